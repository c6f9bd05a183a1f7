"""Heads of 65 to 128 draft rows on both sides of the line between the 128 x 128 tiles and passes of 64 rows, with the scratch that the
library asks for and not a byte more.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route, plan_route_batched, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev, problem  # noqa: F401  (fixture and helper)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k,route", [
    (8192, 256, 80, 10, "slab"),       # a short hidden dimension: passes
    (8192, 256, 83, 10, "slab"),
    (8192, 1024, 82, 10, "tile"),      # lists just fit the scratch
    (8192, 1024, 83, 10, "slab"),      # do not
    (5000, 1024, 65, 9, "tile"),       # a last slab of 8 rows
    (4896, 512, 70, 10, "slab"),
    (4896, 1024, 70, 10, "slab"),      # of 32: too few for a bound, passes
    (2176, 2176, 80, 10, "slab"),      # a large hidden dimension for so few rows
    (2176, 2048, 80, 10, "tile"),
    (40064, 64, 96, 12, "slab"),
    (33024, 1088, 66, 12, "tile"),     # more tiles than compute units; nine parts
    (1000, 1984, 70, 10, "slab"),
    (2000, 1984, 70, 10, "tile"),      # ten parts, the last of one pair
    (1000, 192, 100, 13, "slab"),      # lists of 16 overflow: passes
    (2176, 128, 80, 20, "slab"),       # lists of 32: passes
    (129, 64, 90, 64, "slab"),         # of 64; a last slab of one row
    (129, 1024, 70, 12, "tile"),       # two slabs, one of one row
    (6400, 128, 128, 64, "slab"),
    (3000, 264, 72, 10, "slab"),       # no multiple of 64
])
def test_head_of_65_to_128_rows(ev, oracle_mod, layout, V_act, d, M, k, route):
    import torch
    r = plan_route(M, V_act, d, k, torch.cuda.get_device_properties(0).multi_processor_count)
    assert r["kernel"] == route and r.get("parts", 0) == (route == "tile") and r.get("stages", 4) == (2 if V_act == 33024 else 4)
    W, h, ids = problem(800 + V_act + d, V_act, d, M, V=V_act + 5)
    full = np.zeros((V_act + 5, d), dtype=np.uint16)
    full[ids] = W
    W_act, act_ids = new_matrix(ev, V_act, d, layout), torch.empty(V_act, dtype=torch.int32, device="cuda")
    ev.active_gather(to_dev_bf16(full), to_dev_i32(ids), None, W_act, act_ids)
    n = ev.workspace_bytes(M, V_act, d, k)
    ws = torch.full((n + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), W_act, act_ids, k, workspace=ws[:n]))
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"{layout} V_act={V_act} d={d} M={M} k={k}")
    assert bool((ws[n:] == 0x5a).all())


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k,route,bound", [
    (1000, 700, 256, [64, 1], 10, "tile", 0),                # one launch with the extensions
    (20096, 2048, 64, [30, 30, 30, 20], 10, "tile", 1),      # (row-major: a bound from the extensions' lists)
    (5000, 90, 1024, [60, 40, 28], 10, "tile", 0),           # none: too few lists
    (1000, 20, 192, [50, 78], 8, "tile", 0),                 # the lists just fit the core's scratch
    (1000, 20, 192, [50, 60], 8, "tile", 0),
    (1000, 20, 192, [50, 78], 7, "slab", 0),                 # do not: passes
    (800, 300, 64, [100], 64, "slab", 0),
])
def test_core_of_65_to_128_rows(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, route, bound):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == route and r["bound"] == (bound if layout == "row_major" else 0) and "parts" not in r
    S, M, V = len(lens), sum(lens), V_core + len(lens) * V_arc
    ids = np.random.default_rng(V + M).permutation(V).astype(np.int32)
    W, h = gi.gen_normal_bf16(V, d, 61, 0.05), gi.gen_h(M, d, 62)
    dW, dids, row = to_dev_bf16(W), to_dev_i32(ids), np.arange(V, dtype=np.int32)
    W_core, W_arc = new_matrix(ev, V_core, d, layout), new_matrix(ev, V_arc, d, layout, batch=S)
    scratch = torch.empty(max(V_core, V_arc), dtype=torch.int32, device="cuda")
    ev.active_gather(dW, to_dev_i32(row[:V_core]), None, W_core, scratch[:V_core])
    for s in range(S):
        lo = V_core + s * V_arc
        ev.active_gather(dW, to_dev_i32(row[lo:lo + V_arc]), None, W_arc.sub(s) if layout == "packed" else W_arc[s], scratch[:V_arc])
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = ev.workspace_bytes_segmented(M, V_core, V_arc, S, d, k)
    ws = torch.full((n + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    arc = (W_arc, dids[V_core:].reshape(S, V_arc).contiguous())
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk_segmented(to_dev_bf16(h), W_core, dids[:V_core].clone(), *arc, row_off, k,
                                                                        workspace=ws[:n]))
    for s in range(S):
        a, b, lo = row_off[s], row_off[s + 1], V_core + s * V_arc
        sel = np.concatenate([row[:V_core], row[lo:lo + V_arc]])
        check_head(v[a:b], i[a:b], l[a:b], oracle_mod.logits(h[a:b], W[sel]), ids[sel], k, f"{layout} {V_core} {V_arc} {lens} k={k} sequence {s}")
    assert bool((ws[n:] == 0x5a).all())
