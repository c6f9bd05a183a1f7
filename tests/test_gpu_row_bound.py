"""The batched head where the core's matrix tiles take over a bound of every draft row from the extensions' lists: extensions that
hold all of the best, none of them (every slab's survivors exceed a list) or some, equal logits on both sides of the bound, chunks
that begin anywhere in a tile.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route_batched, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k,arc_scale", [
    (1000, 1000, 256, [60, 1, 70, 3], 10, 1.0),      # 128 x 128 tiles in one launch with the extensions: a slab's own bound, a chunk of a single row
    (1000, 1000, 256, [64, 65, 1], 16, 1.0),         # by halves
    (1100, 500, 128, [40, 40, 60], 10, 1.0),
    (1000, 300, 64, [130], 10, 1.0),
    (1000, 1000, 256, [33, 64, 64], 10, 0.01),       # nothing of the extension is among the best
    (1000, 1000, 256, [33, 64, 64], 10, 40.0),       # nothing of the core is
    (1000, 1000, 256, [33, 64, 64], 1, 1.0),
    (1000, 1000, 256, [33, 64, 64], 10, 0.0),        # every logit of the extensions is 0
    (21700, 1500, 64, [60] * 12, 10, 1.0),           # 256 x 256 tiles: the first best of 16 lists
    (21700, 1500, 64, [64] * 12, 7, 0.05),
    (32700, 2048, 64, [60] * 8, 16, 1.0),            # lists as long as k: the second best
    (32700, 2048, 64, [60] * 8, 16, 0.05),
    (32700, 500, 128, [60] * 8, 10, 1.0),            # of 8 lists
    (1000, 700, 64, [3] * 64, 2, 1.0),               # as many chunks as one launch takes
])
def test_bound_from_extensions(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, arc_scale):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == ("gemm" if V_core > 20000 else "tile")
    if V_core > 20000:
        assert r["bound"] == (2 if k == 16 or V_arc == 500 else 1)
    else:
        assert r["joint"] == (V_arc != 700 or layout == "packed") and r["bound"] == 1 - r["joint"]
    check_bound(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, arc_scale)


def test_bound_from_extensions_of_packed_small_tiles(ev, oracle_mod):
    """Two tiles on every compute unit and little in the second row of them: W through LDS, and a bound."""
    import torch
    V_core, V_arc, d, lens, k = 32700, 1000, 3072, [50, 31, 50], 10
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, "packed")
    assert r["kernel"] == "tile" and r["joint"] == 0 and r["bound"] == 1 and r["split"] == 1
    check_bound(ev, oracle_mod, "packed", V_core, V_arc, d, lens, k, 1.0)


@pytest.mark.parametrize("V_core,V_arc,d,lens,k,arc_scale,bound", [
    (10300, 2048, 128, [60, 1, 70, 3], 10, 1.0, 1),          # 128 x 128 tiles, the first best of 16 lists, a chunk of a single row
    (10300, 2048, 64, [64, 65, 1], 16, 1.0, 2),              # the second best of 16
    (8300, 300, 64, [5] * 26, 8, 1.0, 0),                    # too few lists: a slab's own bound
    (8300, 500, 64, [9] * 16, 10, 1.0, 2),                   # of 8 lists
    (10300, 2048, 64, [33, 64, 64], 10, 0.01, 1),            # nothing of the extension is among the best: more survivors than a list holds
    (10300, 2048, 64, [33, 64, 64], 10, 40.0, 1),            # nothing of the core is
    (10300, 2048, 64, [33, 64, 64], 1, 1.0, 1),
    (10300, 2048, 64, [33, 64, 64], 10, 0.0, 1),             # every logit of the extensions is 0
    (10307, 2048, 64, [33, 64, 64], 13, 0.05, 2),            # a ragged last slab
    (30000, 2048, 64, [50] * 3, 10, 1.0, 1),                 # more tiles than compute units: rings of two stages
    (16300, 1000, 128, [60] * 8, 16, 0.3, 2),
])
def test_bound_from_extensions_of_small_tiles(ev, oracle_mod, V_core, V_arc, d, lens, k, arc_scale, bound):
    """Row-major small tiles that the extensions do not ride with."""
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, "row_major")
    assert r["kernel"] == "tile" and r["joint"] == 0 and r["bound"] == bound
    check_bound(ev, oracle_mod, "row_major", V_core, V_arc, d, lens, k, arc_scale)


def check_bound(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, arc_scale):
    import torch
    S, M = len(lens), sum(lens)
    rng = np.random.default_rng(V_core + V_arc + M + k)
    V = V_core + S * V_arc
    W = gi.gen_normal_bf16(V, d, 41, 0.05)
    Wf = gi.bf16_bits_to_f32(W)
    Wf[V_core:] *= np.float32(arc_scale)
    W = gi.f32_to_bf16_bits(Wf)
    W[V_core - 40:V_core] = W[V_core:V_core + 40]                # rows of the core that equal rows of the first extension
    h = gi.gen_h(M, d, 42)
    ids = rng.permutation(V).astype(np.int32)
    dW, dids, row = to_dev_bf16(W), to_dev_i32(ids), np.arange(V, dtype=np.int32)
    W_core, W_arc = new_matrix(ev, V_core, d, layout), new_matrix(ev, V_arc, d, layout, batch=S)
    scratch = torch.empty(max(V_core, V_arc), dtype=torch.int32, device="cuda")
    ev.active_gather(dW, to_dev_i32(row[:V_core]), None, W_core, scratch[:V_core])
    for s in range(S):
        lo = V_core + s * V_arc
        ev.active_gather(dW, to_dev_i32(row[lo:lo + V_arc]), None, W_arc.sub(s) if layout == "packed" else W_arc[s], scratch[:V_arc])
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk_segmented(
        to_dev_bf16(h), W_core, dids[:V_core].clone(), W_arc, dids[V_core:].reshape(S, V_arc).contiguous(), row_off, k))
    for s in range(S):
        a, b, lo = row_off[s], row_off[s + 1], V_core + s * V_arc
        sel = np.concatenate([row[:V_core], row[lo:lo + V_arc]])
        check_head(v[a:b], i[a:b], l[a:b], oracle_mod.logits(h[a:b], W[sel]), ids[sel], k, f"{layout} {V_core} {V_arc} {lens} k={k} sequence {s}")


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k", [
    (1000, 1000, 256, [60, 1, 70, 3], 10),       # 128 x 128 tiles
    (1000, 1000, 256, [64, 65, 1], 16),
    (1003, 500, 128, [40, 40, 60], 5),           # a last slab of 107 rows
    (10300, 2048, 64, [60, 1, 70, 3], 10),       # (row-major: these by themselves and bounded, those above beside the extensions)
    (10300, 2048, 64, [64, 65, 1], 16),
    (21700, 1500, 64, [60] * 12, 10),            # 256 x 256 tiles
])
def test_bound_loose_for_some_rows(ev, oracle_mod, layout, V_core, V_arc, d, lens, k):
    """Extensions that live in the first half of the hidden dimension, and draft rows that live in either half: where it is
    the second, the extensions' logits are 0 and half of the core's reach the bound; beside them rows that it serves well."""
    import torch
    S, M, V = len(lens), sum(lens), V_core + len(lens) * V_arc
    W, h = gi.gen_normal_bf16(V, d, 43, 0.05), gi.gen_h(M, d, 44)
    W[V_core:, d // 2:] = 0
    h[::3, :d // 2] = 0                                          # (every third draft row; the others see both halves)
    ids = np.random.default_rng(V + M).permutation(V).astype(np.int32)
    dW, dids, row = to_dev_bf16(W), to_dev_i32(ids), np.arange(V, dtype=np.int32)
    W_core, W_arc = new_matrix(ev, V_core, d, layout), new_matrix(ev, V_arc, d, layout, batch=S)
    scratch = torch.empty(max(V_core, V_arc), dtype=torch.int32, device="cuda")
    ev.active_gather(dW, to_dev_i32(row[:V_core]), None, W_core, scratch[:V_core])
    for s in range(S):
        lo = V_core + s * V_arc
        ev.active_gather(dW, to_dev_i32(row[lo:lo + V_arc]), None, W_arc.sub(s) if layout == "packed" else W_arc[s], scratch[:V_arc])
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk_segmented(
        to_dev_bf16(h), W_core, dids[:V_core].clone(), W_arc, dids[V_core:].reshape(S, V_arc).contiguous(), row_off, k))
    for s in range(S):
        a, b, lo = row_off[s], row_off[s + 1], V_core + s * V_arc
        sel = np.concatenate([row[:V_core], row[lo:lo + V_arc]])
        check_head(v[a:b], i[a:b], l[a:b], oracle_mod.logits(h[a:b], W[sel]), ids[sel], k, f"{layout} {V_core} {V_arc} {lens} k={k} sequence {s}")
