"""Few extensions of the batched head: the draft rows of a chunk go to two workgroups.  Chunks of 1, 32, 33 and 64 rows beside each
other, an empty sequence, more than a chunk to a sequence, beside a core of large tiles and of small ones; the same where the extensions ride in
the core's launch instead.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route_batched, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k,core,tiles", [
    (500, 130, 264, [32, 33, 0, 1], 10, "slab", None),      # one launch with the core
    (500, 130, 264, [33, 31, 0, 2], 10, "slab", None),      # a slab of two rows
    (500, 128, 256, [33, 31], 17, "slab", None),
    (700, 700, 2048, [64, 1, 70, 33], 10, "tile", None),
    (700, 90, 512, [150], 64, "tile", None),                # three chunks of one sequence
    (700, 2000, 256, [40, 64, 33], 24, "tile", None),       # pairs of logits as groups
    (700, 1250, 256, [40] * 8, 10, "tile", None),
    (32700, 130, 64, [33, 64, 70, 1, 0, 60, 32, 40, 90], 10, "gemm", 4),      # a slab of two rows; chunks of 33, 64, 1, 32 and 26 rows
    (32700, 700, 64, [64, 65, 33, 150, 80], 24, "gemm", 4), # pairs of logits as groups; three chunks of one sequence
    (32700, 1250, 192, [50] * 8, 10, "gemm", 5),            # taller slabs than without
])
def test_split_rows(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, core, tiles):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == core and r["split"] == (tiles is not None) and r["joint"] == (tiles is None) and tiles in (None, r["arc_tiles"])
    check_batch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k)


@pytest.mark.parametrize("V_core,V_arc,d,lens,k,bound", [
    (10300, 2048, 264, [50, 33, 64], 10, 0),                # d no multiple of 64: slabs, in one launch
    (10300, 2048, 256, [50, 33, 64], 10, 1),                # small tiles, one to a compute unit, that take over a bound
    (10300, 2048, 320, [50, 33, 64], 20, 0),                # none
    (30000, 2048, 64, [50] * 3, 10, 1),                     # in twos, and too few places beside them
])
def test_beside_small_tiles(ev, oracle_mod, V_core, V_arc, d, lens, k, bound):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, "row_major")
    assert r["bound"] == bound and r["split"] == (d % 64 == 0) and r["kernel"] == ("slab" if d == 264 else "tile")
    check_batch(ev, oracle_mod, "row_major", V_core, V_arc, d, lens, k)


def check_batch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k):
    import torch
    S, M, V = len(lens), sum(lens), V_core + len(lens) * V_arc
    ids = np.random.default_rng(V + M).permutation(V).astype(np.int32)
    W, h = gi.gen_normal_bf16(V, d, 51, 0.05), gi.gen_h(M, d, 52)
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
        if a < b:
            sel = np.concatenate([row[:V_core], row[lo:lo + V_arc]])
            check_head(v[a:b], i[a:b], l[a:b], oracle_mod.logits(h[a:b], W[sel]), ids[sel], k, f"{layout} {V_core} {V_arc} {lens} k={k} sequence {s}")
