"""The batched head where the core's slabs or small tiles and the extensions' slabs share one launch.  Ragged last slabs of both,
passes of a core beside each other, sequences without rows, more chunks than a launch takes; lists of every length, and bounds found by halves at
every scale of logits.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route_batched, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def check_batch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k):
    import torch
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
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk_segmented(
        to_dev_bf16(h), W_core, dids[:V_core].clone(), W_arc, dids[V_core:].reshape(S, V_arc).contiguous(), row_off, k))
    for s in range(S):
        a, b, lo = row_off[s], row_off[s + 1], V_core + s * V_arc
        if a < b:
            sel = np.concatenate([row[:V_core], row[lo:lo + V_arc]])
            check_head(v[a:b], i[a:b], l[a:b], oracle_mod.logits(h[a:b], W[sel]), ids[sel], k, f"{layout} {V_core} {V_arc} k={k} sequence {s}")


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k,blocks", [
    (1, 1, 8, [1], 1, 1),                            # one slab of one row in each
    (63, 65, 256, [5, 0, 11], 10, 1),                # two slabs to an extension, one to the core
    (1000, 130, 264, [20, 12], 64, 2),               # pairs of logits as groups; hidden sizes that are no whole chunks
    (700, 300, 2048, [33, 31], 10, 4),               # a full pass
    (700, 300, 512, [40, 30, 33], 13, 4),            # two passes, a chunk across their border
    (333, 70, 264, [1] * 70, 13, 4),                 # two batches of chunks: the core goes with the first
    (20000, 90, 256, [3, 2], 10, 1),                 # many more slabs in the core
])
def test_joint_launch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k, blocks):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens[:64], torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == "slab" and r["joint"] == 1 and r["arc_blocks"] == blocks
    check_batch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k)


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k", [
    (128, 64, 64, [64, 1, 0, 70], 10),               # a tile, a pair of chunks, extensions of one slab
    (300, 65, 320, [140, 30], 10),                   # five pairs; a last tile of 44 rows: fewer groups than k
    (148, 70, 1024, [100, 60], 13),                  # of 20
    (700, 200, 256, [40, 30, 80], 16),               # lists as long as k
    (1100, 130, 2048, [33] * 5, 17),                 # lists of 32
    (700, 90, 192, [60, 100], 64),                   # of 64
    (33000, 100, 256, [16] * 10, 10),                # more tiles than compute units
    (500, 40, 128, [2] * 70, 20),                    # two batches of chunks: the tiles go with the first
])
def test_joint_tiles(ev, oracle_mod, layout, V_core, V_arc, d, lens, k):
    import torch
    r = plan_route_batched(V_core, V_arc, d, k, lens if len(lens) <= 64 else [sum(lens) // 7] * 7, torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == "tile" and r["joint"] == 1
    check_batch(ev, oracle_mod, layout, V_core, V_arc, d, lens, k)


@pytest.mark.parametrize("V_act,k", [(148, 10), (177, 16), (4000, 13), (4000, 16), (4000, 33), (20011, 30)])
def test_bounds_at_every_scale(ev, oracle_mod, V_act, k):
    """Rows of h from 1e-30 to 1e30 and rows of zeros (whose logits are all equal): values against the products, in the scale of each row."""
    d, M = 256, 140
    W, h = gi.gen_normal_bf16(V_act, d, 63, 0.05), gi.gen_h(M, d, 64)
    scale = np.array([1e-30, 1.0, 1e30, 0.0])[np.arange(M) % 4]
    f32 = lambda b: (b.astype(np.uint32) << 16).view(np.float32)  # noqa: E731
    hb = gi.f32_to_bf16_bits((f32(h) * scale[:, None]).astype(np.float32))
    ids = np.random.default_rng(V_act).permutation(V_act).astype(np.int32)
    v, i, _ = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(hb), to_dev_bf16(W), to_dev_i32(ids), k))
    z = oracle_mod.logits(hb, W)
    for m in range(M):
        if scale[m] == 0.0:
            assert np.array_equal(i[m], np.arange(k)) and not v[m].any()
            continue
        best = np.sort(z[m])[::-1][:k]
        err = 1e-5 * np.abs(z[m]).max()                            # (256 products of bf16 summed in 32 bits)
        assert np.all(np.abs(v[m] - best) <= err), f"row {m}"
        slot = np.argsort(ids)[i[m]]
        assert len(set(i[m].tolist())) == k and np.all(np.abs(z[m][slot] - v[m]) <= err), f"row {m}"


@pytest.mark.parametrize("V_act,M,k,zeros", [(5000, 160, 10, 1), (5000, 160, 10, 3), (5000, 160, 10, 4), (4000, 140, 5, 2), (3000, 140, 33, 3)])
def test_few_rows_past_their_lists(ev, oracle_mod, V_act, M, k, zeros):
    """Rows whose logits are all equal, some of the 32 that a wavefront has: up to three go one after the other, more by halves first."""
    d = 128
    W, h = gi.gen_normal_bf16(V_act, d, 65, 0.05), gi.gen_h(M, d, 66)
    empty = np.arange(M) % 32 >= 32 - zeros
    h[empty] = 0
    ids = np.random.default_rng(V_act + zeros).permutation(V_act).astype(np.int32)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), to_dev_bf16(W), to_dev_i32(ids), k))
    assert np.all(i[empty] == np.arange(k)) and not v[empty].any()
    check_head(v[~empty], i[~empty], l[~empty], oracle_mod.logits(h[~empty], W), ids, k, f"V_act={V_act} k={k} zeros={zeros}")
