"""The batched head where the core goes by slabs: its slabs and those of the extensions share one launch.  Ragged last slabs of both,
passes of a core beside each other, sequences without rows, more chunks than a launch takes.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route_batched, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


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
    chunks = plan_route_batched(V_core, V_arc, d, k, lens[:64], torch.cuda.get_device_properties(0).multi_processor_count)
    assert chunks["kernel"] == "slab" and chunks["joint_blocks"] == blocks
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
