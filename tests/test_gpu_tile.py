"""The head for a few hundred draft rows (128 x 128 tiles): both layouts at the edges of tiles, the ring
and the epilogue's paths.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev, problem  # noqa: F401  (fixture and helper)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k", [
    (128, 64, 129, 10),       # one slab, a single pair of chunks, a second tile of one row
    (127, 128, 200, 5),       # a ragged slab, fewer pairs than ring stages
    (129, 256, 256, 10),      # a slab of one row, exactly four pairs
    (1000, 320, 257, 16),     # five pairs, three row tiles, lists full
    (700, 576, 131, 33),      # k past the staged lists
    (300, 4096, 140, 64),     # the benchmark's hidden size, largest k
])
def test_few_hundred_rows(ev, oracle_mod, layout, V_act, d, M, k):
    import torch
    W, h, ids = problem(700 + V_act + d, V_act, d, M, V=V_act + 5)
    full = np.zeros((V_act + 5, d), dtype=np.uint16)
    full[ids] = W
    W_act = new_matrix(ev, V_act, d, layout)
    act_ids = torch.empty(V_act, dtype=torch.int32, device="cuda")
    ev.active_gather(to_dev_bf16(full), to_dev_i32(ids), None, W_act, act_ids)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), W_act, act_ids, k))
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"{layout} V_act={V_act} d={d} M={M} k={k}")
