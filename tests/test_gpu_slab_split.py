"""The slab kernel where several wavefronts share a tile: every slab shape with two and four blocks of draft rows,
short and partial hidden dimensions, both layouts, and every granularity of the bound.  Needs an MI355X: run with
`-m gpu`."""
import numpy as np
import pytest

from helpers import check_head, new_matrix, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev, problem  # noqa: F401  (fixture and helper)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k", [
    (16384, 256, 33, 10),     # 4 tiles per workgroup, a single chunk
    (16390, 512, 17, 33),     # 5, two chunks, a slab of a few rows, pairs of logits as groups
    (24576, 768, 64, 20),     # 6, three chunks
    (28672, 264, 32, 10),     # 7, a chunk and a piece
    (28673, 520, 60, 64),     # 8, two chunks and a piece, k past the groups
    (36864, 1024, 60, 6),     # 9: one wavefront per tile
    (100, 4096, 40, 10),      # two workgroups only
    (5, 72, 20, 5),           # less than a tile
])
def test_split_tiles(ev, oracle_mod, layout, V_act, d, M, k):
    import torch
    W, h, ids = problem(600 + V_act + d, V_act, d, M, V=V_act + 3)
    full = np.zeros((V_act + 3, d), dtype=np.uint16)
    full[ids] = W
    W_act = new_matrix(ev, V_act, d, layout)
    act_ids = torch.empty(V_act, dtype=torch.int32, device="cuda")
    ev.active_gather(to_dev_bf16(full), to_dev_i32(ids), None, W_act, act_ids)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), W_act, act_ids, k))
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"{layout} V_act={V_act} d={d} M={M} k={k}")
