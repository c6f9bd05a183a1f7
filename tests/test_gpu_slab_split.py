"""The slab kernel: every slab height with two and four blocks of draft rows, with tiles shared by several wavefronts and
without, short and partial hidden dimensions, both layouts, and every granularity of the bound.  Needs an MI355X: run
with `-m gpu`."""
import numpy as np
import pytest

from helpers import check_head, new_matrix, plan_route, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev, problem  # noqa: F401  (fixture and helper)

pytestmark = pytest.mark.gpu


CASES = [
    (16384, 256, 33, 10),     # 4 tiles per workgroup, a single chunk
    (16390, 512, 17, 33),     # 5, two chunks, a slab of a few rows, pairs of logits as groups
    (24576, 768, 64, 20),     # 6, three chunks
    (28672, 264, 32, 10),     # 7, a chunk and a piece
    (28673, 520, 60, 64),     # 8, two chunks and a piece, k past the groups
    (36864, 1024, 60, 6),     # 9: one wavefront per tile
    (100, 4096, 40, 10),      # two workgroups only
    (5, 72, 20, 5),           # less than a tile
    (16384, 512, 20, 10),     # 4 with two blocks
    (16390, 520, 60, 20),     # 5 with four; k == lanes of a draft row
    (24570, 256, 20, 24),     # 6 with two; pairs of logits from here on
    (28672, 264, 60, 10),     # 7 with four
    (28673, 512, 30, 20),     # 8 with two
    (36864, 256, 32, 33),     # 9 with two
    (37000, 264, 20, 10),     # 10
    (36999, 512, 40, 40),     # 10, k == lanes
    (41001, 72, 25, 33),      # 12
    (48000, 256, 64, 48),     # 12, k == lanes
    (60000, 256, 24, 10),     # two rounds with two blocks: no tile is shared
    (51446, 512, 40, 10),     # two rounds with four blocks
]


def test_cases_reach_every_shape(ev):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    got = set()
    for V_act, d, M, k in CASES:
        r = plan_route(M, V_act, d, k, cus)
        assert r["kernel"] == "slab"
        got.add((r["tiles"], r["blocks"], r["shared"]))
    want = {(t, b, s) for b in (2, 4) for t, s in ((4, b), (5, 2), (6, 2), (7, 2), (8, 2), (9, 1), (10, 1), (12, 1))}
    assert want <= got, want - got
    assert any(b == 2 and s == 1 and t <= 8 for t, b, s in got)


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k", CASES)
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
