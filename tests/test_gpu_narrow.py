"""The head for up to 16 draft rows: both layouts at the edges of tiles, units, rings and groups of the few-row kernel
(hidden dimension dealt out to the wavefronts, h in registers), and on both sides of the line to the slab kernel.
Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route, to_dev_bf16, to_dev_i32
from test_gpu_parity import ev, problem  # noqa: F401  (fixture and helper)

pytestmark = pytest.mark.gpu


CASES = [
    (1, 8, 1, 1),             # one row, one 16-byte piece
    (16, 64, 16, 16),         # exactly one tile, k == rows
    (17, 72, 3, 10),          # a tile and a row; a unit and a piece
    (4096, 256, 8, 8),        # one tile per workgroup
    (4112, 264, 9, 10),       # one workgroup with a tile more than the others
    (20485, 776, 7, 33),      # six tiles: ring turns of four and of two, a ragged last tile
    (36880, 1288, 2, 10),     # ten tiles: more than one group of partial sums
    (9000, 4096, 16, 64),     # the largest hidden size, all rows, k == 64
    (9000, 4088, 1, 10),
    (9000, 3000, 15, 20),
    (5000, 4104, 4, 10),      # past it: the other kernel
    (170000, 64, 2, 10),      # more tiles than one round of workgroups takes
    (4000, 4096, 16, 64),     # all rows, one tile to a workgroup: the largest hidden size, k == 64
    (4091, 3000, 15, 20),
    (49169, 264, 16, 64),     # all rows, 12 and 13 tiles to a workgroup: more than a round of slabs
    (50003, 776, 13, 33),
    (3000, 2048, 5, 10),      # four, five and seven units to a wavefront
    (5999, 2504, 8, 7),
    (8001, 3504, 2, 10),
    (30000, 256, 8, 10),      # the other kernel: few hidden elements, many tiles
]


def test_cases_reach_both_kernels(ev):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    few = [c for c in CASES if plan_route(c[2], c[0], c[1], c[3], cus)["kernel"] == "narrow"]
    # every number of units per wavefront and ring depth, up to 8 rows and more, one tile to a workgroup and many
    assert {-(-c[1] // 512) for c in few} >= set(range(1, 9))
    assert any(c[2] > 8 and c[0] > 16 * cus for c in few) and any(c[2] > 8 and c[0] <= 16 * cus for c in few)
    assert {c[2] for c in CASES if c not in few} >= {4, 8, 9, 16}


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k", CASES)
def test_few_rows(ev, oracle_mod, layout, V_act, d, M, k):
    import torch
    W, h, ids = problem(500 + V_act + d, V_act, d, M, V=V_act + 5)
    W_act = new_matrix(ev, V_act, d, layout)
    act_ids = torch.empty(V_act, dtype=torch.int32, device="cuda")
    # row i of W is the row of id ids[i]
    full = np.zeros((V_act + 5, d), dtype=np.uint16)
    full[ids] = W
    ev.active_gather(to_dev_bf16(full), to_dev_i32(ids), None, W_act, act_ids)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), W_act, act_ids, k))
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"{layout} V_act={V_act} d={d} M={M} k={k}")


def test_few_rows_equal_logits_order_by_id(ev):
    """All logits equal: every row reaches every bound, and the k smallest ids win."""
    import torch
    V_act, d, k = 5000, 512, 12
    h = torch.zeros((5, d), dtype=torch.bfloat16, device="cuda")
    W = torch.randn((V_act, d), device="cuda").bfloat16()
    ids = np.random.default_rng(3).permutation(3 * V_act)[:V_act].astype(np.int32)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(h, W, to_dev_i32(ids), k))
    assert np.array_equal(i, np.tile(np.sort(ids)[:k], (5, 1))) and not v.any()
    assert np.allclose(l, np.log(V_act), rtol=1e-6)
