"""The head for a few hundred draft rows (128 x 128 tiles): both layouts at the edges of tiles, both ring depths
and the epilogue's paths.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, new_matrix, plan_route, to_dev_bf16, to_dev_i32
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
    # more tiles than compute units: a ring of two stages, two workgroups to a unit
    (20003, 320, 300, 10),    # five pairs, both sides ragged
    (17000, 192, 200, 20),    # three pairs, lists of 32
    (11500, 448, 257, 16),    # seven pairs, a row tile of one row
    (33000, 256, 140, 10),    # four pairs
    (33009, 64, 129, 10),     # a single pair
    (18011, 128, 150, 10),    # two
    (16500, 384, 129, 20),    # six: two after the ring's only turn
    (16500, 2048, 150, 10),   # a few compute units with two tiles
])
def test_few_hundred_rows(ev, oracle_mod, layout, V_act, d, M, k):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert plan_route(M, V_act, d, k, cus) == {"kernel": "tile", "stages": 2 if V_act > 10000 else 4}
    W, h, ids = problem(700 + V_act + d, V_act, d, M, V=V_act + 5)
    full = np.zeros((V_act + 5, d), dtype=np.uint16)
    full[ids] = W
    W_act = new_matrix(ev, V_act, d, layout)
    act_ids = torch.empty(V_act, dtype=torch.int32, device="cuda")
    ev.active_gather(to_dev_bf16(full), to_dev_i32(ids), None, W_act, act_ids)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(h), W_act, act_ids, k))
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"{layout} V_act={V_act} d={d} M={M} k={k}")


@pytest.mark.parametrize("M,V_act,d,k", [
    (200, 700, 128, 33),      # 128 x 128 tiles, lists of 64 slots
    (200, 700, 128, 17),      # lists of 32
    (200, 700, 128, 10),      # lists of 16: the staged ones
    (1999, 6230, 64, 33),     # 256 x 256 tiles
])
def test_a_row_of_nans_leaves_the_others_alone(ev, oracle_mod, M, V_act, d, k):
    """A draft row of NaNs with the sign set has no candidate at all: its lists come out empty, at their own
    places.  The workspace starts full of candidates that would beat everything, so a list that nobody writes
    shows, and so does one that another row's overwrites."""
    import torch
    W, h, ids = problem(800 + M + k, V_act, d, M, V=V_act + 9)
    bad = [5, 130]
    hb = h.copy()
    hb[bad] = 0xFFC0
    ws = torch.empty(ev.workspace_bytes(M, V_act, d, k) // 8, dtype=torch.int64, device="cuda")
    ws.fill_((0x7149F2CA << 32) | 7654321)                 # (1e30, id 7654321)
    v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(to_dev_bf16(hb), to_dev_bf16(W), to_dev_i32(ids), k,
                                                              workspace=ws.view(torch.uint8)))
    good = np.setdiff1d(np.arange(M), bad)
    check_head(v[good], i[good], l[good], oracle_mod.logits(h[good], W), ids, k, f"M={M} V_act={V_act} k={k}")
    assert not np.isfinite(l[bad]).any()                   # (NaN, or -inf: a maximum takes no notice of a NaN)
    # the sign of a NaN that goes through the matrix cores is not ours to say: no candidates, or NaNs of active rows
    empty = i[bad] == -1
    assert np.all(np.isneginf(v[bad][empty])) and np.all(np.isnan(v[bad][~empty])) and np.isin(i[bad][~empty], ids).all()
