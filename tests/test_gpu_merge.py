"""The merge of slab partials at the sizes where it changes shape: one round and several, one thread
per list and several, short lists, long ones, and more candidates at the bound than its list holds.
Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head
from test_gpu_parity import ev, problem, run_head  # noqa: F401  (fixture and helpers)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V_act,M,k", [
    (10, 3, 10),              # one list that holds exactly k
    (65, 5, 64),              # two lists, k close to everything
    (1000, 2, 1),
    (1000, 20, 5),            # sixteen lists of 5, dealt out to the wavefronts
    (4090, 17, 1),            # 64 lists of 1
    (5900, 33, 64),           # 93 lists of 64: fewer than 2 q for every wavefront
    (8448, 60, 64),           # 132: not dealt out
    (900, 140, 10),           # unsorted lists, dealt out a line at a time
    (1024, 7, 33),            # sixteen lists, several threads to a list
    (4100, 2, 63),
    (16400, 3, 11),           # a little more than 256 lists, odd k (lists 8-byte aligned)
    (90001, 1, 64),           # 512 to 1024 lists
    (200003, 2, 10),          # more than one round of 1024 lists
    (140009, 129, 10),        # unsorted lists, more than one round
    (3000, 130, 64),          # unsorted lists of 64 slots
])
def test_merge_shapes(ev, oracle_mod, V_act, M, k):
    W, h, ids = problem(900 + V_act + k, V_act, 64, M, V=V_act + 11)
    v, i, l = run_head(ev, h, W, ids, k)
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"V_act={V_act} M={M} k={k}")


@pytest.mark.parametrize("k", [33, 64])
def test_merge_more_candidates_than_its_list_holds(ev, oracle_mod, k):
    """Every 64th run of 64 rows is far below the rest, which makes the bound useless: nearly all of the
    lists' entries reach it.  The logits are exact (small integers), so the ids are too."""
    V_act, d = 16384, 64
    r = np.arange(V_act)
    W = np.zeros((V_act, d), dtype=np.float32)
    W[:, 0] = np.random.default_rng(5).permutation(V_act) // 64     # 256 values, 64 rows each: ties by id
    W[:, 1] = np.where((r // 64) % 64 == 63, -128.0, 0.0)           # below everything else
    h = np.zeros((2, d), dtype=np.float32)
    h[:, 0], h[:, 1] = 1.0, 2.0
    h[1, 0] = -1.0
    Wb, hb = gi.f32_to_bf16_bits(W), gi.f32_to_bf16_bits(h)
    ids = np.random.default_rng(6).permutation(V_act).astype(np.int32)
    v, i, l = run_head(ev, hb, Wb, ids, k)
    z = oracle_mod.logits(hb, Wb)
    for m in range(2):
        order = np.lexsort((ids, -z[m]))[:k]
        assert np.array_equal(i[m], ids[order]) and np.array_equal(v[m], z[m][order].astype(np.float32))
