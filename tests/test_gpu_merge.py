"""The merge of slab partials at the sizes where it changes shape: one round and several, one thread
per list and several, few lists and many, short ones and long ones, and more candidates at the bound than its list holds.
Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from helpers import check_head, plan_route
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
    (16400, 3, 11),           # 256 lists, odd k (lists 8-byte aligned)
    (90001, 1, 64),           # 256 lists of 64
    (90001, 17, 64),          # 469 lists: 512 threads
    (150000, 20, 10),         # 938 lists: 1024 threads
    (200003, 2, 10),          # lists of workgroups with several tiles
    (200003, 17, 10),         # 1251 lists: more than one round of 1024
    (400005, 33, 64),         # several rounds, long lists
    (140009, 129, 10),        # unsorted lists, more than one round
    (3000, 130, 64),          # unsorted lists of 64 slots
])
def test_merge_shapes(ev, oracle_mod, V_act, M, k):
    W, h, ids = problem(900 + V_act + k, V_act, 64, M, V=V_act + 11)
    v, i, l = run_head(ev, h, W, ids, k)
    check_head(v, i, l, oracle_mod.logits(h, W), ids, k, f"V_act={V_act} M={M} k={k}")


def candidates(z, ids, k, rows, threads):
    """How many keys of the sorted lists of one draft row reach the merge's bound, and how many its list holds: the
    selection of the first round, written out for lists that are dealt out to the wavefronts in turn."""
    key = lambda r: (-z[r], ids[r])                          # noqa: E731
    lists = [sorted(range(a, min(a + rows, len(z))), key=key)[:k] for a in range(0, len(z), rows)]
    waves, sets = threads // 64, threads // 128
    q = -(-k // sets)
    assert threads // 2 < len(lists) < threads and len(lists) >= 2 * q * waves
    taus = [sorted((key(L[0]) for L in lists[w::waves]))[q - 1] for w in range(waves)]
    tau = sorted(taus)[sets - 1]
    return sum(key(r) <= tau for L in lists for r in L), 4096 + k


@pytest.mark.parametrize("k", [33, 64])
def test_merge_falls_back_to_the_exact_selection(ev, k):
    """All that is large sits in the lists of seven of the sixteen wavefronts, and the bound needs eight: thousands of
    keys reach it, more than the list in LDS holds.  The logits are exact (small integers), so the ids are too."""
    import torch
    V_act, d, M = 150000, 64, 18
    r = plan_route(M, V_act, d, k, torch.cuda.get_device_properties(0).multi_processor_count)
    assert r["kernel"] == "slab" and 512 < r["lists"] < 1024
    rng = np.random.default_rng(7)
    lists = np.arange(V_act) // r["rows"]
    W = np.zeros((V_act, d), dtype=np.float32)
    W[:, 0] = rng.integers(0, 250, V_act)
    W[:, 1] = np.where(lists % 16 < 7, 128.0, -128.0)        # 2 x 128 above and below
    h = np.zeros((M, d), dtype=np.float32)
    h[:, 0], h[:, 1] = 1.0, 2.0
    h[1::2, 0] = -1.0
    ids = rng.permutation(V_act).astype(np.int32)
    v, i, l = run_head(ev, gi.f32_to_bf16_bits(h), gi.f32_to_bf16_bits(W), ids, k)
    for m in (0, 1, M - 1):
        z = h[m] @ W.T
        n, room = candidates(z, ids, k, r["rows"], 1024)
        assert n > room, (n, room)
        order = np.lexsort((ids, -z))[:k]
        assert np.array_equal(i[m], ids[order]) and np.array_equal(v[m], z[order])


@pytest.mark.parametrize("k", [33, 64])
def test_merge_with_a_low_run_in_every_64(ev, oracle_mod, k):
    """Every 64th run of 64 rows is far below the rest.  The logits are exact (small integers), so the ids are too."""
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
