"""A logit is a function of its draft row and its weight row alone, wherever in the active set that row sits:
identical rows have identical logits, so that they are ordered by id, and the result depends on the set of ids and
not on their order.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

from helpers import new_matrix, plan_route_batched, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def scattered_copies(rows, copies, d, seed):
    """W [rows, d] on the GPU in which every row occurs `copies` times or once less, in random places, and which
    distinct row each is."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    base = torch.empty(((rows + copies - 1) // copies, d), dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=g)
    group = np.random.default_rng(seed).permutation(np.arange(rows) // copies)
    return base[torch.from_numpy(group).cuda()].contiguous(), group


def check_equal_rows(vals, out_ids, ids, group, where):
    """Among equal rows the logits are equal bit for bit and the smaller id comes first; no id is passed over."""
    of = dict(zip(ids.tolist(), group.tolist()))
    members = {}
    for t in sorted(of):
        members.setdefault(of[t], []).append(t)
    for m in range(len(vals)):
        seen = {}
        for v, t in zip(vals[m].tolist(), out_ids[m].tolist()):
            seen.setdefault(of[t], []).append((v, t))
        for gr, entries in seen.items():
            assert len({v for v, _ in entries}) == 1, f"{where}: row {m}: equal rows, logits {entries}"
            assert [t for _, t in entries] == members[gr][:len(entries)], f"{where}: row {m}: {entries} of {members[gr]}"


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_act,d,M,k", [
    (3000, 4096, 8, 10),       # few draft rows
    (2200, 512, 20, 10),       # slabs of 4 tiles; two chunks of the hidden dimension
    (16390, 2048, 33, 10),     # 5 tiles, eight chunks
    (28700, 1024, 60, 33),     # 8 tiles
    (36864, 1024, 64, 10),     # 9 tiles
    (9000, 4096, 40, 10),
    (9000, 3000, 40, 10),      # no whole number of chunks
    (5000, 1024, 100, 10),     # two passes over the matrix
    (5000, 1024, 80, 10),      # 128 x 128 tiles, in parts
    (3000, 1024, 200, 10),     # 128 x 128 tiles
])
def test_equal_rows_and_order(ev, layout, V_act, d, M, k):
    import torch
    W, group = scattered_copies(V_act, 4, d, V_act + d)
    rng = np.random.default_rng(d)
    ids = rng.choice(2 * V_act, V_act, replace=False).astype(np.int32)
    h = torch.empty((M, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(M))
    W_lm = torch.zeros((2 * V_act, d), dtype=torch.bfloat16, device="cuda")
    W_lm[torch.from_numpy(ids).cuda().long()] = W

    def head(order):
        W_act = new_matrix(ev, V_act, d, layout)
        act_ids = torch.empty(V_act, dtype=torch.int32, device="cuda")
        ev.active_gather(W_lm, to_dev_i32(order), None, W_act, act_ids)
        return [x.cpu().numpy() for x in ev.active_lmhead_topk(h, W_act, act_ids, k)]

    v0, i0, l0 = head(ids)
    check_equal_rows(v0, i0, ids, group, f"{layout} V_act={V_act} d={d} M={M}")
    v1, i1, l1 = head(ids[rng.permutation(V_act)])
    assert np.array_equal(i0, i1) and np.array_equal(v0, v1)
    np.testing.assert_allclose(l0, l1, rtol=1e-6)


@pytest.mark.parametrize("layout", ["packed", "row_major"])
@pytest.mark.parametrize("V_core,V_arc,d,lens,k,core", [
    (16000, 400, 512, [20, 1, 40], 12, "slab"),          # core in one pass of slabs of 4 tiles
    (36864, 900, 1024, [33, 64, 10], 12, "tile"),        # 107 rows: 128 x 128 tiles in a single chain, extensions of 4 tiles
    (36864, 900, 1024, [33, 64, 10], 13, "slab"),        # core in two passes
    (36864, 900, 2048, [33, 64, 10], 13, "slab"),        # a hidden dimension that a call with one set takes in two segments
    (2000, 2000, 2048, [60, 17, 60, 8], 12, "tile"),     # 128 x 128 tiles and slabs
    (10300, 2048, 256, [50, 33, 64], 12, "tile"),        # (row-major: in two launches, rows of the extensions shared out, a bound from their lists)
    (300, 17000, 256, [64], 12, "slab"),
])
def test_equal_rows_in_core_and_extension(ev, layout, V_core, V_arc, d, lens, k, core):
    """Copies of one row in the shared core and in an extension tie as well."""
    import torch
    S, M = len(lens), sum(lens)
    r = plan_route_batched(V_core, V_arc, d, k, lens, torch.cuda.get_device_properties(0).multi_processor_count, layout)
    assert r["kernel"] == core and "parts" not in r and r.get("segments", 1) == 1
    W, group = scattered_copies(V_core + V_arc, 4, d, V_core + d)
    rng = np.random.default_rng(d)
    ids = rng.permutation(2 * (V_core + V_arc)).astype(np.int32)
    W_lm = torch.zeros((len(ids), d), dtype=torch.bfloat16, device="cuda")
    core, first_arc = ids[:V_core], ids[V_core:V_core + V_arc]
    W_lm[torch.from_numpy(ids[:V_core + V_arc]).cuda().long()] = W
    h = torch.empty((M, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(M))
    W_core, ids_core = new_matrix(ev, V_core, d, layout), torch.empty(V_core, dtype=torch.int32, device="cuda")
    ev.active_gather(W_lm, to_dev_i32(core), None, W_core, ids_core)
    W_arc, ids_arc = new_matrix(ev, V_arc, d, layout, batch=S), torch.empty((S, V_arc), dtype=torch.int32, device="cuda")
    for s in range(S):                                       # every sequence the same extension, in another order
        ev.active_gather(W_lm, to_dev_i32(first_arc[rng.permutation(V_arc)]), None,
                         W_arc.sub(s) if layout == "packed" else W_arc[s], ids_arc[s])
    row_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    v, i, _ = (x.cpu().numpy() for x in ev.active_lmhead_topk_segmented(h, W_core, ids_core, W_arc, ids_arc, row_off, k))
    check_equal_rows(v, i, ids[:V_core + V_arc], group, f"{layout} V_core={V_core} V_arc={V_arc} d={d}")
