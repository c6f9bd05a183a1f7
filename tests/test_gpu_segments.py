"""Hidden sizes that are a multiple of 2,048: the slab kernel sums two alternating halves of a row apart, half of the
workgroups of a row-major matrix the other one first.  Against the oracle, both layouts to the bit the same, and equal rows of
neighbouring slabs tie.  Needs an MI355X: run with `-m gpu`."""
import numpy as np
import pytest

from helpers import check_head, new_matrix, plan_route, to_dev_bf16, to_dev_i32
from test_gpu_equal_rows import check_equal_rows
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V_act,d,M,k,tiles,blocks,shared", [
    (4200, 2048, 60, 10, 4, 4, 4),       # four wavefronts to a tile: one segment; the last slab is ragged
    (4200, 2048, 20, 10, 4, 2, 2),       # two segments of four chunks
    (4200, 4096, 20, 10, 4, 2, 2),       # of eight chunks, taken four at a time
    (18000, 2048, 40, 40, 5, 4, 2),      # pairs of logits as groups: more LDS
    (18000, 2048, 12, 10, 5, 1, 1),
    (30000, 2048, 24, 10, 8, 2, 2),
    (33001, 2048, 64, 33, 9, 4, 1),      # one wavefront per tile
    (45000, 2048, 33, 10, 12, 4, 1),     # tallest slabs
    (131080, 2048, 17, 10, 12, 2, 1),    # several rounds, two workgroups on a compute unit
    (5000, 6144, 33, 10, 4, 4, 4),       # one segment
    (18000, 6144, 33, 10, 5, 4, 2),      # three turns of eight chunks: an odd number
    (4200, 6144, 20, 10, 4, 2, 2),
    (4200, 10240, 17, 10, 4, 2, 2),      # five
])
def test_two_segments(ev, oracle_mod, V_act, d, M, k, tiles, blocks, shared):
    import torch
    r = plan_route(M, V_act, d, k, torch.cuda.get_device_properties(0).multi_processor_count)
    assert (r["kernel"], r["tiles"], r["blocks"], r["shared"]) == ("slab", tiles, blocks, shared)
    assert r["segments"] == (1 if shared == 4 else 2)
    rng = np.random.default_rng(V_act + d)
    g = torch.Generator(device="cuda").manual_seed(V_act + M)
    base = torch.empty((V_act // 4 + 1, d), dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=g)
    group = rng.permutation(np.arange(V_act) // 4)
    W = base[torch.from_numpy(group).cuda()].contiguous()
    h = torch.empty((M, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    ids = rng.permutation(V_act).astype(np.int32)
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    ref = oracle_mod.logits(bits(h), bits(base))[:, group]
    got = {}
    for layout in ("packed", "row_major"):
        W_act, act_ids = new_matrix(ev, V_act, d, layout), torch.empty(V_act, dtype=torch.int32, device="cuda")
        ev.active_gather(W, to_dev_i32(np.arange(V_act, dtype=np.int32)), None, W_act, act_ids)
        v, i, l = (x.cpu().numpy() for x in ev.active_lmhead_topk(h, W_act, to_dev_i32(ids), k))
        check_equal_rows(v, i, ids, group, f"{layout} V_act={V_act} d={d} M={M}")
        check_head(v, i, l, ref, ids, k, f"{layout} V_act={V_act} d={d} M={M}")
        got[layout] = (v, i, l)
    for a, b in zip(*got.values()):
        assert np.array_equal(a, b)
