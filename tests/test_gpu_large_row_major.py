"""Row-major matrices that the slab kernel takes past the caches, in whole lines (320 MiB and more): to the bit what it gives on
the packed matrix, also in a last slab of a few rows and a last tile of one.  Needs an MI355X: run with `-m gpu`."""
import pytest

from helpers import new_matrix, plan_route
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V_act,d,M,k,shared", [
    (82017, 2048, 60, 10, 2),      # two segments, two wavefronts to a tile
    (82011, 2048, 20, 10, 1),
    (43001, 4096, 33, 20, 1),      # one wavefront per tile
    (43001, 4096, 12, 10, 1),      # one block of draft rows
    (219009, 768, 64, 10, None),   # one segment
    (656001, 256, 24, 1, None),    # a single chunk
])
def test_past_the_caches(ev, V_act, d, M, k, shared):
    import torch
    r = plan_route(M, V_act, d, k, torch.cuda.get_device_properties(0).multi_processor_count)
    assert r["kernel"] == "slab" and shared in (None, r["shared"]) and V_act * d * 2 >= 320 << 20
    assert r["segments"] == (2 if d % 2048 == 0 else 1)
    g = torch.Generator(device="cuda").manual_seed(V_act)
    W = torch.empty((V_act, d), dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=g)
    h = torch.empty((M, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    W[V_act - 1] = 2 * h[0] / d ** 0.5                             # the last row wins for the first draft row
    ids = torch.randperm(V_act, generator=g, device="cuda").to(torch.int32)
    P, out = new_matrix(ev, V_act, d, "packed"), []
    ev.active_gather(W, torch.arange(V_act, dtype=torch.int32, device="cuda"), None, P, torch.empty_like(ids))
    for W_act in (P, W):
        out.append(ev.active_lmhead_topk(h, W_act, ids, k))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert out[1][1][0, 0] == ids[-1]
    ref = h[:2].double() @ W.double().t()
    torch.testing.assert_close(out[1][0][:2].double(), ref.topk(k, dim=1).values, rtol=1e-4, atol=1e-4)
    torch.testing.assert_close(out[1][2][:2].double(), ref.logsumexp(1), rtol=1e-4, atol=1e-4)
