"""The KL gate on both sides of its launches' lines: rows of logits that start at any 4-byte place and end with one to three logits of their
own, events whose selection and draft logits share a launch and events that are too many for that, hidden states too large for it.  Needs an MI355X: run
with `-m gpu`."""
import numpy as np
import pytest

import evospec_inputs as gi
from test_gpu_kl_gate import check, ev, run  # noqa: F401  (fixture and helpers)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,V,d,K,T", [
    (3, 32769, 64, 256, 1.0),       # a tail of one logit in the last of eight slices
    (2, 40002, 64, 17, 2.0),        # of two
    (2, 131075, 64, 256, 1.0),      # of three, five loads per thread
    (2, 7, 8, 3, 1.0),              # one load and a tail
    (2, 3, 8, 2, 1.0),              # less than a load
    (3, 30001, 64, 5, 1.0),         # one slice
    (64, 4099, 64, 256, 1.0),       # four workgroups to an event: all of a round
    (65, 4099, 64, 256, 1.0),       # one event more: apart
    (256, 300, 64, 64, 1.0),        # one workgroup to an event
    (2, 2000, 64, 130, 1.0),        # the last workgroup has two rows
    (1, 1000, 15352, 20, 1.0),      # the largest hidden state beside the selection's memory, and the next one
    (1, 1000, 15360, 20, 1.0),
])
def test_launches(ev, E, V, d, K, T):
    from oracle import kl_gate
    rng = np.random.default_rng(E + V + K)
    W, h = gi.gen_normal_bf16(V, d, 21, 0.05), gi.gen_h(E, d, 22)
    z = (rng.standard_normal((E, V)) * 2.5).astype(np.float32)
    z[:, -3:] += 6.0                                              # the tail is in the support
    check(run(ev, z, h, W, K, T), kl_gate(z, h, W, K, T), f"E={E} V={V} d={d} K={K}")
