"""Failure events from several threads and streams at once, more of them than there are places for the search's ids on the host: each
thread's events are what a thread by itself gets.  Also behind work that keeps the stream busy for longer than the host looks for the ids.  Needs an
MI355X: run with `-m gpu`."""
import threading

import numpy as np
import pytest

import evospec_inputs as gi
from helpers import to_dev_bf16, to_dev_i32
from test_gpu_parity import ev  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

V, d, n_core, cap, k = 3000, 128, 500, 64, 10


def events(ev, t, Wd, row_ptr, col, out, busy=False):
    import torch
    with torch.cuda.stream(torch.cuda.Stream()):
        core = gi.zipf_ranking(V, 31)[:n_core].astype(np.int32)
        arc = ev.ArcManager(capacity=cap, p0=cap // 2, ghost_cap=cap, max_insert=32, min_residency=1, warmup_events=2, slot_base=n_core, core=core)
        W_act = torch.zeros((n_core + cap, d), dtype=torch.bfloat16, device="cuda")
        act_ids = torch.full((n_core + cap,), -1, dtype=torch.int32, device="cuda")
        ev.active_gather(Wd, to_dev_i32(core), None, W_act, act_ids)
        ws = torch.empty(ev.path_a_workspace_bytes(V, d, k, 32), dtype=torch.uint8, device="cuda")
        rng = np.random.default_rng(t)
        a = torch.zeros((4096, 4096), dtype=torch.bfloat16, device="cuda") if busy else None
        got = []
        for e in range(6):
            h = to_dev_bf16(gi.gen_h(1, d, 100 * t + e))
            for _ in range(100 if busy else 0):
                a = a @ a
            got.append(ev.path_a_event(arc, h, Wd, rng.integers(0, V, 10).astype(np.int32), k, row_ptr, col, 8, W_act, act_ids, ws))
            arc.advance(1)
        torch.cuda.current_stream().synchronize()
        out[t] = (got, act_ids.cpu().numpy(), W_act.cpu().view(torch.int16).numpy())


def test_events_of_threads(ev):
    import torch
    Wd = to_dev_bf16(gi.gen_W_lm(V, d))
    row_ptr, col = gi.bigram_graph(V, 12)
    torch.cuda.synchronize()
    alone, together = {}, {}
    for t in range(20):
        events(ev, t, Wd, row_ptr, col, alone, busy=t == 3)
    threads = [threading.Thread(target=events, args=(ev, t, Wd, row_ptr, col, together)) for t in range(20)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert sorted(together) == list(range(20))
    for t in range(20):
        assert alone[t][0] == together[t][0] and any(alone[t][0])
        assert np.array_equal(alone[t][1], together[t][1]) and np.array_equal(alone[t][2], together[t][2])
