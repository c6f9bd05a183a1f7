"""What a user of the active-vocabulary LM head has it do, as cases that can be measured.

Every case goes through the package's public entry points on inputs that live on the GPU, with the
outputs and the workspace that a decode loop keeps.  Sizes are those of `evospec_inputs.py` and
`bench.py` (a 151,936 x 4,096 LM head, 60 draft rows, top 10) and generic odd ones.

Kinds:
  head       the restricted head on a compact matrix (packed or row-major) or on all of W_lm
  step       the head, with a dynamic-buffer update riding behind it (one call)
  update     a dynamic-buffer update, then the head (two calls)
  batched    several sequences over a shared core, each with its own extension
  gather     a full rebuild of the compact matrix
  kl_gate    the retained-support KL gate over a batch of verification events
  event      a whole failure event: exact search, candidates, admission, insertion
"""
import math

import numpy as np
import torch

import paper_2605_27390_amd as ev

DEV = "cuda"
V_FULL = 151936


def listed():
    return [
        # a small vocabulary and model: a call is launches and latency
        {"name": "tiny head", "kind": "head", "layout": "packed", "V": 8192, "V_act": 1024, "d": 256, "M": 8, "k": 8},
        # one depth of the draft tree: a few rows, after a 256-row refresh of the dynamic buffer
        {"name": "depth update + head", "kind": "update", "layout": "packed", "V": V_FULL, "V_act": 18432, "d": 4096,
         "M": 8, "k": 10, "n": 256},
        # the smallest static core of the budget study, a whole draft tree at once
        {"name": "8k core head", "kind": "head", "layout": "packed", "V": V_FULL, "V_act": 8448, "d": 4096, "M": 60, "k": 10},
        # the decode loop's draft step: 32k core + 4k dynamic ids, 60 tree nodes, 32 admitted ids applied behind it
        {"name": "draft step", "kind": "step", "layout": "packed", "V": V_FULL, "V_act": 36864, "d": 4096, "M": 60, "k": 10,
         "n": 32},
        # a smaller model whose caller keeps the compact matrix row-major
        {"name": "d2048 row-major head", "kind": "head", "layout": "row_major", "V": 128256, "V_act": 32256, "d": 2048,
         "M": 60, "k": 10},
        # sizes that divide nothing: ragged rows, hidden size and tree, a wider top-k
        {"name": "ragged head", "kind": "head", "layout": "packed", "V": 50257, "V_act": 20011, "d": 3000, "M": 37, "k": 20},
        # the unpruned head on W_lm as it is
        {"name": "full-vocabulary head", "kind": "head", "layout": "full", "V": V_FULL, "V_act": V_FULL, "d": 4096, "M": 60,
         "k": 10},
        # batched serving at full load: 16 sequences x 60 rows
        {"name": "batched 16 x 60", "kind": "batched", "layout": "packed", "V": V_FULL, "V_core": 32768, "V_arc": 2048,
         "d": 4096, "S": 16, "M": 960, "ragged": False, "k": 10},
        # a small batch whose trees have different sizes
        {"name": "batched ragged 4", "kind": "batched", "layout": "packed", "V": V_FULL, "V_core": 16384, "V_arc": 1000,
         "d": 4096, "S": 4, "M": 197, "ragged": True, "k": 10},
        # a new active set: the compact matrix is built from W_lm
        {"name": "rebuild", "kind": "gather", "layout": "packed", "V": V_FULL, "V_act": 36864, "d": 4096},
        # the admission gate over one verification round
        {"name": "kl gate 60", "kind": "kl_gate", "V": V_FULL, "d": 4096, "E": 60, "K": 256, "T": 1.0},
        # failure events, one after the other
        {"name": "failure event", "kind": "event", "layout": "packed", "V": V_FULL, "n_core": 32000, "d": 4096, "k": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _hidden(rng, lo=256, hi=4096):
    """Mostly the round hidden sizes of models, sometimes any multiple of 8."""
    if rng.random() < 0.7:
        return rng.choice([x for x in (256, 512, 768, 1024, 1536, 2048, 2560, 3072, 4096) if lo <= x <= hi])
    return 8 * _log(rng, lo // 8, hi // 8)


def _top(rng):
    return 10 if rng.random() < 0.5 else _log(rng, 1, 64)


def draw(rng):
    kind = rng.choice(["head"] * 4 + ["step", "update", "batched", "batched", "gather", "kl_gate", "event"])
    layout = "packed" if rng.random() < 0.7 else "row_major"
    if kind == "head":
        V_act = _log(rng, 1024, 65536)
        return {"kind": kind, "layout": layout, "V": 2 * V_act + rng.randrange(999), "V_act": V_act, "d": _hidden(rng),
                "M": _log(rng, 1, 64) if rng.random() < 0.7 else _log(rng, 65, 512), "k": _top(rng)}
    if kind in ("step", "update"):
        V_act = _log(rng, 4096, 40000)
        return {"kind": kind, "layout": layout, "V": 2 * V_act + rng.randrange(999), "V_act": V_act, "d": _hidden(rng, 1024),
                "M": _log(rng, 1, 64), "k": _top(rng), "n": _log(rng, 1, 32 if kind == "step" else 256)}
    if kind == "batched":
        S = rng.randrange(2, 17)
        return {"kind": kind, "layout": layout, "V": V_FULL, "V_core": _log(rng, 4096, 32768), "V_arc": _log(rng, 128, 2048),
                "d": rng.choice((2048, 4096)), "S": S, "M": rng.randrange(8 * S, 60 * S + 1), "ragged": True, "k": _top(rng)}
    if kind == "gather":
        V_act = _log(rng, 2048, 65536)
        return {"kind": kind, "layout": layout, "V": 2 * V_act + rng.randrange(999), "V_act": V_act, "d": _hidden(rng)}
    if kind == "kl_gate":
        return {"kind": kind, "V": _log(rng, 32000, V_FULL), "d": _hidden(rng), "E": _log(rng, 1, 64),
                "K": 256 if rng.random() < 0.5 else _log(rng, 8, 256), "T": rng.choice((1.0, 2.0))}
    return {"kind": kind, "layout": layout, "V": _log(rng, 32000, V_FULL), "n_core": _log(rng, 4096, 16384), "d": _hidden(rng, 1024),
            "k": 10}


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weights(V, d, g):
    return torch.empty((V, d), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)


def _hidden_states(M, d, g):
    return torch.empty((M, d), dtype=torch.bfloat16, device=DEV).normal_(0.0, 1.0, generator=g)


def _matrix(layout, rows, d, batch=None):
    """An empty compact matrix (or `batch` of them); pad elements start at zero, so that whole buffers compare."""
    if layout == "packed":
        n = ev.matrix_bytes(rows, d, ev.PACKED) // 2 * (batch or 1)
        return ev.PackedMatrix(rows, d, batch=batch, data=torch.zeros(n, dtype=torch.bfloat16, device=DEV))
    return torch.zeros((rows, d) if batch is None else (batch, rows, d), dtype=torch.bfloat16, device=DEV)


def _buffer(W):
    return W.data if isinstance(W, ev.PackedMatrix) else W


def _outputs(M, k):
    return (torch.empty((M, k), dtype=torch.float32, device=DEV), torch.empty((M, k), dtype=torch.int32, device=DEV),
            torch.empty((M,), dtype=torch.float32, device=DEV))


def _row_off(case, seed):
    """Draft rows per sequence: equal, or any split of M with at least one row each."""
    S, M = case["S"], case["M"]
    if not case["ragged"]:
        return [M // S * s for s in range(S)] + [M]
    cuts = np.sort(np.random.default_rng(seed).choice(np.arange(1, M), size=S - 1, replace=False))
    return [0] + [int(x) for x in cuts] + [M]


def _draw_inputs(case, seed):
    """Everything random about a case, from the seed alone."""
    g = _gen(seed)
    kind, V, d = case["kind"], case["V"], case["d"]
    x = {"W_lm": _weights(V, d, g)}
    if kind in ("head", "step", "update", "batched"):
        x["h"] = _hidden_states(case["M"], d, g)
    if case.get("layout") == "full":
        return x
    if kind == "kl_gate":
        # the target's logits: the draft's own, plus what the draft gets wrong
        x["h"] = _hidden_states(case["E"], d, g)
        z = x["h"].float() @ x["W_lm"].float().t()
        x["z"] = z.add_(torch.randn(z.shape, generator=g, device=DEV), alpha=0.5)
        return x
    perm = torch.randperm(V, generator=g, device=DEV).to(torch.int32)
    if kind == "batched":
        x["core"] = perm[:case["V_core"]].clone()
        rest = perm[case["V_core"]:]
        x["arc"] = torch.stack([rest[torch.randperm(rest.numel(), generator=g, device=DEV)[:case["V_arc"]]]
                                for _ in range(case["S"])]).contiguous()
        x["row_off"] = _row_off(case, seed)
    elif kind == "event":
        x["core"] = perm[:case["n_core"]].cpu().numpy()
        r = np.random.default_rng(seed)
        # co-occurrence graph (12 successors per token on average, 64 at most) and the events' own inputs
        deg = np.minimum(r.geometric(1 / 12, size=V) - 1, 64)
        x["row_ptr"] = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        x["col_idx"] = r.integers(0, V, int(x["row_ptr"][-1])).astype(np.int32)
        x["h"] = [_hidden_states(1, d, g) for _ in range(16)]
        x["top"] = [r.choice(V, 10, replace=False).astype(np.int32) for _ in range(16)]
    else:
        x["ids"] = perm[:case["V_act"]].clone()
        if kind in ("step", "update"):
            n = case["n"]
            x["new_ids"] = perm[case["V_act"]:case["V_act"] + n].clone()
            # the dynamic part is the last ninth of the active set
            first = case["V_act"] - max(n, case["V_act"] // 9)
            x["slots"] = (first + torch.randperm(case["V_act"] - first, generator=g, device=DEV)[:n]).to(torch.int32)
    return x


def prepare(case, seed):
    x = _draw_inputs(case, seed)
    kind, d = case["kind"], case["d"]
    s = {"case": case, "W_lm": x["W_lm"], "h": x.get("h")}
    if kind == "kl_gate":
        E, K, V = case["E"], case["K"], case["V"]
        s["z"] = x["z"]
        s["out"] = (torch.empty((E, K), dtype=torch.int32, device=DEV), torch.empty((E, K), dtype=torch.float32, device=DEV),
                    torch.empty((E, K), dtype=torch.float32, device=DEV), torch.empty((E,), dtype=torch.float32, device=DEV))
        s["ws"] = torch.empty(ev.kl_gate_workspace_bytes(E, V), dtype=torch.uint8, device=DEV)
        return s
    if kind == "batched":
        core, arc, S = x["core"], x["arc"], case["S"]
        s["W_core"] = _matrix(case["layout"], core.numel(), d)
        s["ids_core"] = torch.empty_like(core)
        ev.active_gather(x["W_lm"], core, None, s["W_core"], s["ids_core"])
        s["W_arc"] = _matrix(case["layout"], case["V_arc"], d, batch=S)
        s["ids_arc"] = torch.empty_like(arc)
        for i in range(S):
            ev.active_gather(x["W_lm"], arc[i], None, s["W_arc"].sub(i) if case["layout"] == "packed" else s["W_arc"][i],
                             s["ids_arc"][i])
        s["row_off"] = x["row_off"]
        s["ws"] = torch.empty(ev.workspace_bytes_segmented(case["M"], core.numel(), case["V_arc"], S, d, case["k"]),
                              dtype=torch.uint8, device=DEV)
        del s["W_lm"]                                     # (the core and the extensions are all it needs)
        return s
    if kind == "event":
        n = case["n_core"]
        ids = torch.from_numpy(x["core"]).to(DEV)
        s["W_act"] = _matrix(case["layout"], n + 256, d)
        s["ids"] = torch.zeros((n + 256,), dtype=torch.int32, device=DEV)
        ev.active_gather(x["W_lm"], ids, None, s["W_act"], s["ids"])
        s["arc"] = ev.ArcManager(slot_base=n, core=x["core"])
        s["top"], s["row_ptr"], s["col_idx"], s["at"] = x["top"], x["row_ptr"], x["col_idx"], 0
        s["ws"] = torch.empty(ev.path_a_workspace_bytes(case["V"], d, case["k"], 32), dtype=torch.uint8, device=DEV)
        return s
    if case["layout"] == "full":
        s["W_act"], s["ids"] = x["W_lm"], None
    else:
        s["W_act"] = _matrix(case["layout"], case["V_act"], d)
        s["ids"] = torch.empty_like(x["ids"])
        if kind == "gather":
            s["src"] = x["ids"]
            return s
        ev.active_gather(x["W_lm"], x["ids"], None, s["W_act"], s["ids"])
        if kind == "head":
            del s["W_lm"]
    s["new_ids"], s["slots"] = x.get("new_ids"), x.get("slots")
    s["out"] = _outputs(case["M"], case["k"])
    s["ws"] = torch.empty(ev.workspace_bytes(case["M"], case["V_act"], d, case["k"]), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind, k = case["kind"], case.get("k")
    if kind == "head":
        v, i, z = ev.active_lmhead_topk(s["h"], s["W_act"], s["ids"], k, *s["out"], workspace=s["ws"])
        return {"vals": v, "ids": i, "logz": z}
    if kind == "step":
        v, i, z = ev.active_lmhead_topk_then_update(s["h"], s["W_act"], s["ids"], k, s["W_lm"], s["new_ids"], s["slots"],
                                                    *s["out"], workspace=s["ws"])
        return {"vals": v, "ids": i, "logz": z, "act_ids": s["ids"], "W_act": _buffer(s["W_act"])}
    if kind == "update":
        ev.active_gather(s["W_lm"], s["new_ids"], s["slots"], s["W_act"], s["ids"])
        v, i, z = ev.active_lmhead_topk(s["h"], s["W_act"], s["ids"], k, *s["out"], workspace=s["ws"])
        return {"vals": v, "ids": i, "logz": z, "act_ids": s["ids"], "W_act": _buffer(s["W_act"])}
    if kind == "batched":
        v, i, z = ev.active_lmhead_topk_segmented(s["h"], s["W_core"], s["ids_core"], s["W_arc"], s["ids_arc"], s["row_off"], k,
                                                  workspace=s["ws"])
        return {"vals": v, "ids": i, "logz": z}
    if kind == "gather":
        ev.active_gather(s["W_lm"], s["src"], None, s["W_act"], s["ids"])
        return {"act_ids": s["ids"], "W_act": _buffer(s["W_act"])}
    if kind == "kl_gate":
        sup, zt, zq, kl = ev.kl_gate(s["z"], s["h"], s["W_lm"], case["K"], case["T"], *s["out"], workspace=s["ws"])
        return {"support": sup, "target": zt, "draft": zq, "kl": kl}
    j = s["at"] % len(s["top"])
    s["at"] += 1
    pairs = ev.path_a_event(s["arc"], s["h"][j], s["W_lm"], s["top"][j], k, s["row_ptr"], s["col_idx"], 8, s["W_act"], s["ids"],
                            s["ws"])
    s["arc"].advance(3)                                   # decoding steps between two failures
    return {"pairs": np.array(pairs, dtype=np.int32).reshape(-1, 2), "act_ids": s["ids"], "W_act": _buffer(s["W_act"])}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    kind, V, d = case["kind"], case["V"], case["d"]
    row = 2 * d
    if kind == "gather":
        return {"bytes": case["V_act"] * (2 * row + 8), "flops": 0}
    if kind == "kl_gate":
        E, K = case["E"], case["K"]
        return {"bytes": E * (4 * V + K * row + row + 12 * K + 4), "flops": 2 * E * K * d}
    if kind == "event":
        return {"bytes": V * row + row, "flops": 2 * V * d}
    M, k = case["M"], case["k"]
    out = M * (8 * k + 4)
    if kind == "batched":
        rows = case["V_core"] + case["S"] * case["V_arc"]
        return {"bytes": rows * (row + 4) + M * row + out, "flops": 2 * M * (case["V_core"] + case["V_arc"]) * d}
    extra = case["n"] * (2 * row + 12) if kind in ("step", "update") else 0
    ids = 0 if case["layout"] == "full" else 4
    return {"bytes": case["V_act"] * (row + ids) + M * row + out + extra, "flops": 2 * M * case["V_act"] * d}


def tolerance(case):
    if case["kind"] == "gather":
        return "exact"
    if case["kind"] == "kl_gate":
        # the divergence is what is left of two logarithms that nearly cancel (measured: 8e-6 off 64 bits)
        return {"rel": 5e-5, "max": 1e-3, "differ": 0.01}
    # Products of bf16 are exact in 32 bits: what is left is the rounding of 32-bit sums (measured: up to
    # 4e-7 off 64 bits), and ids whose logits are closer than that may trade places.
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gather", "event"):
        return None                                       # bytes and whole numbers
    x = _draw_inputs(case, seed)
    h, W = x["h"].double(), x["W_lm"]
    if kind == "kl_gate":
        K, T = case["K"], case["T"]
        zt, sup = torch.sort(x["z"].double(), dim=1, descending=True, stable=True)
        zt, sup = zt[:, :K].contiguous(), sup[:, :K]
        zq = torch.stack([W[sup[e]].double() @ h[e] for e in range(case["E"])])
        lp, lq = torch.log_softmax(zt / T, 1), torch.log_softmax(zq / T, 1)
        return {"support": None, "target": zt, "draft": zq, "kl": (lp.exp() * (lp - lq)).sum(1)}
    k = case["k"]
    if kind == "batched":
        zc = h @ W[x["core"].long()].double().t()
        vals, logz = [], []
        for s in range(case["S"]):
            lo, hi = x["row_off"][s], x["row_off"][s + 1]
            z = torch.cat([zc[lo:hi], h[lo:hi] @ W[x["arc"][s].long()].double().t()], 1)
            vals.append(torch.topk(z, k, dim=1).values)
            logz.append(torch.logsumexp(z, 1))
        return {"vals": torch.cat(vals), "ids": None, "logz": torch.cat(logz)}
    if case["layout"] == "full":
        ids = None
        z = h @ W.double().t()
    else:
        ids = x["ids"].long()
        if kind == "update":
            ids[x["slots"].long()] = x["new_ids"].long()
        z = h @ W[ids].double().t()
    r = {"vals": torch.topk(z, k, dim=1).values, "ids": None, "logz": torch.logsumexp(z, 1)}
    if kind in ("step", "update"):
        r.update(act_ids=None, W_act=None)
    return r
