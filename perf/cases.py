"""The workloads this framework is timed on: what a program that serves or calibrates an
ACE token-adaptive MoE layer calls, through the package's public entry points.

Three kinds of call:
  layer   one layer forward (`prepare_forward` where the program calls the same buffers
          again, `moe_forward` where every call brings its own shapes)
  tau     `tau_map`: contribution scores of a score pass -> thresholds of skip budgets
  tables  `build_tables`: the offline GSP / RCR tables of one layer

Layer cases carry: T tokens, d hidden, N experts, k slots per token, m expert intermediate
size, dtype, tau (the model's frozen threshold), and the options of the call.
"""
from __future__ import annotations

import functools
import math

import torch

import paper_2609_05228_amd as ace

DEV = "cuda"


def _layer(**kw):
    case = dict(kind="layer", T=1, d=2048, N=128, k=8, m=768, dtype="bf16", tau=0.1155, m_min=1, fusion="max",
                zipf=0.0, m_shared=0, skip_disable=False, write_scores=False, prepared=True)
    case.update(kw)
    return case


def listed():
    return [
        # one new token of one sequence: five dependent launches around 38 MB of weights
        _layer(name="decode_1", T=1),
        # the decode batch of the 48-layer stack: HBM-bound weight streaming
        _layer(name="decode_32", T=32),
        # a batch past the small-batch kernels, its size new on every call (continuous batching)
        _layer(name="batch_131", T=131, prepared=False),
        # a ragged prompt, its size new on every call
        _layer(name="prefill_1021", T=1021, prepared=False),
        # the benchmark's prefill: 4096 tokens at half the slots skipped
        _layer(name="prefill_4096", T=4096),
        # the wider pool: 256 experts, one shared expert, Zipf-skewed routing (matrix-bound experts)
        _layer(name="zipf_8192", T=8192, N=256, m=512, m_shared=512, zipf=1.1, tau=0.0810),
        # the score pass that calibrates tau: the plain top-k layer with the scores written
        _layer(name="score_8192", T=8192, skip_disable=True, write_scores=True),
        # the small fp32 layer
        _layer(name="f32_64", T=64, d=256, N=8, k=2, m=512, dtype="f32", tau=0.45),
        # an fp32 layer of ordinary width on a ragged batch
        _layer(name="f32_517", T=517, d=1024, N=32, k=4, m=512, dtype="f32", tau=0.23, prepared=False),
        # thresholds from one layer's score pass
        dict(name="tau_4096", kind="tau", rows=4096, k=8, m_min=1, n_q=1, q=0.5),
        # one global threshold per budget from the score passes of 48 layers x 8192 tokens
        dict(name="tau_stack", kind="tau", rows=48 * 8192, k=8, m_min=1, n_q=4, q=0.5),
        # the offline tables of one layer
        dict(name="tables_128", kind="tables", d=2048, N=128, m=768, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "batch", "prefill", "f32", "tau", "tables"])
    if kind == "tau":
        k = rng.randint(3, 8)
        return dict(kind="tau", rows=_log_int(rng, 64, 48 * 8192), k=k, m_min=rng.randint(1, min(3, k - 1)),
                    n_q=rng.randint(1, 8), q=round(rng.uniform(0.05, 0.25), 3))
    while True:
        if kind == "tables":
            case = dict(kind="tables", d=128 * _log_int(rng, 1, 16), N=_log_int(rng, 8, 256),
                        m=64 * _log_int(rng, 1, 16), dtype=rng.choice(["bf16", "bf16", "f32"]))
            if case["N"] * case["m"] ** 2 * case["d"] <= 128 * 768 ** 2 * 2048:
                return case
            continue
        lo, hi = dict(decode=(1, 64), batch=(65, 1023), prefill=(1024, 8192), f32=(1, 1024))[kind]
        N = _log_int(rng, 8, 64 if kind == "f32" else 256)
        k = rng.randint(1, min(8, N))
        m = 64 * _log_int(rng, 1, 16)
        d = 128 * _log_int(rng, 2, 8 if kind == "f32" else 16)
        case = _layer(T=_log_int(rng, lo, hi), d=d, N=N, k=k, m=m, dtype="f32" if kind == "f32" else "bf16",
                      tau=round(rng.uniform(0.6, 1.0) / k, 4), m_min=rng.randint(1, k) if rng.random() < 0.2 else 1,
                      fusion=rng.choice(["max"] * 6 + ["min", "mean", "gsp", "rcr", "score"]),
                      zipf=rng.choice([0.0, 0.0, 1.1]),
                      m_shared=rng.choice([0, 0, m, 64 * _log_int(rng, 1, 16)]),
                      skip_disable=rng.random() < 0.2, write_scores=rng.random() < 0.2,
                      prepared=rng.random() < 0.5)
        if N * m * d <= 128 * 768 * 2048 and case["T"] * (k * m + case["m_shared"]) * d <= 8192 * 8 * 768 * 2048:
            return case


# ---------------------------------------------------------------- inputs

def _normal(gen, shape, std, mean, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(mean, std, generator=gen)


def _layer_inputs(case, seed):
    """Activations N(0, 1), RMSNorm scales near one, router and expert weights N(0, 0.02), a
    Zipf router bias where asked for, and tables spread as the ones of such a layer are."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    T, d, N, m, ms = case["T"], case["d"], case["N"], case["m"], case["m_shared"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    x = _normal(gen, (T, d), 1.0, 0.0, dt)
    w = {
        "gamma": _normal(gen, (d,), 0.1, 1.0, dt),
        "w_router": _normal(gen, (N, d), 0.02, 0.0, dt),
        "b_router": None,
        "w_gate": _normal(gen, (N, m, d), 0.02, 0.0, dt),
        "w_up": _normal(gen, (N, m, d), 0.02, 0.0, dt),
        "w_down": _normal(gen, (N, d, m), 0.02, 0.0, dt),
    }
    if case["zipf"] > 0:
        rank = torch.randperm(N, generator=gen, device=DEV) + 1
        w["b_router"] = (-case["zipf"] * rank.double().log()).float()
    if ms:
        w["ws_gate"] = _normal(gen, (ms, d), 0.02, 0.0, dt)
        w["ws_up"] = _normal(gen, (ms, d), 0.02, 0.0, dt)
        w["ws_down"] = _normal(gen, (d, ms), 0.02, 0.0, dt)
    a_gsp = _normal(gen, (N,), 0.001, 1.0, torch.float32)
    a_rcr = _normal(gen, (N,), 0.08, 1.0, torch.float32)
    return x, w, a_gsp, a_rcr


def _scores(case, seed):
    """Contribution scores of a score pass: slots in descending router probability."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rows, k = case["rows"], case["k"]
    z = torch.randn((rows, k), generator=gen, device=DEV).sort(dim=1, descending=True).values * 0.4
    g = z.softmax(dim=1)
    s = g * (1 + 0.08 * torch.randn((rows, k), generator=gen, device=DEV))
    return torch.maximum(g, s / s.sum(dim=1, keepdim=True)).contiguous()


def _budgets(case):
    return ([case["q"]] + [0.1, 0.25, 0.6, 0.05, 0.4, 0.75, 0.9])[:case["n_q"]]


def prepare(case, seed):
    if case["kind"] == "tau":
        return dict(kind="tau", scores=_scores(case, seed), qs=_budgets(case), m_min=case["m_min"])
    if case["kind"] == "tables":
        gen = torch.Generator(device=DEV).manual_seed(seed)
        d, N, m = case["d"], case["N"], case["m"]
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        return dict(kind="tables", weights={
            "gamma": _normal(gen, (d,), 0.1, 1.0, dt),
            "w_router": _normal(gen, (N, d), 0.02, 0.0, dt),
            "w_gate": _normal(gen, (N, m, d), 0.02, 0.0, dt),
            "w_up": _normal(gen, (N, m, d), 0.02, 0.0, dt),
            "w_down": _normal(gen, (N, d, m), 0.02, 0.0, dt)})
    x, w, a_gsp, a_rcr = _layer_inputs(case, seed)
    kw = dict(k=case["k"], tau=case["tau"], m_min=case["m_min"], fusion=case["fusion"],
              skip_disable=case["skip_disable"], write_scores=case["write_scores"])
    if case["prepared"]:
        return dict(kind="prepared", forward=ace.prepare_forward(x, w, a_gsp, a_rcr, **kw))
    return dict(kind="layer", args=(x, w, a_gsp, a_rcr), kw=kw)


def run(state):
    if state["kind"] == "prepared":
        return state["forward"]()
    if state["kind"] == "layer":
        return ace.moe_forward(*state["args"], **state["kw"])
    if state["kind"] == "tau":
        return ace.tau_map(state["scores"], state["qs"], m_min=state["m_min"])
    return ace.build_tables(state["weights"])


# ---------------------------------------------------------------- work and tolerance

@functools.lru_cache(maxsize=None)
def _expected(T, d, N, k, tau, m_min, zipf, skip_disable):
    """(kept slots, experts with a kept slot) that such a routing gives: the same draw of
    logits N(0, 0.02 sqrt(d)) every time, equal tables."""
    gen = torch.Generator().manual_seed(1)
    z = torch.randn((T, N), generator=gen) * (0.02 * math.sqrt(d))
    if zipf > 0:
        z -= zipf * torch.arange(1, N + 1).log()
    top, idx = z.topk(k, dim=1)
    keep = torch.ones((T, k), dtype=torch.bool)
    if not skip_disable:
        keep = top.softmax(dim=1) >= tau
        keep[:, :m_min] = True
    return int(keep.sum()), int(idx[keep].unique().numel())


def work(case):
    if case["kind"] == "tau":
        return {"bytes": 4 * case["rows"] * case["k"], "flops": case["rows"] * case["k"]}
    esz = 2 if case["dtype"] == "bf16" else 4
    d, N, m = case["d"], case["N"], case["m"]
    if case["kind"] == "tables":
        # three symmetric m x m Gram matrices per expert in 64 bits, and the prototype's expert
        return {"bytes": esz * (3 * N * m * d + N * d), "flops": 3 * N * m * m * d + 6 * N * m * d}
    T, k, ms = case["T"], case["k"], case["m_shared"]
    kept, active = _expected(T, d, N, k, case["tau"], case["m_min"], case["zipf"], case["skip_disable"])
    slot_bytes = 13 if case["write_scores"] else 9
    return {"bytes": esz * (3 * active * m * d + 3 * ms * d + N * d + 2 * T * d) + slot_bytes * T * k,
            "flops": 6 * d * m * kept + 6 * T * d * ms + 2 * T * d * N}


def tolerance(case):
    if case["kind"] == "tau":
        return "exact"  # an order statistic: integers, and a midpoint rounded once
    if case["kind"] == "tables":
        # 64-bit sums, the tables rounded to fp32 at the end: one unit in the last place
        return {"rel": 2.5e-7, "max": 5e-7}
    if case["dtype"] == "f32":
        # fp32 sums of up to 2048 products in another order
        return {"rel": 4e-6, "max": 1e-4, "differ": 1e-3}
    # bf16: x_in, H, the expert outputs and y are each rounded to 8 bits; a slot whose score is
    # within fp32 rounding of tau may fall either way, and moves its token's whole row
    return {"rel": 1e-2, "max": 0.9, "differ": 1e-3}


# ---------------------------------------------------------------- in 64 bits

def exact(case, seed):
    if case["kind"] == "tau":
        return _exact_tau(_scores(case, seed), _budgets(case), case["m_min"])
    if case["kind"] == "tables":
        return _exact_tables(prepare(case, seed)["weights"])
    return _exact_layer(case, *_layer_inputs(case, seed))


def _swiglu(x, wg, wu, wd):
    g = x @ wg.double().t()
    return (g * torch.sigmoid(g) * (x @ wu.double().t())) @ wd.double().t()


def _exact_layer(case, x, w, a_gsp, a_rcr):
    T, k, N = case["T"], case["k"], case["N"]
    eps = 1e-6
    xd = x.double()
    xn = xd / (xd.square().mean(dim=1, keepdim=True) + 1e-6).sqrt() * w["gamma"].double()
    z = xn @ w["w_router"].double().t()
    if w["b_router"] is not None:
        z = z + w["b_router"].double()
    z, idx = z.sort(dim=1, descending=True, stable=True)
    z, idx = z[:, :k], idx[:, :k]
    g = z.softmax(dim=1)

    def view(table):
        s = g * table.double()[idx]
        return s / (s.sum(dim=1, keepdim=True) + eps)

    pg, pr = view(a_gsp), view(a_rcr)
    c = {"max": torch.maximum(pg, pr), "min": torch.minimum(pg, pr), "mean": (pg + pr) / 2, "gsp": pg, "rcr": pr,
         "score": g / (g.sum(dim=1, keepdim=True) + eps)}[case["fusion"]]
    if case["skip_disable"]:
        keep, gates = torch.ones_like(idx, dtype=torch.bool), g
    else:
        # tau as the layer gets it: one fp32 scalar
        keep = c >= float(torch.tensor(case["tau"], dtype=torch.float32))
        keep[:, 0] = True
        # restore skipped slots by descending c until m_min are active
        for _ in range(case["m_min"]):
            short = keep.sum(dim=1) < case["m_min"]
            best = c.masked_fill(keep, -1.0).argmax(dim=1)
            keep[short, best[short]] = True
        gates = torch.where(keep, g, torch.zeros_like(g))
        gates = gates / (gates.sum(dim=1, keepdim=True) + eps)
    y = torch.zeros((T, case["d"]), dtype=torch.float64, device=x.device)
    if "ws_gate" in w:
        y += _swiglu(xn, w["ws_gate"], w["ws_up"], w["ws_down"])
    for e in idx[keep].unique().tolist():
        tok, slot = torch.nonzero((idx == e) & keep, as_tuple=True)
        f = _swiglu(xn[tok], w["w_gate"][e], w["w_up"][e], w["w_down"][e])
        y[tok] += gates[tok, slot].unsqueeze(1) * f  # an expert holds a token at most once
    out = dict(y=y, topk_idx=idx.to(torch.int32), keep=keep.to(torch.uint8), gates=gates)
    if case["write_scores"]:
        out["scores"] = c
    return out


def _exact_tau(scores, qs, m_min):
    rows, k = scores.shape
    cand = torch.ones((rows, k), dtype=torch.bool, device=scores.device)
    cand[:, 0] = False
    if m_min > 1:
        # the m_min - 1 highest other slots of a row are never skipped (ties: lower slot first)
        best = scores[:, 1:].sort(dim=1, descending=True, stable=True).indices[:, :m_min - 1] + 1
        cand.scatter_(1, best, False)
    c = scores[cand].double().sort().values
    n = c.numel()
    taus, counts = [], []
    for q in qs:
        mq = min(max(round(q * rows * k), 0), n)
        counts.append(mq)
        if mq == 0 or mq == n:
            taus.append(0.0 if mq == 0 else math.inf)
            continue
        lo, hi = float(c[mq - 1]), float(c[mq])
        if lo == hi:  # a tie: below it or above it, whichever count is closer
            below, above = int((c < lo).sum()), int((c <= lo).sum())
            if abs(below - mq) > abs(above - mq):
                lo, hi = (lo, float(c[above])) if above < n else (math.inf, math.inf)
        taus.append((lo + hi) / 2)
    return dict(tau=torch.tensor(taus, dtype=torch.float64), m_q=torch.tensor(counts, dtype=torch.int64),
                n_cand=torch.tensor([n], dtype=torch.int64))


def _exact_tables(w):
    eps = 1e-6
    gam = w["gamma"].double()
    wr = w["w_router"].double()
    wr = wr - wr.mean(dim=0)
    q = wr / (wr.square().mean(dim=1, keepdim=True).sqrt() + eps)
    gsp, rcr = [], []
    for e in range(wr.shape[0]):
        wg, wu, wd = (w[n][e].double() for n in ("w_gate", "w_up", "w_down"))
        G, U = wg * gam, wu * gam
        D = wd.t() @ wd
        up = U.square().sum().sqrt() * (D * (G @ G.t())).sum().sqrt()
        gate = G.square().sum().sqrt() * (D * (U @ U.t())).sum().sqrt()
        gsp.append((up * gate).sqrt())
        h = wg @ q[e]
        f = wd @ (h * torch.sigmoid(h) * (wu @ q[e]))
        rcr.append(f.square().sum().sqrt() / (q[e].square().sum().sqrt() + eps))
    gsp, rcr = torch.stack(gsp), torch.stack(rcr)
    return dict(a_gsp=gsp / (gsp.mean() + eps), a_rcr=rcr / (rcr.mean() + eps))
