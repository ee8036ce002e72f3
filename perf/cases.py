"""Performance cases of the CIS token loss: what a training program has the library do, over the
sizes, directions, data types and options it is used with.

Three kinds of call are measured, each through the package's public entry points:

  loss     the token loss on logits [T, V], forward only or fused with its gradient, through a
           LossCall (a training loop keeps one per micro-batch shape). The rate-1 CIS path by
           default; with an operator or the decoupled objective, the extended entry points.
  weights  an operator's weights from recorded log-probabilities (weights_ex).
  lmhead   the loss behind the language-model head on hidden states [T, H] and a head weight
           [V, H] (lmhead_loss_fwd / lmhead_loss_bwd), with kept gradient buffers and workspace.

Inputs follow the rollouts of ``workloads``: two engines whose logits differ by a small
perturbation (0.1% of the rows by a large one), ids drawn from the inference engine's softmax,
its log-probabilities recorded in float32, and group-normalised binary advantages.
"""

from __future__ import annotations

import math

import torch

import paper_2609_32444_amd as cis

KAPPA = 5e-3
CLIP_LOW, CLIP_HIGH = 0.2, 0.28
# Operators and their bounds (the package's operator family): op id, lo, hi.
OPS = {"cis": (cis.OP_CIS, 0.0, math.inf), "tis": (cis.OP_TIS, 0.0, 2.0),
       "icepop": (cis.OP_ICEPOP, 0.5, 5.0), "two_sided": (cis.OP_TWO_SIDED, 0.0, math.inf),
       "seq_tis": (cis.OP_SEQ_TIS, 0.0, 2.0), "seq_mis": (cis.OP_SEQ_MIS, 0.5, 2.0)}
LAM = math.expm1(1.0)   # threshold c = 1 on the log-odds displacement

# Rows of a rollout batch are cut into responses of this many tokens (lengths U{lo..hi}).
RESP = (256, 1536)


def _loss(name, T, V, **kw):
    c = dict(name=name, kind="loss", T=T, V=V, dtype="bfloat16", bwd=True, op="cis",
             decoupled=False, mask=1.0, padded=0, peak=0.0)
    c.update(kw)
    return c


def _lm(name, T, V, H, **kw):
    c = dict(name=name, kind="lmhead", T=T, V=V, H=H, bwd=True, op="cis", decoupled=False,
             mask=1.0, chunk=cis.LMHEAD_CHUNK, recompute=False)
    c.update(kw)
    return c


def listed():
    return [
        # A debugging-sized batch in float32: 4 responses of 64 tokens. Launches count.
        _loss("tiny f32 fused", 256, 1024, dtype="float32"),
        # One short response of a large-vocabulary model: fewer rows than the chip has CUs.
        _loss("short response fused", 96, 151936),
        # 16 prompts x 8 padded responses of up to 256 tokens, peaked rows.
        _loss("small fused", 32768, 32768, padded=256, peak=1.0),
        # The packed MoE rollout batch, fused: the step every training iteration takes.
        _loss("rollout fused", 16384, 151936),
        # The same batch, loss and weights only (evaluation, old log-probabilities).
        _loss("rollout forward", 16384, 151936, bwd=False),
        # Wide vocabulary: rows that no longer fit a compute unit's registers; a quarter masked.
        _loss("wide fused", 16384, 262144, mask=0.75),
        # An odd vocabulary (padded row stride, ragged last vector) and an odd row count on the
        # decoupled PPO-clip path with a masking operator.
        _loss("ragged decoupled", 3001, 50257, op="icepop", decoupled=True, mask=0.9),
        # Sequence-level weights of a long-response batch: 64 responses of 8192 tokens.
        dict(name="sequence weights", kind="weights", T=524288, op="seq_tis", resp=8192,
             mask=1.0),
        # The loss behind the LM head on the rollout batch: evaluation, and the training step.
        _lm("head forward", 16384, 151936, 2048, bwd=False),
        _lm("head fwd+bwd", 16384, 151936, 2048),
        # A short ragged micro-batch through a small head, decoupled, a tenth of it masked.
        _lm("head ragged decoupled", 1777, 50257, 1600, op="tis", decoupled=True, mask=0.9),
        # A caller short of memory: small chunks, logits never stored.
        _lm("head recompute", 4096, 151936, 2048, chunk=2048, recompute=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loss", "loss", "loss", "weights", "lmhead", "lmhead"])
    if kind == "weights":
        return dict(kind=kind, T=_log_int(rng, 1000, 1 << 20),
                    op=rng.choice(["cis", "tis", "two_sided", "seq_tis", "seq_mis"]),
                    resp=_log_int(rng, 256, 8192), mask=rng.choice([1.0, 0.75]))
    op, decoupled = rng.choice([("cis", False), ("cis", False), ("cis", True), ("tis", True),
                                ("icepop", True), ("two_sided", False), ("seq_tis", True)])
    if kind == "lmhead":
        while True:
            T, V = _log_int(rng, 256, 16384), _log_int(rng, 8192, 151936)
            H = 8 * _log_int(rng, 64, 512)
            if T * V * H <= 16384 * 151936 * 2048:
                break
        return dict(kind=kind, T=T, V=V, H=H, bwd=rng.random() < 0.7, op=op,
                    decoupled=decoupled, mask=rng.choice([1.0, 0.9]),
                    chunk=rng.choice([1024, 2048, 4096, 4096, 8192]),
                    recompute=rng.random() < 0.2)
    f32 = rng.random() < 0.25
    while True:
        T, V = _log_int(rng, 32, 32768), _log_int(rng, 1024, 262144)
        if T * V * (2 if f32 else 1) <= 16384 * 262144:
            break
    return dict(kind=kind, T=T, V=V, dtype="float32" if f32 else "bfloat16",
                bwd=rng.random() < 0.7, op=op, decoupled=decoupled,
                mask=rng.choice([1.0, 1.0, 0.75]), padded=0, peak=rng.choice([0.0, 0.8]))


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------

def _advantages(n_resp, g, group=16):
    """Group-normalised binary rewards of n_resp responses (a group has at least one of each)."""
    n = (n_resp + group - 1) // group
    r = (torch.rand(n, group, generator=g, device="cuda") < 0.5).double()
    r[:, 0], r[:, 1] = 0.0, 1.0
    a = (r - r.mean(1, keepdim=True)) / (r.std(1, keepdim=True, unbiased=False) + 1e-6)
    return a.reshape(-1)[:n_resp].float()


def _responses(T, lo, hi, seed):
    """Offsets [n + 1] of responses packed back to back over T tokens."""
    gc = torch.Generator().manual_seed(int(seed))
    n = T // lo + 2
    off = torch.cumsum(torch.randint(lo, hi + 1, (n,), generator=gc), 0)
    off = torch.cat([torch.zeros(1, dtype=torch.int64), off[off < T], torch.tensor([T])])
    return off.cuda()


def _sample(z, sd, g):
    """The inference engine: ids ~ softmax(z + delta) and their log-probabilities."""
    zi = (z + sd[:, None] * torch.randn(z.shape, generator=g, device=z.device)).bfloat16().float()
    e = torch.empty_like(zi).exponential_(generator=g)
    y = torch.argmax(zi - torch.log(e), dim=1)
    lse = torch.logsumexp(zi, dim=1)
    return y, (zi.gather(1, y[:, None])[:, 0] - lse).clamp_(max=0.0)


def _rollout(case, seed, logits_of):
    """Per-row inputs of T rows whose training logits logits_of(r0, n) gives in float32."""
    T = case["T"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 2 + 1)
    off = _responses(T, min(RESP[0], max(T // 4, 1)), min(RESP[1], max(T // 2, 1)), seed)
    n_resp = off.numel() - 1
    adv = torch.repeat_interleave(_advantages(n_resp, g), off[1:] - off[:-1])
    sd = torch.full((T,), 0.03, device="cuda")
    sd[torch.rand(T, generator=g, device="cuda") < 0.001] = 2.0
    if case.get("padded"):
        n = case["padded"]
        lens = torch.randint(n // 4, n + 1, (T // n + 1, 1), generator=g, device="cuda")
        mask = (torch.arange(n, device="cuda")[None, :] < lens).reshape(-1)[:T]
    else:
        mask = torch.rand(T, generator=g, device="cuda") < case["mask"]
    ids = torch.empty(T, dtype=torch.int64, device="cuda")
    lq = torch.empty(T, device="cuda")
    old = torch.empty(T, device="cuda") if case["decoupled"] else None
    step = max(1, min(T, (1 << 27) // case["V"]))
    for r0 in range(0, T, step):
        z = logits_of(r0, min(step, T - r0))
        s = slice(r0, r0 + z.shape[0])
        ids[s], lq[s] = _sample(z, sd[s], g)
        if old is not None:  # the training engine's own value at the rollout snapshot
            z += 0.3 * torch.randn(z.shape, generator=g, device="cuda")
            old[s] = z.gather(1, ids[s][:, None])[:, 0] - torch.logsumexp(z, dim=1)
        del z
    n_valid = max(int(mask.sum()), 1)
    return dict(ids=ids, lq=lq, adv=adv.contiguous(), mask=mask.to(torch.uint8).contiguous(),
                old=old, off=off if case["op"].startswith("seq") else None, scale=-1.0 / n_valid)


def _zipf(V):
    return -1.1 * torch.log(torch.arange(1, V + 1, device="cuda", dtype=torch.float32))


def _loss_inputs(case, seed):
    T, V = case["T"], case["V"]
    dt = getattr(torch, case["dtype"])
    epv = 16 // dt.itemsize
    logits = torch.zeros(T, (V + epv - 1) // epv * epv, dtype=dt, device="cuda")[:, :V]
    bias, g = _zipf(V), torch.Generator(device="cuda").manual_seed(int(seed) * 2)

    def rows(r0, n):
        z = bias + 2.0 * torch.randn(n, V, generator=g, device="cuda")
        if case["peak"]:  # confident rows: one logit well above the rest
            at = torch.arange(n, device="cuda")[torch.rand(n, generator=g, device="cuda")
                                                < case["peak"]]
            col = torch.randint(0, V, (at.numel(),), generator=g, device="cuda")
            z[at, col] = z.max(dim=1).values[at] + 4.69
        logits[r0:r0 + n] = z
        return logits[r0:r0 + n].float()

    return dict(logits=logits, **_rollout(case, seed, rows))


def _lm_inputs(case, seed):
    T, V, H = case["T"], case["V"], case["H"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 2)
    w = torch.randn(V, H, generator=g, device="cuda") * (2.0 / math.sqrt(H - 1))
    w[:, 0] = _zipf(V)
    h = torch.randn(T, H, generator=g, device="cuda")
    h[:, 0] = 1.0
    w, h = w.bfloat16(), h.bfloat16()
    return dict(hidden=h, weight=w,
                **_rollout(case, seed, lambda r0, n: (h[r0:r0 + n] @ w.T).float()))


def _weights_inputs(case, seed):
    T = case["T"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    # most sampled tokens are confident: -log p is small for 80% of them
    conf = torch.rand(T, generator=g, device="cuda") < 0.8
    lp = -torch.empty(T, device="cuda").exponential_(generator=g) * torch.where(conf, 0.02, 1.5)
    lq = lp + torch.where(conf, 0.002, 0.03) * torch.randn(T, generator=g, device="cuda")
    mask = (torch.rand(T, generator=g, device="cuda") < case["mask"]).to(torch.uint8)
    off = None
    if case["op"].startswith("seq"):
        off = _responses(T, case["resp"], case["resp"], seed)
    return dict(lp=lp, lq=lq.clamp_(max=0.0), mask=mask, off=off)


def _params(case, scale=1.0):
    op, lo, hi = OPS[case["op"]]
    return cis.params(op, lam=LAM, kappa=KAPPA, lo=lo, hi=hi, clip_low=CLIP_LOW,
                      clip_high=CLIP_HIGH, scale=scale)


def _base(case):
    return case["op"] == "cis" and not case["decoupled"]


def _stats(ws):
    """Views of the statistics block at the workspace's start: the loss in float64, the row
    counts that no tie can move (valid, bad ids, not finite) and the largest |log k|."""
    return {"sum": ws[:8].view(torch.float64), "rows": ws[8:32].view(torch.int64),
            "max_logk": ws[40:48].view(torch.float64)}


def prepare(case, seed):
    s = _prepare(case, seed)
    s["stats"] = _stats(s["call"].workspace if "call" in s else s["ws"])
    return s


def _prepare(case, seed):
    if case["kind"] == "weights":
        s = _weights_inputs(case, seed)
        n_seq = 0 if s["off"] is None else s["off"].numel() - 1
        s["ws"] = torch.empty(cis.workspace_bytes_ex(case["T"], n_seq), dtype=torch.uint8,
                              device="cuda")
        return dict(case=case, params=_params(case), **s)
    if case["kind"] == "lmhead":
        s = _lm_inputs(case, seed)
        n_seq = 0 if s["off"] is None else s["off"].numel() - 1
        bwd, T, V, H = case["bwd"], case["T"], case["V"], case["H"]
        n = cis.lmhead_workspace_bytes(T, V, H, case["chunk"], n_seq, with_grad=bwd,
                                       recompute=bwd and case["recompute"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        if bwd:
            s["dh"] = torch.empty(T, H, device="cuda")
            s["dw"] = torch.empty(V, H, device="cuda")
        return dict(case=case, params=_params(case, s["scale"]), **s)
    s = _loss_inputs(case, seed)
    call = cis.LossCall(s["logits"], s["ids"], s["lq"], s["adv"], s["mask"], lam=LAM,
                        kappa=KAPPA, scale=s["scale"], bwd=case["bwd"],
                        params=None if _base(case) else _params(case, s["scale"]),
                        logp_old=s["old"], seq_offsets=s["off"])
    return dict(case=case, call=call)


def run(state):
    case = state["case"]
    if case["kind"] == "weights":
        out = cis.weights_ex(state["lp"], state["lq"], state["mask"], params=state["params"],
                             seq_offsets=state["off"], workspace=state["ws"])
    elif case["kind"] == "lmhead":
        args = (state["hidden"], state["weight"], state["ids"], state["lq"], state["adv"],
                state["mask"])
        kw = dict(params=state["params"], logp_old=state["old"], seq_offsets=state["off"],
                  chunk=case["chunk"], workspace=state["ws"])
        if case["bwd"]:
            out = cis.lmhead_loss_bwd(*args, **kw, dhidden=state["dh"], dweight=state["dw"],
                                      recompute=case["recompute"])
        else:
            out = cis.lmhead_loss_fwd(*args, **kw)
    else:
        out = state["call"].run()
    # of the workspace, the statistics at its start: they stay on the device
    return {**{k: v for k, v in out.items() if k != "workspace"}, **state["stats"]}


# ------------------------------------------------------------------------------------------
# What a pass cannot do without, and how far correct results may differ
# ------------------------------------------------------------------------------------------

def work(case):
    T = case["T"]
    if case["kind"] == "weights":
        return {"bytes": T * (4 + 4 + 1 + 4 + 1 + 4), "flops": 0}
    rows = 8 + 4 + 4 + 1 + (4 if case["decoupled"] else 0) + 4 + 4 + 1 + 4
    if case["kind"] == "lmhead":
        V, H = case["V"], case["H"]
        n = 2 * (T + V) * H + T * rows + (4 * (T + V) * H if case["bwd"] else 0)
        return {"bytes": n, "flops": 2 * T * V * H * (3 if case["bwd"] else 1)}
    es = 4 if case["dtype"] == "float32" else 2
    valid = T * (0.625 if case["padded"] else case["mask"])
    n = valid * case["V"] * es + (T * case["V"] * es if case["bwd"] else 0) + T * rows
    return {"bytes": int(n), "flops": 0}


def tolerance(case):
    """About four times the largest error against float64, by what the outputs are made of."""
    lm, bwd = case["kind"] == "lmhead", case.get("bwd", False)
    if lm and bwd:      # float32 products whose operand is the gradient rounded to bf16: 3.3e-3
        return {"rel": 1e-2, "differ": 2e-3}
    if bwd and case["dtype"] == "bfloat16":      # gradients rounded once to bf16: 2.1e-3
        return {"rel": 8e-3, "differ": 2e-3}
    if lm:              # displacements from float32 dot products of the logits: 2.8e-5
        return {"rel": 1e-4, "differ": 2e-3}
    return {"rel": 1e-5, "differ": 2e-3}         # float32 sums of a row: 2.1e-6


# ------------------------------------------------------------------------------------------
# The same results in float64, in plain torch
# ------------------------------------------------------------------------------------------

def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _op_weight(case, lp, one_m_p, lq, mask, off):
    lam, kap = _f32(LAM), _f32(KAPPA)
    _, lo, hi = OPS[case["op"]]
    dk = lp - lq
    if case["op"].startswith("seq"):
        s = torch.cumsum(torch.where(mask, dk, 0.0), 0)
        s = torch.cat([torch.zeros_like(s[:1]), s])
        K = torch.exp(s[off[1:]] - s[off[:-1]])
        k = torch.repeat_interleave(K, off[1:] - off[:-1])
    else:
        k = torch.exp(dk)
    cap = 1.0 + lam * torch.clamp(one_m_p, min=kap)
    if case["op"] == "cis":
        return torch.minimum(k, cap)
    if case["op"] == "two_sided":
        return torch.maximum(torch.minimum(k, cap), (1.0 + torch.exp(lp)) / 2)
    if case["op"] in ("tis", "seq_tis"):
        return k.clamp(max=hi)
    return torch.where((k >= lo) & (k <= hi), k, 0.0)


def _exact_rows(case, s, z, r):
    """Per-row outputs and dL/dlogits of rows r with float64 logits z; w0 is the decoupled
    path's weight."""
    y, lq, adv = s["ids"][r], s["lq"][r].double(), s["adv"][r].double()
    mask, scale = s["mask"][r] != 0, _f32(s["scale"])
    e = torch.softmax(z, dim=1)
    lt = z.gather(1, y[:, None])[:, 0] - torch.logsumexp(z, dim=1)
    e.scatter_(1, y[:, None], 0.0)
    one_m_p = e.sum(1)
    if case["decoupled"]:
        w = s["w0"][r]
        rho = torch.exp(lt - s["old"][r].double())
        lo, hi = 1.0 - _f32(CLIP_LOW), 1.0 + _f32(CLIP_HIGH)
        a, b = rho * adv, rho.clamp(lo, hi) * adv
        terms, coef = scale * w * torch.minimum(a, b), scale * w * torch.where(a <= b, a, 0.0)
    else:
        w = _op_weight(case, lt, one_m_p, lq, mask, None)
        terms, coef = scale * w * adv * lt, scale * w * adv
    op_lp = s["old"][r].double() if case["decoupled"] else lt
    op_1mp = -torch.expm1(op_lp) if case["decoupled"] else one_m_p
    rows = dict(logp_train=lt, w=w, terms=terms, eps=_eps(op_lp, op_1mp, lq), logk=op_lp - lq)
    rows = {k: torch.where(mask, v, 0.0) for k, v in rows.items()}
    grad = None
    if case["bwd"]:
        coef = torch.where(mask, coef, 0.0)
        grad = e.mul_(-coef[:, None])
        grad.scatter_(1, y[:, None], (coef * one_m_p)[:, None])
    return rows, grad


def _eps(lp, one_m_p, lq):
    """logit p - logit q, from the two log-probabilities and 1 - p."""
    return (lp - lq) - (torch.log(one_m_p) - torch.log(-torch.expm1(lq)))


def exact(case, seed):
    if case["kind"] == "weights":
        s = _weights_inputs(case, seed)
        lp, lq, mask = s["lp"].double(), s["lq"].double(), s["mask"] != 0
        w = _op_weight(case, lp, -torch.expm1(lp), lq, mask, s["off"])
        return {"w": torch.where(mask, w, 0.0), "acted": None,
                "eps": torch.where(mask, _eps(lp, -torch.expm1(lp), lq), 0.0), "sum": None,
                "rows": None, "max_logk": (lp - lq)[mask].abs().max()[None]}
    lm = case["kind"] == "lmhead"
    s = _lm_inputs(case, seed) if lm else _loss_inputs(case, seed)
    T, V = case["T"], case["V"]
    if case["decoupled"]:
        lo, lq = s["old"].double(), s["lq"].double()
        s["w0"] = _op_weight(case, lo, -torch.expm1(lo), lq, s["mask"] != 0, s["off"])
    names = ("logp_train", "w", "terms", "eps", "logk")
    out = {k: torch.empty(T, dtype=torch.float64, device="cuda") for k in names}
    if lm:
        h, w = s["hidden"].double(), s["weight"].double()
        dh, dw = (torch.zeros_like(h), torch.zeros_like(w)) if case["bwd"] else (None, None)
    elif case["bwd"]:
        grad = torch.empty(T, V, dtype=torch.float64, device="cuda")
    step = max(1, min(T, (1 << 28) // V))
    for r0 in range(0, T, step):
        r = slice(r0, min(T, r0 + step))
        z = h[r] @ w.T if lm else s["logits"][r].double()
        rows, g = _exact_rows(case, s, z, r)
        for k in names:
            out[k][r] = rows[k]
        if g is not None and lm:
            dh[r] = g @ w
            dw += g.T @ h[r]
        elif g is not None:
            grad[r] = g
        del z, g
    out["max_logk"] = out.pop("logk").abs().max()[None]
    out["loss"] = out["terms"].sum()[None]
    out["sum"], out["rows"] = out["loss"], None
    if lm:
        out["acted"] = None
        if case["bwd"]:
            out.update(dhidden=dh, dweight=dw)
    else:
        del out["eps"]
        out["trunc"] = None
        if case["bwd"]:
            out["dlogits"] = grad
    return out
