"""Performance cases of the library: the calls that training and evaluating a draft model makes.

listed() names a few representative calls, draw() gives more of the same ranges, prepare() makes
the inputs a training program has in hand, run() is one call sequence through the public entry
points, work() the bytes and operations no implementation can avoid, exact() the same results from
plain torch in 64 bits.

Ranges: 1 to 16 positions per window, vocabularies of 1,000 to 152,000 entries (two thirds of them
padded to a multiple of 16, the others of any length, as tokenizers with added tokens have), from a
quarter of a million logits per call up to the 1.84e9 of 2048 windows x 7 positions x 128,256.
"""
import math

import torch

import paper_2609_24150_amd as aal
from paper_2609_24150_amd.inputs import make_logits, make_uniforms

DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
BYTES = {"bf16": 2, "fp32": 4}
MOST_ELEMENTS = 2048 * 7 * 128256

# (wtv, eal, kl, tv) weights of the training objectives
WEIGHTS = {
    "wtv": (1.0, 0.0, 0.0, 0.0),
    "kl+eal": (0.0, 0.1, 1.0, 0.0),
    "kl+tv": (0.0, 0.0, 1.0, 1.0),
    "eal": (0.0, 1.0, 0.0, 0.0),
}


def listed():
    return [
        # The smallest call: a unit-test sized EAL step in fp32, bound by latency and launches.
        dict(name="eal-small", op="eal", N=64, K=4, V=1024, dtype="fp32", recipe="c1", td=1.0),
        # One micro-batch of a memory-limited training step: too few windows to fill the device.
        dict(name="wtv-micro", op="wtv", N=12, K=7, V=128256, dtype="bf16", recipe="c2", td=1.0, tt=1.0),
        # The training step of the benchmark: window total variation at full batch.
        dict(name="wtv-train", op="wtv", N=2048, K=7, V=128256, dtype="bf16", recipe="c2", td=1.0, tt=1.0),
        # Greedy-verification training over the largest vocabulary.
        dict(name="eal-train", op="eal", N=1024, K=5, V=151936, dtype="bf16", recipe="c3", td=1.0),
        # Long windows in fp32 at low temperature.
        dict(name="wtv-fp32", op="wtv", N=1024, K=16, V=32000, dtype="fp32", recipe="c4", td=0.5, tt=0.5),
        # A vocabulary with one added token: rows that no vector width divides.
        dict(name="wtv-ragged", op="wtv", N=256, K=7, V=32001, dtype="bf16", recipe="c2", td=1.0, tt=1.0),
        # Validation: the forward pass alone, over windows of ten positions.
        dict(name="wtv-eval", op="wtv", N=256, K=10, V=65536, dtype="bf16", recipe="c2", td=1.0, tt=1.0, grad=False),
        # The anchored greedy recipe over sequences with windows sliding by one, loss and gradient only.
        dict(name="kl-eal-sliding", op="loss", B=2, S=1024, K=7, V=128256, dtype="bf16", recipe="c2", weights="kl+eal",
             td=1.0, tt=1.0, sequences=True, outputs=False),
        # The anchored sampling recipe over short sequences with an unpadded vocabulary.
        dict(name="kl-tv-ragged", op="loss", B=8, S=96, K=5, V=50001, dtype="bf16", recipe="c3", weights="kl+tv",
             td=0.7, tt=0.7, sequences=True),
        # Simulated acceptance of sampled rollouts: eight per prompt.
        dict(name="sim-rollouts", op="sim", P=64, G=8, K=7, V=128256, dtype="bf16", recipe="c5", td=1.0),
        # The policy-gradient stage: 64 groups of eight windows.
        dict(name="grpo-train", op="grpo", groups=64, m=8, K=7, V=128256, dtype="bf16", recipe="c2", td=1.0),
        # One rank's share of a vocabulary split over eight ranks: partials, merge, acceptance, scan, gradient.
        dict(name="wtv-vocab-rank", op="vp", ranks=8, rank=3, N=512, K=7, V=128256, dtype="bf16", recipe="c2",
             td=1.0, tt=1.0),
    ]


def draw(rng):
    op = rng.choice(["eal", "wtv", "wtv", "loss", "loss", "sim", "grpo", "vp"])
    K = rng.choice([1, 2, 3, 4, 5, 6, 7, 7, 8, 8, 9, 10, 11, 12, 13, 14, 15, 16])
    V = int(round(math.exp(rng.uniform(math.log(1000), math.log(152000)))))
    if rng.random() < 2 / 3:
        V = V // 16 * 16
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
    most = MOST_ELEMENTS // (2 if dtype == "fp32" else 1)
    rows = max(K, int(math.exp(rng.uniform(math.log(1 << 18), math.log(most))) / V))
    c = dict(op=op, K=K, V=V, dtype=dtype, td=rng.choice([1.0, 1.0, 0.7, 0.5]))
    if op in ("eal", "wtv"):
        c.update(N=max(1, rows // K), recipe=rng.choice(["c1", "c2", "c3", "c4"]), grad=rng.random() < 0.85)
        if op == "wtv":
            c["tt"] = c["td"]
        if dtype == "bf16" and rng.random() < 0.25:
            c["grad_dtype"] = "fp32"
    elif op == "loss":
        weights = rng.choice(["wtv", "kl+eal", "kl+tv", "eal"])
        seq = rng.random() < 0.7
        S = rng.randint(K, max(K, min(2048, rows))) if seq else K
        c.update(B=max(1, rows // S), S=S, weights=weights, recipe=rng.choice(["c2", "c3"]), tt=c["td"],
                 sequences=seq, grad=rng.random() < 0.85, outputs=rng.random() < 0.5)
        if weights in ("eal", "kl+eal") and rng.random() < 0.3:
            c["labels"] = True
    elif op == "sim":
        G = rng.choice([2, 4, 8])
        c.update(P=max(1, rows // (G * K)), G=G, recipe="c5")
    elif op == "grpo":
        m = rng.choice([2, 4, 8])
        c.update(groups=max(1, int(rows * 0.75) // (m * K)), m=m, recipe="c2")
    else:
        ranks = rng.choice([2, 4, 8])
        c.update(N=max(1, min(rows, most // V // 2) // K), ranks=ranks, rank=rng.randrange(ranks), recipe="c2",
                 tt=c["td"])
    return c


# ----------------------------------------------------------------- inputs
def _slice(c):
    """[v0, v1) of the case's rank: equal slices, the last one takes the rest."""
    per = c["V"] // c["ranks"]
    v0 = c["rank"] * per
    return v0, c["V"] if c["rank"] == c["ranks"] - 1 else v0 + per


def _shape(c):
    if c["op"] in ("eal", "wtv", "vp"):
        return (c["N"], c["K"], c["V"])
    if c["op"] == "loss":
        return (c["B"], c["S"], c["V"])
    if c["op"] == "sim":
        return (c["P"], c["G"], c["K"], c["V"])
    return (c["groups"], c["m"] * c["K"], c["V"])


def _logits(c, seed):
    return make_logits(c["recipe"], _shape(c), DTYPES[c["dtype"]], seed=seed, chunk_elems=1 << 28)


def _reference(z, seed):
    """The reference draft of the policy-gradient stage: the policy perturbed."""
    g = torch.Generator(device=z.device)
    g.manual_seed(seed * 7919 + 17)
    out = torch.empty_like(z)
    for i in range(0, z.shape[0], 8):
        noise = torch.randn(z[i:i + 8].shape, generator=g, device=z.device, dtype=torch.float32)
        out[i:i + 8] = (z[i:i + 8].float() + 0.5 * noise).to(z.dtype)
    return out


def _labels(zt, seed):
    """Ground-truth tokens: the target's greedy token on nine rows of ten, any other token elsewhere."""
    rows, V = math.prod(zt.shape[:-1]), zt.shape[-1]
    g = torch.Generator(device=zt.device)
    g.manual_seed(seed * 104729 + 5)
    other = torch.randint(0, V, (rows,), generator=g, device=zt.device)
    keep = torch.rand(rows, generator=g, device=zt.device) < 0.9
    z = zt.view(rows, V)
    top = torch.cat([z[r0:r1].argmax(-1) for r0, r1 in _chunks(rows, V)])
    return torch.where(keep, top, other).int()


def prepare(case, seed):
    c = case
    zd, zt = _logits(c, seed)
    st = {"case": c, "zd": zd, "zt": zt, "labels": _labels(zt, seed) if c.get("labels") else None}
    if c["op"] == "sim":
        st["u1"], st["u2"] = make_uniforms(_shape(c)[:3], seed)
    elif c["op"] == "grpo":
        st["zref"] = _reference(zd, seed)
    elif c["op"] == "vp":
        # this rank's slices, and the records that the other ranks' all-gathers deliver
        rows, v0, v1 = c["N"] * c["K"], *_slice(c)
        zd, zt = zd.view(rows, -1), zt.view(rows, -1)
        per = c["V"] // c["ranks"]
        parts, accs, cuts = [], [], []
        for r in range(c["ranks"]):
            a, b = r * per, c["V"] if r == c["ranks"] - 1 else (r + 1) * per
            cuts.append((a, zd[:, a:b].contiguous(), zt[:, a:b].contiguous()))
            parts.append(aal.aal_vp_row_partials(cuts[-1][1], cuts[-1][2], a, aal.AAL_VP_WTV, c["td"], c["tt"],
                                                 V_total=c["V"]))
        st["parts_all"] = torch.stack(parts)
        row = aal.aal_vp_merge_rows(st["parts_all"], aal.AAL_VP_WTV, c["td"], c["tt"])
        for _, d, t in cuts:
            accs.append(aal.aal_vp_accept_partials(d, t, row, c["td"], c["tt"]))
        st["acc_all"] = torch.stack(accs)
        _, st["zd"], st["zt"] = cuts[c["rank"]]
        st["v0"] = v0
    return st


def run(state):
    c, zd, zt = state["case"], state["zd"], state["zt"]
    op = c["op"]
    grad = c.get("grad", True)
    gd = DTYPES[c["grad_dtype"]] if "grad_dtype" in c else None
    if op == "eal":
        return aal.aal_eal_fwd_bwd(zd, zt, c["td"], grad=grad, grad_dtype=gd)
    if op == "wtv":
        return aal.aal_wtv_fwd_bwd(zd, zt, c["td"], c["tt"], grad=grad, grad_dtype=gd)
    if op == "loss":
        layout = aal.AAL_LAYOUT_SEQUENCES if c["sequences"] else aal.AAL_LAYOUT_WINDOWS
        return aal.aal_loss_fwd_bwd(zd, zt, c["K"], weights=WEIGHTS[c["weights"]], temp_draft=c["td"],
                                    temp_target=c["tt"], layout=layout, labels=state["labels"], grad=grad,
                                    outputs=c.get("outputs", True))
    if op == "sim":
        return aal.aal_sim_accept_grpo(zd, zt, state["u1"], state["u2"], c["td"])
    if op == "grpo":
        return aal.aal_grpo_fwd_bwd(zd, state["zref"], zt, c["m"], c["K"], temperature=c["td"])
    # one rank's share; the copies stand where a rank's all-gathers write its own records
    mode, td, tt, r = aal.AAL_VP_WTV, c["td"], c["tt"], c["rank"]
    parts_all, acc_all = state["parts_all"], state["acc_all"]
    parts_all[r].copy_(aal.aal_vp_row_partials(zd, zt, state["v0"], mode, td, tt, V_total=c["V"]))
    row = aal.aal_vp_merge_rows(parts_all, mode, td, tt)
    acc_all[r].copy_(aal.aal_vp_accept_partials(zd, zt, row, td, tt))
    out = aal.aal_vp_window_scan(row, acc_all, c["N"], c["K"], mode, td)
    out["grad"] = aal.aal_vp_grad(zd, zt, row, state["v0"], mode, td, tt)
    return out


def work(case):
    c = case
    rows, V, s = math.prod(_shape(c)[:-1]), c["V"], BYTES[c["dtype"]]
    if c["op"] == "vp":
        v0, v1 = _slice(c)
        V = v1 - v0
    sg = 0 if c["op"] == "sim" or not c.get("grad", True) else BYTES[c.get("grad_dtype", c["dtype"])]
    reads = 3 if c["op"] == "grpo" else 2
    # per entry of a row: the exponentials and a multiply-add or two for each tensor and direction
    return {"bytes": float(rows * (V * (reads * s + sg) + 16)), "flops": float(rows * V * 12)}


def tolerance(case):
    c = case
    # Gradients in bf16 round to 2^-9 of each entry (a relative error of about 2e-3 against 64 bits);
    # entries of the window-TV gradient whose q and p agree to rounding may take either side of
    # the subgradient (an entry then changes by its whole size, hence "max").
    out16 = c["op"] != "sim" and c.get("grad", True) and c.get("grad_dtype", c["dtype"]) == "bf16"
    t = {"rel": 6e-3 if out16 else 1e-5}
    if c["op"] in ("wtv", "vp", "loss"):
        t["max"] = 0.9
    if c["op"] == "sim":
        # a draw within rounding of a boundary of the cumulative distribution may take its neighbour
        t.update(rel=2e-2, max=0.99, differ=2e-3)
    if c["op"] == "grpo":
        t["rel"] = max(t["rel"], 1e-4)  # the loss is a sum of terms of both signs
    return t


# ------------------------------------------------------------------ 64 bits
def _chunks(rows, V):
    n = max(1, (1 << 27) // V)
    return [(r, min(rows, r + n)) for r in range(0, rows, n)]


def _first_max(z):
    V = z.shape[-1]
    i = torch.arange(V, device=z.device).expand_as(z)
    return torch.where(z == z.amax(-1, keepdim=True), i, V).amin(-1)


def _window_parts(a):
    """E and dE/da of windows a [..., K] (64 bits)."""
    K = a.shape[-1]
    pre = torch.ones_like(a)
    suf = torch.ones_like(a)
    for k in range(1, K):
        pre[..., k] = pre[..., k - 1] * a[..., k - 1]
        suf[..., K - 1 - k] = 1 + a[..., K - k] * suf[..., K - k]
    return (pre * a).sum(-1), pre * suf


def _row_windows(a, c):
    """E per window and dE/da summed per row, for a in the case's layout."""
    K = c["K"]
    if c["op"] != "loss" or not c["sequences"]:
        return _window_parts(a)
    W = a.shape[1] - K + 1
    E, dw = _window_parts(a.unfold(1, K, 1).contiguous())
    d = torch.zeros_like(a)
    for k in range(K):
        d[:, k:k + W] += dw[..., k]
    return E, d


def _exact_losses(c, zd, zt, labels=None):
    """EAL, WTV, the weighted objectives and the vocabulary-parallel share."""
    shape = zd.shape[:-1]
    V = zd.shape[-1]
    rows = math.prod(shape)
    zd, zt = zd.view(rows, V), zt.view(rows, V)
    td, tt = c["td"], c.get("tt", 1.0)
    if c["op"] == "loss":
        w_wtv, w_eal, w_kl, w_tv = WEIGHTS[c["weights"]]
    else:
        w_wtv, w_eal, w_kl, w_tv = (0.0, 1.0, 0.0, 0.0) if c["op"] == "eal" else (1.0, 0.0, 0.0, 0.0)
    want_p = bool(w_wtv or w_kl or w_tv)
    dev = zd.device
    new = lambda: torch.zeros(rows, dtype=torch.float64, device=dev)  # noqa: E731
    a_tv, qlt, a_eal, kl = new(), new(), new(), new()
    xs = torch.full((rows,), -1, dtype=torch.int64, device=dev)
    for r0, r1 in _chunks(rows, V):
        lq = torch.log_softmax(zd[r0:r1].double() / td, -1)
        if w_eal:
            xs[r0:r1] = _first_max(zt[r0:r1]) if labels is None else labels[r0:r1].long()
            a_eal[r0:r1] = lq.gather(1, xs[r0:r1, None]).squeeze(1).exp()
        if want_p:
            lp = torch.log_softmax(zt[r0:r1].double() / tt, -1)
            q, p = lq.exp(), lp.exp()
            a_tv[r0:r1] = torch.minimum(p, q).sum(-1)
            qlt[r0:r1] = (q * (q < p)).sum(-1)
            if w_kl:
                kl[r0:r1] = (p * (lp - lq)).sum(-1)
    f = lambda t: t.view(shape)  # noqa: E731
    E_tv, d_tv = _row_windows(f(a_tv), c)
    E_eal, d_eal = _row_windows(f(a_eal), c)
    W = E_tv.numel()
    count = torch.zeros(shape, dtype=torch.float64, device=dev)
    if c["op"] == "loss" and c["sequences"]:
        for k in range(c["K"]):
            count[:, k:k + shape[1] - c["K"] + 1] += 1
    else:
        count += 1
    terms = [-E_tv.mean() if w_wtv else 0.0, -E_eal.mean() if w_eal else 0.0, kl.mean() if w_kl else 0.0,
             (count * (1 - f(a_tv))).sum() / (W * c["K"]) if w_tv else 0.0]
    loss = sum(w * t for w, t in zip((w_wtv, w_eal, w_kl, w_tv), terms))
    grad = None
    if c.get("grad", True):
        cut = _slice(c) if c["op"] == "vp" else (0, V)
        grad = torch.empty(rows, cut[1] - cut[0], dtype=torch.float64, device=dev)
        g_tv = ((-w_wtv * d_tv - w_tv * count / c["K"]) / W).reshape(rows)
        g_eal = (-w_eal * d_eal / W).reshape(rows) * a_eal
        for r0, r1 in _chunks(rows, V):
            q = torch.softmax(zd[r0:r1].double() / td, -1)
            g = -g_eal[r0:r1, None] * q
            if w_eal:
                g.scatter_add_(1, xs[r0:r1, None], g_eal[r0:r1, None])
            if want_p:
                p = torch.softmax(zt[r0:r1].double() / tt, -1)
                g += g_tv[r0:r1, None] * q * ((q < p).double() - qlt[r0:r1, None])
                if w_kl:
                    g += w_kl / rows * (q - p)
            grad[r0:r1] = g[:, cut[0]:cut[1]] / td
    loss = torch.as_tensor(loss, dtype=torch.float64).reshape(1)
    if c["op"] == "loss":
        flat = lambda t: t.reshape(-1)  # noqa: E731
        tv = want_p and c.get("outputs", True)
        w_eal = w_eal and c.get("outputs", True)
        return {"loss": loss, "terms": torch.tensor([float(t) for t in terms], dtype=torch.float64),
                "E_tv": flat(E_tv) if tv else None, "E_eal": flat(E_eal) if w_eal else None,
                "accept_tv": a_tv if tv else None, "accept_eal": a_eal if w_eal else None,
                "xstar": xs.int() if c.get("outputs", True) else None,
                "grad": None if grad is None else grad.view(*shape, V)}
    out = {"loss": loss, "E": E_eal if c["op"] == "eal" else E_tv, "accept": f(a_eal if c["op"] == "eal" else a_tv)}
    if c["op"] == "eal":
        out["xstar"] = f(xs).int()
    if c["op"] == "vp":
        out["grad"] = grad
    else:
        out["grad"] = None if grad is None else grad.view(*shape, V)
    return out


def _exact_sim(c, zd, zt, u1, u2):
    P, G, K, V = zd.shape
    rows = P * G * K
    zd, zt, u1, u2 = zd.view(rows, V), zt.view(rows, V), u1.view(rows).double(), u2.view(rows).double()
    tok = torch.empty(rows, dtype=torch.int64, device=zd.device)
    acc = torch.empty(rows, dtype=torch.int32, device=zd.device)
    for r0, r1 in _chunks(rows, V):
        q = torch.softmax(zd[r0:r1].double() / c["td"], -1)
        p = torch.softmax(zt[r0:r1].double() / c["td"], -1)
        cum = q.cumsum(-1)
        x = (cum <= u1[r0:r1, None] * cum[:, -1:]).sum(-1).clamp_(max=V - 1)
        tok[r0:r1] = x
        qx, px = q.gather(1, x[:, None]).squeeze(1), p.gather(1, x[:, None]).squeeze(1)
        acc[r0:r1] = (u2[r0:r1] * qx < px).int()
    acc = acc.view(P, G, K)
    reward = acc.cumprod(-1).sum(-1)
    r = reward.double()
    adv = (r - r.mean(-1, keepdim=True)) / (r.std(-1, unbiased=False, keepdim=True) + 1e-6)
    return {"token": tok.view(P, G, K).int(), "accept": acc, "reward": reward.int(), "advantage": adv}


def _exact_grpo(c, zd, zref, zt):
    B, S, V = zd.shape
    m, K, T = c["m"], c["K"], c["td"]
    rows = B * S
    th, rf, tg = zd.view(rows, V), zref.view(rows, V), zt.view(rows, V)
    sth, srf, xs = (torch.empty(rows, dtype=torch.int64, device=zd.device) for _ in range(3))
    diff = torch.empty(rows, dtype=torch.float64, device=zd.device)
    for r0, r1 in _chunks(rows, V):
        sth[r0:r1], srf[r0:r1], xs[r0:r1] = (_first_max(z[r0:r1]) for z in (th, rf, tg))
        at = sth[r0:r1, None]
        diff[r0:r1] = (torch.log_softmax(th[r0:r1].double() / T, -1).gather(1, at) -
                       torch.log_softmax(rf[r0:r1].double() / T, -1).gather(1, at)).squeeze(1)
    w = lambda t: t.view(B, m, K)  # noqa: E731
    tau_th = w((sth == xs).int()).cumprod(-1).sum(-1)
    tau_rf = w((srf == xs).int()).cumprod(-1).sum(-1)
    R = (tau_th - tau_rf).double()
    A = (R - R.mean(-1, keepdim=True)) / (R.std(-1, unbiased=False, keepdim=True) + 1e-6)
    raw = w(diff).mean(-1)
    log_rho = raw.clamp(-10, 10)
    rho = log_rho.exp()
    s1, s2 = rho * A, rho.clamp(0.8, 1.2) * A
    loss = -torch.minimum(s1, s2).mean()
    inside = ((rho > 0.8) & (rho < 1.2)).double()
    d = torch.where(s1 <= s2, A, A * inside) * rho * ((raw > -10) & (raw < 10))
    coef = (-d / (B * m) / K / T).unsqueeze(-1).expand(B, m, K).reshape(rows)
    grad = torch.empty(rows, V, dtype=torch.float64, device=zd.device)
    for r0, r1 in _chunks(rows, V):
        g = -torch.softmax(th[r0:r1].double() / T, -1)
        g.scatter_add_(1, sth[r0:r1, None], torch.ones(r1 - r0, 1, dtype=torch.float64, device=zd.device))
        grad[r0:r1] = coef[r0:r1, None] * g
    return {"loss": loss.reshape(1), "tau_theta": tau_th.int(), "tau_ref": tau_rf.int(), "advantage": A,
            "log_rho": log_rho, "grad": grad.view(B, S, V)}


def exact(case, seed):
    c = case
    zd, zt = _logits(c, seed)
    if c["op"] == "sim":
        return _exact_sim(c, zd, zt, *make_uniforms(_shape(c)[:3], seed))
    if c["op"] == "grpo":
        return _exact_grpo(c, zd, _reference(zd, seed), zt)
    return _exact_losses(c, zd, zt, _labels(zt, seed) if c.get("labels") else None)
