"""The calls whose speed matters, over the ranges they are made in.

Each case is one pass of the verify/defer step (or of the drafter's sampling
step, or of a whole decoding round) through the Python binding, with seeded
synthetic logits in the shapes of the repository's workloads: a Zipf-ranked
verifier with N(0, 1) noise and a drafter that mostly agrees with it.

Fields of a case: ``op`` (verify, greedy, mix, draft, round), ``B`` sequences,
``gamma`` drafted positions, ``V`` vocabulary, ``dtype``, ``rule`` / ``alpha``
/ ``T`` (mix draws them per sequence), ``stats`` (row statistics and the
sampled mass are returned too, as a program that logs or tunes the deferral
asks for them).
"""
import math

import torch

from paper_2405_19261_amd import spc

CHOW, DIFF, OPT, ALWAYS = 0, 1, 2, 3
TOKEN_V1, TOKEN_V2, TOKEN_V3 = 5, 6, 7
LOSSY, BILD, CHOWLOG, DIFFLOG, OPTLOG = 8, 9, 10, 11, 12
TOKEN_RULES = (TOKEN_V1, TOKEN_V2, TOKEN_V3)
# a rule with an alpha that makes it defer on some rows and not on others
RULE_ALPHA = ((CHOW, 0.4), (DIFF, 0.05), (OPT, 0.1), (ALWAYS, 0.0), (TOKEN_V1, 0.05),
              (TOKEN_V2, 0.05), (TOKEN_V3, 0.3), (LOSSY, 0.2), (BILD, 8.0), (CHOWLOG, 5.0),
              (DIFFLOG, 0.3), (OPTLOG, 0.5))
MIX = ((CHOW, 0.4), (DIFF, 0.05), (OPT, 0.1))
MIX_T = (0.5, 0.7, 1.0)


def _case(name, op, B, gamma, V, dtype, rule=DIFF, alpha=0.05, T=1.0, stats=False):
    return dict(name=name, op=op, B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=alpha,
                T=T, stats=stats)


def listed():
    return [
        # the smallest call: one short-vocabulary sequence, nothing but latency
        _case("tiny_chow_f32", "verify", 1, 4, 1000, "f32", CHOW, 0.5),
        # a T5-sized vocabulary in float32 under the paper's OPT rule
        _case("t5_opt_f32", "verify", 8, 5, 32128, "f32", OPT, 0.1),
        # one interactive sequence at the Gemma vocabulary
        _case("one_diff_bf16", "verify", 1, 7, 256000, "bf16", DIFF, 0.05),
        # the benchmark step: a serving batch at the Gemma vocabulary
        _case("gemma_diff_bf16", "verify", 32, 7, 256000, "bf16", DIFF, 0.05),
        # the same with the deferral statistics logged, under OPT (D_TV of every row)
        _case("gemma_opt_stats_bf16", "verify", 16, 7, 256000, "bf16", OPT, 0.1, stats=True),
        # a token-specific target (Alg. 6)
        _case("gemma_token_bf16", "verify", 32, 7, 256000, "bf16", TOKEN_V2, 0.05),
        # an entropy rule on float32 logits, its statistic logged
        _case("difflog_f32", "verify", 16, 4, 128000, "f32", DIFFLOG, 0.3, T=0.7, stats=True),
        # a vocabulary whose rows start anywhere (no padding to a vector)
        _case("odd_diff_bf16", "verify", 24, 5, 100003, "bf16", DIFF, 0.05),
        # temperature 0, a large batch
        _case("gemma_greedy_bf16", "greedy", 128, 4, 256000, "bf16", OPT, 0.1, T=0.0),
        # a large batch of requests with their own rules and temperatures
        _case("stress_mix_bf16", "mix", 256, 8, 256000, "bf16"),
        # the drafter's step
        _case("draft_bf16", "draft", 32, 1, 256000, "bf16"),
        # a decoding round: gamma drafter steps, then the verification
        _case("round_lossy_bf16", "round", 8, 4, 32128, "bf16", LOSSY, 0.2, T=0.7),
    ]


def draw(rng):
    op = rng.choice(("verify",) * 6 + ("greedy", "mix", "draft", "round"))
    dtype = rng.choice(("bf16", "bf16", "f32"))
    V = int(round(math.exp(rng.uniform(math.log(1000), math.log(256000)))))
    step = rng.choice((1, 8, 128, 128))
    V = max(1000, min(256000, V // step * step))
    if step == 1:
        V |= 1
    gamma = 1 if op == "draft" else rng.randint(1, 8)
    most = 3.0e8 if step == 1 else 1.0e9  # bytes of logits
    rows = most / (2 * V * (2 if dtype == "bf16" else 4))
    top = max(1, min(256, int(rows / (gamma + 1))))
    B = int(round(math.exp(rng.uniform(0.0, math.log(top)))))
    rule, alpha = rng.choice(RULE_ALPHA)
    T = rng.choice((0.7, 1.0, 1.0))
    stats = op in ("verify", "mix") and rng.random() < 0.35
    if op == "greedy":
        rule, alpha, T = OPT, 0.1, 0.0
    if op == "mix":
        rule, alpha, T = DIFF, 0.05, 1.0
    c = _case("", op, B, gamma, V, dtype, rule, alpha, T, stats)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _logits(c, seed):
    """Verifier and drafter logits [B][gamma+1][V] in the case's type, and a generator."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(int(seed) % (1 << 62))
    B, g1, V = c["B"], (1 if c["op"] == "draft" else c["gamma"] + 1), c["V"]
    R = B * g1
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    q = torch.empty((R, V), device=dev, dtype=dt)
    p = torch.empty((R, V), device=dev, dtype=dt)

    def normal(n, s=1.0):
        return torch.randn((n, V), generator=g, device=dev) * s

    noisy = torch.rand(R, generator=g, device=dev) < 0.10
    # mix: a quarter of the sequences have a drafter equal to the verifier, a
    # quarter one unrelated to it
    part = torch.rand(B, generator=g, device=dev).repeat_interleave(g1)
    chunk = max(1, min(R, (1 << 27) // V))
    for r0 in range(0, R, chunk):
        n = min(R, r0 + chunk) - r0
        rank = torch.rand((n, V), generator=g, device=dev).mul_(V).floor_().add_(1.0)
        zp = rank.log_().mul_(-1.2).add_(normal(n))
        zq = zp.mul(0.8).add_(normal(n))
        zq += normal(n, math.sqrt(3.0)) * noisy[r0:r0 + n, None]
        if c["op"] == "mix":
            m = part[r0:r0 + n, None]
            zq = torch.where(m < 0.25, zp, torch.where(m < 0.5, normal(n, 2.0), zq))
        p[r0:r0 + n] = zp.to(dt)
        q[r0:r0 + n] = zq.to(dt)
    return q.view(B, g1, V), p.view(B, g1, V), g


def _drafts(q, T, gamma, g):
    """x ~ softmax(q / T) for the first gamma rows of each sequence (argmax at T = 0)."""
    B, _, V = q.shape
    out = torch.empty((B, gamma), dtype=torch.int32, device=q.device)
    for j in range(gamma):
        for b0 in range(0, B, 64):
            z = q[b0:b0 + 64, j].float()
            t = T[b0:b0 + 64, None]
            if float(T[b0]) == 0.0:
                x = z.argmax(-1)
            else:
                x = torch.multinomial(torch.softmax(z / t, -1), 1, generator=g)[:, 0]
            out[b0:b0 + 64, j] = x.to(torch.int32)
    return out


def prepare(case, seed):
    c = case
    B, gamma, V = c["B"], c["gamma"], c["V"]
    q, p, g = _logits(c, seed)
    dev = q.device
    s = dict(case=c, q=q, p=p)
    if c["op"] == "draft":
        s["rows"] = q.view(B, V)
        s["u"] = torch.rand(B, generator=g, device=dev)
        s["out"] = torch.empty(B, dtype=torch.int32, device=dev)
        del s["p"]
        return s
    T = torch.full((B,), float(c["T"]), device=dev)
    if c["op"] == "mix":
        pick = torch.randint(0, len(MIX), (B,), generator=g, device=dev)
        s["rule_ps"] = torch.tensor([r for r, _ in MIX], dtype=torch.int32, device=dev)[pick]
        s["alpha_ps"] = torch.tensor([a for _, a in MIX], device=dev)[pick]
        T = torch.tensor(MIX_T, device=dev)[
            torch.randint(0, len(MIX_T), (B,), generator=g, device=dev)]
        s["temp_ps"] = T
    s["u"] = torch.rand((B, gamma + 1), generator=g, device=dev)
    # a step's integers live in one record, which a serving loop brings to the
    # host in one copy: draft tokens [B][gamma], accept lengths [B], next tokens [B]
    rec = torch.zeros(B * (gamma + 2), dtype=torch.int32, device=dev)
    s["record"] = rec
    s["draft"] = rec[:B * gamma].view(B, gamma)
    s["defer"] = torch.zeros((B, gamma + 1), dtype=torch.uint8, device=dev)
    s["out"] = (rec[B * gamma:B * (gamma + 1)], rec[B * (gamma + 1):], s["defer"])
    if c["op"] == "round":
        s["q_rows"] = [q[:, j].contiguous() for j in range(gamma)]
        s["u_draft"] = torch.rand((gamma, B), generator=g, device=dev)
    else:
        s["draft"].copy_(_drafts(q, T, gamma, g))
    if c["stats"]:
        s["row_stats"] = torch.zeros((B, gamma + 1, 8), device=dev)
        s["norm"] = torch.zeros(B, device=dev)
    return s


# ------------------------------------------------------------------ the pass
def run(s):
    c = s["case"]
    op = c["op"]
    if op == "draft":
        return {"token": spc.spc_draft_sample(s["rows"], c["T"], uniforms=s["u"], out=s["out"])}
    if op == "greedy":
        spc.spc_greedy_verify(s["q"], s["p"], s["draft"], c["rule"], c["alpha"], out=s["out"])
        return {"record": s["record"], "defer": s["defer"]}
    if op == "round":
        for j, z in enumerate(s["q_rows"]):
            s["draft"][:, j] = spc.spc_draft_sample(z, c["T"], uniforms=s["u_draft"][j])
    if op == "mix" or c["stats"]:
        kw = {}
        if op == "mix":
            kw.update(rule_per_seq=s["rule_ps"], alpha_per_seq=s["alpha_ps"],
                      temp_per_seq=s["temp_ps"],
                      rules_present=sum(1 << r for r, _ in MIX))
        if c["stats"]:
            kw.update(out_row_stats=s["row_stats"], out_sample_norm=s["norm"])
        spc.spc_verify_ex(s["q"], s["p"], s["draft"], s["u"], c["rule"], c["alpha"], c["T"],
                          out=s["out"], **kw)
    else:
        spc.spc_verify(s["q"], s["p"], s["draft"], s["u"], c["rule"], c["alpha"], c["T"],
                       out=s["out"])
    r = {"record": s["record"], "defer": s["defer"]}
    if c["stats"]:
        r.update(row_stats=s["row_stats"], norm=s["norm"])
    return r


def work(case):
    c = case
    eb = 4 if c["dtype"] == "f32" else 2
    B, gamma, V = c["B"], c["gamma"], c["V"]
    if c["op"] == "draft":
        return {"bytes": B * V * eb + 8 * B, "flops": 4 * B * V}
    g1 = gamma + 1
    n = B * g1 * V
    ints = 4 * B * gamma + 4 * B * g1 + 8 * B + B * g1
    w = {"bytes": 2 * n * eb + ints + (4 * B * g1 * 8 + 4 * B if c["stats"] else 0),
         "flops": 8 * n}  # per logit: scale, maximum, exponential, sum
    if c["op"] == "round":
        w["bytes"] += B * gamma * V * eb
        w["flops"] += 4 * B * gamma * V
    return w


def tolerance(case):
    # Statistics come from float32 exponentials summed in float64 and are
    # stored in float32.  An inverse-CDF draw whose uniform lies within
    # rounding of a boundary (about 1e-8 of the mass, against up to 256000
    # boundaries) may land on the neighbouring token.
    # (measured against float64: row statistics 4e-8, the sampled mass 5e-8 to 2e-7)
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}


# ------------------------------------------------------------------ 64 bits
def _rows64(z, T):
    """log-probabilities [n, V] of rows z [n, V] at temperatures T [n], maxima and lse."""
    s = z.double() / T[:, None]
    m = s.max(-1).values
    lse = torch.logsumexp(s, -1)
    return s - lse[:, None], m, lse


def _draw64(w, u):
    """(smallest k with C_k > u W, W) for weights w [V]."""
    C = w.cumsum(0)
    t = u.double() * C[-1]
    k = int(torch.searchsorted(C, t.reshape(1), right=True)[0])
    return min(k, int(w.nonzero()[-1])), float(C[-1])


def _exact_draft(rows, T, u):
    out = torch.empty(rows.shape[0], dtype=torch.int32, device=rows.device)
    for b in range(rows.shape[0]):
        lp, _, _ = _rows64(rows[b:b + 1], torch.full((1,), float(T), device=rows.device).double())
        out[b], _ = _draw64(lp[0].exp(), u[b])
    return out


def exact(case, seed):
    """What run() returns, in float64 torch: the step of Alg. 4 / Alg. 6 row by row."""
    c = case
    B, gamma, V = c["B"], c["gamma"], c["V"]
    if B * (gamma + 1) > 600:  # integers only there, or too long
        return None
    s = prepare(case, seed)
    if c["op"] == "draft":
        return {"token": _exact_draft(s["rows"], c["T"], s["u"])}
    if c["op"] == "round":
        for j in range(gamma):
            s["draft"][:, j] = _exact_draft(s["q_rows"][j], c["T"], s["u_draft"][j])
    dev, g1 = s["q"].device, gamma + 1
    stats = torch.zeros((B, g1, 8), dtype=torch.float64, device=dev)
    norm = torch.zeros(B, dtype=torch.float64, device=dev)
    acc, nxt = s["out"][0], s["out"][1]
    for b in range(B):
        rule = int(s["rule_ps"][b]) if c["op"] == "mix" else c["rule"]
        alpha = float(s["alpha_ps"][b]) if c["op"] == "mix" else float(
            torch.tensor(c["alpha"], dtype=torch.float32))
        T = float(s["temp_ps"][b]) if c["op"] == "mix" else float(
            torch.tensor(c["T"], dtype=torch.float32))
        greedy = T == 0.0
        t = torch.full((g1,), 1.0 if greedy else T, device=dev, dtype=torch.float64)
        lq, mq, zq = _rows64(s["q"][b], t)
        lp, mp, zp = _rows64(s["p"][b], t)
        Q, P = lq.exp(), lp.exp()
        xq, xp = Q.max(-1).values, P.max(-1).values
        aq, ap = s["q"][b].float().argmax(-1), s["p"][b].float().argmax(-1)
        tv = torch.zeros(g1, dtype=torch.float64, device=dev)
        log = torch.zeros_like(tv)
        if rule in (OPT, OPTLOG):
            tv = (aq != ap).double() if greedy else (P - Q).clamp(min=0).sum(-1)
        if rule == BILD:
            log = -(Q * lp).sum(-1)
        if rule == CHOWLOG:
            log = -(Q * lq).sum(-1)
        if rule in (DIFFLOG, OPTLOG):
            log = -(Q * lq).sum(-1) + (P * lp).sum(-1)
        R = None
        if rule in TOKEN_RULES:
            th = xp * (1 - alpha) if rule == TOKEN_V3 else xp - alpha
            R = (Q if rule == TOKEN_V1 else P) < th[:, None]
            tv = (Q * R).sum(-1)
            delta = torch.zeros(g1, dtype=torch.bool, device=dev)
        elif rule == CHOW:
            delta = xq < 1 - alpha
        elif rule in (DIFF, OPT):
            delta = xq < xp - alpha * (tv if rule == OPT else 1.0)
        elif rule == ALWAYS:
            delta = torch.ones(g1, dtype=torch.bool, device=dev)
        elif rule == LOSSY:
            delta = torch.zeros(g1, dtype=torch.bool, device=dev)
        else:
            delta = log > alpha * (tv if rule == OPTLOG else 1.0)
        f = gamma
        for j in range(gamma):
            x = int(s["draft"][b, j])
            if R is not None:
                delta[j] = R[j, x]
                pi = P[j, x] * tv[j] + (0 if R[j, x] else Q[j, x])
            elif rule == LOSSY:
                pi = P[j, x] / (1 - alpha)
            else:
                pi = P[j, x] if delta[j] else Q[j, x]
            if greedy:
                keep = x == int(ap[j] if delta[j] else aq[j])
            else:
                keep = bool(s["u"][b, j].double() < (pi / Q[j, x]).clamp(max=1.0))
            if not keep and f == gamma:
                f = j
        acc[b] = f
        s["defer"][b] = delta.to(torch.uint8)
        if greedy:
            nxt[b] = (ap if delta[f] else aq)[f]
            continue
        if R is not None:
            pi = torch.where(R[f], P[f] * tv[f], Q[f] + P[f] * tv[f])
            w = (pi - Q[f]).clamp(min=0) if f < gamma else pi
        elif f < gamma:
            w = (P[f] - Q[f]).clamp(min=0)
        else:
            w = P[f] if (rule == LOSSY or delta[f]) else Q[f]
        nxt[b], norm[b] = _draw64(w, s["u"][b, gamma])
        stats[b] = torch.stack([mq, zq, xq, mp, zp, xp, tv, log], -1)
    r = {"record": s["record"], "defer": s["defer"]}
    if c["stats"]:
        r.update(row_stats=stats, norm=norm)
    return r
