"""The work that a training program has this library do, as timed and checked cases.

Four kinds, one per public call:

  advantage  curation of the rollout groups of a micro-batch or of a whole step
  logprob    log-prob / entropy / lse of stored logits (scoring a rollout, a reference policy)
  loss       clipped loss and dlogits of stored logits, statistics formed inside the call
             (``lse`` 0) or by a forward call before it (``lse`` 1)
  fused      the same with the LM head fused in: forward only, or with dhidden and dweight

A token case has Q groups of N rollouts; 35 % of the groups have all-equal rewards and carry no
gradient.  ``padded`` cases right-pad every rollout to T / (Q N) rows (9/16 of them valid on
average), the others lay the rollouts end to end.
"""
import math

import numpy as np
import torch

import paper_2602_14338_amd as aero
from paper_2602_14338_amd import binding

EPS = 0.2
ZERO_FRAC = 0.35
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn}
_BYTES = {"f32": 4, "bf16": 2, "f16": 2, "f8": 1}
_CHUNK = 1 << 28   # logits handled at a time outside the timed pass


def listed():
    return [
        # curation of one micro-batch: 8 queries of 8 rollouts, the smallest call of a step
        dict(name="advantage_microbatch", kind="advantage", Q=8, n_lo=8, n_hi=8),
        # curation of a whole step: 256 queries, 8 to 32 rollouts each as the two-stage allocation leaves them
        dict(name="advantage_step", kind="advantage", Q=256, n_lo=8, n_hi=32),
        # a short scoring call on an odd vocabulary whose rows are not 16-byte aligned
        dict(name="logprob_odd_vocab", kind="logprob", dtype="bf16", T=500, V=50257, ld=50257, Q=4, N=8, padded=0,
             entropy=0),
        # old log-probs of a rollout batch, right-padded to 1024 slots
        dict(name="logprob_rollout", kind="logprob", dtype="bf16", T=16384, V=151936, ld=151936, Q=2, N=8, padded=1,
             entropy=1),
        # a small model in single precision: 4 queries x 8 rollouts x 64 tokens
        dict(name="loss_f32_small", kind="loss", dtype="f32", T=2048, V=1024, ld=1024, Q=4, N=8, padded=0, lse=0,
             stats=1, entropy_coef=0.0, kl_coef=0.0),
        # the training micro-batch of the logits path: right-padded, statistics logged
        dict(name="loss_bf16_padded", kind="loss", dtype="bf16", T=16384, V=151936, ld=151936, Q=2, N=8, padded=1,
             lse=0, stats=1, entropy_coef=0.0, kl_coef=0.0),
        # half-precision logits with both optional terms of the loss
        dict(name="loss_f16_terms", kind="loss", dtype="f16", T=4096, V=151936, ld=151936, Q=8, N=8, padded=0, lse=0,
             stats=0, entropy_coef=1e-3, kl_coef=1e-2),
        # forward call (log-probs logged), then the loss call on its lse: a 32K vocabulary, packed
        dict(name="loss_two_calls", kind="loss", dtype="bf16", T=8192, V=32000, ld=32000, Q=16, N=8, padded=0, lse=1,
             stats=0, entropy_coef=0.0, kl_coef=0.0),
        # log-probs of a reference policy straight from hidden states, odd token count
        dict(name="fused_logprob", kind="fused", T=4001, H=1536, V=151936, Q=4, N=8, padded=0, bwd=0, dweight="f32"),
        # one small micro-batch through the fused head: a few hundred tokens against the whole vocabulary
        dict(name="fused_small", kind="fused", T=600, H=1536, V=151936, Q=2, N=8, padded=0, bwd=1, dweight="bf16"),
        # 1.5B-sized head, 16K packed tokens
        dict(name="fused_16k_h1536", kind="fused", T=16384, H=1536, V=151936, Q=8, N=8, padded=0, bwd=1,
             dweight="f32"),
        # 7B-sized head, 32K packed tokens
        dict(name="fused_32k_h3584", kind="fused", T=32768, H=3584, V=152064, Q=128, N=10, padded=0, bwd=1,
             dweight="f32"),
    ]


def _grad_scale(case):
    """Gradients of the narrow-range types are lifted into it; a token's weight is about 1 / T."""
    lift = {"f16": 256, "f8": 8}.get(case["dtype"])
    return 2.0 ** math.floor(math.log2(lift * case["T"])) if lift else 1.0


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["advantage", "logprob", "loss", "loss", "loss", "fused", "fused"])
    if kind == "advantage":
        lo = rng.randint(2, 16)
        return dict(kind=kind, Q=_log_int(rng, 4, 1024), n_lo=lo, n_hi=lo + rng.randint(0, 24))
    Q, N = rng.randint(2, 16), rng.randint(4, 12)
    padded = rng.randint(0, 1)
    if kind == "fused":
        T = _log_int(rng, 100, 16384)
        H = 8 * _log_int(rng, 16, 448) if rng.random() < 0.5 else rng.choice([896, 1536, 2048, 3584])
        V = _log_int(rng, 4000, 152064) if rng.random() < 0.5 else rng.choice([32000, 151936, 152064])
        case = dict(kind=kind, T=T, H=H, V=V, Q=Q, N=N, padded=padded, bwd=int(rng.random() < 0.7),
                    dweight=rng.choice(["f32", "bf16"]))
    else:
        V = _log_int(rng, 1000, 262144) if rng.random() < 0.6 else rng.choice([32000, 151936, 152064, 262144])
        ld = V if rng.random() < 0.5 else (V + 63) // 64 * 64
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32", "f8"])
        T = _log_int(rng, 64, max(65, min(32768, 1200000000 // V)))
        case = dict(kind=kind, dtype=dtype, T=T, V=V, ld=ld, Q=Q, N=N, padded=padded)
        if kind == "logprob":
            case["entropy"] = rng.randint(0, 1)
        else:
            terms = rng.random() < 0.3
            case.update(lse=int(rng.random() < 0.3), stats=rng.randint(0, 1), entropy_coef=1e-3 if terms else 0.0,
                        kl_coef=1e-2 if terms and rng.random() < 0.5 else 0.0)
            if case["lse"]:
                case["stats"] = 0
    if padded:   # whole slots
        case["T"] = max(1, case["T"] // (Q * N)) * Q * N
    return case


# ---------------------------------------------------------------------------------- inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + stream)
    return g


def _rewards(rng, sizes):
    zero = rng.permutation(len(sizes))[:int(round(ZERO_FRAC * len(sizes)))]
    out = []
    for q, n in enumerate(sizes):
        r = np.zeros(n, np.float32)
        if q in zero or n < 2:
            r[:] = float(rng.random() < 0.5)
        else:
            r[rng.permutation(n)[:int(rng.integers(1, n))]] = 1.0
        out.append(r)
    return np.concatenate(out)


def _advantage_inputs(case, seed):
    rng = np.random.default_rng([seed, 1])
    # evenly spread sizes in a drawn order: the number of rollouts depends on the case alone
    sizes = rng.permutation(np.rint(np.linspace(case["n_lo"], case["n_hi"], case["Q"])).astype(np.int64))
    R = int(sizes.sum())
    return dict(offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32), rewards=_rewards(rng, sizes),
                lengths=rng.integers(128, 2049, size=R).astype(np.int32),
                keys=rng.integers(0, 2 ** 32, size=R, dtype=np.uint32))


def _token_structure(case, seed):
    """Owner of every token row (-1: padding), advantage and weight of every rollout (Eq. 1, Eq. 2)."""
    rng = np.random.default_rng([seed, 2])
    Q, N, T = case["Q"], case["N"], case["T"]
    R = Q * N
    u = rng.uniform(0.125, 1.0, size=R)
    if case["padded"]:
        slots = T // R
        lengths = np.maximum(1, np.rint(u * slots)).astype(np.int64)
        owner = np.where(np.arange(slots)[None, :] < lengths[:, None], np.arange(R)[:, None], -1).reshape(-1)
    else:   # the last rollouts are cut at T rows, their recorded length stays the full one
        lengths = np.maximum(1, np.rint(u * (1.1 * T / u.sum()))).astype(np.int64)
        owner = np.repeat(np.arange(R), lengths)[:T]
        owner = np.concatenate([owner, np.full(T - owner.size, -1)])
    r = _rewards(rng, [N] * Q).reshape(Q, N).astype(np.float64)
    sd = r.std(axis=1, keepdims=True)
    adv = np.where(sd > 0, (r - r.mean(axis=1, keepdims=True)) / np.where(sd > 0, sd, 1.0), 0.0).reshape(-1)
    weight = 1.0 / (Q * N * lengths)
    return owner.astype(np.int32), adv.astype(np.float32), weight.astype(np.float32)


def _row_chunks(T, width):
    step = max(1, _CHUNK // width)
    return [(a, min(T, a + step)) for a in range(0, T, step)]


def _old_logprob(cur, seed):
    """Behaviour log-probs: the current ones plus N(0, 0.05^2), the ratio kept clear of the clip edges."""
    g = _gen(seed, 5)
    noise = torch.randn(cur.shape, generator=g, device="cuda", dtype=torch.float64) * 0.05
    for _ in range(4):
        rho = torch.exp(-noise)
        bad = ((rho - (1 - EPS)).abs() < 5e-3) | ((rho - (1 + EPS)).abs() < 5e-3)
        noise = torch.where(bad, torch.randn(cur.shape, generator=g, device="cuda", dtype=torch.float64) * 0.05, noise)
    return (cur + noise).float()


def _inputs(case, seed):
    """Device tensors of a token case; the same for the timed pass and for the 64-bit reference."""
    owner, adv, weight = _token_structure(case, seed)
    T, V = case["T"], case["V"]
    x = dict(owner=torch.from_numpy(owner).cuda(), adv=torch.from_numpy(adv).cuda(),
             weight=torch.from_numpy(weight).cuda())
    valid = x["owner"] >= 0
    cur = torch.zeros(T, dtype=torch.float64, device="cuda")
    if case["kind"] == "fused":
        H = case["H"]
        x["hidden"] = torch.randn(T, H, generator=_gen(seed, 1), device="cuda").bfloat16()
        x["W"] = (torch.randn(V, H, generator=_gen(seed, 2), device="cuda") * 0.02).bfloat16()
        # the head's logits are narrow (about 0.8 at H = 1536): sampled tokens are nearly uniform
        y = torch.randint(0, V, (T,), generator=_gen(seed, 3), device="cuda")
        if case["bwd"]:
            w32 = x["W"].float()
            for a, b in _row_chunks(T, V):
                z = x["hidden"][a:b].float() @ w32.t()
                cur[a:b] = z.gather(1, y[a:b, None])[:, 0].double() - torch.logsumexp(z, 1).double()
    else:
        x["logits"] = torch.empty(T, case["ld"], dtype=_TORCH[case["dtype"]], device="cuda")
        y = torch.empty(T, dtype=torch.int64, device="cuda")
        g, gs = _gen(seed, 1), _gen(seed, 3)
        for a, b in _row_chunks(T, case["ld"]):
            x["logits"][a:b] = (torch.randn(b - a, case["ld"], generator=g, device="cuda") * 3.0).to(x["logits"].dtype)
            z = x["logits"][a:b, :V].float()
            lse = torch.logsumexp(z, 1)
            # tokens sampled from the policy itself
            p = torch.exp(z - lse[:, None])
            u = torch.empty_like(p).exponential_(generator=gs)
            y[a:b] = p.div_(u).argmax(1)
            cur[a:b] = z.gather(1, y[a:b, None])[:, 0].double() - lse.double()
    x["targets"] = torch.where(valid, y, torch.full_like(y, -1)).int()
    x["old"] = torch.where(valid, _old_logprob(cur, seed), torch.zeros((), device="cuda"))
    g = _gen(seed, 6)
    x["ref"] = (cur + torch.randn(T, generator=g, device="cuda", dtype=torch.float64) * 0.1).float()
    return x


def prepare(case, seed):
    f = lambda n: torch.zeros(n, device="cuda")
    if case["kind"] == "advantage":
        x = _advantage_inputs(case, seed)
        Q, R = case["Q"], x["rewards"].size
        d = {k: torch.from_numpy(v.view(np.int32) if v.dtype == np.uint32 else v).cuda() for k, v in x.items()}
        return dict(case=case, x=d, Q=Q, R=R,
                    params=aero.AdvParams(reject_enable=1, posterior_mode=1),
                    out=(f(R), f(R), torch.zeros(R, dtype=torch.uint8, device="cuda"),
                         torch.full((R,), -1, dtype=torch.int32, device="cuda"),
                         torch.zeros(Q + 1, dtype=torch.int32, device="cuda"),
                         torch.zeros(Q, dtype=torch.uint8, device="cuda"),
                         torch.zeros(Q, dtype=torch.uint8, device="cuda")),
                    err=torch.zeros(1, dtype=torch.int32, device="cuda"))
    T, V = case["T"], case["V"]
    x = _inputs(case, seed)
    s = dict(case=case, x=x, R=x["adv"].numel(), err=torch.zeros(1, dtype=torch.int32, device="cuda"),
             logprob=f(T), entropy=f(T), lse=f(T), loss=f(1), clip=f(1))
    if case["kind"] == "loss":
        s["dlogits"] = torch.zeros_like(x["logits"])
        s["ws"] = torch.empty(aero.aero_workspace_bytes(binding.OP_GRPO_LOSS_BWD, T=T, V=V, R=s["R"]),
                              dtype=torch.uint8, device="cuda")
    elif case["kind"] == "fused":
        H = case["H"]
        s["ws"] = torch.empty(aero.aero_workspace_bytes(binding.OP_LMHEAD_FUSED, T=T, V=V, H=H, R=s["R"]),
                              dtype=torch.uint8, device="cuda")
        if case["bwd"]:
            s["dhidden"] = torch.zeros(T, H, dtype=torch.bfloat16, device="cuda")
            s["dweight"] = torch.zeros(V, H, dtype=_TORCH[case["dweight"]], device="cuda")
    return s


# ---------------------------------------------------------------------------------- one pass
def run(s):
    case, x = s["case"], s["x"]
    if case["kind"] == "advantage":
        aero.aero_group_advantage(x["rewards"], x["lengths"], x["offsets"], x["keys"], s["Q"], s["R"], s["params"],
                                  *s["out"], s["err"])
        return s["out"]
    T, V = case["T"], case["V"]
    if case["kind"] == "logprob":
        ent = s["entropy"] if case["entropy"] else None
        aero.aero_logprob_fwd(x["logits"], T, V, case["ld"], x["targets"], None, s["logprob"], ent, s["lse"], s["err"])
        return (s["logprob"], s["lse"]) + ((ent,) if case["entropy"] else ())
    if case["kind"] == "loss":
        terms = case["entropy_coef"] != 0.0
        lse = ent = None
        out = ()
        if case["lse"]:
            lse, ent = s["lse"], s["entropy"] if terms else None
            aero.aero_logprob_fwd(x["logits"], T, V, case["ld"], x["targets"], None, s["logprob"], ent, lse, s["err"])
            out = (s["logprob"], lse)
        stats = case["stats"]
        if stats:
            out = (s["logprob"], s["entropy"], s["lse"])
        aero.aero_grpo_loss_bwd(x["logits"], T, V, case["ld"], x["targets"], lse, x["old"], x["owner"], x["adv"],
                                x["weight"], s["R"], EPS, EPS, _grad_scale(case), s["loss"], s["clip"],
                                s["logprob"] if stats else None, s["dlogits"], s["ws"], s["err"],
                                entropy_out=s["entropy"] if stats else None, lse_out=s["lse"] if stats else None,
                                entropy_coef=case["entropy_coef"], entropy=ent, kl_coef=case["kl_coef"],
                                ref_logprob=x["ref"] if case["kl_coef"] else None)
        return out + (s["loss"], s["clip"], s["dlogits"])
    if not case["bwd"]:
        aero.aero_lmhead_logprob_fused(x["hidden"], x["W"], T, case["H"], V, x["targets"], s["logprob"], s["entropy"],
                                       s["lse"], workspace=s["ws"], err_flag=s["err"])
        return s["logprob"], s["entropy"], s["lse"]
    aero.aero_lmhead_logprob_fused(x["hidden"], x["W"], T, case["H"], V, x["targets"], s["logprob"], s["entropy"],
                                   s["lse"], x["old"], x["owner"], x["adv"], x["weight"], s["R"], EPS, EPS, 1.0,
                                   s["loss"], s["clip"], s["dhidden"], s["dweight"], s["ws"], s["err"])
    return s["logprob"], s["entropy"], s["lse"], s["loss"], s["clip"], s["dhidden"], s["dweight"]


def work(case):
    """Expected counts: valid and gradient-carrying rows vary a little with the seed."""
    if case["kind"] == "advantage":
        R = case["Q"] * (case["n_lo"] + case["n_hi"]) / 2
        return dict(bytes=R * 25 + case["Q"] * 10, flops=R * 20)
    T, V = case["T"], case["V"]
    valid = T * (9 / 16 if case["padded"] else 1.0)
    grad = valid * (1 - round(ZERO_FRAC * case["Q"]) / case["Q"])
    if case["kind"] == "fused":
        H = case["H"]
        b, fl = 2.0 * valid * H + 2.0 * V * H + 16.0 * T, 2.0 * valid * V * H
        if case["bwd"]:   # dhidden, dweight and the two contractions that form them
            b += 2.0 * T * H + (4.0 if case["dweight"] == "f32" else 2.0) * V * H
            fl += 4.0 * grad * V * H
        return dict(bytes=b, flops=fl)
    e = _BYTES[case["dtype"]]
    if case["kind"] == "logprob":
        return dict(bytes=valid * V * e + 16.0 * T, flops=5.0 * valid * V)
    every = case["stats"] or case["lse"] or case["entropy_coef"] != 0.0   # rows whose statistics are wanted
    read = valid if every else grad
    return dict(bytes=(read + T) * V * e + 32.0 * T, flops=9.0 * read * V)


def tolerance(case):
    """About four times the distance from the 64-bit result over the declared ranges."""
    if case["kind"] == "advantage":
        return {"rel": 5e-7}    # formed in 64 bits, rounded once
    if case["kind"] == "logprob":
        return {"rel": 1.2e-6}  # 32-bit sums over exactly widened logits
    if case["kind"] == "fused":
        return {"rel": 1e-2} if case["bwd"] else {"rel": 5e-7}   # 16-bit operands of the gradient products
    # the stored gradient entry's own rounding; in 32 bits the loss, whose terms cancel inside a group (single
    # draws were seen 1.5e-4 off)
    return {"rel": {"f32": 6e-4, "bf16": 7e-3, "f16": 1e-3, "f8": 0.12}[case["dtype"]]}


# ---------------------------------------------------------------------------------- 64-bit reference
def _exact_advantage(case, seed):
    x = _advantage_inputs(case, seed)
    p = aero.AdvParams()
    off, rew, L, keys = x["offsets"], x["rewards"].astype(np.float64), x["lengths"], x["keys"]
    R, Q = rew.size, case["Q"]
    adv, weight, mask = np.zeros(R), np.zeros(R), np.zeros(R, np.uint8)
    zv, cat, counts = np.zeros(Q, np.uint8), np.zeros(Q, np.uint8), np.zeros(Q, np.int64)
    for q in range(Q):
        i = np.arange(off[q], off[q + 1])
        r, n, c = rew[i], i.size, int(rew[i].sum())
        order = np.lexsort((i, keys[i]))          # by (key, index)
        if c == 0 or c == n:
            cat[q], keep = (0 if c == 0 else 3), np.sort(i[order[:p.zero_keep]])
        elif c * p.tau_den < n * p.tau_num:       # all correct rollouts, k per correct one of the others
            wrong = i[order[r[order] != 1.0]][:min(p.k_ratio * c, n - c)]
            cat[q], keep = 1, np.sort(np.concatenate([i[r == 1.0], wrong]))
        else:
            cat[q], keep = 2, i
        cat[q] |= 4 if c <= p.s_rescue else 0
        mask[keep] = 1
        counts[q] = keep.size
        k = rew[keep]
        zv[q] = k.max() == k.min()
        mu, sd = k.mean(), k.std()
        if zv[q]:
            mu = (c + p.alpha0) / (n + p.alpha0 + p.beta0)
            sd = math.sqrt(mu * (1 - mu))
        adv[keep] = (k - mu) / sd
        weight[keep] = 1.0 / (Q * float(keep.size) * L[keep])
    index = np.full(R, -1, np.int32)
    index[:counts.sum()] = np.nonzero(mask)[0]
    return adv, weight, mask, index, np.concatenate([[0], np.cumsum(counts)]).astype(np.int32), zv, cat


def exact(case, seed):
    if case["kind"] == "advantage":
        return tuple(torch.from_numpy(a) for a in _exact_advantage(case, seed))
    x = _inputs(case, seed)
    T, V = case["T"], case["V"]
    d64 = lambda *shape: torch.zeros(shape, dtype=torch.float64, device="cuda")
    valid = x["targets"] >= 0
    i, y = x["owner"].clamp(min=0).long(), x["targets"].clamp(min=0).long()
    A = torch.where(valid, x["adv"].double()[i], d64())
    w = torch.where(valid, x["weight"].double()[i], d64())
    fused, bwd = case["kind"] == "fused", case["kind"] == "loss" or case.get("bwd", 0)
    ec, kc = case.get("entropy_coef", 0.0), case.get("kl_coef", 0.0)
    scale = 1.0 if fused else _grad_scale(case)
    lp, ent, lse, loss = d64(T), d64(T), d64(T), d64()
    if fused:
        W = x["W"].double()
        if bwd:
            dh, dW = d64(T, case["H"]), d64(V, case["H"])
    elif bwd:
        dlogits = d64(T, case["ld"])
    clipped = signal = 0
    for a, b in _row_chunks(T, V * 2):
        z = x["hidden"][a:b].double() @ W.t() if fused else x["logits"][a:b, :V].double()
        ok = valid[a:b]
        s = torch.logsumexp(z, 1)
        pi = torch.exp(z - s[:, None])
        zy = z.gather(1, y[a:b, None])[:, 0]
        H = s - (pi * z).sum(1)
        zero = torch.zeros_like(s)
        lse[a:b], lp[a:b], ent[a:b] = (torch.where(ok, v, zero) for v in (s, zy - s, H))
        if not bwd:
            continue
        rho = torch.exp(lp[a:b] - x["old"][a:b].double())
        Ac, wc = A[a:b], w[a:b]
        lo, hi = 1 - float(np.float32(EPS)), 1 + float(np.float32(EPS))
        loss -= (wc * torch.minimum(rho * Ac, rho.clamp(lo, hi) * Ac)).sum()
        act = torch.where(Ac > 0, rho <= hi, rho >= lo) & (Ac != 0)
        signal += int((Ac != 0).sum())
        clipped += int(((Ac != 0) & ~act).sum())
        g = torch.where(act, -scale * wc * Ac * rho, zero)
        if kc:
            kc32 = float(np.float32(kc))
            d = x["ref"][a:b].double() - lp[a:b]
            loss += (kc32 * wc * torch.where(ok, torch.exp(d) - d - 1, zero)).sum()
            g = g + torch.where(ok, scale * kc32 * wc * (1 - torch.exp(d)), zero)
        dz = -g[:, None] * pi
        dz.scatter_add_(1, y[a:b, None], g[:, None])
        if ec:
            ec32 = float(np.float32(ec))
            loss -= (ec32 * wc * ent[a:b]).sum()
            dz += torch.where(ok, scale * ec32 * wc, zero)[:, None] * pi * (z - s[:, None] + H[:, None])
        if fused:
            rows = torch.nonzero(g)[:, 0]
            dh[a:b] = dz @ W
            dW += dz[rows].t() @ x["hidden"][a:b].double()[rows]
        else:
            dlogits[a:b, :V] = dz
    if case["kind"] == "logprob":
        return (lp, lse) + ((ent,) if case["entropy"] else ())
    if not bwd:
        return lp, ent, lse
    tail = (loss.reshape(1), torch.tensor([clipped / signal if signal else 0.0], dtype=torch.float64, device="cuda"))
    if fused:
        return (lp, ent, lse) + tail + (dh, dW)
    head = (lp, ent, lse) if case["stats"] else (lp, lse) if case["lse"] else ()
    return head + tail + (dlogits,)
