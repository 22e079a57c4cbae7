"""GPU parity for the logits path: group advantages, softmax statistics, clipped loss and
dlogits, each compared element by element with the float64 checker on the same seeded inputs.

Tolerances (stated for the method): masks, kept indices and counts bit-exact; log-probs and
entropy within 2e-3 absolute; loss within 1e-4 relative; dlogits within 1e-2 absolute and,
because |dlogits| <= |g_t| is tiny, also scale-free: within 1e-2 |g_t| plus one bf16 / fp32
rounding of the entry.  Advantages and weights within 1e-6 relative.
"""
import numpy as np
import pytest
import torch

import aero_inputs as ai
from oracle import aero_oracle as orc
from oracle.aero_oracle import AdvParams

pytestmark = pytest.mark.gpu

LP_TOL = 2e-3
ENT_TOL = 2e-3
DZ_ATOL = 1e-2


@pytest.fixture(scope="module")
def gh():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_helpers
    return gpu_helpers


# ------------------------------------------------------------------ group advantage

MODES = [dict(), dict(reject_enable=1), dict(reject_enable=1, posterior_mode=1), dict(posterior_mode=1),
         dict(reject_enable=1, k_ratio=2), dict(reject_enable=1, k_ratio=3, s_rescue=1, zero_keep=2,
                                                posterior_mode=1, alpha0=0.5, beta0=2.0)]


def check_groups(gh, arrays, params, keys="wl"):
    rewards, lengths, offsets, kp = arrays
    ref = orc.group_advantage(rewards, lengths, offsets, kp if keys else None, AdvParams(**params))
    out = gh.run_group_advantage(arrays, params, keys=keys)
    nk = int(ref["kept_offsets"][-1])
    assert np.array_equal(out["keep_mask"].cpu().numpy(), ref["keep_mask"])
    assert np.array_equal(out["kept_offsets"].cpu().numpy(), ref["kept_offsets"])
    assert np.array_equal(out["kept_index"].cpu().numpy()[:nk], ref["kept_index"])
    assert np.array_equal(out["zero_var"].cpu().numpy(), ref["zero_var"])
    assert np.array_equal(out["category"].cpu().numpy(), ref["category"])
    assert int(out["err"].item()) == ref["err"]
    for k in ("adv", "weight"):
        got = out[k].cpu().numpy().astype(np.float64)
        assert np.allclose(got, ref[k], rtol=1e-6, atol=0), k
        assert np.array_equal(got == 0, ref[k] == 0), k
    return ref, out


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg3", "cfg4", "cfg5"])
@pytest.mark.parametrize("mode", range(len(MODES)))
def test_group_advantage_configs(gh, name, mode):
    wl = ai.make_config(name)
    check_groups(gh, (wl.rewards, wl.lengths, wl.group_offsets, wl.keep_priority), MODES[mode])


def test_group_advantage_edge_cases(gh):
    rng = np.random.default_rng(21)
    # big groups (several strides of 64), empty groups, single-rollout groups, tied keys, no keys
    sizes = [0, 1, 200, 0, 65, 64, 2, 3, 129, 0]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    R = int(off[-1])
    rewards = (rng.random(R) < 0.2).astype(np.float32)
    rewards[off[5]:off[6]] = 1.0
    lengths = rng.integers(0, 50, size=R).astype(np.int32)       # includes zero lengths
    keys = rng.integers(0, 3, size=R).astype(np.uint32)
    for params in MODES:
        check_groups(gh, (rewards, lengths, off, keys), params)
        check_groups(gh, (rewards, lengths, off, keys), params, keys=None)
    # Q = 0 and R = 0
    out = gh.run_group_advantage((np.zeros(0, np.float32), np.zeros(0, np.int32), np.array([0], np.int32), None),
                                 dict(), keys=None)
    assert out["kept_offsets"].cpu().tolist() == [0]
    # many groups: the scan spans several entries per thread
    sizes = rng.integers(0, 6, size=5000)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    R = int(off[-1])
    rewards = (rng.random(R) < 0.4).astype(np.float32)
    check_groups(gh, (rewards, rng.integers(1, 9, size=R).astype(np.int32), off,
                      rng.integers(0, 2 ** 32, size=R, dtype=np.uint32)), dict(reject_enable=1, posterior_mode=1))


@pytest.mark.parametrize("seed", range(16))
def test_group_advantage_random_structures(gh, seed):
    """Seeded random group structures (empty, single, several strides of 64 wide), success rates, tied keys
    and hyper-parameters of the curation step, all outputs bit for bit / to 1e-6 against the checker."""
    rng = np.random.default_rng(1000 + seed)
    Q = int(rng.integers(1, 300))
    sizes = np.where(rng.random(Q) < 0.1, rng.integers(65, 200, size=Q), rng.integers(0, 34, size=Q))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    R = int(off[-1])
    p_q = np.repeat(rng.beta(0.5, 0.5, size=Q), sizes)
    rewards = (rng.random(R) < p_q).astype(np.float32)
    lengths = rng.integers(1, 3000, size=R).astype(np.int32)
    keys = rng.integers(0, int(rng.choice([2, 5, 2 ** 32])), size=R).astype(np.uint32)
    tau = [(1, 2), (1, 3), (2, 3), (1, 1)][int(rng.integers(4))]
    params = dict(k_ratio=int(rng.integers(1, 5)), s_rescue=int(rng.integers(0, 4)), tau_num=tau[0], tau_den=tau[1],
                  zero_keep=int(rng.integers(1, 7)), reject_enable=int(rng.integers(2)),
                  posterior_mode=int(rng.integers(2)), alpha0=float(rng.choice([0.5, 1.0, 2.0])),
                  beta0=float(rng.choice([0.5, 1.0, 3.0])))
    check_groups(gh, (rewards, lengths, off, keys), params)
    check_groups(gh, (rewards, lengths, off, keys), params, keys=None)


@pytest.mark.parametrize("Q,lo,hi", [(33, 1, 8), (121, 60, 68), (401, 8, 30), (257, 60, 68), (1500, 20, 60)])
def test_group_advantage_placement_forms(gh, Q, lo, hi):
    """Kept rollouts placed by every workgroup for itself, around and above 8192 rollouts, groups on both sides of the
    64 that a wave holds, the number of groups no multiple of a workgroup's four."""
    rng = np.random.default_rng(Q)
    sizes = rng.integers(lo, hi + 1, size=Q)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    R = int(off[-1])
    assert (R > 8192) == (Q in (257, 1500))
    rewards = (rng.random(R) < np.repeat(rng.beta(0.5, 0.5, size=Q), sizes)).astype(np.float32)
    check_groups(gh, (rewards, rng.integers(1, 3000, size=R).astype(np.int32), off,
                      rng.integers(0, 4, size=R).astype(np.uint32)), dict(reject_enable=1, posterior_mode=1, k_ratio=2))


@pytest.mark.parametrize("Q,R", [(1, 64), (1, 65), (7, 448), (8, 512), (9, 513), (15, 300), (16, 1024), (17, 1025), (33, 8191), (500, 8192), (500, 8193),
                                 (1536, 8192), (1537, 8191), (2047, 2500), (2048, 8192),
                                 (2047, 32768), (2048, 32768), (2048, 32769), (2049, 20000), (1, 8192), (1, 8193), (129, 8256),
                                 (129, 8257), (512, 32768), (511, 32768)])
def test_group_advantage_one_launch(gh, Q, R):
    """One launch up to 2048 groups and 8192 rollouts, without rejection up to 32768 of at most 64 a group on average: around a
    workgroup's 8 groups (16 from 1537 groups on), the rollouts that a workgroup's loads cover, the last call of each form and the
    first of the other; some groups wider than a wave."""
    rng = np.random.default_rng(Q * 100003 + R)
    cuts = np.sort(rng.integers(0, R + 1, size=Q - 1))
    off = np.concatenate([[0], cuts, [R]]).astype(np.int32)      # empty groups and long ones by chance
    rewards = (rng.random(R) < np.repeat(rng.beta(0.5, 0.5, size=Q), np.diff(off))).astype(np.float32)
    lengths = rng.integers(0, 3000, size=R).astype(np.int32)
    keys = rng.integers(0, 50, size=R).astype(np.uint32)
    for params in (dict(reject_enable=1, posterior_mode=1), dict(reject_enable=1, k_ratio=2), dict(), dict(posterior_mode=1)):
        check_groups(gh, (rewards, lengths, off, keys), params)


@pytest.mark.parametrize("Q,R,rejection,launches", [(256, 8192, 1, 1), (300, 8193, 1, 2), (300, 8193, 0, 1), (512, 32768, 0, 1),
                                                    (511, 32768, 0, 2), (1000, 32769, 0, 2), (2048, 8192, 0, 1), (2049, 8192, 0, 2),
                                                    (8193, 20000, 0, 3)])
def test_group_advantage_launches(gh, Q, R, rejection, launches):
    """The call is bound by its launches; the results of every form are in test_group_advantage_one_launch."""
    import paper_2602_14338_amd as aero
    off = np.linspace(0, R, Q + 1).astype(np.int32)
    ints = [gh.dev(np.ones(R, np.int32)), gh.dev(off), gh.dev(np.arange(R, dtype=np.int32))]
    f, b = (lambda n: torch.zeros(n, device=gh.DEV)), (lambda n: torch.zeros(n, dtype=torch.uint8, device=gh.DEV))
    out = [f(R), f(R), b(R), torch.zeros_like(ints[0]), torch.zeros_like(ints[1]), b(Q), b(Q), torch.zeros_like(ints[0][:1])]
    rewards = f(R)
    assert gh.launches(lambda: aero.aero_group_advantage(rewards, *ints, Q, R, aero.AdvParams(reject_enable=rejection), *out)) == launches


@pytest.mark.parametrize("mask_off", [0, 1, 2, 3])
@pytest.mark.parametrize("Q,lo,hi", [(9, 1, 40), (33, 1, 8), (402, 8, 30), (4095, 0, 3), (4097, 0, 3), (8191, 0, 3),
                                     (8195, 0, 3)])
def test_group_advantage_rollouts_outside_the_groups(gh, Q, lo, hi, mask_off):
    """Offsets that start above 0 (all placement forms: one workgroup, every workgroup for itself up to 8192 groups, by a
    scan): the rollouts in front stay unwritten whatever they hold, everything else is as if they were not there, no
    index leaves [0, R).  The same with an empty group in front whose range lies behind the others (8192 groups, and
    8196).  The mask also starts off the 4-byte grid."""
    rng = np.random.default_rng(10 * Q + mask_off)
    sizes = rng.integers(lo, hi + 1, size=Q)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(off[-1])
    rewards = (rng.random(n) < np.repeat(rng.beta(0.5, 0.5, size=Q), sizes)).astype(np.float32)
    lengths = rng.integers(1, 3000, size=n).astype(np.int32)
    keys = rng.integers(0, 4, size=n).astype(np.uint32)
    params = dict(reject_enable=1, posterior_mode=1, k_ratio=2)

    def run(rewards, lengths, off, keys):
        nQ, R = len(off) - 1, len(rewards)
        mask = torch.full((R + 8,), 0xFF, dtype=torch.uint8, device=gh.DEV)
        idx = torch.full((R + 64,), -5, dtype=torch.int32, device=gh.DEV)
        adv, weight = torch.full((R,), 7.0, device=gh.DEV), torch.full((R,), 7.0, device=gh.DEV)
        ko = torch.full((nQ + 1,), -5, dtype=torch.int32, device=gh.DEV)
        zv, cat = (torch.full((nQ,), 9, dtype=torch.uint8, device=gh.DEV) for _ in range(2))
        gh.aero.aero_group_advantage(gh.dev(rewards), gh.dev(lengths), gh.dev(off), gh.dev(keys.view(np.int32)), nQ, R,
                                     gh.aero.AdvParams(**params), adv, weight, mask[mask_off:mask_off + R], idx[:R], ko, zv, cat)
        m = mask.cpu().numpy()
        assert (m[:mask_off] == 0xFF).all() and (m[mask_off + R:] == 0xFF).all() and (idx[R:] == -5).all()
        return dict(adv=adv.cpu().numpy(), weight=weight.cpu().numpy(), keep_mask=m[mask_off:mask_off + R],
                    kept_index=idx[:R].cpu().numpy(), kept_offsets=ko.cpu().numpy(), zero_var=zv.cpu().numpy(),
                    category=cat.cpu().numpy())

    ref = orc.group_advantage(rewards, lengths, off, keys, AdvParams(**params))
    nk = int(ref["kept_offsets"][-1])
    for gap in (0, 1, 37):
        pad = lambda a, v: np.concatenate([np.full(gap, v, a.dtype), a])
        out = run(pad(rewards, 1), pad(lengths, 5), (off + gap).astype(np.int32), pad(keys, 0))
        assert np.array_equal(out["kept_offsets"], ref["kept_offsets"])
        assert np.array_equal(out["kept_index"][:nk], ref["kept_index"] + gap)
        assert np.array_equal(out["keep_mask"][gap:], ref["keep_mask"]) and (out["keep_mask"][:gap] == 0xFF).all()
        assert np.array_equal(out["zero_var"], ref["zero_var"]) and np.array_equal(out["category"], ref["category"])
        for k in ("adv", "weight"):
            assert np.allclose(out[k][gap:], ref[k], rtol=1e-6, atol=0) and (out[k][:gap] == 7.0).all()
    back = np.concatenate([[n], off]).astype(np.int32)           # offsets that descend once: an empty group [n, 0)
    ref = orc.group_advantage(rewards, lengths, back, keys, AdvParams(**params))
    out = run(rewards, lengths, back, keys)
    for k in ("kept_offsets", "keep_mask", "zero_var", "category"):
        assert np.array_equal(out[k], ref[k]), k
    assert np.array_equal(out["kept_index"][:nk], ref["kept_index"])


def test_group_advantage_general_rewards_and_error_flag(gh):
    rng = np.random.default_rng(22)
    sizes = [5, 9, 16, 70]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rewards = rng.normal(size=int(off[-1])).astype(np.float32)
    rewards[off[1]:off[2]] = 0.25                                    # all equal, non-binary
    arrays = (rewards, np.full(len(rewards), 11, np.int32), off, None)
    ref = orc.group_advantage(*arrays, AdvParams())
    out = gh.run_group_advantage(arrays, dict(), keys=None)
    assert np.allclose(out["adv"].cpu().numpy(), ref["adv"], rtol=2e-6, atol=1e-7)
    assert out["zero_var"].cpu().tolist() == [0, 1, 0, 0] and int(out["err"].item()) == 0
    out = gh.run_group_advantage(arrays, dict(reject_enable=1), keys=None)
    assert int(out["err"].item()) & orc.ERR_NONBINARY_REWARD


def test_binding_native_and_general_ways_agree(gh, monkeypatch):
    """A call whose arguments are all plain goes to the library in one native step; forms that are not (an int subclass,
    parameters of a subclass) are converted as ever, with the same results, and what was refused raises the same on both ways."""
    b = gh.aero.binding
    wl = ai.make_config("cfg1")
    rew, ln, off = gh.dev(wl.rewards), gh.dev(wl.lengths), gh.dev(wl.group_offsets)

    class Small(int):
        pass

    class Params(gh.aero.AdvParams):
        pass

    def call(Q=wl.Q, p=gh.aero.AdvParams(reject_enable=1), rewards=rew, mask_dtype=torch.uint8):
        out = [torch.zeros(wl.R, device=gh.DEV), torch.zeros(wl.R, device=gh.DEV),
               torch.zeros(wl.R, dtype=mask_dtype, device=gh.DEV), torch.zeros(wl.R, dtype=torch.int32, device=gh.DEV),
               torch.zeros(wl.Q + 1, dtype=torch.int32, device=gh.DEV), torch.zeros(wl.Q, dtype=torch.uint8, device=gh.DEV),
               torch.zeros(wl.Q, dtype=torch.uint8, device=gh.DEV)]
        b.aero_group_advantage(rewards, ln, off, None, Q, wl.R, p, *out, None)
        return out

    def outcome(**kw):
        try:
            return [o.cpu() for o in call(**kw)]
        except Exception as e:   # noqa: BLE001
            return type(e), str(e)

    assert b._m.group_advantage is not None
    forms = [dict(), dict(Q=Small(wl.Q)), dict(p=Params(reject_enable=1)), dict(p=gh.aero.AdvParams(reject_enable=True)),
             dict(Q=float(wl.Q)), dict(Q=2 ** 40), dict(Q=-1), dict(p=None), dict(rewards=rew.cpu()), dict(rewards=rew.double()),
             dict(rewards=rew.repeat(2)[::2]), dict(mask_dtype=torch.int32), dict(p=gh.aero.AdvParams(k_ratio=0))]
    native = [outcome(**f) for f in forms]
    monkeypatch.setattr(b._m, "group_advantage", lambda *a: NotImplemented)
    for f, got in zip(forms, native):
        want = outcome(**f)
        if isinstance(want, tuple):
            assert got == want, f
        else:
            assert all(torch.equal(x, y) for x, y in zip(got, want)), f


class _Int(int):
    pass


@pytest.mark.parametrize("entry", ["group_advantage", "logprob_fwd", "loss_bwd", "loss_bwd noalloc", "loss_bwd given lse", "fused"])
def test_binding_native_step_of_every_call(gh, monkeypatch, entry):
    """Plain arguments go through the native step, which answers with a status; what is not plain it leaves alone, with
    NotImplemented.  Either way the results, or the error, are those of the general way.  Every argument has a value of its own, so that
    two that change places show."""
    b, native = gh.aero.binding, entry.split()[0]
    T, V, H, R, ld = 70, 333, 40, 7, 340
    rng = np.random.default_rng(5)
    f = lambda *s, scale=1.0: gh.dev((rng.normal(size=s) * scale).astype(np.float32))   # noqa: E731
    z = f(T, ld, scale=2.0).bfloat16()
    hid, w = f(T, H).bfloat16(), f(V, H, scale=0.3).bfloat16()
    tg = gh.dev(rng.integers(-1, V, size=T).astype(np.int32))
    own = gh.dev(rng.integers(-2, R, size=T).astype(np.int32))
    active = gh.dev(rng.integers(0, 2, size=T).astype(np.uint8))
    old, ref, lse, ent = f(T, scale=0.1) - 5.8, f(T, scale=0.1) - 5.7, f(T, scale=0.1) + 7.0, f(T, scale=0.1) + 4.0
    adv, wt = f(R) + 0.3, f(R, scale=0.1).abs() + 0.05
    sizes = np.array([8, 30, 2, 65, 9, 1, 5])
    off = gh.dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    n = int(sizes.sum())
    rew = gh.dev(rng.integers(0, 2, size=n).astype(np.float32))
    lens, keys = (gh.dev(rng.integers(1, 999, size=n).astype(np.int32)) for _ in range(2))
    ws = torch.empty(max(gh.aero.aero_workspace_bytes(op, T=T, V=V, H=H, R=R) for op in (b.OP_GRPO_LOSS_BWD, b.OP_LMHEAD_FUSED)),
                     dtype=torch.uint8, device=gh.DEV)
    new = lambda *s, dtype=torch.float32: torch.full(s, 7, dtype=dtype, device=gh.DEV)   # noqa: E731

    def call(**kw):
        g = lambda k, v: kw.get(k, v)   # noqa: E731
        err = new(1, dtype=torch.int32) * 0
        lp, en, ls, loss, clip = new(T), new(T), new(T), new(1), new(1)
        mid = (g("T", T), g("V", V))
        tail = dict(entropy_coef=g("entropy_coef", 0.03), kl_coef=0.05, ref_logprob=g("ref", ref))
        rest = (g("old", old), own, adv, wt, g("R", R), 0.15, g("eps_hi", 0.25), 3.0)
        if entry == "group_advantage":
            p = gh.aero.AdvParams(k_ratio=g("k_ratio", 2), s_rescue=1, tau_num=2, tau_den=3, zero_keep=3, reject_enable=1,
                                  posterior_mode=1, alpha0=g("alpha0", 1.5), beta0=0.5)
            out = [new(n), new(n), new(n, dtype=torch.uint8), new(n, dtype=torch.int32), new(8, dtype=torch.int32),
                   new(7, dtype=torch.uint8), new(7, dtype=torch.uint8)]
            b.aero_group_advantage(g("old", rew), lens, off, keys, g("R", 7), n, p, *out, err)
        elif entry == "logprob_fwd":
            out = [lp, en, ls]
            b.aero_logprob_fwd(g("z", z), *mid, ld, g("tg", tg), active, *out, err)
        elif entry == "fused":
            out = [lp, en, ls, loss, clip, new(T, H, dtype=torch.bfloat16), new(V, H, dtype=g("dw", torch.float32))]
            b.aero_lmhead_logprob_fused(g("z", hid), w, mid[0], H, mid[1], g("tg", tg), lp, en, ls, *rest, loss, clip, out[5], out[6],
                                        ws, err, dweight_accumulate=g("accumulate", False), **tail)
        else:
            d = new(T, ld, dtype=g("dw", torch.bfloat16))
            given = entry == "loss_bwd given lse"
            out = [loss, clip, lp, d] + ([] if given else [en, ls])
            head = (g("z", z), *mid, ld, g("tg", tg), lse if given else None, *rest, loss, clip, lp, d)
            tail.update(dict(entropy=ent) if given else dict(entropy_out=en, lse_out=ls))
            if entry == "loss_bwd noalloc":
                b.aero_grpo_loss_bwd_noalloc(*head, err, **tail)
            else:
                b.aero_grpo_loss_bwd(*head, ws, err, **tail)
        return out + [err]

    answers = []
    step = getattr(b._m, native)
    general = []

    def watched(*a):
        answers.append(NotImplemented if general else step(*a))
        return answers[-1]
    monkeypatch.setattr(b._m, native, watched)

    def outcome(kw):
        try:
            return call(**kw)
        except Exception as e:   # noqa: BLE001
            return type(e), str(e)

    plain = [dict(), dict(R=-1)] + {"group_advantage": [dict(k_ratio=1, alpha0=2)], "logprob_fwd": [dict(V=300)],
                                    "fused": [dict(dw=torch.bfloat16, accumulate=True), dict(dw=torch.float16)]}.get(entry, [dict(eps_hi=1)])
    if entry == "logprob_fwd":
        plain[1] = dict(T=-1)
    other = {"group_advantage": [dict(R=_Int(7)), dict(R=2.0), dict(k_ratio=True), dict(k_ratio=1.5), dict(alpha0="x"), dict(old=rew.cpu()),
                                 dict(old=rew.double())]}.get(
        entry, [dict(T=_Int(T)), dict(T=float(T)), dict(V=2 ** 40), dict(tg=tg.long()), dict(tg=tg.cpu()), dict(z=z.double()),
                dict(z=z.t().contiguous().t())])
    if entry.startswith("loss"):
        other += [dict(dw=torch.float32), dict(eps_hi=np.float64(0.25)), dict(eps_hi="x"), dict(ref=ref.double())]
    if entry == "fused":
        other += [dict(accumulate=1), dict(dw=torch.float64), dict(z=hid.float())]
    for kw in plain + other:
        answers.clear()
        got = outcome(kw)
        assert len(answers) == 1 and (type(answers[0]) is int if kw in plain else answers[0] is NotImplemented), (kw, answers)
        general.append(True)
        want = outcome(kw)
        general.clear()
        if isinstance(want, tuple):
            assert got == want, kw
        else:
            assert isinstance(got, list) and all(torch.equal(x, y) for x, y in zip(got, want)), kw
            assert not (got[0] == 7).all(), kw


# ------------------------------------------------------------------ softmax statistics

def check_fwd(gh, wl, row_active=None, targets=None, offset_elems=0):
    targets = wl.targets if targets is None else targets
    host = wl.logits_rows(0, wl.T)
    ref = orc.logprob_fwd(host, wl.dtype, wl.V, targets, row_active)
    if offset_elems:   # misaligned base pointer: slice a flat buffer
        flat = np.concatenate([np.zeros(offset_elems, host.dtype), host.reshape(-1)])
        d = gh.logits_to_dev(flat, wl.dtype)[offset_elems:]
    else:
        d = gh.logits_to_dev(host, wl.dtype)
    lp, ent, lse, err = gh.run_fwd(d, wl.T, wl.V, wl.ld, targets, row_active)
    ignored = targets < 0
    if row_active is not None:
        ignored |= row_active == 0
    for got, want, tol in ((lp, ref[0], LP_TOL), (ent, ref[1], ENT_TOL), (lse, ref[2], LP_TOL)):
        g = got.cpu().numpy().astype(np.float64)
        assert np.isfinite(g).all()
        assert np.abs(g - want).max() <= tol
        assert not g[ignored].any()                 # ignored rows give exact zeros
    return err


def test_fwd_cfg1_full(gh):
    assert check_fwd(gh, ai.make_config("cfg1")) == 0


@pytest.mark.parametrize("V,ld", [(1000, 1000), (1000, 1008), (4999, 4999), (4999, 5008), (32768, 32768),
                                  (151936, 151936), (152064, 152064), (262144, 262152), (7, 8), (1, 1), (65, 72)])
def test_fwd_bf16_shapes(gh, V, ld):
    slots = 4 if V > 100000 else 12
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots)
    active = (wl.token_rollout >= 0).astype(np.uint8)
    assert check_fwd(gh, wl) == 0
    assert check_fwd(gh, wl, row_active=active) == 0


@pytest.mark.parametrize("V,ld", [(1024, 1024), (1023, 1023), (5000, 5004), (151936, 151936)])
def test_fwd_f32_shapes(gh, V, ld):
    wl = ai.make_config("cfg1", V=V, ld=ld, L=2)
    assert check_fwd(gh, wl) == 0


# fp16 storage (beyond the paper's bf16 runs, App. C): same definitions on binary16 values, the
# checker widens them exactly.  "Parity unpinned" by the paper in the sense that no experiment of
# it uses this format; the arithmetic is the pinned one.
@pytest.mark.parametrize("V,ld", [(1000, 1000), (4999, 5008), (151936, 151936), (65, 72), (7, 8)])
def test_fwd_f16_shapes(gh, V, ld):
    slots = 4 if V > 100000 else 12
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots, dtype="f16")
    active = (wl.token_rollout >= 0).astype(np.uint8)
    assert check_fwd(gh, wl) == 0
    assert check_fwd(gh, wl, row_active=active) == 0
    assert check_fwd(gh, wl, offset_elems=3) == 0          # misaligned base: scalar path


# 8-bit float storage (4 exponent, 3 mantissa bits).  Parity unpinned by the paper (it trains in bf16,
# App. C); the arithmetic is the pinned one, the widening is pinned bit for bit on the host.
@pytest.mark.parametrize("V,ld", [(1000, 1008), (4999, 5008), (151936, 151936), (65, 80), (7, 16), (5000, 5003)])
def test_fwd_f8_shapes(gh, V, ld):
    slots = 4 if V > 100000 else 12
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots, dtype="f8e4m3")
    active = (wl.token_rollout >= 0).astype(np.uint8)
    assert check_fwd(gh, wl) == 0
    assert check_fwd(gh, wl, row_active=active) == 0
    assert check_fwd(gh, wl, offset_elems=3) == 0          # misaligned base: scalar path


@pytest.mark.parametrize("dtype,V", [("bf16", 32776), ("bf16", 40961), ("f32", 16385), ("f32", 70003)])
@pytest.mark.parametrize("T", [255, 256, 257])
def test_fwd_rows_around_one_per_cu(gh, T, V, dtype):
    """Long rows take 1024 threads each up to a row per CU, 512 beyond."""
    rng = np.random.default_rng(T + V)
    z = rng.normal(0, 3, size=(T, V)).astype(np.float32)
    host = z if dtype == "f32" else ai.f32_to_bf16_bits(z)
    tg = rng.integers(0, V, size=T).astype(np.int32)
    tg[::7] = -1
    ref = orc.logprob_fwd(host, dtype, V, tg)
    lp, ent, lse, err = gh.run_fwd(gh.logits_to_dev(host, dtype), T, V, V, tg)
    assert err == 0
    for got, want, tol in ((lp, ref[0], LP_TOL), (ent, ref[1], ENT_TOL), (lse, ref[2], LP_TOL)):
        g = got.cpu().numpy()
        assert np.abs(g - want).max() <= tol and not g[tg < 0].any()


def test_fwd_misaligned_base_and_bad_targets(gh):
    wl = ai.make_config("cfg2", V=4096, slots=6, len_lo=1, len_hi=6)
    assert check_fwd(gh, wl, offset_elems=3) == 0
    tg = wl.targets.copy()
    tg[::5] = -1
    assert check_fwd(gh, wl, targets=tg) == 0
    tg[1] = wl.V          # outside the vocabulary: ignored row + error bit, no fault
    tg[2] = 2 ** 31 - 1
    host = wl.logits_rows(0, wl.T)
    lp, ent, lse, err = gh.run_fwd(gh.logits_to_dev(host, "bf16"), wl.T, wl.V, wl.ld, tg)
    assert err & 2 and lp[1].item() == 0 and lse[2].item() == 0
    assert torch.isfinite(lp).all()


def test_fwd_large_magnitudes(gh):
    """Rows whose maximum moves a lot along the row and logits far outside exp's fp32 range."""
    V = 20000
    rng = np.random.default_rng(31)
    z = rng.normal(0, 3, size=(6, V)).astype(np.float32)
    z[0] += np.linspace(-300, 300, V, dtype=np.float32)       # maximum at the very end
    z[1] += np.linspace(300, -300, V, dtype=np.float32)       # maximum at the start
    z[2] *= 100.0
    z[3] = 5.0                                                # uniform row
    z[4, :] = -200.0
    z[4, 77] = 200.0                                          # one dominant logit
    z[5] -= 5000.0
    tg = np.array([V - 1, 0, 5, 6, 77, 9], np.int32)
    for dtype in ("f32", "bf16"):
        host = z if dtype == "f32" else ai.f32_to_bf16_bits(z)
        ref = orc.logprob_fwd(host, dtype, V, tg)
        lp, ent, lse, err = gh.run_fwd(gh.logits_to_dev(host, dtype), 6, V, V, tg)
        scale = np.maximum(1.0, np.abs(ref[2]))
        assert (np.abs(lp.cpu().numpy() - ref[0]) <= LP_TOL * scale).all()
        assert (np.abs(lse.cpu().numpy() - ref[2]) <= LP_TOL * scale).all()
        assert (np.abs(ent.cpu().numpy() - ref[1]) <= ENT_TOL * scale).all()


def test_fwd_empty(gh):
    z = torch.zeros((0, 16), dtype=torch.bfloat16, device=gh.DEV)
    gh.run_fwd(z, 0, 16, 16, np.zeros(0, np.int32))


# ------------------------------------------------------------------ loss and dlogits

def elt_rounding(dtype, ref_abs):
    """One rounding of the stored gradient entry: bf16 has 8 significant bits, fp32 24, fp16 11
    and a fixed grid of 2^-24 below 2^-14 (subnormals), the 8-bit float 4 and a grid of 2^-9 below 2^-6."""
    if dtype == "f16":
        return ref_abs * 2.0 ** -11 + 2.0 ** -25
    if dtype == "f8e4m3":
        return ref_abs * 2.0 ** -4 + 2.0 ** -10
    return ref_abs * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -23) + 1e-30


def check_loss_bwd(gh, wl, params, sigma_old=0.05, use_oracle_lse=True, inplace=False, grad_scale=1.0,
                   expect_clip=False, stats=False, entropy_coef=0.0, kl_coef=0.0, adv_map=None, strict_loss=False,
                   untouched=None):
    """adv_map: replaces the group-relative advantages by adv_map(adv) before both sides see them
    (supplied advantages; e.g. abs makes every term of the loss carry one sign).
    strict_loss: the loss must meet the pure 1e-4 relative bound (well-conditioned case).
    untouched: "half" or "all" - that share of the padding rows is handed to the library as
    AERO_ROW_UNTOUCHED; their gradient rows must keep what the buffer held before the call, everything
    else must come out as for plain padding (the checker sees plain padding)."""
    host = wl.logits_rows(0, wl.T)
    tr_gpu = wl.token_rollout.copy()
    chosen = np.zeros(0, dtype=np.int64)
    if untouched is not None:
        pads = np.flatnonzero(wl.token_rollout < 0)
        chosen = pads if untouched == "all" else pads[::2]
        assert chosen.size > 0
        tr_gpu[chosen] = gh.binding.AERO_ROW_UNTOUCHED
    ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, wl.keep_priority, AdvParams(**params))
    if adv_map is not None:
        ga["adv"] = adv_map(ga["adv"].astype(np.float32)).astype(np.float64)
    active = (wl.token_rollout >= 0).astype(np.uint8)
    lp_ref, ent_ref, lse_ref = orc.logprob_fwd(host, wl.dtype, wl.V, wl.targets, active)
    old = ai.draw_old_logprob(lp_ref, wl.seed, sigma=sigma_old)
    eps = np.float32(wl.eps)
    # log-probs of a reference policy: the behaviour ones moved by seeded noise (input data only)
    ref_lp = (old + np.random.default_rng(wl.seed + 77).normal(0, 0.2, size=old.shape)).astype(np.float32) \
        if kl_coef != 0.0 else None
    ref = orc.grpo_loss_bwd(host, wl.dtype, wl.V, wl.targets, old, wl.token_rollout, ga["adv"].astype(np.float32),
                            ga["weight"].astype(np.float32), eps, eps, grad_scale, entropy_coef=entropy_coef,
                            kl_coef=kl_coef, ref_logprob=ref_lp)
    d = gh.logits_to_dev(host, wl.dtype)
    lse_d = gh.dev(lse_ref.astype(np.float32)) if use_oracle_lse else None
    before = gh.raw_bits(d)[torch.from_numpy(chosen).to(gh.DEV)].clone() if (inplace and chosen.size) else None
    out = gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, wl.targets, lse_d, old, tr_gpu,
                          ga["adv"], ga["weight"], eps=float(eps), grad_scale=grad_scale, inplace=inplace, stats=stats,
                          entropy_coef=entropy_coef,
                          entropy=ent_ref if (use_oracle_lse and entropy_coef != 0.0) else None,
                          kl_coef=kl_coef, ref_logprob=ref_lp)
    assert out["err"] == 0
    loss = out["loss"].item()
    gh.assert_loss(loss, ref["loss"], ref["loss_terms"], strict=strict_loss)
    assert abs(out["clip_frac"].item() - ref["clip_frac"]) < 1e-6
    if expect_clip:
        assert 0.02 < ref["clip_frac"] < 0.98
    lp = out["logprob"].cpu().numpy().astype(np.float64)
    if stats:   # statistics for every valid row, as the forward call would give them
        assert np.abs(lp - lp_ref).max() <= LP_TOL and not lp[active == 0].any()
        for key, want in (("entropy", ent_ref), ("lse", lse_ref)):
            got = out[key].cpu().numpy().astype(np.float64)
            assert np.abs(got - want).max() <= LP_TOL and not got[active == 0].any()
    else:
        assert np.abs(lp - ref["logprob"]).max() <= LP_TOL
    dz = gh.to_np64(out["dlogits"])[:, :wl.V]
    want = ref["dlogits"]
    if chosen.size:   # not written at all: the rows hold what the buffer held before the call
        rows = gh.raw_bits(out["dlogits"])[torch.from_numpy(chosen).to(gh.DEV)]
        if inplace:
            assert torch.equal(rows, before)
        else:
            assert torch.equal(rows, gh.raw_bits(gh.full_like_seven(out["dlogits"][:1])).expand_as(rows))
        dz[chosen] = 0.0
    assert np.isfinite(dz).all()
    # stated for the unscaled gradient; an 8-bit stored entry's own rounding (2^-4 relative) is allowed on top
    stored = elt_rounding(wl.dtype, np.abs(want)) if wl.dtype == "f8e4m3" else 0.0
    assert (np.abs(dz - want) <= DZ_ATOL * max(1.0, grad_scale) + stored).all()
    # scale of a row: |g_t| for the surrogate, |e_t| (|p ln p| + p H_t) <= |e_t| (1 + H_t) for the entropy term
    scale = np.abs(ref["g"]) + np.abs(ref["e"]) * (1.0 + ent_ref)
    bound = 1e-2 * scale[:, None] + elt_rounding(wl.dtype, np.abs(want))
    assert (np.abs(dz - want) <= bound).all()
    dead = (ref["g"] == 0) & (ref["e"] == 0)
    dead[chosen] = False
    bits = gh.raw_bits(out["dlogits"])[:, :wl.V]
    assert not bits[torch.from_numpy(dead).to(gh.DEV)].any()       # exactly +0, sign bit included
    if wl.ld > wl.V and not inplace:                                # pad columns are not written
        assert gh.all_seven(out["dlogits"][:, wl.V:])
    return ref, out


def test_loss_bwd_cfg1_full(gh):
    wl = ai.make_config("cfg1")
    ref, _ = check_loss_bwd(gh, wl, dict())
    assert (ref["g"] == 0).sum() >= 2 * 8 * 64      # the two all-equal groups
    check_loss_bwd(gh, wl, dict(), use_oracle_lse=False)
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, expect_clip=True)
    check_loss_bwd(gh, wl, dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, inplace=True, grad_scale=64.0)


def test_entropy_bonus_cfg1(gh):
    """Entropy bonus (Table 8 coefficient and a large one): rows of the all-equal groups now
    carry the entropy-only gradient, rows of dropped rollouts stay exactly +0."""
    wl = ai.make_config("cfg1")
    ref0, _ = check_loss_bwd(gh, wl, dict())
    for coef in (1e-3, 0.05):
        ref, _ = check_loss_bwd(gh, wl, dict(), entropy_coef=coef)
        assert (ref["e"] != 0).sum() > (ref0["g"] != 0).sum() and ref["loss"] < ref0["loss"]
        assert ((ref["g"] == 0) & (ref["e"] != 0)).any()
        check_loss_bwd(gh, wl, dict(), use_oracle_lse=False, sigma_old=0.3, expect_clip=True, entropy_coef=coef,
                       grad_scale=16.0)
    # curation drops rollouts (weight 0): their rows have neither term
    ref, _ = check_loss_bwd(gh, wl, dict(reject_enable=1, posterior_mode=1), entropy_coef=0.01, inplace=True)
    assert ((ref["e"] == 0) & (wl.token_rollout >= 0)).any()


# 151936 and 32768 take the single-pass kernels (streaming / one workgroup per row) when lse is not given
@pytest.mark.parametrize("V,ld,slots", [(151936, 151936, 6), (32768, 32768, 8), (4999, 4999, 10), (1000, 1008, 10)])
def test_entropy_bonus_cfg2_reduced(gh, V, ld, slots):
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots)
    check_loss_bwd(gh, wl, dict(), entropy_coef=1e-3)
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, use_oracle_lse=False, expect_clip=True, entropy_coef=0.02, stats=True)


@pytest.mark.parametrize("cfg,kw", [("cfg1", dict()), ("cfg2", dict(V=151936, ld=151936, slots=6, len_lo=1, len_hi=6)),
                                    ("cfg2", dict(V=32768, ld=32768, slots=8, len_lo=1, len_hi=8)),
                                    ("cfg2", dict(V=4999, ld=4999, slots=10, len_lo=1, len_hi=10))])
def test_kl_penalty(gh, cfg, kw):
    """Eq. 2's beta term: every token of a weighted rollout is pulled towards the reference policy,
    also in the all-equal groups and on clipped tokens; alone and together with the entropy bonus."""
    wl = ai.make_config(cfg, **kw)
    ref0, _ = check_loss_bwd(gh, wl, dict(), sigma_old=0.3)
    ref, _ = check_loss_bwd(gh, wl, dict(), sigma_old=0.3, kl_coef=0.04, expect_clip=True)
    assert ref["loss"] > ref0["loss"] and (ref["g"] != 0).sum() > (ref0["g"] != 0).sum()
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, use_oracle_lse=False, kl_coef=0.04)   # one-call route, penalty alone
    check_loss_bwd(gh, wl, dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False, kl_coef=0.04,
                   entropy_coef=1e-3, grad_scale=4.0, stats=True)


def test_kl_penalty_needs_the_reference_logprobs(gh):
    wl = ai.make_config("cfg1")
    d = gh.logits_to_dev(wl.logits_rows(0, wl.T), wl.dtype)
    with pytest.raises(Exception):
        gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, wl.targets, None, np.zeros(wl.T), wl.token_rollout,
                        np.zeros(wl.R), np.zeros(wl.R), kl_coef=0.1)


def test_entropy_bonus_needs_the_entropy_array(gh):
    wl = ai.make_config("cfg1")
    d = gh.logits_to_dev(wl.logits_rows(0, wl.T), wl.dtype)
    lse = torch.zeros(wl.T, device=gh.DEV)
    with pytest.raises(Exception):
        gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, wl.targets, lse, np.zeros(wl.T), wl.token_rollout,
                        np.zeros(wl.R), np.zeros(wl.R), entropy_coef=1e-3)


# V >= 8192 with aligned rows takes the single-pass kernel when lse is not given: 151936 and
# 163840 (its largest row) use 20 vectors per thread, 32768 and 8200 (ragged tail) use 8;
# 163848 is one vector too long and falls back to forward + gradient passes, as do the others
# (262144: the largest vocabularies in use).
@pytest.mark.parametrize("V,ld,slots", [(151936, 151936, 6), (4999, 4999, 10), (1000, 1008, 10), (32768, 32768, 10),
                                        (8200, 8200, 10), (163840, 163848, 4), (163848, 163848, 4),
                                        (262144, 262144, 4)])
def test_loss_bwd_cfg2_reduced(gh, V, ld, slots):
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots)
    check_loss_bwd(gh, wl, dict())
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, use_oracle_lse=False, expect_clip=True)
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, use_oracle_lse=False, stats=True)
    check_loss_bwd(gh, wl, dict(), inplace=True)
    check_loss_bwd(gh, wl, dict(), inplace=True, use_oracle_lse=False, stats=True, grad_scale=3.0)


@pytest.mark.parametrize("V,ld,slots", [(151936, 151936, 6), (4999, 4999, 10), (1000, 1008, 10), (32768, 32768, 8)])
def test_loss_bwd_f16(gh, V, ld, slots):
    """fp16 logits and gradients.  grad_scale lifts the gradient entries out of fp16's subnormal
    range, as a caller training in fp16 would; the unscaled run checks the rounding to that grid."""
    def wl():
        return ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots, dtype="f16")
    check_loss_bwd(gh, wl(), dict(), grad_scale=4096.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, expect_clip=True, grad_scale=4096.0, stats=True)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, inplace=True, grad_scale=4096.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3)
    check_loss_bwd(gh, wl(), dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False,
                   entropy_coef=1e-3, kl_coef=0.04, grad_scale=4096.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, adv_map=lambda a: np.abs(a) + np.float32(0.25), strict_loss=True)


@pytest.mark.parametrize("V,ld,slots", [(151936, 151936, 6), (4999, 5008, 10), (1000, 1003, 10), (32768, 32768, 8)])
def test_loss_bwd_f8(gh, V, ld, slots):
    """8-bit float logits and gradients.  The gradient entries are far below the format's grid (2^-9), so a
    grad_scale lifts them (512: the largest entries of these short-response batches stay below the format's
    maximum of 448); the unscaled run checks that everything rounds to that grid (mostly to zero)."""
    def wl():
        return ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots, dtype="f8e4m3")
    check_loss_bwd(gh, wl(), dict(), grad_scale=512.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, expect_clip=True, grad_scale=512.0, stats=True)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, inplace=True, grad_scale=512.0,
                   untouched="half")
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3)
    check_loss_bwd(gh, wl(), dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False,
                   entropy_coef=1e-3, kl_coef=0.04, grad_scale=512.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, adv_map=lambda a: np.abs(a) + np.float32(0.25), strict_loss=True)


def test_f8_gradient_rounding_bit_exact(gh):
    """The narrowing of gradient entries to the 8-bit float, bit for bit.  Rows [0, -384] with lse = 0 and the
    second token sampled have p = (1, 0) exactly, so with weight 1, ratio 1 and advantage -x the stored entry of
    the sampled token is x itself: every representable value, every midpoint of two neighbours (ties to even),
    values around the subnormal grid, and magnitudes beyond 448 (saturate) are compared with the host rounding
    (itself pinned against torch)."""
    grid = orc.widen(np.arange(127, dtype=np.uint8), "f8e4m3")
    mid = (grid[:-1] + grid[1:]) / 2
    rng = np.random.default_rng(5)
    x = np.concatenate([grid, mid, np.nextafter(mid.astype(np.float32), np.float32(0)),
                        np.nextafter(mid.astype(np.float32), np.float32(1e9)),
                        np.abs(rng.standard_normal(2000)) * 30, np.abs(rng.standard_normal(500)) * 0.01,
                        [449.0, 463.9, 464.0, 479.9, 480.0, 1e4, 3e38, 2.0 ** -10, 2.0 ** -11, 1e-30]]).astype(np.float32)
    x = np.concatenate([x, -x])
    x = x[x != 0]                       # advantage 0 switches the row off
    T = len(x)
    want = ai.f32_to_f8e4m3_bits(x)
    for V in (2, 16):                   # 2: rows of 2 bytes, element-wise stores; 16: one 16-byte vector per row
        z = np.tile(ai.f32_to_f8e4m3_bits(np.float32([0.0] + [-384.0] * (V - 1))), (T, 1))
        targets = np.ones(T, np.int32)
        lse = np.zeros(T, np.float32)
        old = np.full(T, -384.0, np.float32)          # = the current log-prob: ratio exactly 1, never clipped
        out = gh.run_loss_bwd(gh.logits_to_dev(z, "f8e4m3"), T, V, V, targets, gh.dev(lse), old,
                              np.arange(T, dtype=np.int32), -x.astype(np.float64), np.ones(T), eps=0.2)
        assert out["err"] == 0
        got = gh.raw_bits(out["dlogits"]).cpu().numpy()
        assert np.array_equal(got[:, 1], want)            # g (1 - p_1) = x
        assert np.array_equal(got[:, 0], want ^ 0x80)     # g (0 - p_0) = -x
        assert not (got[:, 2:] & 0x7F).any()              # -x * 0: a zero of either sign


# One pass over the logits: a row of n 16-byte vectors goes to workgroups of 64 / 256 / 512 / 1024 threads up to
# n = 512 / 2048 / 4096 / 8192, to the streaming kernel up to 20480, to its form that reads part of a row again up to 81920
# and takes two passes beyond; an odd pitch puts every row at another offset from 16 bytes.
@pytest.mark.parametrize("dtype,V,ld,slots", [
    ("bf16", 4096, 4096, 9), ("bf16", 4104, 4107, 9), ("bf16", 16391, 16391, 6), ("bf16", 32775, 32777, 5),
    ("bf16", 65543, 65543, 4), ("bf16", 163847, 163849, 3), ("bf16", 3, 5, 40), ("bf16", 9, 9, 40),
    ("f16", 16393, 16395, 6), ("f16", 151937, 151939, 3),
    ("f32", 2048, 2049, 9), ("f32", 8197, 8197, 6), ("f32", 81920, 81922, 3), ("f32", 81927, 81927, 3), ("f32", 2, 3, 40),
    ("f8e4m3", 8207, 8209, 6), ("f8e4m3", 131103, 131107, 3), ("f8e4m3", 17, 19, 40),
    # enough rows for one pass over fp16 and 8-bit rows that stream (96 and 192), and too few
    ("f16", 151937, 151939, 7), ("f16", 65549, 65551, 6), ("f16", 65549, 65551, 5), ("f16", 65549, 65549, 17),
    ("f8e4m3", 131103, 131107, 13), ("f8e4m3", 131103, 131107, 11),
    # rows that a CU does not hold: one vector more than it does, an odd number of rounds more, the longest, too few rows (16-bit
    # under 54 and, the longest, 213, fp32 under 24 or 10 MB, 8-bit under 256 MB)
    ("bf16", 163855, 163857, 3), ("bf16", 163848, 163848, 2), ("bf16", 262144, 262144, 4), ("f16", 180001, 180003, 3),
    ("f32", 81931, 81931, 2), ("f32", 152064, 152064, 2), ("f32", 327683, 327683, 2), ("f32", 327684, 327684, 2),
    ("f8e4m3", 327713, 327715, 12), ("bf16", 163855, 163857, 12), ("f16", 180001, 180003, 12), ("bf16", 163847, 163847, 11),
    ("f32", 262144, 262147, 2), ("f32", 262148, 262148, 2)])
def test_single_pass_edges(gh, dtype, V, ld, slots):
    def wl():
        return ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots - 1, dtype=dtype)
    gs = {"f16": 4096.0, "f8e4m3": 256.0}.get(dtype, 1.0)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, stats=True, grad_scale=gs, untouched="half")
    check_loss_bwd(gh, wl(), dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False, inplace=True,
                   grad_scale=gs, entropy_coef=0.01, kl_coef=0.04)


@pytest.mark.parametrize("T", [512, 513])
def test_loss_only_f8_rows(gh, T):
    """8-bit rows without a gradient, one pass up to 512 rows and the forward pass alone beyond: loss, clip fraction and
    log-probs as in the call that also forms the gradient (32-bit sums in another order)."""
    V, R = 65568, 40
    g = torch.Generator(device=gh.DEV)
    g.manual_seed(T)
    z = (torch.randn(T, V, generator=g, device=gh.DEV) * 3).to(torch.float8_e4m3fn)
    rng = np.random.default_rng(T)
    tg = rng.integers(0, V, size=T).astype(np.int32)
    tr = rng.integers(-2, R, size=T).astype(np.int32)
    args = (z, T, V, V, tg, None, np.full(T, -12.0, np.float32), tr, np.abs(rng.normal(size=R)) + 0.1, np.full(R, 1.0 / T))
    full, only = gh.run_loss_bwd(*args), gh.run_loss_bwd(*args, want_dlogits=False)
    assert full["loss"].item() != 0.0
    assert abs(full["loss"].item() - only["loss"].item()) <= 1e-6 * abs(full["loss"].item())
    assert full["clip_frac"].item() == only["clip_frac"].item()
    assert (full["logprob"] - only["logprob"]).abs().max() <= 4e-6    # two steps of a value near 12


@pytest.mark.parametrize("off_z,off_d", [(1, 1), (3, 11), (5, 13), (2, 7)])
@pytest.mark.parametrize("V", [777, 70003])
def test_loss_bwd_at_element_offsets(gh, V, off_z, off_d):
    """Logits and gradient that start off the 16-byte grid, alike (one pass) and differently (two passes): the same
    results as from aligned buffers up to a rounding of the stored entry, nothing written around the rows."""
    wl = ai.make_config("cfg2", V=V, slots=5, len_lo=1, len_hi=5)
    host = wl.logits_rows(0, wl.T)
    ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, wl.keep_priority, AdvParams())
    old = np.full(wl.T, -12.0, np.float32)
    n = wl.T * V

    def run(oz, od):
        z = torch.zeros(n + 16, dtype=torch.bfloat16, device=gh.DEV)
        z[oz:oz + n] = gh.logits_to_dev(host, "bf16").reshape(-1)
        dz = torch.full((n + 32,), 7.0, dtype=torch.bfloat16, device=gh.DEV)
        ws = torch.empty(gh.aero.aero_workspace_bytes(gh.binding.OP_GRPO_LOSS_BWD, T=wl.T, V=V, R=wl.R), dtype=torch.uint8,
                         device=gh.DEV)
        loss = torch.zeros(1, device=gh.DEV)
        gh.aero.aero_grpo_loss_bwd(z[oz:oz + n].view(wl.T, V), wl.T, V, V, gh.dev(wl.targets), None, gh.dev(old),
                                gh.dev(wl.token_rollout), gh.dev(ga["adv"].astype(np.float32)),
                                gh.dev(ga["weight"].astype(np.float32)), wl.R, 0.2, 0.2, 1.0, loss, None, None,
                                dz[od:od + n].view(wl.T, V), ws)
        assert (dz[:od] == 7.0).all() and (dz[od + n:] == 7.0).all()
        return loss.item(), dz[od:od + n].double()
    loss_a, dz_a = run(0, 0)
    loss_b, dz_b = run(off_z, off_d)
    assert abs(loss_a - loss_b) <= 1e-5 * abs(loss_a) + 1e-9
    # the same sums in another order: 32-bit differences, which move a stored entry by one step of bf16 at most
    assert ((dz_a - dz_b).abs() <= 2.0 ** -7 * dz_a.abs() + 1e-30).all()


@pytest.mark.parametrize("dtype,V,T,terms", [("f8e4m3", 1310720, 206, False), ("f8e4m3", 327713, 820, True),
                                             ("bf16", 655360, 205, False), ("f16", 655360, 205, True), ("f32", 327680, 205, False)])
def test_rows_held_in_part_against_two_passes(gh, dtype, V, T, terms):
    """256 MB of rows that a CU does not hold, among them the longest it takes: the gradient of one pass (dlogits as aligned as the
    logits) and of two (one element off), up to a step of the stored entry; a quarter of the rows padding or left alone."""
    store = {"f8e4m3": torch.float8_e4m3fn, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    assert T * (V * store.itemsize // 16) * 16 >= 2 ** 28
    R, n = 24, T * V
    g = torch.Generator(device=gh.DEV)
    g.manual_seed(V)
    z = torch.empty(T, V, dtype=store, device=gh.DEV)
    for a in range(0, T, 32):
        z[a:a + 32] = (torch.randn(min(32, T - a), V, generator=g, device=gh.DEV) * 3).to(store)
    rng = np.random.default_rng(V)
    tg = rng.integers(0, V, size=T).astype(np.int32)
    tr = np.where(rng.random(T) < 0.25, rng.integers(-2, 0, size=T), rng.integers(0, R, size=T)).astype(np.int32)
    adv, weight = rng.normal(size=R).astype(np.float32), rng.uniform(0.5, 1.0, size=R).astype(np.float32)
    lp, _, lse, _ = gh.run_fwd(z, T, V, V, tg, want_entropy=False)
    old = lp.cpu().numpy() + rng.normal(0, 0.1, size=T).astype(np.float32)
    scale = {"f16": 4096.0, "f8e4m3": 256.0}.get(dtype, 1.0)

    def run(front):
        dz = torch.zeros(n + 32, dtype=store, device=gh.DEV)
        ws = torch.empty(gh.aero.aero_workspace_bytes(gh.binding.OP_GRPO_LOSS_BWD, T=T, V=V, R=R), dtype=torch.uint8, device=gh.DEV)
        loss = torch.zeros(1, device=gh.DEV)
        kw = dict(entropy_coef=0.02, kl_coef=0.04, ref_logprob=gh.dev(old + np.float32(0.05))) if terms else {}
        gh.aero.aero_grpo_loss_bwd(z, T, V, V, gh.dev(tg), None, gh.dev(old), gh.dev(tr), gh.dev(adv), gh.dev(weight), R, 0.2, 0.2,
                                   scale, loss, None, None, dz[front:front + n].view(T, V), ws, **kw)
        assert not dz[:front].float().any() and not dz[front + n:].float().any()
        return loss.item(), dz[front:front + n].view(T, V)
    (one, d1), (two, d2) = run(0), run(1)
    assert abs(one - two) <= 1e-6 * weight.sum() * T
    # Statistics summed in another order, and the log-partition of two passes rounded to 32 bits (2^-20 at 13), move an entry by some
    # 2e-6 of itself, a stored one by a step of its type on top: 2^-7, 2^-10 and 2^-3 of itself, or the smallest step (bf16: none
    # to speak of, fp16 2^-24, 8-bit 2^-9).  The entropy term's pi c w (z - lse + H) is what cancellation leaves: three sums
    # of up to 32 in 32 bits, 2^-20 each, whatever the entry comes to (fp32, whose bound would be that alone, goes without).
    step = {"bf16": (2.0 ** -7, 0.0), "f16": (2.0 ** -10, 2.0 ** -24), "f8e4m3": (2.0 ** -3, 2.0 ** -9), "f32": (2.0 ** -22, 0.0)}[dtype]
    for a in range(0, T, 16):
        x, y = d1[a:a + 16].float(), d2[a:a + 16].float()
        bound = (step[0] + 1e-5) * x.abs() + step[1] + 1e-30
        if terms:
            bound += torch.exp(z[a:a + 16].float() - lse[a:a + 16, None]) * (scale * 0.02 * weight.max() * 2.0 ** -18)
        assert ((x - y).abs() <= bound).all(), a
    live = torch.from_numpy(tr >= 0).to(gh.DEV)
    assert d1[live][:8].float().any(dim=1).any() and not d1[~live].float().any()


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes_all_storage_types(gh, seed):
    """Seeded random vocabulary sizes, row pitches (aligned and not), batch shapes, storage types and call
    variants: statistics, loss and gradient against the checker as in the fixed cases."""
    rng = np.random.default_rng(2000 + seed)
    dtype = ["bf16", "f32", "f16", "f8e4m3"][seed % 4]
    V = int(rng.choice([rng.integers(1, 64), rng.integers(64, 3000), rng.integers(3000, 40000)]))
    ld = V + int(rng.choice([0, 0, rng.integers(1, 40)]))
    slots = int(rng.integers(3, 13))

    def wl():
        return ai.make_config("cfg2", seed=100 + seed, V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots - 1, dtype=dtype)
    active = (wl().token_rollout >= 0).astype(np.uint8)
    assert check_fwd(gh, wl()) == 0
    assert check_fwd(gh, wl(), row_active=active, offset_elems=int(rng.integers(0, 9))) == 0
    gs = {"f16": 4096.0, "f8e4m3": 256.0}.get(dtype, float(rng.choice([1.0, 3.0])))
    for _ in range(3):
        terms = rng.random() < 0.4
        check_loss_bwd(gh, wl(), dict(reject_enable=int(rng.integers(2)), posterior_mode=int(rng.integers(2))),
                       sigma_old=float(rng.choice([0.05, 0.3])), use_oracle_lse=bool(rng.integers(2)),
                       inplace=bool(rng.integers(2)), grad_scale=gs, stats=False,
                       entropy_coef=0.01 if terms else 0.0, kl_coef=0.04 if terms and rng.random() < 0.5 else 0.0,
                       untouched=[None, "half", "all"][int(rng.integers(3))])


def test_loss_bwd_cfg3_reduced(gh):
    wl = ai.make_config("cfg3", V=151936, T=320, Q=64, len_lo=1, len_hi=12)
    ref, _ = check_loss_bwd(gh, wl, dict())
    assert (ref["g"] == 0).any() and (ref["g"] != 0).any()
    wl = ai.make_config("cfg3", V=151936, T=320, Q=64, len_lo=1, len_hi=12)
    check_loss_bwd(gh, wl, dict(), sigma_old=0.3, use_oracle_lse=False, stats=True)
    check_loss_bwd(gh, wl, dict(reject_enable=1), sigma_old=0.3, use_oracle_lse=False)
    wl = ai.make_config("cfg3", V=8000, T=700, Q=64, len_lo=1, len_hi=12)
    check_loss_bwd(gh, wl, dict(reject_enable=1), sigma_old=0.3, use_oracle_lse=False, expect_clip=True)
    check_loss_bwd(gh, wl, dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, expect_clip=True)


def test_streaming_kernel_optional_terms_several_rows_per_workgroup(gh):
    """V = 151936 with 320 rows: more rows than compute units, so the persistent workgroups of the
    streaming single-pass kernel refill their slots with a second row and draw it from the row
    counter, here in the variant that carries the optional terms (entropy bonus, Table 8; KL
    penalty, Eq. 2's beta term) and with the gradient written over the logits."""
    def wl():
        return ai.make_config("cfg3", V=151936, T=320, Q=64, len_lo=1, len_hi=12)
    ref, _ = check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, entropy_coef=0.02, expect_clip=True)
    assert ((ref["g"] == 0) & (ref["e"] != 0)).any()
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, kl_coef=0.04, stats=True)
    ref, _ = check_loss_bwd(gh, wl(), dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False,
                            kl_coef=0.04, entropy_coef=1e-3, inplace=True, grad_scale=4.0)
    assert (ref["e"] == 0).any() and (ref["e"] != 0).any()      # dropped rollouts: rows with neither term
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, inplace=True)      # plain variant, in place
    check_loss_bwd(gh, wl(), dict(reject_enable=1), use_oracle_lse=False, inplace=True, stats=True)


@pytest.mark.parametrize("inplace,terms", [(False, False), (True, True), (True, False), (False, True)])
@pytest.mark.parametrize("dtype,V,ld,T", [("bf16", 70003, 70005, 624), ("f16", 65549, 65551, 2496), ("f32", 32777, 32779, 2496),
                                          ("f8e4m3", 230001, 230003, 1456),
                                          ("bf16", 66003, 66005, 2048), ("bf16", 66003, 66005, 2049),   # the order's one workgroup, several
                                          ("bf16", 164003, 164005, 832), ("f32", 110001, 110003, 624),
                                          ("f8e4m3", 1300001, 1300003, 416)])   # held in part
def test_streaming_rows_of_changing_alignment(gh, dtype, V, ld, T, inplace, terms):
    """Several rows per workgroup of the streaming kernel, each at another offset from 16 bytes than the one whose slots
    it takes over, after gradient rows and after rows that are only filled with zeros (padding, advantage 0) or
    left alone: bit for bit what calls on 208 rows give, where every workgroup has one row (208 rows begin on the
    16-byte grid at any pitch)."""
    R, step = 24, 208
    g = torch.Generator(device=gh.DEV)
    g.manual_seed(V)
    store = {"f8e4m3": torch.float8_e4m3fn, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    z = torch.empty(T, ld, dtype=store, device=gh.DEV)
    for a in range(0, T, step):
        z[a:a + step] = (torch.randn(min(step, T - a), ld, generator=g, device=gh.DEV) * 3).to(store)
    rng = np.random.default_rng(V)
    tg = rng.integers(0, V, size=T).astype(np.int32)
    tg[:8], tg[8:16] = np.arange(8), V - 1 - np.arange(8)          # in the ragged ends
    tr = np.where(rng.random(T) < 0.25, rng.integers(-2, 0, size=T), rng.integers(0, R, size=T)).astype(np.int32)
    adv, weight = rng.normal(size=R), rng.uniform(0.5, 1.0, size=R)
    adv[:6], weight[6:9] = 0.0, 0.0
    lp, _, _, _ = gh.run_fwd(z, T, V, ld, tg, want_entropy=False)
    old = lp.cpu().numpy() + rng.normal(0, 0.1, size=T).astype(np.float32)
    kw = dict(grad_scale={"f16": 4096.0, "f8e4m3": 256.0}.get(dtype, 1.0), inplace=inplace, stats=True)
    if terms:
        kw.update(entropy_coef=0.02, kl_coef=0.04)

    def run(a, b):
        part = z[a:b].clone() if a == 0 and b == T else z[a:b]   # the whole call on a copy: in place, the parts follow
        if terms:
            kw["ref_logprob"] = old[a:b] + 0.05
        return gh.run_loss_bwd(part, b - a, V, ld, tg[a:b], None, old[a:b], tr[a:b], adv, weight, **kw)
    whole = run(0, T)
    assert whole["err"] == 0 and torch.isfinite(whole["loss"]).all()
    loss = 0.0
    for a in range(0, T, step):
        b = min(T, a + step)
        out = run(a, b)
        loss += out["loss"].item()
        for k in ("logprob", "entropy", "lse"):
            assert torch.equal(out[k], whole[k][a:b]), k
        assert torch.equal(gh.raw_bits(out["dlogits"])[:, :V], gh.raw_bits(whole["dlogits"][a:b])[:, :V])
    written = gh.raw_bits(whole["dlogits"])[torch.from_numpy(tr >= 0).to(gh.DEV)][:, :V]
    assert written.any(dim=1).float().mean() > 0.5
    assert abs(loss - whole["loss"].item()) <= 1e-6 * T


# 151936 with 384 rows: the streaming kernel with several rows per workgroup; 32768: one workgroup per row;
# 4999 / 1000: the forward + gradient route (row kernels); with the checker's lse: the gradient kernels alone
# (151936: one vector per thread in segments).
@pytest.mark.parametrize("V,ld,slots,dtype", [(151936, 151936, 24, "bf16"), (32768, 32768, 10, "bf16"),
                                              (4999, 4999, 10, "bf16"), (1000, 1008, 10, "f32"),
                                              (151936, 151936, 6, "f16")])
def test_untouched_padding_rows(gh, V, ld, slots, dtype):
    """Padding rows marked AERO_ROW_UNTOUCHED: no gradient row is written for them (the buffer keeps its
    contents), their scalar outputs are 0, and every other row - plain padding included - is as before."""
    def wl():
        return ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=1, len_hi=slots - 1, dtype=dtype)
    gs = 4096.0 if dtype == "f16" else 1.0
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, untouched="half", grad_scale=gs)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, untouched="all", stats=True, grad_scale=gs)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=True, untouched="half", grad_scale=gs)
    check_loss_bwd(gh, wl(), dict(), sigma_old=0.3, use_oracle_lse=False, untouched="half", inplace=True, grad_scale=gs)
    check_loss_bwd(gh, wl(), dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=False,
                   untouched="all", entropy_coef=1e-3, kl_coef=0.04, grad_scale=gs)


# Well-conditioned losses: every term carries one sign, so nothing cancels and the stated
# tolerance (1e-4 relative) is enforced with no rounding floor.
@pytest.mark.parametrize("cfg,kw", [("cfg1", dict()),
                                    ("cfg2", dict(V=151936, ld=151936, slots=6, len_lo=1, len_hi=6)),
                                    ("cfg3", dict(V=151936, T=320, Q=64, len_lo=1, len_hi=12)),
                                    ("cfg2", dict(V=4999, ld=4999, slots=10, len_lo=1, len_hi=10))])
def test_loss_strict_tolerance_one_sign_advantages(gh, cfg, kw):
    for route in (True, False):   # statistics given / computed in the call (single pass where it applies)
        check_loss_bwd(gh, ai.make_config(cfg, **kw), dict(), sigma_old=0.3, use_oracle_lse=route, expect_clip=True,
                       adv_map=lambda a: np.abs(a) + np.float32(0.25), strict_loss=True)
        check_loss_bwd(gh, ai.make_config(cfg, **kw), dict(), sigma_old=0.05, use_oracle_lse=route,
                       adv_map=lambda a: -np.abs(a) - np.float32(0.25), strict_loss=True)


@pytest.mark.parametrize("cfg,kw", [("cfg1", dict()), ("cfg3", dict(V=151936, T=320, Q=64, len_lo=1, len_hi=12))])
def test_loss_strict_tolerance_posterior_mode(gh, cfg, kw):
    """Every group all-wrong: in posterior mode (Strategy 2) each kept rollout gets the same negative
    advantage (-1/3 at n = 8 with the uniform prior), the loss is a sum of one-signed terms."""
    for route in (True, False):
        wl = ai.make_config(cfg, **kw)
        wl.rewards[:] = 0.0
        ref, _ = check_loss_bwd(gh, wl, dict(reject_enable=1, posterior_mode=1), sigma_old=0.3, use_oracle_lse=route,
                                expect_clip=True, strict_loss=True)
        assert (ref["g"] != 0).any() and ref["loss"] > 0


# up to 4096 tokens of the shortest rows and 16384 of longer ones the loss takes the first workgroup of the gradient launch
@pytest.mark.parametrize("T,V", [(1, 8), (63, 8), (4096, 8), (4097, 8), (16384, 1040), (16385, 1040), (700, 17000), (65, 40001)])
def test_loss_beside_the_gradient_rows(gh, T, V):
    """The loss and the clip fraction of a call that writes gradient rows are those of one that does not: the same terms in
    64-bit sums of another order, so they differ by one rounding to 32 bits at most."""
    rng = np.random.default_rng(T + V)
    z = gh.logits_to_dev((rng.normal(size=(T, V)) * 2).astype(np.float32), torch.float32)
    y = rng.integers(0, V, size=T).astype(np.int32)
    lp, _, lse = gh.run_fwd(z, T, V, V, y)[:3]
    R = min(T, 50)
    args = (z, T, V, V, y, lse, lp.cpu().numpy() + rng.normal(size=T) * 0.3, (np.arange(T) % R).astype(np.int32),
            rng.normal(size=R) + 0.5, np.full(R, 1.0 / T))
    alone, beside = gh.run_loss_bwd(*args, want_dlogits=False), gh.run_loss_bwd(*args)
    a, b = alone["loss"].item(), beside["loss"].item()
    assert a != 7.0 and abs(a - b) <= 2.0 ** -23 * abs(a)
    assert alone["clip_frac"].item() == beside["clip_frac"].item()
    assert torch.isfinite(beside["dlogits"]).all() and not (beside["dlogits"] == 7.0).any()


def test_loss_is_run_to_run_identical_and_loss_only_mode(gh):
    wl = ai.make_config("cfg3", V=8000, T=3000, Q=64, len_lo=1, len_hi=40)
    host = wl.logits_rows(0, wl.T)
    ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, None, AdvParams())
    lp_ref, _, lse_ref = orc.logprob_fwd(host, wl.dtype, wl.V, wl.targets)
    old = ai.draw_old_logprob(lp_ref, 5, sigma=0.2)
    d = gh.logits_to_dev(host, wl.dtype)
    outs = [gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, wl.targets, None, old, wl.token_rollout, ga["adv"], ga["weight"],
                            want_dlogits=(k < 2)) for k in range(3)]
    assert outs[0]["loss"].view(torch.int32).item() == outs[1]["loss"].view(torch.int32).item()
    assert outs[0]["loss"].view(torch.int32).item() == outs[2]["loss"].view(torch.int32).item()
    assert torch.equal(outs[0]["dlogits"].view(torch.int16), outs[1]["dlogits"].view(torch.int16))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_log_of_the_row_sum_is_rounded_once(gh, dtype):
    """Rows of n zeros among logits of -200: the sum of exponentials is n exactly, so what is left of the error is the
    logarithm's.  Log-partition and log-prob within half a step of the result, and 4.5e-8: the logarithm of
    a factor of n in [1/sqrt 2, sqrt 2), below 0.36, is off by a step of at most 3e-8, and its sum with the
    remainder of n's power of two by half a step of 1.5e-8."""
    V = T = 4096
    z = np.where(np.arange(V)[None, :] <= np.arange(T)[:, None], np.float32(0), np.float32(-200))
    want = np.log(np.arange(1, T + 1, dtype=np.float64))
    bound = np.spacing(want.astype(np.float32)).astype(np.float64) / 2 + 4.5e-8
    host = ai.f32_to_bf16_bits(z).reshape(T, V) if dtype == "bf16" else z
    lp, _, lse, _ = gh.run_fwd(gh.logits_to_dev(host, dtype), T, V, V, np.zeros(T, np.int32), want_entropy=False)
    assert (np.abs(gh.to_np64(lse) - want) <= bound).all()
    assert (np.abs(gh.to_np64(lp) + want) <= bound).all()


@pytest.mark.parametrize("dtype,V,ld,slots", [("bf16", 500, 503, 9), ("bf16", 9000, 9000, 6), ("f32", 40001, 40003, 5)])
def test_sampled_token_at_minus_infinity(gh, dtype, V, ld, slots):
    """A sampled token whose logit is -inf: probability and ratio are 0, so the row is clipped or without gradient and
    the loss stays finite, as with a logit of -1e30 (one workgroup per row, streaming, and two calls)."""
    wl = ai.make_config("cfg2", V=V, ld=ld, slots=slots, len_lo=2, len_hi=slots, dtype=dtype)
    host = wl.logits_rows(0, wl.T)
    rows = np.flatnonzero(wl.token_rollout >= 0)[::3]
    def masked(x):
        h = host.copy()
        h[rows, wl.targets[rows]] = ai.f32_to_bf16_bits(np.float32([x]))[0] if dtype == "bf16" else np.float32(x)
        return h
    ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, wl.keep_priority, AdvParams())
    old = np.full(wl.T, -12.0, np.float32)
    a32, w32 = ga["adv"].astype(np.float32), ga["weight"].astype(np.float32)
    ref = orc.grpo_loss_bwd(masked(-1e30), dtype, V, wl.targets, old, wl.token_rollout, a32, w32, np.float32(0.2),
                            np.float32(0.2), 1.0)
    assert (a32[wl.token_rollout[rows]] > 0).any() and (a32[wl.token_rollout[rows]] < 0).any()
    z = gh.logits_to_dev(masked(-np.inf), dtype)
    _, _, lse, _ = gh.run_fwd(z, wl.T, V, ld, wl.targets, want_entropy=False)
    for given in (None, lse):
        out = gh.run_loss_bwd(z, wl.T, V, ld, wl.targets, given, old, wl.token_rollout, a32, w32)
        gh.assert_loss(out["loss"].item(), ref["loss"], ref["loss_terms"])
        dz = gh.to_np64(out["dlogits"])[:, :V]
        assert (np.abs(dz - ref["dlogits"]) <= 1e-2 * np.abs(ref["g"])[:, None] + 2.0 ** -8 * np.abs(ref["dlogits"])).all()


def test_bad_rollout_index_and_empty_batch(gh):
    wl = ai.make_config("cfg2", V=512, slots=4, len_lo=4, len_hi=4)
    host = wl.logits_rows(0, wl.T)
    ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, None, AdvParams())
    tr = wl.token_rollout.copy()
    tr[3] = wl.R + 5
    d = gh.logits_to_dev(host, wl.dtype)
    out = gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, wl.targets, None, np.zeros(wl.T, np.float32) - 6.0, tr,
                          ga["adv"], ga["weight"])
    assert out["err"] & 4 and not out["dlogits"][3].float().any()
    out = gh.run_loss_bwd(d[:0], 0, wl.V, wl.ld, np.zeros(0, np.int32), None, np.zeros(0, np.float32),
                          np.zeros(0, np.int32), ga["adv"], ga["weight"])
    assert out["loss"].item() == 0.0 and out["clip_frac"].item() == 0.0


def test_raw_c_abi_call_without_the_binding(gh):
    """aero_logprob_fwd called through ctypes directly: plain device addresses and sizes, the NULL
    (default) stream, status code returned; results against the checker."""
    import ctypes as C
    from paper_2602_14338_amd import binding
    lib = C.CDLL(binding.library_path())
    p, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
    lib.aero_logprob_fwd.restype = i32
    lib.aero_logprob_fwd.argtypes = [p, i32, i64, i32, i64, p, p, p, p, p, p, p]
    wl = ai.make_config("cfg2", V=4999, ld=5008, slots=5, len_lo=1, len_hi=5)
    host = wl.logits_rows(0, wl.T)
    ref = orc.logprob_fwd(host, "bf16", wl.V, wl.targets)
    z = gh.logits_to_dev(host, "bf16")
    tg = gh.dev(wl.targets)
    lp, ent, lse = (torch.full((wl.T,), 7.0, device=gh.DEV) for _ in range(3))
    torch.cuda.synchronize()
    st = lib.aero_logprob_fwd(z.data_ptr(), 1, wl.T, wl.V, wl.ld, tg.data_ptr(), None, lp.data_ptr(), ent.data_ptr(),
                              lse.data_ptr(), None, None)
    assert st == 0
    torch.cuda.synchronize()
    for got, want in ((lp, ref[0]), (ent, ref[1]), (lse, ref[2])):
        assert np.abs(got.cpu().numpy().astype(np.float64) - want).max() <= LP_TOL
    assert lib.aero_logprob_fwd(z.data_ptr(), 1, wl.T, wl.V, wl.V - 1, tg.data_ptr(), None, lp.data_ptr(), None,
                                lse.data_ptr(), None, None) == 2      # AERO_ERR_SHAPE: ld < V
    assert lib.aero_logprob_fwd(z.data_ptr(), 5, wl.T, wl.V, wl.ld, tg.data_ptr(), None, lp.data_ptr(), None,
                                lse.data_ptr(), None, None) == 3      # AERO_ERR_DTYPE


def test_ignored_rows_are_not_flagged(gh):
    """Padding rows (rollout index -1) and rows switched off with row_active may hold anything in
    their other fields, e.g. a sampled-token id past the vocabulary: no error bit, zero outputs.
    Covers the forward call, the two-call loss route, and both single-pass kernels."""
    for V, slots in ((512, 6), (32768, 6), (151936, 4)):
        wl = ai.make_config("cfg2", V=V, slots=slots, len_lo=1, len_hi=slots - 1)
        host = wl.logits_rows(0, wl.T)
        pad = wl.token_rollout < 0
        assert pad.any()
        tg = wl.targets.copy()
        tg[pad] = V + 7
        ga = orc.group_advantage(wl.rewards, wl.lengths, wl.group_offsets, None, AdvParams())
        d = gh.logits_to_dev(host, wl.dtype)
        lp, ent, lse, err = gh.run_fwd(d, wl.T, wl.V, wl.ld, tg, (~pad).astype(np.uint8))
        assert err == 0 and not lp[torch.from_numpy(pad).to(gh.DEV)].any()
        _, _, _, err = gh.run_fwd(d, wl.T, wl.V, wl.ld, tg, None)      # not switched off: flagged
        assert err == 2
        old = np.full(wl.T, -12.0, np.float32)
        for lse_arg in (lse, None):
            out = gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, tg, lse_arg, old, wl.token_rollout, ga["adv"], ga["weight"])
            assert out["err"] == 0
            assert not out["dlogits"][torch.from_numpy(pad).to(gh.DEV)].float().any()
        tr = wl.token_rollout.copy()
        tr[~pad] = np.where(np.arange((~pad).sum()) % 3 == 0, wl.R + 1, tr[~pad])   # real bad indices are flagged
        out = gh.run_loss_bwd(d, wl.T, wl.V, wl.ld, tg, None, old, tr, ga["adv"], ga["weight"])
        assert out["err"] == 4


def test_host_side_argument_errors(gh):
    import paper_2602_14338_amd as aero
    z = torch.zeros((4, 16), dtype=torch.bfloat16, device=gh.DEV)
    t = torch.zeros(4, dtype=torch.int32, device=gh.DEV)
    f = torch.zeros(4, device=gh.DEV)
    with pytest.raises(aero.AeroError, match="leading dimension"):
        aero.aero_logprob_fwd(z, 4, 16, 8, t, None, f, f, f)
    with pytest.raises(aero.AeroError, match="leading dimension"):
        aero.aero_logprob_fwd(z, 4, 0, 16, t, None, f, f, f)
    with pytest.raises(aero.AeroError, match="NULL"):
        aero.aero_logprob_fwd(z, 4, 16, 16, None, None, f, f, f)
    with pytest.raises(aero.AeroError, match="unsupported dtype"):
        aero.aero_logprob_fwd(z.to(torch.float64), 4, 16, 16, t, None, f, f, f)
    with pytest.raises(aero.AeroError, match="workspace"):
        aero.aero_grpo_loss_bwd(z, 4, 16, 16, t, None, f, t, f, f, 4, 0.2, 0.2, 1.0, f[:1], None, None, None,
                                torch.zeros(8, dtype=torch.uint8, device=gh.DEV))
