"""cover_token_sample through the C ABI against the oracle's token_sample (the same Gumbel-max
construction over its own Philox4x32-10 implementation): the drawn token agrees, except where
two perturbed scores are closer than the fp32 arithmetic of the kernel can separate (then the
kernel's token must be one of the tied maxima of the oracle's fp64 scores), and the
probability agrees to 1e-4 relative.  LLaDA vocabulary in bf16, ragged vocabularies in both
dtypes (the per-thread tail), several temperatures, seeds above 2^32 and steps."""
import numpy as np
import pytest
import torch

import oracle
from helpers import announce
from paper_2602_06161_amd import cover, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,V,dtype,T,seed,step", [
    (64, 126464, "bf16", 0.1, 0, 0), (64, 126464, "bf16", 0.3, 12345, 7),
    (32, 126464, "bf16", 1.0, (1 << 40) + 3, 99), (33, 1001, "f32", 0.2, 5, 1),
    (17, 1003, "bf16", 0.5, 6, 2), (8, 3, "f32", 1.0, 9, 4)])
def test_sample_matches_oracle(R, V, dtype, T, seed, step):
    announce(f"token sample R{R} V{V} {dtype} T{T}")
    a = synth.token_inputs(R, V, seed=R + V, dtype=dtype)
    logits = a["buffer"].cuda()[:, :V]
    tok, prob = cover.cover_token_sample(logits, T, seed, step)
    torch.cuda.synchronize()
    tok, prob = tok.cpu().numpy(), prob.cpu().numpy()
    x = a["logits"].float().numpy()
    rtok, rp, y = oracle.token_sample(x, np.float32(T), seed, step)
    same = tok == rtok
    for r in np.nonzero(~same)[0]:
        ymax = y[r].max()
        assert ymax - y[r, tok[r]] <= 1e-4 * max(1.0, abs(ymax)), f"row {r}: not a near tie"
    assert (~same).sum() <= max(1, R // 50)
    assert np.allclose(prob[same], rp[same], rtol=1e-4, atol=1e-7)


def test_same_seed_same_draws_and_steps_differ():
    announce("token sample determinism")
    a = synth.token_inputs(16, 4096, seed=1)
    logits = a["buffer"].cuda()[:, :4096]
    t1, _ = cover.cover_token_sample(logits, 1.0, 42, 3)
    t2, _ = cover.cover_token_sample(logits, 1.0, 42, 3)
    t3, _ = cover.cover_token_sample(logits, 1.0, 42, 4)
    torch.cuda.synchronize()
    assert torch.equal(t1, t2) and not torch.equal(t1, t3)


@pytest.mark.parametrize("R,V,dtype,T", [
    (6, 4096, "bf16", 0.2), (6, 16384 + 8, "bf16", 0.3), (6, 32771, "bf16", 1.0), (6, 9001, "f32", 0.3),
    (6, 4, "f32", 1.0), (258, 2055, "bf16", 0.5), (258, 8200, "f32", 0.1)])
def test_sample_skips_only_losers(R, V, dtype, T):
    """Rows on which the race's bound works hardest: one level (every token takes part), rising
    and falling logits (the bound moves late, or at once), one token far above the rest in the
    first, a middle and the last place, and masked logits (-inf, the type's lowest value) from
    the start of the row.  Both workgroup sizes (rows up to and past 256), whole and partial
    rounds of loads.  Tolerances as above."""
    announce(f"token sample bound R{R} V{V} {dtype} T{T}")
    rng = np.random.default_rng(V + R)
    ramp = np.linspace(-12.0, 12.0, V)
    low = -3.3895e38  # finite in bf16 and fp32
    x = np.empty((R, V))
    for r in range(R):
        k = r % 6
        x[r] = (0.5, ramp, ramp[::-1], 0.0, 0.0, 0.0)[k]
        if k == 3:
            x[r] = rng.normal(0, 2, V)
            x[r, (0, V // 2, V - 1)[(r // 6) % 3]] = 40.0
        elif k == 4:
            x[r] = rng.normal(0, 2, V)
            x[r, : V // 2] = -np.inf
        elif k == 5:
            x[r] = rng.normal(0, 2, V)
            x[r, : V - V // 4] = low
    dt = synth.TORCH_DTYPE[dtype]
    per = 8 if dtype == "bf16" else 4
    buf = torch.zeros((R, (V + per - 1) // per * per), dtype=dt)
    buf[:, :V] = torch.from_numpy(x).to(dt)
    tok, prob = cover.cover_token_sample(buf.cuda()[:, :V], T, 77, 5)
    torch.cuda.synchronize()
    tok, prob = tok.cpu().numpy(), prob.cpu().numpy()
    rtok, rp, y = oracle.token_sample(buf[:, :V].double().numpy(), np.float32(T), 77, 5)
    same = tok == rtok
    for r in np.nonzero(~same)[0]:
        assert y[r].max() - y[r, tok[r]] <= 1e-4 * max(1.0, abs(y[r].max())), f"row {r}: not a near tie"
    assert (~same).sum() <= max(1, R // 50)
    assert np.allclose(prob[same], rp[same], rtol=1e-4, atol=1e-7)


@pytest.mark.parametrize("R,V,dtype", [(9, 4099, "f32"), (9, 8200, "bf16"), (270, 1003, "f32"), (9, 6, "bf16")])
def test_sample_stays_in_range(R, V, dtype):
    """Rows outside the contract, and finite logits whose quotient by T is not: +inf in the first
    round of loads, in a later one and in several places, -inf everywhere, NaN among ordinary
    logits and alone, quotients beyond fp32 at both ends.  The token indexes an embedding, so it
    is in [0, V) whatever the row; where the row has +inf or ordinary logits beside -inf and NaN
    it is one that holds no less."""
    announce(f"token sample range R{R} V{V} {dtype}")
    rng = np.random.default_rng(V)
    x = rng.normal(0, 2, (R, V))
    kinds = [lambda r: r.__setitem__(0, np.inf), lambda r: r.__setitem__(V - 1, np.inf),
             lambda r: r.__setitem__(slice(V // 3, V // 3 + 2), np.inf), lambda r: r.fill(-np.inf),
             lambda r: r.__setitem__(slice(0, V // 2), np.nan), lambda r: r.fill(np.nan),
             lambda r: r.__setitem__(V // 2, 3.0e38), lambda r: r.fill(-3.0e38), lambda r: None]
    for r in range(R):
        kinds[r % len(kinds)](x[r])
    dt = synth.TORCH_DTYPE[dtype]
    per = 8 if dtype == "bf16" else 4
    buf = torch.zeros((R, (V + per - 1) // per * per), dtype=dt)
    buf[:, :V] = torch.from_numpy(x).to(dt)
    for T in (0.1, 1.0e-6, 1.0e-40, 1.0e30):
        tok, _ = cover.cover_token_sample(buf.cuda()[:, :V], T, 3, 1)
        torch.cuda.synchronize()
        tok = tok.cpu().numpy()
        assert ((0 <= tok) & (tok < V)).all(), f"T {T}: {tok.min()} .. {tok.max()}"
        for r in range(R):
            got = x[r, tok[r]]
            if np.isposinf(x[r]).any():
                assert np.isposinf(got), f"T {T} row {r}"
            elif not np.isnan(x[r]).all():
                assert not np.isnan(got), f"T {T} row {r}"
            if r % len(kinds) == 6 and T <= 0.1:
                assert tok[r] == V // 2, f"T {T} row {r}"


def test_sample_repeats_at_near_ties():
    """64 tokens per row whose perturbed scores agree within fp32 rounding of their logits, and
    whole rows of one level (in two of these calls two tokens share the largest u exactly): the
    draw is the same in every launch and for both workgroup sizes, and a token of the largest
    score.  1e-6: the score's error, 2^-23 of E in its logarithm and 2^-24 in the mantissa's."""
    announce("token sample near ties")
    R, V, T = 300, 4096, 0.5
    rng = np.random.default_rng(8)
    for step in (1, 11):
        u = oracle.sample_uniforms(R, V, 77, step)
        g = -np.log(-np.log(u))
        near = np.full((R, V), -40.0, np.float32)
        for r in range(R):
            at = rng.choice(V, 64, replace=False)
            near[r, at] = (np.float64(np.float32(T)) * (7.0 - g[r, at])).astype(np.float32)
        for name, x in (("near", near), ("flat", np.full((R, V), 1.5, np.float32))):
            dev = torch.from_numpy(x).cuda()
            draws = [cover.cover_token_sample(dev, T, 77, step)[0].cpu().numpy() for _ in range(8)]
            draws += [cover.cover_token_sample(dev[:200], T, 77, step)[0].cpu().numpy() for _ in range(8)]
            for d in draws[1:]:
                assert np.array_equal(d, draws[0][: len(d)]), f"{name} step {step}: {(d != draws[0][:len(d)]).sum()} rows differ"
            y = x.astype(np.float64) / T + g
            if name == "flat":
                assert (np.sort(u, 1)[:, -1] == np.sort(u, 1)[:, -2]).any()
                assert np.array_equal(draws[0], y.argmax(1))
            assert (y.max(1) - y[np.arange(R), draws[0]]).max() <= 1e-6


@pytest.mark.parametrize("R,V,dtype", [(400, 32000, "bf16"), (64, 32003, "f32"), (200, 126464, "bf16"), (40, 5, "f32")])
@pytest.mark.parametrize("T", [0.1, 0.3, 1.0])
def test_sample_probability_error(R, V, dtype, T):
    """The probability is a share of the row's sum: not above 1 (a raised token takes nearly all
    of many of these rows), and within 1.5e-6 of the exact one: 2^-24 |z| ln 2 for the rounding of
    log2 e / T in the terms beside the maximum (|z| about 20 where a term still counts: 8e-7),
    two ulp of the exponentials and 2^-23 for the sums of a thread's few chunks and the tree."""
    announce(f"token sample probability R{R} V{V} {dtype} T{T}")
    g = torch.Generator().manual_seed(V + R)
    per = 8 if dtype == "bf16" else 4
    x = 2.0 * torch.randn(R, (V + per - 1) // per * per, generator=g)
    top = torch.randint(0, V, (R,), generator=g)
    x[torch.arange(R), top] += 14.0 * torch.rand(R, generator=g)
    x = x.to(synth.TORCH_DTYPE[dtype])
    tok, prob = cover.cover_token_sample(x.cuda()[:, :V], T, 11, 2)
    torch.cuda.synchronize()
    assert prob.max().item() <= 1.0
    z = x[:, :V].double() / float(np.float32(T))
    want = torch.exp(z[torch.arange(R), tok.cpu().long()] - torch.logsumexp(z, 1))
    err = ((prob.cpu().double() - want) / want)[want > 1e-3].abs()
    assert err.max().item() <= 1.5e-6, f"{err.max().item():.2e}"
    print(f"probability error rms {err.pow(2).mean().sqrt().item():.1e} max {err.max().item():.1e}")


@pytest.mark.parametrize("R", [5, 260])
@pytest.mark.parametrize("V,dtype", [(255, "f32"), (257, "f32"), (512, "bf16"), (521, "bf16"), (4104, "bf16"),
                                     (8196, "f32"), (16385, "bf16"), (32776, "bf16")])
def test_sample_partial_rounds(R, V, dtype):
    """Rows whose last round of loads leaves waves, or some of a wave's loads, without a chunk
    (these do nothing), one chunk past a whole round, and the winner among the last tokens."""
    announce(f"token sample partial rounds R{R} V{V} {dtype}")
    rng = np.random.default_rng(V)
    x = rng.normal(0, 1, (R, V))
    x[::2, -9:] += 12.0
    dt = synth.TORCH_DTYPE[dtype]
    per = 8 if dtype == "bf16" else 4
    buf = torch.zeros((R, (V + per - 1) // per * per), dtype=dt)
    buf[:, :V] = torch.from_numpy(x).to(dt)
    tok, prob = cover.cover_token_sample(buf.cuda()[:, :V], 0.8, 4, 6)
    torch.cuda.synchronize()
    rtok, rp, y = oracle.token_sample(buf[:, :V].double().numpy(), np.float32(0.8), 4, 6)
    tok, prob = tok.cpu().numpy(), prob.cpu().numpy()
    assert (y.max(1) - y[np.arange(R), tok]).max() <= 1e-6  # the score's error, as above
    same = tok == rtok
    assert np.allclose(prob[same], rp[same], rtol=2e-6, atol=1e-7)
