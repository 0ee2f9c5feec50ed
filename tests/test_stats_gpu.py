"""GPU producers of the selection signals (cover_token_stats, cover_attn_stats, through the
C ABI) against the fp64 oracle.

Tolerances, from the arithmetic:
  token stats: the log-sum-exp is an fp32 sum of V exp2 terms (each within 2 ulp), taken as
    per-thread runs of at most ~V/8192 chunks and a 1024-way tree, so the relative error of
    the sum stays below (V/8192*8 + 10) * 2^-23 ~ 2e-5 for V = 126464; logp = x_y - lz then
    errs by that much absolutely, conf = 1/sum relatively.  argmax is decided on the stored
    values, which both sides compare exactly: bit-exact.
  attention masses: the weights are exp(s - lse) with the lse of cover_attn_fwd, whose row
    sum adds the bf16-rounded probabilities the PV product uses (each within 2^-9); the lse
    is therefore within 2^-9 of the exact one and every weight within that relative error,
    which sums of positive weights keep: rtol 2^-9 ~ 2e-3 (plus 1e-6 absolute for masses of
    rows with nothing in them)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import announce
from paper_2602_06161_amd import cover, synth

pytestmark = pytest.mark.gpu

TOK_ATOL = 3e-5
TOK_RTOL = 3e-5
MASS_RTOL = 2e-3
MASS_ATOL = 1e-6


def _dev(t):
    """The logits on the GPU with their padded row stride."""
    V = t["logits"].shape[1]
    return t["buffer"].cuda()[:, :V]


def _token_check(t):
    logits, tokens = t["logits"], t["tokens"]
    lg, cf, am = cover.cover_token_stats(_dev(t), tokens.cuda())
    torch.cuda.synchronize()
    r_lp, r_cf, r_am = oracle.token_stats(oracle._f64(logits), tokens.numpy())
    assert np.array_equal(am.cpu().numpy(), r_am), "argmax differs"
    np.testing.assert_allclose(lg.cpu().numpy(), r_lp, rtol=0, atol=TOK_ATOL)
    np.testing.assert_allclose(cf.cpu().numpy(), r_cf, rtol=TOK_RTOL, atol=0)


@pytest.mark.parametrize("R,V,dtype", [(8, 126464, "bf16"), (5, 1003, "f32"), (3, 1001, "bf16"),
                                       (2, 1, "f32"), (7, 8, "bf16"), (4, 50000, "f32")])
def test_token_stats_vs_oracle(R, V, dtype):
    announce(f"token stats R{R} V{V} {dtype}")
    t = synth.token_inputs(R, V, seed=V, dtype=dtype)
    _token_check(t)


def test_token_stats_llada_block():
    """The LM-head output of the 256 generated positions of a LLaDA-8B step (vocab 126464)."""
    announce("token stats R256 V126464 bf16")
    t = synth.token_inputs(256, 126464, seed=1)
    _token_check(t)


def test_token_stats_ties_and_bad_tokens():
    announce("token stats ties / bad tokens")
    t = synth.token_inputs(6, 4096, seed=3, dtype="f32")
    x = t["buffer"]  # V = 4096 needs no padding: the buffer is the logits
    x[1, 100] = x[1, 3000] = x[1].max() + 1.0     # tie: the smaller index wins
    x[2, :] = 0.5                                   # all equal: index 0, conf = 1/V
    tok = t["tokens"].clone()
    tok[3], tok[4] = -1, 4096                       # outside [0, V): NaN, no read
    lg, cf, am = cover.cover_token_stats(x.cuda(), tok.cuda())
    torch.cuda.synchronize()
    am, lg, cf = am.cpu().numpy(), lg.cpu().numpy(), cf.cpu().numpy()
    assert am[1] == 100 and am[2] == 0
    assert abs(cf[2] - 1.0 / 4096) < 1e-9
    assert np.isnan(lg[3]) and np.isnan(lg[4])
    ok = [0, 1, 2, 5]
    r_lp, r_cf, r_am = oracle.token_stats(oracle._f64(x[ok]), tok[ok].numpy())
    np.testing.assert_allclose(lg[ok], r_lp, atol=TOK_ATOL, rtol=0)
    assert np.array_equal(am[ok], r_am)


@pytest.mark.parametrize("dtype,V", [("bf16", 5), ("f32", 3), ("bf16", 8197), ("f32", 4099), ("bf16", 65539), ("f32", 32771)])
def test_token_stats_where_the_maximum_lies(dtype, V):
    """The row's maximum in the first and last whole chunk, in the tail past the last one, tied
    within a chunk, across waves and with the tail (the smallest index wins), and large logits
    (the sum's reference is a rounded product of the maximum)."""
    announce(f"token stats maximum positions {dtype} V {V}")
    t = synth.token_inputs(8, V, seed=V, dtype=dtype)
    x = t["buffer"]
    top = x[:, :V].max().item() + 1.0
    n = 8 if dtype == "bf16" else 4
    last = max(V // n * n - 1, 0)
    marks = [(0,), (last,), (V - 1,), (min(1, last), min(2, last)), (V // 2, V - 1), (0, V // 2, last), (V - 2,), (0, V - 1)]
    for r, where in enumerate(marks):
        for j in where:
            x[r, j] = top
    x[6, :V] = x[6, :V] * 8.0 + 300.0
    lg, cf, am = cover.cover_token_stats(x.cuda()[:, :V], t["tokens"].cuda())
    torch.cuda.synchronize()
    xd = x[:, :V].double()
    lz = torch.logsumexp(xd, 1)
    want = xd.gather(1, t["tokens"].long()[:, None])[:, 0] - lz
    assert all(am[r].item() == int((xd[r] == xd[r].max()).nonzero()[0]) for r in range(8))
    # logp: fp32 rounding of numbers up to |x| (2^-24 of 600, twice) and of the sum
    np.testing.assert_allclose(lg.cpu().numpy(), want.numpy(), atol=1e-4, rtol=0)
    np.testing.assert_allclose(cf.cpu().numpy(), torch.exp(xd.max(1).values - lz).numpy(), rtol=TOK_RTOL)


@pytest.mark.parametrize("dtype,V", [("bf16", 5), ("f32", 3), ("bf16", 20), ("bf16", 8197), ("f32", 4099), ("f32", 40003)])
def test_token_stats_masked_and_large_logits(dtype, V):
    """Logits at the type's lowest value (a masked vocabulary) in whole chunks from the start of
    the row, in the tail and everywhere but one; -inf in the same places; rows of one huge level;
    and logits so large that their reference's rounding is no small number.  Finite and exact to
    the tolerances above, relative to the size of the logits where that is the rounding."""
    announce(f"token stats masked {dtype} V {V}")
    dt = synth.TORCH_DTYPE[dtype]
    per = 8 if dtype == "bf16" else 4
    low = torch.finfo(dt).min
    g = torch.Generator().manual_seed(V)
    x = torch.randn(13, (V + per - 1) // per * per, generator=g) * 2
    x[0, : V // 2] = low
    x[1, V // 2:] = low
    x[2] = low
    x[2, V // 3] = 1.0
    x[3] = low                                   # finite: V equal logits
    x[4, : V // 2] = -torch.inf
    x[5] = -torch.inf
    x[5, V - 1] = 0.5
    x[6] = 3.0e38
    x[7, V // 2] = 3.0e38
    x[8] *= 1.0e8                                # the reference's rounding is several units
    x[9] *= -1.0e5
    x[10, V - 1] = low
    x[11, : V - 1] = low
    x[12] *= -1.0e31
    x = x.to(dt)
    tok = torch.full((13,), V - 1, dtype=torch.int32)
    lg, cf, am = cover.cover_token_stats(x.cuda()[:, :V], tok.cuda())
    torch.cuda.synchronize()
    xd = x[:, :V].double()
    top = xd.max(1).values
    total = torch.exp(xd - top[:, None]).sum(1)
    assert torch.equal(am.cpu().long(), (xd == top[:, None]).long().argmax(1))
    np.testing.assert_allclose(cf.cpu().numpy(), (1 / total).numpy(), rtol=TOK_RTOL)
    # the log of the sum is rounded to fp32, and so is its difference with a logit of that size
    want = (xd[:, V - 1] - top - total.log()).numpy()
    size = torch.maximum(top.abs(), xd[:, V - 1].abs()).numpy()
    got = lg.cpu().numpy().astype(np.float64)
    inf = np.isinf(want)
    assert np.array_equal(got[inf], np.full(inf.sum(), -np.inf))
    assert (np.abs(got[~inf] - want[~inf]) <= TOK_ATOL + 2.0**-22 * size[~inf]).all()
    x[0], x[1] = -torch.inf, torch.nan           # no number in the row: still a token of the vocabulary
    _, cf, am = cover.cover_token_stats(x.cuda()[:2, :V], want_logp=False)
    assert torch.equal(am.cpu(), torch.zeros(2, dtype=torch.int32)) and cf.isnan().all().item()


@pytest.mark.parametrize("dtype,V", [("bf16", 7), ("f32", 6), ("bf16", 523), ("f32", 1030), ("bf16", 16397), ("f32", 8201)])
def test_token_stats_ties_within_a_wave(dtype, V):
    """Several threads of one wave hold the row's maximum: neighbouring and distant chunks, a
    thread's second chunk against another's first, chunks against the tail, whole rows of one
    level.  The smallest index wins."""
    announce(f"token stats ties in a wave {dtype} V {V}")
    t = synth.token_inputs(8, V, seed=V + 1, dtype=dtype)
    x = t["buffer"]
    n = 8 if dtype == "bf16" else 4
    top = x[:, :V].max().item() + 1.0
    second = 1024 * n
    ties = [(n + 1, 3 * n), (5 * n + 2, 2 * n + 3, 4 * n), (V - 1, V - 2), (V - 1, n), (second + 2 * n, n + 2),
            (second + n, 3 * n + 1, V - 1), range(V), range(V // 2, V)]
    for r, where in enumerate(ties):
        for j in where:
            x[r, j % V] = top
    _, cf, am = cover.cover_token_stats(x.cuda()[:, :V], want_logp=False)
    torch.cuda.synchronize()
    xd = x[:, :V].double()
    assert torch.equal(am.cpu().long(), (xd == xd.max(1, keepdim=True).values).long().argmax(1))
    np.testing.assert_allclose(cf.cpu().numpy(), torch.exp(xd.max(1).values - torch.logsumexp(xd, 1)).numpy(), rtol=TOK_RTOL)


def _stats_case(a, r0, masked, drafted):
    t = {k: a[k].cuda() for k in ("q", "k_live", "v_live", "k_cache", "v_cache", "seed_idx", "n_seed")}
    _, lse = cover.cover_attn_fwd(t["q"], t["k_live"], t["v_live"], t["k_cache"], t["v_cache"],
                                  t["seed_idx"], t["n_seed"])
    m, d = torch.as_tensor(masked).cuda(), torch.as_tensor(drafted).cuda()
    d_in, d_out = cover.cover_attn_stats(t["q"], t["k_live"], t["k_cache"], t["seed_idx"],
                                         t["n_seed"], lse, m, d, r0)
    d_in2, d_out2 = cover.cover_attn_stats(t["q"], t["k_live"], t["k_cache"], t["seed_idx"],
                                           t["n_seed"], lse, m, d, r0)
    torch.cuda.synchronize()
    assert torch.equal(d_in, d_in2) and torch.equal(d_out, d_out2), "not deterministic"
    r_in, r_out = oracle.attn_stats(a["q"], a["k_live"], a["k_cache"], a["seed_idx"].numpy(),
                                    a["n_seed"].numpy(), r0, np.asarray(masked), np.asarray(drafted))
    np.testing.assert_allclose(d_in.cpu().numpy(), r_in, rtol=MASS_RTOL, atol=MASS_ATOL)
    np.testing.assert_allclose(d_out.cpu().numpy(), r_out, rtol=MASS_RTOL, atol=MASS_ATOL)


@pytest.mark.parametrize("d,r0,Lr", [(64, 120, 80), (128, 0, 200), (128, 150, 50), (64, 199, 1),
                                     (128, 37, 96)])
def test_attn_stats_vs_oracle(d, r0, Lr):
    """Ragged regions and query blocks, GQA, seeds inside the region (their diagonal takes the
    live key) and outside it."""
    announce(f"attn stats d{d} r0 {r0} Lr {Lr}")
    a = synth.attn_inputs("tiny", seed=d + r0, max_seeds=12, B=2, Hq=4, Hkv=2, L=200, d=d,
                          dtype="bf16", prompt=0, unmasked_gen=200, n_seeds=12)
    rng = np.random.default_rng(r0 + Lr)
    # put some seeds inside the region so its diagonal is exercised
    si = a["seed_idx"].numpy().copy()
    for b in range(2):
        inside = np.sort(rng.choice(np.arange(r0, r0 + Lr), size=min(4, Lr), replace=False))
        rest = np.setdiff1d(si[b][si[b] >= 0], inside)[:8]
        row = np.sort(np.concatenate([inside, rest])).astype(np.int32)
        si[b, :] = -1
        si[b, :row.size] = row
        a["n_seed"][b] = row.size
    a["seed_idx"] = torch.from_numpy(si)
    masked = (rng.integers(0, 2, (2, Lr))).astype(np.uint8)
    drafted = (rng.integers(0, 4, (2, Lr)) == 0).astype(np.uint8)
    _stats_case(a, r0, masked, drafted)


@pytest.mark.parametrize("B,Hq,Hkv,L,r0,Lr", [
    (2, 4, 2, 1100, 0, 1100),    # 35 key tiles in 18 groups of 2, the last group one tile
    (1, 32, 32, 2048, 0, 2048),  # 64 key tiles in 8 groups of 8
    (1, 28, 4, 1500, 300, 1111),  # 35 tiles in 9 groups of 4, the last group three tiles (GQA)
])
def test_attn_stats_key_groups(B, Hq, Hkv, L, r0, Lr):
    """Key groups of several 32-key tiles (the next tile of a group is prefetched while the
    current one is used) and a shorter last group, with seeds inside and outside the region."""
    announce(f"attn stats key groups B{B} Hq{Hq} Hkv{Hkv} L{L} r0 {r0} Lr {Lr}")
    a = synth.attn_inputs("tiny", seed=L + Hq, max_seeds=40, B=B, Hq=Hq, Hkv=Hkv, L=L, d=128,
                          dtype="bf16", prompt=0, unmasked_gen=L, n_seeds=40)
    rng = np.random.default_rng(Lr)
    masked = (rng.integers(0, 2, (B, Lr))).astype(np.uint8)
    drafted = (rng.integers(0, 8, (B, Lr)) == 0).astype(np.uint8)
    _stats_case(a, r0, masked, drafted)


def test_attn_stats_long_seed_lists():
    """Seed lists longer than the 512 positions fetched with the seed count (the rest are read
    in a loop), with entries outside [0, L) inside the count and junk past it (ignored), and a
    batch row without seeds; the oracle gets the cleaned lists."""
    B, Hq, Hkv, L, r0, Lr, ms = 2, 4, 2, 1100, 100, 900, 800
    announce(f"attn stats long seed lists B{B} Hq{Hq} L{L} max_seeds {ms}")
    a = synth.attn_inputs("tiny", seed=77, max_seeds=ms, B=B, Hq=Hq, Hkv=Hkv, L=L, d=128,
                          dtype="bf16", prompt=0, unmasked_gen=L, n_seeds=0)
    rng = np.random.default_rng(77)
    si = rng.integers(-50, L + 50, size=(B, ms)).astype(np.int32)  # junk everywhere
    good = np.sort(rng.choice(L, size=700, replace=False)).astype(np.int32)
    si[0, :700] = good
    si[0, 700:703] = [-5, L, L + 9]  # inside the count, outside [0, L)
    counts = np.array([703, 0], np.int32)
    clean = np.full((B, ms), -1, np.int32)
    clean[0, :700] = good
    a["seed_idx"], a["n_seed"] = torch.from_numpy(si), torch.from_numpy(counts)
    masked = (rng.integers(0, 2, (B, Lr))).astype(np.uint8)
    drafted = (rng.integers(0, 4, (B, Lr)) == 0).astype(np.uint8)
    t = {k: a[k].cuda() for k in ("q", "k_live", "v_live", "k_cache", "v_cache", "seed_idx", "n_seed")}
    _, lse = cover.cover_attn_fwd(t["q"], t["k_live"], t["v_live"], t["k_cache"], t["v_cache"],
                                  t["seed_idx"], t["n_seed"])
    m, d = torch.as_tensor(masked).cuda(), torch.as_tensor(drafted).cuda()
    d_in, d_out = cover.cover_attn_stats(t["q"], t["k_live"], t["k_cache"], t["seed_idx"],
                                         t["n_seed"], lse, m, d, r0)
    torch.cuda.synchronize()
    r_in, r_out = oracle.attn_stats(a["q"], a["k_live"], a["k_cache"], clean,
                                    np.array([700, 0], np.int32), r0, masked, drafted)
    np.testing.assert_allclose(d_in.cpu().numpy(), r_in, rtol=MASS_RTOL, atol=MASS_ATOL)
    np.testing.assert_allclose(d_out.cpu().numpy(), r_out, rtol=MASS_RTOL, atol=MASS_ATOL)


def test_attn_stats_workspace_checked():
    """A caller workspace smaller than the launch needs, or of the wrong dtype, is refused
    before anything is enqueued."""
    announce("attn stats workspace checks")
    a = synth.stats_inputs("llada", seed=0)
    t = {k: a[k].cuda() for k in ("q", "k_live", "v_live", "k_cache", "v_cache", "seed_idx", "n_seed")}
    _, lse = cover.cover_attn_fwd(t["q"], t["k_live"], t["v_live"], t["k_cache"], t["v_cache"],
                                  t["seed_idx"], t["n_seed"])
    m, d = a["masked"].cuda(), a["drafted"].cuda()
    B, Hq, _, _ = a["q"].shape
    need = cover.attn_stats_workspace(B, Hq, m.shape[1])
    args = (t["q"], t["k_live"], t["k_cache"], t["seed_idx"], t["n_seed"], lse, m, d, a["r0"])
    with pytest.raises(ValueError):
        cover.cover_attn_stats(*args, workspace=torch.empty(need - 1, device="cuda"))
    with pytest.raises(ValueError):
        cover.cover_attn_stats(*args, workspace=torch.empty(need, device="cuda", dtype=torch.float64))
    d_in, d_out = cover.cover_attn_stats(*args, workspace=torch.empty(need, device="cuda"))
    r_in, r_out = cover.cover_attn_stats(*args)
    torch.cuda.synchronize()
    assert torch.equal(d_in, r_in) and torch.equal(d_out, r_out)


@pytest.mark.parametrize("name", ["llada", "dream"])
def test_attn_stats_workload(name):
    """The generated block of the LLaDA-8B and Dream-7B layer shapes: 256 region positions,
    128 still masked, 15 drafted."""
    announce(f"attn stats {name}")
    a = synth.stats_inputs(name, seed=0)
    _stats_case(a, a["r0"], a["masked"].numpy(), a["drafted"].numpy())


@pytest.mark.parametrize("B,Hq,Hkv,Lr,d", [
    (1, 4, 2, 31, 128), (1, 32, 8, 300, 64),   # one tile per workgroup: eight waves share it
    (1, 128, 8, 128, 64),                      # two tiles: four waves each
    (2, 64, 8, 190, 128),                      # three: two waves each
    (1, 256, 8, 33, 128),                      # two tiles, the second of one position
    (2, 128, 8, 250, 64),                      # eight: one wave each
    (2, 128, 8, 289, 64), (2, 128, 8, 600, 64),  # ten and nineteen: two tiles per wave
    (1, 4, 2, 1100, 128), (1, 128, 8, 1100, 128)])  # more listed tiles than LDS holds at a time
def test_attn_stats_lists(B, Hq, Hkv, Lr, d):
    """The lists of masked queries and drafted keys, at every division of a workgroup's waves:
    all or none of the positions masked or drafted, single ones, counts at the edges of a
    32-row tile, and seeds that are themselves masked and drafted (their diagonal is live)."""
    announce(f"attn stats lists B{B} Hq{Hq} Lr {Lr} d{d}")
    L, r0 = Lr + 45, 24
    a = synth.attn_inputs("tiny", seed=Lr + Hq, max_seeds=24, B=B, Hq=Hq, Hkv=Hkv, L=L, d=d,
                          dtype="bf16", prompt=0, unmasked_gen=L, n_seeds=24)
    seeds = a["seed_idx"].numpy() - r0
    for case in range(4):
        masked, drafted = np.zeros((B, Lr), np.uint8), np.zeros((B, Lr), np.uint8)
        if case == 0:
            masked[:] = 1
            drafted[:, Lr - 1] = 1
        elif case == 1:
            drafted[:] = 255  # nonzero is a member
        elif case == 2:
            masked[:, : min(32, Lr)] = 1
            drafted[:, Lr - min(33, Lr):] = 1
            for b in range(B):
                inside = seeds[b][(seeds[b] >= 0) & (seeds[b] < Lr)]
                masked[b, inside] = drafted[b, inside] = 1
        else:
            masked[:, 0] = 1
        _stats_case(a, r0, masked, drafted)
