"""GPU parity of cover_attn_fwd (through the C ABI) against the fp64 oracle.

Bar: fp32 max-abs 1e-5; bf16 |gpu - oracle| <= 2e-2 + 1e-2 |oracle| on out and 2e-2 on lse.
Small shapes are compared on every row (several query/key tiles and a ragged tail), so are
sequences of more than 64 key stages with seeds in every stage window and seed lists longer
than the on-chip list; the LLaDA-8B and Dream-7B layer shapes are compared on every row and
the batched long-context shape on two whole batch rows, in the launch configuration the
benchmark times.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import announce, check_attn, to_dev
from paper_2602_06161_amd import cover, synth

pytestmark = pytest.mark.gpu


def _run(a, scale=None, **kw):
    q, kl, vl, kc, vc, si, ns = to_dev(a)
    out, lse = cover.cover_attn_fwd(q, kl, vl, kc, vc, si, ns, scale=scale or 0.0, **kw)
    torch.cuda.synchronize()
    return out, lse


def _oracle(a, scale=None, rows=None, mode="fast"):
    args = [a[k] for k in ("q", "k_live", "v_live", "k_cache", "v_cache", "seed_idx", "n_seed")]
    return oracle.attn(*args, scale=scale or a["scale"], mode=mode, rows=rows)


def _custom(seed, B, Hq, Hkv, L, d, n_seeds, dtype="bf16", positions=None, max_seeds=None):
    cfg = synth.AttnConfig("custom", B, Hq, Hkv, L, d, dtype, 0, L, n_seeds, "independent")
    a = synth.attn_inputs(cfg, seed=seed, max_seeds=max_seeds)
    if positions is not None:
        pos = np.array(sorted(positions), np.int32)
        si = np.full((B, max(len(pos), max_seeds or 0)), -1, np.int32)
        si[:, : len(pos)] = pos
        a["seed_idx"] = torch.from_numpy(si)
        a["n_seed"] = torch.full((B,), len(pos), dtype=torch.int32)
    return a


def test_tiny_f32_every_row():
    announce("tiny fp32 B1 H2 L64 d64, 4 seeds")
    a = synth.attn_inputs("tiny", seed=0)
    out, lse = _run(a)
    ref, lref = _oracle(a, mode="literal")
    check_attn(out, lse, ref, lref, torch.float32, "tiny")


@pytest.mark.parametrize("shape", [(2, 4, 2, 150, 128, 7), (1, 3, 1, 97, 64, 30), (1, 1, 1, 1, 128, 1)])
def test_f32_multi_tile_ragged(shape):
    B, Hq, Hkv, L, d, n = shape
    announce(f"fp32 B{B} Hq{Hq} Hkv{Hkv} L{L} d{d} seeds{n}")
    a = _custom(1, B, Hq, Hkv, L, d, n, dtype="f32")
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.float32, str(shape))


@pytest.mark.parametrize("L,d,n", [(15, 64, 3), (16, 128, 16), (17, 64, 2), (33, 128, 5), (127, 64, 9),
                                   (129, 128, 20), (260, 64, 700)])
def test_f32_tile_edges(L, d, n):
    """One to eight waves per workgroup, whole and partial 16-row tiles, second tiles of a wave,
    and a seed list longer than the positions fetched with its count."""
    announce(f"fp32 L{L} d{d} seeds{n}")
    a = _custom(L, 1, 2, 1, L, d, min(n, L), dtype="f32")
    if n > L:  # the list's tail: entries outside [0, L), ignored
        junk = torch.full((1, n - L), L + 7, dtype=torch.int32)
        a["seed_idx"] = torch.cat([junk, a["seed_idx"][:, :L]], 1).contiguous()
        a["n_seed"] = torch.full((1,), n, dtype=torch.int32)
    out, lse = _run(a)
    if n > L:
        a["seed_idx"], a["n_seed"] = a["seed_idx"][:, n - L:].contiguous(), torch.full((1,), L, dtype=torch.int32)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.float32, f"L{L} d{d}")


@pytest.mark.parametrize("B,L,d,n", [(43, 33, 64, 3), (33, 49, 128, 9), (64, 17, 64, 17), (8, 250, 64, 30)])
def test_f32_one_wave_per_workgroup(B, L, d, n):
    """From 2048 query tiles on one wave walks all key tiles: whole and ragged, seeds in any."""
    announce(f"fp32 one wave B{B} L{L} d{d} seeds{n}")
    a = _custom(L + d, B, 16, 4, L, d, n, dtype="f32")
    assert B * 16 * -(-L // 16) >= 2048
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.float32, f"B{B} L{L} d{d}")


def test_f32_more_tiles_than_workgroups():
    """Past 2^20 query tiles a workgroup takes several: one-token sequences, whose output is
    their own value row."""
    announce("fp32 B2^20+5 L1")
    B = (1 << 20) + 5
    x = torch.randn(B, 1, 1, 64, device="cuda")
    out, lse = cover.cover_attn_fwd(x, x, x, x, x)
    torch.cuda.synchronize()
    assert torch.equal(out, x)
    want = (x.double() ** 2).sum(-1) / 8.0
    assert torch.allclose(lse.double(), want, rtol=1e-5, atol=1e-5)


BF16_SHAPES = [
    (1, 2, 2, 64, 128, 4),
    (2, 4, 2, 300, 128, 12),
    (1, 4, 4, 200, 64, 20),
    (1, 2, 1, 129, 128, 40),
    (2, 3, 3, 45, 64, 5),
    (1, 1, 1, 1, 128, 1),
    (1, 7, 1, 520, 128, 33),
]


@pytest.mark.parametrize("shape", BF16_SHAPES, ids=[str(s) for s in BF16_SHAPES])
def test_bf16_every_row(shape):
    B, Hq, Hkv, L, d, n = shape
    announce(f"bf16 B{B} Hq{Hq} Hkv{Hkv} L{L} d{d} seeds{n}")
    a = _custom(2, B, Hq, Hkv, L, d, n)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, str(shape))


def test_bf16_seeds_on_every_diagonal_block():
    # each wave's diagonal block: workgroup halves x key parities, plus tile edges
    pos = [0, 5, 31, 32, 63, 64, 100, 127, 128, 150, 191, 192, 255]
    announce(f"bf16 diagonal blocks L256 seeds {pos}")
    a = _custom(3, 1, 2, 2, 256, 128, 0, positions=pos)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, "diag-blocks")


@pytest.mark.parametrize("d", [64, 128])
def test_bf16_every_position_a_seed(d):
    announce(f"bf16 all positions seeds L96 d{d}")
    a = _custom(4, 1, 2, 2, 96, d, 0, positions=range(96))
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, "all-seeds")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("L,n,layout,late", [(1, 1, "head", False), (32, 17, "head", False), (64, 40, "token", False),
                                             (65, 3, "head", False), (193, 100, "head", False),
                                             (449, 25, "token", True), (577, 200, "head", True)])
def test_bf16_edges_of_both_kernels(d, many, L, n, layout, late):
    """Up to 256 tiles of 32 query rows a call runs on the block kernel, beyond (many) on the
    four-wave kernel: whole and ragged stages and query tiles, one to eighteen stages, tiles with
    more and fewer than 16 seed rows, grouped heads, token-major strides, and (late) scores that
    outgrow the first stage's by more than 2^24 (rescaled, or the tile computed again)."""
    per = -(-L // 32)
    Hq = 2 * (128 // per + 1) if many else 2
    assert (Hq * per > 256) == many
    announce(f"bf16 d{d} Hq{Hq} L{L} seeds{n} {layout} late {late}")
    a = _custom(L, 1, Hq, Hq // 2, L, d, n)
    if late:
        for k in ("k_live", "k_cache"):
            a[k][:, :, 3 * L // 4:] *= 40.0
    if layout == "token":
        for k in ("q", "k_live", "v_live", "k_cache", "v_cache"):
            a[k] = a[k].transpose(1, 2).contiguous().transpose(1, 2)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    assert not late or np.abs(lref).max() > 30
    check_attn(out, lse, ref, lref, torch.bfloat16, f"d{d} L{L} many {many}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,n,how", [(1001, 24, "rise"), (1001, 24, "one"), (1024, 0, "fall"), (700, 700, "rise"),
                                     (640, 130, "first")])
def test_bf16_scores_outgrow_the_reference(d, L, n, how):
    """Scores that rise from stage to stage by more than the reference maximum tolerates, in every
    row or in one head's last stages only, or fall; every position a seed (the cached diagonal,
    which must not move the reference, the largest score); and a first stage far below the rest."""
    announce(f"bf16 d{d} L{L} seeds{n} scores {how}")
    a = _custom(L, 1, 16, 4, L, d, n)
    up = torch.linspace(0, 40, L)[:, None]
    lift = {"rise": up, "fall": up.flip(0), "one": torch.where(up > 35, 30.0, 0.0),
            "first": torch.where(torch.arange(L)[:, None] < 64, -80.0, 0.0)}[how]
    direction = torch.nn.functional.normalize(torch.ones(d), dim=0)
    heads = slice(0, 1) if how == "one" else slice(None)
    for k in ("k_live", "k_cache"):
        a[k] = a[k].float()
        a[k][:, heads] += lift * direction * d ** 0.5 / 4
        a[k] = a[k].bfloat16()
    a["q"] = (a["q"].float() * 0.5 + 4 * direction).bfloat16()
    if n == L:  # a seed's own cached key, which its row does not see, above everything else
        a["k_cache"] = (a["k_cache"].float() + 3 * direction).bfloat16()
    out, lse = _run(a)
    ref, lref = _oracle(a)
    # the lse of scores in the hundreds: bf16 scores' fp32 sums, 2^-22 of their size on top
    check_attn(out, None, ref, None, torch.bfloat16, f"d{d} {how}")
    err = np.abs(lse.double().cpu().numpy().reshape(lref.shape) - lref)
    assert (err <= 2e-2 + 2.0**-20 * np.abs(lref)).all()


def test_zero_seeds_and_no_seed_arrays():
    announce("bf16 zero seeds / max_seeds 0")
    a = _custom(5, 1, 4, 2, 200, 128, 6)
    a["n_seed"][:] = 0
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, "n_seed=0")
    q, kl, vl, kc, vc, _, _ = to_dev(a)
    out2, lse2 = cover.cover_attn_fwd(q, kl, vl, kc, vc)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


def test_nonseed_cache_rows_are_never_read():
    announce("bf16 non-seed cache rows = NaN")
    a = _custom(6, 2, 4, 2, 256, 128, 10)
    out, lse = _run(a)
    b2 = dict(a)
    kc, vc = a["k_cache"].clone(), a["v_cache"].clone()
    for b in range(2):
        non = np.setdiff1d(np.arange(256), a["seed_idx"][b, : a["n_seed"][b]].numpy())
        kc[b][:, non] = float("nan")
        vc[b][:, non] = float("inf")
    b2["k_cache"], b2["v_cache"] = kc, vc
    out2, lse2 = _run(b2)
    assert torch.isfinite(out2.float()).all()
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


def test_out_of_range_entries_are_ignored():
    announce("bf16 seed lists with entries outside [0, L); a row with none inside")
    L = 200
    a = _custom(16, 2, 4, 2, L, 128, 0, max_seeds=8)
    si = np.array([[-7, 5, L, 130, L + 1000, 64, -1, 199],
                   [-1, L, L + 3, -100, 0, 0, 0, 0]], np.int32)
    ns = np.array([8, 4], np.int32)
    kept = [[5, 130, 64, 199], []]
    a["seed_idx"], a["n_seed"] = torch.from_numpy(si), torch.from_numpy(ns)
    kc, vc = a["k_cache"].clone(), a["v_cache"].clone()
    for b in range(2):   # cache rows that are not seeds must never be read
        non = np.setdiff1d(np.arange(L), kept[b])
        kc[b][:, non] = float("nan")
        vc[b][:, non] = float("inf")
    a["k_cache"], a["v_cache"] = kc, vc
    out, lse = _run(a)
    assert torch.isfinite(out.float()).all()
    ref_in = dict(a)
    rsi = np.full((2, 4), -1, np.int32)
    rsi[0] = kept[0]
    ref_in["seed_idx"] = torch.from_numpy(rsi)
    ref_in["n_seed"] = torch.tensor([4, 0], dtype=torch.int32)
    ref, lref = _oracle(ref_in)
    check_attn(out, lse, ref, lref, torch.bfloat16, "out-of-range entries")


def test_seed_row_ignores_its_own_cached_kv():
    announce("bf16 perturb one seed's own cached K/V")
    a = _custom(7, 1, 2, 2, 256, 128, 9)
    out, lse = _run(a)
    i = int(a["seed_idx"][0, 3])
    b2 = dict(a)
    kc, vc = a["k_cache"].clone(), a["v_cache"].clone()
    kc[0, :, i] += 3.0
    vc[0, :, i] -= 2.0
    b2["k_cache"], b2["v_cache"] = kc, vc
    out2, lse2 = _run(b2)
    assert torch.equal(out[0, :, i], out2[0, :, i]) and torch.equal(lse[0, :, i], lse2[0, :, i])
    others = [j for j in range(256) if j != i]
    assert not torch.equal(out[0][:, others], out2[0][:, others])


def test_repeat_runs_bitwise_equal():
    announce("bf16 determinism")
    a = synth.attn_inputs("llada", seed=1)
    o1, l1 = _run(a)
    o2, l2 = _run(a)
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


def test_dominant_cached_diagonal():
    # Cached diagonal keys aligned with their own query: alpha_i -> 1, the regime where the
    # post-hoc closed form cancels; the in-softmax substitution must still match.
    announce("bf16 dominant cached diagonal")
    a = _custom(8, 1, 2, 2, 192, 128, 16)
    kc = a["k_cache"].float()
    q = a["q"].float()
    for i in a["seed_idx"][0, : a["n_seed"][0]].tolist():
        for h in range(2):
            qi = q[0, h, i]
            kc[0, h, i] = 8.0 * qi / qi.norm() * np.sqrt(128)
    a["k_cache"] = kc.to(torch.bfloat16)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, "dominant-diag")


def test_peaky_scores_force_rescaling():
    announce("bf16 scale 1.0 (peaky rows)")
    a = _custom(9, 1, 2, 1, 384, 128, 12)
    out, lse = _run(a, scale=1.0)
    ref, lref = _oracle(a, scale=1.0)
    check_attn(out, lse, ref, lref, torch.bfloat16, "scale=1")


def test_strided_token_major_layout():
    announce("bf16 [B,L,H,d] strided views")
    a = _custom(10, 2, 4, 2, 160, 128, 8)
    q, kl, vl, kc, vc, si, ns = to_dev(a)
    t = lambda x: x.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)  # same values, token-major
    qs, kls, vls, kcs, vcs = map(t, (q, kl, vl, kc, vc))
    assert qs.stride(2) == 4 * 128
    out, lse = cover.cover_attn_fwd(qs, kls, vls, kcs, vcs, si, ns)
    torch.cuda.synchronize()
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, "strided")


def _sample_rows(a, rng, heads_per_batch=None, n_random=256):
    c = a["cfg"]
    rows = []
    for b in range(c.B):
        heads = range(c.Hq) if heads_per_batch is None else rng.choice(c.Hq, heads_per_batch, replace=False)
        for h in heads:
            for i in a["seed_idx"][b, : a["n_seed"][b]].tolist():
                rows.append((b * c.Hq + h) * c.L + i)
    rows += rng.integers(0, c.B * c.Hq * c.L, n_random).tolist()
    return np.unique(np.array(rows, np.int64))


@pytest.mark.parametrize("name,hpb", [("llada", None), ("dream", None), ("batched", 4)])
def test_full_size_config_sampled_rows(name, hpb):
    announce(f"{name} full size, sampled rows")
    a = synth.attn_inputs(name, seed=0)
    out, lse = _run(a)
    rows = _sample_rows(a, np.random.default_rng(0), hpb)
    ref, lref = _oracle(a, rows=rows)
    c = a["cfg"]
    o = out.reshape(-1, c.d)[torch.from_numpy(rows).cuda()]
    l = lse.reshape(-1)[torch.from_numpy(rows).cuda()]
    check_attn(o, l, ref, lref, torch.bfloat16, name)
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()


def _explicit(seed, B, Hq, Hkv, L, d, per_row, max_seeds=None):
    """Inputs with an explicit seed list per batch row (per_row[b]: positions, any order)."""
    cfg = synth.AttnConfig("custom", B, Hq, Hkv, L, d, "bf16", 0, L, 0, "independent")
    a = synth.attn_inputs(cfg, seed=seed, max_seeds=0)
    ms = max_seeds if max_seeds is not None else max(len(p) for p in per_row)
    si = np.full((B, ms), -1, np.int32)
    ns = np.zeros((B,), np.int32)
    for b, pos in enumerate(per_row):
        pos = np.array(sorted(set(int(x) for x in pos)), np.int32)
        assert pos.size <= ms and (pos.size == 0 or (pos[0] >= 0 and pos[-1] < L))
        si[b, : pos.size] = pos
        ns[b] = pos.size
    a["seed_idx"], a["n_seed"] = torch.from_numpy(si), torch.from_numpy(ns)
    return a


def _stage_spanning_seeds(L, rng, extra=0):
    """Seeds on the first and last rows of stages 0, 31, 32, 33, 63, 64, 65 (64 keys per stage;
    those that exist below L), the last position, plus `extra` random positions."""
    pos = {0, L - 1}
    for s in (0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 127, 128):
        for r in (0, 17, 63):
            if s * 64 + r < L:
                pos.add(s * 64 + r)
    if extra:
        pos |= set(rng.choice(L, size=extra, replace=False).tolist())
    return sorted(pos)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("L", [4200, 8200])
def test_long_sequence_every_row(L, d):
    """More than 64 key stages (the per-stage seed windows are refreshed every 32 stages and
    looked up past stage 64), a ragged last stage (4200 = 65 x 64 + 40; 8200 = 128 x 64 + 8),
    seeds in stages 0..128 including the last position, and a second batch row with its own
    seed set."""
    rng = np.random.default_rng(L + d)
    rows = [_stage_spanning_seeds(L, rng), rng.choice(L, size=40, replace=False)]
    Hq = 2 if L < 8000 else 1
    announce(f"bf16 long sequence B2 Hq{Hq} Hkv1 L{L} d{d}, {len(rows[0])}/40 seeds")
    a = _explicit(20 + L, 2, Hq, 1, L, d, rows)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, f"long L{L} d{d}")


@pytest.mark.parametrize("d", [128, 64])
def test_more_than_256_seeds(d):
    """Seed lists longer than the 256 entries staged on chip (the rest is read from memory):
    300 and 257 seeds in two batch rows, over more than 64 stages in the first."""
    rng = np.random.default_rng(300 + d)
    rows = [rng.choice(4200, size=300, replace=False), rng.choice(2000, size=257, replace=False)]
    announce(f"bf16 B2 Hq4 Hkv2 L4200 d{d}, 300 / 257 seeds")
    a = _explicit(31 + d, 2, 4, 2, 4200, d, rows, max_seeds=320)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, f"300 seeds d{d}")


@pytest.mark.parametrize("name", ["llada", "dream"])
def test_full_size_config_every_row(name):
    """Every output row of the LLaDA-8B and Dream-7B layer shapes against the oracle, in the
    launch configuration the benchmark times."""
    announce(f"{name} full size, every row")
    a = synth.attn_inputs(name, seed=0)
    out, lse = _run(a)
    ref, lref = _oracle(a)
    check_attn(out, lse, ref, lref, torch.bfloat16, name)


def test_batched_whole_batch_rows():
    """Two whole batch rows (all 32 heads x 2048 positions each) of the batched long-context
    shape, each batch row with its own 64 seeds."""
    announce("batched B8 H32 L2048, batch rows 0 and 5 whole")
    a = synth.attn_inputs("batched", seed=0)
    out, lse = _run(a)
    c = a["cfg"]
    per = c.Hq * c.L
    rows = np.concatenate([np.arange(b * per, (b + 1) * per, dtype=np.int64) for b in (0, 5)])
    ref, lref = _oracle(a, rows=rows)
    o = out.reshape(-1, c.d)[torch.from_numpy(rows).cuda()]
    l = lse.reshape(-1)[torch.from_numpy(rows).cuda()]
    check_attn(o, l, ref, lref, torch.bfloat16, "batched rows 0, 5")
