"""GPU parity of cover_attn_rect (a block of query rows against all keys, the prefix-cache
form of Sec. 6.6) through the C ABI: each output row must equal the oracle's COVER attention
row at the same absolute position of the full-length problem (Sec. 5.1, App. B.1), within
the bf16 tolerance of the square kernel.  Cases: the LLaDA generated block, small blocks,
every key-split count regime (including splits with no keys), GQA, ragged lengths with
seeds on the first and last positions, seeds outside the block, every position a seed, the
whole sequence as the block, a single position, no seeds."""
import numpy as np
import pytest
import torch

import oracle
from helpers import announce, check_attn, to_dev
from paper_2602_06161_amd import cover, synth

pytestmark = pytest.mark.gpu


def _custom(seed, B, Hq, Hkv, L, n_seeds, positions=None):
    cfg = synth.AttnConfig("custom", B, Hq, Hkv, L, 128, "bf16", 0, L, n_seeds, "independent")
    a = synth.attn_inputs(cfg, seed=seed)
    if positions is not None:
        pos = np.array(sorted(positions), np.int32)
        a["seed_idx"] = torch.from_numpy(np.tile(pos, (B, 1)))
        a["n_seed"] = torch.full((B,), len(pos), dtype=torch.int32)
    return a


def _check(a, q_off, Lq, n_split=None, seeds=True, where=""):
    announce(f"rect {where} q_off={q_off} Lq={Lq} n_split={n_split}")
    q, kl, vl, kc, vc, si, ns = to_dev(a)
    if not seeds:
        si = ns = None
    qb = q[:, :, q_off:q_off + Lq].contiguous()
    out, lse = cover.cover_attn_rect(qb, kl, vl, kc, vc, q_off, si, ns, n_split=n_split)
    torch.cuda.synchronize()
    B, Hq, L, d = a["q"].shape
    rows = np.array([(b * Hq + h) * L + i for b in range(B) for h in range(Hq)
                     for i in range(q_off, q_off + Lq)], np.int64)
    osi = a["seed_idx"] if seeds else torch.zeros((B, 0), dtype=torch.int32)
    ons = a["n_seed"] if seeds else torch.zeros(B, dtype=torch.int32)
    ref_o, ref_l = oracle.attn(a["q"], a["k_live"], a["v_live"], a["k_cache"], a["v_cache"], osi,
                               ons, scale=a["scale"], mode="fast", rows=rows)
    check_attn(out, lse, ref_o.reshape(B, Hq, Lq, d), ref_l.reshape(B, Hq, Lq), torch.bfloat16,
               where)
    return out, lse


def test_llada_generated_block():
    a = synth.attn_inputs("llada", seed=0)
    _check(a, 768, 256, where="llada")


@pytest.mark.parametrize("q_off,Lq", [(800, 32), (896, 64), (768, 32), (992, 32)])
def test_small_blocks(q_off, Lq):
    a = synth.attn_inputs("llada", seed=1)
    _check(a, q_off, Lq, where="llada small block")


@pytest.mark.parametrize("n_split", [1, 3, 7, 32, 40])
def test_split_counts(n_split):
    # asked for; at 32 stages the launch uses one range whatever it is given (test_split_form has
    # shapes that use theirs, also with ranges without keys)
    a = synth.attn_inputs("llada", seed=2)
    _check(a, 768, 256, n_split=n_split, where="splits")


def test_gqa_dream_block():
    a = synth.attn_inputs("dream", seed=0)
    _check(a, 512, 256, where="dream")


def test_ragged_with_edge_seeds():
    a = _custom(3, 2, 4, 2, 1000, 0, positions=[5, 900, 910, 933, 976, 999])
    _check(a, 900, 77, n_split=3, where="ragged")
    _check(a, 923, 77, n_split=5, where="ragged block at the end")


def test_every_position_a_seed():
    a = _custom(4, 1, 2, 2, 256, 0, positions=list(range(256)))
    _check(a, 100, 100, where="all seeds")


def test_whole_sequence_matches_square_kernel():
    a = synth.attn_inputs("llada", seed=5)
    out, lse = _check(a, 0, 1024, where="whole sequence")
    q, kl, vl, kc, vc, si, ns = to_dev(a)
    sq, slse = cover.cover_attn_fwd(q, kl, vl, kc, vc, si, ns)
    torch.cuda.synchronize()
    assert (out.float() - sq.float()).abs().max().item() < 4e-2
    assert (lse - slse).abs().max().item() < 4e-2


def test_single_position_and_no_seeds():
    a = _custom(6, 1, 2, 2, 1, 0, positions=[0])
    _check(a, 0, 1, where="L=1 seed")
    a = synth.attn_inputs("llada", seed=7)
    _check(a, 768, 256, seeds=False, where="no seeds")


@pytest.mark.parametrize("case", ["llada256", "llada32", "llada64_896", "dream", "ragged",
                                  "ragged_end", "all_seeds", "short", "L1", "no_seeds",
                                  "long_seed_list", "batch_gqa"])
def test_single_launch_form(case):
    """n_split = 1: the single-launch kernel (key split across the waves of a workgroup,
    merged in LDS), on every case shape above plus short sequences (waves without stages)
    and seed lists longer than the part fetched into LDS."""
    if case == "llada256":
        _check(synth.attn_inputs("llada", seed=10), 768, 256, n_split=1, where=case)
    elif case == "llada32":
        _check(synth.attn_inputs("llada", seed=11), 992, 32, n_split=1, where=case)
    elif case == "llada64_896":
        _check(synth.attn_inputs("llada", seed=12), 896, 64, n_split=1, where=case)
    elif case == "dream":
        _check(synth.attn_inputs("dream", seed=13), 512, 256, n_split=1, where=case)
    elif case == "ragged":
        _check(_custom(14, 2, 4, 2, 1000, 0, positions=[5, 900, 910, 933, 976, 999]), 900, 77,
               n_split=1, where=case)
    elif case == "ragged_end":
        _check(_custom(15, 2, 4, 2, 1000, 0, positions=[0, 31, 32, 923, 999]), 923, 77,
               n_split=1, where=case)
    elif case == "all_seeds":
        _check(_custom(16, 1, 2, 2, 256, 0, positions=list(range(256))), 100, 100, n_split=1,
               where=case)
    elif case == "short":  # 4 stages for 8 waves; 3 stages, the last ragged
        _check(_custom(17, 1, 2, 1, 100, 0, positions=[3, 50, 99]), 40, 60, n_split=1, where=case)
        _check(_custom(18, 1, 2, 2, 70, 0, positions=[69]), 0, 70, n_split=1, where=case)
    elif case == "L1":
        _check(_custom(19, 1, 2, 2, 1, 0, positions=[0]), 0, 1, n_split=1, where=case)
    elif case == "no_seeds":
        _check(synth.attn_inputs("llada", seed=20), 768, 256, n_split=1, seeds=False, where=case)
    elif case == "long_seed_list":  # 700 seeds: 512 through LDS, the rest by plain loads
        rng = np.random.default_rng(21)
        pos = rng.choice(1024, size=700, replace=False)
        _check(_custom(21, 1, 2, 2, 1024, 0, positions=pos.tolist()), 600, 200, n_split=1,
               where=case)
    elif case == "batch_gqa":
        _check(_custom(22, 3, 8, 2, 640, 0, positions=[1, 100, 333, 500, 639]), 480, 160,
               n_split=1, where=case)


def test_single_launch_long_sequence():
    """The single launch at L = 4200 (132 stages of 32 keys, 16-17 per wave, the last ragged)
    with seeds in the first, middle and last stages and a block of 256 rows whose 256
    workgroups keep the single launch the default form."""
    pos = [0, 31, 1500, 2047, 2048, 2049, 3999, 4000, 4100, 4191, 4199]
    a = _custom(23, 1, 32, 32, 4200, 0, positions=pos)
    assert cover.rect_splits(1, 32, 256, 4200) == 1
    _check(a, 3944, 256, where="L4200 block at the end")
    _check(a, 1900, 64, n_split=1, where="L4200 middle block")


@pytest.mark.parametrize("n_split", [1, 3])
def test_distinct_seed_lists_per_batch_row(n_split):
    """Each batch row has its own seed list and count: none, a few in and out of the block,
    and a long list with entries past its count (padded with -1, ignored)."""
    L, ms = 700, 40
    cfg = synth.AttnConfig("custom", 3, 4, 2, L, 128, "bf16", 0, L, ms, "independent")
    a = synth.attn_inputs(cfg, seed=24)
    rng = np.random.default_rng(24)
    si = np.full((3, ms), -1, np.int32)
    counts = [0, 5, 33]
    si[1, :5] = [0, 333, 500, 517, 699]
    si[2, :33] = np.sort(rng.choice(L, size=33, replace=False))
    si[2, 33:] = rng.choice(L, size=ms - 33)  # past the count: must be ignored
    a["seed_idx"] = torch.from_numpy(si)
    a["n_seed"] = torch.tensor(counts, dtype=torch.int32)
    osi = torch.from_numpy(np.where(np.arange(ms)[None, :] < np.array(counts)[:, None], si, -1).astype(np.int32))
    q, kl, vl, kc, vc, sid, nsd = to_dev(a)
    q_off, Lq = 480, 150
    announce(f"rect distinct seeds per row n_split={n_split}")
    qb = q[:, :, q_off:q_off + Lq].contiguous()
    out, lse = cover.cover_attn_rect(qb, kl, vl, kc, vc, q_off, sid, nsd, n_split=n_split)
    torch.cuda.synchronize()
    B, Hq, _, d = a["q"].shape
    rows = np.array([(b * Hq + h) * L + i for b in range(B) for h in range(Hq)
                     for i in range(q_off, q_off + Lq)], np.int64)
    ref_o, ref_l = oracle.attn(a["q"], a["k_live"], a["v_live"], a["k_cache"], a["v_cache"], osi,
                               a["n_seed"], scale=a["scale"], mode="fast", rows=rows)
    check_attn(out, lse, ref_o.reshape(B, Hq, Lq, d), ref_l.reshape(B, Hq, Lq), torch.bfloat16,
               "distinct seeds")


@pytest.mark.parametrize("L,Lq,q_off,n_split,pos", [
    (2100, 77, 2023, 4, [0, 31, 32, 525, 1056, 2023, 2050, 2099]),     # the last range's last stage ragged
    (2100, 33, 700, 40, [699, 700, 710, 732, 2099]),                   # ranges without keys
    (2048, 8, 2040, 2, list(range(0, 2048, 3))),                       # a long seed list, every stage patched
    (3000, 1, 1500, 11, [1500]),                                       # one row, a seed
    (2500, 64, 0, 7, list(range(2500))),                               # every position a seed
    (5000, 100, 4000, 256, [4000 + 5 * i for i in range(20)])])
def test_split_form(L, Lq, q_off, n_split, pos):
    """Key ranges in separate workgroups and the merge, at shapes where the call uses the ranges
    it is given (from 48 stages of 32 keys two beat one), against the oracle and bit for bit
    against a second call."""
    a = _custom(L + n_split, 1, 2, 1, L, 0, positions=pos)
    out, lse = _check(a, q_off, Lq, n_split=n_split, where="split form")
    out2, lse2 = _check(a, q_off, Lq, n_split=n_split, where="split form again")
    assert torch.equal(out, out2) and torch.equal(lse, lse2)


def test_split_form_batch_and_heads():
    """Key ranges with several batch rows, grouped heads and a seed list of its own per row (one
    empty, one with entries past its count)."""
    B, Hq, Hkv, L, Lq, q_off, ms = 3, 4, 2, 2100, 20, 1990, 12
    a = synth.attn_inputs(synth.AttnConfig("custom", B, Hq, Hkv, L, 128, "bf16", 0, L, ms, "independent"), seed=31)
    rng = np.random.default_rng(31)
    si = np.sort(rng.choice(L, (B, ms), replace=False)).astype(np.int32)
    si[2, :4] = [0, 1990, 2001, 2099]
    counts = [0, ms, 4]
    a["seed_idx"], a["n_seed"] = torch.from_numpy(si), torch.tensor(counts, dtype=torch.int32)
    ignored = torch.from_numpy(np.where(np.arange(ms)[None] < np.array(counts)[:, None], si, -1).astype(np.int32))
    q, kl, vl, kc, vc, sid, nsd = to_dev(a)
    for n_split in (2, 4, 16):
        announce(f"rect split form batch n_split={n_split}")
        out, lse = cover.cover_attn_rect(q[:, :, q_off:q_off + Lq].contiguous(), kl, vl, kc, vc, q_off, sid, nsd,
                                         n_split=n_split)
        torch.cuda.synchronize()
        rows = np.array([(b * Hq + h) * L + i for b in range(B) for h in range(Hq)
                         for i in range(q_off, q_off + Lq)], np.int64)
        ref_o, ref_l = oracle.attn(a["q"], a["k_live"], a["v_live"], a["k_cache"], a["v_cache"], ignored,
                                   a["n_seed"], scale=a["scale"], mode="fast", rows=rows)
        check_attn(out, lse, ref_o.reshape(B, Hq, Lq, 128), ref_l.reshape(B, Hq, Lq), torch.bfloat16, str(n_split))


@pytest.mark.parametrize("B,Hq,L,Lq,n_split", [(1, 32, 2100, 64, 64), (2, 28, 1000, 100, 8), (4, 32, 700, 70, 3)])
def test_more_ranges_than_pay(B, Hq, L, Lq, n_split):
    """Calls that ask for more key ranges than finish soonest use fewer: same rows, and nothing
    outside the workspace they were given."""
    a = _custom(B + L, B, Hq, Hq // 4, L, 9)
    q, kl, vl, kc, vc, si, ns = to_dev(a)
    need = cover.rect_workspace(B, Hq, Lq, n_split)
    ws = torch.full((need + 4096,), 7.0, device="cuda")
    qb = q[:, :, L - Lq:].contiguous()
    announce(f"rect ranges B{B} Hq{Hq} L{L} Lq{Lq} n_split={n_split}")
    out, lse = cover.cover_attn_rect(qb, kl, vl, kc, vc, L - Lq, si, ns, n_split=n_split, workspace=ws[:need])
    one, one_lse = cover.cover_attn_rect(qb, kl, vl, kc, vc, L - Lq, si, ns, n_split=1)
    torch.cuda.synchronize()
    assert (ws[need:] == 7.0).all()
    # both round the same softmax to bf16 in their own order: 2^-8 of an output of up to 4
    assert (out.float() - one.float()).abs().max().item() < 2e-2
    assert (lse - one_lse).abs().max().item() < 1e-2


def test_workspace_smaller_than_the_default_splits():
    """A workspace of the caller's that holds fewer splits than rect_splits picks, as a plain call
    and with the arguments marshalled once."""
    B, Hq, Hkv, L, Lq = 2, 28, 4, 32768, 8
    announce("rect small workspace")
    g = torch.Generator(device="cuda").manual_seed(6)
    q = torch.randn(B, Hq, Lq, 128, generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(B, Hkv, L, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    ws = torch.full((cover.rect_workspace(B, Hq, Lq, 5) + 1024,), 7.0, device="cuda")
    out, lse = cover.cover_attn_rect(q, k, v, k, v, L - Lq, workspace=ws[:-1024])
    p = cover.PreparedRect(q, k, v, k, v, L - Lq, workspace=ws[:-1024])
    p()
    one, one_lse = cover.cover_attn_rect(q, k, v, k, v, L - Lq, n_split=1)
    torch.cuda.synchronize()
    assert p.n_split == 5 and torch.equal(p.out, out) and (ws[-1024:] == 7.0).all()
    assert (out.float() - one.float()).abs().max().item() < 2e-2  # as above
    assert (lse - one_lse).abs().max().item() < 1e-2


def test_rows_further_apart_than_32_bit_offsets():
    """Key rows 2^26 elements apart (the four K/V tensors interleaved in one buffer), with the key
    ranges that such strides need."""
    B, Hq, Hkv, L, Lq, d, gap = 1, 4, 2, 40, 20, 128, 1 << 26
    g = torch.Generator(device="cuda").manual_seed(4)
    buf = torch.empty((L - 1) * gap + 8 * d, device="cuda", dtype=torch.bfloat16)
    views = [torch.as_strided(buf, (B, Hkv, L, d), (0, d, gap, 1), 2 * d * i) for i in range(4)]
    plain = [torch.randn(B, Hkv, L, d, generator=g, device="cuda").bfloat16() for _ in range(4)]
    for v, p in zip(views, plain):
        v.copy_(p)
    q = torch.randn(B, Hq, Lq, d, generator=g, device="cuda").bfloat16()
    si = torch.tensor([[3, 25, 31, 32, 39]], device="cuda", dtype=torch.int32)
    ns = torch.tensor([5], device="cuda", dtype=torch.int32)
    for n_split in (2, 3):
        announce(f"rect wide rows n_split={n_split}")
        out, lse = cover.cover_attn_rect(q, views[0], views[1], views[2], views[3], 20, si, ns, n_split=n_split)
        want, want_lse = cover.cover_attn_rect(q, *plain, 20, si, ns, n_split=1)
        torch.cuda.synchronize()
        assert (out.float() - want.float()).abs().max().item() < 2e-2  # as above
        assert (lse - want_lse).abs().max().item() < 1e-2
    del buf, views
    torch.cuda.empty_cache()
