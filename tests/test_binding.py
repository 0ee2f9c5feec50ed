"""The calls' native forms (csrc/host.cpp) against their Python forms: the same outputs bit for
bit, caller-given outputs returned as the same objects, and the same errors.  A torch function
mode (here a default device) sends a call to its Python form."""
import pytest
import torch

from helpers import announce
from paper_2602_06161_amd import cover


def test_native_forms_leave_what_is_out_of_the_ordinary():
    """CPU tensors, non-tensors, subclasses and wrong argument counts are handed back (None);
    nothing is enqueued and no error is left behind."""
    h = cover.host()
    x = torch.zeros(2, 8)
    t = torch.zeros(2, dtype=torch.int32)
    assert h.token_stats(x, t, True, True, True, 0) is None
    assert h.token_stats("x", None, False, True, True, 0) is None
    assert h.token_stats() is None
    assert h.token_sample(x, "hot", 1, 1, True, 0) is None
    with pytest.raises(ValueError):
        cover.cover_token_stats(x, t[:1])
    with pytest.raises(TypeError):
        h.bind(1)
    with pytest.raises(ValueError):
        h.bind(0, 0, 0, 0, 0, 0, 0)


def _problem(layout):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    B, Hq, Hkv, L, d, gen = 2, 4, 2, 90, 64, 40

    def r(H):
        if layout == "token":
            return torch.randn(B, L, H, d, generator=g, device="cuda").bfloat16().transpose(1, 2)
        return torch.randn(B, H, L, d, generator=g, device="cuda").bfloat16()

    q, k, v, kc, vc = r(Hq), r(Hkv), r(Hkv), r(Hkv), r(Hkv)
    si = torch.tensor([[52, 60, 89], [51, 70, 71]], device="cuda", dtype=torch.int32)
    ns = torch.tensor([3, 2], device="cuda", dtype=torch.int32)
    lse = torch.full((B, Hq, L), 5.0, device="cuda")
    masked = (torch.rand(B, gen, generator=g, device="cuda") < 0.5).to(torch.uint8)
    drafted = masked * (torch.rand(B, gen, generator=g, device="cuda") < 0.3).to(torch.uint8)
    logits = torch.randn(B * gen, 1000, generator=g, device="cuda")[:, :997]
    logits_bf16 = torch.randn(B * gen, 1000, generator=g, device="cuda").bfloat16()[:, :993]
    toks = torch.randint(0, 900, (B, gen), generator=g, device="cuda", dtype=torch.int32)
    conf = torch.rand(B, gen, generator=g, device="cuda")
    top = torch.randint(0, 900, (B, gen), generator=g, device="cuda", dtype=torch.int32)
    return locals()


def _calls(p):
    """name -> a call of the binding's function on fresh copies of what it updates in place."""
    B, gen, L = p["B"], p["gen"], p["L"]
    flags = torch.ones(B, gen, device="cuda", dtype=torch.uint8)
    att = (p["q"], p["k"], p["v"], p["kc"], p["vc"])
    mass = (p["q"], p["k"], p["kc"], p["si"], p["ns"], p["lse"], p["masked"], p["drafted"], L - gen)

    def update(seeds):
        t, rm = p["toks"].clone(), torch.zeros_like(p["toks"])
        s = (p["si"], p["ns"]) if seeds else (None, None)
        return (t, rm) + tuple(cover.cover_decode_update(t, p["top"], p["conf"], *s, rm, 7, 0.5, 4, 3, L - gen))

    return {
        "fwd": lambda: cover.cover_attn_fwd(*att, p["si"], p["ns"]),
        "fwd_plain": lambda: cover.cover_attn_fwd(*att, scale=0.2, want_lse=False),
        "stats": lambda: cover.cover_token_stats(p["logits"], p["toks"].reshape(-1)),
        "stats_conf": lambda: cover.cover_token_stats(p["logits_bf16"], want_logp=False),
        "sample": lambda: cover.cover_token_sample(p["logits"], 0.7, -3, 2**33 + 1),
        "sample_token": lambda: cover.cover_token_sample(p["logits"], 1, 9, 0, want_prob=False),
        "masses": lambda: cover.cover_attn_stats(*mass),
        "masses_scaled": lambda: cover.cover_attn_stats(*mass[:3], None, None, *mass[5:], scale=0.3),
        "select": lambda: cover.cover_select_seeds(-p["conf"], p["conf"], p["conf"], flags, 5, L - gen),
        "select_plain": lambda: cover.cover_select_seeds(-p["conf"], p["conf"], p["conf"], flags, 5, want_score=False),
        "update": lambda: update(True),
        "update_noseeds": lambda: update(False),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["head", "token"])
def test_native_and_python_forms_agree(layout):
    p = _problem(layout)
    for name, call in _calls(p).items():
        announce(f"binding {name} {layout}")
        native = call()
        with torch.device("cuda"):
            python = call()
        torch.cuda.synchronize()
        assert len(native) == len(python), name
        for a, b in zip(native, python):
            assert (a is None) == (b is None), name
            if a is not None:
                assert a.shape == b.shape and a.stride() == b.stride() and a.dtype == b.dtype and a.device == b.device
                if name == "select" or name == "select_plain":
                    a, b = a[..., :5], b[..., :5]
                assert torch.equal(a, b), name


@pytest.mark.gpu
def test_given_outputs_and_streams():
    announce("binding given outputs, another stream")
    p = _problem("head")
    want, wl = cover.cover_attn_fwd(p["q"], p["k"], p["v"], p["kc"], p["vc"], p["si"], p["ns"])
    out, lse = torch.empty_like(want), torch.empty_like(wl)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a, b = cover.cover_attn_fwd(p["q"], p["k"], p["v"], p["kc"], p["vc"], p["si"], p["ns"], out=out, lse=lse)
    s.synchronize()
    assert a is out and b is lse and torch.equal(out, want) and torch.equal(lse, wl)
    out.zero_()
    torch.cuda.synchronize()
    cover.cover_attn_fwd(p["q"], p["k"], p["v"], p["kc"], p["vc"], p["si"], p["ns"], out=out, lse=lse, stream=s)
    s.synchronize()
    assert torch.equal(out, want)


@pytest.mark.gpu
@pytest.mark.parametrize("python_form", [False, True])
def test_errors_are_the_same(python_form):
    announce(f"binding errors, python form {python_form}")
    p = _problem("head")
    q, k, v, kc, vc, si, ns = (p[n] for n in ("q", "k", "v", "kc", "vc", "si", "ns"))
    x, toks = p["logits"], p["toks"].reshape(-1)
    bad = [
        (ValueError, lambda: cover.cover_attn_fwd(q, k, v[:, :1], kc, vc)),
        (ValueError, lambda: cover.cover_attn_fwd(q, k, v, kc, vc, si.long(), ns)),
        (ValueError, lambda: cover.cover_attn_fwd(q, k, v, kc, vc, out=torch.empty_like(q).float())),
        (TypeError, lambda: cover.cover_attn_fwd(*(t.half() for t in (q, k, v, kc, vc)))),
        (cover.CoverError, lambda: cover.cover_attn_fwd(q, k, v, kc, vc, scale=-1.0)),
        (ValueError, lambda: cover.cover_token_stats(x.double())),
        (ValueError, lambda: cover.cover_token_stats(x, toks.long())),
        (cover.CoverError, lambda: cover.cover_token_stats(torch.randn(4, 997, device="cuda"), toks[:4])),
        (cover.CoverError, lambda: cover.cover_token_sample(x, 0.0, 1, 1)),
        (ValueError, lambda: cover.cover_attn_stats(q, k, kc, si, ns, p["lse"][:, :1], p["masked"], p["drafted"], 50)),
        (ValueError, lambda: cover.cover_attn_stats(q, k, kc, si, ns, p["lse"], p["masked"], p["drafted"], 50,
                                                    workspace=torch.empty(1, device="cuda"))),
        (cover.CoverError, lambda: cover.cover_attn_stats(q, k, kc, si, ns, p["lse"], p["masked"], p["drafted"], 51)),
        (ValueError, lambda: cover.cover_select_seeds(x, x, x, x, 3)),
        (cover.CoverError, lambda: cover.cover_select_seeds(*(p["conf"],) * 3, p["masked"], 3, 2**31 - 1)),
        (ValueError, lambda: cover.cover_decode_update(p["toks"], p["top"], p["conf"].double(), si, ns, p["toks"], 7,
                                                       0.5, 4, 3)),
        (cover.CoverError, lambda: cover.cover_decode_update(p["toks"], p["top"], p["conf"], si, ns,
                                                             torch.zeros_like(p["toks"]), 7, 0.5, 4, 3, min_draft=5)),
    ]
    for kind, call in bad:
        with pytest.raises(kind):
            if python_form:
                with torch.device("cuda"):
                    call()
            else:
                call()
