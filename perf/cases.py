"""The calls whose speed this library is judged by, as a program that decodes with it makes them.

Five kinds, over the ranges that the library's configurations, tests and benchmark use:
  attn    one layer's override attention (cover_attn_fwd), optionally with the seed selection
          that ends a step; bf16 with head size 128 or 64, and fp32; head-major tensors
          ([B,H,L,d] contiguous, arguments marshalled once) or token-major ones ([B,L,H,d], as
          a projection writes them, through the plain call)
  block   the same attention for one block of query rows against all keys (cover_attn_rect)
  token   statistics of the LM head's logits: log p, confidence, argmax (cover_token_stats), or
          temperature sampling (cover_token_sample)
  masses  in/out attention masses of the generated region (cover_attn_stats)
  tail    everything a decoding step does after the model: confidence and draft token, state
          update, log p of the tokens now in place, attention masses, seed selection
"""
import math

import torch

from paper_2602_06161_amd import cover

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _attn(name, B, Hq, Hkv, L, d, seeds, dtype="bf16", layout="head", gen=256, select=False):
    return {"name": name, "kind": "attn", "B": B, "Hq": Hq, "Hkv": Hkv, "L": L, "d": d, "seeds": seeds,
            "dtype": dtype, "layout": layout, "gen": gen, "select": select}


def _block(name, B, Hq, Hkv, L, Lq, q_off, seeds):
    return {"name": name, "kind": "block", "B": B, "Hq": Hq, "Hkv": Hkv, "L": L, "d": 128, "seeds": seeds,
            "dtype": "bf16", "Lq": Lq, "q_off": q_off}


def _token(name, op, R, V, dtype="bf16", T=0.0):
    return {"name": name, "kind": "token", "op": op, "R": R, "V": V, "dtype": dtype, "T": T}


def _masses(name, B, Hq, Hkv, L, d, gen, seeds):
    return {"name": name, "kind": "masses", "B": B, "Hq": Hq, "Hkv": Hkv, "L": L, "d": d, "gen": gen,
            "seeds": seeds, "dtype": "bf16"}


def _tail(name, Hq, Hkv, L, gen, V, seeds):
    return {"name": name, "kind": "tail", "B": 1, "Hq": Hq, "Hkv": Hkv, "L": L, "d": 128, "gen": gen, "V": V,
            "seeds": seeds, "dtype": "bf16"}


def listed():
    return [
        # the smallest call: an fp32 layer of a few tokens, as an integration checks itself with
        _attn("attn_f32_small", 1, 2, 2, 64, 64, 4, dtype="f32", gen=64),
        # the step of the benchmark: one LLaDA-8B layer's attention and the selection
        _attn("step_llada", 1, 32, 32, 1024, 128, 16, select=True),
        # a grouped-query layer (Dream-7B) inside a model: token-major projections
        _attn("attn_dream", 1, 28, 4, 768, 128, 32, layout="token"),
        # a serving batch of long responses: the largest call
        _attn("attn_batched", 8, 32, 32, 2048, 128, 64, gen=512),
        # head size 64, a length that fills no tile
        _attn("attn_d64_ragged", 4, 16, 16, 1001, 64, 24),
        # prefix-cache decoding: one 64-token block, and the whole generated block
        _block("block_64", 1, 32, 32, 1024, 64, 832, 16),
        _block("block_256", 1, 32, 32, 1024, 256, 768, 16),
        # the same behind a long prompt, a grouped-query model's small block
        _block("block_long", 1, 32, 8, 8192, 64, 8064, 16),
        # the LM head's logits of the generated block (LLaDA-8B vocabulary)
        _token("token_stats", "stats", 256, 126464),
        # stochastic decoding's draw from the same logits
        _token("token_sample", "sample", 256, 126464, T=0.3),
        # attention masses of the generated region of a serving batch
        _masses("masses_batched", 8, 32, 32, 2048, 128, 512, 64),
        # what follows the model in every step
        _tail("step_tail", 32, 32, 1024, 256, 126464, 16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    heads = [(32, 32), (28, 4), (32, 8), (16, 16), (12, 12), (40, 8)]
    kind = rng.choice(["attn", "attn", "attn", "block", "block", "token", "token", "masses", "tail"])
    if kind == "attn" and rng.random() < 0.15:
        L = _log_int(rng, 40, 640)
        c = _attn("", rng.randint(1, 2), *rng.choice([(2, 2), (4, 2), (8, 8)]), L, rng.choice([64, 128]),
                  rng.randint(0, min(16, L // 8)), dtype="f32", gen=min(L, 64))
    elif kind == "attn":
        Hq, Hkv = rng.choice(heads)
        L = _log_int(rng, 100, 3000)
        most = 8 * 32 * 2048 * 2048 / (Hq * L * L)  # no larger than the largest listed
        B = _log_int(rng, 1, max(1, min(8, int(most))))
        gen = min(L, rng.choice([64, 128, 256, 512]))
        c = _attn("", B, Hq, Hkv, L, rng.choice([128, 128, 64]), rng.randint(0, min(64, gen // 4)),
                  layout=rng.choice(["head", "token"]), gen=gen, select=rng.random() < 0.4)
    elif kind == "block":
        Hq, Hkv = rng.choice(heads)
        L = _log_int(rng, 256, 16384)
        Lq = min(L, _log_int(rng, 8, 256))
        B = rng.randint(1, 2)
        c = _block("", B, Hq, Hkv, L, Lq, L - Lq - rng.randint(0, min(L - Lq, 128)), rng.randint(0, 32))
    elif kind == "token":
        op = rng.choice(["stats", "sample"])
        c = _token("", op, _log_int(rng, 16, 512), _log_int(rng, 8000, 160000), rng.choice(["bf16", "bf16", "f32"]),
                   round(rng.uniform(0.1, 1.0), 2) if op == "sample" else 0.0)
    elif kind == "masses":
        Hq, Hkv = rng.choice(heads)
        gen = _log_int(rng, 64, 768)
        c = _masses("", rng.randint(1, 8), Hq, Hkv, gen + _log_int(rng, 16, 1500), rng.choice([128, 128, 64]), gen,
                    rng.randint(0, gen // 8))
    else:
        Hq, Hkv = rng.choice(heads)
        gen = _log_int(rng, 64, 512)
        c = _tail("", Hq, Hkv, gen + _log_int(rng, 16, 1500), gen, _log_int(rng, 30000, 160000), rng.randint(4, 32))
    del c["name"]
    return c


# ---- inputs ----------------------------------------------------------------------------------
def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)


def _unmasked(g, B, gen):
    """Half of the generated positions, per row: bool [B, gen]."""
    rank = torch.rand(B, gen, generator=g, device="cuda").argsort(1).argsort(1)
    return rank < max(1, gen // 2)


def _seed_lists(g, unmasked, first, n):
    """n seeds per row among the unmasked generated positions, ascending: int32 [B, n], [B]."""
    B, gen = unmasked.shape
    n = min(n, max(1, gen // 2))
    if n == 0:
        return None, None
    key = torch.rand(B, gen, generator=g, device="cuda").masked_fill(~unmasked, 2.0)
    idx = key.argsort(1)[:, :n].sort(1).values + first
    return idx.to(torch.int32).contiguous(), torch.full((B,), n, device="cuda", dtype=torch.int32)


def _layer(c, g):
    """q, live and cached k/v of one layer and the seeds.  The caches differ from the live states
    by a tenth of their spread, as one decoding step moves them."""
    B, Hq, Hkv, L, d = (c[k] for k in ("B", "Hq", "Hkv", "L", "d"))
    dt = TORCH[c["dtype"]]
    gen = min(c.get("gen", 256), L)

    def tensor(H, n):
        if c.get("layout") == "token":
            return _normal(g, B, n, H, d, dtype=dt).transpose(1, 2)
        return _normal(g, B, H, n, d, dtype=dt)

    s = {"q": tensor(Hq, c.get("Lq", L)), "k": tensor(Hkv, L), "v": tensor(Hkv, L)}
    for x in ("k", "v"):
        s[x + "c"] = s[x] + 0.1 * tensor(Hkv, L)
    um = _unmasked(g, B, gen)
    s["seed_idx"], s["n_seed"] = _seed_lists(g, um, L - gen, c["seeds"])
    s["unmasked"], s["first"], s["gen"] = um, L - gen, gen
    return s


def _select_inputs(c, g, s):
    """Selection inputs of the generated region: Beta(5, 1) confidences, masses of N(0, 1)
    attention scores, the step's seeds excluded."""
    B, gen = s["unmasked"].shape
    conf = torch.rand(B, gen, generator=g, device="cuda").clamp_min(1e-6).pow(0.2)
    flags = s["unmasked"].to(torch.uint8)
    if s["seed_idx"] is not None:
        flags.scatter_(1, s["seed_idx"].long() - s["first"], 3)

    def mass(n):
        return torch.exp(_normal(g, B, gen, n) - 0.5).sum(2) / c["L"]

    return {"logp": conf.log().contiguous(), "d_in": mass(max(1, gen // 2)), "d_out": mass(15), "flags": flags}


def _logits(g, R, V, dtype):
    """N(0, 2^2) logits with one raised token per row (near-uniform to near-certain rows), rows
    padded to 16 bytes; and the token in place: the raised one on even rows, any on odd ones."""
    per = 8 if dtype == "bf16" else 4
    x = 2.0 * _normal(g, R, (V + per - 1) // per * per)
    top = torch.randint(0, V, (R,), generator=g, device="cuda")
    x[torch.arange(R, device="cuda"), top] += 14.0 * torch.rand(R, generator=g, device="cuda")
    other = torch.randint(0, V, (R,), generator=g, device="cuda")
    even = torch.arange(R, device="cuda") % 2 == 0
    return x.to(TORCH[dtype])[:, :V], torch.where(even, top, other).to(torch.int32)


def _heads(s, c, h):
    """float64 q rows, live and override k/v of query head h of every batch row, [B, n, d]."""
    x = h // (c["Hq"] // c["Hkv"])
    k, v = s["k"][:, x].double(), s["v"][:, x].double()
    ko, vo = k.clone(), v.clone()
    if s["seed_idx"] is not None:
        for b in range(c["B"]):
            j = s["seed_idx"][b].long()
            ko[b, j] = s["kc"][b, x, j].double()
            vo[b, j] = s["vc"][b, x, j].double()
    return s["q"][:, h].double(), k, v, ko, vo


def _scores(s, c, q, k, ko, off):
    """Scaled scores of the query rows (positions off ...) on the override keys, a seed row's own
    column on its live key; and that column's seeds as (batch row, query row, position)."""
    x = torch.bmm(q, ko.transpose(1, 2).contiguous()) / math.sqrt(c["d"])
    own = []
    if s["seed_idx"] is not None:
        for b in range(c["B"]):
            j = s["seed_idx"][b].long()
            j = j[(j >= off) & (j < off + q.shape[1])]
            x[b, j - off, j] = (q[b, j - off] * k[b, j]).sum(1) / math.sqrt(c["d"])
            own.append((b, j - off, j))
    return x, own


def _exact_attn(s, c, off):
    out = torch.empty(s["q"].shape, device="cuda", dtype=torch.float64)
    lse = torch.empty(s["q"].shape[:3], device="cuda", dtype=torch.float64)
    for h in range(c["Hq"]):
        q, k, v, ko, vo = _heads(s, c, h)
        x, own = _scores(s, c, q, k, ko, off)
        lse[:, h] = torch.logsumexp(x, 2)
        w = torch.exp(x - lse[:, h][:, :, None])
        o = torch.bmm(w, vo)
        for b, r, j in own:
            o[b, r] += w[b, r, j][:, None] * (v[b, j] - vo[b, j])
        out[:, h] = o
    return out, lse


def _region_lse(s, c):
    """The forward pass's lse, fp32 [B, Hq, L] (its rows outside the region are not read)."""
    lse = torch.zeros(c["B"], c["Hq"], c["L"], device="cuda", dtype=torch.float64)
    a, n = s["first"], s["gen"]
    for h in range(c["Hq"]):
        q, k, _, ko, _ = _heads(s, c, h)
        x, _ = _scores(s, c, q[:, a:a + n], k, ko, a)
        lse[:, h, a:a + n] = torch.logsumexp(x, 2)
    return lse.float()


def _exact_masses(s, c, masked, drafted):
    a, n = s["first"], s["gen"]
    m, f = masked.double(), drafted.double()
    d_in, d_out = torch.zeros_like(m), torch.zeros_like(m)
    for h in range(c["Hq"]):
        q, k, _, ko, _ = _heads(s, c, h)
        x, _ = _scores(s, c, q[:, a:a + n], k, ko, a)
        w = torch.exp(x[:, :, a:a + n] - s["lse"][:, h, a:a + n].double()[:, :, None])
        d_in += torch.bmm(m[:, None], w)[:, 0] / c["Hq"]
        d_out += torch.bmm(w, f[:, :, None].contiguous())[:, :, 0] / c["Hq"]
    return d_in, d_out


def _mass_inputs(g, s):
    """Masked positions of the region, and up to 15 of them just drafted."""
    masked = ~s["unmasked"]
    key = torch.rand(masked.shape, generator=g, device="cuda").masked_fill(~masked, 2.0)
    drafted = (key.argsort(1).argsort(1) < 15) & masked
    return masked.to(torch.uint8), drafted.to(torch.uint8)


MASK_ID = 126336  # the [MASK] token where the vocabulary has it; otherwise the last token


def prepare(case, seed):
    c, g = case, _rng(seed)
    kind = c["kind"]
    if kind == "token":
        logits, tokens = _logits(g, c["R"], c["V"], c["dtype"])
        return {"c": c, "logits": logits, "tokens": tokens, "seed": seed}
    s = _layer(c, g)
    s["c"] = c
    if kind == "attn":
        if c["layout"] == "head":
            s["attn"] = cover.PreparedAttn(s["q"], s["k"], s["v"], s["kc"], s["vc"], s["seed_idx"], s["n_seed"])
        if c["select"]:
            s["sel"] = _select_inputs(c, g, s)
            s["select"] = cover.PreparedSelect(s["sel"]["logp"], s["sel"]["d_in"], s["sel"]["d_out"],
                                               s["sel"]["flags"], max(16, c["seeds"]), s["first"])
    elif kind == "block":
        s["block"] = cover.PreparedRect(s["q"], s["k"], s["v"], s["kc"], s["vc"], c["q_off"], s["seed_idx"],
                                        s["n_seed"])
    else:
        s["lse"] = _region_lse(s, c)
        s["workspace"] = torch.empty(max(1, cover.attn_stats_workspace(c["B"], c["Hq"], s["gen"])), device="cuda",
                                     dtype=torch.float32)
        if kind == "masses":
            s["masked"], s["drafted"] = _mass_inputs(g, s)
        else:
            s["logits"], s["raised"] = _logits(g, s["gen"], c["V"], "bf16")
            s["mask_id"] = min(MASK_ID, c["V"] - 1)
            other = torch.randint(0, c["V"], (1, s["gen"]), generator=g, device="cuda", dtype=torch.int32)
            kept = torch.where(torch.rand(1, s["gen"], generator=g, device="cuda") < 0.7, s["raised"][None], other)
            kept = torch.where(kept == s["mask_id"], kept - 1, kept)
            s["tokens"] = torch.where(s["unmasked"], kept, torch.full_like(kept, s["mask_id"]))
            s["remask"] = torch.randint(0, 4, (1, s["gen"]), generator=g, device="cuda", dtype=torch.int32)
    return s


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind == "attn":
        if c["layout"] == "head":
            s["attn"]()
            out, lse = s["attn"].out, s["attn"].lse
        else:
            out, lse = cover.cover_attn_fwd(s["q"], s["k"], s["v"], s["kc"], s["vc"], s["seed_idx"], s["n_seed"])
        if not c["select"]:
            return {"out": out, "lse": lse}
        s["select"]()
        return {"out": out, "lse": lse, "seeds": s["select"].seed_idx, "n": s["select"].n_seed,
                "score": s["select"].score}
    if kind == "block":
        s["block"]()
        return {"out": s["block"].out, "lse": s["block"].lse}
    if kind == "token" and c["op"] == "stats":
        logp, conf, top = cover.cover_token_stats(s["logits"], s["tokens"])
        return {"logp": logp, "conf": conf, "top": top}
    if kind == "token":
        token, prob = cover.cover_token_sample(s["logits"], c["T"], s["seed"], 3)
        return {"token": token, "prob": prob}
    if kind == "masses":
        d_in, d_out = cover.cover_attn_stats(s["q"], s["k"], s["kc"], s["seed_idx"], s["n_seed"], s["lse"],
                                             s["masked"], s["drafted"], s["first"], workspace=s["workspace"])
        return {"d_in": d_in, "d_out": d_out}
    # the tail of a step: the previous state is kept, its copy is updated in place
    _, conf, top = cover.cover_token_stats(s["logits"], want_logp=False)
    tokens, remask = s["tokens"].clone(), s["remask"].clone()
    flags, drafted, counts = cover.cover_decode_update(tokens, top[None], conf[None], s["seed_idx"], s["n_seed"],
                                                       remask, s["mask_id"], 0.5, 15, 5, s["first"])
    logp, _, _ = cover.cover_token_stats(s["logits"], tokens[0], want_conf=False, want_argmax=False)
    masked = (tokens == s["mask_id"]).to(torch.uint8)
    d_in, d_out = cover.cover_attn_stats(s["q"], s["k"], s["kc"], s["seed_idx"], s["n_seed"], s["lse"], masked,
                                         drafted, s["first"], workspace=s["workspace"])
    seeds, n, score = cover.cover_select_seeds(logp[None], d_in, d_out, flags, 16, s["first"])
    return {"conf": conf, "top": top, "tokens": tokens, "remask": remask, "counts": counts, "logp": logp,
            "d_in": d_in, "d_out": d_out, "seeds": seeds, "n": n, "score": score}


def work(case):
    c = case
    esz = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "token":
        # the logits once; sampling's random numbers and logarithms, and the exponentials of
        # either sum, are of the path but no floating-point contraction: a few per token
        return {"bytes": c["R"] * (c["V"] * esz + 16), "flops": 4 * c["R"] * c["V"]}
    B, Hq, Hkv, L, d = (c[k] for k in ("B", "Hq", "Hkv", "L", "d"))
    if c["kind"] in ("attn", "block"):
        n = c.get("Lq", L)
        kv = 2 * B * Hkv * (L + c["seeds"]) * d * esz
        return {"bytes": kv + 2 * B * Hq * n * d * esz + 4 * B * Hq * n, "flops": 4 * B * Hq * n * L * d}
    n = min(c["gen"], L)
    masses = {"bytes": B * (Hq + Hkv) * n * d * esz + 4 * B * Hq * n + 10 * B * n, "flops": 2 * B * Hq * n * n * d}
    if c["kind"] == "masses":
        return masses
    # the logits are read for the confidences and, once the state is updated, one of each row
    return {"bytes": masses["bytes"] + n * c["V"] * esz + 64 * n, "flops": masses["flops"] + 4 * n * c["V"]}


def tolerance(case):
    c = case
    if c["kind"] in ("attn", "block"):
        return {"rel": 1e-5} if c["dtype"] == "f32" else {"rel": 1e-2}
    if c["kind"] == "tail":
        return {"rel": 1e-5, "differ": 0.01}  # seeds at near-equal scores
    if c["kind"] == "token" and c["op"] == "sample":
        return {"rel": 1e-5, "differ": 0.01}  # perturbed scores tied within fp32
    return {"rel": 1e-5}


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    if c["kind"] == "token":
        x = s["logits"].double()
        if c["op"] == "sample":
            return None  # the draw is defined by the generator's bits
        lz = torch.logsumexp(x, 1)
        logp = x.gather(1, s["tokens"].long()[:, None])[:, 0] - lz
        return {"logp": logp, "conf": torch.exp(x.max(1).values - lz), "top": None}
    if c["kind"] == "attn":
        out, lse = _exact_attn(s, c, 0)
        got = {"out": out, "lse": lse}
        if c["select"]:
            z = s["sel"]
            score = -z["logp"].double() * (1 + z["d_in"].double()) / (1 + z["d_out"].double())
            got.update(seeds=None, n=None, score=torch.where(s["unmasked"], score, torch.zeros_like(score)))
        return got
    if c["kind"] == "block":
        out, lse = _exact_attn(s, c, c["q_off"])
        return {"out": out, "lse": lse}
    if c["kind"] == "masses":
        d_in, d_out = _exact_masses(s, c, s["masked"], s["drafted"])
        return {"d_in": d_in, "d_out": d_out}
    x = s["logits"].double()
    lz = torch.logsumexp(x, 1)
    return {"conf": torch.exp(x.max(1).values - lz), "top": None, "tokens": None, "remask": None, "counts": None,
            "logp": None, "d_in": None, "d_out": None, "seeds": None, "n": None, "score": None}
