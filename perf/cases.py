"""What a program that serves batched speculative sampling asks of this library, as cases to be timed.

A case is a dict of plain values.  Its `kind` says which public entry points one pass goes through:

  step   one verification step of a model: bass_attention_plan once, bass_verify_attention_planned with the
         step's K/V rows for every attention layer, then the acceptance -- from probability rows
         (bass_spec_accept) or from the logits (bass_warp_accept)
  call   the same for a caller that keeps no plan: bass_append_verify_attention per layer, bass_spec_accept
  fill   prompts written into fresh caches: bass_kv_append per layer
  move   sequences moved between caches: bass_kv_gather (bass_kv_gather_int8 for codes) and, for bf16 and
         fp32 caches, bass_kv_append of the rows into another cache
  rows   probability rows from the logits of both models (bass_warp_probs twice), then bass_spec_accept

Lengths belong to the case (they follow from its `lens` number, so that work() knows them); tensors are
drawn from the seed.  Layers of one step have caches of their own, as in a model, so a pass reads each byte
of its caches once and the last-level cache does not hold them from one pass to the next.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2404_15778_amd as bass

DEV = "cuda:0"


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "kv": "bf16", "B": 8, "kmax": 6, "q_lo": 1, "Hq": 32, "Hkv": 32, "D": 128, "ctx_lo": 512,
         "ctx_hi": 2048, "log_ctx": False, "layers": 32, "V": 50000, "sample": "logits", "temperature": 0.2, "top_p": 0.95, "lens": 1}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: two short sequences, fp32, 4 heads of 64 (the tiny configuration of the tests), no
        # plan kept, a toy vocabulary.  Latency, launches and host work.
        _case("call_fp32_tiny", "call", kv="fp32", B=2, kmax=4, q_lo=3, Hq=4, Hkv=4, D=64, ctx_lo=37, ctx_hi=90, layers=1, V=64,
              sample="probs"),
        # One user at a terminal: a single sequence, 7 drafts (where the draft-length heuristic starts).
        _case("step_mha_b1", "step", B=1, kmax=8, q_lo=8),
        # The benchmark's step: 8 sequences, 32 layers, acceptance from probability rows.
        _case("step_mha_b8", "step", sample="probs"),
        # A large batch of very different lengths, 128 to 8192 tokens (fewer layers: a layer is 2 GB of keys and values).
        _case("step_mha_b32_ragged", "step", B=32, kmax=8, ctx_lo=128, ctx_hi=8192, log_ctx=True, layers=4),
        # Grouped-query heads, 8 query heads per kv head, long contexts, a large vocabulary.
        _case("step_gqa_b16", "step", B=16, kmax=6, q_lo=2, Hq=64, Hkv=8, ctx_lo=1024, ctx_hi=4096, layers=16, V=131072),
        # The benchmark's step on INT8 caches.
        _case("step_mha_int8_b8", "step", kv="int8kv"),
        # Grouped-query heads on INT8 caches, 8 tokens each: 64 query rows per kv head, the most that is taken.
        _case("step_gqa_int8_b16", "step", kv="int8kv", B=16, kmax=8, q_lo=4, Hq=64, Hkv=8, ctx_lo=1024, ctx_hi=4096, layers=16),
        # Long drafts: 31 drafts and the last token, at the limit of the draft-length heuristic.
        _case("step_mha_draft32_b8", "step", kmax=32, q_lo=16, layers=16),
        # A smaller model: 16 heads of 64, odd lengths, an odd vocabulary, flat sampling (temperature 1).
        _case("step_mha_d64_b13", "step", B=13, kmax=5, Hq=16, Hkv=16, D=64, ctx_lo=65, ctx_hi=1021, layers=24, V=32001,
              temperature=1.0, top_p=0.9),
        # The other direction of the cache: prompts quantized into INT8 caches.
        _case("fill_int8_b8", "fill", kv="int8kv", kmax=2048, layers=4),
        # Sequences read back from one bf16 cache and written into another (swapped out, or rearranged).
        _case("move_bf16_b8", "move", kmax=2048, layers=4),
        # Sampling of a large batch over a large vocabulary with the probability rows kept.
        _case("rows_b32_v128k", "rows", B=32, kmax=8, V=131072),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("step", "call", "fill", "move", "rows"), (10, 2, 2, 2, 2))[0]
    c = _case("", kind, lens=rng.randrange(1 << 20))
    del c["name"]
    c["temperature"] = rng.choice((0.2, 0.2, 0.6, 1.0))
    c["top_p"] = rng.choice((0.95, 0.95, 0.9, 1.0))
    V = _log_int(rng, 8000, 131072)
    c["V"] = V if rng.random() < 0.4 else V - V % 8  # most vocabularies are padded, not all
    c["B"] = _log_int(rng, 1, 32)
    if kind == "rows":
        c["kmax"] = rng.randint(1, 8)
        return c
    c["kv"] = rng.choices(("bf16", "int8kv", "fp32"), (5, 3, 0) if kind == "step" else (2, 2, 1))[0]
    if kind == "call":
        c.update(kv="fp32", B=rng.randint(1, 4), Hq=8, Hkv=rng.choice((2, 4, 8)), D=rng.choice((32, 64, 128)), layers=1,
                 V=rng.randint(64, 4096), sample="probs", ctx_lo=rng.randint(1, 64), ctx_hi=rng.randint(65, 512),
                 kmax=rng.randint(1, 8))
        return c
    c["Hq"], c["Hkv"], c["D"] = rng.choice(((32, 32, 128), (32, 32, 128), (64, 8, 128), (32, 8, 128), (16, 16, 64), (32, 8, 64)))
    g = c["Hq"] // c["Hkv"]
    c["sample"] = rng.choice(("logits", "logits", "probs"))
    if kind in ("fill", "move"):
        c["ctx_hi"] = c["kmax"] = _log_int(rng, 128, 4096)
        c["ctx_lo"] = max(1, c["kmax"] // rng.randint(1, 8))
    else:
        c["kmax"] = min(_log_int(rng, 1, 33), 64 // g)
        c["q_lo"] = rng.randint(1, c["kmax"])
        c["ctx_hi"] = _log_int(rng, 128, 8192)
        c["ctx_lo"] = max(1, c["ctx_hi"] // rng.randint(1, 16))
        c["log_ctx"] = rng.random() < 0.5
    # as many layers as a model has, or as the largest listed step moves (5 GB), whichever is less
    c["layers"] = 1
    c["layers"] = max(1, min(32, int(4.5e9 / work(c)["bytes"]), int(12e9 / (2 * c["B"] * (c["ctx_hi"] + 64) * c["Hkv"] * c["D"] * 2))))
    if kind != "step":
        c["layers"] = min(c["layers"], 4)
    while c["B"] > 1 and work(c)["bytes"] > 5.5e9:  # one layer alone moves more than that: fewer sequences
        c["B"] //= 2
    return c


# ---- lengths ------------------------------------------------------------------------------------

def _lengths(c):
    """(cached tokens, query tokens) of every sequence."""
    rng = np.random.default_rng([c["lens"], c["B"], c["ctx_hi"], c["kmax"]])
    if c["log_ctx"]:
        ctx = np.rint(np.exp(rng.uniform(math.log(c["ctx_lo"]), math.log(c["ctx_hi"]), size=c["B"]))).astype(np.int32)
    else:
        ctx = rng.integers(c["ctx_lo"], c["ctx_hi"] + 1, size=c["B"]).astype(np.int32)
    nq = rng.integers(min(c["q_lo"], c["kmax"]), c["kmax"] + 1, size=c["B"]).astype(np.int32)
    return ctx, nq


def _desc(c, **kw):
    d = bass.make_desc(c["B"], c["kmax"], c["Hq"], c["Hkv"], c["D"], c["ctx_hi"] + (0 if c["kind"] in ("fill", "move") else c["kmax"] + 2),
                       c["kv"], 1.0 / math.sqrt(c["D"]))
    return d.replace(**kw) if kw else d


# ---- inputs -------------------------------------------------------------------------------------

def _randn(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype)


def _i32(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.int32, device=DEV)


def _context(c, gen, ctx):
    """The rows of every layer's and sequence's cached context, in the order in which they are drawn: (layer, sequence, K, V)."""
    et = torch.float32 if c["kv"] == "fp32" else torch.bfloat16
    for l in range(c["layers"]):
        for b in range(c["B"]):
            shape = (1, int(ctx[b]), c["Hkv"], c["D"])
            K = _randn(gen, shape, et)
            yield l, b, K, _randn(gen, shape, et)


def _step_rows(c, gen):
    """Queries and new K and V rows of every layer, drawn after the context."""
    et = torch.float32 if c["kv"] == "fp32" else torch.bfloat16
    lead, Hq, Hkv, D = (c["layers"], c["B"], c["kmax"]), c["Hq"], c["Hkv"], c["D"]
    # grouped-query recipe: scores of unit variance come from smaller queries
    q_mult = 1.0 if Hq == Hkv else 1.0 / math.sqrt(D)
    Q = _randn(gen, lead + (Hq, D), torch.float32).mul_(q_mult).to(et)
    K = _randn(gen, lead + (Hkv, D), et)
    return Q, K, _randn(gen, lead + (Hkv, D), et)


def _prepare_caches(c, s, gen, ctx):
    """One slab for all layers' K and one for their V, the cached context of every sequence in place."""
    d = s.desc
    size = bass.bass_kv_cache_bytes(d)
    s.Kslab = torch.zeros((c["layers"], size), dtype=torch.uint8, device=DEV)
    s.Vslab = torch.zeros((c["layers"], size), dtype=torch.uint8, device=DEV)
    per_seq, zero = size // c["B"], torch.zeros(1, dtype=torch.int32, device=DEV)
    for l, b, K, V in _context(c, gen, ctx):
        at = slice(b * per_seq, (b + 1) * per_seq)
        bass.bass_kv_append(d.replace(B=1, kmax=K.shape[1]), s.Kslab[l, at], s.Vslab[l, at], K, V, zero, s.ctx[b:b + 1])
    s.K, s.V = list(s.Kslab), list(s.Vslab)


def _prepare_logits(c, gen, k):
    """Logits of the main model ~ N(0, 3^2), of the draft model the same plus N(0, 1)."""
    lt = torch.randn((c["B"], k + 1, c["V"]), generator=gen, device=DEV) * 3.0
    ld = lt[:, :k] + torch.randn((c["B"], k, c["V"]), generator=gen, device=DEV)
    return lt, ld


def _sample(rows, gen):
    """One token of every row."""
    cdf = rows.double().cumsum(-1)
    u = torch.rand(rows.shape[:-1] + (1,), generator=gen, device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf, u * cdf[..., -1:], right=True).squeeze(-1).clamp_(max=rows.shape[-1] - 1).to(torch.int32)


def _prepare_acceptance(c, s, gen, n_draft):
    k = c["kmax"] - 1  # a step verifies the last token and its drafts
    lt, ld = _prepare_logits(c, gen, k)
    rows = torch.empty_like(ld)
    if c["kind"] == "rows" or c["sample"] == "logits":
        if k:
            bass.bass_warp_probs(ld, c["temperature"], c["top_p"], rows)  # what the draft model sampled its drafts from
        s.logits_main, s.logits_draft = lt, ld
    else:
        s.p, rows = torch.softmax(lt, -1), torch.softmax(ld, -1)
        s.q = rows
    s.tok = _sample(rows, gen) if k else torch.zeros((c["B"], 0), dtype=torch.int32, device=DEV)
    s.n_draft = _i32(n_draft)
    s.u = torch.rand((c["B"], k + 1), generator=gen, device=DEV, dtype=torch.float32)
    s.n_accept = torch.zeros(c["B"], dtype=torch.int32, device=DEV)
    s.next_token = torch.zeros(c["B"], dtype=torch.int32, device=DEV)
    if c["kind"] == "rows":
        s.p, s.q = torch.empty_like(lt), torch.empty_like(ld)
    elif c["sample"] == "logits":
        s.accept_ws = torch.empty(bass.bass_warp_accept_workspace_bytes(c["B"], k, c["V"]), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    ctx, nq = _lengths(c)
    s = SimpleNamespace(case=c, status=torch.zeros(1, dtype=torch.int32, device=DEV))
    if c["kind"] == "rows":
        _prepare_acceptance(c, s, gen, nq - 1)
        return s
    s.desc = _desc(c)
    s.ctx, s.nq = _i32(ctx), _i32(nq)
    B, kmax, Hq, Hkv, D = (c[n] for n in ("B", "kmax", "Hq", "Hkv", "D"))
    et = torch.float32 if c["kv"] == "fp32" else torch.bfloat16
    if c["kind"] in ("fill", "move"):
        s.zero = torch.zeros(B, dtype=torch.int32, device=DEV)
        if c["kind"] == "move":
            _prepare_caches(c, s, gen, ctx)
            if c["kv"] == "int8kv":
                new = lambda *shape, dtype: [torch.zeros(shape, dtype=dtype, device=DEV) for _ in range(c["layers"])]  # noqa: E731
                s.codes = [new(B, kmax, Hkv, D, dtype=torch.int8) for _ in range(2)]
                s.scales = [new(B, kmax, Hkv, dtype=torch.float32) for _ in range(2)]
            else:
                s.rows = [torch.zeros((c["layers"], B, kmax, Hkv, D), dtype=et, device=DEV) for _ in range(2)]
                s.to = [torch.zeros_like(s.Kslab) for _ in range(2)]
        else:
            s.Kslab = torch.zeros((c["layers"], bass.bass_kv_cache_bytes(s.desc)), dtype=torch.uint8, device=DEV)
            s.Vslab = torch.zeros_like(s.Kslab)
            s.Kn = [_randn(gen, (B, kmax, Hkv, D), et) for _ in range(c["layers"])]
            s.Vn = [_randn(gen, (B, kmax, Hkv, D), et) for _ in range(c["layers"])]
        return s
    _prepare_caches(c, s, gen, ctx)
    s.Q, s.Kn, s.Vn = (list(t) for t in _step_rows(c, gen))
    s.Oall = torch.zeros((c["layers"], B, kmax, Hq, D), dtype=torch.float32, device=DEV)
    s.O = list(s.Oall)
    s.ws = bass.alloc_workspace(s.desc, DEV)
    s.plan = bass.alloc_plan(s.desc, DEV)
    _prepare_acceptance(c, s, gen, nq - 1)
    return s


# ---- one pass -----------------------------------------------------------------------------------

def _accept(s):
    c = s.case
    if c["kind"] != "rows" and c["sample"] == "logits":
        bass.bass_warp_accept(s.logits_main, s.logits_draft if c["kmax"] > 1 else None, c["temperature"], c["top_p"],
                              s.tok if c["kmax"] > 1 else None, s.n_draft, s.u, s.n_accept, s.next_token, s.accept_ws, None, s.status)
    else:
        bass.bass_spec_accept(s.p, s.q if c["kmax"] > 1 else None, s.tok if c["kmax"] > 1 else None, s.n_draft, s.u, s.n_accept,
                              s.next_token, None, s.status)


def _words(t):
    """An opaque cache as 32-bit words."""
    return t.view(torch.int32)


def run(state):
    s, c = state, state.case
    if c["kind"] == "rows":
        bass.bass_warp_probs(s.logits_main, c["temperature"], c["top_p"], s.p, s.status)
        if c["kmax"] > 1:
            bass.bass_warp_probs(s.logits_draft, c["temperature"], c["top_p"], s.q, s.status)
        _accept(s)
        return {"p": s.p, "q": s.q, "n_accept": s.n_accept, "next_token": s.next_token, "status": s.status}
    if c["kind"] == "fill":
        for l in range(c["layers"]):
            bass.bass_kv_append(s.desc, s.Kslab[l], s.Vslab[l], s.Kn[l], s.Vn[l], s.zero, s.ctx, s.status)
        return {"K": _words(s.Kslab), "V": _words(s.Vslab), "status": s.status}
    if c["kind"] == "move":
        if c["kv"] == "int8kv":
            for l in range(c["layers"]):
                bass.bass_kv_gather_int8(s.desc, s.K[l], s.V[l], s.codes[0][l], s.codes[1][l], s.scales[0][l], s.scales[1][l], s.zero,
                                         s.ctx, s.status)
            return {"codes": s.codes, "scales": s.scales, "status": s.status}
        for l in range(c["layers"]):
            bass.bass_kv_gather(s.desc, s.K[l], s.V[l], s.rows[0][l], s.rows[1][l], s.zero, s.ctx, s.status)
            bass.bass_kv_append(s.desc, s.to[0][l], s.to[1][l], s.rows[0][l], s.rows[1][l], s.zero, s.ctx, s.status)
        return {"rows": s.rows, "K": _words(s.to[0]), "V": _words(s.to[1]), "status": s.status}
    if c["kind"] == "call":
        for l in range(c["layers"]):
            bass.bass_append_verify_attention(s.desc, s.Q[l], s.Kn[l], s.Vn[l], s.K[l], s.V[l], s.ctx, s.nq, s.O[l], None, s.ws, s.status)
    else:
        bass.bass_attention_plan(s.desc, s.ctx, s.nq, bass.PLAN_APPEND, 0, s.plan, s.status)
        for l in range(c["layers"]):
            bass.bass_verify_attention_planned(s.desc, s.Q[l], s.Kn[l], s.Vn[l], s.K[l], s.V[l], s.plan, s.O[l], None, s.ws, s.status)
    _accept(s)
    return {"O": s.Oall, "K": _words(s.Kslab), "V": _words(s.Vslab), "n_accept": s.n_accept, "next_token": s.next_token, "status": s.status}


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    c = case
    ctx, nq = (x.astype(np.int64) for x in _lengths(c))
    B, V, k = c["B"], c["V"], c["kmax"] - 1
    if c["kind"] == "rows":
        rows = B * (2 * k + 1) * V * 4
        return {"bytes": 2 * rows + B * (2 if k else 1) * V * 4, "flops": rows}
    row_elems = c["Hkv"] * c["D"]
    kv_row = {"bf16": 2 * row_elems, "fp32": 4 * row_elems, "int8kv": row_elems + 4 * c["Hkv"]}[c["kv"]]  # one cached K (or V) row
    new_row = (4 if c["kv"] == "fp32" else 2) * row_elems  # as the model gives it
    tokens = int(ctx.sum())
    if c["kind"] == "fill":
        return {"bytes": c["layers"] * 2 * tokens * (new_row + kv_row), "flops": 0}
    if c["kind"] == "move":
        passes = 2 * kv_row if c["kv"] == "int8kv" else 4 * kv_row
        return {"bytes": c["layers"] * 2 * tokens * passes, "flops": 0}
    q_bytes = (4 if c["kv"] == "fp32" else 2) * int(nq.sum()) * c["Hq"] * c["D"]
    layer = 2 * tokens * kv_row + 2 * int(nq.sum()) * (new_row + kv_row) + q_bytes + 4 * B * c["kmax"] * c["Hq"] * c["D"]
    seen = int((nq * ctx + nq * (nq + 1) // 2).sum())
    rows = B * (2 if k else 1) if c["sample"] == "probs" else B * (2 * k + 1)
    return {"bytes": c["layers"] * layer + rows * V * 4, "flops": c["layers"] * 4 * seen * c["Hq"] * c["D"]}


def tolerance(case):
    """Caches, codes, tokens and counts are whole numbers and exact everywhere.  Attention outputs and probability
    rows were compared with the same computation in 64 bits on the listed cases (one layer, up to four sequences);
    stated here is about four times the largest difference seen:
      bf16 and INT8 caches (probabilities rounded to bf16)  rel 1.3e-3 .. 1.75e-3, max 6.6e-3 .. 2.1e-2
      fp32 caches                                           rel 2.9e-7, max 1.3e-6
      probability rows                                      rel 3.1e-8, max 2.1e-7"""
    if case["kind"] in ("fill", "move"):
        return "exact"
    if case["kind"] == "rows":
        return {"rel": 1.3e-7, "max": 8e-7}
    if case["kv"] == "fp32":
        return {"rel": 1.2e-6, "max": 5.5e-6}
    return {"rel": 7e-3, "max": 8.5e-2}


# ---- what a pass returns, in 64 bits ----------------------------------------------------------------

def _represented(x, c):
    """Rows as an attention over this cache sees them: the values themselves, or code * scale of INT8 rows, in 64 bits."""
    if c["kv"] != "int8kv":
        return x.double()
    x = x.float()  # every step below is one operation in 32 bits
    amax = x.abs().amax(-1, keepdim=True)
    codes = torch.round(x * torch.where(amax > 0, 127.0 / amax, torch.zeros_like(amax)))
    return codes.double() * (amax / 127.0).double()


def _warped(z, temperature, top_p):
    """Probability rows: temperature, the shortest prefix of the sorted tokens that reaches top_p, renormalised."""
    p = torch.softmax(z.double() / temperature, -1)
    if top_p >= 1.0:
        return p
    sorted_p, order = torch.sort(p, dim=-1, descending=True, stable=True)
    before = sorted_p.cumsum(-1) - sorted_p
    p = torch.zeros_like(p).scatter_(-1, order, torch.where(before < top_p, sorted_p, torch.zeros_like(sorted_p)))
    return p / p.sum(-1, keepdim=True)


def exact(case, seed):
    c = case
    if c["kind"] in ("fill", "move"):
        return None  # whole numbers and copies
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    ctx, nq = _lengths(c)
    if c["kind"] == "rows":
        p, q = (torch.stack([_warped(z, c["temperature"], c["top_p"]) for z in t]) if t.numel() else t.double()
                for t in _prepare_logits(c, gen, c["kmax"] - 1))
        return {"p": p, "q": q, "n_accept": None, "next_token": None, "status": None}
    Hq, Hkv, D = c["Hq"], c["Hkv"], c["D"]
    g, scale = Hq // Hkv, 1.0 / math.sqrt(D)
    at_context = gen.get_state()
    for _ in _context(c, gen, ctx):
        pass
    Q, Kn, Vn = _step_rows(c, gen)
    gen.set_state(at_context)
    O = torch.zeros((c["layers"], c["B"], c["kmax"], Hq, D), dtype=torch.float64, device=DEV)
    for l, b, K, V in _context(c, gen, ctx):
        L, n = int(ctx[b]), int(nq[b])
        K = _represented(torch.cat([K[0], Kn[l, b, :n]]), c).permute(1, 2, 0).contiguous()  # [Hkv, D, L + n]
        V = _represented(torch.cat([V[0], Vn[l, b, :n]]), c).permute(1, 0, 2).contiguous()
        q = _represented(Q[l, b, :n], c).view(n, Hkv, g, D).permute(1, 0, 2, 3).reshape(Hkv, n * g, D)
        s = torch.matmul(q, K).mul_(scale).view(Hkv, n, g, L + n)
        hidden = torch.arange(L + n, device=DEV) > L + torch.arange(n, device=DEV).unsqueeze(1)
        s.masked_fill_(hidden.view(1, n, 1, L + n), float("-inf"))
        o = torch.matmul(torch.softmax(s, -1).view(Hkv, n * g, L + n), V)
        O[l, b, :n] = o.view(Hkv, n, g, D).permute(1, 0, 2, 3).reshape(n, Hq, D)
    return {"O": O, "K": None, "V": None, "n_accept": None, "next_token": None, "status": None}
