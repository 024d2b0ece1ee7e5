"""The work that a program composing cached context has libpkv do, as timed cases.

A case is one pass through the public entry points of ``paper_2606_17107_amd.pkv``
with what such a program keeps at hand: caches, position arrays, block tables,
segment records, attention descriptors and the split workspace.  Splices go
through the tensor-level calls (one per request); attention layers go through
the descriptor-level calls that a serving loop issues once per layer.

  listed()              the fixed cases
  draw(rng)             one more case of the same ranges
  prepare(case, seed)   inputs on the GPU, made from the seed alone
  run(state)            one pass; returns the output tensors
  work(case)            bytes and flops the pass cannot do without
  tolerance(case)       how far another correct implementation may be off
  exact(case, seed)     the same outputs in float64 from plain torch
"""
import math
import random

import torch

from paper_2606_17107_amd import pkv

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
ELEM = {"bf16": 2, "f32": 4}
STYLES = {"half": pkv.PKV_ROPE_HALF, "interleaved": pkv.PKV_ROPE_INTERLEAVED}


# ---- the cases --------------------------------------------------------------

def _splice(entry, dtype, layers, kv_heads, head_dim, v_dim, tokens, src0, dst0, slots, theta, rope_dim=None,
            rope_offset=0, style="half", page=0):
    """A chunk of `tokens` moved from positions src0.. to dst0.. of a `slots`-slot cache."""
    return dict(kind="splice", entry=entry, dtype=dtype, layers=layers, kv_heads=kv_heads, head_dim=head_dim,
                v_dim=v_dim, tokens=tokens, src0=src0, dst0=dst0, slots=slots, theta=theta,
                rope_dim=rope_dim or head_dim, rope_offset=rope_offset, style=style, page=page)


def _attention(variant, layers, seqs, heads, kv_heads, head_dim, queries, kv_min, kv_max, window=0, page=0,
               ragged=False):
    """Suffix attention of up to `queries` tokens a sequence over caches of kv_min..kv_max slots."""
    return dict(kind="attention", variant=variant, dtype="f32" if variant == "f32" else "bf16", layers=layers,
                seqs=seqs, heads=heads, kv_heads=kv_heads, head_dim=head_dim,
                v_dim=512 if variant == "mla" else head_dim, queries=queries, kv_min=kv_min, kv_max=kv_max,
                window=window, page=page, ragged=ragged)


def _compose(layers, kv_heads, head_dim, seqs, skills, ctx_min, ctx_max, theta):
    """Every sequence splices the same library of skills at offsets of its own, in one call."""
    return dict(kind="compose", dtype="bf16", layers=layers, kv_heads=kv_heads, head_dim=head_dim, seqs=seqs,
                skills=",".join(str(n) for n in skills), ctx_min=ctx_min, ctx_max=ctx_max, theta=theta)


def listed():
    def named(name, case):
        return dict(case, name=name)

    return [
        # The smallest use: a short skill spliced into a small fp32 cache, then its suffix attends.  Latency,
        # launches and the binding's own cost are all there is.
        named("tiny_f32_step", dict(kind="step", dtype="f32", layers=1, heads=4, kv_heads=2, head_dim=64, tokens=128,
                                    src0=0, dst0=300, slots=512, queries=16, theta=10000.0)),
        # A 4096-token skill into every layer of an 8B-class GQA cache, with the rescaled frequency table such
        # a model is deployed with.
        named("splice_gqa8b_table", _splice("table", "bf16", 32, 8, 128, 128, 4096, 0, 2000, 8256, 500000.0)),
        # A 16k-token skill of an MLA cache: only the 64 k_pe channels of each 576-channel row rotate.
        named("splice_mla", _splice("theta", "bf16", 27, 1, 576, 0, 16384, 0, 8192, 32896, 10000.0, rope_dim=64,
                                    rope_offset=512, style="interleaved")),
        # The same 8B-class cache behind a block table (a serving engine's pool of 64-slot pages), with the
        # odd lengths and offsets that requests have.
        named("splice_paged", _splice("paged", "bf16", 32, 8, 128, 128, 3001, 0, 517, 8256, 500000.0, page=64)),
        # Many users, one library: 16 sequences each splice three skills in one call (a pipeline stage of 8
        # layers of the 8B shape).
        named("compose_batched", _compose(8, 8, 128, 16, (1024, 2048, 4096), 8192, 12288, 500000.0)),
        # One layer of the 8B shape, as a model issues it: a 64-token suffix over a spliced 8k context.
        named("attn_gqa8b_layer", _attention("gqa", 1, 1, 32, 8, 128, 64, 8256, 8256)),
        # One layer of the batched composition: 16 ragged contexts, 256 suffix tokens each.
        named("attn_batched_layer", _attention("gqa", 1, 16, 32, 8, 128, 256, 8448, 12544)),
        # One layer of a long prefill: 1024 suffix tokens over a 49k spliced context.
        named("attn_long32k_layer", _attention("gqa", 1, 1, 28, 4, 128, 1024, 50176, 50176)),
        # The same suffix in a sliding-window layer.
        named("attn_window_layer", _attention("gqa", 1, 1, 28, 4, 128, 1024, 50176, 50176, window=4096)),
        # Token-by-token generation over the composed contexts, one layer, paged pool: one query a sequence.
        named("attn_decode_paged", _attention("gqa", 1, 16, 32, 8, 128, 1, 8448, 12544, page=64)),
        # One layer of the MLA suffix (absorbed form).
        named("attn_mla_layer", _attention("mla", 1, 1, 16, 1, 576, 128, 32896, 32896)),
        # Token-by-token generation over MLA caches.
        named("attn_mla_decode", _attention("mla", 1, 16, 16, 1, 576, 1, 4096, 32768)),
    ]


MAX_SPLICE_BYTES = 3.9e9    # about the composition's
MAX_FLOPS = 7.0e11          # about the long prefill's


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_splice(rng):
    entry = rng.choice(["theta", "theta", "table", "paged"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    mla = entry == "theta" and dtype == "bf16" and rng.random() < 0.4
    tokens = _log_int(rng, 128, 32768)
    layers = 1 if dtype == "f32" else _log_int(rng, 1, 32)
    if mla:
        shape = dict(kv_heads=1, head_dim=576, v_dim=0, rope_dim=64, rope_offset=512, style="interleaved")
    else:
        d = rng.choice([64, 128])
        shape = dict(kv_heads=rng.choice([2, 4, 8]), head_dim=d, v_dim=d)
    src0 = rng.randint(0, 4096)
    dst0 = rng.randint(0, 8192)
    slots = dst0 + tokens + rng.randint(0, 4096)
    return _splice(entry, dtype, layers, tokens=tokens, src0=src0, dst0=dst0, slots=slots,
                   theta=rng.choice([1e4, 5e5, 1e6]), page=rng.choice([32, 64, 128]) if entry == "paged" else 0,
                   **shape)


def _draw_compose(rng):
    skills = tuple(_log_int(rng, 256, 4096) for _ in range(3))
    ctx = sum(skills) + rng.randint(64, 4096)
    return _compose(rng.choice([1, 2, 4, 8]), rng.choice([4, 8]), 128, rng.randint(1, 16), skills, ctx,
                    ctx + rng.randint(0, 4096), 5e5)


def _draw_attention(rng):
    variant = rng.choice(["gqa", "gqa", "gqa", "mla", "f32"])
    if variant == "f32":
        heads, kv_heads, d = rng.choice([(4, 2, 64), (8, 2, 64), (8, 8, 128)])
        kv = _log_int(rng, 128, 2048)
        return _attention(variant, 1, rng.randint(1, 4), heads, kv_heads, d, _log_int(rng, 1, 64), max(64, kv // 2), kv,
                          ragged=rng.random() < 0.5)
    decode = rng.random() < 0.35
    seqs = rng.choice([1, 1, 2, 5, 16]) if not decode else _log_int(rng, 1, 16)
    queries = 1 if decode else _log_int(rng, 2, 1024)
    heads, kv_heads, d = (16, 1, 576) if variant == "mla" else rng.choice([(32, 8, 128), (28, 4, 128), (14, 2, 64),
                                                                           (8, 8, 128)])
    kv_max = _log_int(rng, 512, 50176)
    kv_min = rng.randint(kv_max // 2, kv_max)
    window = rng.choice([1024, 4096]) if variant == "gqa" and rng.random() < 0.25 else 0
    return _attention(variant, 1, seqs, heads, kv_heads, d, min(queries, kv_min), kv_min, kv_max, window=window,
                      page=rng.choice([0, 0, 32, 64]), ragged=not decode and rng.random() < 0.5)


def draw(rng):
    while True:
        kind = rng.random()
        case = _draw_attention(rng) if kind < 0.6 else _draw_splice(rng) if kind < 0.85 else _draw_compose(rng)
        w = work(case)
        if w["bytes"] <= MAX_SPLICE_BYTES and w["flops"] <= MAX_FLOPS:
            return case


# ---- geometry (fixed by the case, not by the seed) ----------------------------

def _lengths(case):
    """(queries, kv length) of every sequence of an attention case."""
    r = random.Random(case["kv_max"] * 131 + case["seqs"] * 7 + case["queries"])
    out = []
    for _ in range(case["seqs"]):
        kv = r.randint(case["kv_min"], case["kv_max"])
        nq = r.randint(1, case["queries"]) if case["ragged"] else case["queries"]
        out.append((nq, kv))
    return out


def _plan(case):
    """Segments of a composition: skills in shuffled order at disjoint offsets of every context."""
    skills = [int(n) for n in case["skills"].split(",")]
    base = [sum(skills[:i]) for i in range(len(skills))]
    r = random.Random(case["ctx_max"] * 131 + case["seqs"])
    src0 = [r.randint(0, 2048) for _ in skills]
    segs, slot0 = [], 0
    for _ in range(case["seqs"]):
        ctx = r.randint(case["ctx_min"], case["ctx_max"])
        order = list(range(len(skills)))
        r.shuffle(order)
        cuts = sorted(r.randint(0, ctx - sum(skills)) for _ in skills)
        pos = 0
        for k, cut in zip(order, cuts):
            segs.append(dict(src_slot0=base[k], dst_seq_base=slot0, n_tokens=skills[k], src_pos0=src0[k],
                             dst_pos0=cut + pos, dst_seq_len=ctx))
            pos += skills[k]
        slot0 += ctx
    return segs, sum(skills), slot0, max(skills)


def _omega(case):
    """Per-pair frequencies: the plain schedule, or (entry "table") the rescaled one of long-context 8B
    models: wavelengths above 8192 divided by 8, below 2048 kept, interpolated between."""
    r = case.get("rope_dim", case["head_dim"])
    w = case["theta"] ** (-torch.arange(0, r, 2, dtype=torch.float64) / r)
    if case.get("entry") != "table":
        return w
    wl = 2 * math.pi / w
    mix = (8192 / wl - 1) / 3
    return torch.where(wl < 2048, w, torch.where(wl > 8192, w / 8, (1 - mix) * w / 8 + mix * w))


# ---- inputs -------------------------------------------------------------------

class _Normal:
    """N(0,1) draws of one seeded generator, in order, on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def __call__(self, shape, dtype, gain=1.0):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, gain, generator=self.g)

    def permutation(self, n):
        return torch.randperm(n, generator=self.g, device="cuda")


def _ints(values, dtype=torch.int32):
    return torch.tensor(values, dtype=dtype, device="cuda")


def _arange(lo, n):
    return torch.arange(lo, lo + n, dtype=torch.int32, device="cuda")


def _inputs(case, seed):
    """Tensors of one case.  Post-RoPE keys and queries are N(0,1) like unrotated ones (a rotation keeps
    the distribution); GQA queries have gain 2, so that the scaled scores have the spread of trained heads
    (about 2) and the softmax is not flat."""
    n = _Normal(seed)
    dt = DTYPES[case["dtype"]]
    s = {}
    if case["kind"] == "attention":
        lens = _lengths(case)
        rows = sum(q for q, _ in lens)
        L, Hkv, d = case["layers"], case["kv_heads"], case["head_dim"]
        s["q"] = n((L, rows, case["heads"], d), dt, 1.0 if case["variant"] == "mla" else 2.0)
        if case["page"]:
            page = case["page"]
            per_seq = max(-(-kv // page) for _, kv in lens)
            pages = per_seq * len(lens) + 16
            s["table"] = n.permutation(pages)[: per_seq * len(lens)].to(torch.int32).view(len(lens), per_seq)
            s["k"] = n((L, pages, page, Hkv, d), dt)
            s["v"] = s["k"][..., :512] if case["variant"] == "mla" else n((L, pages, page, Hkv, case["v_dim"]), dt)
        else:
            s["k"] = n((L, Hkv, sum(kv for _, kv in lens), d), dt)
            s["v"] = s["k"][..., :512] if case["variant"] == "mla" else n(s["k"].shape[:3] + (case["v_dim"],), dt)
        s["q_pos"] = _ints([kv - q + i for q, kv in lens for i in range(q)])
        s["kv_len"] = _ints([kv for _, kv in lens])
        return s
    L, H, d = case["layers"], case["kv_heads"], case["head_dim"]
    if case["kind"] == "compose":
        _, src, slots, _ = _plan(case)
        for name, tokens in (("src_k", src), ("src_v", src), ("dst_k", slots), ("dst_v", slots)):
            s[name] = n((L, H, tokens, d), dt)
        return s
    T, dv = case["tokens"], case.get("v_dim", d)
    s["src_k"] = n((L, H, T, d), dt)
    s["src_v"] = n((L, H, T, dv), dt) if dv else None
    if case.get("page"):
        page = case["page"]
        entries = -(-case["slots"] // page)
        s["table"] = n.permutation(entries + 16)[:entries].to(torch.int32).view(1, entries)
        s["dst_k"] = n((L, entries + 16, page, H, d), dt)
        s["dst_v"] = n((L, entries + 16, page, H, dv), dt) if dv else None
    else:
        s["dst_k"] = n((L, H, case["slots"] + case.get("queries", 0), d), dt)
        s["dst_v"] = n((L, H, case["slots"] + case.get("queries", 0), dv), dt) if dv else None
    s["src_pos"] = _arange(case["src0"], T)
    s["dst_pos"] = _arange(case["dst0"], T)
    if case["kind"] == "step":
        s["q"] = n((L, case["queries"], case["heads"], d), dt, 2.0)
        s["q_pos"] = _arange(case["slots"], case["queries"])
        s["kv_len"] = _ints([case["slots"] + case["queries"]])
    return s


def _scale(case):
    return 1.0 / math.sqrt(192 if case.get("variant") == "mla" else case["head_dim"])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    s["scale"] = _scale(case)
    if case["kind"] == "step":
        s["out"] = torch.zeros_like(s["q"])
    elif case["kind"] == "compose":
        segs, _, _, longest = _plan(case)
        s["segs"], s["n_segs"], s["longest"] = pkv.make_segments(segs, "cuda"), len(segs), longest
    elif case["kind"] == "splice":
        s["omega"] = _omega(case).tolist()
    else:
        lens = _lengths(case)
        H, Hkv, d = case["heads"], case["kv_heads"], case["head_dim"]
        s["out"] = torch.zeros(s["q"].shape[:3] + (case["v_dim"],), dtype=s["q"].dtype, device="cuda")
        s["cu_q"] = _ints([0] + torch.tensor([q for q, _ in lens]).cumsum(0).tolist())
        s["kv_base"] = _ints([0] + torch.tensor([kv for _, kv in lens]).cumsum(0).tolist()[:-1], torch.int64)
        variant = pkv.PKV_ATTN_MLA if case["variant"] == "mla" else pkv.PKV_ATTN_GQA
        many = len(lens) > 1
        k, v = s["k"], s["v"]
        if case["page"]:   # the pool seen as [layer][head][slot][channel], for the descriptor's strides
            k, v = k[:, 0].transpose(1, 2), v[:, 0].transpose(1, 2)
        desc = pkv.make_attn_desc(s["q"], k, v, s["out"], max(kv for _, kv in lens), n_seqs=len(lens),
                                  cu_q=s["cu_q"] if many else None,
                                  kv_base=s["kv_base"] if many and not case["page"] else None,
                                  max_q=max(q for q, _ in lens), variant=variant, window=case["window"])
        if case["page"]:
            desc.cache_slots = s["table"].shape[1] * case["page"]
            s["paging"] = pkv.make_paging(s["table"], s["k"], s["v"])
        s["desc"] = desc
        s["bytes"] = pkv.pkv_attention_workspace_size(desc, H, Hkv, d)
        s["workspace"] = torch.empty(max(16, s["bytes"]), dtype=torch.uint8, device="cuda")
    return s


# ---- one pass -------------------------------------------------------------------

def _ok(status):
    if status != pkv.PKV_OK:
        raise pkv.PkvError(status, pkv.pkv_last_error())


def run(s):
    c = s["case"]
    if c["kind"] == "attention":
        args = (s["q"], s["k"], s["v"], s["out"], s["q_pos"], s["kv_len"], c["heads"], c["kv_heads"], c["head_dim"],
                s["scale"], s["desc"])
        if c["page"]:
            _ok(pkv.pkv_suffix_attention_paged(*args, s["paging"], s["workspace"], s["bytes"]))
        else:
            _ok(pkv.pkv_suffix_attention(*args, s["workspace"], s["bytes"]))
        return s["out"]
    if c["kind"] == "compose":
        pkv.reposition_splice_batched(s["src_k"], s["src_v"], s["dst_k"], s["dst_v"], s["segs"], s["n_segs"],
                                      s["longest"], c["theta"], c["head_dim"])
        return s["dst_k"], s["dst_v"]
    ends = (s["src_k"], s["src_v"], s["dst_k"], s["dst_v"], s["src_pos"], s["dst_pos"])
    if c["kind"] == "step":
        pkv.reposition_splice(*ends, c["theta"], c["head_dim"])
        pkv.suffix_attention(s["q"], s["dst_k"], s["dst_v"], s["out"], s["q_pos"], s["kv_len"], s["scale"],
                             c["slots"] + c["queries"])
        return s["dst_k"], s["dst_v"], s["out"]
    where = dict(rope_offset=c["rope_offset"], rope_style=STYLES[c["style"]])
    if c["entry"] == "paged":
        pkv.reposition_splice_paged(*ends, s["table"], c["theta"], c["rope_dim"], dst_capacity=c["slots"], **where)
    elif c["entry"] == "table":
        pkv.reposition_splice_freqs(*ends, s["omega"], c["rope_dim"], **where)
    else:
        pkv.reposition_splice(*ends, c["theta"], c["rope_dim"], **where)
    return s["dst_k"], s["dst_v"]


# ---- what a pass cannot do without ------------------------------------------------

def _attention_work(case, lens):
    """Keys some query sees, read once; queries read and outputs written; 2 (d + d_v) flops a visible pair."""
    d, dv, window = case["head_dim"], case.get("v_dim", case["head_dim"]), case.get("window", 0)
    row = d if case.get("variant") == "mla" else d + dv
    keys = pairs = 0
    for nq, kv in lens:
        first = max(0, kv - nq - window + 1) if window else 0
        keys += kv - first
        pairs += sum(min(kv - nq + i + 1, window) if window else kv - nq + i + 1 for i in range(nq))
    rows = sum(q for q, _ in lens)
    eb, L = ELEM[case["dtype"]], case["layers"]
    return (keys * case["kv_heads"] * row + rows * case["heads"] * (d + dv)) * eb * L, 2 * (d + dv) * case["heads"] * pairs * L


def work(case):
    eb = ELEM[case["dtype"]]
    if case["kind"] == "attention":
        nbytes, flops = _attention_work(case, _lengths(case))
        return {"bytes": nbytes, "flops": flops}
    if case["kind"] == "compose":
        segs, src, _, _ = _plan(case)
        tokens = sum(sg["n_tokens"] for sg in segs)
        per = case["layers"] * case["kv_heads"] * case["head_dim"]
        return {"bytes": 2 * (src + tokens) * per * eb, "flops": 3 * tokens * per}
    row = case["head_dim"] + case.get("v_dim", case["head_dim"])
    per = case["tokens"] * case["layers"] * case["kv_heads"]
    nbytes, flops = 2 * per * row * eb, 3 * per * case.get("rope_dim", case["head_dim"])
    if case["kind"] == "step":
        more, mul = _attention_work(case, [(case["queries"], case["slots"] + case["queries"])])
        nbytes, flops = nbytes + more, flops + mul
    return {"bytes": nbytes, "flops": flops}


# ---- results ----------------------------------------------------------------------

def tolerance(case):
    if case["kind"] == "attention":
        # bf16: probabilities and outputs are rounded to 8 bits, 2.2e-3 off the 64-bit result in the
        # 2-norm.  fp32: sums of some thousand products, 8e-7 off.
        return {"rel": 5e-6, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.1}
    if case["dtype"] == "f32":   # fp32 rotations and, in a whole step, the attention's sums
        return {"rel": 5e-6, "max": 1e-4}
    # One rounding to bf16 of an fp32 rotation: two implementations differ by an ulp in few elements.
    return {"rel": 1e-3, "max": 0.02}


def _turned(k, delta, case):
    """Keys [..., tokens, d] with their rotary slice turned by delta [tokens], in float64."""
    r, o = case.get("rope_dim", case["head_dim"]), case.get("rope_offset", 0)
    ang = delta.double()[:, None] * _omega(case).cuda()[None, :]
    c, s = ang.cos(), ang.sin()
    k = k.double()
    part = k[..., o:o + r].clone()
    if case.get("style", "half") == "half":
        a, b = part[..., : r // 2], part[..., r // 2:]
        k[..., o:o + r // 2], k[..., o + r // 2:o + r] = a * c - b * s, a * s + b * c
    else:
        a, b = part[..., 0::2], part[..., 1::2]
        k[..., o:o + r:2], k[..., o + 1:o + r:2] = a * c - b * s, a * s + b * c
    return k


def _attend(q, k, v, q_pos, scale, window):
    """Causal (and windowed) softmax attention of one KV head in float64: q [rows, G, d], k, v [kv, *]."""
    kv = k.shape[0]
    out = torch.empty(q.shape[:2] + (v.shape[1],), dtype=torch.float64, device=q.device)
    k64, v64 = k.double().contiguous(), v.double().contiguous()
    step = max(1, int(2.5e8 // (kv * q.shape[1])))
    for lo in range(0, q.shape[0], step):
        p = q_pos[lo:lo + step].long()
        x = q[lo:lo + step].double().reshape(-1, q.shape[2]) @ k64.t().contiguous()
        x = (x * scale).view(len(p), q.shape[1], kv)
        j = torch.arange(kv, device=q.device)
        hidden = j[None, :] > p[:, None]
        if window:
            hidden |= j[None, :] <= p[:, None] - window
        x.masked_fill_(hidden[:, None, :], -math.inf)
        w = torch.softmax(x, -1)
        out[lo:lo + step] = (w.view(-1, kv) @ v64).view(len(p), q.shape[1], -1)
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "attention":
        lens, G = _lengths(case), case["heads"] // case["kv_heads"]
        out = torch.empty(s["q"].shape[:3] + (case["v_dim"],), dtype=torch.float64, device="cuda")
        row, slot = 0, 0
        for i, (nq, kv) in enumerate(lens):
            for layer in range(case["layers"]):
                for g in range(case["kv_heads"]):
                    if case["page"]:
                        ids = s["table"][i].long()
                        k = s["k"][layer, ids, :, g].reshape(-1, s["k"].shape[-1])[:kv]
                        v = s["v"][layer, ids, :, g].reshape(-1, s["v"].shape[-1])[:kv]
                    else:
                        k, v = s["k"][layer, g, slot:slot + kv], s["v"][layer, g, slot:slot + kv]
                    heads = slice(g * G, (g + 1) * G)
                    out[layer, row:row + nq, heads] = _attend(s["q"][layer, row:row + nq, heads], k, v,
                                                              s["q_pos"][row:row + nq], _scale(case),
                                                              case["window"])
            row, slot = row + nq, slot + kv
        return out
    dk = s["dst_k"].double()
    dv = None if s["dst_v"] is None else s["dst_v"].double()
    if case["kind"] == "compose":
        for sg in _plan(case)[0]:
            n = sg["n_tokens"]
            src = slice(sg["src_slot0"], sg["src_slot0"] + n)
            lo = sg["dst_seq_base"] + sg["dst_pos0"]
            delta = torch.full((n,), sg["dst_pos0"] - sg["src_pos0"], device="cuda")
            dk[:, :, lo:lo + n] = _turned(s["src_k"][:, :, src], delta, case)
            dv[:, :, lo:lo + n] = s["src_v"][:, :, src].double()
        return dk, dv
    turned = _turned(s["src_k"], s["dst_pos"] - s["src_pos"], case)
    p = s["dst_pos"].long()
    if case.get("page"):
        ids, at = s["table"][0].long()[p // case["page"]], p % case["page"]
        dk[:, ids, at] = turned.transpose(1, 2)
        if dv is not None:
            dv[:, ids, at] = s["src_v"].double().transpose(1, 2)
    else:
        dk[:, :, p] = turned
        if dv is not None:
            dv[:, :, p] = s["src_v"].double()
    if case["kind"] != "step":
        return dk, dv
    G = case["heads"] // case["kv_heads"]
    # the suffix attends over the keys as the cache stores them
    out = torch.cat([_attend(s["q"][0, :, g * G:(g + 1) * G], dk[0, g], dv[0, g], s["q_pos"], _scale(case), 0)
                     for g in range(case["kv_heads"])], 1)[None]
    return dk, dv, out
