"""What a program that serves long contexts with this library spends its time on, as measurable cases.

A case is a dict of plain sizes; `kind` names the user's operation:
  layer      ParallelCompLayer.forward: chunk prefill with scores, chunk and token selection, KV
             compaction, global attention of the query block
  prefill    ParallelCompLayer.chunk_prefill alone (no selection follows in this layer)
  stream     StreamingParallelComp.forward: the same layer with the chunks arriving in batches
  decode     DecodeCache.step for a few tokens over the compressed 16-bit cache and the growing tail
  decode8    DecodeCacheFp8.step, the same over the 8-bit cache
  cache8     building the 8-bit cache from the selected tokens (pc_gather_kv_amax,
             pc_kv_quantize_fp8_amax) and the query block's attention over it (pc_parallel_attn_fp8)
  selfinfo   chunk selection by self-information from the language model's logits

The inputs are drawn on the GPU from the seed: unit-variance keys and values, queries with a gain
that gives logits a standard deviation of about 2 (a row's weight sits on a few dozen keys, as in
a trained model), a heavy first key in every chunk, and a fifth of the chunks carrying the query's
mean direction in their keys, so that chunks and tokens differ in relevance.
"""
import math
import random

import torch

import paper_2502_14317_amd as pc
from paper_2502_14317_amd.layer import (DecodeCache, DecodeCacheFp8, ParallelCompLayer,
                                        StreamingParallelComp, fp8_alloc)

BF16 = torch.bfloat16


# ------------------------------------------------------------------------------------------ cases
def _layer(name, C, w, wq, hq, hkv, d, base, kc, kt, obs=32, kind="layer", batch=0, ragged=False,
           lam=0.0, cls=0):
    case = {"kind": kind, "chunks": C, "w": w, "wq": wq, "hq": hq, "hkv": hkv, "d": d, "base": base,
            "keep_chunks": kc, "keep_tokens": kt, "obs": obs, "batch": batch, "ragged": ragged,
            "lam": lam, "cls": cls}
    return dict(case, name=name) if name else case


def _decode(name, kind, B, seg, kt, tail, tokens, hq, hkv, d, base, ragged=False):
    case = {"kind": kind, "batch": B, "segs": seg, "keep_tokens": kt, "tail": tail, "tokens": tokens,
            "hq": hq, "hkv": hkv, "d": d, "base": base, "ragged": ragged}
    return dict(case, name=name) if name else case


def _cache8(name, B, C, rows, seg, kt, nq, hq, hkv, d, base):
    case = {"kind": "cache8", "batch": B, "chunks": C, "rows": rows, "segs": seg, "keep_tokens": kt,
            "nq": nq, "hq": hq, "hkv": hkv, "d": d, "base": base}
    return dict(case, name=name) if name else case


def _selfinfo(name, C, tokens, vocab, keep):
    case = {"kind": "selfinfo", "chunks": C, "tokens": tokens, "vocab": vocab, "keep_chunks": keep}
    return dict(case, name=name) if name else case


def listed():
    return [
        # a short prompt through a small model: launches and latency, not arithmetic
        _layer("layer_tiny", 4, 512, 64, 8, 8, 64, 1e4, 2, 128),
        # one pre-training window of a Llama-2-7B-shaped layer (the paper's table starts at one chunk)
        _layer("layer_one_chunk", 1, 3584, 512, 32, 32, 128, 1e4, 1, 1792),
        # documents of unequal length with attention calibration and every query row voting (Eq. 6
        # as printed); no size a multiple of a tile
        _layer("layer_ragged", 12, 2011, 203, 32, 8, 128, 5e5, 5, 701, obs=203, ragged=True, lam=1.5, cls=100),
        # 128K tokens, Llama-3-8B-shaped layer: the workload the benchmark quotes
        _layer("layer_128k_gqa", 16, 7680, 512, 32, 8, 128, 5e5, 8, 2048),
        # 128K tokens, Llama-2-7B-shaped layer: many shorter chunks, one KV head per query head
        _layer("layer_128k_mha", 36, 3584, 512, 32, 32, 128, 1e4, 12, 1024),
        # 512K tokens, prefill and scores only: the longest context
        _layer("prefill_512k", 64, 8192, 512, 32, 8, 128, 5e5, 0, 0, kind="prefill"),
        # the 128K layer with the chunks arriving four at a time (memory-bound deployments)
        _layer("stream_128k", 16, 7680, 512, 32, 8, 128, 5e5, 8, 2048, kind="stream", batch=4),
        # one user's answer, token by token: small cache, latency of a step
        _decode("decode_one", "decode", 1, 8, 2048, 512, 8, 32, 8, 128, 5e5),
        # sixteen users' answers over 64K kept tokens each: the cache is read once per token
        _decode("decode_batch", "decode", 16, 32, 2048, 512, 2, 32, 8, 128, 5e5),
        # the same from the 8-bit cache
        _decode("decode_batch_8bit", "decode8", 16, 32, 2048, 512, 2, 32, 8, 128, 5e5),
        # after the prefill of four sequences: 8-bit cache from the selected tokens, then the
        # query block's attention over it
        _cache8("cache_8bit_build", 4, 16, 4096, 8, 2048, 512, 32, 8, 128, 5e5),
        # chunk selection by the paper's own criterion at a Llama-3 vocabulary
        _selfinfo("selfinfo_llama3", 16, 512, 128256, 8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "prefill", "stream", "decode", "decode8", "cache8", "selfinfo"])
    hq, hkv, d = rng.choice([(32, 8, 128), (32, 32, 128), (32, 8, 128), (8, 8, 64), (16, 4, 128), (24, 8, 64)])
    base = rng.choice([1e4, 5e5])
    if kind in ("layer", "prefill", "stream"):
        C, w, wq = _log_int(rng, 1, 36), _log_int(rng, 300, 7680), _log_int(rng, 24, 512)
        kc, kt = rng.randint(1, min(C, 12)), _log_int(rng, max(1, w // 8), max(2, w // 2))
        obs = rng.choice([8, 32, 32, wq])
        obs = min(obs, wq)
        if kind == "prefill":
            return _layer(None, C, w, wq, hq, hkv, d, base, 0, 0, obs, kind="prefill")
        if kind == "stream":
            return _layer(None, max(2, C), w, wq, hq, hkv, d, base, min(kc, max(2, C)), kt, obs,
                          kind="stream", batch=rng.randint(1, max(1, C // 2)))
        ragged = rng.random() < 0.3 and C <= 16
        return _layer(None, C, w, wq, hq, hkv, d, base, kc, kt, obs, ragged=ragged,
                      lam=0.05 * obs if ragged else 0.0, cls=min(100, w // 4) if ragged else 0)
    if kind in ("decode", "decode8"):
        return _decode(None, kind, _log_int(rng, 1, 16), _log_int(rng, 1, 32), _log_int(rng, 700, 2048),
                       _log_int(rng, 24, 512), rng.randint(1, 8), hq, hkv, d, base, ragged=rng.random() < 0.4)
    if kind == "cache8":
        C = rng.randint(2, 16)
        kt = _log_int(rng, 128, 2048)
        return _cache8(None, rng.randint(1, 4), C, kt + _log_int(rng, 64, 2048), rng.randint(1, min(C, 8)),
                       kt, _log_int(rng, 24, 512), hq, hkv, d, base)
    return _selfinfo(None, rng.randint(2, 16), _log_int(rng, 16, 512),
                     8 * rng.randint(4000, 16032), rng.randint(1, 2))


# ------------------------------------------------------------------------------------------ inputs
def _lens(case):
    """Context rows of every chunk: full in a plain layer, from w down to about w / 3 in a ragged one."""
    C, w = case["chunks"], case["w"]
    if not case["ragged"]:
        return [w] * C
    return [max(1, w - (c * c * 131 + 29 * c) % max(1, 2 * w // 3)) for c in range(C)]


def _normal(gen, shape, gain=1.0):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=BF16)
    return x if gain == 1.0 else x.mul_(gain)


def _layer_inputs(case, seed):
    C, w, wq, hq, hkv, d = (case[k] for k in ("chunks", "w", "wq", "hq", "hkv", "d"))
    L, lens = w + wq, _lens(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = _normal(gen, (C, L, hq, d), 2.0), _normal(gen, (C, L, hkv, d)), _normal(gen, (C, L, hkv, d))
    qq, kq, vq = (x[0, w:].clone() for x in (q, k, v))                 # the query rows, the same in every chunk
    u = qq.float().view(wq, hkv, hq // hkv, d).mean(dim=(0, 2))
    u = (0.25 * math.sqrt(d) * u / u.norm(dim=-1, keepdim=True)).to(BF16)
    relevant = random.Random(seed).sample(range(C), max(1, C // 5))
    for c in range(C):
        n = lens[c]
        if c in relevant:
            k[c, :n] += u
        k[c, 0] *= 1.5
        q[c, n:n + wq], k[c, n:n + wq], v[c, n:n + wq] = qq, kq, vq
    return q, k, v, lens


def _segments(gen, case):
    shape = (case["batch"], case["segs"], case["hkv"], case["keep_tokens"], case["d"])
    return _normal(gen, shape), _normal(gen, shape)


def _decode_inputs(case, seed):
    """Compressed segments, their lengths (None: full), tail rows (keys rotated), the new tokens' q, k, v."""
    B, S, kt, tail, T, hq, hkv, d = (case[k] for k in ("batch", "segs", "keep_tokens", "tail", "tokens", "hq", "hkv", "d"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kc, vc = _segments(gen, case)
    seg_len = None
    if case["ragged"]:
        seg_len = torch.randint(kt // 2, kt + 1, (B, S), generator=gen, device="cuda", dtype=torch.int32)
    k_tail, v_tail = _normal(gen, (B, tail, hkv, d)), _normal(gen, (B, tail, hkv, d))
    return (kc, vc, seg_len, k_tail, v_tail, _normal(gen, (T, B, 1, hq, d), 2.0), _normal(gen, (T, B, 1, hkv, d)),
            _normal(gen, (T, B, 1, hkv, d)))


def _cache8_inputs(case, seed):
    """Source rows of K and V, the kept chunks and tokens, the query block's q, k, v."""
    B, C, rows, S, kt, nq, hq, hkv, d = (case[k] for k in ("batch", "chunks", "rows", "segs", "keep_tokens", "nq", "hq", "hkv", "d"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    src, i32 = (B, C, rows, hkv, d), torch.int32
    chunk_idx = torch.rand((B, C), generator=gen, device="cuda").argsort(dim=1)[:, :S].to(i32).contiguous()
    tok_idx = torch.rand((B, S, hkv, rows), generator=gen, device="cuda").argsort(dim=-1)[..., :kt]
    tok_idx = tok_idx.sort(dim=-1).values.to(i32).contiguous()
    return (_normal(gen, src), _normal(gen, src), chunk_idx, tok_idx, _normal(gen, (B, nq, hq, d), 2.0),
            _normal(gen, (B, nq, hkv, d)), _normal(gen, (B, nq, hkv, d)))


def _selfinfo_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    C, T, V = case["chunks"], case["tokens"], case["vocab"]
    return (_normal(gen, (C, T, V), 2.0),
            torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("layer", "prefill", "stream"):
        q, k, v, lens = _layer_inputs(case, seed)
        sizes = (case["w"], case["wq"], case["hq"], case["hkv"], case["d"], case["obs"], case["base"],
                 case["keep_chunks"], case["keep_tokens"])
        s = {"case": case, "q": q, "k": k, "v": v, "lens": lens, "dev_lens": None}
        if kind == "stream":
            s["layer"] = StreamingParallelComp(case["chunks"], case["batch"], *sizes)
            return s
        cal = (case["lam"], 0, case["cls"]) if case["cls"] else None
        s["layer"] = ParallelCompLayer(case["chunks"], *sizes, calibration=cal)
        if case["ragged"]:
            s["dev_lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
        return s
    if kind in ("decode", "decode8"):
        B, S, kt, tail, T, hq, hkv, d = (case[k] for k in ("batch", "segs", "keep_tokens", "tail", "tokens", "hq", "hkv", "d"))
        kc, vc, seg_len, k_tail, v_tail, q, k, v = _decode_inputs(case, seed)
        if kind == "decode":
            cache = DecodeCache(B, S, kt, hq, hkv, d, case["base"])
        else:
            cache = DecodeCacheFp8(B, S, kt, tail + T, hq, hkv, d, case["base"])
        cache.load(kc, vc, seg_len, k_tail, v_tail)
        return {"case": case, "cache": cache, "q": q, "k": k, "v": v,
                "outs": torch.empty((T, B, 1, hq, d), dtype=BF16, device="cuda")}
    f32 = torch.float32
    if kind == "cache8":
        B, C, rows, S, kt, nq, hq, hkv, d = (case[k] for k in ("batch", "chunks", "rows", "segs", "keep_tokens", "nq", "hq", "hkv", "d"))
        k_src, v_src, chunk_idx, tok_idx, q, k_self, v_self = _cache8_inputs(case, seed)
        kc = torch.empty((B, S, hkv, kt, d), dtype=BF16, device="cuda")
        return {"case": case, "k_src": k_src, "v_src": v_src, "chunk_idx": chunk_idx, "tok_idx": tok_idx,
                "kc": kc, "vc": torch.empty_like(kc),
                "k_amax": torch.empty((B, S, hkv), dtype=f32, device="cuda"),
                "v_amax": torch.empty((B, S, hkv), dtype=f32, device="cuda"),
                "k8": fp8_alloc(B, S, hkv, kt, d), "v8": fp8_alloc(B, S, hkv, kt, d),
                "k_scale": torch.empty((B, S, hkv), dtype=f32, device="cuda"),
                "v_scale": torch.empty((B, S, hkv), dtype=f32, device="cuda"),
                "q": q, "k_self": k_self, "v_self": v_self,
                "out": torch.empty((B, nq, hq, d), dtype=BF16, device="cuda"),
                "lse": torch.empty((B, hq, nq), dtype=f32, device="cuda"),
                "ws": pc.alloc_workspace(pc.pc_parallel_attn_fp8_workspace_bytes(B, nq, S, kt, 0, hq, hkv, d, True))}
    C, T, keep = (case[k] for k in ("chunks", "tokens", "keep_chunks"))
    logits, targets = _selfinfo_inputs(case, seed)
    return {"case": case, "logits": logits, "targets": targets,
            "nll": torch.empty((C, T), dtype=f32, device="cuda"),
            "info": torch.empty((C,), dtype=f32, device="cuda"),
            "idx": torch.empty((keep,), dtype=torch.int32, device="cuda"),
            "top": torch.empty((keep,), dtype=f32, device="cuda")}


# ------------------------------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("layer", "prefill"):
        layer, lens, wq = s["layer"], s["lens"], case["wq"]
        if kind == "prefill":
            layer.chunk_prefill(s["q"], s["k"], s["v"])
        elif s["dev_lens"] is None:
            layer.forward(s["q"], s["k"], s["v"])
        else:
            layer.forward(s["q"], s["k"], s["v"], chunk_lens=s["dev_lens"], first_len=lens[0])
        out = {"tok_score": layer.tok_score, "chunk_score": layer.chunk_score}
        if s["dev_lens"] is None:
            out.update(o=layer.o, lse=layer.lse, k_rope=layer.k_rope)
        else:           # rows behind a short sequence are padding and hold nothing
            out.update(o=[layer.o[c, :n + wq] for c, n in enumerate(lens)],
                       lse=[layer.lse[c, :, :n + wq] for c, n in enumerate(lens)],
                       k_rope=[layer.k_rope[c, :n + wq] for c, n in enumerate(lens)], tok_cnt=layer.tok_cnt)
        if kind == "layer":
            # the compacted K / V are rows of k_rope and v at tok_idx, copied bit for bit
            out.update(chunk_idx=layer.chunk_idx, tok_idx=layer.tok_idx, global_o=layer.global_o,
                       global_lse=layer.global_lse)
        return out
    if kind == "stream":
        layer = s["layer"]
        layer.forward(s["q"], s["k"], s["v"])
        return {"chunk_score": layer.chunk_score, "queue_id": layer.queue_id, "queue_score": layer.queue_score,
                "queue_slot": layer.queue_slot, "tok_idx": layer.tok_idx, "o": layer.o, "lse": layer.lse,
                "k_rope": layer.k_rope, "global_o": layer.global_o, "global_lse": layer.global_lse}
    if kind in ("decode", "decode8"):
        cache, tail = s["cache"], case["tail"]
        # an answer starts behind the query block: the tail is set back to it, then grows by a row a
        # token; every step's output goes to a buffer of its own, where the layer behind finds it
        tail_len = cache.seg_len[:, -1] if kind == "decode" else cache.tail_len
        tail_len.fill_(tail)
        for t in range(case["tokens"]):
            cache.out = s["outs"][t]
            cache.step(s["q"][t], s["k"][t], s["v"][t], 7680 + tail + t)
        if kind == "decode":
            k_tail, v_tail = cache.kc[:, -1, :, :tail + case["tokens"]], cache.vc[:, -1, :, :tail + case["tokens"]]
        else:
            k_tail, v_tail = cache.k_tail, cache.v_tail
        return {"outs": s["outs"], "lse": cache.lse, "tail_len": tail_len, "k_tail": k_tail, "v_tail": v_tail}
    if kind == "cache8":
        B, C, rows, S, kt, nq, hq, hkv, d = (case[k] for k in ("batch", "chunks", "rows", "segs", "keep_tokens", "nq", "hq", "hkv", "d"))
        pc.pc_gather_kv_amax(s["k_src"], s["v_src"], s["chunk_idx"], s["tok_idx"], B, C, rows, S, hkv, kt, d,
                             s["kc"], s["vc"], s["k_amax"], s["v_amax"])
        pc.pc_kv_quantize_fp8_amax(s["kc"], s["vc"], s["k_amax"], s["v_amax"], None, B, S, kt, hkv, d,
                                   s["k8"], s["v8"], s["k_scale"], s["v_scale"])
        pc.pc_parallel_attn_fp8(s["q"], s["k8"], s["v8"], s["k_scale"], s["v_scale"], None, None, None, None, 0,
                                B, nq, S, kt, hq, hkv, d, rows, case["base"], 0.0, s["out"], s["lse"], s["ws"],
                                k_self=s["k_self"], v_self=s["v_self"])
        return {k: s[k] for k in ("kc", "vc", "k_amax", "v_amax", "k8", "v8", "k_scale", "v_scale", "out", "lse")}
    C, T, V, keep = (case[k] for k in ("chunks", "tokens", "vocab", "keep_chunks"))
    pc.pc_chunk_self_information(s["logits"], s["targets"], C, T, V, True, s["nll"], s["info"])
    pc.pc_select_chunks_topk(s["info"], C, keep, s["idx"], s["top"])
    return {k: s[k] for k in ("nll", "info", "idx", "top")}


# ------------------------------------------------------------------------------------------ bounds
def work(case):
    kind = case["kind"]
    if kind in ("layer", "prefill", "stream"):
        wq, hq, hkv, d, obs = (case[k] for k in ("wq", "hq", "hkv", "d", "obs"))
        kc, kt = case["keep_chunks"], case["keep_tokens"]
        lens = _lens(case)
        rows = sum(n + wq for n in lens)
        flops = sum(4.0 * d * hq * (n + wq) * (n + wq + 1) / 2 + 2.0 * d * hq * obs * (n + wq) for n in lens)
        # q in, o out, k and v in, rotated keys out, lse and scores out
        n_bytes = 2.0 * rows * d * (2 * hq + 3 * hkv) + 4.0 * rows * hq + 4.0 * sum(lens) * hkv
        if kc:
            flops += 4.0 * d * hq * (wq * kc * kt + wq * (wq + 1) / 2)
            n_bytes += 8.0 * kc * hkv * kt * d + 4.0 * wq * d * hq        # compacted K / V in and out, query block
        return {"bytes": n_bytes, "flops": flops}
    if kind in ("decode", "decode8"):
        B, S, kt, tail, T, hq, hkv, d = (case[k] for k in ("batch", "segs", "keep_tokens", "tail", "tokens", "hq", "hkv", "d"))
        seg_rows = S * kt * (0.75 if case["ragged"] else 1.0)
        elem = 2.0 if kind == "decode" else 1.0
        per_token = B * hkv * d * 2.0 * (seg_rows * elem + (tail + 0.5 * T) * 2.0) + 4.0 * B * hq * d
        return {"bytes": T * per_token, "flops": T * 4.0 * B * hq * d * (seg_rows + tail)}
    if kind == "cache8":
        B, S, kt, nq, hq, hkv, d = (case[k] for k in ("batch", "segs", "keep_tokens", "nq", "hq", "hkv", "d"))
        kept = 2.0 * B * S * hkv * kt * d                                    # values of K and V
        # rows read, compacted rows written, codes written and read by the attention
        return {"bytes": kept * (2 + 2 + 1 + 1) + 2.0 * B * nq * d * (2 * hq + 2 * hkv),
                "flops": 4.0 * B * hq * d * (nq * S * kt + nq * (nq + 1) / 2)}
    return {"bytes": 2.0 * case["chunks"] * case["tokens"] * case["vocab"],
            "flops": 4.0 * case["chunks"] * case["tokens"] * case["vocab"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "selfinfo":
        return {"rel": 1e-6}        # 32-bit sums of a vocabulary row: 5e-8 from the sum in 64 bits
    # bf16 operands, probabilities and outputs: 3e-3 to 5.4e-3 from the same attention in 64 bits, so two
    # correct implementations lie up to 8e-3 apart (codes, scales and lengths stay exact)
    if kind in ("decode", "decode8", "cache8"):
        return {"rel": 1e-2}
    # Scores are good to a few 1e-6, so of two tokens that close at the k-th place
    # either may be kept: the kept list of one (chunk, head) then shifts between their places.
    return {"rel": 1e-2, "differ": 0.01}


# ------------------------------------------------------------------------------------------ in 64 bits
def _rope64(x, pos, base):
    """Rotation of the pairs (i, i + d / 2) of x [..., rows, d] at the positions pos [rows]."""
    d = x.shape[-1]
    theta = base ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    ang = pos.to(torch.float64)[:, None] * theta
    c, s, a, b = ang.cos(), ang.sin(), x[..., :d // 2], x[..., d // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _attend64(q, k, v, offset=None, votes=0):
    """softmax(q k^T / sqrt(d)) v for q [rows, d] and its logsumexp, rows in blocks; row r sees the keys up to
    r + offset (None: all); votes: also the sum over the last `votes` rows of the probability of every key."""
    n, d = q.shape
    out, lse = torch.empty_like(q), torch.empty(n, dtype=torch.float64, device=q.device)
    score = torch.zeros(k.shape[0], dtype=torch.float64, device=q.device) if votes else None
    kt = k.t().contiguous()
    for r0 in range(0, n, 2048):
        r1 = min(r0 + 2048, n)
        m = k.shape[0] if offset is None else min(k.shape[0], r1 + offset)
        s = (q[r0:r1] @ kt[:, :m].contiguous()) / math.sqrt(d)
        if offset is not None:
            rows = torch.arange(r0, r1, device=q.device)[:, None]
            s.masked_fill_(torch.arange(m, device=q.device)[None] > rows + offset, float("-inf"))
        lse[r0:r1] = torch.logsumexp(s, dim=1)
        p = s.sub_(lse[r0:r1, None]).exp_()
        out[r0:r1] = p @ v[:m]
        if r1 > n - votes:
            score[:m] += p[max(0, n - votes - r0):].sum(dim=0)
    return out, lse, score


def _exact_layer(case, seed):
    C, w, wq, hq, hkv, d, obs = (case[k] for k in ("chunks", "w", "wq", "hq", "hkv", "d", "obs"))
    kc, kt, stream = case["keep_chunks"], case["keep_tokens"], case["kind"] == "stream"
    q, k, v, lens = _layer_inputs(case, seed)
    G, L, dev, f64 = hq // hkv, w + wq, "cuda", torch.float64
    tok = torch.zeros((C, hkv, w), dtype=f64, device=dev)
    o, lse, kr, q0, k_kept = [], [], [], None, []
    for c, n in enumerate(lens):
        pos = torch.arange(n + wq, device=dev)
        qc = _rope64(q[c, :n + wq].transpose(0, 1).to(f64), pos, case["base"])
        kcx = _rope64(k[c, :n + wq].transpose(0, 1).to(f64), pos, case["base"])
        vcx = v[c, :n + wq].transpose(0, 1).to(f64)
        oc, lc = [], []
        for h in range(hq):
            x, y, z = _attend64(qc[h], kcx[h // G], vcx[h // G], 0, obs)
            oc.append(x.float()); lc.append(y); tok[c, h // G, :n] += z[:n]
        o.append(torch.stack(oc, dim=1)); lse.append(torch.stack(lc)); kr.append(kcx.transpose(0, 1).float())
        if c == 0 and kc:
            q0, k_self, v_self = qc[:, n:], kcx[:, n:], vcx[:, n:]
    chunk = tok.sum(dim=(1, 2))
    out = {"chunk_score": chunk}
    if case["ragged"]:
        out.update(tok_score=tok, o=o, lse=lse, k_rope=kr, tok_cnt=None)
    elif stream:                     # the batch buffers hold the last batch, behind it rows of the one before
        b = min(case["batch"], C)
        last = [max(c for c in range(C) if c % b == i) for i in range(b)]
        out.update(o=torch.stack([o[c] for c in last]), lse=torch.stack([lse[c] for c in last]),
                   k_rope=torch.stack([kr[c] for c in last]))
    else:
        out.update(tok_score=tok, o=torch.stack(o), lse=torch.stack(lse), k_rope=torch.stack(kr))
    if kc:
        go = torch.empty((1, wq, hq, d), dtype=f64, device=dev)
        gl = torch.empty((1, hq, wq), dtype=f64, device=dev)
        kept = chunk.argsort(descending=True, stable=True)[:kc].tolist()
        for g in range(hkv):
            ks, vs = [], []
            for c in kept:
                t = tok[c, g, :lens[c]].clone()
                if case["cls"]:
                    head = t[:case["cls"]]
                    head[head > case["lam"]] = -1.0
                idx = t.argsort(descending=True, stable=True)[:kt]
                idx = idx[t[idx] >= 0]
                ks.append(kr[c][idx, g].to(f64)); vs.append(v[c, idx, g].to(f64))
            ks, vs = torch.cat(ks + [k_self[g]]), torch.cat(vs + [v_self[g]])
            for h in range(g * G, (g + 1) * G):
                go[0, :, h], gl[0, h], _ = _attend64(q0[h], ks, vs, ks.shape[0] - wq)
        out.update(global_o=go, global_lse=gl, tok_idx=None)
        out.update({"queue_id": None, "queue_score": None, "queue_slot": None} if stream else {"chunk_idx": None})
    return out


def _exact_decode(case, seed):
    B, tail, T, hq, hkv, d = (case[k] for k in ("batch", "tail", "tokens", "hq", "hkv", "d"))
    kc, vc, seg_len, k_tail, v_tail, q, k, v = _decode_inputs(case, seed)
    if case["kind"] == "decode8":
        kc, vc = ((c * s[..., None, None]).to(torch.float64) for c, s in (_e4m3(x, seg_len) for x in (kc, vc)))
    G, f64 = hq // hkv, torch.float64
    pos = 7680 + tail + torch.arange(T, device="cuda")
    outs = torch.empty((T, B, 1, hq, d), dtype=f64, device="cuda")
    lse = torch.empty((B, hq, 1), dtype=f64, device="cuda")
    for b in range(B):
        n = [case["keep_tokens"]] * case["segs"] if seg_len is None else seg_len[b].tolist()
        for g in range(hkv):
            new = _rope64(k[:, b, 0, g].to(f64), pos, case["base"])
            ks = torch.cat([kc[b, s, g, :m].to(f64) for s, m in enumerate(n)] + [k_tail[b, :, g].to(f64), new])
            vs = torch.cat([vc[b, s, g, :m].to(f64) for s, m in enumerate(n)] + [v_tail[b, :, g].to(f64), v[:, b, 0, g].to(f64)])
            for h in range(g * G, (g + 1) * G):
                x, y, _ = _attend64(_rope64(q[:, b, 0, h].to(f64), pos, case["base"]), ks, vs, ks.shape[0] - T)
                outs[:, b, 0, h], lse[b, h, 0] = x, y[-1]
    return {"outs": outs, "lse": lse, "tail_len": None, "k_tail": None, "v_tail": None}


def _e4m3(x, seg_len=None):
    """The 8-bit cache's values: E4M3 codes (as numbers) of the valid rows of x [B, S, hkv, rows, d] over a scale."""
    x = x.float()
    if seg_len is not None:
        x = x * (torch.arange(x.shape[3], device=x.device) < seg_len[:, :, None, None])[..., None]
    scale = x.abs().amax(dim=(3, 4)) / 448.0
    scale = torch.where(scale > 0, scale, torch.ones_like(scale))
    return (x / scale[..., None, None]).to(torch.float8_e4m3fn).float(), scale


def _exact_cache8(case, seed):
    B, C, S, kt, nq, hq, hkv, d = (case[k] for k in ("batch", "chunks", "segs", "keep_tokens", "nq", "hq", "hkv", "d"))
    k_src, v_src, chunk_idx, tok_idx, q, k_self, v_self = _cache8_inputs(case, seed)
    G, f64 = hq // hkv, torch.float64
    b_, g_ = torch.arange(B, device="cuda").view(B, 1, 1, 1), torch.arange(hkv, device="cuda").view(1, 1, hkv, 1)
    where = (b_, chunk_idx.long()[:, :, None, None], tok_idx.long(), g_)
    kc, vc = k_src[where], v_src[where]
    (k8, k_scale), (v8, v_scale) = _e4m3(kc), _e4m3(vc)
    out = torch.empty((B, nq, hq, d), dtype=f64, device="cuda")
    lse = torch.empty((B, hq, nq), dtype=f64, device="cuda")
    pos = case["rows"] + torch.arange(nq, device="cuda")
    for b in range(B):
        for g in range(hkv):
            ks = torch.cat([(k8[b, :, g].to(f64) * k_scale[b, :, g, None, None]).flatten(0, 1), k_self[b, :, g].to(f64)])
            vs = torch.cat([(v8[b, :, g].to(f64) * v_scale[b, :, g, None, None]).flatten(0, 1), v_self[b, :, g].to(f64)])
            for h in range(g * G, (g + 1) * G):
                out[b, :, h], lse[b, h], _ = _attend64(_rope64(q[b, :, h].to(f64), pos, case["base"]), ks, vs, ks.shape[0] - nq)
    return {"kc": None, "vc": None, "k_amax": None, "v_amax": None, "k8": None, "v8": None,
            "k_scale": k_scale, "v_scale": v_scale, "out": out, "lse": lse}


def _exact_selfinfo(case, seed):
    logits, targets = _selfinfo_inputs(case, seed)
    nll = []
    for c in range(case["chunks"]):
        x = logits[c].to(torch.float64)
        nll.append(torch.logsumexp(x, dim=1) - x.gather(1, targets.long()[:, None])[:, 0])
    nll = torch.stack(nll)
    return {"nll": nll, "info": -nll.sum(dim=1), "idx": None, "top": None}


def exact(case, seed):
    """What run() returns, in 64 bits (codes, copies and lists of places: None)."""
    kind = case["kind"]
    if kind in ("layer", "prefill", "stream"):
        return _exact_layer(case, seed)
    return {"decode": _exact_decode, "decode8": _exact_decode, "cache8": _exact_cache8, "selfinfo": _exact_selfinfo}[kind](case, seed)
