"""The work that serving with this engine consists of, as measurable cases.

A case is one pass through the public entry points: prefill and decode calls of a pipeline stage on
resident weights, a cold start from pinned host memory, the KV-cache move of a consolidation, and the
attention of one layer through its own entry point. Shapes are those of ``workloads`` (the tiny model,
7B, 13B and 8B-GQA); weights are N(0, 0.02) with norm gains around one, hidden states N(0, 1), all made
on the GPU from the seed. ``exact`` is the same decoder in 64 bits, in plain torch.
"""
from __future__ import annotations

import math
import random
import struct

import torch

from paper_2502_15524_amd import hs, pipeline
from workloads import MODELS

DEV = "cuda"
BLOCK = 16  # tokens per KV block


def listed():
    return [
        # The smallest whole model: a 32-token prompt and 16 decode steps, embedding to logits.
        # Latency and launches are all there is.
        dict(name="tiny-generate", kind="generate", model="tiny", begin=0, end=2, seqs=1, lo=32, hi=32, steps=16),
        # One 512-token prompt through layers of a middle stage: the prefill of a cold-started pipeline.
        dict(name="7b-prefill-1x512", kind="prefill", model="llama2-7b", begin=8, end=10, seqs=1, lo=512, hi=512, steps=0),
        # A full batch of equal prompts through one layer.
        dict(name="7b-prefill-8x1024", kind="prefill", model="llama2-7b", begin=16, end=17, seqs=8, lo=1024, hi=1024, steps=0),
        # Ragged prompts with grouped-query heads, the largest prefill of the workloads.
        dict(name="8b-prefill-ragged16", kind="prefill", model="llama3-8b", begin=8, end=9, seqs=16, lo=128, hi=2048, steps=0),
        # A few short chat turns: more rows than a decode step has, far fewer than a document.
        dict(name="13b-prefill-short4", kind="prefill", model="llama2-13b", begin=5, end=6, seqs=4, lo=17, hi=96, steps=0),
        # One user's decode in the middle of the pipeline.
        dict(name="7b-decode-b1", kind="decode", model="llama2-7b", begin=8, end=10, seqs=1, lo=512, hi=512, steps=8),
        # The last stage of a merged worker: takes over 16 ragged caches and decodes, LM head included.
        dict(name="8b-decode-b16-head", kind="decode", model="llama3-8b", begin=31, end=32, seqs=16, lo=128, hi=2048, steps=8),
        # A busy worker: more sequences than one 16-token MFMA chunk holds.
        dict(name="13b-decode-b40", kind="decode", model="llama2-13b", begin=20, end=21, seqs=40, lo=64, hi=1024, steps=8),
        # The cold start itself: the layer's weights stream from pinned memory while the prompt prefills.
        dict(name="7b-cold-1x512", kind="cold", model="llama2-7b", begin=8, end=9, seqs=1, lo=512, hi=512, steps=0),
        # Consolidation: a stage's cache gathered, scattered into another worker and gathered there again.
        dict(name="8b-kv-move", kind="move", model="llama3-8b", begin=4, end=8, seqs=16, lo=128, hi=2048, steps=0),
        # The attention of one layer over long prompts, by itself.
        dict(name="13b-attn-prefill-4x2048", kind="attn_prefill", model="llama2-13b", begin=0, end=1, seqs=4, lo=2048, hi=2048, steps=0),
        # The attention of one decode step over long ragged caches, RoPE and cache append included.
        dict(name="8b-attn-decode-b32", kind="attn_decode", model="llama3-8b", begin=0, end=1, seqs=32, lo=256, hi=4096, steps=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: prompts of 16 to 16K tokens in 1 to 16 sequences, decode batches of 1 to 64, every model."""
    kind = rng.choices(["prefill", "decode", "attn_prefill", "attn_decode", "move", "generate"], [8, 7, 2, 2, 1, 1])[0]
    if kind == "generate":
        n = rng.randint(1, 6)
        hi = rng.randint(2, 60)
        return dict(kind=kind, model="tiny", begin=0, end=2, seqs=n, lo=rng.randint(1, hi), hi=hi, steps=rng.randint(4, 16))
    model = rng.choice(["llama2-7b", "llama2-13b", "llama3-8b"])
    layers = MODELS[model].n_layers
    if kind == "prefill":
        n = _log_int(rng, 1, 16)
        total = _log_int(rng, max(16, 2 * n), 9000 if model == "llama2-13b" else 15000)
        hi = max(2, min(4096, 2 * total // (n + 1)))
        lo = max(1, min(hi, int(hi * rng.uniform(0.1, 1.0))))
        head = rng.random() < 0.2  # the last stage: one row of logits a sequence
        begin = layers - 1 if head else rng.randint(1, layers - 2)
        return dict(kind=kind, model=model, begin=begin, end=begin + 1, seqs=n, lo=lo, hi=hi, steps=0)
    if kind == "decode":
        n = _log_int(rng, 1, 64)
        hi = _log_int(rng, 32, min(4000, 60000 // n))
        head = rng.random() < 0.3
        begin = layers - 1 if head else rng.randint(1, layers - 2)
        return dict(kind=kind, model=model, begin=begin, end=begin + 1, seqs=n, lo=rng.randint(max(1, hi // 8), hi), hi=hi, steps=rng.randint(4, 8))
    if kind == "attn_prefill":
        n = _log_int(rng, 1, 8)
        hi = _log_int(rng, 64, min(8192, 16000 // n))
        return dict(kind=kind, model=model, begin=0, end=1, seqs=n, lo=rng.randint(max(1, hi // 4), hi), hi=hi, steps=0)
    if kind == "attn_decode":
        n = _log_int(rng, 1, 64)
        hi = _log_int(rng, 64, min(8192, 120000 // n))
        return dict(kind=kind, model=model, begin=0, end=1, seqs=n, lo=rng.randint(max(1, hi // 8), hi), hi=hi, steps=0)
    n = _log_int(rng, 1, 16)
    hi = _log_int(rng, 64, 2048)
    return dict(kind="move", model=model, begin=4, end=4 + rng.randint(1, 3), seqs=n, lo=rng.randint(max(1, hi // 8), hi), hi=hi, steps=0)


# ------------------------------------------------------------------ inputs


def lengths(case):
    """Prompt or cache lengths of the case's sequences."""
    r = random.Random("%d %d %d" % (case["seqs"], case["lo"], case["hi"]))
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["seqs"])]


def _normal(seed, what, shape, std, mean=0.0):
    """bf16 normal values on the GPU, from the seed and the tensor's name alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(random.Random("%d %s" % (seed, what)).getrandbits(48))
    x = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(mean, std, generator=g)
    return x.to(torch.bfloat16)


def weight(cfg, seed, layer, kind):
    """One tensor of the model, [out][in] (gains and embedding as usual)."""
    h, d = cfg.hidden, cfg.head_dim
    shape = dict(attn_norm=(h,), ffn_norm=(h,), final_norm=(h,), wq=(cfg.n_heads * d, h), wk=(cfg.n_kv_heads * d, h),
                 wv=(cfg.n_kv_heads * d, h), wo=(h, cfg.n_heads * d), wgate=(cfg.ffn, h), wup=(cfg.ffn, h),
                 wdown=(h, cfg.ffn), embed=(cfg.vocab, h), lm_head=(cfg.vocab, h))[kind]
    if kind.endswith("norm"):
        return _normal(seed, "%d %s" % (layer, kind), shape, 0.1, 1.0)
    # an embedding of unit scale stands for the residual stream of a trained model
    return _normal(seed, "%d %s" % (layer, kind), shape, 1.0 if kind == "embed" else 0.02)


def _tile(w):
    """Row-major [rows][cols] -> the tiled matrix format of the weight image (include/hs.h)."""
    rows, cols = w.shape
    kp = -(-cols // 64) * 64
    if kp != cols:
        w = torch.nn.functional.pad(w, (0, kp - cols))
    v = w.view(rows // 8, 8, kp // 64, 8, 8).permute(2, 0, 1, 3, 4)  # [kb][nb][row][chunk][8]
    r = torch.arange(8, device=w.device)
    return v[:, :, r[:, None], r[None, :] ^ r[:, None]].reshape(-1)


def _halves(w, d):
    """The two RoPE halves of every head interleaved in groups of 16 rows."""
    n, k = w.shape
    return w.view(n // d, 2, d // 32, 16, k).transpose(1, 2).reshape(n, k)


def image(cfg, seed, begin, end):
    """The packed weight image of layers [begin, end) in pinned host memory."""
    descs, nbytes = hs.hs_weight_layout(pipeline.hs_cfg(cfg), begin, end)
    buf = pipeline.PinnedBuffer(nbytes)
    host = torch.from_numpy(buf.numpy())
    for t in descs:
        w = lambda kind: weight(cfg, seed, t["layer"], kind)  # noqa: E731, B023
        kind = t["kind"]
        if kind == hs.HS_W_QKV:
            x = _tile(torch.cat([_halves(w("wq"), cfg.head_dim), _halves(w("wk"), cfg.head_dim), w("wv")]))
        elif kind == hs.HS_W_GATEUP:
            x = _tile(torch.stack([w("wgate").view(-1, 16, cfg.hidden), w("wup").view(-1, 16, cfg.hidden)], 1).reshape(-1, cfg.hidden))
        elif kind in (hs.HS_W_O, hs.HS_W_DOWN, hs.HS_W_LM_HEAD):
            x = _tile(w({hs.HS_W_O: "wo", hs.HS_W_DOWN: "wdown", hs.HS_W_LM_HEAD: "lm_head"}[kind]))
        else:
            x = w({hs.HS_W_EMBED: "embed", hs.HS_W_ATTN_NORM: "attn_norm", hs.HS_W_FFN_NORM: "ffn_norm", hs.HS_W_FINAL_NORM: "final_norm"}[kind])
        host[t["offset"]:t["offset"] + t["bytes"]].copy_(x.reshape(-1).view(torch.uint8))
    return buf


def _blocks(n):
    return -(-n // BLOCK)


def cache(cfg, seed, begin, end, lens):
    """Random post-RoPE keys and values, [layer][block][K | V][kv head][slot][d], zero past each sequence's end."""
    x = _normal(seed, "cache", (end - begin, sum(map(_blocks, lens)), 2, cfg.n_kv_heads, BLOCK, cfg.head_dim), 1.25)
    at = 0
    for n in lens:
        at += _blocks(n)
        if n % BLOCK:
            x[:, at - 1, :, :, n % BLOCK:] = 0
    return x


def blob(cfg, seed, begin, end, lens):
    """A KV blob (include/hs.h) of these sequences on the GPU, and its header and records."""
    x = cache(cfg, seed, begin, end, lens).reshape(-1).view(torch.uint8)
    off = -(-(64 + 16 * len(lens)) // 256) * 256
    head = struct.pack("<4sIIiiiiiiIQQQ", b"HSKV", 1, 1, begin, end, cfg.n_kv_heads, cfg.head_dim, BLOCK, len(lens), 0, off, x.numel(), off + x.numel())
    head += b"".join(struct.pack("<qii", i, n, _blocks(n)) for i, n in enumerate(lens))
    head += bytes(off - len(head))
    return torch.cat([torch.frombuffer(bytearray(head), dtype=torch.uint8).to(DEV), x]), head


def _stage_inputs(case, seed, rows, what):
    cfg = MODELS[case["model"]]
    if case["begin"] == 0:
        g = torch.Generator(device=DEV)
        g.manual_seed(random.Random("%d %s" % (seed, what)).getrandbits(48))
        return torch.randint(0, cfg.vocab, (rows,), dtype=torch.int32, device=DEV, generator=g)
    return _normal(seed, what, (rows, cfg.hidden), 1.0)


def _tables(cfg, n):
    """cos and sin of pos * base^(-2 i / d), float64 [n][d / 2]."""
    i = torch.arange(cfg.head_dim // 2, dtype=torch.float64, device=DEV)
    a = torch.arange(n, dtype=torch.float64, device=DEV)[:, None] * cfg.rope_base ** (-2.0 * i / cfg.head_dim)
    return a.cos(), a.sin()


def _attn_inputs(case, seed):
    cfg, lens = MODELS[case["model"]], lengths(case)
    rows = sum(lens) if case["kind"] == "attn_prefill" else len(lens)
    return _normal(seed, "qkv", (rows, (cfg.n_heads + 2 * cfg.n_kv_heads) * cfg.head_dim), 1.25)


def prepare(case, seed):
    cfg, lens, kind = MODELS[case["model"]], lengths(case), case["kind"]
    d, n = cfg.head_dim, len(lens)
    if kind == "attn_prefill":
        cu = [0]
        for k in lens:
            cu.append(cu[-1] + k)
        return dict(case=case, cfg=cfg, qkv=_attn_inputs(case, seed), cu=cu,
                    out=torch.zeros((cu[-1], cfg.n_heads * d), dtype=torch.bfloat16, device=DEV))
    if kind == "attn_decode":
        # the blocks of the sequences lie in the pool as a block manager's free list leaves them: mixed
        pool = cache(cfg, seed, 0, 1, lens)[0]
        order = list(range(pool.shape[0]))
        random.Random("order %d" % seed).shuffle(order)
        table = torch.zeros((n, max(map(_blocks, lens))), dtype=torch.int32)
        at = 0
        for i, k in enumerate(lens):
            table[i, :_blocks(k)] = torch.tensor(order[at:at + _blocks(k)], dtype=torch.int32)
            at += _blocks(k)
        mixed = torch.empty_like(pool)
        mixed[torch.tensor(order, device=DEV)] = pool
        cos, sin = (t.float() for t in _tables(cfg, max(lens)))
        return dict(case=case, cfg=cfg, qkv=_attn_inputs(case, seed), pool=mixed, table=table.to(DEV), cos=cos, sin=sin,
                    ctx=torch.tensor(lens, dtype=torch.int32, device=DEV), max_ctx=max(lens),
                    out=torch.zeros((n, cfg.n_heads * d), dtype=torch.bfloat16, device=DEV))

    begin, end, steps = case["begin"], case["end"], case["steps"]
    last = end == cfg.n_layers
    prefills = kind in ("prefill", "generate", "cold")
    img = image(cfg, seed, begin, end)

    def stage():
        st = pipeline.Stage(cfg, begin, end, max_seqs=n, max_ctx=max(lens) + steps, max_batch_tokens=sum(lens) if prefills else n)
        st.load(img)
        st.sync()
        return st

    s = dict(case=case, cfg=cfg, ids=list(range(n)), lens=lens, stage=stage(), rows=sum(lens))
    if kind == "move":
        s["other"] = stage()
        given, head = blob(cfg, seed, begin, end, lens)
        hs.hs_kv_import_many(s["stage"].h, [(given.data_ptr(), given.numel(), head)])
        s["sent"], s["back"] = torch.zeros_like(given), torch.zeros_like(given)
        s["stage"].sync()
    elif kind == "decode":
        s["blob"], s["head"] = blob(cfg, seed, begin, end, lens)
    if prefills:
        s["in"] = _stage_inputs(case, seed, sum(lens), "prompt")
        s["out"] = torch.zeros(n, dtype=torch.int32, device=DEV) if last else torch.zeros((sum(lens), cfg.hidden), dtype=torch.bfloat16, device=DEV)
    if steps:
        s["step_in"] = [_stage_inputs(case, seed, n, "step %d" % k) for k in range(steps)]
        s["step_out"] = torch.zeros((steps, n), dtype=torch.int32, device=DEV) if last else torch.zeros((steps, n, cfg.hidden), dtype=torch.bfloat16, device=DEV)
    if last:
        s["logits"] = torch.zeros((int(prefills) + steps, n, cfg.vocab), dtype=torch.float32, device=DEV)
    if kind == "cold":
        s["image"] = img
    else:
        img.close()
    return s


# -------------------------------------------------------------------- run


def run(s):
    case, cfg, kind = s["case"], s["cfg"], s["case"]["kind"]
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "attn_prefill":
        hs.hs_k_attn_prefill(s["qkv"].data_ptr(), s["out"].data_ptr(), s["cu"], cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, stream)
        return s["out"]
    if kind == "attn_decode":
        qkv, out = s["qkv"], s["out"]
        hs.hs_k_attn_decode_rope(qkv.data_ptr(), qkv.shape[1], s["pool"].data_ptr(), s["table"].data_ptr(), s["ctx"].data_ptr(),
                                 s["cos"].data_ptr(), s["sin"].data_ptr(), s["max_ctx"], out.data_ptr(), out.shape[1], len(out),
                                 cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, s["table"].shape[1], s["max_ctx"], stream)
        return dict(out=out, pool=s["pool"])

    st, ids = s["stage"], s["ids"]
    if kind == "move":
        size = hs.hs_kv_export(st.h, ids, s["sent"].data_ptr(), s["sent"].numel(), stream)
        head = hs.hs_kv_export_head(st.h, ids)
        hs.hs_kv_import_many(s["other"].h, [(s["sent"].data_ptr(), size, head)], stream)
        hs.hs_kv_export(s["other"].h, ids, s["back"].data_ptr(), s["back"].numel(), stream)
        for i in ids:
            hs.hs_seq_free(s["other"].h, i)
        return dict(sent=s["sent"], back=s["back"])

    last, result = "logits" in s, {}
    at = 0
    if kind == "decode":
        hs.hs_kv_import_many(st.h, [(s["blob"].data_ptr(), s["blob"].numel(), s["head"])], stream)
    else:
        if kind == "cold":
            hs.hs_stage_invalidate_weights(st.h)
            st.load(s["image"])
        st.prefill(ids, s["lens"], s["in"].data_ptr(), s["out"].data_ptr(), s["logits"][0].data_ptr() if last else 0, stream)
        at = 1
        if not last:
            result["prefill"] = s["out"]
    for k in range(case["steps"]):
        st.decode(ids, s["step_in"][k].data_ptr(), s["step_out"][k].data_ptr(), s["logits"][at + k].data_ptr() if last else 0, stream)
    for i in ids:
        hs.hs_seq_free(st.h, i)
    if last:
        result["logits"] = s["logits"]
    elif case["steps"]:
        result["decode"] = s["step_out"]
    return result


# ------------------------------------------------------------ work, tolerance


def work(case):
    """Weights are read once a call (a decode step is a call), each cached key and value once a step."""
    cfg, lens, kind = MODELS[case["model"]], lengths(case), case["kind"]
    d, h, n, total = cfg.head_dim, cfg.hidden, len(lens), sum(lens)
    kv_tok = 2 * cfg.n_kv_heads * d * 2  # bytes of a token's key and value in one layer
    attn = lambda pairs: 4.0 * cfg.n_heads * d * pairs  # noqa: E731
    causal = sum(k * (k + 1) / 2 for k in lens)
    if kind == "attn_prefill":
        return dict(bytes=total * (2 * cfg.n_heads + 2 * cfg.n_kv_heads) * d * 2, flops=attn(causal))
    if kind == "attn_decode":
        return dict(bytes=total * kv_tok + n * (2 * cfg.n_heads + 4 * cfg.n_kv_heads) * d * 2, flops=attn(total))
    layers = case["end"] - case["begin"]
    if kind == "move":
        return dict(bytes=6 * total * kv_tok * layers, flops=0)
    per_layer = (cfg.n_heads + 2 * cfg.n_kv_heads) * d * h + cfg.n_heads * d * h + 3 * h * cfg.ffn
    head = cfg.vocab * h if case["end"] == cfg.n_layers else 0
    out_row = cfg.vocab * 4 if head else h * 2
    nbytes = flops = 0.0
    if kind != "decode":
        rows = n if head else total
        nbytes += 2 * (layers * per_layer + head) + total * h * 2 + rows * out_row + layers * total * kv_tok
        flops += 2.0 * (layers * per_layer * total + head * n) + layers * attn(causal)
    if kind == "cold":
        nbytes += 2 * layers * per_layer  # the upload writes what the layers read
    if kind == "decode":
        nbytes += 2 * total * kv_tok * layers  # the caches taken over
    for k in range(case["steps"]):
        nbytes += 2 * (layers * per_layer + head) + n * (h * 2 + out_row) + layers * (total + (k + 1) * n) * kv_tok
        flops += 2.0 * n * (layers * per_layer + head) + layers * attn(total + (k + 1) * n)
    return dict(bytes=nbytes, flops=flops)


def kind_is_attention(case):
    return case["kind"] in ("attn_prefill", "attn_decode")


def tolerance(case):
    if case["kind"] == "move":
        return "exact"  # bytes
    # bf16 storage, float32 sums. Measured on MI355X against exact(): one layer's attention 0.0019 to 0.003 of
    # the norm, a layer or two of a stage 0.0038 to 0.0072 (each rounding to bf16 is half of 2^-8).
    return dict(rel=0.01 if kind_is_attention(case) else 0.02)


# ------------------------------------------------------------------ 64 bits


def _norm64(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, cos, sin):
    """Rotate-half RoPE of [rows][heads][d] with each row's own angles [rows][d / 2]."""
    a, b = x.chunk(2, -1)
    c, s = cos[:, None], sin[:, None]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend64(q, k, v, first):
    """Causal attention of queries [m][heads][d] at positions first, first + 1, ... over [n][kv heads][d]."""
    m, n, group = q.shape[0], k.shape[0], q.shape[1] // k.shape[1]
    out = torch.empty_like(q)
    ahead = torch.arange(n, device=q.device)[None, :] > torch.arange(first, first + m, device=q.device)[:, None]
    for h in range(q.shape[1]):
        p = (q[:, h] @ k[:, h // group].T) / math.sqrt(q.shape[2])
        out[:, h] = torch.softmax(p.masked_fill_(ahead, -math.inf), -1) @ v[:, h // group]
    return out


def _layer64(cfg, w, x, seqs, cos, sin):
    """One decoder layer on rows x; seqs: (first row, end row, cached keys, cached values) of each sequence.
    Returns the rows and each sequence's keys and values with the new rows joined."""
    d, nh, nkv = cfg.head_dim, cfg.n_heads, cfg.n_kv_heads
    u = _norm64(x, w("attn_norm"), cfg.rms_eps)
    q, k, v = ((u @ w(name).double().T).view(len(x), -1, d) for name in ("wq", "wk", "wv"))
    mixed, joined = torch.empty((len(x), nh * d), dtype=torch.float64, device=x.device), []
    for b, e, ck, cv in seqs:
        at = slice(len(ck), len(ck) + e - b)
        kk = torch.cat([ck, _rope64(k[b:e], cos[at], sin[at])])
        vv = torch.cat([cv, v[b:e]])
        mixed[b:e] = _attend64(_rope64(q[b:e], cos[at], sin[at]), kk, vv, len(ck)).reshape(e - b, -1)
        joined.append((kk, vv))
    x = x + mixed @ w("wo").double().T
    u = _norm64(x, w("ffn_norm"), cfg.rms_eps)
    act = torch.nn.functional.silu(u @ w("wgate").double().T) * (u @ w("wup").double().T)
    return x + act @ w("wdown").double().T, joined


def exact(case, seed):
    cfg, lens, kind = MODELS[case["model"]], lengths(case), case["kind"]
    d, nh, nkv = cfg.head_dim, cfg.n_heads, cfg.n_kv_heads
    if kind == "move":
        return None
    if kind == "attn_prefill":
        q, k, v = (t.double().view(-1, t.shape[1] // d, d) for t in _attn_inputs(case, seed).split([nh * d, nkv * d, nkv * d], 1))
        at, outs = 0, []
        for n in lens:
            outs.append(_attend64(q[at:at + n], k[at:at + n], v[at:at + n], 0))
            at += n
        return torch.cat(outs).reshape(sum(lens), -1)

    def kept(x, layer, i):
        """Keys and values of sequence i in a cache laid out by blocks, each [tokens][kv heads][d] in 64 bits."""
        b = sum(map(_blocks, lens[:i]))
        part = x[layer, b:b + _blocks(lens[i])].double().permute(1, 0, 3, 2, 4).reshape(2, -1, nkv, d)
        return part[0, :lens[i]], part[1, :lens[i]]

    cos, sin = _tables(cfg, max(lens) + case["steps"])
    if kind == "attn_decode":
        q, k, v = (t.double().view(-1, t.shape[1] // d, d) for t in _attn_inputs(case, seed).split([nh * d, nkv * d, nkv * d], 1))
        x = cache(cfg, seed, 0, 1, lens)
        outs = []
        for i, n in enumerate(lens):
            at = slice(n - 1, n)
            ck, cv = kept(x, 0, i)
            kk = torch.cat([ck[:-1], _rope64(k[i:i + 1], cos[at], sin[at])])
            vv = torch.cat([cv[:-1], v[i:i + 1]])
            outs.append(_attend64(_rope64(q[i:i + 1], cos[at], sin[at]), kk, vv, n - 1))
        return dict(out=torch.cat(outs).reshape(len(lens), -1), pool=None)

    begin, end, last = case["begin"], case["end"], case["end"] == cfg.n_layers
    n, steps = len(lens), case["steps"]
    empty = torch.empty((0, nkv, d), dtype=torch.float64, device=DEV)
    if kind == "decode":
        given = cache(cfg, seed, begin, end, lens)
        kv = [[kept(given, l, i) for i in range(n)] for l in range(end - begin)]
    else:
        kv = [[(empty, empty)] * n for _ in range(end - begin)]
    result, logits = {}, []

    def rows_in(x):
        return weight(cfg, seed, -1, "embed")[x.long()].double() if begin == 0 else x.double()

    def forward(x, ends):
        for l in range(begin, end):
            seqs = [(b, e, *kv[l - begin][i]) for i, (b, e) in enumerate(ends)]
            x, kv[l - begin] = _layer64(cfg, lambda k: weight(cfg, seed, l, k), x, seqs, cos, sin)  # noqa: B023
        if last:
            x = x[[e - 1 for _, e in ends]]
            logits.append(_norm64(x, weight(cfg, seed, -1, "final_norm"), cfg.rms_eps) @ weight(cfg, seed, -1, "lm_head").double().T)
        return x

    if kind != "decode":
        ends, at = [], 0
        for k in lens:
            ends.append((at, at + k))
            at += k
        x = forward(rows_in(_stage_inputs(case, seed, at, "prompt")), ends)
        if not last:
            result["prefill"] = x
    outs = [forward(rows_in(_stage_inputs(case, seed, n, "step %d" % k)), [(i, i + 1) for i in range(n)]) for k in range(steps)]
    if last:
        result["logits"] = torch.stack(logits)
    elif steps:
        result["decode"] = torch.stack(outs)
    return result
