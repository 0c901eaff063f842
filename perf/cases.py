"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  Its "kind" names the public entry points that it goes through:

  layers   ss_decoder_layers_forward: the decoder layers over the new rows of every sequence, against the cache
  verify   ss_verify_forward: embedding, layers, final norm and LM head
  draft    ss_draft_step with sampling: the same, then softmax and one token per sequence
  step     ss_speculative_step, greedy: K draft calls, the verify pass, the acceptance and the roll-back
  accept   ss_speculative_accept_logits: the rejection step from the logits of both models
  sample   ss_softmax, ss_top_k_filter, ss_top_p_filter, ss_speculative_accept: the rejection step with selection rules
  greedy   ss_greedy_accept

Every call that appends to a cache is followed by the truncation that a rejected draft brings
(ss_kv_cache_truncate, on the device), so a pass leaves the lengths as it found them.
"""
import hashlib
import math
from types import SimpleNamespace

import torch

import paper_2311_04951_amd as sv

# decoder shapes: d_model, heads, head_dim, d_ff, vocabulary
SHAPES = {
    "small": (256, 4, 64, 688, 1024),      # the fp32 pair of the smoke test and its draft
    "tiny": (128, 2, 64, 344, 1024),
    "1b": (2048, 32, 64, 5632, 32000),     # heads of 64
    "3b": (3072, 24, 128, 8192, 32000),    # a draft of the size that goes with the 13B-shaped target
    "7b": (4096, 32, 128, 11008, 32000),
    "13b": (5120, 40, 128, 13824, 32000),
}
QUANT_BITS = {"none": 16, "int8": 8, "int4": 4}


def _c(name, kind, **values):
    return dict({"name": name, "kind": kind}, **values)


def _layers(name, shape, layers, quant, batch, rows, context):
    return _c(name, "layers", shape=shape, layers=layers, quant=quant, batch=batch, rows=rows, context=context)


def listed():
    return [
        # the smallest call: one token of a small fp32 draft, all launches and latency
        _c("draft small f32", "draft", shape="small", layers=2, batch=1, context=40),
        # one row of a 3B-shaped draft (two of its layers and the LM head): a step of plain decoding, or a draft's call
        _c("verify 3B-shape 1 row", "verify", shape="3b", layers=2, batch=1, rows=1, context=300),
        # a layer of the usual verify pass, K = 4, at a long prompt
        _layers("layer 7B-shape 5 rows", "7b", 1, "none", 1, 5, 1024),
        # K = 5 on the wider target of the size ratio 13B : 3B, an odd context
        _layers("layer 13B-shape 6 rows", "13b", 1, "none", 1, 6, 2001),
        # weight-only quantised targets; several layers, so that the matrices don't stay in the caches
        _layers("4 layers int8 5 rows", "7b", 4, "int8", 1, 5, 200),
        _layers("8 layers int4 5 rows", "7b", 8, "int4", 1, 5, 200),
        # a batch of sequences of different lengths (up to 4096 positions) verifies K = 8 draft tokens each
        _layers("layer 7B-shape 8x9 rows", "7b", 1, "none", 8, 9, 4080),
        # prefill of a batch: chunks of 16 tokens of 16 prompts
        _layers("prefill 7B-shape 16x16 rows", "7b", 1, "none", 16, 16, 500),
        # a whole greedy step of the 7B-shaped target with its first two layers as the draft
        _c("step 7B-shape greedy K 4", "step", shape="7b", layers=32, draft_layers=2, K=4, context=260),
        # the rejection step of a large batch over a large vocabulary
        _c("accept 64 x K 8 x 128256", "accept", batch=64, K=8, vocab=128256),
        # the rejection step of one sequence with top-k and top-p
        _c("sample 1 x K 4 x 32000", "sample", batch=1, K=4, vocab=32000, top_k=200, top_p=0.9),
        # greedy acceptance of a batch
        _c("greedy 8 x K 8 x 128256", "greedy", batch=8, K=8, vocab=128256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layers"] * 6 + ["verify", "draft", "step", "accept", "sample", "greedy"])
    if kind == "layers":
        quant = rng.choice(["none", "none", "int8", "int4"])
        shape = rng.choice(["1b", "3b", "7b", "13b"])
        batch = rng.choice([1, 1, 1, _log(rng, 2, 16)])
        rows = _log(rng, 1, 16)
        return dict(kind=kind, shape=shape, layers={"none": 1, "int8": 2, "int4": 3}[quant], quant=quant, batch=batch, rows=rows,
                    context=_log(rng, 16, 4080 if batch <= 8 else 2000))
    if kind == "verify":
        return dict(kind=kind, shape=rng.choice(["small", "1b", "3b", "7b"]), layers=rng.randint(1, 3), batch=rng.choice([1, 1, 3]),
                    rows=_log(rng, 1, 16), context=_log(rng, 16, 2000))
    if kind == "draft":
        return dict(kind=kind, shape=rng.choice(["small", "tiny"]), layers=rng.randint(1, 4), batch=_log(rng, 1, 8), context=_log(rng, 4, 500))
    if kind == "step":
        return dict(kind=kind, shape=rng.choice(["1b", "3b", "7b"]), layers=rng.randint(4, 16), draft_layers=rng.randint(1, 3), K=rng.randint(1, 8),
                    context=_log(rng, 16, 2000))
    vocab = rng.choice([32000, 32000, 50257, 128256, _log(rng, 1000, 130000)])
    K = rng.randint(1, 10)
    batch = _log(rng, 1, 32)
    if kind == "sample":
        return dict(kind=kind, batch=batch, K=K, vocab=vocab, top_k=rng.choice([0, 40, _log(rng, 2, 2000)]), top_p=rng.choice([1.0, 0.95, 0.8, 0.3]))
    return dict(kind=kind, batch=batch, K=K, vocab=vocab)


# ------------------------------------------------------------------------------------------------ inputs

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, name):
    g = torch.Generator(device=_dev())
    g.manual_seed(int.from_bytes(hashlib.sha256(f"{seed}:{name}".encode()).digest()[:7], "little"))
    return g


def _normal(seed, name, shape, std, mean=0.0, dtype=torch.float32):
    x = torch.randn(shape, generator=_gen(seed, name), device=_dev(), dtype=torch.float32)
    return x.mul_(std).add_(mean).to(dtype)


def _uniforms(seed, name, shape):
    """Multiples of 2^-24 in [0, 1)."""
    return torch.randint(0, 1 << 24, shape, generator=_gen(seed, name), device=_dev(), dtype=torch.int32).to(torch.float32) / (1 << 24)


def _tokens(seed, name, shape, vocab):
    return torch.randint(0, vocab, shape, generator=_gen(seed, name), device=_dev(), dtype=torch.int32)


def _shape(case):
    d, heads, hd, ff, vocab = SHAPES[case["shape"]]
    f32 = case["shape"] in ("small", "tiny")
    return SimpleNamespace(n_layers=case["layers"], d_model=d, n_heads=heads, head_dim=hd, d_ff=ff, vocab=vocab, rope_base=10000.0, rms_eps=1e-5,
                           dtype="f32" if f32 else "bf16")


def _storage(s):
    return torch.float32 if s.dtype == "f32" else torch.bfloat16


def _layer(case, seed, l):
    """Layer l in the packed form the library streams.  In a "step" the layers behind the draft's write a tenth as much into the
    residual stream, so that the draft predicts its target the way a trained one does and some tokens are accepted."""
    s = _shape(case)
    W, dt = s.n_heads * s.head_dim, _storage(s)
    late = 0.1 if case["kind"] == "step" and l >= case["draft_layers"] else 1.0
    return {"wqkv": _normal(seed, f"wqkv{l}", (3 * W, s.d_model), 0.02, dtype=dt), "wo": _normal(seed, f"wo{l}", (s.d_model, W), 0.02 * late, dtype=dt),
            "wgu": _normal(seed, f"wgu{l}", (2 * s.d_ff, s.d_model), 0.02, dtype=dt),
            "wd": _normal(seed, f"wd{l}", (s.d_model, s.d_ff), 0.02 * late, dtype=dt),
            "g1": _normal(seed, f"g1{l}", (s.d_model,), 0.02, 1.0), "g2": _normal(seed, f"g2{l}", (s.d_model,), 0.02, 1.0)}


def _ends(case, seed):
    """Embedding, final gain and LM head."""
    s = _shape(case)
    dt = _storage(s)
    return {"embed": _normal(seed, "embed", (s.vocab, s.d_model), 0.02, dtype=dt), "gf": _normal(seed, "gf", (s.d_model,), 0.02, 1.0),
            "lm_head": _normal(seed, "lm_head", (s.vocab, s.d_model), 0.02, dtype=dt)}


def _lengths(case):
    """Cached positions of every sequence: the first has all of the context, the others up to a quarter fewer."""
    b, n = case.get("batch", 1), case["context"]
    return [n - (n * i) // (4 * b) for i in range(b)]


def _context(case, seed, l, b, n):
    """Keys (already rotated) and values of layer l of sequence b."""
    s = _shape(case)
    W = s.n_heads * s.head_dim
    return _normal(seed, f"k{l}.{b}", (n, W), 1.0, dtype=_storage(s)), _normal(seed, f"v{l}.{b}", (n, W), 1.0, dtype=_storage(s))


def _model(case, seed, layers, ends=None, n_layers=None):
    s = _shape(case)
    s.n_layers = n_layers or s.n_layers
    quant = case.get("quant", "none")
    return sv.Model(s, ends, max_rows=max(16, case.get("batch", 1) * case.get("rows", 1)), max_pos=case["context"] + 64, packed_layers=layers,
                    int8_weights=quant == "int8", int4_weights=quant == "int4")


class _Cache:
    """A cache with its context, the call that sets the lengths back, and views of what a pass of `rows` rows appends."""

    def __init__(self, case, seed, model, n_layers, rows):
        s = _shape(case)
        self.lens = _lengths(case)
        B, H, hd, dt = len(self.lens), s.n_heads, s.head_dim, _storage(s)
        self.kv = sv.KVCache(model, B, case["context"] + 40)
        for l in range(n_layers):
            for b, n in enumerate(self.lens):
                sv.ss_kv_cache_append(self.kv, l, b, 0, *_context(case, seed, l, b, n))
        sv.ss_kv_cache_set_len(self.kv, self.lens)
        self.lens_dev = torch.tensor(self.lens, dtype=torch.int32, device=_dev())
        # the layout is the one that the C header gives
        S = (case["context"] + 40 + 63) // 64 * 64
        half = n_layers * B * H * S * hd * dt.itemsize
        keys = self.kv.buf[:half].view(dt).view(n_layers, B, H, S, hd)
        values = self.kv.buf[half:2 * half].view(dt).view(n_layers, B, H, S // 64, hd, 64)
        self.appended = {"k": [keys[:, b, :, n:n + rows] for b, n in enumerate(self.lens)],
                         "v": [values[:, b, :, n // 64:(n + rows - 1) // 64 + 1] for b, n in enumerate(self.lens)]}

    def back(self):
        sv.ss_kv_cache_truncate(self.kv, self.lens_dev, self.lens)


def _sampling_inputs(case, seed):
    """Draft logits N(0, 2), target logits the same plus N(0, 0.5) and a bonus row N(0, 2); the draft's tokens are drawn from its rows."""
    B, K, V = case["batch"], case["K"], case["vocab"]
    ql = _normal(seed, "q", (B, K, V), 2.0)
    pl = torch.empty((B, K + 1, V), dtype=torch.float32, device=_dev())
    pl[:, :K] = ql + _normal(seed, "noise", (B, K, V), 0.5)
    pl[:, K] = _normal(seed, "bonus", (B, V), 2.0)
    return pl, ql, _uniforms(seed, "u", (B, K + 1))


def _draw_tokens(q, seed):
    """One token of every row of q by the inverse of its cumulative sums."""
    B, K, V = q.shape
    c = q.reshape(B * K, V).double().cumsum(1)
    u = _uniforms(seed, "ud", (B * K, 1)).double() * c[:, -1:]
    return torch.searchsorted(c, u, right=True).clamp_(max=V - 1).to(torch.int32).view(B, K)


def prepare(case, seed):
    kind = case["kind"]
    st = SimpleNamespace(case=case)
    if kind in ("layers", "verify", "draft", "step"):
        s = _shape(case)
        packed = [_layer(case, seed, l) for l in range(s.n_layers)]
        ends = None if kind == "layers" else _ends(case, seed)
        st.model = _model(case, seed, packed, ends)
        rows = case["K"] + 1 if kind == "step" else case.get("rows", 1)
        st.cache = _Cache(case, seed, st.model, s.n_layers, rows)
        B = case.get("batch", 1)
        if kind == "layers":
            st.h0 = _normal(seed, "h", (B * rows, s.d_model), 1.0)
            st.h = torch.empty_like(st.h0)
        elif kind == "verify":
            st.tokens = _tokens(seed, "tokens", (B, rows), s.vocab)
            st.logits = torch.empty((B, rows, s.vocab), dtype=torch.float32, device=_dev())
        elif kind == "draft":
            st.tokens = _tokens(seed, "tokens", (B, 1), s.vocab)
            st.u = _uniforms(seed, "u", (B,))
            st.q = torch.empty((B, s.vocab), dtype=torch.float32, device=_dev())
            st.out = torch.empty((B,), dtype=torch.int32, device=_dev())
        else:
            nd = case["draft_layers"]
            st.draft = _model(case, seed, packed[:nd], ends, n_layers=nd)
            st.draft_cache = _Cache(case, seed, st.draft, nd, rows)
            st.first = _tokens(seed, "tokens", (2,), s.vocab)
            st.buf = sv.StepBuffers(case["K"], s.vocab, int(st.first[0]), _dev())
        return st
    pl, ql, st.u = _sampling_inputs(case, seed)
    B, K, V = case["batch"], case["K"], case["vocab"]
    st.na = torch.empty(B, dtype=torch.int32, device=_dev())
    st.nx = torch.empty(B, dtype=torch.int32, device=_dev())
    st.pl = pl
    if kind == "accept":
        st.ql, st.d = ql, _draw_tokens(ql.softmax(-1), seed)
    elif kind == "sample":
        q = ql.softmax(-1)
        if 0 < case["top_k"] < V:
            q = torch.where(q >= q.topk(case["top_k"], -1).values[..., -1:], q, 0.0)
            q = q / q.sum(-1, keepdim=True)
        st.q, st.d, st.p = q.contiguous(), _draw_tokens(q, seed), torch.empty_like(pl)
    else:   # three of four draft tokens are the target's own choice
        st.d = torch.where(_uniforms(seed, "hit", (B, K)) < 0.75, pl[:, :K].argmax(-1).to(torch.int32), _tokens(seed, "miss", (B, K), V)).contiguous()
    return st


# ------------------------------------------------------------------------------------------------ a pass

def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "layers":
        st.h.copy_(st.h0)
        sv.ss_decoder_layers_forward(st.model, st.cache.kv, st.h, case["batch"], case["rows"])
        st.cache.back()
        return {"h": st.h, "appended": st.cache.appended}
    if kind == "verify":
        sv.ss_verify_forward(st.model, st.cache.kv, st.tokens, case["rows"], st.logits)
        st.cache.back()
        return {"logits": st.logits, "appended": st.cache.appended}
    if kind == "draft":
        sv.ss_draft_step(st.model, st.cache.kv, st.tokens, 1, 1.0, st.u, st.q, st.q.shape[1], st.out)
        st.cache.back()
        return {"q": st.q, "token": st.out, "appended": st.cache.appended}
    if kind == "step":
        st.buf.feed.copy_(st.first)
        st.buf.n_feed.value = 1
        a, y, d = sv.ss_speculative_step(st.model, st.cache.kv, st.draft, st.draft_cache.kv, st.buf, 0.0)
        st.cache.back()
        st.draft_cache.back()
        return {"logits": st.buf.logits, "accepted": a, "next": y, "draft": d, "appended": st.cache.appended}
    if kind == "accept":
        sv.ss_speculative_accept_logits(st.pl, st.ql, 1.0, st.d, st.u, n_accepted=st.na, next_token=st.nx)
        return {"n_accepted": st.na, "next": st.nx}
    if kind == "sample":
        p = sv.ss_softmax(st.pl, 1.0, st.p)
        if case["top_k"]:
            sv.ss_top_k_filter(p, case["top_k"], p)
        if case["top_p"] < 1.0:
            sv.ss_top_p_filter(p, case["top_p"], p)
        sv.ss_speculative_accept(p, st.q, st.d, st.u, n_accepted=st.na, next_token=st.nx)
        return {"p": p, "n_accepted": st.na, "next": st.nx}
    sv.ss_greedy_accept(st.pl, st.d, n_accepted=st.na, next_token=st.nx)
    return {"n_accepted": st.na, "next": st.nx}


# ------------------------------------------------------------------------------------------------ work and tolerance

def work(case):
    kind = case["kind"]
    if kind in ("layers", "verify", "draft", "step"):
        s = _shape(case)
        d, W, F, V = s.d_model, s.n_heads * s.head_dim, s.d_ff, s.vocab
        e = 4 if s.dtype == "f32" else 2
        bits = QUANT_BITS[case.get("quant", "none")] if e == 2 else 32
        params = 4 * W * d + 3 * d * F
        lens = _lengths(case)

        def forward(n_layers, M, lens, head_rows):
            """One forward pass: every matrix, the cached and the new keys and values, the hidden rows (or embeddings) and the logits."""
            R = len(lens) * M
            scales = {16: 0, 32: 0, 8: 4 * (3 * W + 2 * d + 2 * F), 4: 4 * params // 128}[bits]
            by = n_layers * (params * bits // 8 + scales + 8 * d + 2 * W * e * sum(n + 2 * M for n in lens)) + R * d * 4
            fl = n_layers * (2 * params * R + 4 * W * M * sum(n + (M + 1) / 2 for n in lens))
            if head_rows:
                by += V * d * e + 4 * head_rows * V
                fl += 2 * V * d * head_rows
            return by, fl

        if kind == "layers":
            by, fl = forward(s.n_layers, case["rows"], lens, 0)
            by += 4 * len(lens) * case["rows"] * d      # the hidden rows come and go
        elif kind == "verify":
            by, fl = forward(s.n_layers, case["rows"], lens, len(lens) * case["rows"])
        elif kind == "draft":
            by, fl = forward(s.n_layers, 1, lens, len(lens))
        else:
            by, fl = forward(s.n_layers, case["K"] + 1, lens, case["K"] + 1)
            for i in range(case["K"]):
                b1, f1 = forward(case["draft_layers"], 1, [lens[0] + i], 1)
                by, fl = by + b1, fl + f1
        return {"bytes": by, "flops": fl}
    B, K, V = case["batch"], case["K"], case["vocab"]
    if kind == "accept":        # the logits of both models
        return {"bytes": 4 * B * (2 * K + 1) * V, "flops": 4 * B * (2 * K + 1) * V}
    if kind == "sample":        # the target's logits read, its probabilities written, one row of the draft's read
        return {"bytes": 4 * B * (2 * (K + 1) + 1) * V, "flops": 6 * B * (K + 1) * V}
    return {"bytes": 4 * B * (K + 1) * V, "flops": B * (K + 1) * V}


def tolerance(case):
    """About four times the largest error over all outputs, measured against the same computation in 64 bits that rounds only what the cache
    holds.  A bf16 model keeps its sums and hidden rows in 32 bits (4e-6 to 8e-6 in the hidden rows of one layer, 1.4e-5 in the logits behind
    two); the largest error is that of the appended keys and values, where a value near the middle between two bf16 numbers falls to either
    side: 1.4e-4 within three layers, 4e-4 behind 8 int4 layers, 6e-4 behind 32 layers."""
    if case["kind"] == "greedy":
        return "exact"
    if case["kind"] == "accept":        # whole numbers: one differs where a uniform meets a boundary within the last bits
        return {"rel": 0.0, "differ": 0.01}
    if case["kind"] == "sample":        # sums of up to 130000 32-bit numbers
        return {"rel": 1e-5}
    if case["shape"] in ("small", "tiny"):
        return {"rel": 1.5e-6}
    return {"rel": 2.5e-3 if case["kind"] == "step" else 6e-4 if case.get("quant", "none") == "none" else 1.6e-3}


# ------------------------------------------------------------------------------------------------ the same in 64 bits

def _dequantised(w, quant):
    """The matrix that the quantised model stands for, by the rule of the C header, in 64 bits."""
    if quant == "none":
        return w.double()
    top = 127.0 if quant == "int8" else 7.0
    g = w.double().view((w.shape[0], -1, 128) if quant == "int4" else (w.shape[0], 1, -1))
    amax = g.abs().amax(-1, keepdim=True)
    # the rule divides in 32 bits: a 64-bit quotient of 32-bit numbers, rounded to 32 bits, is that quotient
    scale = torch.where(amax > 0, (amax / top).float().double(), 1.0)
    return (torch.round((g / scale).float()).clamp_(-top, top).double() * scale).view(w.shape)


def _norm64(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain.double()


def _layer64(case, s, w, h, ctx, lens, M):
    """h [B, M, d] through one layer; ctx[b] = (keys, values) [n, W] in 64 bits.  Returns h and the new keys and values [B][M, W]
    (64 bits throughout: what the cache's type rounds off is part of the library's error)."""
    quant, H, hd, W = case.get("quant", "none"), s.n_heads, s.head_dim, s.n_heads * s.head_dim
    B = h.shape[0]
    qkv = _norm64(h, w["g1"], s.rms_eps) @ _dequantised(w["wqkv"], quant).t()
    q, k, v = (t.reshape(B, M, H, hd) for t in qkv.split(W, -1))
    j = torch.arange(hd // 2, device=h.device, dtype=torch.float64)
    inv = s.rope_base ** (-2.0 * j / hd)
    out = torch.empty((B, M, W), dtype=torch.float64, device=h.device)
    new = []
    for b in range(B):
        ang = (lens[b] + torch.arange(M, device=h.device, dtype=torch.float64))[:, None, None] * inv

        def turn(x):
            lo, hi = x[..., :hd // 2], x[..., hd // 2:]
            return torch.cat([lo * ang.cos() - hi * ang.sin(), lo * ang.sin() + hi * ang.cos()], -1)

        qb = turn(q[b])
        kb, vb = turn(k[b]), v[b]
        new.append((kb.reshape(M, W), vb.reshape(M, W)))
        K = torch.cat([ctx[b][0].reshape(-1, H, hd), kb], 0).permute(1, 2, 0).contiguous()     # [H, hd, n]
        V = torch.cat([ctx[b][1].reshape(-1, H, hd), vb], 0).permute(1, 0, 2).contiguous()     # [H, n, hd]
        score = torch.bmm(qb.permute(1, 0, 2).contiguous(), K) / math.sqrt(hd)
        n = K.shape[-1]
        seen = torch.arange(n, device=h.device)[None, :] <= (n - M + torch.arange(M, device=h.device))[:, None]
        score = score.masked_fill(~seen, -math.inf).softmax(-1)
        out[b] = torch.bmm(score, V).permute(1, 0, 2).reshape(M, W)
    h = h + out @ _dequantised(w["wo"], quant).t()
    gate, up = (_norm64(h, w["g2"], s.rms_eps) @ _dequantised(w["wgu"], quant).t()).split(s.d_ff, -1)
    return h + (gate * torch.sigmoid(gate) * up) @ _dequantised(w["wd"], quant).t(), new


def _forward64(case, s, weights, h, contexts, lens, M):
    """All layers; contexts[l][b] is replaced by the one with the new rows behind it.  Returns h and what every layer appended."""
    appended = []
    for l, w in enumerate(weights):
        h, new = _layer64(case, s, w() if callable(w) else w, h, contexts[l], lens, M)
        contexts[l] = [tuple(torch.cat([c, n], 0) for c, n in zip(cb, nb)) for cb, nb in zip(contexts[l], new)]
        appended.append(new)
    return h, appended


def _appended64(case, s, contexts, lens, M):
    """What `_Cache.appended` shows: the new keys, and the blocks of 64 positions that hold the new values."""
    H, hd = s.n_heads, s.head_dim
    ks, vs = [], []
    for b, n in enumerate(lens):
        ks.append(torch.stack([c[b][0][n:n + M].reshape(M, H, hd).permute(1, 0, 2) for c in contexts]))
        first, last = n // 64, (n + M - 1) // 64
        rows = []
        for c in contexts:
            v = c[b][1][first * 64:n + M]
            v = torch.cat([v, v.new_zeros((last + 1 - first) * 64 - v.shape[0], v.shape[1])], 0)
            rows.append(v.reshape(last + 1 - first, 64, H, hd).permute(2, 0, 3, 1))
        vs.append(torch.stack(rows))
    return {"k": ks, "v": vs}


def _contexts64(case, seed, n_layers):
    lens = _lengths(case)
    return [[tuple(t.double() for t in _context(case, seed, l, b, n)) for b, n in enumerate(lens)] for l in range(n_layers)]


def _head64(s, ends, h):
    return _norm64(h, ends["gf"], s.rms_eps) @ ends["lm_head"].double().t()


def _pick64(w, u):
    """The token of 64-bit integer weights [V] by the integer inverse of their running sums (None: they are all 0)."""
    c = w.cumsum(0)
    total = int(c[-1])
    if total == 0:
        return None
    threshold = (int(round(float(u) * (1 << 24))) * total) >> 24
    return int(torch.searchsorted(c, torch.tensor([threshold], device=w.device), right=True)[0])


def _weights64(p):
    return (p.clamp(min=0.0) * 4294967296.0).to(torch.int64)


def _accept64(p, q, d, u):
    """The rejection step on 64-bit probabilities [B, K + 1, V] and [B, K, V]."""
    B, K = d.shape
    at = d.long()[..., None]
    pd, qd = p[:, :K].gather(-1, at)[..., 0], q.gather(-1, at)[..., 0]
    ok = ((pd >= qd) | (u[:, :K].double() * qd < pd)).cpu()
    na, nx = [], []
    for b in range(B):
        a = next((i for i in range(K) if not ok[b, i]), K)
        tok = _pick64(_weights64(p[b, a] - q[b, a]), u[b, K]) if a < K else None
        if tok is None:
            tok = _pick64(_weights64(p[b, a]), u[b, K])
        na.append(a)
        nx.append(int(p[b, a].argmax()) if tok is None else tok)
    return torch.tensor(na, dtype=torch.int32), torch.tensor(nx, dtype=torch.int32)


def _kept64(p, keep_sorted):
    """Rows of p restricted to the tokens that keep_sorted(weights in descending order) names, and renormalised."""
    w = _weights64(p).clamp_(max=(1 << 32) - 1)
    order = w.argsort(dim=-1, descending=True, stable=True)
    kept = keep_sorted(w.gather(-1, order))
    mask = torch.zeros_like(kept).scatter_(-1, order, kept)
    z = torch.where(mask, w, 0).sum(-1, keepdim=True).double() / 4294967296.0
    return torch.where(mask, p / z, 0.0)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("layers", "verify", "draft", "step"):
        s = _shape(case)
        lens = _lengths(case)
        B = len(lens)
        M = case["K"] + 1 if kind == "step" else case.get("rows", 1)
        contexts = _contexts64(case, seed, s.n_layers)
        weights = [lambda l=l: _layer(case, seed, l) for l in range(s.n_layers)]
        if kind == "layers":
            h = _normal(seed, "h", (B * M, s.d_model), 1.0).double().view(B, M, -1)
            h, _ = _forward64(case, s, weights, h, contexts, lens, M)
            return {"h": h.reshape(B * M, -1), "appended": _appended64(case, s, contexts, lens, M)}
        ends = _ends(case, seed)
        if kind in ("verify", "draft"):
            tokens = _tokens(seed, "tokens", (B, M), s.vocab)
            h, _ = _forward64(case, s, weights, ends["embed"][tokens.long()].double(), contexts, lens, M)
            logits, appended = _head64(s, ends, h), _appended64(case, s, contexts, lens, M)
            if kind == "verify":
                return {"logits": logits, "appended": appended}
            q = logits[:, -1].softmax(-1)
            u = _uniforms(seed, "u", (B,))
            return {"q": q, "token": torch.tensor([_pick64(_weights64(q[b]), u[b]) for b in range(B)], dtype=torch.int32), "appended": appended}
        nd = case["draft_layers"]
        draft_weights, draft_contexts = [_layer(case, seed, l) for l in range(nd)], [list(c) for c in contexts[:nd]]
        tokens = [int(_tokens(seed, "tokens", (2,), s.vocab)[0])]
        for i in range(case["K"]):
            h = ends["embed"][tokens[-1:]].double()[None]
            h, _ = _forward64(case, s, draft_weights, h, draft_contexts, [lens[0] + i], 1)
            tokens.append(int(_head64(s, ends, h)[0, 0].argmax()))
        h, _ = _forward64(case, s, weights, ends["embed"][tokens].double()[None], contexts, lens, M)
        logits = _head64(s, ends, h)[0]
        best = logits.argmax(-1).tolist()
        a = next((i for i in range(case["K"]) if tokens[i + 1] != best[i]), case["K"])
        return {"logits": logits, "accepted": a, "next": best[a], "draft": tokens[1:], "appended": _appended64(case, s, contexts, lens, M)}
    st = prepare(case, seed)
    if kind == "greedy":
        best = st.pl.argmax(-1).cpu()
        d, K = st.d.cpu(), case["K"]
        na = [next((i for i in range(K) if int(d[b, i]) != int(best[b, i])), K) for b in range(d.shape[0])]
        return {"n_accepted": torch.tensor(na, dtype=torch.int32), "next": torch.stack([best[b, a] for b, a in enumerate(na)]).to(torch.int32)}
    p = st.pl.double().softmax(-1)
    if kind == "accept":
        na, nx = _accept64(p, st.ql.double().softmax(-1), st.d, st.u)
        return {"n_accepted": na, "next": nx}
    V, k = case["vocab"], case["top_k"]
    if 0 < k < V:
        p = _kept64(p, lambda w: (torch.arange(V, device=w.device) < k).expand_as(w))
    if case["top_p"] < 1.0:
        grid = round(case["top_p"] * (1 << 24))

        def nucleus(w):
            c = w.cumsum(-1)
            goal = (grid * c[..., -1:] + (1 << 24) - 1) >> 24
            return c - w < goal

        p = _kept64(p, nucleus)
    na, nx = _accept64(p, st.q.double(), st.d, st.u)
    return {"p": p, "n_accepted": na, "next": nx}
