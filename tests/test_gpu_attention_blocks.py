"""The attention of one split in blocks of 64 positions (bf16, heads of 64 and 128, calls of 256 and more (sequence, head) units at 256 and
more positions): lengths at the edges of blocks and of the round over the wavefronts, sequences of very different lengths."""
import ctypes
import math

import pytest
import torch

import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev


def _want(q, k, v, lens, M):
    """64-bit attention; q [B, M, H, hd], k / v per sequence [n + M, H, hd]."""
    out = torch.empty_like(q, dtype=torch.float64)
    for b, n in enumerate(lens):
        s = torch.einsum("mhe,phe->hmp", q[b].double(), k[b].double()) / math.sqrt(q.shape[-1])
        seen = torch.arange(n + M, device=q.device)[None, :] <= n + torch.arange(M, device=q.device)[:, None]
        out[b] = torch.einsum("hmp,phe->mhe", s.masked_fill(~seen, -math.inf).softmax(-1), v[b].double())
    return out


# head size, heads, cached positions, rows per sequence, d_ff
LAYERS = [
    (128, 32, [252, 0, 63, 64, 65, 191, 192, 193], 4, 256), (128, 32, [511, 510, 512, 448, 449, 447, 1, 250], 1, 256), (128, 40, [300, 255, 256, 257, 319, 320, 17, 128], 9, 256),
    (128, 32, [1000, 40, 575, 576, 577, 300, 2, 900], 16, 11008), (64, 32, [252, 0, 63, 64, 65, 511, 512, 513], 3, 256), (64, 64, [700, 255, 256, 639, 640], 16, 256)]
# ... of which these, by the bytes of a pass, ask for keys and values with the non-temporal bit (a wide d_ff, or many positions in a call of at most 16 rows)
STREAMED = [(128, 32, [1000, 40, 575, 576, 577, 300, 2, 900], 16, 4608), (64, 64, [700, 255, 256, 639, 640], 16, 4096), (128, 32, [1280 + 9 * i for i in range(16)], 1, 256)]


def _streams(hd, heads, lens, M, ff):
    """The library's own choice for a bf16 model of one layer whose matrices are few enough to be asked for without the bit."""
    W = hd * heads
    matrices = 2 * (4 * W * W + 3 * W * ff)
    rows = len(lens) * M
    assert rows <= 16 or matrices < 256 << 20
    f = sv.lib().ss_dev_streams_kv
    f.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int]
    return bool(f(matrices, 4 * W * sum(lens), rows))


def test_keys_and_values_are_streamed_where_the_cache_does_not_hold_them():
    f = sv.lib().ss_dev_streams_kv
    f.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int]
    MB = 1 << 20
    # up to 16 rows ask for every matrix with the bit: keys and values have the cache of 256 MB to themselves
    assert [f(400 * MB, kv * MB, 16) for kv in (0, 136, 262, 319, 320, 500)] == [0, 0, 0, 0, 1, 1]
    # more rows: with the matrices that come without it
    assert [f(118 * MB, kv * MB, 17) for kv in (0, 64, 105, 106, 500)] == [0, 0, 0, 1, 1]
    assert [f(plain * MB, 0, 256) for plain in (0, 223, 224)] == [0, 0, 1]
    assert not any(_streams(*c) for c in LAYERS if c[4] == 256 and c[1] == 32) and all(_streams(*c) for c in STREAMED)


@pytest.mark.gpu
@pytest.mark.parametrize("hd,heads,lens,M,ff", LAYERS + STREAMED)
def test_layer_attention_against_64_bits(hd, heads, lens, M, ff):
    """A layer whose d_ff part is nearly nothing and whose O projection is the identity: h grows by the attention's result.  Queries, weights and
    results carry 16 bits (two planes), sums 32: 2^-16 of values around 1, and of the sum of the weights, which is 1."""
    B, W, d = len(lens), heads * hd, heads * hd
    g = torch.Generator(device=dev()).manual_seed(hd + heads)
    r = lambda *s: torch.randn(s, generator=g, device=dev())
    eye = torch.eye(d, device=dev(), dtype=torch.bfloat16)
    L = {"wqkv": (r(3 * W, d) * 0.02).to(torch.bfloat16), "wo": eye, "wgu": torch.zeros(2 * ff, d, device=dev(), dtype=torch.bfloat16),
         "wd": torch.zeros(d, ff, device=dev(), dtype=torch.bfloat16), "g1": torch.ones(d, device=dev()), "g2": torch.ones(d, device=dev())}
    gm = sv.Model(si.DecoderShape(1, d, heads, hd, ff, 64, dtype="bf16"), None, max_rows=B * M, max_pos=max(lens) + 64, packed_layers=[L])
    kv = sv.KVCache(gm, B, max(lens) + 40)
    S = (max(lens) + 40 + 63) // 64 * 64
    for b, n in enumerate(lens):
        if n:
            sv.ss_kv_cache_append(kv, 0, b, 0, r(n, W).to(torch.bfloat16), r(n, W).to(torch.bfloat16))
    sv.ss_kv_cache_set_len(kv, lens)
    h = r(B * M, d)
    out = sv.ss_decoder_layers_forward(gm, kv, h.clone(), B, M)
    cache = kv.buf.view(torch.bfloat16)[:2 * B * heads * S * hd].view(2, B, heads, S, hd)
    k = [cache[0, b, :, :n + M].permute(1, 0, 2).float() for b, n in enumerate(lens)]
    v = [cache[1, b].reshape(heads, S // 64, hd, 64).permute(0, 1, 3, 2).reshape(heads, S, hd)[:, :n + M].permute(1, 0, 2).float() for b, n in enumerate(lens)]
    x = h.double()
    q = (x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5)) @ L["wqkv"][:W].double().t()
    q = q.view(B, M, heads, hd)
    pos = torch.tensor(lens, device=dev(), dtype=torch.float64)[:, None] + torch.arange(M, device=dev(), dtype=torch.float64)
    ang = pos[..., None] * 10000.0 ** (-2.0 * torch.arange(hd // 2, device=dev(), dtype=torch.float64) / hd)
    cs, sn = ang.cos()[:, :, None], ang.sin()[:, :, None]
    lo, hi = q[..., :hd // 2], q[..., hd // 2:]
    q = torch.cat([lo * cs - hi * sn, lo * sn + hi * cs], -1)
    want = _want(q, k, v, lens, M).reshape(B * M, W)
    got = out.double() - x
    # a score's error: 2^-17 of each of hd products of about 1 x 1.3, over sqrt(hd), and the fp32 rotation; results of up to 4: 1e-4 is ten of them
    assert float((got - want).norm() / want.norm()) < 3e-5
    assert float((got - want).abs().max()) < 3e-4


@pytest.mark.gpu
@pytest.mark.parametrize("hd,heads", [(128, 32), (64, 32), (128, 40)])
def test_positions_behind_the_end_need_not_be_numbers(hd, heads):
    """What a longer sequence left behind the half block (32 positions) that holds the end: the same bits as with zeros.  Positions between the end and the
    next multiple of 32 are multiplied with weights of zero, here and in every other attention kernel: they have to be finite and are zeros here."""
    lens, M, d, S = [257, 270, 284, 320, 14, 383, 321, 510], 4, heads * hd, 640
    g = torch.Generator(device=dev()).manual_seed(hd + heads)
    r = lambda *s: torch.randn(s, generator=g, device=dev())
    L = {"wqkv": (r(3 * d, d) * 0.02).to(torch.bfloat16), "wo": torch.eye(d, device=dev(), dtype=torch.bfloat16), "wgu": torch.zeros(512, d, device=dev(), dtype=torch.bfloat16),
         "wd": torch.zeros(d, 256, device=dev(), dtype=torch.bfloat16), "g1": torch.ones(d, device=dev()), "g2": torch.ones(d, device=dev())}
    gm = sv.Model(si.DecoderShape(1, d, heads, hd, 256, 64, dtype="bf16"), None, max_rows=len(lens) * M, max_pos=S, packed_layers=[L])
    h, k, v = r(len(lens) * M, d), [r(n, d) for n in lens], [r(n, d) for n in lens]
    out = []
    for behind in (0.0, math.nan, math.inf):
        kv = sv.KVCache(gm, len(lens), S)
        for b, n in enumerate(lens):
            full = torch.full((2, S, d), behind, device=dev())
            full[:, :(n + M + 31) // 32 * 32] = 0
            full[0, :n], full[1, :n] = k[b], v[b]
            sv.ss_kv_cache_append(kv, 0, b, 0, full[0].to(torch.bfloat16), full[1].to(torch.bfloat16))
        sv.ss_kv_cache_set_len(kv, lens)
        out.append(sv.ss_decoder_layers_forward(gm, kv, h.clone(), len(lens), M))
    assert bool(out[0].isfinite().all()) and torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
