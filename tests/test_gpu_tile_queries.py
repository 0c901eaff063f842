"""Calls of more than 16 rows over cached positions, bf16, int8 and int4 matrices: queries, keys, values and their rotation for every tile of the
QKV product, with K split and not.  (A layer without cached positions shows its values alone: a softmax over one position is 1.)"""
import ctypes
import math

import pytest
import torch

import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev
from test_gpu_tile_quantised import _dequantised, _rms

# rows, d_model, heads of 128: every (rows of a block, columns, K split or not) that the choice can come to with up to 40 heads
SHAPES = {16: [(17, 136, 2), (17, 2056, 2), (17, 2048, 16), (18, 3080, 24), (33, 136, 2), (33, 1160, 2), (40, 2056, 16), (33, 3072, 24), (49, 136, 2), (49, 1032, 2), (129, 136, 24),
               (50, 1160, 16), (129, 136, 40), (129, 2048, 12), (161, 136, 2), (161, 1032, 2), (288, 128, 24), (161, 1160, 12), (81, 136, 2), (81, 1032, 2), (200, 136, 40), (81, 4104, 24)],
          8: [(17, 144, 2), (17, 2064, 2), (18, 3088, 24), (33, 144, 2), (33, 2048, 2), (33, 2048, 24), (49, 144, 2), (49, 1040, 2), (288, 144, 24), (72, 4096, 32), (129, 3072, 12), (81, 144, 16),
              (81, 1168, 8), (256, 144, 40), (161, 4112, 12), (200, 144, 24), (200, 2064, 8), (100, 3088, 40)],
          4: [(17, 128, 2), (17, 2048, 2), (18, 2176, 24), (33, 128, 2), (33, 1024, 2), (40, 2048, 24), (49, 128, 2), (49, 1152, 2), (288, 128, 24), (72, 4096, 32), (129, 2176, 12), (81, 128, 16),
              (81, 1152, 8), (256, 128, 40), (161, 3072, 12), (200, 128, 24), (200, 2176, 8), (100, 3072, 24), (288, 640, 24), (64, 640, 2), (96, 1024, 8), (320, 128, 40)]}
QKV, D_FF = 3, 128


def _tile(bits, R, d, heads):
    L = sv.lib()
    L.ss_dev_gemm_tile_bits.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    out, W = (ctypes.c_int * 3)(), 128 * heads
    L.ss_dev_gemm_tile_bits(bits, QKV, R, 3 * W, d, 4 * max(3 * W, 2 * D_FF, d) * ((R + 15) // 16) * 64, out)
    return out[0], out[1], out[2] > 1


@pytest.mark.parametrize("bits", [16, 8, 4])
def test_the_shapes_below_meet_every_tile_of_the_qkv_product(bits):
    met = {_tile(bits, *s) for s in SHAPES[bits]}
    for rows in (32, 48, 80, 96, 128):
        for cols in (64, 96, 192) if bits == 16 and rows < 96 else (96, 192):
            assert {m[2] for m in met if m[:2] == (rows, cols)}, (rows, cols)
        assert {m[2] for m in met if m[0] == rows} == {False, True}, rows


def _rotated(x, pos):
    """x [rows, heads, 128], halves rotated by the row's position."""
    ang = pos.double()[:, None] * 10000.0 ** (-2.0 * torch.arange(64, device=x.device, dtype=torch.float64) / 128)
    cs, sn = ang.cos()[:, None], ang.sin()[:, None]
    lo, hi = x[..., :64], x[..., 64:]
    return torch.cat([lo * cs - hi * sn, lo * sn + hi * cs], -1)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,i", [(b, i) for b in SHAPES for i in range(len(SHAPES[b]))])
def test_one_layer_over_cached_positions_against_64_bits(bits, i):
    """One row per sequence behind 0 to 6 positions.  Activations carry 16 bits (two planes), sums, scales and the rotation 32; keys and values go
    to the cache in bf16, and the rest starts from what it holds."""
    R, d, heads = SHAPES[bits][i]
    W = 128 * heads
    g = torch.Generator(device=dev()).manual_seed(R + bits)
    r = lambda *s: torch.randn(s, generator=g, device=dev())
    n = lambda *s: (r(*s) * 0.02).to(torch.bfloat16)
    # (entries of 0.02 would leave scores of a short K near zero, and with them whatever a query is)
    L = {"wqkv": (r(3 * W, d) / math.sqrt(d)).to(torch.bfloat16), "wo": n(d, W), "wgu": n(2 * D_FF, d), "wd": n(d, D_FF), "g1": torch.ones(d, device=dev()), "g2": torch.ones(d, device=dev())}
    gm = sv.Model(si.DecoderShape(1, d, heads, 128, D_FF, 64, dtype="bf16"), None, max_rows=R, max_pos=64, packed_layers=[L], int8_weights=bits == 8, int4_weights=bits == 4)
    kv = sv.KVCache(gm, R, 16)
    lens = [b % 7 for b in range(R)]
    for b, m in enumerate(lens):
        if m:
            sv.ss_kv_cache_append(kv, 0, b, 0, r(m, W).to(torch.bfloat16), r(m, W).to(torch.bfloat16))
    sv.ss_kv_cache_set_len(kv, lens)
    h = r(R, d)
    out = sv.ss_decoder_layers_forward(gm, kv, h.clone(), R, 1)

    w = {k: _dequantised(v, bits) if bits < 16 else v.double() for k, v in L.items() if k[0] == "w"}
    q, k, v = (_rms(h, L["g1"]) @ w["wqkv"].t()).view(R, 3, heads, 128).unbind(1)
    pos = torch.tensor(lens, device=dev())
    q, k = _rotated(q, pos), _rotated(k, pos)
    cache = kv.buf.view(torch.bfloat16)[:2 * R * W * 64].view(2, R, heads, 64 * 128)
    keys = cache[0].view(R, heads, 64, 128).permute(0, 2, 1, 3).double()       # [R, 64, heads, 128]
    values = cache[1].view(R, heads, 128, 64).permute(0, 3, 1, 2).double()
    rows = torch.arange(R, device=dev())
    # half a unit of bf16 and the sum's own error, turned by at most sqrt(2) (see test_gpu_tile_gemm.py)
    assert float(((keys[rows, pos] - k).abs() - 2.0 ** -8 * k.abs()).max()) < 1e-4
    assert float(((values[rows, pos] - v).abs() - 2.0 ** -8 * v.abs()).max()) < 1e-4
    seen = torch.arange(7, device=dev())[None, :] <= pos[:, None]
    s = (q[:, None] * keys[:, :7]).sum(-1) / math.sqrt(128)                      # [R, 7, heads]
    p = s.masked_fill(~seen[..., None], -math.inf).softmax(1)
    attn = torch.where(seen[..., None, None], p[..., None] * values[:, :7], 0.0).sum(1).reshape(R, W)
    x = h.double() + attn @ w["wo"].t()
    gate, up = (_rms(x, L["g2"]) @ w["wgu"].t()).split(D_FF, -1)
    x = x + (gate * torch.sigmoid(gate) * up) @ w["wd"].t()
    # a score's error: 2^-17 of each of 128 products around 1, over sqrt(128); then that of the four products
    assert float((out.double() - x).norm() / x.norm()) < 2e-5
    assert float((out.double() - x).abs().max()) < 1e-3
