"""Calls of more than 16 rows with int8 and int4 matrices: every tile of the GEMM that there is for them, ragged rows, columns and (int8) K."""
import ctypes

import pytest
import torch

import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev

STORE, RESID, SWIGLU, QKV = range(4)
# rows, d_model, heads of 128, d_ff: K and columns that end inside a tile, K split and not, one row block and several, the last one nearly empty
LAYERS = {8: [(17, 1040, 8, 1744), (18, 1040, 8, 13824), (40, 1040, 8, 13824), (72, 1040, 8, 13824), (40, 1040, 8, 16528), (33, 1040, 8, 1744), (49, 1040, 12, 1744), (80, 4096, 32, 1040), (81, 1040, 8, 1744), (96, 2048, 64, 11008), (128, 1040, 8, 2064), (18, 4096, 32, 144),
              (128, 2048, 32, 8192), (129, 1040, 12, 1744), (161, 144, 40, 11008), (192, 1040, 32, 5632), (256, 4096, 32, 2064), (250, 144, 16, 11008), (272, 1040, 8, 1744)],
          4: [(17, 1024, 8, 1792), (18, 1024, 8, 13824), (40, 1024, 8, 13824), (72, 1024, 8, 13824), (40, 1024, 8, 16512), (33, 1024, 8, 1792), (49, 1152, 12, 1792), (80, 4096, 32, 1152), (81, 1024, 9, 1792), (96, 2048, 64, 11008), (128, 1024, 8, 2048), (18, 4096, 32, 128),
              (128, 2048, 32, 8192), (129, 1152, 12, 1792), (161, 128, 40, 11008), (192, 1024, 32, 5632), (256, 4096, 32, 2048), (250, 128, 16, 11008), (272, 1024, 8, 1792)]}
# what those leave out of each product's own tiles; the last of int8 has matrices of more than 256 MB, which are asked for with the non-temporal bit
LAYERS[8] += [(40, 4096, 32, 2064), (100, 3088, 40, 1744), (120, 4096, 32, 1040), (144, 4112, 24, 4096), (192, 4096, 32, 2064), (288, 144, 40, 4096), (24, 128, 2, 11008), (161, 4112, 12, 272),
              (288, 4112, 2, 272), (40, 144, 1, 272), (40, 5120, 40, 13824)]
LAYERS[4] += [(40, 4096, 32, 2048), (100, 3072, 24, 1792), (120, 4096, 32, 1024), (144, 4096, 24, 4096), (192, 4096, 32, 2048), (288, 128, 40, 4096), (24, 128, 2, 11008), (256, 3072, 12, 1024),
              (288, 256, 2, 128), (40, 512, 1, 128), (320, 640, 1, 4096)]
HEADS = [(17, 333), (24, 32000), (40, 50257), (72, 32000), (72, 5003), (90, 32000), (200, 32000)]      # rows, columns; K 256
HEADS += [(40, 1000), (40, 32000), (32, 50257), (48, 33000)]                                           # one round of workgroups and more


def _met(bits):
    L = sv.lib()
    L.ss_dev_gemm_tile_bits.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    out, met = (ctypes.c_int * 3)(), set()

    def tile(epi, R, N, K, ws):
        L.ss_dev_gemm_tile_bits(bits, epi, R, N, K, ws, out)
        met.add((epi, out[0], out[1], out[2] > 1))

    for R, d, heads, ff in LAYERS[bits]:
        W = 128 * heads
        for epi, N, K in ((QKV, 3 * W, d), (RESID, d, W), (SWIGLU, ff, d), (RESID, d, ff)):
            tile(epi, R, N, K, 4 * max(3 * W, 2 * ff, d) * ((R + 15) // 16) * 64)
    for R, V in HEADS:
        tile(STORE, R, V, 256, 0)
    return met


@pytest.mark.parametrize("bits", [8, 4])
def test_the_shapes_below_meet_every_tile(bits):
    met = _met(bits)
    for epis, built in (((QKV, SWIGLU), {(r, c) for r in (32, 48, 80, 96, 128) for c in (96, 192)} | {(r, 128) for r in (32, 48, 80)}),
                        ((RESID, STORE), {(32, 64), (32, 128), (48, 64), (48, 128), (80, 64), (80, 128), (96, 128), (128, 128)})):
        assert {m[1:3] for m in met if m[0] in epis} == built
    assert {m[3] for m in met if m[0] == QKV} == {m[3] for m in met if m[0] == RESID} == {False, True}


@pytest.mark.parametrize("bits", [8, 4])
def test_the_shapes_below_meet_every_tile_of_every_product(bits):
    """Every epilogue is a kernel of its own, with its own registers, columns and ends."""
    met = _met(bits)
    rows, plain = (32, 48, 80, 96, 128), {(32, 64), (32, 128), (48, 64), (48, 128), (80, 64), (80, 128), (96, 128), (128, 128)}
    built = {(QKV, r, c) for r in rows for c in (96, 192)} | {(SWIGLU, r, c) for r in rows for c in (96, 192)} | {(SWIGLU, r, 128) for r in (32, 48, 80)}
    assert {m[:3] for m in met} == built | {(e, r, c) for e in (STORE, RESID) for r, c in plain}
    # with K split and not, wherever the choice comes to it
    for r in rows:
        assert {s for e, rr, c, s in met if (e, rr) == (RESID, r)} >= ({True} if r > 80 else {False, True}), r


def test_a_few_groups_of_k():
    """int4, K of up to 512, more than 48 rows of QKV or gate/up: blocks of 96 rows.  A residual projection of 256 < K < 512, both widths: K in one piece."""
    L = sv.lib()
    L.ss_dev_gemm_tile_bits.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    out = (ctypes.c_int * 3)()

    def tile(bits, epi, R, N, K):
        L.ss_dev_gemm_tile_bits(bits, epi, R, N, K, 1 << 30, out)
        return tuple(out)

    for epi in (QKV, SWIGLU):
        for K in (128, 256, 512):
            assert [tile(4, epi, R, 384, K)[0] for R in (32, 48, 49, 80, 96, 128)] == [32, 48, 96, 96, 96, 96]
            assert tile(8, epi, 80, 384, K)[0] == 80
        assert tile(4, epi, 80, 384, 640)[0] == 80
    for bits in (8, 4):
        assert [tile(bits, RESID, R, 128, 384)[2] for R in (18, 80, 256)] == [1, 1, 1] and tile(bits, RESID, 80, 256, 256)[2] > 1 and tile(bits, RESID, 18, 128, 768)[2] > 1


def _dequantised(w, bits):
    """The matrix that a quantised model stands for, in 64 bits: scales of 32 bits, entries of q."""
    top = 127.0 if bits == 8 else 7.0
    g = w.double().view((w.shape[0], 1, -1) if bits == 8 else (w.shape[0], -1, 128))
    amax = g.abs().amax(-1, keepdim=True)
    # the rule divides in 32 bits: a 64-bit quotient of 32-bit numbers, rounded to 32 bits, is that quotient
    scale = torch.where(amax > 0, (amax / top).float().double(), 1.0)
    return (torch.round((g / scale).float()).clamp_(-top, top).double() * scale).view(w.shape)


def _rms(x, g):
    x = x.double()
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-5) * g.double()


@pytest.mark.gpu
@pytest.mark.parametrize("bits,i", [(b, i) for b in (8, 4) for i in range(len(LAYERS[b]))])
def test_one_layer_against_64_bits(bits, i):
    """A layer without cached positions, one row per sequence, whose attention is the row's own value: four products.  Activations carry 16
    bits (two planes), sums and scales 32: 1e-5 relative, the bound of the bf16 matrices."""
    R, d, heads, ff = LAYERS[bits][i]
    W = heads * 128
    g = torch.Generator(device=dev()).manual_seed(R + bits)
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(torch.bfloat16)
    L = {"wqkv": n(3 * W, d), "wo": n(d, W), "wgu": n(2 * ff, d), "wd": n(d, ff), "g1": torch.ones(d, device=dev()), "g2": torch.ones(d, device=dev())}
    gm = sv.Model(si.DecoderShape(1, d, heads, 128, ff, 64, dtype="bf16"), None, max_rows=R, max_pos=64, packed_layers=[L], int8_weights=bits == 8, int4_weights=bits == 4)
    h = torch.randn((R, d), generator=g, device=dev())
    kv = sv.KVCache(gm, R, 16)
    out = sv.ss_decoder_layers_forward(gm, kv, h.clone(), R, 1)
    v = kv.buf.view(torch.bfloat16)[R * W * 64:].view(R, heads, 128, 64)[..., 0].reshape(R, W).double()
    want = _rms(h, L["g1"]) @ _dequantised(L["wqkv"][2 * W:].contiguous(), bits).t()
    # half a unit of bf16 and the sum's own error (see test_gpu_tile_gemm.py)
    assert float(((v - want).abs() - 2.0 ** -8 * want.abs()).max()) < 5e-5
    x = h.double() + v @ _dequantised(L["wo"], bits).t()
    gate, up = (_rms(x, L["g2"]) @ _dequantised(L["wgu"], bits).t()).split(ff, -1)
    x = x + (gate * torch.sigmoid(gate) * up) @ _dequantised(L["wd"], bits).t()
    assert float((out.double() - x).norm() / x.norm()) < 1e-5
    assert float((out.double() - x).abs().max()) < 1e-3


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("R,V", HEADS)
def test_a_head_against_64_bits(R, V, bits):
    g = torch.Generator(device=dev()).manual_seed(R + V)
    d = 256
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(torch.bfloat16)
    ends = {"embed": n(V, d), "gf": torch.ones(d, device=dev()), "lm_head": n(V, d)}
    gm = sv.Model(si.DecoderShape(0, d, 4, 64, 128, V, dtype="bf16"), ends, max_rows=R, max_pos=64, packed_layers=[], int8_weights=bits == 8, int4_weights=bits == 4)
    toks = torch.randint(0, V, (R, 1), generator=g, device=dev(), dtype=torch.int32)
    got = sv.ss_verify_forward(gm, sv.KVCache(gm, R, 16), toks, 1)[:, 0].double()
    want = _rms(ends["embed"][toks[:, 0].long()].float(), ends["gf"]) @ _dequantised(ends["lm_head"], bits).t()
    assert float((got - want).norm() / want.norm()) < 1e-5
    assert float((got - want).abs().max()) < 1e-4
