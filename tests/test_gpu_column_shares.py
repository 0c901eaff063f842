"""Calls of at most 16 rows: the output columns of every GEMM dealt out evenly over the workgroups (one to eight quads each, one or several
workgroups per compute unit, the last quad in part), ragged K, every kind of matrix and both operand layouts (up to 8 rows, more)."""
import ctypes

import pytest
import torch

import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev

KINDS = ["f32", "bf16", "int8", "int4"]
ROWS = [1, 2, 5, 8, 9, 16]
# d_model, heads of 128, d_ff: shares of 1, 2 - 3, 5 - 6 and 7 - 8 quads in each of the four matrices of a layer
LAYERS = [(256, 2, 384), (1152, 16, 2816), (2304, 32, 5632), (5248, 40, 8192), (1152, 64, 11008), (1152, 80, 13824), (7168, 2, 384)]
RAGGED = {"f32": -52, "bf16": -56, "int8": -16, "int4": 0}      # added to a d_model of 1152 and a d_ff of 384: K ends inside a step (int4: half way)
VOCABS = [1, 6, 333, 3001, 5003, 8190, 11264, 32000, 50257]


def _share(epi, R, N):
    L = sv.lib()
    L.ss_dev_gemm_share.argtypes = [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    L.ss_dev_gemm_share.restype = None
    out = (ctypes.c_int * 3)()
    L.ss_dev_gemm_share(epi, R, N, out)
    groups, quads, rest = out
    return groups, quads, rest


def test_shares_cover_the_columns_and_every_size_is_met():
    """No GPU: shares add up, differ by one quad at most, hold eight at most; the shapes below meet every one that a kernel is built for."""
    STORE, RESID, SWIGLU, QKV = range(4)
    met = set()
    for R in ROWS:
        for epi, N in [(e, n) for d, h, ff in LAYERS for e, n in ((QKV, 384 * h), (RESID, d), (SWIGLU, ff))] + [(STORE, v) for v in VOCABS]:
            groups, quads, rest = _share(epi, R, N)
            assert groups * quads + rest == (N // 8 if epi == QKV else -(-N // 4)) and 0 <= rest < groups and 1 <= quads + (rest > 0) <= 8
            met.add((epi, R > 8, groups > 256, (quads + (rest > 0) + 1) // 2))
    for more in (False, True):
        for epi in (STORE, SWIGLU, QKV):
            assert {ei for e, m, many, ei in met if (e, m, many) == (epi, more, False)} == {1, 2, 3, 4}, (epi, more)
            # several workgroups per unit: shares of up to 4 quads and of 7 or 8 up to 8 rows, of 5 or 6 and of 7 or 8 beyond - no others, of any matrix
            assert {ei for e, m, many, ei in met if (e, m, many) == (epi, more, True)} == ({3, 4} if more else {2, 4}), (epi, more)
        assert {ei for e, m, many, ei in met if (e, m) == (RESID, more)} == {1, 2, 3, 4}


@pytest.mark.parametrize("R", [1, 8, 9, 16])
def test_no_matrix_has_a_share_that_no_kernel_is_built_for(R):
    """No GPU: of all sizes up to 300000 columns, those with more than one workgroup per compute unit."""
    for epi in range(4):
        for N in range(96 if epi == 3 else 8193, 300000, 96 if epi == 3 else 7):
            groups, quads, rest = _share(epi, R, N)
            ei = (quads + (rest > 0) + 1) // 2
            assert ei <= 4 and (groups <= 256 or ei in ((2, 4) if R <= 8 else (3, 4))), (epi, N)


def _rms(x, eps=1e-5):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps)


def _matrix(w, kind):
    """What a matrix of this kind stands for, by the rule of the C header, in 64 bits."""
    if kind in ("f32", "bf16"):
        return w.double()
    top = 127.0 if kind == "int8" else 7.0
    g = w.double().view((w.shape[0], -1, 128) if kind == "int4" else (w.shape[0], 1, -1))
    amax = g.abs().amax(-1, keepdim=True)
    scale = torch.where(amax > 0, (amax / top).float().double(), 1.0)
    return (torch.round((g / scale).float()).clamp_(-top, top).double() * scale).view(w.shape)


def _model(kind, shape, ends, layers):
    return sv.Model(shape, ends, max_rows=16, max_pos=64, packed_layers=layers, int8_weights=kind == "int8", int4_weights=kind == "int4")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d,heads,ff", LAYERS)
def test_two_layers_against_64_bits(d, heads, ff, kind):
    """Two layers without cached positions, one row per sequence: the attention of a row is its own value, so a layer is four products
    and the norms between them (deferred ones).  Activations carry 16 bits at least, sums 32: 1e-5 relative a layer."""
    d += RAGGED[kind] if d == 1152 else 0
    ff += RAGGED[kind] if ff == 384 else 0
    W, dt = heads * 128, torch.float32 if kind == "f32" else torch.bfloat16
    g = torch.Generator(device=dev()).manual_seed(d + ff)
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(dt)
    layer = lambda: {"wqkv": n(3 * W, d), "wo": n(d, W), "wgu": n(2 * ff, d), "wd": n(d, ff), "g1": 1 + n(d).float(), "g2": 1 + n(d).float()}
    layers = [layer(), layer()]
    gm = _model(kind, si.DecoderShape(2, d, heads, 128, ff, 64, dtype="f32" if kind == "f32" else "bf16"), None, layers)
    ref = [{k: (_matrix(v, kind) if k[0] == "w" else v.double()) for k, v in L.items()} for L in layers]
    for R in ROWS:
        h = torch.randn((R, d), generator=g, device=dev())
        kv = sv.KVCache(gm, R, 16)
        out = sv.ss_decoder_layers_forward(gm, kv, h.clone(), R, 1).double()
        values = kv.buf.view(dt)[2 * R * W * 64:].view(2, R, heads, 128, 64)[..., 0].reshape(2, R, W).double()
        x = h.double()
        for L, v in zip(ref, values):
            want = (_rms(x) * L["g1"]) @ L["wqkv"][2 * W:].t()
            # half a unit of the cache's type and the sum's own error
            assert float(((v - want).abs() - (2.0 ** -8 if dt == torch.bfloat16 else 0) * want.abs()).max()) < 5e-5, R
            x = x + v @ L["wo"].t()
            gate, up = ((_rms(x) * L["g2"]) @ L["wgu"].t()).split(ff, -1)
            x = x + (gate * torch.sigmoid(gate) * up) @ L["wd"].t()
        assert float((out - x).norm() / x.norm()) < 2e-5, R
        assert float((out - x).abs().max()) < 2e-3, R


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("V", VOCABS)
def test_a_head_against_64_bits(V, kind):
    """No layers: the norm of the embedded row times the head, the columns of the last share in part.  Sums of up to 1152 products in 32 bits:
    1e-5 of the outputs' rms, 0.02 sqrt(1152).  int4 entries are multiplied as q + 136 (even ones) and q + 24 (odd ones), and a group's
    sum starts at what these biases add to it: 136 sqrt(64) and 24 sqrt(64), 1105 together, whose roundings (2^-24 of it, some four to a group)
    the scale, 0.01, and nine groups leave at 1105 * 2^-24 * 0.01 * 2 * 3 = 4e-6, 6e-6 of that rms: six times that."""
    d = 1152 + RAGGED[kind]
    g = torch.Generator(device=dev()).manual_seed(V)
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(torch.float32 if kind == "f32" else torch.bfloat16)
    ends = {"embed": n(V, d), "gf": torch.ones(d, device=dev()), "lm_head": n(V, d)}
    gm = _model(kind, si.DecoderShape(0, d, 2, 64, 128, V, dtype="f32" if kind == "f32" else "bf16"), ends, [])
    head = _matrix(ends["lm_head"], kind)
    for R in ROWS:
        toks = torch.randint(0, V, (R, 1), generator=g, device=dev(), dtype=torch.int32)
        out = torch.full((R * V + 64,), 7.0, device=dev())
        got = sv.ss_verify_forward(gm, sv.KVCache(gm, R, 16), toks, 1, out[:R * V].view(R, 1, V))[:, 0].double()
        want = _rms(ends["embed"][toks[:, 0].long()].double()) @ head.t()
        rms = 0.02 * d ** 0.5
        assert float((got - want).square().mean().sqrt()) < (4e-5 if kind == "int4" else 1e-5) * rms, R
        assert float((got - want).abs().max()) < 2e-4 * rms, R
        assert bool((out[R * V:] == 7.0).all()), R
