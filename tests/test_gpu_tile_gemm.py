"""Calls of more than 16 rows with bf16 matrices: every tile of the GEMM (32, 48, 80 and 128 rows per workgroup with every column count
that there is, K split and not: test_tile_coverage.py asks the library which tile each shape below takes), ragged rows, columns and K."""
import pytest
import torch

import oracle
import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev, maxabs, weights_to_device

pytestmark = pytest.mark.gpu


def _rms(x, g, eps):
    x = x.double()
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


@pytest.mark.parametrize("batch,rows", [(2, 9), (2, 16), (3, 11), (3, 16), (5, 10), (5, 16), (6, 16), (9, 16), (16, 16), (17, 16)])
def test_ragged_batches_match_the_oracle(batch, rows):
    """18 to 272 rows; 333 columns in the head (a ragged last tile), K of 256, 688 (ends inside a stage of 64 and of 128) and 40 (d_ff: less
    than a stage).  Tolerance of the bf16 path: 2e-2 on logits."""
    for d, ff in ((256, 688), (128, 40)):
        shape = si.DecoderShape(2, d, d // 64, 64, ff, 333, dtype="bf16")
        w = si.decoder_weights(shape, seed=81)
        gm = sv.Model(shape, weights_to_device(w), max_rows=batch * rows, max_pos=128)
        om = oracle.Model(shape, w)
        toks = si.token_ids(81, "t", (batch, rows), shape.vocab)
        kv = sv.KVCache(gm, batch, 64)
        got = sv.ss_verify_forward(gm, kv, toks.to(dev()), rows)
        assert sv.ss_kv_cache_get_len(kv).tolist() == [rows] * batch
        for b in {0, batch // 2, batch - 1}:
            ref = om.forward(om.new_kv(64), toks[b].numpy())
            assert maxabs(got[b], ref) < 2e-2 and maxabs(got[b], ref) < 2e-2 * abs(ref).max()


LAYERS = [(R, d, heads, ff) for d, heads, ff in ((4096, 32, 1032), (1536, 12, 4104)) for R in (17, 33, 49, 72, 81, 128, 160, 256)]
# what those leave out: short K (few rows, many columns: wide tiles, no split), 7B- and 13B-shaped gate/up, the widest there is
LAYERS += [(17, 136, 8, 11008), (33, 136, 8, 11008), (81, 136, 8, 13824), (129, 136, 8, 11008), (17, 136, 64, 65536), (33, 136, 64, 65536), (49, 136, 64, 344),
           (17, 1096, 16, 344), (33, 1096, 16, 344), (129, 136, 40, 344), (1024, 2056, 16, 344), (144, 4096, 32, 11008), (256, 4096, 32, 11008)]
HEADS = [(R, V, 72) for R in (17, 40, 72, 200) for V in (333, 32000, 50257)]      # rows, columns, K


@pytest.mark.parametrize("R,d,heads,ff", LAYERS)      # K split four ways and less; columns and K that end inside a tile
def test_one_layer_against_64_bits(R, d, heads, ff):
    """A whole layer without cached positions, one row per sequence: the attention of a row is its own value, so the layer is four
    products.  bf16 matrices are exact, activations carry 16 bits (two planes), sums 32: 1e-5 relative."""
    W = heads * 128
    g = torch.Generator(device=dev()).manual_seed(R)
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(torch.bfloat16)
    L = {"wqkv": n(3 * W, d), "wo": n(d, W), "wgu": n(2 * ff, d), "wd": n(d, ff), "g1": torch.ones(d, device=dev()), "g2": torch.ones(d, device=dev())}
    shape = si.DecoderShape(1, d, heads, 128, ff, 64, dtype="bf16")
    gm = sv.Model(shape, None, max_rows=R, max_pos=64, packed_layers=[L])
    h = torch.randn((R, d), generator=g, device=dev())
    kv = sv.KVCache(gm, R, 16)
    out = sv.ss_decoder_layers_forward(gm, kv, h.clone(), R, 1)
    # the values as the cache holds them (bf16: one near the middle between two numbers may fall to either side, so the rest starts from these)
    v = kv.buf.view(torch.bfloat16)[R * W * 64:].view(R, heads, 128, 64)[..., 0].reshape(R, W).double()
    want = _rms(h, L["g1"], 1e-5) @ L["wqkv"][2 * W:].double().t()
    # half a unit of bf16, 2^-8 |want| at most, and the sum's own error: 4096 terms of 0.02 N(0, 1) times what two bf16 planes leave of an
    # activation (2^-18 rms), 64 * 0.02 * 2^-18 = 5e-6 rms; ten times that for the largest of 10^6
    assert float(((v - want).abs() - 2.0 ** -8 * want.abs()).max()) < 5e-5
    x = h.double() + v @ L["wo"].double().t()
    gate, up = (_rms(x, L["g2"], 1e-5) @ L["wgu"].double().t()).split(ff, -1)
    x = x + (gate * torch.sigmoid(gate) * up) @ L["wd"].double().t()
    assert float((out.double() - x).norm() / x.norm()) < 1e-5
    assert float((out.double() - x).abs().max()) < 1e-3


@pytest.mark.parametrize("R,V,d", HEADS)
def test_a_head_against_64_bits(R, V, d):
    """No layers: the norm of the embedded row times the head.  Activations of 16 bits, sums of 72 products in 32: 1e-5 relative."""
    g = torch.Generator(device=dev()).manual_seed(R + V)
    n = lambda *s: (torch.randn(s, generator=g, device=dev()) * 0.02).to(torch.bfloat16)
    ends = {"embed": n(V, d), "gf": torch.ones(d, device=dev()), "lm_head": n(V, d)}
    gm = sv.Model(si.DecoderShape(0, d, 2, 32, 64, V, dtype="bf16"), ends, max_rows=R, max_pos=64, packed_layers=[])
    toks = torch.randint(0, V, (R, 1), generator=g, device=dev(), dtype=torch.int32)
    got = sv.ss_verify_forward(gm, sv.KVCache(gm, R, 16), toks, 1)[:, 0].double()
    want = _rms(ends["embed"][toks[:, 0].long()].float(), ends["gf"], 1e-5) @ ends["lm_head"].double().t()
    assert float((got - want).norm() / want.norm()) < 1e-5
    assert float((got - want).abs().max()) < 1e-4


@pytest.mark.parametrize("d,ff", [(128, 344), (256, 688), (768, 1032)])
@pytest.mark.parametrize("batch,rows", [(32, 16), (33, 16), (57, 9), (64, 16)])      # 512 rows: the blocks of any call; 513 and more: those of the cost
def test_many_rows_of_a_short_k_match_the_oracle(batch, rows, d, ff):
    shape = si.DecoderShape(1, d, d // 64, 64, ff, 333, dtype="bf16")
    w = si.decoder_weights(shape, seed=82)
    gm = sv.Model(shape, weights_to_device(w), max_rows=batch * rows, max_pos=64)
    om = oracle.Model(shape, w)
    toks = si.token_ids(82, "t", (batch, rows), shape.vocab)
    got = sv.ss_verify_forward(gm, sv.KVCache(gm, batch, 64), toks.to(dev()), rows)
    for b in {0, batch // 2, batch - 1}:
        assert maxabs(got[b], om.forward(om.new_kv(64), toks[b].numpy())) < 2e-2
