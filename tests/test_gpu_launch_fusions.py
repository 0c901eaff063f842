"""What rides on another launch of the forward pass: the embedding with the first norm, the lengths with the last
projection, the final norm with the last projection, the hidden rows worked on where the caller holds them."""
import pytest
import torch

import oracle
import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev, maxabs, weights_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,rows", [(1, 1), (3, 5), (3, 8), (5, 16)])      # 1, 15 rows; 24 and 80 rows take the wide kernels
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_that_the_caller_holds_unaligned(dtype, batch, rows):
    """ss_decoder_layers_forward on rows at an address that is only 4-byte aligned: the same numbers as on aligned ones (the norm
    of the first layer adds its squares in another order: a few units of 2^-24), and every length moves by the rows of the call."""
    shape = si.DecoderShape(2, 256, 4, 64, 344, 500, dtype=dtype)
    w = si.decoder_weights(shape, seed=71)
    gm = sv.Model(shape, weights_to_device(w), max_rows=80, max_pos=256)
    h0 = si.normal(71, "h", (batch * rows, 256), 1.0).to(dev())
    arena = torch.zeros(batch * rows * 256 + 8, device=dev())
    outs = []
    for at in (0, 1):
        kv = sv.KVCache(gm, batch, 100)
        lens = [7 + 3 * b for b in range(batch)]
        sv.ss_kv_cache_set_len(kv, lens)
        h = arena[at:at + h0.numel()].view_as(h0)
        h.copy_(h0)
        sv.ss_decoder_layers_forward(gm, kv, h, batch, rows)
        assert sv.ss_kv_cache_get_len(kv).tolist() == [n + rows for n in lens]
        outs.append(h.clone())
    scale = float(outs[0].abs().max())
    assert float((outs[0] - outs[1]).abs().max()) <= 2e-5 * scale      # bf16: a rounded key or value may fall to the other side


@pytest.mark.parametrize("d", [256, 264, 100])      # final norm deferred; not deferrable (264); a row that is not a multiple of 256 loads
@pytest.mark.parametrize("batch,rows", [(1, 1), (2, 7), (1, 16), (3, 12)])
def test_embedding_and_final_norm_on_other_launches_match_the_oracle(d, batch, rows):
    shape = si.DecoderShape(1, d, 2, 64, 2 * d, 333, dtype="f32")
    w = si.decoder_weights(shape, seed=72)
    gm = sv.Model(shape, weights_to_device(w), max_rows=48, max_pos=128)
    om = oracle.Model(shape, w)
    toks = si.token_ids(72, "t", (batch, rows), shape.vocab)
    toks[0, 0] = shape.vocab + 5                                        # clamped to the last token, and flagged
    kv = sv.KVCache(gm, batch, 64)
    got = sv.ss_verify_forward(gm, kv, toks.to(dev()), rows)
    assert sv.ss_device_status(gm) == 1
    toks[0, 0] = shape.vocab - 1
    for b in range(batch):
        assert maxabs(got[b], om.forward(om.new_kv(64), toks[b].numpy())) < 1e-4
