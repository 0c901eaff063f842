"""What rides on another launch of the forward pass: the embedding with the first norm, the lengths with the last
projection, the final norm with the last projection, the hidden rows worked on where the caller holds them."""
import pytest
import torch

import oracle
import paper_2311_04951_amd as sv
import seeded_inputs as si
from gpu_util import dev, maxabs, weights_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,rows", [(1, 1), (3, 5), (3, 8), (5, 16)])      # 1, 15 rows; 24 and 80 rows take the GEMMs of more than 16
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


@pytest.mark.parametrize("V", [1, 3, 1000, 4096, 8193, 32000, 50257, 128256])
@pytest.mark.parametrize("B,K", [(1, 0), (2, 4), (9, 15), (200, 8)])
def test_greedy_acceptance_by_segments(V, B, K):
    """Rows cut into segments, one to many, aligned and not, with ties across segments, infinities and NaNs, and a workspace that
    holds no pairs at all: the lowest index of the largest value, NaNs aside."""
    if B * V > 4_000_000:
        B = max(1, 4_000_000 // V)
    x = torch.randint(-4, 5, (B, K + 1, V), generator=torch.Generator().manual_seed(V + B)).float()     # ties everywhere
    x[0, 0] = -torch.inf
    if V > 5:
        x[-1, -1, 5] = torch.inf
        x[-1, -1, 0] = torch.nan
        x[0, K, V - 1] = 9.0
    best = torch.where(x.isnan(), -torch.inf, x).argmax(-1).to(torch.int32)
    first = torch.where(x.isnan(), -torch.inf, x) == torch.where(x.isnan(), -torch.inf, x).max(-1, keepdim=True).values
    best = first.float().argmax(-1).to(torch.int32)                                 # the lowest index
    d = best[:, :K].clone()
    d[torch.rand(d.shape, generator=torch.Generator().manual_seed(1)) < 0.2] += 1
    want_n = [next((i for i in range(K) if d[b, i] != best[b, i]), K) for b in range(B)]
    tight = sv.ss_workspace_init(torch.empty(256 + 65536 + 4 * B * (K + 1) + 16, dtype=torch.uint8, device=dev()))
    for ws in (None, tight):
        na, nx = sv.ss_greedy_accept(x.to(dev()), d.contiguous().to(dev()), ws=ws)
        assert na.tolist() == want_n
        assert nx.tolist() == [int(best[b, n]) for b, n in enumerate(want_n)]


@pytest.mark.parametrize("V", [64, 1000, 1027, 6144, 6145, 16384, 16388])      # one launch up to 6144; one statistics segment up to 16384
def test_a_draft_step_in_one_sampling_launch_gives_the_bits_of_the_separate_ones(V):
    shape = si.DecoderShape(1, 256, 4, 64, 344, V, dtype="f32")
    gm = sv.Model(shape, weights_to_device(si.decoder_weights(shape, seed=73)), max_rows=16, max_pos=64)
    for batch, T in ((1, 1.0), (5, 0.3)):
        toks = si.token_ids(73, "t", (batch, 1), V).to(dev())
        u = si.uniforms(73, f"u{batch}", (batch,)).to(dev())
        ld = V + 3
        q = torch.full((batch, ld), -1.0, device=dev())
        out = torch.empty(batch, dtype=torch.int32, device=dev())
        sv.ss_draft_step(gm, sv.KVCache(gm, batch, 32), toks, 1, T, u, q, ld, out)
        logits = sv.ss_verify_forward(gm, sv.KVCache(gm, batch, 32), toks, 1)
        p = sv.ss_softmax(logits.reshape(batch, 1, V), T)
        assert torch.equal(q[:, :V], p[:, 0]) and bool((q[:, V:] == -1).all())
        none = torch.zeros(1, dtype=torch.int32, device=dev())
        _, tok = sv.ss_speculative_accept(p, p, none, u.reshape(batch, 1).contiguous())      # K = 0: a plain sample
        assert out.tolist() == tok.tolist()


@pytest.mark.skipif(torch.cuda.is_available() and torch.cuda.mem_get_info()[0] < 120 << 30, reason="the model's buffers take 80 GB")
def test_few_rows_of_a_model_whose_activation_planes_pass_4_gib():
    """A model sized for so many rows that one activation plane of max_rows x d_ff holds more than 2^32 bytes: calls of a few rows
    give the bits that the same weights give in a small model (their GEMMs address the planes with 32 bits)."""
    shape = si.DecoderShape(1, 256, 4, 64, 32768, 64, dtype="bf16")
    w = weights_to_device(si.decoder_weights(shape, seed=74))
    toks = si.token_ids(74, "t", (1, 5), shape.vocab).to(dev())
    outs = []
    for max_rows in (16, 65552):
        assert max_rows == 16 or max_rows * shape.d_ff * 2 > 1 << 32
        gm = sv.Model(shape, w, max_rows=max_rows, max_pos=32)
        kv = sv.KVCache(gm, 1, 16)
        outs.append(sv.ss_verify_forward(gm, kv, toks, 5).clone())
        torch.cuda.synchronize()
        del kv, gm
    assert torch.equal(outs[0], outs[1])


@pytest.mark.skipif(torch.cuda.is_available() and torch.cuda.mem_get_info()[0] < 120 << 30, reason="the model's buffers take 40 to 80 GB")
@pytest.mark.parametrize("max_rows", [32800, 65552])      # planes 2 and 4 GiB apart
@pytest.mark.parametrize("grid8", [False, True])
def test_the_persistent_kernel_on_a_model_whose_activation_planes_lie_far_apart(grid8, max_rows):
    """Both planes are read through one buffer descriptor with 32-bit offsets: the bits of a small model with the same weights."""
    shape = si.DecoderShape(1, 256, 4, 64, 32768, 64, dtype="bf16")
    w = weights_to_device(si.decoder_weights(shape, seed=75))
    toks = si.token_ids(75, "t", (1, 5), shape.vocab).to(dev())
    outs = []
    for rows in (16, max_rows):
        gm = sv.Model(shape, w, max_rows=rows, max_pos=32)
        sv.ss_model_set_persistent(gm, True)
        if grid8:
            sv.ss_model_set_persistent_options(gm, 8, True)
        kv = sv.KVCache(gm, 1, 16)
        outs.append(sv.ss_verify_forward(gm, kv, toks, 5).clone())
        assert sv.ss_device_status(gm) == 0
        del kv, gm
    assert bool(torch.isfinite(outs[0]).all()) and torch.equal(outs[0], outs[1])


def test_greedy_acceptance_of_rows_that_hold_nothing_but_nan_and_minus_infinity():
    """NaNs lose to everything, minus infinity included, wherever the cuts between segments fall; a row of NaNs alone gives index 0."""
    V = 20000                                                       # four segments of 5000 in a workspace that holds their pairs
    x = torch.full((1, 4, V), -torch.inf)
    x[0, 0, :5000] = torch.nan                                      # the whole first segment
    x[0, 1, :12345] = torch.nan                                     # two segments and part of the third
    x[0, 2] = torch.nan
    x[0, 2, V - 1] = -torch.inf                                     # one number, the last
    x[0, 3] = torch.nan
    want = [5000, 12345, V - 1, 0]
    for K in range(4):
        rows = x[:, 3 - K:].contiguous().to(dev())                  # every row is a position's and, in its turn, the first mismatch
        best = want[3 - K:]
        for n in range(K + 1):
            d = torch.tensor([best[:K]], dtype=torch.int32)
            if n < K:
                d[0, n] += 1
            for ws in (None, sv.ss_workspace_init(torch.empty(256 + 65536 + 4 * (K + 1) + 16, dtype=torch.uint8, device=dev()))):
                na, nx = sv.ss_greedy_accept(rows, d.to(dev()), ws=ws)
                assert (na.tolist(), nx.tolist()) == ([n], [best[n]]), (K, n, ws is None)
