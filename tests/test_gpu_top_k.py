"""Top-k selection on the GPU path (Section 3 lists it with top-p): the filter against the oracle bit for bit
(same kept set including ties and zero-weight tails, same renormalised values), alone and ahead of top-p, the
distribution the filtered rejection step emits on the kernels themselves, and the loops that use it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2311_04951_amd as sv
import seeded_inputs as si
from paper_2311_04951_amd import generate as gen
from gpu_util import dev, weights_to_device

pytestmark = pytest.mark.gpu


def _bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("V", [2, 64, 1000, 4095, 4096, 4097, 8191, 8192, 8193, 16384, 16385, 32769])
def test_the_cut_among_ties_is_the_oracles(V):
    """Equal weights in every place, in every other and in none but the ends of the wavefronts' parts: the last kept one found in the first
    part, at the ends of parts and in the last, whatever number of looks a part takes (up to 4096, 8192, 16384 entries and beyond)."""
    rows = np.full((3, V), 1.0 / V, dtype=np.float32)
    rows[1, 1::2] = 0.25 / V
    part = ((V + 15) // 16 + 63) // 64 * 64
    rows[2] = 0.25 / V
    for v in range(0, V, part):
        rows[2, v] = rows[2, min(v + part, V) - 1] = 1.0 / V
    g = torch.from_numpy(rows).to(dev())
    for k in sorted({k for k in (1, 2, 3, part - 1, part, part + 1, V // 2, V // 2 + 1, V - 2, V - 1) if 1 <= k < V}):
        got = sv.ss_top_k_filter(g, k)
        assert np.array_equal(_bits(got.cpu().numpy()), _bits(oracle.top_k_filter(rows, k))), (V, k)
    for top_p in (1e-6, 0.5, 0.9999):
        got = sv.ss_top_p_filter(g, top_p)
        assert np.array_equal(_bits(got.cpu().numpy()), _bits(oracle.top_p_filter(rows, top_p))), (V, top_p)


@pytest.mark.parametrize("V", [7, 1000, 32000, 50257, 128256])
def test_filter_equals_oracle_bit_for_bit(V):
    rows = oracle.softmax(si.normal(5, f"tk{V}", (7, V), 2.0).numpy(), 0.8)
    rows[1] = np.float32(1.0 / V)                       # every weight equal: the cut falls among ties
    rows[2] = 0.0
    rows[2, V // 3] = 1.0                               # one-hot: k > 1 reaches into the tokens without a weight
    rows[3] = 0.0                                       # nothing has a weight: returned unchanged
    rows[4, : V // 2] = rows[4, 0]                      # a block of equal weights among others
    rows[4] /= rows[4].sum()
    rows[5, V // 2:] = 0.0                              # half the row without a weight
    rows[5] /= rows[5].sum()
    rows[6, ::2] = rows[6, 1]                           # ties interleaved with other weights
    g = torch.from_numpy(rows).to(dev())
    for k in sorted({1, 2, 5, min(50, V - 1), V // 2, V // 2 + 1, V - 1}):
        want = oracle.top_k_filter(rows, k)
        got = sv.ss_top_k_filter(g, k)
        assert np.array_equal(_bits(got.cpu().numpy()), _bits(want)), (V, k)
        assert torch.equal(g, torch.from_numpy(rows).to(dev()))                 # the input is not touched
    # in place on the library's own softmax output, then top-p on top of it: the order the loops use
    logits = si.normal(6, f"tkl{V}", (3, V), 2.0)
    p = sv.ss_softmax(logits.to(dev()), 0.7)
    k = min(40, V - 1)
    want = oracle.select(p.cpu().numpy(), top_k=k, top_p=0.8)
    sv.ss_top_k_filter(p, k, p)
    sv.ss_top_p_filter(p, 0.8, p)
    assert np.array_equal(_bits(p.cpu().numpy()), _bits(want))
    # k >= V is the identity, k < 1 is refused
    assert torch.equal(sv.ss_top_k_filter(g, V), g) and torch.equal(sv.ss_top_k_filter(g, V + 5), g)
    with pytest.raises(sv.SpecVerifyError):
        sv.ss_top_k_filter(g, 0)


def test_gpu_filtered_rejection_step_emits_the_filtered_target():
    """On the kernels themselves: 2^18 sequences share one pair of rows over 12 tokens, both filtered to their 5 most
    probable tokens by the library; each sequence draws d ~ q', runs the rejection step and emits a token.  The
    histogram must be the filtered target p' (chi-square over its 5 tokens, p-value > 1e-4; the unfiltered target is
    rejected) and no token outside p' may appear."""
    from scipy import stats
    B, V, k, D = 1 << 18, 12, 5, dev()
    g = torch.Generator().manual_seed(78)
    p1 = torch.softmax(torch.randn(V, generator=g), 0)
    q1 = torch.softmax(torch.randn(V, generator=g) * 1.5, 0)
    pf = sv.ss_top_k_filter(p1.to(D)[None], k)[0]
    qf = sv.ss_top_k_filter(q1.to(D)[None], k)[0]
    assert int((pf > 0).sum()) == k and int((qf > 0).sum()) == k and bool(((pf > 0) != (qf > 0)).any())
    p = pf.repeat(B, 1, 1).repeat(1, 2, 1).contiguous()
    q = qf.repeat(B, 1, 1).contiguous()
    ud = si.uniforms(78, "chi_ud", (B, 1), device=D)
    ua = si.uniforms(78, "chi_ua", (B, 2), device=D)
    zf, zi = torch.zeros(1, device=D), torch.zeros(1, dtype=torch.int32, device=D)
    _, d = sv.ss_speculative_accept(q, zf, zi, ud)
    na, nx = sv.ss_speculative_accept(p, q, d[:, None].contiguous(), ua)
    emitted = torch.where(na == 1, d, nx).cpu().numpy()
    counts = np.bincount(emitted, minlength=V).astype(np.float64)
    pe = pf.double().cpu().numpy()
    keep = pe > 0
    assert counts[~keep].sum() == 0
    pk = pe[keep] / pe.sum()
    chi = ((counts[keep] - B * pk) ** 2 / (B * pk)).sum()
    assert stats.chi2.sf(chi, k - 1) > 1e-4
    pu = p1.double().numpy()
    assert stats.chi2.sf(((counts - B * pu) ** 2 / (B * pu)).sum(), V - 1) < 1e-12


def _pair(seed):
    tw = si.decoder_weights(si.TINY_TARGET, seed)
    dshape, dw = si.early_exit_draft(si.TINY_TARGET, tw, 1)
    gt = sv.Model(si.TINY_TARGET, weights_to_device(tw), max_rows=16, max_pos=256)
    gd = sv.Model(dshape, weights_to_device(dw), max_rows=16, max_pos=256)
    return gt, gd, tw, dshape, dw


def test_draft_step_samples_from_the_filtered_row():
    gt = _pair(2)[0]
    V = si.TINY_TARGET.vocab
    prompt = si.token_ids(2, "prompt", (10,), V)
    kv = sv.KVCache(gt, 1, 64)
    gen.prefill(gt, kv, prompt[:-1].tolist())
    feed = prompt[-1:].to(torch.int32).to(dev())[None]
    u = si.uniforms(2, "u", (1,)).to(dev())
    q = torch.empty(V, dtype=torch.float32, device=dev())
    tok = torch.empty(1, dtype=torch.int32, device=dev())
    sv.ss_draft_step(gt, kv, feed, 1, 1.0, u, q, V, tok)
    plain = q.cpu().numpy().copy()
    for top_k, top_p in ((7, 1.0), (7, 0.5), (V, 1.0)):
        sv.ss_kv_cache_set_len(kv, [9])
        sv.ss_draft_step(gt, kv, feed, 1, 1.0, u, q, V, tok, top_p=top_p, top_k=top_k)
        want = oracle.select(plain, top_k=top_k if top_k < V else 0, top_p=top_p)
        assert np.array_equal(_bits(q.cpu().numpy()), _bits(want)), (top_k, top_p)
        assert int(tok[0]) == oracle.sample(want, float(u[0])) and want[int(tok[0])] > 0
    with pytest.raises(sv.SpecVerifyError):
        sv.ss_draft_step(gt, kv, feed, 1, 1.0, u, q, V, tok, top_k=-1)


@pytest.mark.parametrize("K,top_k,top_p", [(3, 6, 1.0), (5, 20, 0.9)])
def test_speculative_loop_with_top_k(K, top_k, top_p):
    gt, gd, tw, dshape, dw = _pair(3)
    V = si.TINY_TARGET.vocab
    prompt = si.token_ids(3, "prompt", (20,), V).numpy().tolist()
    n_new = 40
    ud, ua = si.uniforms(3, "ud", (n_new, K)).numpy(), si.uniforms(3, "ua", (n_new, K + 1)).numpy()
    seen = []
    one, st1 = gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua, top_p=top_p, top_k=top_k)
    calls, st0 = gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua, top_p=top_p, top_k=top_k,
                                          observer=lambda s: seen.append({k: (v.detach().cpu().numpy().copy() if hasattr(v, "detach") else v) for k, v in s.items()}))
    assert one == calls and st1["accepted"] == st0["accepted"]                               # one call per step = call by call
    assert one != gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua, top_p=top_p)[0]   # the filter is not ignored
    for s in seen:
        assert np.count_nonzero(s["p"][0, 0]) <= top_k and np.count_nonzero(s["q"][0, 0]) <= top_k
        ona, onx = oracle.speculative_accept(s["p"], s["q"], s["draft"], ua[s["step"]][None])
        assert ona.tolist() == s["n_accepted"].tolist() and onx.tolist() == s["next"].tolist()
        assert s["p"][0, int(ona[0]), int(onx[0])] > 0                                       # the emitted token is one of the target's kept tokens
    # identical models: everything accepted; the stream is autoregressive sampling under the same rules
    steps = n_new // (K + 1)
    same, st = gen.speculative_generate(gt, gt, prompt, steps * (K + 1), K, 1.0, ud, ua, top_p=top_p, top_k=top_k)
    assert all(a == K for a in st["accepted"])
    u_ar = np.concatenate([np.concatenate([ud[s], ua[s, K:]]) for s in range(steps)])
    assert same == gen.autoregressive_generate(gt, prompt, steps * (K + 1), 1.0, u_ar, top_p=top_p, top_k=top_k)
    # top_k = 1 is greedy decoding, whatever the draft proposes
    greedy = gen.autoregressive_generate(gt, prompt, 24, 0.0)
    assert gen.speculative_generate(gt, gd, prompt, 24, K, 1.0, ud, ua, top_k=1)[0] == greedy
