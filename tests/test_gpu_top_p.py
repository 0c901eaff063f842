"""Top-p selection on the GPU path (Section 3 names it beside argmax): the filter against the oracle bit for
bit (same kept set, same renormalised values), and the loops that use it."""
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


@pytest.mark.parametrize("V", [7, 1000, 32000, 50257])
def test_filter_equals_oracle_bit_for_bit(V):
    rows = oracle.softmax(si.normal(5, f"tp{V}", (6, V), 2.0).numpy(), 0.8)
    rows[1] = np.float32(1.0 / V)                       # every weight equal: the boundary falls among ties
    rows[2] = 0.0
    rows[2, V // 3] = 1.0                               # one-hot
    rows[3] = 0.0                                       # nothing has a weight: returned unchanged
    rows[4, : V // 2] = rows[4, 0]                      # a block of equal weights among others
    rows[4] /= rows[4].sum()
    g = torch.from_numpy(rows).to(dev())
    for top_p in (1e-6, 0.1, 0.5, 0.9, 0.999, 0.9999999):
        want = oracle.top_p_filter(rows, top_p)
        got = sv.ss_top_p_filter(g, top_p)
        assert np.array_equal(_bits(got.cpu().numpy()), _bits(want)), (V, top_p)
        assert torch.equal(g, torch.from_numpy(rows).to(dev()))                 # the input is not touched
    # in place, and on the library's own softmax output
    logits = si.normal(6, f"tl{V}", (3, V), 2.0)
    p = sv.ss_softmax(logits.to(dev()), 0.7)
    want = oracle.top_p_filter(p.cpu().numpy(), 0.8)
    sv.ss_top_p_filter(p, 0.8, p)
    assert np.array_equal(_bits(p.cpu().numpy()), _bits(want))
    # top_p >= 1 is the identity, top_p <= 0 is refused
    assert torch.equal(sv.ss_top_p_filter(g, 1.0), g)
    with pytest.raises(sv.SpecVerifyError):
        sv.ss_top_p_filter(g, 0.0)


def _pair(seed):
    tw = si.decoder_weights(si.TINY_TARGET, seed)
    dshape, dw = si.early_exit_draft(si.TINY_TARGET, tw, 1)
    gt = sv.Model(si.TINY_TARGET, weights_to_device(tw), max_rows=16, max_pos=256)
    gd = sv.Model(dshape, weights_to_device(dw), max_rows=16, max_pos=256)
    return gt, gd


def test_draft_step_samples_from_the_filtered_row():
    gt, _ = _pair(2)
    V = si.TINY_TARGET.vocab
    prompt = si.token_ids(2, "prompt", (10,), V)
    kv = sv.KVCache(gt, 1, 64)
    gen.prefill(gt, kv, prompt[:-1].tolist())
    feed = prompt[-1:].to(torch.int32).to(dev())[None]
    u = si.uniforms(2, "u", (1,)).to(dev())
    q = torch.empty(V, dtype=torch.float32, device=dev())
    tok = torch.empty(1, dtype=torch.int32, device=dev())
    # the unfiltered row first (same cache state: roll the appended row back)
    sv.ss_draft_step(gt, kv, feed, 1, 1.0, u, q, V, tok)
    plain = q.cpu().numpy().copy()
    sv.ss_kv_cache_set_len(kv, [9])
    sv.ss_draft_step(gt, kv, feed, 1, 1.0, u, q, V, tok, top_p=0.5)
    want = oracle.top_p_filter(plain, 0.5)
    assert np.array_equal(_bits(q.cpu().numpy()), _bits(want))
    assert int(tok[0]) == oracle.sample(want, float(u[0])) and want[int(tok[0])] > 0


@pytest.mark.parametrize("K,top_p", [(3, 0.6), (5, 0.9)])
def test_speculative_loop_with_top_p(K, top_p):
    gt, gd = _pair(3)
    V = si.TINY_TARGET.vocab
    prompt = si.token_ids(3, "prompt", (20,), V).numpy().tolist()
    n_new = 40
    ud, ua = si.uniforms(3, "ud", (n_new, K)).numpy(), si.uniforms(3, "ua", (n_new, K + 1)).numpy()
    seen = []
    one, st1 = gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua, top_p=top_p)
    calls, st0 = gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua, top_p=top_p,
                                          observer=lambda s: seen.append({k: (v.detach().cpu().numpy().copy() if hasattr(v, "detach") else v) for k, v in s.items()}))
    assert one == calls and st1["accepted"] == st0["accepted"]
    assert one != gen.speculative_generate(gt, gd, prompt, n_new, K, 1.0, ud, ua)[0]          # the filter is not ignored
    for s in seen:
        # the rows the rejection step saw are filtered rows (fixed points of the filter's kept set), and the
        # step's decisions are the oracle's on those rows
        assert np.count_nonzero(s["p"][0, 0]) < V and np.count_nonzero(s["q"][0, 0]) < V
        ona, onx = oracle.speculative_accept(s["p"], s["q"], s["draft"], ua[s["step"]][None])
        assert ona.tolist() == s["n_accepted"].tolist() and onx.tolist() == s["next"].tolist()
        assert s["p"][0, int(ona[0]), int(onx[0])] > 0                                       # the emitted token lies in the target's nucleus
    # identical models: everything accepted; the stream is autoregressive top-p sampling with the interleaved uniforms
    steps = n_new // (K + 1)
    same, st = gen.speculative_generate(gt, gt, prompt, steps * (K + 1), K, 1.0, ud, ua, top_p=top_p)
    assert all(a == K for a in st["accepted"])
    u_ar = np.concatenate([np.concatenate([ud[s], ua[s, K:]]) for s in range(steps)])
    assert same == gen.autoregressive_generate(gt, prompt, steps * (K + 1), 1.0, u_ar, top_p=top_p)


@pytest.mark.parametrize("V", [1, 2, 32768, 32769, 70001])      # the longest row that stays on chip, and longer ones
def test_both_filters_where_the_route_changes_equal_oracle_bit_for_bit(V):
    """Rows that fit the on-chip copy and rows that don't, aligned and not (a leading dimension of V on an odd offset), with the
    boundary among a few tokens, among more than are ranked one by one, and among more than the list of candidates holds; with
    weights of 2^32 (probability 1 and more), of zero, and values that are no probabilities."""
    rows = oracle.softmax(si.normal(8, f"r{V}", (6, V), 2.0).numpy(), 1.0)
    rows[1] = np.float32(1.0 / V)                                                # all in one bin, equal
    rows[2] = (1.0 + np.arange(V, dtype=np.float32) / (64.0 * V)) / V            # all in one or two bins, different
    rows[3, V // 2:] = 0.0                                                       # half without a weight
    rows[4, 0] = 1.0
    rows[4, V // 2] = 3.0                                                        # more than 1
    rows[5] = -rows[5]
    rows[5, V - 1] = 0.25
    arena = torch.zeros(6 * V + 8, device=dev())
    for at in (0, 1):
        g = arena[at:at + 6 * V].view(6, V)
        g.copy_(torch.from_numpy(rows))
        out = torch.empty_like(arena)[at:at + 6 * V].view(6, V)
        for top_p in (0.003, 0.5, 0.97):
            assert np.array_equal(_bits(sv.ss_top_p_filter(g, top_p, out).cpu().numpy()), _bits(oracle.top_p_filter(rows, top_p))), (V, top_p, at)
        for k in sorted({1, max(1, V // 100), max(1, (2 * V) // 3), max(1, V - 1)} - {V}):
            assert np.array_equal(_bits(sv.ss_top_k_filter(g, k, out).cpu().numpy()), _bits(oracle.top_k_filter(rows, k))), (V, k, at)


@pytest.mark.parametrize("V", [1, 5, 4096, 32770])
def test_negative_zeros_have_no_weight(V):
    """-0.0 among the entries (what a masked product leaves): no weight, whatever a maximum of -0 and +0 is."""
    rows = oracle.softmax(si.normal(9, f"z{V}", (3, V), 2.0).numpy(), 1.0)
    rows[0, ::3] = -0.0
    rows[1, : V // 2 + 1] = -0.0
    rows[2] = -0.0                                                               # nothing has a weight: returned unchanged
    g = torch.from_numpy(rows).to(dev())
    for top_p in (0.01, 0.5, 0.99):
        assert np.array_equal(_bits(sv.ss_top_p_filter(g, top_p).cpu().numpy()), _bits(oracle.top_p_filter(rows, top_p))), (V, top_p)
    for k in sorted({1, V // 2, V - 1} - {0, V}):                                # (beyond half of V: into the tokens without a weight)
        assert np.array_equal(_bits(sv.ss_top_k_filter(g, k).cpu().numpy()), _bits(oracle.top_k_filter(rows, k))), (V, k)


@pytest.mark.parametrize("V", [127, 1025, 4097, 32767, 36865])
def test_crowded_bins_and_unaligned_rows_equal_oracle_bit_for_bit(V):
    """Bins that hold a few tokens, some hundred (the bounds of what is ranked and listed) and most of the row, alone and between other
    tokens, in rows whose entries are read word by word: equal weights, weights within one bin, every second entry equal, a flat tail."""
    n = si.normal(11, f"c{V}", (9, V), 1.0).numpy()
    n[0] *= 0.001                                                        # all within one bin or two
    n[1] *= 0.01
    n[2, ::2] = n[2, 0]
    n[3, V // 8:] = -3.0
    n[4] *= 4.0
    for r, top in ((5, 192), (6, 193), (7, 2048), (8, 2049)):            # as many tokens in the top bin
        n[r, :top] = 9.0 + 1e-4 * n[r, :top]
    rows = oracle.softmax(n, 1.0)
    g = torch.from_numpy(rows).to(dev())
    for top_p in (0.02, 0.5, 0.95):
        assert np.array_equal(_bits(sv.ss_top_p_filter(g, top_p).cpu().numpy()), _bits(oracle.top_p_filter(rows, top_p))), (V, top_p)
    for k in sorted({1, 64, 100, 192, 193, V // 2, V - 2} - {V}):
        if k < V:
            assert np.array_equal(_bits(sv.ss_top_k_filter(g, k).cpu().numpy()), _bits(oracle.top_k_filter(rows, k))), (V, k)


@pytest.mark.parametrize("V", [32000, 128256])
def test_rows_of_equal_weights_take_no_multiple_of_the_time_of_others(V):
    """Equal weights meet in one bin: were every entry an atomic addition of its own, the row would take seven to eleven times as long
    as one of a softmax; with the additions of a wavefront put together it takes about three."""
    def us(x, f):
        out = torch.empty_like(x)
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                f(x, out)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    usual = torch.softmax(2 * si.normal(10, f"u{V}", (1, V), 1.0).to(dev()), -1)
    flat = torch.full_like(usual, 1.0 / V)
    mixed = torch.where(torch.arange(V, device=dev()) % 2 == 0, flat, usual)     # ... and where they lie between others
    for f in (lambda x, o: sv.ss_top_k_filter(x, 200, o), lambda x, o: sv.ss_top_p_filter(x, 0.9, o)):
        times = [us(x, f) for x in (usual, flat, mixed)]
        assert max(times) < 4.5 * times[0], times


@pytest.mark.parametrize("V", [8192, 8193, 18432, 18433, 32000, 32768, 32771, 50260])
def test_rows_with_few_candidates_equal_oracle_bit_for_bit(V):
    """Rows whose kept tokens are looked for among candidates (top-p from 8193 entries on, top-k from 18433): as many tokens with a weight as the candidates' list
    holds, one fewer and one more, few and none; the heaviest token in the row's last entries; ties at the boundary; more tokens above the
    bound than the list holds (all in the first units of a few threads); aligned rows and others, in place and not."""
    n = si.normal(12, f"f{V}", (8, V), 2.0).numpy()
    rows = oracle.softmax(n, 1.0)
    for r, nnz in enumerate((1535, 1536, 1537, 60)):
        rows[r, np.argsort(rows[r])[: V - nnz]] = 0.0
    rows[4, V - 3:] = (0.3, 0.2, 0.1)
    rows[5, np.argsort(rows[5])[-200:-20]] = rows[5].max() / 2          # 180 ties below the twenty heaviest
    rows[6] = 2.0 ** -33                                                # nothing has a weight but one token
    rows[6, V // 2] = 0.5
    rows[7].reshape(-1)[: V // 4096 * 4096].reshape(-1, 4096)[:, :1600] += 0.01
    arena = torch.zeros(8 * V + 8, device=dev())
    for at in (0, 1):
        g = arena[at:at + 8 * V].view(8, V)
        for k in (1, 30, 100, 511, 512, 513, 1536, 1537):
            want = oracle.top_k_filter(rows, k)
            g.copy_(torch.from_numpy(rows))
            assert np.array_equal(_bits(sv.ss_top_k_filter(g, k, torch.empty_like(arena)[at:at + 8 * V].view(8, V)).cpu().numpy()), _bits(want)), (V, k, at)
            assert np.array_equal(_bits(sv.ss_top_k_filter(g, k, g).cpu().numpy()), _bits(want)), (V, k, at)
        for top_p in (0.01, 0.7, 0.999):
            want = oracle.top_p_filter(rows, top_p)
            g.copy_(torch.from_numpy(rows))
            assert np.array_equal(_bits(sv.ss_top_p_filter(g, top_p, torch.empty_like(arena)[at:at + 8 * V].view(8, V)).cpu().numpy()), _bits(want)), (V, top_p, at)
            assert np.array_equal(_bits(sv.ss_top_p_filter(g, top_p, g).cpu().numpy()), _bits(want)), (V, top_p, at)
