"""No-GPU check: the shapes of test_gpu_tile_gemm.py meet every tile of the GEMM for more than 16 rows, by the library's own choice."""
import ctypes

import paper_2311_04951_amd as sv
import test_gpu_tile_gemm as shapes

STORE, RESID, SWIGLU, QKV = range(4)


def _tile(epi, R, N, K, ws_bytes):
    L = sv.lib()
    L.ss_dev_gemm_tile.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    L.ss_dev_gemm_tile.restype = None
    out = (ctypes.c_int * 3)()
    L.ss_dev_gemm_tile(epi, R, N, K, ws_bytes, out)
    return tuple(out)


def test_every_tile_is_met():
    met = set()
    for R, d, heads, ff in shapes.LAYERS:
        W = 128 * heads
        ws = 4 * max(3 * W, 2 * ff, d) * ((R + 15) // 16) * 64          # the workspace of a model of R rows
        for epi, N, K in ((QKV, 3 * W, d), (RESID, d, W), (SWIGLU, ff, d), (RESID, d, ff)):
            rows, cols, splits = _tile(epi, R, N, K, ws)
            met.add((epi, rows, cols, splits > 1))
    for R, V, d in shapes.HEADS:
        rows, cols, splits = _tile(STORE, R, V, d, 0)
        met.add((STORE, rows, cols, splits > 1))
    built = {(e, r, c) for e in (QKV, SWIGLU) for r in (32, 48, 80, 128) for c in (64, 96, 192) if (r, c) != (128, 64)}
    built |= {(e, r, c) for e in (STORE, RESID) for r in (32, 48, 80, 128) for c in (64, 128)}
    assert {m[:3] for m in met} == built
    for epi in (QKV, RESID):
        for rows in (32, 48, 80, 128):
            assert {s for e, r, c, s in met if (e, r) == (epi, rows)} == {False, True}, (epi, rows)
    assert not any(s for e, r, c, s in met if e in (STORE, SWIGLU))


def test_many_rows_of_a_short_k_take_small_blocks():
    """1024 rows of models of 128 to 512: a launch of a few stages is bound by its ends; blocks of 128 rows, or K split, where small blocks fill the chip are slower."""
    for d, heads, ff, want in ((128, 2, 384, [(32, 64, 1), (32, 64, 1), (32, 96, 1), (32, 64, 1)]), (256, 4, 768, [(32, 96, 1), (32, 64, 1), (80, 96, 1), (32, 64, 2)]),
                               (512, 8, 1536, [(80, 96, 1), (32, 64, 1), (128, 96, 1)])):
        W = 64 * heads
        ws = 4 * max(3 * W, 2 * ff, d) * 1024
        got = [_tile(epi, 1024, N, K, ws) for epi, N, K in ((QKV, 3 * W, d), (RESID, d, W), (SWIGLU, ff, d), (RESID, d, ff))]
        assert got[:len(want)] == want, d
