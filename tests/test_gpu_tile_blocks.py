"""The tile GEMM in blocks of 96 rows, gate and up in 128 columns, and column shares and row blocks that do not fill whole rounds of the eight XCDs."""
import ctypes

import pytest
import torch

import paper_2311_04951_amd as sv
from test_gpu_tile_gemm import test_one_layer_against_64_bits as _layer_against_64_bits

# two and three row blocks, the last one full or nearly empty; K split and not; d_ff that ends inside a tile and, as K, inside a stage
LAYERS = [(161, 1536, 12, 4104), (192, 4096, 32, 1032), (192, 136, 8, 344), (185, 1096, 16, 1736), (257, 4096, 32, 1032), (288, 136, 40, 11008), (270, 2056, 16, 13824)]
# gate and up of more than 256 shares of 96 columns and at most 256 of 128: the fewest and the most, K that ends inside a stage
WIDE = [(17, 1040, 8, 12304), (32, 1096, 8, 16384), (33, 1040, 8, 13824), (48, 136, 8, 12312), (49, 1096, 8, 16376), (80, 1040, 8, 13824)]
STORE, RESID, SWIGLU, QKV = range(4)


def _tiles():
    L = sv.lib()
    L.ss_dev_gemm_tile.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    met, ragged = set(), set()
    for R, d, heads, ff in LAYERS:
        W = 128 * heads
        for epi, N, K in ((QKV, 3 * W, d), (RESID, d, W), (SWIGLU, ff, d), (RESID, d, ff)):
            out = (ctypes.c_int * 3)()
            L.ss_dev_gemm_tile(epi, R, N, K, 4 * max(3 * W, 2 * ff, d) * ((R + 15) // 16) * 64, out)
            rows, cols, splits = out
            met.add((epi, rows, cols))
            columns = 32 * ((ff + 15) // 16) if epi == SWIGLU else (N + 15) // 16 * 16
            ragged.add((-(-columns // cols) % 8 != 0, -(-R // rows)))
    return met, ragged


def test_the_shapes_below_meet_every_tile_of_96_rows():
    met, ragged = _tiles()
    assert {m for m in met if m[1] == 96} == {(e, 96, c) for e in (QKV, SWIGLU) for c in (96, 192)} | {(RESID, 96, c) for c in (64, 128)}
    assert {(r, n) for r in (False, True) for n in (2, 3)} <= ragged      # column shares that are no multiple of 8, over two and three row blocks


def test_gate_and_up_of_one_round_take_128_columns():
    L = sv.lib()
    L.ss_dev_gemm_tile_bits.argtypes = [ctypes.c_int] * 5 + [ctypes.c_size_t, ctypes.POINTER(ctypes.c_int)]
    out = (ctypes.c_int * 3)()

    def tile(bits, R, F, K):
        L.ss_dev_gemm_tile_bits(bits, SWIGLU, R, F, K, 0, out)
        return out[0], out[1]

    for bits in (16, 8, 4):
        for R, d, _, ff in WIDE:
            assert tile(bits, R, ff, d) == (32 if R <= 32 else 48 if R <= 48 else 80, 128)
        for R, F in ((40, 12288), (40, 16400), (81, 13824), (160, 8192)):     # one round of 96 columns; two of 128; more than one row block
            assert tile(bits, R, F, 4096)[1] != 128


@pytest.mark.gpu
@pytest.mark.parametrize("R,d,heads,ff", LAYERS + WIDE)
def test_one_layer_of_these_blocks_against_64_bits(R, d, heads, ff):
    """The bound of the shapes with other tiles: 16 bits of the activations, sums in 32."""
    _layer_against_64_bits(R, d, heads, ff)


@pytest.mark.gpu
@pytest.mark.parametrize("V", [333, 32000])
def test_a_head_of_96_row_blocks_against_64_bits(V):
    from test_gpu_tile_gemm import test_a_head_against_64_bits
    test_a_head_against_64_bits(180, V, 72)
