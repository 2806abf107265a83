"""The product of more than 32 rows, whose waves take block columns of their own: each of its instances (columns of a block; tiles of batch rows
and of channels, waves of a workgroup; codes of 1 bit as 128 + q or 1 + q / 2), whole and with column splits, in one group of batch rows and in several, with row
groups past the matrix's end, fewer block columns than waves, a last wave with fewer than the others, more of them than a wave has lanes,
blocks of 1 bit, and tiles of two block rows.  Reference and bounds are those of the edges' test."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_mp_gemm_edges as edges

pytestmark = pytest.mark.gpu
ALL = [1, 2, 3, 4, 5, 6, 7, 8]

CASES = {
    "many 128,2,2,8,0": [
        (256, 256, 64, 128, [0] + ALL, 117, 0),
        (96, 128 * 27, 32, 128, [1, 2, 3, 4], 80, 8),          # column splits
        (32, 128 * 42, 32, 128, [3, 5, 6], 64, 0),             # and row groups of which one is in the matrix
    ],
    "many 64,2,2,8,0": [
        (288, 64 * 4, 32, 64, [3, 5, 6], 76, 0),
        (96, 64 * 42, 32, 64, [2, 8], 127, 24),
        (32, 64 * 126, 32, 64, [0] + ALL, 46, 0),
        (64, 64 * 512, 64, 64, [4, 7], 128, 0),                # the widest row
    ],
    "many 128,3,2,8,0": [
        (2176, 256, 128, 128, [2, 8], 120, 0),
        (416, 128 * 34, 32, 128, [0] + ALL, 125, 0),
        (5504, 128, 64, 128, [2, 8], 46, 0),                   # one group of rows
    ],
    "many 64,3,2,8,0": [
        (2976, 256, 32, 64, [2, 4, 8], 90, 0),
        (384, 64 * 50, 64, 64, ALL, 80, 0),
        (7296, 64 * 6, 32, 64, [1, 4, 8], 49, 0),
    ],
    "many 128,3,4,4,0": [
        (2848, 256, 32, 128, [1, 2, 3, 4, 8], 110, 0),
        (4160, 128, 64, 128, [3, 5, 6], 51, 8),
    ],
    "many 64,3,4,4,0": [
        (2848, 64 * 4, 32, 64, ALL, 102, 0),
        (4672, 64 * 82, 64, 64, [2, 4, 8], 95, 0),
        (8640, 64 * 258, 32, 64, [2, 8], 128, 0),              # a wave with more block columns than lanes
        (12672, 64, 64, 64, [0] + ALL, 60, 0),
    ],
    "many 128,4,4,4,0": [
        (5888, 256, 128, 128, [1, 2, 3, 4], 101, 0),
        (16480, 128, 32, 128, [1, 4, 8], 54, 0),
    ],
    "many 64,4,4,4,0": [
        (13312, 256, 256, 64, [0, 1, 2, 3, 4], 109, 0),
        (16768, 64, 128, 64, [1, 4, 8], 50, 8),
    ],
    "many 128,4,4,8,0": [
        (4256, 128 * 5, 32, 128, [3, 5, 6], 118, 0),
        (1152, 128 * 83, 128, 128, [3, 5, 6], 100, 8),
        (4672, 128 * 6, 64, 128, [1, 4, 8], 98, 0),
        (8640, 128 * 5, 64, 128, [0] + ALL, 54, 0),
    ],
    "many 64,4,4,8,0": [
        (5920, 64 * 5, 32, 64, ALL, 116, 0),
        (3328, 64 * 48, 256, 64, [2, 4, 8], 106, 0),
        (8320, 64 * 5, 64, 64, [1, 2, 3, 4], 52, 0),
    ],
    "many 128,2,2,8,1": [(32, 128 * 40, 32, 128, [0, 1], 39, 8)],
    "many 128,3,2,8,1": [(5504, 128, 128, 128, [0, 1], 43, 0)],
    "many 128,3,4,4,1": [(4224, 128, 128, 128, [1, 4, 8], 55, 0)],
    "many 128,4,4,4,1": [(8224, 128, 32, 128, [0, 1], 59, 0)],
    "many 128,4,4,8,1": [(9152, 128 * 5, 32, 128, [0, 1], 59, 0)],
    "many 64,2,2,8,1": [(32, 64 * 60, 32, 64, [1], 45, 0)],
    "many 64,3,2,8,1": [(5472, 64, 32, 64, [1, 4, 8], 33, 0)],
    "many 64,3,4,4,1": [(4160, 64, 64, 64, [1, 4, 8], 50, 0)],
    "many 64,4,4,4,1": [(17696, 64 * 9, 32, 64, [0, 1], 50, 0)],
    "many 64,4,4,8,1": [(8384, 64 * 9, 64, 64, [1], 59, 0)],
}


@pytest.mark.parametrize("R,C,m,n,bits,batch,pad,one_bit", [case + (128 if name.endswith(",0") else 2,) for name, cases in CASES.items() for case in cases])
def test_product_by_columns(orc, R, C, m, n, bits, batch, pad, one_bit):
    edges.test_product_edges(orc, R, C, m, n, bits, batch, pad, one_bit)
