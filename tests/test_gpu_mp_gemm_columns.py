"""The product of more than 32 rows whose waves take block columns of their own: each of its shapes, whole and with column splits, with row
groups past the matrix's end, fewer block columns than waves, a last wave with fewer than the others, more of them than a wave has lanes,
and tiles of two block rows.  Reference and bounds are those of the edges' test."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_mp_gemm_edges as edges

pytestmark = pytest.mark.gpu
ALL = [1, 2, 3, 4, 5, 6, 7, 8]


@pytest.mark.parametrize("R,C,m,n,bits,batch,pad", [
    # two by two tiles; with column splits
    (256, 256, 64, 128, [0] + ALL, 117, 0),
    (96, 128 * 27, 32, 128, [1, 2, 3, 4], 80, 8),
    (288, 64 * 4, 32, 64, [3, 5, 6], 76, 0),
    (96, 64 * 42, 32, 64, [2, 8], 127, 24),
    # three by two
    (2176, 256, 128, 128, [2, 8], 120, 0),
    (416, 128 * 34, 32, 128, [0] + ALL, 125, 0),
    (2976, 256, 32, 64, [2, 4, 8], 90, 0),
    (384, 64 * 50, 64, 64, ALL, 80, 0),
    # three by four, 256 threads
    (2848, 256, 32, 128, [1, 2, 3, 4, 8], 110, 0),
    (2848, 64 * 4, 32, 64, ALL, 102, 0),
    (4672, 64 * 82, 64, 64, [2, 4, 8], 95, 0),
    # four by four, 256 threads; (the last: three by four) a wave with more block columns than lanes
    (5888, 256, 128, 128, [1, 2, 3, 4], 101, 0),
    (13312, 256, 256, 64, [0, 1, 2, 3, 4], 109, 0),
    (8640, 64 * 258, 32, 64, [2, 8], 128, 0),
    # four by four, 512 threads
    (4256, 128 * 5, 32, 128, [3, 5, 6], 118, 0),
    (1152, 128 * 83, 128, 128, [3, 5, 6], 100, 8),
    (5920, 64 * 5, 32, 64, ALL, 116, 0),
    (3328, 64 * 48, 256, 64, [2, 4, 8], 106, 0),
    (64, 64 * 512, 64, 64, [4, 7], 128, 0),               # the widest row
])
def test_product_by_columns(orc, R, C, m, n, bits, batch, pad):
    edges.test_product_edges(orc, R, C, m, n, bits, batch, pad)
