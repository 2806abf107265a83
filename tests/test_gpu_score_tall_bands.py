"""Channel scores of plans large enough for bands of 512 rows, bit for bit against the oracle: rows that end inside a band and inside an octet
run of it, matrices of one band, columns that end inside a segment and inside a panel, and next to them plans just too small."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_score_bands as bands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [
    [(4104, 8)] * 52,                                       # 468 workgroups of 512 rows (884 of 256: two turns)
    [(4608, 24)] * 50 + [(520, 4104), (8, 4096)],           # whole bands, and matrices that are less than one
    [(1000, 520)] * 256,                                    # 512 workgroups
    [(4104, 8)] * 44,                                       # 396: too few
    [(4104, 8)] * 60,                                       # 540: two turns, as 1020 of 256 rows take
])
def test_score_tall_bands(orc, shapes):
    bands.test_score_bands(orc, shapes)
