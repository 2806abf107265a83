"""Offsets by the single launch and by three, at the edges of the tiles and of the line between them, for levels of every
candidate (nine of them: the one that the permuted table does not hold) and level arrays that start anywhere."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 15, 8191, 8192, 8193, 16384 + 24, 131072, 196608 - 8, 196608, 196608 + 8, 524288 - 8, 524288, 524288 + 8])
@pytest.mark.parametrize("bits", [[3], [1, 2, 4, 8], [0, 1, 2, 3, 4, 5, 6, 7, 8]])
def test_offsets(N, bits):
    print("[case] offsets", N, bits, flush=True)
    dev = torch.device("cuda:0")
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    rows = next(r for r in range(1, N + 1) if N % r == 0 and N // r <= 4096)
    mats = (rows + 4095) // 4096
    while rows % mats:
        mats += 1
    plan = sb.Plan(ctx, [(rows // mats * 8, N // rows * 8)] * mats, 8, 8, bits)
    assert plan.num_blocks() == N
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    lv = np.random.default_rng(N).integers(0, len(bits), N).astype(np.uint8)
    want = np.concatenate([[0], np.cumsum(8 * np.asarray(bits, np.int64)[lv])])
    for shift in (0, 1, 7):
        buf = torch.zeros(N + 8, dtype=torch.uint8, device=dev)
        level = buf[shift:shift + N]
        level.copy_(torch.from_numpy(lv))
        off = torch.full((N + 3,), -1, dtype=torch.int64, device=dev)
        plan.offsets(level, off, ws)
        np.testing.assert_array_equal(off[:N + 1].cpu().numpy(), want)
        assert off[N + 1:].tolist() == [-1, -1]
    plan.close()
    ctx.close()
