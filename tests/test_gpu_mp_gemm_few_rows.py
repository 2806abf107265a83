"""The kernels for few rows at the edges of their choices: 16 and 8 waves a workgroup (one turn of the chip), x straight from
memory (up to 4 rows) and by way of LDS, one to four groups of 16 rows with a ragged last one, 32, 64 and 128 channels a
workgroup of the kernel with column splits, a pitch, pruned blocks, every bitwidth.  Bound as for the other products: terms of size
|B| scale |x| and |zero| |x| in fp32, where the codes' offset is 128 (up to 32 rows) or 2^c (more rows, bitwidths up to 5):
2^-22 of their sum for the largest error, 2^-24 for the root mean square."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu

ALL = [1, 2, 3, 4, 5, 6, 7, 8]


@pytest.mark.parametrize("R,C,m,n,bits,batch,pad", [
    (8192, 128 * 17, 128, 128, ALL, 4, 0),                # 256 workgroups: 16 waves, x from memory
    (8192, 128 * 17, 128, 128, [1, 2, 4, 7], 5, 8),       # by way of LDS
    (8224, 128 * 17, 32, 128, [2, 5], 4, 8),              # 257: 8 waves
    (8224, 128 * 17, 32, 128, [0] + ALL, 5, 0),
    (8224, 64 * 20, 32, 64, ALL, 4, 0),
    (8224, 64 * 20, 32, 64, [0] + ALL, 13, 24),
    (64, 128 * 17, 32, 128, [0] + ALL, 9, 0),
    (64, 128 * 24, 32, 128, ALL, 16, 0),
    (64, 128 * 33, 32, 128, ALL, 15, 0),
    (96, 64 * 25, 32, 64, [0] + ALL, 16, 0),
    (96, 64 * 25, 32, 64, ALL, 3, 8),
    (32, 64 * 512, 32, 64, [1, 3], 16, 0),                # the widest row: 64 blocks a wave
    (96, 64 * 7, 32, 64, ALL, 17, 8),                     # a second group of one row
    (64, 128 * 9, 32, 128, [0] + ALL, 31, 0),
    (64, 128 * 28, 64, 128, [1, 4, 6], 32, 0),
    (64, 128 * 5, 32, 128, ALL, 33, 8),                   # three groups: more than 32 rows
    (96, 64 * 40, 32, 64, [0] + ALL, 47, 0),
    (64, 64 * 3, 64, 64, [1, 2, 4], 64, 0),
    (4128, 128 * 4, 32, 128, ALL, 33, 0),                 # three groups, two turns
    (4128, 64 * 5, 32, 64, ALL, 48, 8),
    (16416, 128 * 3, 32, 128, [3, 8], 16, 0),             # 513 workgroups of 32 channels: 64 each
    (4128, 128 * 65, 32, 128, [1, 2], 16, 0),             # column splits, ragged last workgroup
    (8192, 128 * 10, 64, 128, ALL, 32, 0),                # two groups, two turns
    (16448, 128 * 6, 64, 128, [2, 7], 29, 8),             # 257 of 64 channels: 128 each
    (3072, 128 * 60, 64, 128, [2, 4], 30, 0),             # 64
    (4128, 64 * 40, 32, 64, ALL, 20, 0),                  # 32 and 64 channels of 64-column blocks, splits
    (1024, 64 * 100, 32, 64, [0, 3, 5], 25, 8),
    (13344, 64 * 20, 32, 64, [2, 8], 12, 0),
])
def test_product_of_few_rows(orc, R, C, m, n, bits, batch, pad):
    print("[case] product of few rows", R, C, m, n, bits, batch, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(R + C + batch)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(R, C)], m, n, bits)
    N = plan.num_blocks()
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    level = rng.integers(0, len(bits), N).astype(np.uint8)
    off = orc.offsets(level, m, n, bits)
    codes = np.zeros(max(int(off[-1]), 16), np.uint8)
    scale, zero = np.zeros(N * m, np.float32), np.zeros(N * m, np.float32)
    W = orc.f32_to_bf16(0.02 * rng.standard_normal((R, C)))
    orc.pack(W, m, n, bits, level, off, 0, codes, scale, zero)
    xb = orc.f32_to_bf16(rng.standard_normal((batch, C)))
    x = torch.full((batch, C + pad), float("nan"), dtype=torch.bfloat16, device=dev)   # what lies past the columns is not read
    x[:, :C] = torch.from_numpy(xb.view(np.int16)).view(torch.bfloat16)
    args = [torch.from_numpy(t).to(dev) for t in (level, off, codes, scale, zero)]
    y = torch.full((batch + 1, R), -7.0, device=dev)
    plan.mp_gemm(0, x[:, :C], *args, y, ws)
    torch.cuda.synchronize()
    assert torch.all(y[batch] == -7.0)
    What = torch.from_numpy(orc.dequant(codes, scale, zero, level, off, 0, R, C, m, n, bits)).double()
    xf = torch.from_numpy(orc.bf16_to_f32(xb)).double()
    ref = (xf @ What.T).numpy()
    nbc = C // n
    offset = {1: 128, 6: 128, 7: 128} if batch > 32 else {b: 128 for b in range(1, 8)}
    most = np.array([2.0 ** b + offset.get(b, 2.0 ** b) for b in bits])      # of |B|, in codes
    mag = np.abs(zero.reshape(N, m)) + scale.reshape(N, m) * most[level][:, None]
    mag = mag.reshape(R // m, nbc, m).transpose(0, 2, 1).reshape(R, nbc)
    bound = np.abs(xf.numpy()).reshape(batch, nbc, n).sum(2) @ mag.T
    err = np.abs(y[:batch].cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= bound * 2.0 ** -22 + 1e-30), float((err / (bound + 1e-300)).max())
    assert np.sqrt((err ** 2).mean()) <= 2.0 ** -24 * np.sqrt((bound ** 2).mean())
    plan.close()
    ctx.close()
