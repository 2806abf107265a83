"""Blocks of 1 bit, whose codes enter as 128 + q in the kernels of up to 32 rows and as that or, in some products of 33 to 64 rows, as 1 + q / 2 in
those of more (`narrow`: the sizes of these, which the narrow kernel takes or that of many rows).  Bound of a result: terms of size |B| scale |x| and |zero| |x| in fp32, with |B| up to 129 or, in units of
scale, 4; 2^-22 of their sum for the largest error.  What a row of x gives in products of 32 and of more rows then differs by the sum of both bounds at
most."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C,m,n,narrow", [(64, 128 * 5, 32, 128, (33, 47, 48, 64)), (2048, 1024, 32, 128, (33, 47, 48, 64)), (96, 64 * 40, 32, 64, (33, 47, 48, 64)),
                                            (4096, 4096, 64, 128, (33, 48, 64)), (8192, 64 * 32, 128, 64, (33, 48))])
@pytest.mark.parametrize("bits", [[1], [0, 1, 4]])
def test_one_bit_blocks_at_every_size_of_a_launch(orc, R, C, m, n, narrow, bits):
    print("[case] one bit", R, C, n, bits, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(R + C)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(R, C)], m, n, bits)
    N, nbc, most_rows = plan.num_blocks(), C // n, 97
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    level = rng.integers(0, len(bits), N).astype(np.uint8)
    off = orc.offsets(level, m, n, bits)
    codes = np.zeros(max(int(off[-1]), 16), np.uint8)
    scale, zero = np.zeros(N * m, np.float32), np.zeros(N * m, np.float32)
    W = orc.f32_to_bf16(0.02 * rng.standard_t(4, (R, C)))
    orc.pack(W, m, n, bits, level, off, 0, codes, scale, zero)
    x = torch.from_numpy(rng.standard_normal((most_rows, C)).astype(np.float32)).to(torch.bfloat16)
    What = torch.from_numpy(orc.dequant(codes, scale, zero, level, off, 0, R, C, m, n, bits)).to(dev).double()
    xd = x.to(dev)
    ref = xd.double() @ What.t().contiguous()
    sums = xd.double().abs().view(most_rows, nbc, n).sum(2)
    args = [torch.from_numpy(t).to(dev) for t in (level, off, codes, scale, zero)]

    def bound(offset):
        most = np.array([0 if b == 0 else 2 ** b + (offset if b == 1 else 128) for b in bits], np.float64)
        mag = np.abs(zero.reshape(N, m)) + scale.reshape(N, m) * most[level][:, None]
        mag = mag.reshape(R // m, nbc, m).transpose(0, 2, 1).reshape(R, nbc)
        return 2.0 ** -22 * (sums @ torch.from_numpy(np.ascontiguousarray(mag.T)).to(dev)) + 1e-30

    wide, fine = bound(128), bound(2)
    got = {}
    for batch in (32, 33, 47, 48, 64, 65, 96, 97):
        y = torch.full((batch, R), -7.0, device=dev)
        plan.mp_gemm(0, xd[:batch], *args, y, ws)
        got[batch] = y.double()
        limit = fine if batch in narrow else wide
        assert bool(((got[batch] - ref[:batch]).abs() <= limit[:batch]).all()), batch
        rows = min(batch, 32)
        assert bool(((got[batch][:rows] - got[32][:rows]).abs() <= (limit + wide)[:rows]).all()), batch
        rms = ref.square().mean().sqrt()
        print("  %d rows: off by %.1e of the root mean square, from 32 rows by %.1e" % (
            batch, (got[batch] - ref[:batch]).abs().max() / rms, (got[batch][:rows] - got[32][:rows]).abs().max() / rms))
    plan.close()
    ctx.close()
