"""The products for up to 16 and for more than 32 batch rows at the edges of their work split: batch tiles and groups, row
groups past the matrix's end, odd numbers of block columns, column splits, workgroup shapes, every bitwidth with and
without pruned blocks.  Tolerance: a kernel sums terms of size |B| scale |x| in fp32, where B scale is at most the span of
the block row (2^c scale) and the offset that the codes carry (128 scale; 2^c scale for most bitwidths of the products for
many rows), and zero |x|.  The bound is 2^-22 of the sum of all of them for the largest error and 2^-24 for the root mean
square."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu

ALL = [1, 2, 3, 4, 5, 6, 7, 8]


# A product, and the kernels that it runs on a whole device: "first", "narrow" or "many", and the instance (columns of a block and, of the
# first, batch tiles, row groups, small offset; narrow, waves, small offset, x by way of LDS; many, see the test of its instances).
CASES = [
    # up to 16 rows: fewer block columns than waves, one more than the waves, odd numbers of blocks a wave
    (32, 128, 32, 128, [3], 1, 0, "narrow 128,16,0,0"),
    (96, 128 * 17, 32, 128, [0] + ALL, 3, 8, "narrow 128,16,0,0"),
    (64, 128 * 35, 64, 128, ALL, 8, 0, "narrow 128,16,0,1"),
    (96, 128 * 16, 32, 128, ALL, 9, 0, "narrow 128,16,0,1"),
    (64, 128 * 48, 64, 128, [2, 5, 7], 16, 24, "first 128,1,1,0"),
    (64, 64 * 33, 32, 64, [0] + ALL, 2, 0, "narrow 64,16,0,0"),
    (160, 64 * 130, 32, 64, [1, 3, 6, 8], 16, 8, "first 64,1,1,0"),
    (64, 128 * 80, 32, 128, [2, 4], 1, 0, "first 128,1,1,0"),         # 5 blocks a wave
    (64, 64 * 144, 32, 64, [2, 4], 5, 0, "first 64,1,1,0"),           # 9
    # more: few block columns and rows
    (32, 128, 32, 128, [4], 33, 0, "narrow 128,16,1,1"),              # one block, three groups of rows, the last of one
    (160, 128 * 5, 32, 128, ALL, 48, 8, "narrow 128,16,1,1"),
    (192, 128 * 8, 64, 128, [0] + ALL, 49, 0, "narrow 128,16,1,1"),   # four groups
    (96, 64 * 9, 32, 64, ALL, 64, 16, "narrow 64,16,1,1"),
    (64, 64 * 5, 32, 64, [1], 50, 0, "narrow 64,16,1,1"),
    (96, 128 * 10, 32, 128, ALL, 40, 0, "narrow 128,16,1,1"),
    (32, 128, 32, 128, ALL[2:3], 40, 1 << 20, "narrow 128,16,1,1 narrow 128,16,1,1"),     # a pitch past 32-bit offsets of a batch group: 32 rows a launch, then 8
    # many rows: a last group of one row; one with a ragged last tile; 1 bit; column splits
    (128, 64 * 16, 64, 64, [0, 3, 5, 7, 8], 65, 0, "many 64,2,2,8,0"),
    (256, 128 * 6, 128, 128, [2, 6], 113, 0, "many 128,2,2,8,0"),
    (8192, 256, 128, 128, [1, 4, 8], 70, 0, "many 128,3,4,4,0"),
    (12288, 256, 128, 128, [3, 8], 128, 0, "many 128,4,4,4,0"),
    (12288, 192, 64, 64, ALL, 100, 0, "many 64,4,4,4,0"),
    (64, 128 * 3, 32, 128, [2, 4, 8], 200, 0, "many 128,2,2,8,0 many 128,2,2,8,0"),           # a second launch
    (64, 128 * 4, 32, 128, [1], 80, 0, "many 128,2,2,8,0"),
    (64, 64 * 400, 64, 64, [2, 5, 8], 64, 0, "many 64,2,2,8,0"),
    (320, 128 * 46, 32, 128, [1, 3, 7], 90, 0, "many 128,2,2,8,0"),
    (16512, 128 * 16, 128, 128, [2, 3], 70, 0, "many 128,2,2,8,0"),
    (16512, 64 * 40, 128, 64, [3, 4], 81, 0, "many 64,3,2,8,0"),
    (8320, 128 * 32, 128, 128, [2, 3], 65, 0, "many 128,2,2,8,0"),
    # 64 rows, and the rest by the kernels for few
    (16512, 64 * 12, 128, 64, [1], 70, 0, "many 64,4,4,4,0 first 64,1,1,1"),
    (24704, 64 * 16, 128, 64, [1], 81, 0, "many 64,4,4,4,0 first 64,2,2,1"),
    (16416, 128 * 9, 32, 128, [1, 4, 8], 66, 0, "many 128,4,4,4,0 narrow 128,8,1,1"),
    # up to 16 rows: column splits, several turns
    (32, 128 * 49, 32, 128, [2, 6], 16, 0, "first 128,1,1,0"),        # 4 blocks a wave, four column splits
    (32, 64 * 80, 32, 64, [1, 2], 16, 0, "first 64,1,1,0"),           # five
    (8320, 64 * 16, 128, 64, [1, 2], 7, 0, "narrow 64,8,0,1"),
    (12288, 128 * 16, 128, 128, [2, 6], 16, 0, "narrow 128,8,0,1"),
    (8224, 128 * 3, 32, 128, [4, 8], 7, 0, "narrow 128,8,0,1"),
]


@pytest.mark.parametrize("R,C,m,n,bits,batch,pad", [case[:7] for case in CASES])
def test_product_edges(orc, R, C, m, n, bits, batch, pad, one_bit=128):
    print("[case] product", R, C, m, n, bits, batch, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(R + C + batch)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(m, n), (R, C)], m, n, bits)
    N, base = plan.num_blocks(), 1
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    level = rng.integers(0, len(bits), N).astype(np.uint8)
    off = orc.offsets(level, m, n, bits)
    codes = np.zeros(max(int(off[-1]), 16), np.uint8)
    scale, zero = np.zeros(N * m, np.float32), np.zeros(N * m, np.float32)
    W = orc.f32_to_bf16(0.02 * rng.standard_t(4, size=(R, C)))
    orc.pack(W, m, n, bits, level, off, base, codes, scale, zero)
    xb = orc.f32_to_bf16(rng.standard_normal((batch, C)))
    x = torch.full((batch, C + pad), float("nan"), dtype=torch.bfloat16, device=dev)   # what lies past the columns is not read
    x[:, :C] = torch.from_numpy(xb.view(np.int16)).view(torch.bfloat16)
    args = [torch.from_numpy(t).to(dev) for t in (level, off, codes, scale, zero)]
    y = torch.full((batch + 1, R), -7.0, device=dev)
    plan.mp_gemm(1, x[:, :C], *args, y, ws)
    again = torch.empty_like(y[:batch])
    plan.mp_gemm(1, x[:, :C], *args, again, ws)
    torch.cuda.synchronize()
    assert torch.equal(y[:batch], again) and torch.all(y[batch] == -7.0)
    What = orc.dequant(codes, scale, zero, level, off, base, R, C, m, n, bits).astype(np.float64)
    xf = orc.bf16_to_f32(xb).astype(np.float64)
    ref = xf @ What.T
    nbc = C // n
    offset = {1: one_bit, 6: 128, 7: 128} if batch > 32 else {b: 128 for b in range(1, 8)}
    most = np.array([2.0 ** b + offset.get(b, 2.0 ** b) for b in bits])      # of |B|, in codes
    mag = (np.abs(zero.reshape(N, m)) + scale.reshape(N, m) * most[level][:, None])[base:]
    mag = mag.reshape(R // m, nbc, m).transpose(0, 2, 1).reshape(R, nbc)
    bound = np.abs(xf).reshape(batch, nbc, n).sum(2) @ mag.T
    err = np.abs(y[:batch].cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= bound * 2.0 ** -22 + 1e-30), float((err / (bound + 1e-300)).max())
    assert np.sqrt((err ** 2).mean()) <= 2.0 ** -24 * np.sqrt((bound ** 2).mean())
    plan.close()
    ctx.close()


@pytest.mark.parametrize("R,C,m,n,batch", [(1024, 4096, 128, 128, 100), (256, 8192, 32, 64, 64), (32, 16384, 32, 128, 33), (64, 32768, 64, 64, 128),
                                           (2048, 4096, 128, 128, 250)])
def test_product_does_not_depend_on_the_rest_of_the_plan(R, C, m, n, batch):
    """A matrix alone in its plan and next to one whose stages need a far larger workspace: the same bits, and nothing is
    written behind the workspace that the plan asks for."""
    print("[case] product alone and in company", R, C, m, n, batch, flush=True)
    dev = torch.device("cuda:0")
    bits, g = [2, 3, 4, 8], torch.Generator(device=dev)
    g.manual_seed(R + C)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    w = (0.02 * torch.randn(R, C, generator=g, device=dev)).to(torch.bfloat16)
    x = torch.randn(batch, C, generator=g, device=dev).to(torch.bfloat16)
    nb = (R // m) * (C // n)
    lv = torch.randint(0, 4, (nb,), generator=g, device=dev).to(torch.uint8)
    out = []
    for shapes in ([(R, C)], [(R, C), (16384, 16384)]):
        plan = sb.Plan(ctx, shapes, m, n, bits)
        N, need = plan.num_blocks(), plan.workspace_bytes()
        ws = torch.full((need + 65536,), 0x5A, dtype=torch.uint8, device=dev)
        level = torch.zeros(N, dtype=torch.uint8, device=dev)
        level[:nb] = lv
        off = torch.empty(N + 1, dtype=torch.int64, device=dev)
        plan.offsets(level, off, ws)
        codes = torch.zeros(int(off[-1]), dtype=torch.uint8, device=dev)
        scale, zero = torch.zeros(N * m, device=dev), torch.zeros(N * m, device=dev)
        plan.pack(0, w, level, off, codes, scale, zero)
        y = torch.full((batch, R), -7.0, device=dev)
        plan.mp_gemm(0, x, level, off, codes, scale, zero, y, ws)
        torch.cuda.synchronize()
        assert torch.all(ws[need:] == 0x5A)
        out.append(y)
        plan.close()
    assert torch.equal(out[0], out[1])
    ctx.close()
