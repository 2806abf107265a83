"""The cost table of rows wider than 16384 elements, whose weights and sensitivities share LDS and whose columns two or four workgroups share,
bit for bit against the oracle: the narrowest and the widest row, rows with and without overlapping pieces, parts that end inside a lane group's chunks or
have none at all, both numbers of parts, every number of candidates, the reordered weights as an output, and a pitch; and a matrix of few such rows, by
way of a copy in the workspace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu


# n, R, C, m, bits, pad; workgroups that share a row (0: a copy in the workspace), and 1 KiB pieces of sensitivities and weights with the same place
CASES = [
    (64, 64, 16448, 32, [3], 0, 4, 0),                      # four parts, the last one empty
    (128, 256, 16512, 8, [1, 2, 3, 4, 5, 6, 7, 8], 0, 4, 0),
    (64, 160, 26624, 8, [0, 2, 4], 8, 4, 0),                # the last row without overlap, pitched
    (64, 160, 26688, 8, [0, 2, 4], 0, 4, 1),                # and the first with it
    (64, 160, 26816, 8, [0, 2, 4], 8, 4, 1),
    (128, 192, 27264, 64, [2, 3, 4], 0, 4, 3),
    (64, 192, 28608, 64, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 4, 14),
    (64, 136, 32768, 8, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 4, 38),
    (128, 64, 32768, 16, [1, 8], 0, 4, 34),
    (128, 1160, 16640, 8, [2, 5], 0, 2, 0),                 # 145 units of one octet
    (64, 1096, 17344, 8, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 2, 0),
    (64, 520, 25600, 8, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 2, 0),     # 65 units; the last row without overlap
    (64, 520, 25664, 8, [0, 1, 2, 3, 4, 5, 6, 7, 8], 8, 2, 2),
    (128, 1040, 28672, 16, [1, 2, 3, 4, 5, 6], 0, 2, 12),
    (64, 1048, 24640, 8, [1, 2, 4, 8], 16, 2, 0),
    (64, 520, 32768, 8, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 2, 42),    # the most overlap
    (64, 8, 16448, 8, [2, 8], 8, 0, 0),                     # few rows
    (128, 128, 32768, 32, [0, 1, 4], 0, 0, 0),
    (128, 248, 16512, 8, [1, 2, 3, 4, 8], 16, 0, 0),
    (64, 64, 28672, 64, [0, 1, 2, 3, 4, 5, 6, 7, 8], 0, 0, 0),
]


@pytest.mark.parametrize("n,R,C,m,bits,pad", [case[:6] for case in CASES])
def test_cost_of_wide_rows(orc, n, R, C, m, bits, pad):
    print("[case] cost of wide rows", n, R, C, bits, flush=True)
    dev = torch.device("cuda:0")
    W, S = synth.make_matrix("student_t", R, C, seed=R + C)
    rng = np.random.default_rng(R + C)
    rp, cp = rng.permutation(R).astype(np.int32), rng.permutation(C).astype(np.int32)
    Wn, Sn = synth.bf16_bits(W), S.numpy()
    Wp, Sp = orc.gather(Wn, Sn, rp, cp)
    want = orc.cost_table(Wp, Sp, m, n, bits)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(R, C)], m, n, bits)
    need = plan.workspace_bytes()
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device=dev)
    Wd = torch.full((R, C + pad), float("nan"), dtype=torch.bfloat16, device=dev)
    Sd = torch.full((R, C + pad), float("nan"), device=dev)
    Wd[:, :C], Sd[:, :C] = W.to(dev), S.to(dev)
    cost = torch.zeros(plan.num_blocks(), len(bits), device=dev)
    w_re = torch.empty(R, C, dtype=torch.bfloat16, device=dev)
    perms = [torch.from_numpy(p).to(dev) for p in (rp, cp)]
    for out in (None, w_re):
        cost.fill_(-1.0)
        plan.gather_cost_all([sb.matrix(Wd[:, :C], Sd[:, :C])], *perms, out, cost, ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(cost.cpu().numpy().view(np.uint32), want.reshape(cost.shape).view(np.uint32))
    np.testing.assert_array_equal(synth.bf16_bits(w_re.cpu()).view(np.uint16), np.asarray(Wp).view(np.uint16))
    assert torch.all(ws[need:] == 0x5A)
    plan.close()
    ctx.close()
