"""Searches on 32- and 256-column blocks score the matrices and write their reordered copies in one pass over the originals: copies
and table equal those of gather and cost table one after the other, bit for bit.  Every row class of the kernel (up to 4096,
8192, 16384 columns, wider), rows whose chunks do not fill the lanes, few and many candidates, pitched inputs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 256])
@pytest.mark.parametrize("m,cols,bits", [(8, (256, 768, 4096), [2, 3]), (16, (1280, 2304), [1, 2, 3, 4]), (32, (512, 4352, 8192), [0, 1, 2, 4]),
                                         (128, (8448, 3840), [1, 2, 3, 4, 8]), (64, (14336, 16384), [4]), (8, (12544, 256), [0, 1, 2, 3, 4, 8]),
                                         (16, (16640, 9984), [1, 2, 3, 4, 5, 6, 7, 8]), (8, (2816, 14336), [0, 1, 2, 3, 4, 5, 6, 7, 8]),
                                         (256, (2048, 12032), [1, 2, 3, 4, 5, 6, 7])])
def test_one_pass_with_copies(m, n, cols, bits):
    print("[case] copies", m, n, cols, bits, flush=True)
    dev = torch.device("cuda:0")
    shapes = [(m * (1 + i) if m > 8 else 24, c) for i, c in enumerate(cols)]
    data = []
    for i, (r, c) in enumerate(shapes):
        w, s = synth.make_matrix("outlier_chan" if i else "student_t", r, c, seed=3, tid=2 * i, device=dev)
        wp, sp = torch.zeros(r, c + 8 * i, dtype=w.dtype, device=dev), torch.zeros(r, c + 4 * i, device=dev)
        wp[:, :c], sp[:, :c] = w, s
        data.append((wp[:, :c], sp[:, :c]))
    data[0][0][:, : n] = 0.5                                # groups of one value
    mats = [sb.matrix(w, s) for w, s in data]
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, shapes, m, n, bits)
    assert not plan.gather_cost_supported()
    N, elems, avg = plan.num_blocks(), sum(r * c for r, c in shapes), 0.5 * (bits[0] + bits[-1])
    ws = torch.empty(plan.workspace_bytes() + 4096, dtype=torch.uint8, device=dev)
    ws[plan.workspace_bytes():] = 171
    z = lambda k, dt=torch.float32: torch.zeros(k, dtype=dt, device=dev)
    rp, cp = z(sum(r for r, _ in shapes), torch.int32), z(sum(c for _, c in shapes), torch.int32)
    w_re, s_re, cost = z(elems, torch.bfloat16), z(elems), z((N, plan.K))
    level, off, codes = z(N, torch.uint8), z(N + 1, torch.int64), z(max(plan.codes_bytes_bound(avg), 16), torch.uint8)
    scale, zero = z(N * m), z(N * m)
    out = sb.Outputs(rp.data_ptr(), cp.data_ptr(), w_re.data_ptr(), s_re.data_ptr(), cost.data_ptr(), level.data_ptr(), off.data_ptr(),
                     codes.data_ptr(), codes.numel(), scale.data_ptr(), zero.data_ptr())
    plan.search(mats, avg, out, ws)
    w2, s2, cost2 = torch.empty_like(w_re), torch.empty_like(s_re), torch.empty_like(cost)
    plan.gather_all(mats, rp, cp, w2, s2, ws)
    plan.cost_table_all(w2, s2, cost2, ws)
    torch.cuda.synchronize()
    assert torch.equal(w_re.view(torch.int16), w2.view(torch.int16))
    assert torch.equal(s_re.view(torch.int32), s2.view(torch.int32))
    assert torch.equal(cost.view(torch.int32), cost2.view(torch.int32))
    assert bool((ws[plan.workspace_bytes():] == 171).all())
    plan.close()
    ctx.close()
