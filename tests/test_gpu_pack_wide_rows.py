"""Packing of rows wider than 16384 elements, whose columns two workgroups share: at the edges of the halves (a chunk past them, the
second half nearly empty, both full), for units that do not fill the pairs, next to matrices of other row classes; against
packing of the reordered copy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shapes,bits", [(64, [(8, 16448)], [1, 2, 3, 4, 8]), (128, [(24, 16512), (8, 512)], [2, 3, 4]), (128, [(40, 28672)], [0, 3, 8]),
                                           (64, [(16, 32704), (8, 32768), (24, 32704)], [4, 7]), (128, [(72, 32768)], [1, 2, 3, 4, 5, 6, 7, 8]),
                                           (128, [(136, 20480), (8, 16384), (16, 20480)], [1, 2, 4])])
def test_pack_wide_rows(n, shapes, bits):
    print("[case] pack wide", n, shapes, bits, flush=True)
    dev = torch.device("cuda:0")
    m = 8
    data = [synth.make_matrix("outlier_chan", r, c, seed=7, tid=2 * i, device=dev) for i, (r, c) in enumerate(shapes)]
    mats = [sb.matrix(w, s) for w, s in data]
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, shapes, m, n, bits)
    N = plan.num_blocks()
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    rp = torch.empty(sum(r for r, _ in shapes), dtype=torch.int32, device=dev)
    cp = torch.empty(sum(c for _, c in shapes), dtype=torch.int32, device=dev)
    plan.reorder_all(mats, rp, cp, ws)
    w_re = torch.empty(sum(r * c for r, c in shapes), dtype=torch.bfloat16, device=dev)
    plan.gather_all(mats, rp, cp, w_re, None, ws)
    g = torch.Generator(device=dev)
    g.manual_seed(N)
    level = torch.randint(0, len(bits), (N,), generator=g, device=dev).to(torch.uint8)
    off = torch.empty(N + 1, dtype=torch.int64, device=dev)
    plan.offsets(level, off, ws)
    got = []
    for fused in (True, False):
        codes = torch.full((int(off[-1]) + 64,), 0xA5, dtype=torch.uint8, device=dev)
        scale, zero = torch.full((N * m + 4,), -1.0, device=dev), torch.full((N * m + 4,), -1.0, device=dev)
        if fused:
            plan.gather_pack_all(mats, rp, cp, level, off, codes, scale, zero, ws)
        else:
            plan.pack_all(w_re, level, off, codes, scale, zero, ws)
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in (codes, scale, zero)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    assert (got[0][0][-64:] == 0xA5).all()
    plan.close()
    ctx.close()
