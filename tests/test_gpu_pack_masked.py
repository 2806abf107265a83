"""Packing of the original weights by the instances for devices whose 16-bit loads leave half of a register as it was (a library that
takes every device for one): the same codes, scales and origins as packing of the reordered copy.  Each row class, few and many
bits, ragged rows."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shapes,bits", [(64, [(16, 4096), (24, 192)], [0, 1, 2, 3, 4, 5, 6, 7, 8]), (128, [(24, 7808), (8, 4224)], [2, 4]),
                                           (128, [(16, 16384)], [1, 8]), (64, [(8, 16448), (16, 32768)], [3, 4])])
def test_masked_instances(n, shapes, bits):
    print("[case] pack masked", n, shapes, bits, flush=True)
    prev, path = sb.LIB_PATH, sb.variant_path("masked")
    assert os.path.exists(path), "build the variant first: python -m paper_2602_17698_amd.build --tests"
    sb.use_library(path)
    try:
        dev, m = torch.device("cuda:0"), 8
        data = [synth.make_matrix("outlier_chan", r, c, seed=9, tid=2 * i, device=dev) for i, (r, c) in enumerate(shapes)]
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
            scale, zero = torch.full((N * m,), -1.0, device=dev), torch.full((N * m,), -1.0, device=dev)
            if fused:
                plan.gather_pack_all(mats, rp, cp, level, off, codes, scale, zero, ws)
            else:
                plan.pack_all(w_re, level, off, codes, scale, zero, ws)
            torch.cuda.synchronize()
            got.append([t.cpu().numpy() for t in (codes, scale, zero)])
        for a, b in zip(*got):
            np.testing.assert_array_equal(a, b)
        plan.close()
        ctx.close()
    finally:
        sb.use_library(prev)
