"""The reorder-gather at the edges of its staging: rows of one KiB and of more than the waves of a workgroup take in one
turn, rows that end inside a KiB, one to eight rows per workgroup and a last workgroup with fewer, both workgroup sizes.
Values are moved, so they are exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C", [(8, 8), (24, 256), (40, 520), (24, 1032), (16, 3080), (24, 4104), (40, 6152), (16, 8200), (24, 12296),
                                 (8, 16384), (24, 16392), (8, 27144), (8, 28680), (8, 32768)])
def test_gather_edges(R, C):
    print("[case] gather", R, C, flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(R + C)
    shapes = [(R, C), (16, 64), (R + 8, C)]
    W = [torch.randint(-2**15, 2**15, (r, c + 8), generator=g, device=dev, dtype=torch.int16).view(torch.bfloat16) for r, c in shapes]
    S = [torch.randint(-2**31, 2**31, (r, c + 4), generator=g, device=dev, dtype=torch.int64).to(torch.int32).view(torch.float32) for r, c in shapes]
    perm = lambda n: torch.randperm(n, generator=g, device=dev).to(torch.int32)
    rps, cps = [perm(r) for r, _ in shapes], [perm(c) for _, c in shapes]
    mats = [sb.matrix(w[:, :c], s[:, :c]) for w, s, (_, c) in zip(W, S, shapes)]
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, shapes, 8, 8, [2, 4])
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    n = sum(r * c for r, c in shapes)
    w_re, s_re = torch.empty(n, dtype=torch.bfloat16, device=dev), torch.empty(n, device=dev)
    plan.gather_all(mats, torch.cat(rps), torch.cat(cps), w_re, s_re, ws)
    w_one, s_one = torch.empty(R, C, dtype=torch.bfloat16, device=dev), torch.empty(R, C, device=dev)
    plan.gather(0, mats[0], rps[0], cps[0], w_one, s_one)
    torch.cuda.synchronize()
    at = 0
    for w, s, rp, cp, (r, c) in zip(W, S, rps, cps, shapes):
        want_w = w.view(torch.int16)[rp.long()][:, cp.long()].cpu().numpy()
        want_s = s.view(torch.int32)[rp.long()][:, cp.long()].cpu().numpy()
        np.testing.assert_array_equal(w_re[at:at + r * c].view(torch.int16).view(r, c).cpu().numpy(), want_w)
        np.testing.assert_array_equal(s_re[at:at + r * c].view(torch.int32).view(r, c).cpu().numpy(), want_s)
        if at == 0:
            np.testing.assert_array_equal(w_one.view(torch.int16).cpu().numpy(), want_w)
            np.testing.assert_array_equal(s_one.view(torch.int32).cpu().numpy(), want_s)
        at += r * c
    plan.close()
    ctx.close()
