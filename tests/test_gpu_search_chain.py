"""A search is enqueued whole and its result read at the end: it equals the stages called one by one, also when it is stopped by
max_iters, when it takes several workgroups or the two-pass route, and when another plan of the context had its turn in between.
And where its workgroups give up waiting for each other: what was enqueued behind them does nothing, and both are done again."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb
from paper_2602_17698_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [(256, 512), (64, 1024), (512, 512), (128, 2048)]        # three column classes, not in order


def outputs(plan, shapes, m, avg, dev):
    N, elems = plan.num_blocks(), sum(r * c for r, c in shapes)
    z = lambda n, dt=torch.float32: torch.zeros(n, dtype=dt, device=dev)
    return dict(rp=z(sum(r for r, _ in shapes), torch.int32), cp=z(sum(c for _, c in shapes), torch.int32),
                w=z(elems, torch.bfloat16), s=z(elems), cost=z((N, plan.K)), level=z(N, torch.uint8), off=z(N + 1, torch.int64),
                codes=z(max(plan.codes_bytes_bound(avg), 16), torch.uint8), scale=z(N * m), zero=z(N * m))


@pytest.mark.parametrize("m,n,max_iters", [(16, 64, 100000), (32, 128, 1), (8, 32, 100000), (8, 8, 2), (8, 64, 3)])
def test_search_equals_its_stages(m, n, max_iters):
    print("[case] search chain", m, n, max_iters, flush=True)
    dev = torch.device("cuda:0")
    bits, avg = [1, 2, 4], 2.3
    data = [synth.make_matrix("student_t", r, c, seed=5, tid=2 * i, device=dev) for i, (r, c) in enumerate(SHAPES)]
    mats = [sb.matrix(w, s) for w, s in data]
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plans = [sb.Plan(ctx, SHAPES, m, n, bits), sb.Plan(ctx, SHAPES[2:], m, n, bits)]
    got = []
    for plan, sh, ms, iters in ((plans[0], SHAPES, mats, max_iters), (plans[1], SHAPES[2:], mats[2:], 100000), (plans[0], SHAPES, mats, max_iters)):
        ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
        o = outputs(plan, sh, m, avg, dev)
        p = {k: t.data_ptr() for k, t in o.items()}
        out = sb.Outputs(p["rp"], p["cp"], p["w"], p["s"], p["cost"], p["level"], p["off"], p["codes"], o["codes"].numel(),
                         p["scale"], p["zero"])
        rc, st = plan.search(ms, avg, out, ws, max_iters=iters)
        torch.cuda.synchronize()
        got.append((rc, st, o))
    plan, ws, o = plans[0], torch.empty(plans[0].workspace_bytes(), dtype=torch.uint8, device=dev), outputs(plans[0], SHAPES, m, avg, dev)
    plan.reorder_all(mats, o["rp"], o["cp"], ws)
    plan.gather_all(mats, o["rp"], o["cp"], o["w"], o["s"], ws)
    plan.cost_table_all(o["w"], o["s"], o["cost"], ws)
    rc, st, _ = plan.allocate(o["cost"], avg, o["level"], ws, max_iters=max_iters)
    plan.offsets(o["level"], o["off"], ws)
    plan.pack_all(o["w"], o["level"], o["off"], o["codes"], o["scale"], o["zero"], ws)
    torch.cuda.synchronize()
    for rc_s, st_s, o_s in (got[0], got[2]):
        assert (rc_s, st_s) == (rc, st) and st["iters"] > 0
        for k in ("rp", "cp", "cost", "level", "off", "codes", "scale", "zero"):
            np.testing.assert_array_equal(o_s[k].cpu().numpy(), o[k].cpu().numpy(), err_msg=k)
    assert (rc == sb.ERR_MAX_ITERS) == (max_iters < 10)
    for p in plans:
        p.close()
    ctx.close()


# one pass with rows that two workgroups share, two passes, copies in one pass; offsets in one launch and in three; tables in
# registers and in memory
@pytest.mark.parametrize("shapes,m,n", [([(256, 8192), (128, 20480), (192, 4096)], 8, 64), ([(512, 4096), (256, 2048)], 8, 16),
                                        ([(512, 4096), (64, 1024)], 8, 32), ([(4096, 4096)], 8, 8), ([(8192, 4096 + 64)], 8, 8)])
def test_search_whose_workgroups_give_up(shapes, m, n):
    dev = torch.device("cuda:0")
    bits, avg = [1, 2, 4, 8], 2.9
    path = sb.variant_path("impatient")
    assert os.path.exists(path), "build the variant first: python -m paper_2602_17698_amd.build --tests"
    data = [synth.make_matrix("student_t", r, c, seed=11, tid=2 * i, device=dev) for i, (r, c) in enumerate(shapes)]
    mats = [sb.matrix(w, s) for w, s in data]
    prev, got = sb.LIB_PATH, []
    try:
        for lib in (prev, path, path):
            print("[case] search gives up", shapes, n, os.path.basename(lib), flush=True)
            sb.use_library(lib)
            ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
            plan = sb.Plan(ctx, shapes, m, n, bits)
            assert plan.num_blocks() > 2048                  # more than one workgroup
            ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
            o = outputs(plan, shapes, m, avg, dev)
            p = {k: t.data_ptr() for k, t in o.items()}
            out = sb.Outputs(p["rp"], p["cp"], p["w"], p["s"], p["cost"], p["level"], p["off"], p["codes"], o["codes"].numel(),
                             p["scale"], p["zero"])
            rc, st = plan.search(mats, avg, out, ws)
            got.append((rc, st, {k: t.cpu().numpy() for k, t in o.items() if k not in ("w", "s")}))
            plan.close()
            ctx.close()
    finally:
        sb.use_library(prev)
    for rc, st, o in got[1:]:
        assert (rc, st) == got[0][:2]
        for k, t in o.items():
            np.testing.assert_array_equal(t, got[0][2][k], err_msg=k)
