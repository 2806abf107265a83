"""The resident search kernel at the edges of its work split (blocks per workgroup, blocks in registers or in
memory, one workgroup or several), and the single-workgroup search behind a wait that was given up."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


@pytest.fixture(params=["", "impatient"])
def ctx(request, dev):
    """A context of the default build, and of the one whose workgroups give up waiting for each other at once."""
    prev, path = sb.LIB_PATH, sb.variant_path(request.param)
    assert os.path.exists(path), "build the variant first: python -m paper_2602_17698_amd.build --tests"
    sb.use_library(path)
    try:
        c = sb.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
        yield c
        c.close()
    finally:
        sb.use_library(prev)


def plan_with_blocks(ctx, N, bits, dev):
    b = next(b for b in range(1, N + 1) if N % b == 0 and N // b <= 4096)
    plan = sb.Plan(ctx, [(8 * (N // b), 8 * b)], 8, 8, bits)
    assert plan.num_blocks() == N
    return plan, torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)


def table(N, bits, seed):
    rng = np.random.default_rng(seed)
    c = np.exp(2.0 * rng.normal(size=(N, 1))) * 4.0 ** -np.asarray(bits, np.float64) * np.exp(0.2 * rng.normal(size=(N, len(bits))))
    return c.astype(np.float32)


# 2048 blocks per workgroup, 32 x 2048 the change to 4096 each, 128 x 4096 the last table held in registers
@pytest.mark.parametrize("N,bits,avg", [(1, [2, 3], 2.5), (2047, [2, 3, 4], 2.75), (2048, [1, 2, 3, 4, 8], 2.25),
                                        (2050, [1, 2, 3, 4], 2.5), (65536, [0, 2, 4, 8], 2.9), (65540, [1, 2, 3, 4], 2.5),
                                        (524288, [1, 2, 3, 4, 8], 2.25), (524304, [2, 3, 4], 2.75)])
def test_allocate_at_the_edges_of_the_work_split(orc, ctx, dev, N, bits, avg):
    say("allocate", N, bits, avg, sb.LIB_PATH)
    cost = table(N, bits, N)
    plan, ws = plan_with_blocks(ctx, N, bits, dev)
    level = torch.full((N,), 255, dtype=torch.uint8, device=dev)
    rc, st, tr = plan.allocate(torch.from_numpy(cost).to(dev), avg, level, ws, trace_cap=500)
    rc_o, level_o, st_o, tr_o = orc.allocate(cost, bits, avg, want_trace=True)
    assert (rc, st, tr) == (rc_o, st_o, tr_o)
    np.testing.assert_array_equal(level.cpu().numpy(), level_o)
    plan.close()


def test_allocate_where_values_lie_outside_the_first_bins(orc, ctx, dev):
    """Infinite and negative gains next to ordinary ones, and all gains but one below zero: the boundary falls
    into an outermost bin of the first round."""
    for name in ("infinite", "negative"):
        say(name)
        bits, N = [2, 3, 4], 6000
        cost = table(N, bits, 5)
        if name == "infinite":
            cost[:40, 0] = 3e38                          # (huge gains: a few values far above the rest)
            cost[40:80, 1] = cost[40:80, 0] * 2          # negative first steps
        else:
            cost = np.ascontiguousarray(cost[:, ::-1])
            cost[17] = [4, 2, 1]
        plan, ws = plan_with_blocks(ctx, N, bits, dev)
        for avg in (2.0, 2.01, 2.7, 3.0):
            level = torch.empty(N, dtype=torch.uint8, device=dev)
            rc, st, tr = plan.allocate(torch.from_numpy(cost).to(dev), avg, level, ws, gamma0=0.3, trace_cap=500)
            rc_o, level_o, st_o, tr_o = orc.allocate(cost, bits, avg, gamma0=0.3, want_trace=True)
            assert (rc, st, tr) == (rc_o, st_o, tr_o), avg
            np.testing.assert_array_equal(level.cpu().numpy(), level_o)
        plan.close()


@pytest.mark.parametrize("N", [2048, 2050, 524304, 3147776])     # the last: more workgroups than a search takes
def test_propose_at_the_edges_of_the_work_split(orc, ctx, dev, N):
    say("propose", N, sb.LIB_PATH)
    bits = [1, 2, 3, 4, 8]
    plan, ws = plan_with_blocks(ctx, N, bits, dev)
    rng = np.random.default_rng(N)
    level = rng.integers(0, len(bits), N).astype(np.uint8)
    used = int(np.asarray(bits)[level].sum())
    for case in range(4):
        s_up = rng.standard_normal(N).astype(np.float32) if case % 2 else rng.integers(-2, 6, N).astype(np.float32)
        s_dn = np.abs(rng.standard_normal(N)).astype(np.float32) - np.float32(0.1 * (case == 3))
        avg, k = (used + [0, N // 50, -3, 0][case]) / N + 1e-9, max(1, N // [20, 9, 30, 2][case])
        lv = torch.from_numpy(level).to(dev)
        d_up, d_dn = torch.from_numpy(s_up).to(dev), torch.from_numpy(s_dn).to(dev)
        kind, want, winfo = orc.propose(s_up, s_dn, level, bits, avg, k)
        out = torch.empty_like(lv)
        info = plan.propose(d_up, d_dn, lv, avg, k, out, ws)
        assert info["kind"] == kind and all(info[f] == winfo[f] for f in ("n_up", "n_dn", "bits_before", "bits_after"))
        np.testing.assert_array_equal(out.cpu().numpy(), want)
        plan.propose(d_up, d_dn, lv, avg, k, lv, ws, want_info=False)        # in place, without the host's answer
        torch.cuda.synchronize()
        np.testing.assert_array_equal(lv.cpu().numpy(), want)
    plan.close()


def _freed(s_up, s_dn, level, bits, k):
    """Step bits that the lowered set of a swap frees: the first h by s_down outside the first h by s_up."""
    h, K, widths = max(1, k // 2), len(bits), np.asarray(bits)
    up = np.flatnonzero(level < K - 1)
    raised = up[np.argsort(-s_up[up], kind="stable")][:h]
    dn = np.setdiff1d(np.flatnonzero(level > 0), raised)
    dn = dn[np.argsort(s_dn[dn], kind="stable")][:h]
    return int((widths[level[dn]] - widths[level[dn] - 1]).sum())


@pytest.mark.parametrize("N", [1500, 6000, 524304])       # one workgroup, several, blocks in memory
def test_propose_on_levels_over_budget(orc, ctx, dev, N):
    """The bits in use exceed the budget by more, as much and less than the lowered set frees: what does not fit is not
    proposed, and the counts are those of the levels written."""
    say("propose over budget", N, sb.LIB_PATH)
    bits = [1, 2, 4, 5]
    plan, ws = plan_with_blocks(ctx, N, bits, dev)
    rng = np.random.default_rng(N + 1)
    for case in ("far", "one too many", "all of it", "one left", "nobody to lower", "nobody to raise"):
        level = rng.integers(0, len(bits), N).astype(np.uint8)
        s_up, s_dn = rng.standard_normal(N).astype(np.float32), np.abs(rng.standard_normal(N)).astype(np.float32)
        k = N // 20
        if case == "nobody to lower":                     # all above the lowest candidate are in the raised set
            level[:] = 0
            some = rng.choice(N, k // 4, replace=False)
            level[some], s_up[some] = 1, 50.0 + s_up[some]
        elif case == "nobody to raise":
            level[:] = len(bits) - 1
        used, freed = int(np.asarray(bits)[level].sum()), _freed(s_up, s_dn, level, bits, k)
        over = {"far": N, "one too many": freed + 1, "all of it": freed, "one left": freed - 1, "nobody to lower": k // 4,
                "nobody to raise": 2 * N}[case]
        avg = (used - over) / N + 1e-9
        kind, want, winfo = orc.propose(s_up, s_dn, level, bits, avg, k)
        out = torch.full((N,), 77, dtype=torch.uint8, device=dev)
        info = plan.propose(torch.from_numpy(s_up).to(dev), torch.from_numpy(s_dn).to(dev), torch.from_numpy(level).to(dev),
                            avg, k, out, ws)
        got = out.cpu().numpy()
        assert info["kind"] == kind and all(info[f] == winfo[f] for f in winfo), (case, info, kind, winfo)
        np.testing.assert_array_equal(got, want, err_msg=case)
        assert int(np.asarray(bits)[got].sum()) == info["bits_after"], case
    plan.close()


@pytest.fixture
def unaided(dev):
    """A context of a library that does not repeat a search that was given up."""
    prev, path = sb.LIB_PATH, sb.variant_path("noretry")
    assert os.path.exists(path), "build the variant first: python -m paper_2602_17698_amd.build --tests"
    sb.use_library(path)
    try:
        c = sb.Context(device=0, stream=torch.cuda.current_stream().cuda_stream)
        yield c
        c.close()
    finally:
        sb.use_library(prev)


# 3, 128 and 128 workgroups; "both signs": entries that fall and rise, whose changes have sums with all upper bits set, added up
# as two halves: the lower ones carry, the upper ones wrap
@pytest.mark.parametrize("N", [6000, 524288, 524304])
@pytest.mark.parametrize("kind", ["falling", "both signs"])
def test_the_resident_workgroups_finish_by_themselves(orc, unaided, dev, N, kind):
    say("no second try", N, kind)
    bits = [1, 2, 3, 4]
    cost = table(N, bits, N) if kind == "falling" else np.random.default_rng(N).random((N, 4), dtype=np.float32)
    plan, ws = plan_with_blocks(unaided, N, bits, dev)
    level = torch.full((N,), 255, dtype=torch.uint8, device=dev)
    rc, st, tr = plan.allocate(torch.from_numpy(cost).to(dev), 2.5, level, ws, trace_cap=500)
    rc_o, level_o, st_o, tr_o = orc.allocate(cost, bits, 2.5, want_trace=True)
    assert (rc, st, tr) == (rc_o, st_o, tr_o)
    assert any(t["delta_fixed"] < 0 for t in tr)
    np.testing.assert_array_equal(level.cpu().numpy(), level_o)
    s_up, s_dn = (np.ascontiguousarray(cost[:, i]) for i in (0, 2))
    kind, want, winfo = orc.propose(s_up, s_dn, level_o, bits, 2.6, N // 20)
    info = plan.propose(torch.from_numpy(s_up).to(dev), torch.from_numpy(s_dn).to(dev), level, 2.6, N // 20, level, ws)
    assert info["kind"] == kind and all(info[f] == winfo[f] for f in winfo)
    np.testing.assert_array_equal(level.cpu().numpy(), want)
    plan.close()


def test_propose_with_the_most_workgroups(orc, unaided, dev):
    """256 of them, the largest number of parts that a sum has, in a swap whose two sets meet in many blocks."""
    N, bits = 1 << 22, [1, 2, 3, 4]
    say("no second try", N)
    plan, ws = plan_with_blocks(unaided, N, bits, dev)
    rng = np.random.default_rng(2)
    level = rng.integers(0, 4, N).astype(np.uint8)
    s_up = rng.random(N, dtype=np.float32)
    s_dn = np.ascontiguousarray(1 - s_up)
    avg, k = int(np.asarray(bits)[level].sum()) / N + 1e-9, N // 3
    kind, want, winfo = orc.propose(s_up, s_dn, level, bits, avg, k)
    out = torch.full((N,), 77, dtype=torch.uint8, device=dev)
    info = plan.propose(torch.from_numpy(s_up).to(dev), torch.from_numpy(s_dn).to(dev), torch.from_numpy(level).to(dev), avg, k, out, ws)
    assert kind == 2 and info["kind"] == kind and all(info[f] == winfo[f] for f in winfo)
    np.testing.assert_array_equal(out.cpu().numpy(), want)
    plan.close()


def test_propose_replays_from_a_captured_graph(orc, dev):
    say("propose in a graph")
    N, bits = 9000, [1, 2, 3, 4]
    stream = torch.cuda.Stream()
    ctx = sb.Context(device=0, stream=stream.cuda_stream)
    plan, ws = plan_with_blocks(ctx, N, bits, dev)
    rng = np.random.default_rng(1)
    level = rng.integers(0, 4, N).astype(np.uint8)
    avg = int(np.asarray(bits)[level].sum()) / N + 1e-9
    d_up, d_dn = torch.empty(N, device=dev), torch.empty(N, device=dev)
    lv, out = torch.from_numpy(level).to(dev), torch.empty(N, dtype=torch.uint8, device=dev)
    call = lambda: plan.propose(d_up, d_dn, lv, avg, 450, out, ws, want_info=False)
    d_up.zero_(), d_dn.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        call()
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    for replay in range(4):
        s_up, s_dn = rng.standard_normal(N).astype(np.float32), np.abs(rng.standard_normal(N)).astype(np.float32)
        d_up.copy_(torch.from_numpy(s_up)), d_dn.copy_(torch.from_numpy(s_dn))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), orc.propose(s_up, s_dn, level, bits, avg, 450)[1])
    plan.close()
    ctx.close()
