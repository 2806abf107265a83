"""Searches and single steps of at most 64 blocks, which one wave does by ranking: at both sides of that line, with shared values,
uneven steps, blocks in both sets, budgets below and above what is in use, few iterations; against the oracle (whole numbers: equal)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


@pytest.mark.parametrize("N", [1, 2, 16, 33, 63, 64, 65])
@pytest.mark.parametrize("bits", [[4], [2, 8], [2, 3, 4], [0, 1, 3, 8], [1, 2, 3, 4, 5, 6, 7, 8], [0, 1, 2, 3, 4, 5, 6, 7, 8]])
def test_few_blocks(orc, N, bits):
    print("[case] search of few blocks", N, bits, flush=True)
    dev = torch.device("cuda:0")
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(N * 8, 8)], 8, 8, bits)
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    rng = np.random.default_rng(1000 * N + len(bits))
    K = len(bits)
    falling = -np.sort(-rng.random((N, K)), axis=1)
    for case, cost in enumerate((falling, np.round(falling * 3), rng.random((N, K)) - 0.4, np.round(rng.random((N, K)) * 2), np.zeros((N, K)))):
        cost = np.ascontiguousarray(cost, dtype=np.float32)
        for avg in (bits[0], bits[0] + 0.37 * (bits[-1] - bits[0]), bits[0] + 0.8 * (bits[-1] - bits[0]), bits[-1] + 1):
            for gamma, cap in ((1.0, 500), (0.3, 500), (0.04, 3)):
                level = torch.full((N,), 255, dtype=torch.uint8, device=dev)
                kw = dict(gamma0=gamma, gammaT=0.01, max_iters=cap, init_mode=case & 1)
                got = plan.allocate(torch.from_numpy(cost).to(dev), avg, level, ws, trace_cap=500, **kw)
                rc, want, st, tr = orc.allocate(cost, bits, avg, want_trace=True, **kw)
                assert got == (sb.ERR_MAX_ITERS if rc else 0, st, tr), (case, avg, gamma)
                np.testing.assert_array_equal(level.cpu().numpy(), want)
        lv = rng.integers(0, K, N).astype(np.uint8)
        used = int(np.asarray(bits)[lv].sum())
        out = torch.empty(N, dtype=torch.uint8, device=dev)
        for slack in (0, 1, 5, N, -1, -N):
            b = (used + slack + 0.5) / N
            if b < bits[0]:
                continue
            for up, dn in ((cost[:, 0], cost[:, -1]), (-cost[:, 0], cost[:, 0]), (cost[:, -1], -cost[:, -1])):
                up, dn = np.ascontiguousarray(up), np.ascontiguousarray(dn)
                for k in (1, max(1, N // 3), 2 * N):
                    kind, want, winfo = orc.propose(up, dn, lv, bits, b, k)
                    info = plan.propose(torch.from_numpy(up).to(dev), torch.from_numpy(dn).to(dev), torch.from_numpy(lv).to(dev), b, k, out, ws)
                    assert info["kind"] == kind and all(info[f] == winfo[f] for f in winfo), (case, slack, k)
                    np.testing.assert_array_equal(out.cpu().numpy(), want)
    plan.close()
    ctx.close()
