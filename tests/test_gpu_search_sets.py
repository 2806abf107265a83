"""Sets of the search that meet or share words: blocks that are both the best to raise and the cheapest to lower (the two sides are
chosen side by side and then apart), values shared by many blocks (their places decide), steps of different widths (a part
of the raised set fits).  One workgroup, several, and a table in memory; against the oracle."""
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


def tables(N, bits, seed):
    """Rows that fall steeply after a flat step, in half of the blocks; few distinct values."""
    rng = np.random.default_rng(seed)
    cost = -np.sort(-rng.random((N, len(bits))), axis=1)
    odd = rng.random(N) < 0.5
    at = rng.integers(0, len(bits), N)
    j = np.arange(len(bits))[None, :]
    steep = np.where(j <= at[:, None], 4.0, 0.25) + rng.integers(0, 3, (N, 1))
    cost = np.where(odd[:, None], steep, cost)
    return cost.astype(np.float32), np.round(cost * 8).astype(np.float32)


@pytest.mark.parametrize("N,bits,avg", [(40, [1, 2, 3], 2.2), (700, [1, 2, 4, 8], 3.1), (2049, [2, 4, 8], 4.6), (9001, [1, 2, 3, 4, 8], 2.7),
                                        (70000, [0, 1, 3, 8], 2.4), (540000, [1, 2, 8], 2.3)])
def test_sets_that_meet_and_values_that_are_shared(orc, N, bits, avg):
    print("[case] search sets", N, bits, flush=True)
    dev = torch.device("cuda:0")
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    rows = next(r for r in range(1, N + 1) if N % r == 0 and N // r <= 4096)
    mats = (rows + 4095) // 4096
    while rows % mats:
        mats += 1
    plan = sb.Plan(ctx, [(rows // mats * 8, N // rows * 8)] * mats, 8, 8, bits)
    assert plan.num_blocks() == N
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device=dev)
    rng = np.random.default_rng(N)
    for case, cost in enumerate(tables(N, bits, N + 1)):
        for gamma in (0.3, 0.04):
            level = torch.full((N,), 255, dtype=torch.uint8, device=dev)
            got = plan.allocate(torch.from_numpy(cost).to(dev), avg, level, ws, gamma0=gamma, gammaT=0.01, trace_cap=500)
            rc, want, st, tr = orc.allocate(cost, bits, avg, gamma0=gamma, gammaT=0.01, want_trace=True)
            assert got == (rc, st, tr), (case, gamma)
            np.testing.assert_array_equal(level.cpu().numpy(), want)
        lv = rng.integers(0, len(bits), N).astype(np.uint8)
        used = int(np.asarray(bits)[lv].sum())
        s_up, s_dn = (np.ascontiguousarray(cost[:, c]) for c in (0, -1))
        out = torch.empty(N, dtype=torch.uint8, device=dev)
        for slack in (0, 1, 3, N // 50 + 2, -1, -N):
            b = (used + slack + 0.5) / N
            if b < bits[0]:
                continue
            for up in (s_up, -s_up):
                kind, want, winfo = orc.propose(up, s_dn, lv, bits, b, max(1, N // 9))
                info = plan.propose(torch.from_numpy(up).to(dev), torch.from_numpy(s_dn).to(dev), torch.from_numpy(lv).to(dev), b,
                                    max(1, N // 9), out, ws)
                assert info["kind"] == kind and all(info[f] == winfo[f] for f in winfo), (case, slack)
                np.testing.assert_array_equal(out.cpu().numpy(), want)
    plan.close()
    ctx.close()
