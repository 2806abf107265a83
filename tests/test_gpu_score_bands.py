"""Channel scores of plans whose band height differs, bit for bit against the oracle: rows that end inside a band, the
smallest bands, 128 bands and just below the next height, and plans of many matrices."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [
    [(8, 8)], [(520, 512)], [(1032, 4104), (24, 520)], [(1024, 8)], [(16384, 8)], [(16392, 8)], [(32768, 16)], [(2056, 16392)],
    [(512, 520)] * 60, [(264, 8)] * 110, [(264, 8)] * 200,
])
def test_score_bands(orc, shapes):
    print("[case] score bands", len(shapes), shapes[0], flush=True)
    rng = np.random.default_rng(sum(r * c for r, c in shapes) % 1000)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, shapes, 8, 8, [2, 4])
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device="cuda:0")
    S = [np.abs(rng.standard_normal(s)).astype(np.float32) ** 3 for s in shapes]
    Sd = [torch.from_numpy(s).to("cuda:0") for s in S]
    M = [sb.matrix(None, s) for s in Sd]
    nr, nc = sum(r for r, _ in shapes), sum(c for _, c in shapes)
    rp, cp = (torch.full((k,), -1, dtype=torch.int32, device="cuda:0") for k in (nr, nc))
    plan.reorder_all(M, rp, cp, ws)
    want = [orc.channel_scores(s) for s in S]
    np.testing.assert_array_equal(rp.cpu().numpy(), np.concatenate([orc.argsort_desc(r) for r, _ in want]))
    np.testing.assert_array_equal(cp.cpu().numpy(), np.concatenate([orc.argsort_desc(c) for _, c in want]))
    last = len(shapes) - 1
    rs, cs = torch.empty(shapes[last][0], device="cuda:0"), torch.empty(shapes[last][1], device="cuda:0")
    plan.channel_scores(last, M[last], rs, cs, ws)
    np.testing.assert_array_equal(rs.cpu().numpy().view(np.uint32), want[last][0].view(np.uint32))
    np.testing.assert_array_equal(cs.cpu().numpy().view(np.uint32), want[last][1].view(np.uint32))
    plan.close()
    ctx.close()
