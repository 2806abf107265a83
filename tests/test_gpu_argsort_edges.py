"""The argsort around its chunks of 1024 channels, against the oracle: one channel more and less than a chunk, several chunks
with many ties across them, the longest arrays, pieces shorter and longer than a chunk.  Orders are exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_17698_amd import binding as sb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C,kind", [
    (8, 1016, "ties"), (1016, 1024, "ties"), (1032, 1528, "ties"), (2048, 2056, "equal"), (5000, 8, "ties"),
    (8, 32768, "ties"), (32768, 8, "few"), (3064, 1544, "special"),
])
def test_argsort_edges(orc, R, C, kind):
    print("[case] argsort", R, C, kind, flush=True)
    rng = np.random.default_rng(R * 7 + C)
    if kind == "equal":
        S = np.ones((R, C), np.float32)
    elif kind == "few":                       # almost every channel ties
        S = (rng.random((R, C)) < 0.001).astype(np.float32)
    else:
        S = rng.integers(0, 3, (R, C)).astype(np.float32)
    if kind == "special":                     # sums of 0, and sums that overflow
        S[rng.random(R) < 0.3] = 0.0
        S[5] = S[1700] = np.float32(3e38)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(R, C)], 8, 8, [2, 4])
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device="cuda:0")
    Sd = torch.from_numpy(S).to("cuda:0")
    rs, cs = torch.empty(R, device="cuda:0"), torch.empty(C, device="cuda:0")
    rp = torch.full((R,), -1, dtype=torch.int32, device="cuda:0")
    cp = torch.full((C,), -1, dtype=torch.int32, device="cuda:0")
    M = sb.matrix(None, Sd)
    plan.channel_scores(0, M, rs, cs, ws)
    plan.reorder(0, M, rp, cp, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(rp.cpu().numpy(), orc.argsort_desc(rs.cpu().numpy()))
    np.testing.assert_array_equal(cp.cpu().numpy(), orc.argsort_desc(cs.cpu().numpy()))
    plan.close()
    ctx.close()


@pytest.mark.parametrize("n,piece", [(4096, 64), (4096, 1024), (6144, 2048), (7680, 1280), (6000, 8)])
def test_argsort_pieces(orc, n, piece):
    print("[case] argsort in pieces", n, piece, flush=True)
    rng = np.random.default_rng(n + piece)
    ctx = sb.Context(0, torch.cuda.current_stream().cuda_stream)
    plan = sb.Plan(ctx, [(n, 8), (16, 8)], 8, 8, [2, 4])
    ws = torch.empty(plan.workspace_bytes(), dtype=torch.uint8, device="cuda:0")
    S = [torch.from_numpy(rng.integers(0, 9, s).astype(np.float32)).to("cuda:0") for s in [(n, 8), (16, 8)]]
    rp = torch.full((n + 16,), -1, dtype=torch.int32, device="cuda:0")
    cp = torch.full((16,), -1, dtype=torch.int32, device="cuda:0")
    plan.reorder_coupled_all([sb.matrix(None, s) for s in S], [0, sb.DIM_FIXED], [sb.DIM_INDEPENDENT, sb.DIM_FIXED], 1, [piece],
                             rp, cp, ws)
    torch.cuda.synchronize()
    score = S[0].cpu().numpy().sum(1, dtype=np.float32)               # whole numbers: exact in any order
    np.testing.assert_array_equal(rp[:n].cpu().numpy(), orc.argsort_desc_pieces(score, piece))
    np.testing.assert_array_equal(rp[n:].cpu().numpy(), np.arange(16))
    np.testing.assert_array_equal(cp[:8].cpu().numpy(), orc.argsort_desc(S[0].cpu().numpy().sum(0, dtype=np.float32)))
    plan.close()
    ctx.close()
