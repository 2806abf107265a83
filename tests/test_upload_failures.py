"""A call that fails while the plan's page-locked image is made leaves the plan as it was: the next call sends the same image and
launches the same kernels as on a plan that never saw a failure."""
import pytest

from recording_runtime import record

SCRIPT = r"""
import os
if not os.path.exists(sb.LIB_PATH):
    from paper_2602_17698_amd import build
    build.build()
shapes = [(64, 128 * (i + 1)) for i in range(31)]                # as many column classes as matrices: the tables fill their slots
ctx = sb.Context(0, 0)
rows, cols = sum(r for r, _ in shapes), sum(c for _, c in shapes)
mats = [sb.Matrix(fake(2 * r * c), fake(4 * r * c), r, c, c, c) for r, c in shapes]
a = {k: fake(1 << 24) for k in ("rp", "cp", "w", "s", "cost", "level", "off", "codes", "scale", "zero", "ws")}
calls = {
    "gather_all": lambda p: p.gather_all(mats, a["rp"], a["cp"], a["w"], a["s"], a["ws"]),
    "gather_cost_all": lambda p: p.gather_cost_all(mats, a["rp"], a["cp"], None, a["cost"], a["ws"]),
    "gather_pack_all": lambda p: p.gather_pack_all(mats, a["rp"], a["cp"], a["level"], a["off"], a["codes"], a["scale"], a["zero"], a["ws"]),
    "cost_table_all": lambda p: p.cost_table_all(a["w"], a["s"], a["cost"], a["ws"]),
    "pack_all": lambda p: p.pack_all(a["w"], a["level"], a["off"], a["codes"], a["scale"], a["zero"], a["ws"]),
    "reorder_all": lambda p: p.reorder_all(mats, a["rp"], a["cp"], a["ws"]),
}
out = {}
for name, call in calls.items():
    for what, nth in (("hipHostMalloc", 1), ("hipEventCreateWithFlags", 1), ("hipEventCreateWithFlags", 2)):
        logs = []
        for broken in (False, True):
            plan = sb.Plan(ctx, shapes, 64, 128, [1, 2, 4])
            status = 0
            log()
            if broken:
                fail(what, nth)
                try:
                    call(plan)
                except sb.SbitsError as e:
                    status = e.status
                failed = log()
            call(plan), call(plan), call(plan)                   # (each image at least once)
            after = [line for line in log() if not line.startswith("event")]
            plan.close()
            if broken:
                failed += log()
            logs.append((status, after))
        events = [line for line in failed if line.startswith("event")]
        out["%s, %s %d" % (name, what, nth)] = [logs[0], logs[1], [line for line in failed if not line.startswith("event")], len(events)]
answer(out)
"""


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    return record(tmp_path_factory.mktemp("recorder"), SCRIPT)


def test_the_next_call_is_as_on_a_new_plan(runs):
    for name, (whole, broken, failed, _) in runs.items():
        assert whole[0] == 0 and broken[0] == -7, name                          # SBITS_ERR_HIP
        assert sum(line.startswith("launch") for line in whole[1]) >= 3, name
        assert whole[1] == broken[1], name
        assert failed == [], name                                               # nothing was enqueued
