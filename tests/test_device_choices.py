"""Choices that the host makes by size and by device, on devices that need not be there."""
import re

import pytest

from recording_runtime import record

PACK = r"""
ctx_of = lambda ecc: (device(256, ecc), sb.Context(0, 0))[1]
out = {}
for ecc in (1, 0):
    for n, cols in ((64, 4096), (64, 8192), (128, 16384), (128, 28672)):
        ctx = ctx_of(ecc)
        plan = sb.Plan(ctx, [(64, cols)], 32, n, [1, 2, 4])
        mats = [sb.Matrix(fake(128 * cols), fake(256 * cols), 64, cols, cols, cols)]
        a = [fake(1 << 24) for _ in range(8)]
        log()
        plan.gather_pack_all(mats, a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7])
        pack = [line.split()[1] for line in log() if line.startswith("launch")]
        try:
            rc = plan.gather_cost_all(mats, a[0], a[1], None, a[2], a[7])
        except sb.SbitsError as e:
            rc = e.status
        out["%d %d %d" % (ecc, n, cols)] = [pack, rc]
        plan.close()
        ctx.close()
answer(out)
"""


def test_packing_of_original_weights_is_for_any_device(tmp_path):
    """Where 16-bit loads leave half of a register as it was, packing takes the instances that mask it; scoring is refused there."""
    for key, (pack, cost) in record(tmp_path, PACK).items():
        ecc = key[0] == "1"
        assert len(pack) == 1 and "gather_pack_kernel" in pack[0], key
        assert pack[0].count("Lb1E") == (0 if ecc else 2), key                  # (WIDE and MASK)
        assert cost == (0 if ecc else -8), key                                  # SBITS_ERR_UNIMPLEMENTED


OFFSETS = r"""
ctx = sb.Context(0, 0)
out = {}
for rows, cols in ((8, 8), (24576, 512), (24584, 512), (26624, 1024), (8192, 4096)):
    plan = sb.Plan(ctx, [(rows, cols)], 8, 8, [1, 2, 4])
    log()
    plan.offsets(fake(1 << 20), fake(1 << 23), fake(1 << 23))
    out[plan.num_blocks()] = len(log())
    plan.close()
answer(out)
"""


def test_offsets_in_one_launch_where_that_is_faster(tmp_path):
    for n, launches in record(tmp_path, OFFSETS).items():
        assert launches == (1 if int(n) <= 196608 else 3), n


PARTITION = r"""
out = {}
for cus in (256, 32):
    device(cus, 1)
    ctx = sb.Context(0, 0)
    class X:
        def __init__(self, batch, ld): self.shape, self.ld = (batch, ld), ld
        def data_ptr(self): return fake(1 << 20)
        def stride(self, i): return self.ld
    for name, n, shape, batch in (("narrow, 64 workgroups", 128, (2048, 1024), 3), ("first, 64-column blocks", 64, (2048, 8192), 20),
                                  ("first, two on a CU", 128, (2048, 16384), 4), ("first, 32 rows", 128, (4096, 8192), 32)):
        plan = sb.Plan(ctx, [shape], 32, n, [2, 4])
        a = [fake(1 << 24) for _ in range(8)]
        log()
        plan.mp_gemm(0, X(batch, shape[1]), a[0], a[1], a[2], a[3], a[4], a[5], a[6])
        out["%s %d" % (name, cus)] = [line.split()[1:6] for line in log() if line.startswith("launch")]
        plan.close()
    plan = sb.Plan(ctx, [(8192, 512)], 64, 128, [2, 4])
    mats = [sb.Matrix(fake(1 << 23), fake(1 << 24), 8192, 512, 512, 512)]
    log()
    plan.gather_pack_all(mats, *[fake(1 << 23) for _ in range(8)])
    out["packing %d" % cus] = [line.split()[1:6] for line in log() if line.startswith("launch")]
    plan.close()
    ctx.close()
answer(out)
"""


def test_workgroups_follow_the_compute_units_and_sums_do_not(tmp_path):
    """On a partition of 32 compute units the shape of the workgroups is another one, the kernel, which decides the order of the
    sums, the same."""
    got = record(tmp_path, PARTITION)
    base = lambda launches: [launch[0].split("sbits")[1].split("kernel")[0] for launch in launches]
    for key in got:
        if key.endswith(" 256"):
            assert base(got[key]) == base(got[key[:-3] + "32"]), key
    grid = lambda key: [int(v) for v in got[key][0][2].split(",")]
    block = lambda key: int(got[key][0][4])
    assert block("narrow, 64 workgroups 256") == 1024 and block("narrow, 64 workgroups 32") == 512
    assert block("first, 64-column blocks 32") >= block("first, 64-column blocks 256")
    assert block("first, two on a CU 256") == 256 and block("first, two on a CU 32") == 512
    assert grid("packing 256")[0] == 512 and grid("packing 32")[0] == 256          # octets: 2 and 4 a workgroup


SCORES = r"""
out = []
for cus in (256, 32):
    device(cus, 1)
    ctx = sb.Context(0, 0)
    for shapes in ([(2048, 2048)], [(4096, 4096)], [(16384, 8192)], [(12288, 12288)], [(9728, 16384)], [(1536, 4096)] * 11, [(768, 8)] * 43, [(4104, 8)] * 30,
                   [(8192, 20480)], [(3072, 3072)] * 3, [(8192, 16384)], [(4096, 4096)] * 12, [(14336, 4096)] * 16,
                   [(8704, 5120), (8192, 4608)]):
        plan = sb.Plan(ctx, shapes, 8, 8, [2, 4])
        mats = [sb.Matrix(fake(1 << 28), fake(1 << 29), r, c, c, c) for r, c in shapes]
        log()
        plan.reorder_all(mats, fake(1 << 20), fake(1 << 20), fake(1 << 28))
        launch = [line.split() for line in log() if "score_partial" in line]
        tall = sum(-(-r // 256) * -(-c // 4096) for r, c in shapes)
        out.append([cus, tall, int(launch[0][3].split(",")[0]), int(launch[0][-1]), sum(r * c for r, c in shapes) / (256 * 4096)])
        plan.close()
    ctx.close()
answer(out)
"""


def test_workgroups_of_the_scores_have_a_cu_each_or_share_it_evenly(tmp_path):
    """Bands of fewer than 256 rows are made only while every workgroup finds a CU of its own, or while the work is that of 200; where there
    are more workgroups than CUs all the same, two of them fit a CU's 160 KiB of LDS."""
    seen = record(tmp_path, SCORES)
    for cus, tall, grid, lds, work in seen:
        assert grid <= max(256, tall) or (grid <= 512 and work * grid / tall <= 205), (cus, tall, grid)
        assert lds <= (80 if grid > cus else 160) * 1024, (cus, tall, grid, lds)
    assert sum(128 < tall < 192 for _, tall, _, _, _ in seen) >= 4 and sum(128 < grid < 192 for _, _, grid, _, _ in seen) >= 8
    assert sum(256 < grid <= 512 and grid > tall for _, tall, grid, _, _ in seen) == 4


PACK_ALL = r"""
ctx = sb.Context(0, 0)
out = []
for n in (8, 16, 32, 64, 128, 512):
    for mib in (16, 32, 41, 64, 128, 160, 192, 256):
        plan = sb.Plan(ctx, [(64 * mib, 8192)], 8, n, [2, 4])
        a = [fake(1 << 29) for _ in range(12)]
        packs = lambda: [line.split()[1] for line in log() if " _ZN5sbits11pack_kernel" in line]
        log()
        plan.pack_all(*a[:7])
        again = packs()
        if n != 64 and n != 128:                  # (those are packed from the matrices themselves)
            try:
                plan.search([sb.Matrix(a[0], a[1], 64 * mib, 8192, 8192, 8192)], 3.0, sb.Outputs(*a[2:10], 1 << 40, *a[10:12]), fake(1 << 29))
            except sb.SbitsError:                 # (nothing ran: there is no result to finish with)
                pass
        out.append([n, mib, again, packs()])
        plan.close()
answer(out)
"""


def test_packing_of_copies_keeps_weights_in_the_caches_where_they_fit(tmp_path):
    """Blocks of up to 64 columns, weights that fit the memory-side cache with their codes: by ordinary loads where they are packed again, not in a search."""
    bounds = {8: (24, 144), 16: (40, 176), 32: (40, 208), 64: (72, 208)}
    for n, mib, again, search in record(tmp_path, PACK_ALL):
        lo, hi = bounds.get(n, (0, 0))
        name = "pack_kernelILi%dELb%dE"
        assert len(again) == 1 and name % (n // 8, lo < mib <= hi) in again[0], (n, mib, again)
        assert len(search) >= (n not in (64, 128)) and all(name % (n // 8, 0) in kernel for kernel in search), (n, mib, search)


COST = r"""
ctx = sb.Context(0, 0)
out = []
for shapes, n, bits, m in %r:
    plan = sb.Plan(ctx, shapes, m, n, bits)
    mats = [sb.Matrix(fake(2 * r * c), fake(4 * r * c), r, c, c, c) for r, c in shapes]
    a = [fake(1 << 24) for _ in range(4)]
    log()
    plan.gather_cost_all(mats, a[0], a[1], None, a[2], a[3])
    launches = [line.split()[1:] for line in log() if line.startswith("launch")]
    out.append([[v[0] for v in launches], plan.workspace_bytes(), [[int(v[2].split(",")[0]), int(v[4]), int(v[6])] for v in launches if "gather_cost_wide" in v[0]]])
    plan.close()
answer(out)
"""


def test_cost_of_few_wide_rows_goes_by_a_copy(tmp_path):
    """One matrix of its width with few rows beyond 16384 elements: reordered into the workspace, then scored; else in one pass."""
    nine, five, three, two = list(range(9)), [1, 2, 3, 4, 8], [2, 3, 4], [2, 8]
    cases = [([(8, 32768)], 128, three, 1), ([(128, 32768)], 64, three, 1), ([(136, 32768)], 128, three, 0), ([(128, 32768)], 128, five, 1),
             ([(136, 32768)], 64, nine, 0), ([(248, 16512)], 128, nine, 1), ([(8, 16512)], 128, two, 0), ([(8, 16448)], 64, two, 1), ([(8, 20480), (8, 20480)], 64, three, 0),
             ([(64, 4096), (8, 20480), (160, 25088)], 64, nine, 2), ([(64, 16384)], 64, nine, 0)]
    for (shapes, n, bits, copies), (kernels, ws, _) in zip(cases, record(tmp_path, COST % ([c[:3] + (8,) for c in cases],))):
        assert sum("13gather_kernel" in k for k in kernels) == 2 * copies, (shapes, kernels)
        assert sum("gather_cost_wide" in k for k in kernels) == len({c for _, c in shapes if c > 16384}) - copies, (shapes, kernels)
        wide = [r * c for r, c in shapes if c > 16384]
        assert ws > (6 * max(wide) if copies else 0), (shapes, ws)


def test_cases_of_wide_rows_have_the_parts_and_the_overlap_that_they_are_meant_for(tmp_path):
    """The tests of the cost of wide rows on the device, against the grid and the LDS of their launches."""
    pytest.importorskip("torch")
    import test_gpu_cost_wide_rows as wide
    seen = record(tmp_path, COST % ([([(R, C)], n, bits, m) for n, R, C, m, bits, *_ in wide.CASES],))
    for (n, R, C, m, bits, pad, parts, overlap), (_, _, launches) in zip(wide.CASES, seen):
        assert len(launches) == (parts > 0), (n, R, C)
        for grid, threads, lds in launches:
            sums = 4 // parts * threads // (n // 8) * len(bits) * 4
            assert grid == -(-R // 64) * 8 * parts, (n, R, C, grid)          # (an octet a workgroup, eight apart)
            assert -(-2 * C // 1024) - -(4 * C) // 1024 - (lds - sums) // 1024 == overlap, (n, R, C, lds)


PRODUCTS = r"""
class X:
    def __init__(self, batch, ld): self.shape, self.ld = (batch, ld), ld
    def data_ptr(self): return fake(1 << 20)
    def stride(self, i): return self.ld
ctx = sb.Context(0, 0)
out = []
for R, C, m, n, bits, batch, pad in %r:
    plan = sb.Plan(ctx, [(m, n), (R, C)], m, n, bits)
    a = [fake(1 << 24) for _ in range(7)]
    log()
    plan.mp_gemm(1, X(batch, C + pad), *a)
    out.append([line.split()[1] for line in log() if line.startswith("launch")])
    plan.close()
answer(out)
"""


def launched(tmp_path, products):
    """The kernels of each product (R, C, m, n, bits, rows of x, pitch - C): "first", "narrow" or "many" and the instance."""
    out = []
    for kernels in record(tmp_path, PRODUCTS % (products,)):
        names = [re.search(r"mp_gemm_(narrow_|many_|finish_)?kernel(?:I(\w+)E)?E", k) for k in kernels]
        out.append(" ".join((m[1] or "first_")[:-1] + " " + ",".join(re.findall(r"L[ib](\d+)E", m[2] + "E")) for m in names if m[1] != "finish_"))
    return out


def test_wide_matrices_take_the_kernel_of_many_rows(tmp_path):
    """Shapes for which the estimates once favoured a kernel that is up to 1.23 times slower there."""
    products = [(704, 22144, 64, 128, [3, 5, 6], 110, 0), (2304, 25856, 128, 128, [2, 3, 4], 53, 0), (6400, 22784, 128, 128, [4], 63, 0),
                (1536, 25088, 128, 128, [1, 2, 3, 4, 8], 98, 0), (2304, 24832, 32, 128, [2, 3, 4], 61, 0), (1088, 28160, 32, 128, [0, 1, 2, 3, 4], 115, 0)]
    for product, kernels in zip(products, launched(tmp_path, products)):
        assert kernels.startswith("many "), (product, kernels)


def test_products_with_codes_of_1_bit_take_the_faster_kernel(tmp_path):
    """33 to 64 rows whose codes of 1 bit enter as 1 + q / 2: in the narrow kernel or in that of many rows, by their times; 128 + q stays in the latter."""
    products = [(19968, 8576, 64, 64, [1, 2, 3, 4], 42, 0), (6368, 2624, 32, 64, [1, 2, 3, 4], 33, 0), (1984, 14336, 32, 128, [1, 2, 3, 4], 44, 0),
                (96, 640, 32, 64, [1, 4], 40, 0), (14304, 4032, 32, 64, [0, 1, 2, 3, 4], 62, 0), (14304, 4032, 32, 64, [0, 2, 3, 4], 62, 0)]
    kinds = [k.split(" ")[0] + k[-1] for k in launched(tmp_path, products)]
    assert kinds == ["many1", "many1", "many1", "narrow1", "many0", "many0"]


def test_cases_of_the_products_run_the_kernels_that_they_are_meant_for(tmp_path):
    """The tests of the products on the device, whose cases are chosen by kernel and instance: which one a product takes goes by estimates."""
    pytest.importorskip("torch")
    import test_gpu_mp_gemm_columns as columns
    import test_gpu_mp_gemm_edges as edges
    cases = edges.CASES + [case + (name,) for name, group in columns.CASES.items() for case in group]
    for case, kernels in zip(cases, launched(tmp_path, [case[:7] for case in cases])):
        assert kernels == case[7], case
    assert len(columns.CASES) == 20                          # (all instances)
