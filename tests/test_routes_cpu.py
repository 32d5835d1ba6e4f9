"""Which kernel a list takes: lists for which both kernels were timed, by what their plans counted, take the faster one, and a list
whose plan there was no memory for keeps a kernel that needs none.  Runs on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
M = 1_000_000


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "routes")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", os.path.join(ROOT, "tests", "sanitize", "routes_driver.cpp"), "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr

    def ask(*fields):
        res = subprocess.run([exe], input=" ".join(str(f) for f in fields) + "\n", capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        return res.stdout.strip()
    return ask


# rank, nonzeros, nonzeros per segment, different coordinates and common share of a sample, share of the segments that are cut up,
# and share of the nonzeros in them
@pytest.mark.parametrize("rank,nnz,per,distinct,common,cut,long,route", [
    (16, 11 * M, 20, 30_000, 1.0, 0.09, 0.33, "walk"),     # uneven rows over rows that an L2 holds: 100 us, and 112 on the pieces
    (16, 40 * M, 20, 59_000, 0.99, 0.09, 0.33, "walk"),    # 434 and 451
    (16, 34 * M, 13.5, 58_000, 0.85, 0.03, 0.14, "walk"),  # power-law columns: 290 and 357
    (16, 40 * M, 150, 30_000, 1.0, 0.73, 0.96, "walk"),    # 277 and 303
    (16, 22 * M, 9.4, 13_500, 0.97, 0.01, 0.03, "walk"),   # 203 and 213
    (16, 27 * M, 15, 85_700, 0.75, 0.03, 0.14, "walk"),    # power-law columns of a large operand: 0.90
    (16, 40 * M, 16, 106_000, 0.9, 0.05, 0.2, "pieces"),   # 608 and 603
    (16, 11 * M, 12, 24_000, 0.02, 0.02, 0.1, "pieces"),   # near the diagonal: 229 and 137
    (16, 24 * M, 9, 30_000, 1.0, 0.0, 0.0, "pieces"),      # rows of one length: 253 and 231
    (16, 40 * M, 3, 30_000, 1.0, 0.0, 0.0, "walk"),        # very many in short segments
    (16, 15 * M, 3, 30_000, 1.0, 0.0, 0.0, "pieces"),
    (16, 10 * M, 20, 30_000, 1.0, 0.09, 0.33, "pieces"),   # short lists
    (8, 40 * M, 20, 30_000, 1.0, 0.09, 0.33, "walk"),      # 295 and 309
    (8, 31 * M, 15, 62_000, 0.85, 0.05, 0.39, "walk"),     # power-law columns: 258 and 287
    (8, 11 * M, 20, 30_000, 1.0, 0.09, 0.33, "walk"),      # 90 and 91
    (8, 20 * M, 11.6, 3_429, 1.0, 0.03, 0.65, "pieces"),   # TTM over power-law fibers: 170 and 155
    (8, 10 * M, 20, 30_000, 1.0, 0.09, 0.33, "pieces"),
    (8, 40 * M, 32, 30_000, 1.0, 0.22, 0.56, "pieces"),    # 281 and 269
    (8, 40 * M, 20, 30_000, 1.0, 0.0, 0.0, "pieces"),      # 292 and 248
    (8, 40 * M, 16, 106_000, 0.9, 0.05, 0.2, "pieces"),    # 458 and 444
    (8, 40 * M, 3, 30_000, 1.0, 0.0, 0.0, "pieces"),
    (32, 40 * M, 20, 30_000, 1.0, 0.09, 0.33, "pieces"),
])
def test_segments_take_the_faster_kernel(routes, rank, nnz, per, distinct, common, cut, long, route):
    nseg = int(nnz / per)
    joins = int(cut * nseg)
    assert routes("segreduce", rank, nnz, nseg, nnz // 1400, distinct, common, joins, nseg - joins + int(long * nnz / 30)) == route


@pytest.mark.parametrize("rank,nnz,route", [(8, 11 * M, "walk"), (16, 11 * M, "walk"), (16, 10 * M, "pieces"), (32, 40 * M, "pieces")])
def test_segments_without_a_plan(routes, rank, nnz, route):
    """"pieces" means that the caller finds no plan and takes the kernels that need none."""
    assert routes("segreduce", rank, nnz, nnz // 30, 0, 0, 0.0, 0, 0) == route


POWER = (4_000, 13_500, 4 * M)                             # rows of C in 32768 nonzeros, rows of B in 32768 fibers, nonzeros of the longest slice
UNIFORM = {3_000: (3_000, 16_100, 790), 8_000: (7_900, 32_100, 1600), 15_000: (13_300, 16_100, 950), 30_000: (19_900, 28_000, 950),
           60_000: (25_300, 32_100, 1600), 300_000: (31_000, 16_100, 1750)}


@pytest.mark.parametrize("rank,power,r3,r8,r15,r30,r60,r300", [
    # faster on the wavefronts (w) or the walk (-), 44 M nonzeros; "?": within 2 %
    (9, "w", "w", "w", "w", "w", "?", "-"),
    (10, "w", "w", "w", "w", "w", "-", "-"),
    (15, "w", "?", "w", "w", "-", "-", "-"),
    (16, "w", "?", "?", "?", "-", "-", "?"),
    (20, "w", "w", "w", "w", "w", "?", "-"),
    (32, "w", "?", "?", "-", "-", "-", "-"),
    (34, "w", "-", "-", "-", "-", "-", "-"),
    (40, "w", "w", "w", "w", "-", "-", "-"),
    (62, "w", "w", "w", "-", "-", "-", "-"),
    (64, "w", "-", "w", "w", "w", "w", "?"),
    (96, "w", "?", "w", "w", "?", "-", "-"),
    (128, "w", "w", "w", "w", "w", "w", "-"),
])
def test_mttkrp_takes_the_faster_kernel(routes, rank, power, r3, r8, r15, r30, r60, r300):
    n = 44 * M
    facts = [(3.6, POWER), (2.25, UNIFORM[3_000]), (5, UNIFORM[8_000]), (3, UNIFORM[15_000]), (3, UNIFORM[30_000]), (5, UNIFORM[60_000]),
             (6, UNIFORM[300_000])]
    for want, (per, fact) in zip((power, r3, r8, r15, r30, r60, r300), facts):
        if want != "?":
            assert routes("mttkrp", rank, n, int(n / per), *fact) == ("wave" if want == "w" else "walk"), (rank, per, fact)


@pytest.mark.parametrize("rank,nnz,per,route", [
    (16, 150 * M, 4, "wave"), (64, 20 * M, 3.46, "wave"), (16, 41 * M, 3.6, "walk"), (10, 5 * M, 3, "walk"), (10, 6 * M, 3, "wave"), (20, 2_700_000, 3, "wave"),
    (20, 2_600_000, 3, "walk"), (32, 10 * M, 3, "walk"), (40, 1_100_000, 3, "wave"), (40, 1 * M, 3, "walk"), (8, 60 * M, 3, "walk"), (48, 60 * M, 3, "walk"),
    (33, 60 * M, 3, "walk"), (66, 60 * M, 3, "walk"), (10, 60 * M, 1.9, "walk"), (40, 60 * M, 8.1, "walk"), (10, 60 * M, 30, "wave")])
def test_mttkrp_by_size(routes, rank, nnz, per, route):
    assert routes("mttkrp", rank, nnz, int(nnz / per), *POWER) == route


def test_mttkrp_without_samples(routes):
    """A list whose plan there was no memory for counts as one whose rows come from memory."""
    for rank in range(1, 129):
        want = "wave" if 18 <= rank <= 30 and rank % 2 == 0 else "walk"
        assert routes("mttkrp", rank, 3 * M, M, 32768, 32768, 100_000) == want
        assert routes("mttkrp", rank, 44 * M, 11 * M, 32768, 32768, 100_000) == "walk"
