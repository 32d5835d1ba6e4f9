"""SpMV with the sweep over long rows: long vectors on either side of the rule, an odd number of columns (the last interval of the
vector is ragged), rows around the sweep's length, rows cut into several units, pieces of one nonzero and of many, empty rows."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu

MIN_COLS = 5 << 17


def _line(ncols):
    """Nonzeros in rows of 128 and more from which on the sweep runs."""
    return 4 * ncols + (4 << 20)


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


def _matrix(ncols, clustered, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    lens = torch.cat([torch.tensor([0, 127, 128, 129, 4095, 4096, 4097, 8193, 60_000, 0, 1]), torch.randint(0, 127, (30_000,)),
                      torch.full((_line(ncols) // 900 + 50,), 900), torch.tensor([0, 5, 0])]).cuda()
    rows = torch.repeat_interleave(lens)
    # distinct columns of a row: its nonzeros in equal strides from a random start; clustered rows lie in an eighth of the columns
    k = torch.arange(rows.numel(), device="cuda") - (torch.cumsum(lens, 0) - lens)[rows]
    width = torch.full_like(lens, ncols)
    if clustered:
        width[torch.rand(lens.numel(), device="cuda", generator=g) < 0.05] = ncols // 8
    start = (torch.rand(lens.numel(), device="cuda", generator=g, dtype=torch.float64) * ncols).long()
    cols = (start[rows] + k * (width // lens.clamp(min=1))[rows]) % ncols
    keys = torch.sort(rows * ncols + cols).values
    rows, cols = torch.div(keys, ncols, rounding_mode="floor"), keys % ncols
    vals = torch.rand(rows.numel(), dtype=torch.float64, device="cuda", generator=g) * 2 - 1
    return lens.numel(), rows.int(), cols.int(), vals


@pytest.mark.parametrize("layout", ["csr", "dcsr"])
@pytest.mark.parametrize("ncols,clustered", [(MIN_COLS, False), (MIN_COLS - 1, False), (700_001, True), (MIN_COLS + 4099, False)])
def test_sweep_against_the_oracle(comet, layout, ncols, clustered):
    n, rows, cols, vals = _matrix(ncols, clustered, ncols)
    A = comet.from_levels((fmt.pack_csr if layout == "csr" else fmt.pack_dcsr)(n, ncols, rows, cols, vals))
    print("spmv sweep %s ncols=%d nnz=%d heavy=%s" % (layout, ncols, vals.numel(), A.heavy_plan()), flush=True)
    assert A.heavy_plan()[1] >= _line(ncols)           # so that the sweep runs from MIN_COLS columns on
    x = gen.dense_operand(3, 0, (ncols, 1)).reshape(-1)
    old = gen.dense_operand(4, 0, (n, 1)).reshape(-1)
    ref, absum = oracle.spmv(np_(rows), np_(cols), np_(vals), (n, ncols), np_(x))
    y = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmv(A, x.cuda(), y)
    assert_values_close(np_(y), ref, absum, "spmv sweep")
    for _ in range(3):
        assert torch.equal(y, comet.comet_spmv(A, x.cuda())), "two runs differ"
    # on the sweep the sums are formed in another order than in the plain kernel, which tells the two apart; below it they are the same
    plain = comet.comet_spmv(A.set_variant(3), x.cuda())
    A.set_variant(0)
    assert torch.equal(y, plain) == (ncols < MIN_COLS)
    z = old.cuda()
    comet.comet_spmv_axpby(A, 0.75, x.cuda(), -0.5, z)
    assert_values_close(np_(z), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "spmv sweep axpby")
    # a value that no nonzero reads must not reach the result, wherever the kernels touch the vector
    unused = torch.ones(ncols, dtype=torch.bool, device="cuda")
    unused[cols.long()] = False
    w = x.cuda()
    w[unused] = float("nan")
    w[0] = x[0] if not bool(unused[0]) else float("inf")
    assert torch.equal(y, comet.comet_spmv(A, w))


def test_order_of_the_sums_is_fixed(comet):
    """Sums that rounding tells apart: the nonzeros of a row are large and of both signs, so that another order of the additions
    gives another result.  The order is the program's, whatever else runs on the device."""
    n, rows, cols, vals = _matrix(MIN_COLS, True, 7)
    vals = torch.where(torch.arange(vals.numel(), device="cuda") % 3 == 0, 1e8, 1.0) * vals
    A = comet.from_levels(fmt.pack_csr(n, MIN_COLS, rows, cols, vals))
    x = gen.dense_operand(5, 0, (MIN_COLS, 1)).reshape(-1).cuda()
    y = comet.comet_spmv(A, x)
    side, noise = torch.cuda.Stream(), torch.ones(1 << 24, device="cuda")
    for _ in range(20):
        with torch.cuda.stream(side):
            noise = noise * 1.0000001
        assert torch.equal(y, comet.comet_spmv(A, x))
    side.synchronize()


def test_sweep_replays_from_a_captured_graph(comet):
    """After reserve a call only launches kernels; replays, with eager work between them, give the eager result bit for bit."""
    n, rows, cols, vals = _matrix(MIN_COLS, False, 8)
    A = comet.from_levels(fmt.pack_csr(n, MIN_COLS, rows, cols, vals))
    assert A.heavy_plan()[1] >= _line(MIN_COLS)
    A.reserve(1)
    x = gen.dense_operand(6, 0, (MIN_COLS, 1)).reshape(-1).cuda()
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        comet.comet_spmv(A, x, y)
    want = comet.comet_spmv(A, x)
    for rep in range(3):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), "replay %d differs from the eager result" % rep


@pytest.mark.parametrize("R", [1, 32])
def test_columns_in_any_order(comet, R):
    """The default creation does not check that the columns of a row increase.  Long rows in another order have no windows: the
    kernels that take any order run, and the result is right."""
    n, rows, cols, vals = _matrix(MIN_COLS, False, 9)
    lens = torch.bincount(rows.long(), minlength=n)
    end = torch.cumsum(lens, 0)
    p = torch.arange(rows.numel(), device="cuda")
    back = end[rows.long()] - 1 - (p - (end - lens)[rows.long()])           # every row back to front
    L = fmt.pack_csr(n, MIN_COLS, rows, cols, vals)
    L.crd[1], L.vals = cols[back].contiguous(), vals[back].contiguous()
    A = comet.from_levels(L, comet.COMET_BORROW)
    assert A.heavy_plan() == (0, 0)
    B = gen.dense_operand(3, 0, (MIN_COLS, R))
    got = comet.comet_spmv(A, B.reshape(-1).cuda()) if R == 1 else comet.comet_spmm(A, B.cuda())
    ref, absum = oracle.spmm(np_(rows), np_(cols), np_(vals), (n, MIN_COLS), np_(B))
    assert_values_close(np_(got).reshape(n, R), ref, absum, "columns back to front R=%d" % R)
