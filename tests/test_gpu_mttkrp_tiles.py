"""MTTKRP on its tile sizes: fibers and slices that end just before, at and behind the boundaries of chunks of 1024
nonzeros, slices over few and over many of them, every lane-group layout, lists on either side of the size rules, and fibers
and slices without nonzeros between the pieces' tiles."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu

LINE = 3 << 20                 # nonzeros from which on the tiles hold 4096
# fibers of each slice
EDGES = [[1023], [1], [1024], [1025], [15, 16, 17, 31, 32, 33, 63, 64], [1] * 40, [3000, 2, 5], [1] * 1500, [30000], [7] * 5000, [2, 1021], [1]]


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


def _tensor(slices, root=None):
    """Slice s is stored at coordinate 2 s + 1, or at root[s] of root[-1] rows; fiber f of a slice at 3 f; coordinates of a fiber are
    consecutive.  Half of the rows are stored, which is when the others are cleared one by one."""
    nfib = torch.tensor([len(s) for s in slices])
    lens = torch.tensor([n for s in slices for n in s])
    slice_of = torch.repeat_interleave(torch.arange(len(slices)), nfib)
    f_in = torch.arange(lens.numel()) - (torch.cumsum(nfib, 0) - nfib)[slice_of]
    fiber = torch.repeat_interleave(torch.arange(lens.numel()), lens)
    k = torch.arange(fiber.numel()) - (torch.cumsum(lens, 0) - lens)[fiber]
    root = torch.cat([2 * torch.arange(len(slices)) + 1, torch.tensor([2 * len(slices)])]) if root is None else torch.tensor(root)
    dims = (int(root[-1]), 3 * int(nfib.max()), int(lens.max()))
    vals = gen.dense_operand(9, 0, (fiber.numel(), 1)).reshape(-1)
    return dims, root[slice_of][fiber].int(), (3 * f_in)[fiber].int(), k.int(), vals


def _check(comet, slices, R, variant=2, root=None):
    dims, i, j, k, vals = _tensor(slices, root)
    print("mttkrp tiles R=%d nnz=%d" % (R, vals.numel()), flush=True)
    X = comet.from_levels(fmt.pack_csf3(dims, i, j, k, vals).to("cuda")).set_variant(variant)
    B, C, old = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2]), (2, dims[0])))
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(B), np_(C))
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, [None, B.to("cuda"), C.to("cuda")], M)
    assert_values_close(np_(M), ref, absum, "mttkrp R=%d" % R)
    assert torch.equal(M, comet.comet_mttkrp(X, 0, [None, B.to("cuda"), C.to("cuda")])), "two runs differ"
    D = old.to("cuda")
    comet.comet_mttkrp_axpby(X, 0, 0.75, [None, B.to("cuda"), C.to("cuda")], -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby R=%d" % R)


@pytest.mark.parametrize("variant", [2, 3])                              # pieces up to rank 33, and the walk
@pytest.mark.parametrize("R", [1, 3, 8, 10, 16, 20, 32, 33, 48, 64, 96, 128])
def test_edges_of_chunks(comet, R, variant):
    _check(comet, EDGES, R, variant)


@pytest.mark.parametrize("variant", [2, 3])                              # the line is the walk's; at this rank pieces take both sides
@pytest.mark.parametrize("nnz", [LINE - 1, LINE])
def test_both_sides_of_the_size_rule(comet, nnz, variant):
    each = [700, 3, 1, 5000, 40]
    n = nnz // sum(each)
    slices = [each] * n
    if nnz - n * sum(each):
        slices = slices + [[nnz - n * sum(each)]]
    _check(comet, slices, 10, variant)


# nonzeros up to which lists take the pieces, by what the rule sees: short slices of several nonzeros per fiber, the same behind a
# slice cut over many tiles, and a nonzero per fiber
LINES = [("short", 8, 25 << 15), ("short", 16, 25 << 14), ("short", 33, 3 << 18), ("short", 20, 9 << 18), ("short", 9, 9 << 18), ("short", 6, 5 << 20),
         ("long", 8, 9 << 18), ("long", 32, 9 << 17), ("long", 11, 5 << 18), ("ones", 10, 3 << 18), ("ones", 33, 1 << 18), ("ones", 24, 3 << 18)]


@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("shape,R,line", LINES)
def test_both_sides_of_the_rules_for_pieces(comet, shape, R, line, more):
    each = [1] * 7 if shape == "ones" else [40, 3, 1, 500, 17, 16, 1]
    first = [[300] * 100] if shape == "long" else []                    # 30 chunks
    rest = line + more - sum(map(sum, first))
    n = rest // sum(each)
    _check(comet, first + [each] * n + ([[rest - n * sum(each)]] if rest - n * sum(each) else []), R)


@pytest.mark.parametrize("variant", [2, 3])
@pytest.mark.parametrize("R", [1, 6, 10, 16, 35])
@pytest.mark.parametrize("longest", [40, 600])
def test_rows_between_stored_slices(comet, R, longest, variant):
    """Rows that are not stored, in runs of 1, 2, 40 and more, in front of the first slice, behind the last, and in front of slices of
    every kind: in one record, in several (more than 16 pieces), cut by a tile boundary, over many tiles.  With beta each of them has
    to be scaled exactly once, and an infinite alpha must not reach them.  (longest 600: too long a run for the kernel over pieces
    to clear at ranks from 10 on.)"""
    kinds = [[3], [1] * 20, [40, 1, 2], [1] * 50, [300, 7], [17, 16, 33, 1], [1], [2] * 200]
    slices = [kinds[(s * s + s // 3) % len(kinds)] for s in range(1200)] + [[500] * 40, [1] * 3, [90] * 9]
    gaps = [longest if s == 77 else 40 if s == 400 else (0, 0, 1, 0, 2, 0, 0)[s % 7] for s in range(len(slices))]
    gaps[0], gaps[-3] = 3, 2
    root, at = [], -1
    for gap in gaps:
        at += gap + 1
        root.append(at)
    root.append(at + 1 + 5)                                             # rows of M
    assert 2 * len(slices) >= root[-1]
    _check(comet, slices, R, variant, root)
    dims, i, j, k, vals = _tensor(slices, root)
    X = comet.from_levels(fmt.pack_csf3(dims, i, j, k, vals).to("cuda")).set_variant(variant)
    B, C, old = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2]), (2, dims[0])))
    D = old.to("cuda")
    comet.comet_mttkrp_axpby(X, 0, float("inf"), [None, B.to("cuda"), C.to("cuda")], -0.5, D)
    none = np.ones(dims[0], dtype=bool)
    none[root[:-1]] = False
    assert np.array_equal(np_(D)[none], -0.5 * np_(old)[none])


@pytest.mark.parametrize("R", [1, 6, 16, 35])
@pytest.mark.parametrize("stored_every", [1, 3])
def test_fibers_and_slices_without_nonzeros(comet, R, stored_every):
    """Runs of empty fibers and of slices without fibers, long enough to fill tiles of the pieces, at either end and between
    nonzeros; with the rows behind the last slice cleared by a gap (1), or all rows together (3).  An infinite alpha must not
    reach rows that receive nothing."""
    g = torch.Generator().manual_seed(R)
    slices = []
    for n in (0, 0, 700, 1, 0, 40, 5, 0, 300, 2000, 0):
        slices.append([0] * n)                                          # empty fibers only, or no fiber at all
        slices.append([0] * 130 + [int(x) for x in torch.randint(0, 40, (60,), generator=g)] + [0] * (n % 200))
        slices.append([])
        slices += [[1], [0, 1], [1, 0]] * 25
    slices.append([])
    nfib = torch.tensor([len(x) for x in slices])
    lens = torch.tensor([n for x in slices for n in x])
    pos2 = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(nfib, 0)]).int()
    pos3 = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lens, 0)]).int()
    crd1 = (stored_every * torch.arange(len(slices)) + stored_every - 1).int()
    crd2 = (torch.arange(lens.numel()) - (torch.cumsum(nfib, 0) - nfib).repeat_interleave(nfib)).int()
    fiber = torch.repeat_interleave(torch.arange(lens.numel()), lens)
    k = (torch.arange(fiber.numel()) - (torch.cumsum(lens, 0) - lens)[fiber]).int()
    i = crd1[torch.repeat_interleave(torch.arange(len(slices)), nfib)[fiber]]
    dims = (stored_every * len(slices) + 4, int(nfib.max()) + 1, int(lens.max()) + 1)
    vals = gen.dense_operand(3, 1, (fiber.numel(), 1)).reshape(-1)
    print("mttkrp empties R=%d every=%d nnz=%d fibers=%d" % (R, stored_every, vals.numel(), lens.numel()), flush=True)
    d = lambda t: t.to("cuda").contiguous()
    X = comet.comet_tensor_create(dims, [comet.COMET_CU] * 3, [d(torch.tensor([0, len(slices)], dtype=torch.int32)), d(pos2), d(pos3)],
                                  [d(crd1), d(crd2), d(k)], d(vals)).set_variant(2)
    B, C, old = (gen.dense_operand(5, n, (e, R)) for n, e in ((0, dims[1]), (1, dims[2]), (2, dims[0])))
    ref, absum = oracle.mttkrp(np_(i), np_(crd2[fiber]), np_(k), np_(vals), dims, np_(B), np_(C))
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, [None, d(B), d(C)], M)
    assert_values_close(np_(M), ref, absum, "empties R=%d" % R)
    D = old.to("cuda")
    comet.comet_mttkrp_axpby(X, 0, 0.75, [None, d(B), d(C)], -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "empties axpby R=%d" % R)
    if stored_every == 1:
        D = old.to("cuda")
        comet.comet_mttkrp_axpby(X, 0, float("inf"), [None, d(B), d(C)], -0.5, D)
        none = np.ones(dims[0], dtype=bool)
        none[np_(i)] = False
        assert np.array_equal(np_(D)[none], -0.5 * np_(old)[none])


@pytest.mark.parametrize("values", [1 << 29, 1 << 32])
@pytest.mark.parametrize("level", [1, 2])
@pytest.mark.parametrize("R", [4, 5])
def test_factors_whose_offsets_leave_32_bits(comet, R, level, values):
    """A factor just above 2^29 values (row offsets in bytes) and 2^32 values (in doubles), its first and last rows among
    those that are read."""
    wide = values // R + 3
    dims = (50, 7, 9)
    g = torch.Generator().manual_seed(R)
    i, j, k = torch.meshgrid(torch.arange(dims[0]), torch.arange(dims[1]), torch.arange(dims[2]), indexing="ij")
    keep = torch.rand(i.shape, generator=g) < 0.6
    i, j, k = (x[keep].int() for x in (i, j, k))
    vals = torch.rand(i.numel(), dtype=torch.float64, generator=g) * 2 - 1
    spread = torch.linspace(0, wide - 1, dims[level], dtype=torch.float64).long()        # where the coordinates of the level go
    spread[-1] = wide - 1
    far = spread[(j if level == 1 else k).long()].int()
    tdims = (dims[0], wide, dims[2]) if level == 1 else (dims[0], dims[1], wide)
    X = comet.from_levels(fmt.pack_csf3(tdims, i, far if level == 1 else j, far if level == 2 else k, vals).to("cuda")).set_variant(2)
    small = [gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2]))]
    F = torch.empty((wide, R), dtype=torch.float64, device="cuda")
    F[spread.cuda()] = small[level - 1].cuda()
    BC = [s.cuda() for s in small]
    BC[level - 1] = F
    print("mttkrp wide factor R=%d level=%d rows=%d nnz=%d" % (R, level, wide, vals.numel()), flush=True)
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, [None] + BC, M)
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(small[0]), np_(small[1]))
    assert_values_close(np_(M), ref, absum, "wide factor R=%d level=%d" % (R, level))


@pytest.mark.parametrize("R", [1, 7, 16, 20, 33, 42, 64, 100, 128])
def test_slices_over_many_tiles_of_the_walk(comet, R):
    """Slices cut over 64 and more tiles of the walk, whose partial sums a workgroup adds up per block of 16 columns: at ranks
    whose last block leaves threads idle, at several slices in a row, and with short slices between them."""
    long_slice = [300] * 280                                            # 84 000 nonzeros: 82 chunks of 1024
    slices = [long_slice, [1], long_slice, [7, 2000, 1], long_slice, long_slice, [3] * 300, [66_000], long_slice * 2, [1023], long_slice * 3, [5]]
    assert sum(map(sum, slices)) < LINE                                 # in chunks
    _check(comet, slices, R, 3)


@pytest.mark.parametrize("op", ["ttv", "ttv_coo", "spmv"])
def test_chains_over_many_tiles_at_rank_one(comet, op):
    """Segments of 64 and more tiles of 4096 nonzeros, one behind the other and with short ones between them, on a vector that
    does not fit LDS: every one ends among the tiles of another workgroup of the fix-up, wherever it begins."""
    n = 400_003
    lens = [280_000, 5, 262_144, 262_145, 1, 399_999, 4096, 300_000, 300_000, 12_000, 2]
    rows = torch.repeat_interleave(torch.arange(len(lens)), torch.tensor(lens))
    cols = torch.cat([torch.arange(m) for m in lens])
    vals = gen.dense_operand(7, 0, (rows.numel(), 1)).reshape(-1)
    x = gen.dense_operand(7, 1, (n, 1)).reshape(-1)
    print("chains %s nnz=%d" % (op, vals.numel()), flush=True)
    ref, absum = oracle.spmv(np_(rows), np_(cols), np_(vals), (len(lens), n), np_(x))
    if op == "spmv":
        A = comet.from_levels(fmt.pack_csr(len(lens), n, rows.int(), cols.int(), vals).to("cuda"), comet.COMET_LEAN).set_variant(2)
        got = comet.comet_spmv(A, x.cuda())
        y = torch.ones(len(lens), dtype=torch.float64, device="cuda")
        comet.comet_spmv_axpby(A, 0.5, x.cuda(), 2.0, y)
        assert_values_close(np_(y), 0.5 * ref + 2.0, 0.5 * absum + 2.0, "chains axpby")
    else:
        dims = (1, len(lens), n)
        i = torch.zeros_like(rows).int()
        T = fmt.pack_csf3(dims, i, rows.int(), cols.int(), vals) if op == "ttv" else fmt.pack_coo(dims, (i, rows.int(), cols.int()), vals)
        got = comet.comet_ttv(comet.from_levels(T.to("cuda")).set_variant(2), 2, x.cuda()).vals()
    assert_values_close(np_(got), ref, absum, "chains %s" % op)
