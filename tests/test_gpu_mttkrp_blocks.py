"""MTTKRP on lists long enough for wavefronts that take blocks of nonzeros: fibers and slices that end at every place of a block, a
lane group and a run of 1024 nonzeros, blocks with as many fibers or slices as nonzeros, every layout of the rows, operands whose row
offsets need 64 bits; and lists that keep the walk over nonzeros: below the sizes, with rows of C spread over more than the caches hold, with an empty
fiber or slice.  Which of the two ran shows in the last bits: they add in different orders, and the walk is what variant 3 takes."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


def _lists(nnz):
    """Fiber lengths and the fibers of each slice: 2 to 8 nonzeros per fiber in all, exactly nnz of them."""
    g = np.random.default_rng(7)
    fibers, slices = [], []

    def add(of):
        slices.append(len(of))
        fibers.extend(of)

    total = 0
    while total < nnz:
        start = len(fibers)
        for n in (1023, 1024, 1025, 31, 32, 33, 63, 64, 65, 7, 8, 9):
            add([n])                                                    # a slice of one fiber
        add([1] * 700)                                                  # as many fibers as nonzeros, no slice ends for 700
        for _ in range(400):
            add([1])                                                    # every nonzero is a slice
        for _ in range(150):
            add(list(g.integers(1, 4, int(g.integers(1, 6)))))          # several slices in a lane group
        add([64] * 40 + [1] * 130 + [8] * 300 + [16] * 64)
        add(list(g.integers(1, 12, 3000)))                              # one slice over many runs
        add(list(g.integers(1, 12, int(g.integers(100, 400)))))
        total += sum(fibers[start:])
    over = total - nnz
    while over:
        cut = min(over, fibers[-1] - 1) if slices[-1] == 1 or fibers[-1] > 1 else 0
        if cut:
            fibers[-1] -= cut
            over -= cut
        elif slices[-1] > 1:
            fibers.pop()
            slices[-1] -= 1
            over -= 1
        else:
            fibers.pop()
            slices.pop()
            over -= 1
    assert sum(fibers) == nnz and 2 * len(fibers) <= nnz <= 8 * len(fibers)
    return torch.tensor(np.array(fibers)), torch.tensor(slices)


def _tensor(nnz, spread):
    """Fibers begin at one of `spread` different rows of C."""
    lens, nfib = _lists(nnz)
    fiber = torch.repeat_interleave(torch.arange(lens.numel()), lens)
    slice_of = torch.repeat_interleave(torch.arange(nfib.numel()), nfib)
    j = torch.arange(lens.numel()) - (torch.cumsum(nfib, 0) - nfib)[slice_of]
    k = torch.arange(fiber.numel()) - (torch.cumsum(lens, 0) - lens)[fiber] + fiber * 7 % spread
    dims = (nfib.numel() * 4 // 3 + 5, int(nfib.max()) + 2, int(lens.max()) + spread)
    i = slice_of + slice_of // 3                                        # three of four rows are stored
    return dims, i[fiber].int(), j[fiber].int(), k.int(), gen.dense_operand(9, 0, (nnz, 1)).reshape(-1)


_kept = {}


def _case(nnz, spread=6000):
    if (nnz, spread) not in _kept:
        _kept.clear()
        _kept[nnz, spread] = _tensor(nnz, spread)
    return _kept[nnz, spread]


SMALL = 1 << 20                                                         # from here on at even ranks above 32
NEAR, FAR = 6000, 40000
CASES = [(SMALL, NEAR, 34, True), (SMALL, NEAR, 44, True), (SMALL + 1, NEAR, 40, True), (SMALL + 63, NEAR, 50, True), (SMALL + 700, NEAR, 62, True),
         (SMALL - 1, NEAR, 40, False), (SMALL, FAR, 40, False), (SMALL, FAR, 62, False),
         (5 << 19, NEAR, 20, True), ((5 << 19) + 31, NEAR, 30, True), ((5 << 19) - 1, NEAR, 20, False),
         ((5 << 20) + 1, NEAR, 9, True), ((5 << 20) + 1, NEAR, 10, True), ((5 << 20) + 1, NEAR, 15, True), ((5 << 20) + 1, FAR, 10, False),
         ((10 << 20) + 5, 9000, 32, True), ((10 << 20) + 5, 9000, 64, True), ((10 << 20) + 5, 9000, 96, True), ((10 << 20) + 5, 9000, 128, True),
         ((10 << 20) + 5, FAR, 32, False), ((40 << 20) + 1, NEAR, 16, True), ((40 << 20) - 1, NEAR, 16, False)]


@pytest.mark.parametrize("nnz,spread,R,blocks", CASES)
def test_blocks(comet, nnz, spread, R, blocks):
    dims, i, j, k, vals = _case(nnz, spread)
    print("mttkrp blocks R=%d nnz=%d spread=%d" % (R, nnz, spread), flush=True)
    T = fmt.pack_csf3(dims, i, j, k, vals).to("cuda")
    X, plain = comet.from_levels(T).set_variant(2), comet.from_levels(T).set_variant(3)
    B, C, old = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2]), (2, dims[0])))
    factors = [None, B.to("cuda"), C.to("cuda")]
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(B), np_(C))
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, factors, M)
    assert_values_close(np_(M), ref, absum, "mttkrp R=%d" % R)
    assert torch.equal(M, comet.comet_mttkrp(X, 0, factors)), "two runs differ"
    assert torch.equal(M, comet.comet_mttkrp(plain, 0, factors)) != blocks
    D = old.to("cuda")
    comet.comet_mttkrp_axpby(X, 0, 0.75, factors, -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby R=%d" % R)


@pytest.mark.parametrize("level", [1, 2])
@pytest.mark.parametrize("nnz,R", [(SMALL, 34), ((5 << 20) + 1, 11)])
def test_row_offsets_beyond_4_gib(comet, nnz, R, level):
    """The coordinates of a level spread over more than 4 GiB of operand rows, the last row among them."""
    dims, i, j, k, vals = _case(nnz)
    wide = (1 << 29) // R + 7
    spread = torch.linspace(0, wide - 1, dims[level], dtype=torch.float64).long()
    spread[-1] = wide - 1
    crd = [i, j, k]
    crd[level] = spread[crd[level].long()].int()
    tdims = list(dims)
    tdims[level] = wide
    X = comet.from_levels(fmt.pack_csf3(tdims, *crd, vals).to("cuda")).set_variant(2)
    small = [gen.dense_operand(5, n, (dims[n + 1], R)) for n in (0, 1)]
    F = torch.empty((wide, R), dtype=torch.float64, device="cuda")
    F[spread.cuda()] = small[level - 1].cuda()
    BC = [s.cuda() for s in small]
    BC[level - 1] = F
    print("mttkrp blocks wide R=%d level=%d rows=%d" % (R, level, wide), flush=True)
    M = comet.comet_mttkrp(X, 0, [None] + BC)
    assert not torch.equal(M, comet.comet_mttkrp(X.set_variant(3), 0, [None] + BC))
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(small[0]), np_(small[1]))
    assert_values_close(np_(M), ref, absum, "wide R=%d level=%d" % (R, level))


@pytest.mark.parametrize("empty", ["fiber", "slice"])
def test_lists_with_something_empty(comet, empty):
    """One fiber, or slice, without nonzeros behind the others: its row receives nothing."""
    dims, i, j, k, vals = _case(SMALL)
    R = 34
    T = fmt.pack_csf3(dims, i, j, k, vals)
    last_row = int(T.crd[0][-1])
    if empty == "fiber":
        T.crd[1] = torch.cat([T.crd[1], torch.tensor([dims[1] - 1], dtype=torch.int32)])
        T.pos[2] = torch.cat([T.pos[2], T.pos[2][-1:]])
        T.pos[1][-1] += 1
    else:
        T.crd[0] = torch.cat([T.crd[0], torch.tensor([last_row + 1], dtype=torch.int32)])
        T.pos[1] = torch.cat([T.pos[1], T.pos[1][-1:]])
        T.pos[0][-1] += 1
    X = comet.from_levels(T.to("cuda")).set_variant(2)
    B, C = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2])))
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(B), np_(C))
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, [None, B.to("cuda"), C.to("cuda")], M)
    assert_values_close(np_(M), ref, absum, "empty %s" % empty)
    assert torch.equal(M, comet.comet_mttkrp(X.set_variant(3), 0, [None, B.to("cuda"), C.to("cuda")]))


def test_reserved_scratch_serves_every_rank(comet):
    """After reserve the calls of every rank up to it allocate nothing (a capture would refuse that), whichever kernel each takes."""
    dims, i, j, k, vals = _case((5 << 20) + 1)
    T = fmt.pack_csf3(dims, i, j, k, vals).to("cuda")
    X, fresh = comet.from_levels(T).set_variant(2), comet.from_levels(T).set_variant(2)
    X.reserve(62)
    ranks = (2, 9, 10, 16, 20, 34, 40, 62)
    factors = {R: [None] + [gen.dense_operand(5, n, (d, R)).cuda() for n, d in ((0, dims[1]), (1, dims[2]))] for R in ranks}
    out = {R: torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda") for R in ranks}
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        for R in ranks:
            comet.comet_mttkrp(X, 0, factors[R], out[R])
    want = {R: comet.comet_mttkrp(fresh, 0, factors[R]) for R in ranks}
    for rep in range(3):
        for R in ranks:
            out[R].fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for R in ranks:
            assert torch.equal(out[R], want[R]), "replay %d rank %d" % (rep, R)


def test_reserve_takes_what_the_routes_need(comet):
    """32 M nonzeros, 30 per fiber, and a fiber without any, so that no rank is taken by blocks: the pieces of TTM need most, 46 MB at
    rank 128.  A summary per 1024 nonzeros would be 64."""
    n, per = 32_000_000, 30
    fibers = n // per
    i32 = dict(dtype=torch.int32, device="cuda")
    fiber_ends = torch.cat([torch.arange(fibers + 1, **i32) * per, torch.tensor([fibers * per], **i32)])
    slices = 1000
    slice_ends = torch.arange(slices + 1, **i32) * (fibers // slices)
    slice_ends[-1] = fibers + 1
    k = torch.arange(fibers * per, **i32) % per
    j = torch.arange(fibers + 1, **i32)
    X = comet.comet_tensor_create((slices, fibers + 1, per), [comet.COMET_CU] * 3, [torch.tensor([0, slices], **i32), slice_ends, fiber_ends],
                                  [torch.arange(slices, **i32), j, k], torch.ones(fibers * per, dtype=torch.float64, device="cuda"), comet.COMET_VALIDATE | comet.COMET_LEAN)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    X.reserve(128)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < 55 << 20


@pytest.mark.parametrize("variant", [2, 3])
@pytest.mark.parametrize("nnz,R", [(300_001, 20), (SMALL + 63, 50), ((5 << 19) + 31, 20), ((5 << 20) + 1, 11)])
def test_factors_that_are_not_finite(comet, nnz, R, variant):
    """Blocks, pieces (the shortest list) and the walk.  Slices that name no such row have the result that they have without it, bit for
    bit, though kernels load row 0 of C and the last fiber's row of B behind the list's end; the others infinity where all products are positive, and
    else something that is not finite (which depends on what is added up before it is multiplied)."""
    dims, i, j, k, vals = _case(nnz)
    print("mttkrp not finite R=%d nnz=%d variant=%d" % (R, nnz, variant), flush=True)
    B, C = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2])))
    last = int(j[-1])
    for positive in (True, False):
        v, b, c = (x.abs() + 0.1 if positive else x for x in (vals, B, C))
        X = comet.from_levels(fmt.pack_csf3(dims, i, j, k, v).to("cuda")).set_variant(variant)
        want = comet.comet_mttkrp(X, 0, [None, b.cuda(), c.cuda()])
        for what in ("B", "C"):
            bad_b, bad_c = b.clone(), c.clone()
            if what == "B":
                bad_b[[last, 2500]] = float("inf")
                names = (j == last) | (j == 2500)
            else:
                bad_c[[0, 1234]] = float("inf")
                names = (k == 0) | (k == 1234)
            rows = torch.zeros(dims[0], dtype=torch.bool)
            rows[i[names].long().unique()] = True
            assert rows.any() and not rows.all()
            M = comet.comet_mttkrp(X, 0, [None, bad_b.cuda(), bad_c.cuda()])
            assert torch.equal(M[~rows.cuda()], want[~rows.cuda()]), what
            hit = M[rows.cuda()]
            assert bool((hit == float("inf")).all() if positive else (~torch.isfinite(hit)).all()), what
