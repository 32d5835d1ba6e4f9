"""Performance cases of the sparse x dense contraction library: what its users have it do, over the real range.

A user keeps a tensor handle (level arrays and values resident in device memory) and calls one of the five
contractions on it again and again with dense operands: SpMV and SpMM in a solver or a feature propagation, TTV,
TTM and MTTKRP in a tensor decomposition.  The sizes are those of the library's own configurations (up to
10^6 x 10^6 matrices, tensors of 50 to 150 million nonzeros with power-law modes), smaller and odd ones between
them and the smallest calls, where a launch is most of the time.  Values are fp64 and indices int32, the only types
that the library has.

A case is a dict of plain values:
  op          spmv, spmm, ttv, ttm, mttkrp
  fmt         csr, dcsr (matrices); csf, coo (tensors)
  I, J, K     mode sizes (K: tensors only)
  nnz, fibers tensors: number of nonzeros and of different coordinates without the last level's, exactly
  a_i, a_j, a_k   tensors: Zipf exponent of the indices of a mode (0: uniform)
  row_alpha, row_cap   matrices: row lengths are min(Zipf(row_alpha), row_cap); row_alpha 0: every row has row_cap
  band        matrices: columns lie at most this far from the diagonal (0: anywhere)
  stored      matrices: share of the rows that have nonzeros at all
  R           columns of the dense operands
  mode        tensors: the mode that is contracted (ttv, ttm) or produced (mttkrp)
  accumulate  the product is added to half of the old result, in place
"""
import functools

import numpy as np
import torch

import paper_2102_05187_amd as comet

F64 = 8          # bytes of a value
I32 = 4          # bytes of an index
ALPHA, BETA = 0.75, 0.5


def _matrix(op, fmt, I, J, row_alpha, row_cap, R, band=0, stored=1.0, accumulate=False, **kw):
    return dict(kw, op=op, fmt=fmt, I=I, J=J, row_alpha=row_alpha, row_cap=row_cap, R=R, band=band, stored=stored,
                accumulate=accumulate)


def _tensor(op, fmt, dims, alphas, nnz, fibers, R, mode, accumulate=False, **kw):
    return dict(kw, op=op, fmt=fmt, I=dims[0], J=dims[1], K=dims[2], a_i=alphas[0], a_j=alphas[1], a_k=alphas[2],
                nnz=nnz, fibers=fibers, R=R, mode=mode, accumulate=accumulate)


def _order(case):
    """Modes of the levels: the produced mode first or the contracted one last."""
    mode = case["mode"]
    rest = [m for m in range(3) if m != mode]
    return [mode, *rest] if case["op"] == "mttkrp" else [*rest, mode]


def listed():
    return [
        # the smallest solver step: one SpMV of a few microseconds in a loop of many
        _matrix("spmv", "csr", 4096, 4096, 0, 10, 1, name="spmv_csr_4096"),
        # one step of a graph iteration on a power-law matrix whose vector fits no compute unit's LDS
        _matrix("spmv", "csr", 1_000_000, 1_000_000, 1.8, 10_000, 1, name="spmv_csr_1m"),
        # the smallest matrix with a block of vectors
        _matrix("spmm", "csr", 4096, 4096, 0, 10, 32, name="spmm_csr_4096_r32"),
        # the library's headline: a power-law matrix times a tall dense matrix (graph features, a block of vectors)
        _matrix("spmm", "csr", 1_000_000, 1_000_000, 1.8, 10_000, 32, name="spmm_csr_1m_r32"),
        # a matrix with local structure (a mesh in its natural numbering) and empty rows, stored doubly compressed;
        # a number of columns that is no power of two, added to the old result
        _matrix("spmm", "dcsr", 300_007, 270_011, 1.4, 500, 20, band=2000, stored=0.8, accumulate=True,
                name="spmm_dcsr_band_r20"),
        # tensor times vector at the size of the library's configuration
        _tensor("ttv", "csf", (20_000, 20_000, 20_000), (1.3, 1.3, 1.3), 50_000_000, 8_430_000, 1, 2,
                name="ttv_csf_50m"),
        # the same on a coordinate list as it comes from a file, of ordinary size, with a longer vector
        _tensor("ttv", "coo", (2003, 5003, 60_013), (1.3, 1.3, 1.2), 5_000_011, 637_003, 1, 2, name="ttv_coo_5m"),
        # one step of a Tucker decomposition at the size of the library's configuration
        _tensor("ttm", "csf", (200_000, 100_000, 5000), (1.5, 1.5, 0), 100_000_000, 6_520_000, 16, 2, name="ttm_csf_100m_r16"),
        # the same along the first mode (the tensor stored again for it), of ordinary size and with more columns
        _tensor("ttm", "csf", (30_011, 9001, 1009), (1.4, 1.4, 0), 8_000_009, 1_622_003, 32, 0,
                name="ttm_mode0_r32"),
        # one step of a CP decomposition at the size of the library's configuration: the largest pass
        _tensor("mttkrp", "csf", (2_000_000, 1_000_000, 20_000), (1.4, 1.4, 1.4), 150_000_000, 37_500_000, 16, 0,
                name="mttkrp_csf_150m_r16"),
        # the same for the second mode, of ordinary size and with a high rank
        _tensor("mttkrp", "csf", (700_001, 400_009, 9001), (1.4, 1.4, 1.4), 20_000_003, 5_776_001, 64, 1,
                name="mttkrp_mode1_r64"),
        # a decomposition of a small tensor with a rank that fits no vector width, added to the old result
        _tensor("mttkrp", "csf", (4001, 809, 211), (1.2, 1.2, 1.1), 100_003, 41_011, 10, 0, accumulate=True,
                name="mttkrp_small_r10"),
    ]


# ---- drawn cases ---------------------------------------------------------------------------------------------------
MOST_WORK = 150_000_000 * 16                 # nonzeros times columns of the largest listed case
RANKS = (8, 16, 16, 32, 32, 64)


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _columns(rng):
    """The number of dense columns: mostly the usual powers of two, else anything up to 64."""
    return rng.choice(RANKS) if rng.random() < 0.6 else rng.randint(2, 64)


def draw(rng):
    op = rng.choice(("spmv", "spmm", "ttv", "ttm", "mttkrp"))
    if op in ("spmv", "spmm"):
        I = _log(rng, 4000, 1_000_000)
        J = min(1_000_000, max(2000, int(I * rng.uniform(0.5, 2.0))))
        R = 1 if op == "spmv" else _columns(rng)
        fixed = rng.random() < 0.3
        band = 0 if rng.random() < 0.6 else _log(rng, 200, 20_000)
        cap = rng.randint(3, 40) if fixed else min(_log(rng, 100, 10_000), (2 * band if band else J) // 4)
        case = _matrix(op, rng.choice(("csr", "csr", "dcsr")), I, J, 0 if fixed else round(rng.uniform(1.5, 2.2), 2), cap, R,
                       band=band, stored=rng.choice((1.0, 1.0, round(rng.uniform(0.3, 1.0), 2))),
                       accumulate=rng.random() < 0.3)
        while _matrix_size(case)[1] * max(R, 16) > MOST_WORK // 2:
            case["I"] = case["I"] * 2 // 3
        return case
    R = 1 if op == "ttv" else _columns(rng)
    dims, alphas, full = {"ttv": ((20_000,) * 3, (1.3,) * 3, 50_000_000),
                          "ttm": ((200_000, 100_000, 5000), (1.5, 1.5, 0), 100_000_000),
                          "mttkrp": ((2_000_000, 1_000_000, 20_000), (1.4,) * 3, 150_000_000)}[op]
    # the configuration's tensor, made smaller in all modes; the smaller ones are less dense, as in use
    nnz = _log(rng, 100_000, min(full, MOST_WORK // R))
    scale = (nnz / full) ** 0.28
    dims = tuple(max(50, int(d * scale * rng.uniform(0.8, 1.3))) for d in dims)
    fmt, mode = "csf", 0 if op == "mttkrp" else 2
    if rng.random() < 0.3:
        mode = rng.randrange(3)
    elif rng.random() < 0.3:
        fmt = "coo"
    case = _tensor(op, fmt, dims, alphas, nnz, 0, R, mode, accumulate=op == "mttkrp" and rng.random() < 0.3)
    case["fibers"] = int(0.97 * _distinct(_draws(case), [_modes(case)[m] for m in _order(case)[:2]]))
    return case


# ---- inputs --------------------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _zipf_table(n, alpha):
    """CDF of the bounded Zipf law on 0 .. n-1 (host)."""
    c = np.cumsum(np.arange(1, n + 1, dtype=np.float64) ** -alpha)
    return c / c[-1]


def _rand(n, g):
    return torch.rand(n, dtype=torch.float64, device="cuda", generator=g)


def _dense(shape, g):
    return _rand(shape, g).mul_(2).sub_(1)


class _Mode:
    """Indices of one mode: Zipf over ranks, ranks scattered over the coordinates."""

    def __init__(self, size, alpha, g):
        self.size, self.table = size, None
        if alpha:
            self.table = torch.from_numpy(_zipf_table(size, alpha)).cuda()
            self.place = torch.randperm(size, device="cuda", generator=g)

    def draw(self, n, g):
        if self.table is None:
            return torch.randint(self.size, (n,), device="cuda", generator=g)
        return self.place[torch.searchsorted(self.table, _rand(n, g), right=True).clamp_(max=self.size - 1)]


def _coordinates(case, g):
    """Exactly nnz distinct coordinates of a tensor with exactly the stated number of fibers, sorted by mode 0, 1, 2."""
    dims, nnz, fibers, order = (case["I"], case["J"], case["K"]), case["nnz"], case["fibers"], _order(case)
    modes = [_Mode(dims[m], case[("a_i", "a_j", "a_k")[m]], g) for m in order]
    J, K = dims[order[1]], dims[order[2]]
    keys, chunk, found = torch.empty(0, dtype=torch.int64, device="cuda"), min(1 << 28, 6 * nnz), 0
    while found < fibers or keys.numel() - (found - fibers) < nnz:
        i, j, k = (m.draw(chunk, g) for m in modes)
        keys = torch.unique(torch.cat([keys, torch.unique(i.mul_(J).add_(j).mul_(K).add_(k))]))
        del i, j, k
        ij, size = torch.unique_consecutive(torch.div(keys, K, rounding_mode="floor"), return_counts=True)
        found = ij.numel()
    # fibers with one nonzero go until the number of fibers is right, then nonzeros that leave a fiber standing
    single = (size == 1).nonzero().flatten()
    gone = single[torch.randperm(single.numel(), device="cuda", generator=g)[:found - fibers]]
    first = torch.cumsum(size, 0) - size
    drop = torch.zeros(keys.numel(), dtype=torch.bool, device="cuda")
    drop[first[gone]] = True
    spare = torch.ones_like(drop)
    spare[first] = False
    spare = spare.nonzero().flatten()
    u = _rand(spare.numel(), g)
    drop[spare[u < u.sort().values[keys.numel() - (found - fibers) - nnz]]] = True
    keys = keys[~drop]
    out = [None] * 3
    out[order[2]], keys = keys % K, torch.div(keys, K, rounding_mode="floor")
    out[order[1]], out[order[0]] = keys % J, torch.div(keys, J, rounding_mode="floor")
    if order != [0, 1, 2]:
        by = torch.argsort((out[0] * dims[1] + out[1]) * dims[2] + out[2])
        out = [c[by] for c in out]
    return [c.int() for c in out]


def _starts(ids, n):
    """pos array of n segments from the sorted segment numbers of their members."""
    pos = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(ids, minlength=n), 0, out=pos[1:])
    return pos.int()


def _root(n):
    return torch.tensor([0, n], dtype=torch.int32, device="cuda")


def _csf(dims, i, j, k, vals):
    ij, fiber = torch.unique_consecutive(i.long() * dims[1] + j, return_inverse=True)
    crd0, slice_ = torch.unique_consecutive(torch.div(ij, dims[1], rounding_mode="floor"), return_inverse=True)
    return comet.comet_tensor_create(
        dims, [comet.COMET_CU] * 3, [_root(crd0.numel()), _starts(slice_, crd0.numel()), _starts(fiber, ij.numel())],
        [crd0.int(), (ij % dims[1]).int(), k], vals)


def _coo(dims, i, j, k, vals):
    return comet.comet_tensor_create(dims, [comet.COMET_CN, comet.COMET_S, comet.COMET_S],
                                     [_root(vals.numel()), None, None], [i, j, k], vals)


def _make_matrix(case, g):
    I, J, cap = case["I"], case["J"], case["row_cap"]
    if case["row_alpha"]:
        # the unbounded law cut off at the cap: the longest rows hold the whole tail
        table = torch.from_numpy(_zipf_table(50 * cap, case["row_alpha"])).cuda()
        lengths = (torch.searchsorted(table, _rand(I, g), right=True) + 1).clamp_(max=cap)
    else:
        lengths = torch.full((I,), cap, device="cuda")
    if case["stored"] < 1:
        lengths *= _rand(I, g) < case["stored"]
    rows = torch.repeat_interleave(lengths)
    if case["band"]:
        middle = torch.div(rows * J, I, rounding_mode="floor")
        cols = (middle + torch.randint(-case["band"], case["band"] + 1, (rows.numel(),), device="cuda", generator=g)).clamp_(0, J - 1)
    else:
        cols = torch.randint(J, (rows.numel(),), device="cuda", generator=g)
    keys = torch.unique(rows * J + cols)
    rows, cols = torch.div(keys, J, rounding_mode="floor"), (keys % J).int()
    vals = _dense(keys.numel(), g)
    if case["fmt"] == "csr":
        size = torch.tensor([I], dtype=torch.int32, device="cuda")
        return comet.comet_tensor_create((I, J), [comet.COMET_D, comet.COMET_CU], [size, _starts(rows, I)], [None, cols], vals)
    crd0, row = torch.unique_consecutive(rows, return_inverse=True)
    return comet.comet_tensor_create((I, J), [comet.COMET_CU] * 2, [_root(crd0.numel()), _starts(row, crd0.numel())],
                                     [crd0.int(), cols], vals)


class _View:
    """Memory of a result handle as torch sees it; the tensor made from it keeps the handle alive."""

    def __init__(self, Y, ptr, shape, typestr):
        self.owner = Y
        self.__cuda_array_interface__ = {"shape": shape, "typestr": typestr, "data": (ptr, False), "version": 2}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op, R = case["op"], case["R"]
    s = {"op": op, "accumulate": case["accumulate"]}
    if op in ("spmv", "spmm"):
        s["A"] = _make_matrix(case, g)
        s["B"] = _dense((case["J"],) if op == "spmv" else (case["J"], R), g)
        s["C"] = _dense((case["I"],) if op == "spmv" else (case["I"], R), g)
        return s
    dims, mode = (case["I"], case["J"], case["K"]), case["mode"]
    s["mode"] = mode
    order = _order(case)
    ijk = _coordinates(case, g)
    vals = _dense(case["nnz"], g)
    if case["fmt"] == "csf" and order == [0, 1, 2]:
        s["X"] = _csf(dims, *ijk, vals)
    else:
        s["X"] = _coo(dims, *ijk, vals)
        if order != [0, 1, 2]:
            s["X"] = comet.comet_tensor_reorder(s["X"], order)
    if op == "mttkrp":
        s["factors"] = [None if m == mode else _dense((dims[m], R), g) for m in range(3)]
        s["M"] = _dense((dims[mode], R), g)
        return s
    # the result's handle is made once, with a product that is zero, and written by every pass
    s["D"] = _dense((dims[mode],) if op == "ttv" else (dims[mode], R), g)
    call = comet.comet_ttv if op == "ttv" else comet.comet_ttm
    s["Y"] = call(s["X"], mode, torch.zeros_like(s["D"]))
    info = s["Y"].info()
    n = info.nvals // R
    s["out"] = [torch.as_tensor(_View(s["Y"], info.vals, (n,) if op == "ttv" else (n, R), "<f8"), device="cuda")]
    if case["fmt"] == "coo" and order == [0, 1, 2]:
        s["out"] += [torch.as_tensor(_View(s["Y"], info.crd[l], (n,), "<i4"), device="cuda") for l in range(2)]
    return s


def run(s):
    op = s["op"]
    if op == "ttv":
        comet.comet_ttv(s["X"], s["mode"], s["D"], s["Y"])
        return s["out"]
    if op == "ttm":
        comet.comet_ttm(s["X"], s["mode"], s["D"], s["Y"])
        return s["out"]
    if s["accumulate"]:
        if op == "spmv":
            return comet.comet_spmv_axpby(s["A"], ALPHA, s["B"], BETA, s["C"])
        if op == "spmm":
            return comet.comet_spmm_axpby(s["A"], ALPHA, s["B"], BETA, s["C"])
        return comet.comet_mttkrp_axpby(s["X"], s["mode"], ALPHA, s["factors"], BETA, s["M"])
    if op == "spmv":
        return comet.comet_spmv(s["A"], s["B"], s["C"])
    if op == "spmm":
        return comet.comet_spmm(s["A"], s["B"], s["C"])
    return comet.comet_mttkrp(s["X"], s["mode"], s["factors"], s["M"])


# ---- work ----------------------------------------------------------------------------------------------------------
def _bins(size, alpha):
    """A mode's indices in groups of about equal probability: (how many, the probability of one of them)."""
    if not alpha:
        return np.array([float(size)]), np.array([1.0 / size])
    edges = np.unique(np.round(np.geomspace(1, size + 1, 40)).astype(np.int64)) - 1
    total = np.concatenate([[0.0], _zipf_table(size, alpha)])
    count = np.diff(edges).astype(np.float64)
    return count, np.diff(total[edges]) / count


def _distinct(draws, modes):
    """Expected number of different coordinates among so many draws."""
    count = p = np.ones(1)
    for m in modes:
        n, q = _bins(*m)
        count, p = np.multiply.outer(count, n).ravel(), np.multiply.outer(p, q).ravel()
    return float((count * -np.expm1(-draws * p)).sum())


def _modes(case):
    return [(case["I"], case["a_i"]), (case["J"], case["a_j"]), (case["K"], case["a_k"])]


def _draws(case):
    """How many draws give nnz different coordinates."""
    lo, hi = float(case["nnz"]), 1000.0 * case["nnz"]
    for _ in range(40):
        mid = (lo * hi) ** 0.5
        lo, hi = (mid, hi) if _distinct(mid, _modes(case)) < case["nnz"] else (lo, mid)
    return lo


def _matrix_size(case):
    """Expected (stored rows, nonzeros, columns that occur)."""
    I, J, cap = case["I"], case["J"], case["row_cap"]
    if case["row_alpha"]:
        p = np.diff(_zipf_table(50 * cap, case["row_alpha"]), prepend=0.0)
        p = np.append(p[:cap - 1], p[cap - 1:].sum())
    else:
        p = np.append(np.zeros(cap - 1), 1.0)
    width = min(J, 2 * case["band"] + 1) if case["band"] else J
    length = float((p * width * -np.expm1(np.arange(1, cap + 1) * np.log1p(-1.0 / width))).sum())
    rows = I * case["stored"]
    return rows, rows * length, J * -np.expm1(-rows * length / J)


def work(case):
    """Each level array, value and touched operand row read once, each result element written once."""
    R = case["R"]
    if case["op"] in ("spmv", "spmm"):
        rows, nnz, cols = _matrix_size(case)
        levels = I32 * (case["I"] if case["fmt"] == "csr" else 2 * rows) + (I32 + F64) * nnz
        result = F64 * R * case["I"] * (2 if case["accumulate"] else 1)
        return {"bytes": levels + F64 * R * cols + result, "flops": 2 * R * nnz}
    nnz, fibers, mode = case["nnz"], case["fibers"], case["mode"]
    sizes, draws = _modes(case), _draws(case)
    seen = [_distinct(draws, [m]) for m in sizes]
    if case["op"] == "mttkrp":
        levels = (I32 + F64) * nnz + 2 * I32 * (fibers + seen[mode])
        operands = F64 * R * (sum(seen) - seen[mode])
        result = F64 * R * sizes[mode][0] * (2 if case["accumulate"] else 1)
        return {"bytes": levels + operands + result, "flops": 2 * R * (nnz + fibers)}
    if case["fmt"] == "coo":                              # the result's coordinates are written too
        levels = (3 * I32 + F64) * nnz + 2 * I32 * fibers
    else:
        levels = (I32 + F64) * nnz + I32 * fibers
    return {"bytes": levels + F64 * R * (fibers + seen[mode]), "flops": 2 * R * nnz}


def tolerance(case):
    """64-bit sums in any order; every other correct order stays well within this."""
    return {"rel": 1e-12, "max": 1e-10}
