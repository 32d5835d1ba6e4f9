"""The MTTKRP walk on both tile sizes: fibers and slices that end just before, at and behind the boundaries of chunks of 1024
nonzeros, slices over few and over many of them, every lane-group layout, and lists on either side of the size rule."""
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


def _tensor(slices):
    """Slice s is stored at coordinate 2 s + 1; fiber f of a slice at 3 f; coordinates of a fiber are consecutive."""
    nfib = torch.tensor([len(s) for s in slices])
    lens = torch.tensor([n for s in slices for n in s])
    slice_of = torch.repeat_interleave(torch.arange(len(slices)), nfib)
    f_in = torch.arange(lens.numel()) - (torch.cumsum(nfib, 0) - nfib)[slice_of]
    fiber = torch.repeat_interleave(torch.arange(lens.numel()), lens)
    k = torch.arange(fiber.numel()) - (torch.cumsum(lens, 0) - lens)[fiber]
    dims = (2 * len(slices) + 1, 3 * int(nfib.max()), int(lens.max()))
    vals = gen.dense_operand(9, 0, (fiber.numel(), 1)).reshape(-1)
    return dims, (2 * slice_of + 1)[fiber].int(), (3 * f_in)[fiber].int(), k.int(), vals


def _check(comet, slices, R):
    dims, i, j, k, vals = _tensor(slices)
    print("mttkrp tiles R=%d nnz=%d" % (R, vals.numel()), flush=True)
    X = comet.from_levels(fmt.pack_csf3(dims, i, j, k, vals).to("cuda")).set_variant(2)
    B, C, old = (gen.dense_operand(5, n, (d, R)) for n, d in ((0, dims[1]), (1, dims[2]), (2, dims[0])))
    ref, absum = oracle.mttkrp(np_(i), np_(j), np_(k), np_(vals), dims, np_(B), np_(C))
    M = torch.full((dims[0], R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_mttkrp(X, 0, [None, B.to("cuda"), C.to("cuda")], M)
    assert_values_close(np_(M), ref, absum, "mttkrp R=%d" % R)
    assert torch.equal(M, comet.comet_mttkrp(X, 0, [None, B.to("cuda"), C.to("cuda")])), "two runs differ"
    D = old.to("cuda")
    comet.comet_mttkrp_axpby(X, 0, 0.75, [None, B.to("cuda"), C.to("cuda")], -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby R=%d" % R)


@pytest.mark.parametrize("R", [1, 3, 8, 10, 16, 20, 32, 33, 48, 64, 96, 128])
def test_edges_of_chunks(comet, R):
    _check(comet, EDGES, R)


@pytest.mark.parametrize("nnz", [LINE - 1, LINE])
def test_both_sides_of_the_size_rule(comet, nnz):
    each = [700, 3, 1, 5000, 40]
    n = nnz // sum(each)
    slices = [each] * n
    if nnz - n * sum(each):
        slices = slices + [[nnz - n * sum(each)]]
    _check(comet, slices, 10)
