"""SpMM at ranks 8 and 16 over lists that a walk over tiles of 4096 nonzeros takes, because their rows differ in length and all
parts of the list use the same operand rows (from 10 M nonzeros on; very long lists of short rows are in
test_gpu_rank16_walk.py): rows that end around the boundaries of walkers (64 and 128 nonzeros) and tiles, rows over many tiles, empty rows, plain and
accumulating."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu
J = 40000


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


@pytest.fixture(scope="module")
def matrix():
    ends = {64 * m + d for m in range(1, 130) for d in (-1, 0, 1)} | {4096 * m + d for m in range(3, 40) for d in (-1, 0, 1)}
    ends = [0] + sorted(ends)
    edges = []
    for n in range(1, len(ends)):
        edges += [ends[n] - ends[n - 1]] + [0] * (n % 3 == 0)      # a row that ends just there; an empty one behind every third
    edges = torch.tensor(edges, dtype=torch.int64)
    tail = torch.tensor([0, 30000, 0, 0, 12288, 4096, 1, 4095, 8193, 0], dtype=torch.int64)
    lens = torch.cat([edges, tail, torch.full((270_000,), 37), torch.zeros(50, dtype=torch.int64), torch.full((300_000,), 2), tail])
    rows, cols, vals = gen.matrix_from_row_lengths(lens.numel(), J, lens, 12, "cuda")
    assert vals.numel() > 10 << 20
    return lens.numel(), rows, cols, vals


@pytest.mark.parametrize("R", [8, 16])
@pytest.mark.parametrize("layout", ["csr", "dcsr"])
def test_rows_around_walkers_and_tiles(comet, matrix, layout, R):
    I, rows, cols, vals = matrix
    pack = fmt.pack_csr if layout == "csr" else fmt.pack_dcsr
    A = comet.from_levels(pack(I, J, rows, cols, vals), comet.COMET_VALIDATE | comet.COMET_LEAN).set_variant(2)
    B, old = gen.dense_operand(3, 0, (J, R)), gen.dense_operand(4, 0, (I, R))
    print("long list %s R=%d nnz=%d" % (layout, R, vals.numel()), flush=True)
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B.to("cuda"), C)
    ref, absum = oracle.spmm(np_(rows), np_(cols), np_(vals), (I, J), np_(B))
    assert_values_close(np_(C), ref, absum, "long list %s R=%d" % (layout, R))
    assert torch.equal(C, comet.comet_spmm(A, B.to("cuda"))), "two runs differ"
    D = old.to("cuda")
    comet.comet_spmm_axpby(A, 0.75, B.to("cuda"), -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby %s R=%d" % (layout, R))
