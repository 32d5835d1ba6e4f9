"""SpMM at rank 16 over more than 24 Mi nonzeros in rows of four on average, which a walk over tiles of 4096 nonzeros takes: rows
that end around the boundaries of walkers (128 nonzeros) and tiles, rows over many tiles, empty rows, plain and accumulating; and
the same rows with longer ones behind them, which the piece kernel takes."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu
J, R = 40000, 16


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


@pytest.mark.parametrize("layout,rest", [("csr", 4), ("dcsr", 4), ("csr", 9)])
def test_rows_around_walkers_and_tiles(comet, layout, rest):
    ends = {128 * m + d for m in range(1, 70) for d in (-1, 0, 1)} | {4096 * m + d for m in range(3, 40) for d in (-1, 0, 1)}
    ends = [0] + sorted(ends)
    edges = []
    for n in range(1, len(ends)):
        edges += [ends[n] - ends[n - 1]] + [0] * (n % 3 == 0)      # a row that ends just there; an empty one behind every third
    edges = torch.tensor(edges, dtype=torch.int64)
    tail = torch.tensor([0, 30000, 0, 0, 12288, 4096, 1, 4095, 8193, 0], dtype=torch.int64)
    lens = torch.cat([edges, tail, torch.full((25_200_000 // rest,), rest), tail])
    rows, cols, vals = gen.matrix_from_row_lengths(lens.numel(), J, lens, 12, "cuda")
    I, nnz = lens.numel(), vals.numel()
    assert nnz > 24 << 20
    print("rank-16 walk %s rest=%d nnz=%d" % (layout, rest, nnz), flush=True)
    A = comet.from_levels((fmt.pack_csr if layout == "csr" else fmt.pack_dcsr)(I, J, rows, cols, vals),
                          comet.COMET_VALIDATE | comet.COMET_LEAN).set_variant(2)
    B, old = gen.dense_operand(3, 0, (J, R)), gen.dense_operand(4, 0, (I, R))
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B.to("cuda"), C)
    ref, absum = oracle.spmm(np_(rows), np_(cols), np_(vals), (I, J), np_(B))
    assert_values_close(np_(C), ref, absum, "rank-16 walk %s" % layout)
    assert torch.equal(C, comet.comet_spmm(A, B.to("cuda"))), "two runs differ"
    D = old.to("cuda")
    comet.comet_spmm_axpby(A, 0.75, B.to("cuda"), -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby %s" % layout)
