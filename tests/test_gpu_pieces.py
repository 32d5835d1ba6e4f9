"""The rank-R kernel over pieces: segment lengths around its limits (pieces of 32, whole segments of 48, tiles of 768 and
1472 units), segments over many tiles, empty ones, every row layout, with and without accumulation."""
import numpy as np
import pytest
import torch

import oracle
from synth import formats as fmt
from synth import generate as gen
from util import assert_values_close, np_

pytestmark = pytest.mark.gpu

EDGES = [1, 0, 31, 32, 33, 47, 48, 49, 2, 63, 64, 65, 0, 0, 95, 96, 97, 3, 767, 768, 769, 1, 1535, 1536, 1537, 700, 40, 5000, 7, 20000, 0]


@pytest.fixture(scope="module")
def comet():
    from paper_2102_05187_amd import build
    build.build_if_missing()
    import paper_2102_05187_amd as c
    return c


def _edges():
    # behind them tiles that end with empty rows next to a few long ones
    lens = torch.tensor(EDGES * 2 + [1] * 1500 + [0] * 900 + [2, 48, 49] * 300 + [0, 30000] + ([20, 24, 28] + [0] * 900) * 4,
                        dtype=torch.int64)
    return (lens.numel(), 40000), gen.matrix_from_row_lengths(lens.numel(), 40000, lens, 5)


@pytest.mark.parametrize("R", [2, 3, 4, 7, 8, 9, 10, 16, 20, 31, 32, 33, 34, 48, 63, 64, 66, 96, 100, 127, 128])
@pytest.mark.parametrize("layout", ["csr", "dcsr"])
def test_edges_of_pieces(comet, layout, R):
    (I, J), (rows, cols, vals) = _edges()
    pack = fmt.pack_csr if layout == "csr" else fmt.pack_dcsr
    A = comet.from_levels(pack(I, J, rows, cols, vals).to("cuda")).set_variant(2)
    B = gen.dense_operand(3, 0, (J, R))
    print("pieces %s R=%d nnz=%d" % (layout, R, vals.numel()), flush=True)
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B.to("cuda"), C)
    ref, absum = oracle.spmm(np_(rows), np_(cols), np_(vals), (I, J), np_(B))
    assert_values_close(np_(C), ref, absum, "pieces %s R=%d" % (layout, R))
    again = comet.comet_spmm(A, B.to("cuda"))
    assert torch.equal(C, again), "two runs differ"
    old = gen.dense_operand(4, 0, (I, R))
    D = old.to("cuda")
    comet.comet_spmm_axpby(A, 0.75, B.to("cuda"), -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "pieces axpby R=%d" % R)


@pytest.mark.parametrize("R", [20, 33])
def test_many_nonzeros_take_large_tiles(comet, R):
    n = 650_000
    lens = gen.zipf_row_lengths(n, 1.75, 4000, 3)
    lens[::7] = 0
    rows, cols, vals = gen.matrix_from_row_lengths(n, n, lens, 6, "cuda")
    assert vals.numel() > 10 << 20
    A = comet.from_levels(fmt.pack_csr(n, n, rows, cols, vals))
    B = gen.dense_operand(3, 0, (n, R))
    print("large tiles R=%d nnz=%d" % (R, vals.numel()), flush=True)
    C = comet.comet_spmm(A, B.to("cuda"))
    ref, absum = oracle.spmm(np_(rows.cpu()), np_(cols.cpu()), np_(vals.cpu()), (n, n), np_(B))
    assert_values_close(np_(C), ref, absum, "large tiles R=%d" % R)


@pytest.mark.parametrize("R", [20, 128])
def test_most_partial_sums_in_a_tile(comet, R):
    # rows of 65 are three pieces each, more than rows of any other length give: 22 whole ones in a large tile and cut ones at its ends
    n = 165_000
    lens = torch.full((n,), 65, dtype=torch.int64)
    rows, cols, vals = gen.matrix_from_row_lengths(n, 50_000, lens, 7, "cuda")
    assert vals.numel() > 10 << 20
    A = comet.from_levels(fmt.pack_csr(n, 50_000, rows, cols, vals))
    B = gen.dense_operand(3, 0, (50_000, R))
    print("partial sums R=%d nnz=%d" % (R, vals.numel()), flush=True)
    C = comet.comet_spmm(A, B.to("cuda"))
    ref, absum = oracle.spmm(np_(rows.cpu()), np_(cols.cpu()), np_(vals.cpu()), (n, 50_000), np_(B))
    assert_values_close(np_(C), ref, absum, "partial sums R=%d" % R)


@pytest.mark.parametrize("R", [20, 32, 33, 64, 128])
@pytest.mark.parametrize("layout", ["csr", "dcsr"])
def test_edges_of_large_tiles(comet, layout, R):
    """The same edges where tiles are large: rows around a whole tile, over few and over many tiles, empty ones."""
    lens = torch.tensor([1, 0, 31, 32, 33, 47, 48, 49, 64, 65, 97, 1471, 1472, 1473, 2944, 2945, 0, 20000, 30000, 0] + [33, 0, 49, 2] * 200,
                        dtype=torch.int64)
    lens = torch.cat([lens, torch.full((200_000,), 37, dtype=torch.int64), lens])
    I, J = lens.numel(), 40000
    rows, cols, vals = gen.matrix_from_row_lengths(I, J, lens, 8, "cuda")
    assert vals.numel() > 7 << 20
    pack = fmt.pack_csr if layout == "csr" else fmt.pack_dcsr
    A = comet.from_levels(pack(I, J, rows, cols, vals)).set_variant(2)
    B, old = gen.dense_operand(3, 0, (J, R)), gen.dense_operand(4, 0, (I, R))
    print("large tiles %s R=%d nnz=%d" % (layout, R, vals.numel()), flush=True)
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B.to("cuda"), C)
    ref, absum = oracle.spmm(np_(rows.cpu()), np_(cols.cpu()), np_(vals.cpu()), (I, J), np_(B))
    assert_values_close(np_(C), ref, absum, "large tiles %s R=%d" % (layout, R))
    D = old.to("cuda")
    comet.comet_spmm_axpby(A, 0.75, B.to("cuda"), -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "axpby R=%d" % R)


@pytest.mark.parametrize("R", [2, 16, 18, 33, 34, 64, 66, 96, 100, 128])
@pytest.mark.parametrize("layout", ["csr", "dcsr"])
def test_operands_of_4_gib(comet, layout, R):
    """Row offsets beyond 32 bits in bytes, first and last rows of the operand among them; every layout for such operands."""
    J = (1 << 32) // (8 * R) + 3
    lens = torch.tensor([1, 0, 2, 33, 48, 49, 3000, 0, 5] * 20, dtype=torch.int64)
    rows, cols, vals = gen.matrix_from_row_lengths(lens.numel(), J, lens, 9)
    start = torch.cumsum(lens, 0) - lens
    cols[start[lens > 1]] = 0
    cols[(start + lens - 1)[lens > 1]] = J - 1
    I = lens.numel()
    A = comet.from_levels((fmt.pack_csr if layout == "csr" else fmt.pack_dcsr)(I, J, rows, cols, vals).to("cuda")).set_variant(2)
    print("large operand %s R=%d J=%d" % (layout, R, J), flush=True)
    B = torch.rand((J, R), dtype=torch.float64, device="cuda")
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B, C)
    used, where = torch.unique(cols.long(), return_inverse=True)
    ref, absum = oracle.spmm(np_(rows), np_(where.int()), np_(vals), (I, used.numel()), np_(B[used.cuda()]))
    assert_values_close(np_(C), ref, absum, "large operand %s R=%d" % (layout, R))
    D = torch.ones_like(C)
    comet.comet_spmm_axpby(A, 0.75, B, -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5, 0.75 * absum + 0.5, "large operand axpby R=%d" % R)


@pytest.mark.parametrize("R", [2, 8])
def test_without_memory_for_the_plan(comet, R):
    """A handle whose piece plan (4 bytes per row here) does not fit is made all the same, and its products are right."""
    I, J, step = 48_000_000, 1000, 12
    pos = torch.div(torch.arange(I + 1, device="cuda") + step - 1, step, rounding_mode="floor").int()
    nnz = int(pos[-1])
    crd = torch.randint(0, J, (nnz,), device="cuda", dtype=torch.int32)
    vals = torch.rand(nnz, dtype=torch.float64, device="cuda")
    B = torch.rand((J, R), dtype=torch.float64, device="cuda")
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    size = torch.tensor([I], dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while True:                                   # all but about 100 MB of the device memory, without touching it
        free = torch.cuda.mem_get_info()[0] - (100 << 20)
        if free < 16 << 20 or len(held) > 2000:
            break
        try:
            held.append(torch.empty(min(free // 2 + (8 << 20), 8 << 30), dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            break
    print("no plan R=%d left=%d MB" % (R, torch.cuda.mem_get_info()[0] >> 20), flush=True)
    try:
        A = comet.comet_tensor_create([I, J], [comet.COMET_D, comet.COMET_CU], [size, pos], [None, crd], vals, 0)
    finally:
        del held
        torch.cuda.empty_cache()
    comet.comet_spmm(A.set_variant(2), B, C)
    assert torch.equal(C[::step], vals[:, None] * B[crd.long()])
    C[::step] = 0.0
    assert torch.count_nonzero(C) == 0


@pytest.mark.parametrize("R", [10, 20, 32, 33, 48, 64, 100, 128])
def test_rows_spread_over_a_large_operand(comet, R):
    """Nonzeros that hardly ever come back to an operand row take another number of loads per piece; the same edges."""
    lens = torch.tensor(([n for n in EDGES if n < 100] + list(range(1, 50))) * 120 + [5000, 20000], dtype=torch.int64)
    I, J = lens.numel(), 1_000_000 if R < 32 else 400_000
    rows, cols, vals = gen.matrix_from_row_lengths(I, J, lens, 8)
    part = torch.unique(cols[:1 << 18]).numel()
    print("spread R=%d nnz=%d distinct=%d" % (R, vals.numel(), part), flush=True)
    assert vals.numel() > 1 << 18 and part * (R * 8 if R % 16 == 0 else R * 8 + 120) > 33 << 20
    A = comet.from_levels(fmt.pack_csr(I, J, rows, cols, vals).to("cuda"), comet.COMET_LEAN).set_variant(2)
    B, old = gen.dense_operand(3, 0, (J, R)), gen.dense_operand(4, 0, (I, R))
    C = torch.full((I, R), float("nan"), dtype=torch.float64, device="cuda")
    comet.comet_spmm(A, B.to("cuda"), C)
    ref, absum = oracle.spmm(np_(rows), np_(cols), np_(vals), (I, J), np_(B))
    assert_values_close(np_(C), ref, absum, "spread R=%d" % R)
    D = old.to("cuda")
    comet.comet_spmm_axpby(A, 0.75, B.to("cuda"), -0.5, D)
    assert_values_close(np_(D), 0.75 * ref - 0.5 * np_(old), 0.75 * absum + 0.5 * np.abs(np_(old)), "spread axpby R=%d" % R)
