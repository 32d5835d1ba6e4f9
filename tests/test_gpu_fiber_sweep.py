"""The heavy-fiber sweep of TTM: fibers whose pieces inside a window of operand rows end at every place of a block of 16, empty
pieces, one window and many with a ragged last one, and operand rows that are not finite beside fibers that do not name them."""
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


def _tensor(K, window):
    """Just over 2^20 nonzeros in fibers of 256 and more, with short ones between them: fiber f has 256 + f % 33 consecutive
    coordinates from a start that moves along the mode, so that pieces of 0 to 33 nonzeros lie on both sides of every window's
    edge, or it fills half of the mode."""
    g = np.random.default_rng(11)
    fibers, total = [], 0
    edges = list(range(window, K, window)) or [K // 2]
    while total < (1 << 20) + 5000:
        f = len(fibers)
        if f % 7 == 0:
            c = np.flatnonzero(g.random(K) < 0.5)
        elif f % 7 == 1:
            c = np.sort(g.choice(K, 1 + f % 40, replace=False))
        else:
            n = min(256 + f % 33, K)
            at = edges[f % len(edges)] - (f // 7) % 40 - (0 if f % 2 else n - 20)
            at = min(max(at, 0), K - n)
            c = np.arange(at, at + n)
        if f % 7 != 1 and len(c) < 256:
            c = np.arange(256)
        fibers.append(c)
        total += len(c)
    k = torch.from_numpy(np.concatenate(fibers)).to(torch.int64)
    f = torch.from_numpy(np.repeat(np.arange(len(fibers)), [len(c) for c in fibers]))
    J = 11
    vals = torch.from_numpy(g.uniform(-1, 1, k.numel()))
    return ((len(fibers) + J - 1) // J, J, K), f // J, f % J, k, vals


@pytest.mark.parametrize("R,K", [(16, 700), (16, 1024), (16, 3000), (16, 8192), (32, 512), (32, 2500), (32, 8191)])
def test_pieces_of_every_length(comet, R, K):
    dims, i, j, k, vals = _tensor(K, 16384 // R)
    print("fiber sweep R=%d K=%d nnz=%d" % (R, K, vals.numel()), flush=True)
    X = comet.from_levels(fmt.pack_csf3(dims, i, j, k, vals).to("cuda"))
    assert X.heavy_plan()[0] > 0
    U = gen.dense_operand(4, 0, (K, R))
    Y = comet.comet_ttm(X, 2, U.cuda())
    torch.cuda.synchronize()
    first = np_(Y.vals()).reshape(-1, R).copy()
    ref = oracle.ttm(np_(i), np_(j), np_(k), np_(vals), dims, np_(U))
    assert_values_close(first, ref["vals"], ref["abs"], "fiber sweep R=%d K=%d" % (R, K))
    # a row of the operand that is not finite: in the results of the fibers that name it, and in no other
    bad = K // 3
    named = np.zeros(first.shape[0], bool)
    fiber = np_(i).astype(np.int64) * dims[1] + np_(j)
    named[np.unique(fiber[np_(k) == bad])] = True
    assert named.any() and not named.all()
    U[bad] = float("inf")
    comet.comet_ttm(X, 2, U.cuda(), Y)
    torch.cuda.synchronize()
    got = np_(Y.vals()).reshape(-1, R)
    assert np.array_equal(got[~named], first[~named])
    assert not np.isfinite(got[named]).any()
