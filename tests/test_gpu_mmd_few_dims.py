"""Pair sums and MMDs of sets of up to 2048 sounds where the dimensions are too
few (or, for one sum, so many) that all pairs in float64 are quicker than
sorting: at the edges of the 4 and 32 staged dimensions, of the tiles and of
the line between the two ways, against the float64 oracle.

Bound: differences of float32 values are within 2^-53 relative in float64 and a
sum of non-negative terms passes through fewer than 33 + 16 + 2048 additions on
the GPU (a run of at most 8 chunks of 32 dimensions per accumulator, 16 pairs a
thread, trees) and up to 4096 in the oracle: 7e-13 relative in all, 1e-12 here.
"""
import numpy as np
import pytest
import torch

from oracle import mmd as OM

pytestmark = pytest.mark.gpu
REL = 1e-12


@pytest.fixture(scope="module")
def nb():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2104_12922_amd import nebula
    return nebula


def _set(seed, n, dim):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, dim, generator=g) * 3.0 - 5.0
    x[torch.rand(n, dim, generator=g) < 0.2] = -13.815511
    return x.float()


@pytest.mark.parametrize("n,m,dim", [(2048, 2048, 1), (2000, 2000, 3), (1100, 1100, 4), (1100, 1090, 5),
                                     (1025, 2048, 31), (1, 2048, 32), (2048, 1, 33), (300, 300, 36),
                                     (700, 650, 100), (65, 63, 60000), (64, 64, 65537)])
def test_matches_oracle(nb, n, m, dim):
    X, Y = _set(n + dim, n, dim), _set(m + dim + 1, m, dim)
    x, y = X.cuda(), Y.cuda()
    sxy, sxx, syy = (OM.l1_distance_sum(a.double().numpy(), b.double().numpy())
                     for a, b in ((X, Y), (X, X), (Y, Y)))
    got = nb.mmd_l1(x, y).cpu().numpy()
    for a, b in zip(got[1:], (sxy, sxx, syy)):
        assert abs(a - b) <= REL * b, (a, b)
    scale = 2 * sxy / (n * m) + sxx / (n * n) + syy / (m * m)
    assert abs(got[0] - (2 * sxy / (n * m) - sxx / (n * n) - syy / (m * m))) <= REL * scale
    assert np.array_equal(nb.mmd_l1(x, y).cpu().numpy(), got)
    assert float(nb.mmd_l1(x, x)[0]) == 0.0
    if min(n, m) > 256 or max(n, m) <= 256:            # (float32 runs for one much smaller set)
        one = float(nb.l1_pair_sum(x, y))
        assert abs(one - sxy) <= REL * sxy


def test_strided_rows_and_values_that_are_not_finite(nb):
    wide, Y = _set(1, 1200, 20), _set(2, 1300, 9)
    A, B = wide.cuda()[:, 3:12], Y.cuda()
    s = float(nb.l1_pair_sum(A, B))
    assert s == float(nb.l1_pair_sum(A.contiguous(), B))
    ref = OM.l1_distance_sum(wide[:, 3:12].double().numpy(), Y.double().numpy())
    assert abs(s - ref) <= REL * ref
    for v in (float("inf"), float("-inf"), float("nan")):
        X = wide[:, 3:12].clone()
        X[77, 4] = v
        got = nb.mmd_l1(X.cuda(), B).cpu().numpy()
        assert np.isnan(got[2]) and np.isfinite(got[3])
        assert np.isnan(got[1]) if v != v else got[1] == float("inf")
