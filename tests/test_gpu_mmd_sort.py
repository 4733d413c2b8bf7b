"""Pair sums by sorting (sets of up to 2048 sounds) on the GPU against the
float64 oracle, at the edges of the kernel's register counts (32 R values a
set, R = 4 .. 64) and of its 16- and 8-dimension tiles.

Bound: every term of a sum is non-negative and float64: a gap is off by at
most 2^-53 relative, and a sum passes through fewer than 200 additions, so the
GPU's sum is within 210 * 2^-53 = 2.4e-14 relative; the oracle adds up to 4096
row sums one by one (4.6e-13).  1e-12 covers both."""

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


def _sets(seed, n, m, dim):
    g = torch.Generator().manual_seed(seed)
    X = torch.randn(n, dim, generator=g) * 3.0 - 5.0
    Y = torch.randn(m, dim, generator=g) * 4.0 - 4.0
    floor = -13.815511                                    # silent frames: many equal values
    X[torch.rand(n, dim, generator=g) < 0.2] = floor
    Y[torch.rand(m, dim, generator=g) < 0.3] = floor
    return X.float(), Y.float()


def _sums(X, Y):
    X, Y = X.cpu().double().numpy(), Y.cpu().double().numpy()
    return [OM.l1_distance_sum(a, b) for a, b in ((X, Y), (X, X), (Y, Y))]


@pytest.mark.parametrize("n,m,dim", [(128, 128, 2740), (127, 100, 4099), (129, 256, 1031),
                                     (257, 512, 301), (512, 130, 400), (513, 1000, 97),
                                     (1024, 1024, 49), (1025, 90, 111), (2048, 2048, 17),
                                     (2048, 1, 33)])
def test_sorted_sums_match_oracle(nb, n, m, dim):
    X, Y = _sets(n + m + dim, n, m, dim)
    got = nb.mmd_l1(X.cuda(), Y.cuda()).cpu().numpy()
    sxy, sxx, syy = _sums(X, Y)
    for a, b in zip(got[1:], (sxy, sxx, syy)):
        assert abs(a - b) <= REL * b, (a, b)
    scale = 2 * sxy / (n * m) + sxx / (n * n) + syy / (m * m)
    assert abs(got[0] - (2 * sxy / (n * m) - sxx / (n * n) - syy / (m * m))) <= REL * scale
    again = nb.mmd_l1(X.cuda(), Y.cuda()).cpu().numpy()
    assert np.array_equal(got, again)
    assert float(nb.mmd_l1(X.cuda(), X.cuda())[0]) == 0.0


def test_integers_are_bit_exact(nb):
    g = torch.Generator().manual_seed(5)
    X = torch.randint(-8, 9, (300, 900), generator=g).float()
    Y = torch.randint(-6, 11, (200, 900), generator=g).float()
    got = nb.mmd_l1(X.cuda(), Y.cuda()).cpu().numpy()
    assert list(got[1:]) == _sums(X, Y)


def test_strided_rows(nb):
    wide, B = _sets(9, 700, 650, 315)
    A = wide.cuda()[:, 3:303]                             # unaligned rows, stride 315
    B = B.cuda()[:, :300].contiguous()
    s = float(nb.l1_pair_sum(A, B))
    assert s == float(nb.l1_pair_sum(A.contiguous(), B))
    ref = _sums(A, B)[0]
    assert abs(s - ref) <= REL * ref


@pytest.mark.parametrize("x,y", [(float("inf"), None), (float("nan"), None), (None, float("nan")),
                                 (float("inf"), float("inf")), (float("inf"), float("-inf")),
                                 (None, float("-inf")), (3.4028234e38, None)])
def test_values_that_are_not_finite(nb, x, y):
    X, Y = _sets(4, 260, 250, 700)
    if x is not None:
        X[17, 5] = x
    if y is not None:
        Y[240, 5] = y
    got = nb.mmd_l1(X.cuda(), Y.cuda()).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = _sums(X, Y)
    for a, b in zip(got[1:], ref):
        if np.isfinite(b):
            assert abs(a - b) <= REL * b
        else:
            assert np.isnan(a) if np.isnan(b) else a == b
