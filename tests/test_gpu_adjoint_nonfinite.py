"""The render adjoint on cotangents and parameters that are not finite or nearly
as large as float32 goes: an adjoint reaches only the parameters that the sample
depends on (a ramp that is not passed, shape weights without a sum), and a large
one does not overflow before its sums do.  Against the float64 oracle, by the
criterion of test_gpu_adjoint."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import philox
from test_gpu_adjoint import check, oracle_grad

pytestmark = pytest.mark.gpu
B = 6
DECAY, RELEASE, NOTE_OFF = [3, 8, 13, 18, 23, 28], [5, 10, 15, 20, 25, 30], [1]


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2104_12922_amd as S
    return S


def _inputs(N):
    u = philox.sample_params(5, np.arange(B)).astype(np.float32).astype(np.float64)
    g = np.random.default_rng(2).standard_normal((B, N)).astype(np.float32)
    return u, g


def _grad(S, u, g, table):
    return S.synth_render_backward(torch.tensor(u, dtype=torch.float32).cuda(), torch.tensor(g).cuda(),
                                   table).cpu().numpy()


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("N", [700, 13000])
def test_ramps_that_are_not_passed(S, value, N):
    table = W.default_nebula().table()
    table[1] = (1.0, 4.0, 1.0, 0.0)                     # the note and every attack outlast the sound
    for b in range(2, 32, 5):
        table[b] = (1.0, 2.0, 1.0, 0.0)
    u, g = _inputs(N)
    g[np.arange(B), np.arange(B) * 101 + 7] = value
    ref = oracle_grad(u, g, N, table)
    got = _grad(S, u, g, table)
    for p in DECAY + RELEASE + NOTE_OFF:
        assert np.all(ref[:, p] == 0.0) and np.all(got[:, p] == 0.0), p
    assert not np.isfinite(got).all()


def test_shape_weights_without_a_sum(S):
    table = W.default_nebula().table()
    u, g = _inputs(700)
    u[:, 35] = np.nan                                   # a shape weight of the first LFO
    got = _grad(S, u, g, table)
    assert np.isfinite(got[:, 36:40]).all()


@pytest.mark.parametrize("scale", [1e30, 1e37])
@pytest.mark.parametrize("period", [100, 768])
def test_large_cotangents(S, scale, period):
    table = W.default_nebula().table()
    N = 9 * period
    u, g = _inputs(N)
    g[np.arange(B), N - 1 - np.arange(B) * 37] = scale
    rc = 44100.0 / period
    got = S.synth_render_backward(torch.tensor(u, dtype=torch.float32).cuda(), torch.tensor(g).cuda(),
                                  table, control_rate=rc).cpu().numpy()
    assert not np.isnan(got).any()                      # (a pitch's gradient may itself pass 3.4e38)
    if period == 100:
        assert np.isfinite(got).all()
        check(got, oracle_grad(u, g, N, table))
