"""FM operators of negative frequency (a nebula whose ratios are below 0: the
frequency is limited from above only) against the float64 oracle: within half
the sample rate, across 0, at exactly half, and far beyond it, where the phase
passes several cycles a sample.  The bound is test_gpu_fm's: the phase of each
sample is within 2^-22 cycles of the float64 one, inside its EPS."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fm as OFM
from test_gpu_fm import _bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(-3.0, -0.5), (-2.0, 2.0), (-600.0, -100.0)])
def test_negative_ratios(lo, hi):
    from paper_2104_12922_amd import fm
    tab = W.fm_default_nebula().table()
    for b in OFM.OP_BASE:
        tab[b] = (lo, hi, 1.0, 0.0)
    u = fm.fm_sample_params(21, batch=6)
    uu = u.cpu().numpy().astype(np.float64)
    y = fm.fm_render(u, tab, n_samples=13001).cpu().numpy()
    ref = OFM.render_uniform(torch.tensor(uu), 13001, tab).numpy()
    err = np.abs(y - ref).max(1)
    assert np.all(err <= _bound(uu, tab)), err


def test_minus_half_the_sample_rate():
    from paper_2104_12922_amd import fm
    tab = W.fm_default_nebula().table()
    tab[0] = (69.0, 69.0, 1.0, 0.0)
    for b in OFM.OP_BASE:
        tab[b] = (-44100.0 / 880.0, -44100.0 / 880.0, 1.0, 0.0)
        tab[b + 1] = (0.0, 0.0, 1.0, 0.0)
    u = fm.fm_sample_params(22, batch=3)
    uu = u.cpu().numpy().astype(np.float64)
    y = fm.fm_render(u, tab, n_samples=6500).cpu().numpy()
    ref = OFM.render_uniform(torch.tensor(uu), 6500, tab).numpy()
    assert np.all(np.abs(y - ref).max(1) <= _bound(uu, tab))


def test_minus_infinity_is_not_a_number():
    from paper_2104_12922_amd import fm
    tab = W.fm_default_nebula().table()
    tab[0] = (1e6, 1e6, 1.0, 0.0)                      # 440 2^(1e6 / 12): above the largest float64
    tab[OFM.OP_BASE[3]] = (-1.0, -1.0, 1.0, 0.0)
    u = fm.fm_sample_params(23, batch=2)
    y = fm.fm_render(u, tab, n_samples=500)
    uu = torch.tensor(u.cpu().numpy().astype(np.float64))
    assert bool((torch.isnan(y).cpu() == torch.isnan(OFM.render_uniform(uu, 500, tab))).all())
