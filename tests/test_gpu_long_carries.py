"""Chunk-start carries of long voices (more than 32 chunks: sums and updates in
launches of their own) are bit for bit those of a voice walked by one workgroup,
around the workgroups' 16 chunks, the 64 of an update step and the 256 staged at
a time; uniform and ragged, at 1, 2 and 4 runs a segment and with clamped
increments."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
CHUNK = 6200


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2104_12922_amd as S
    return S


@pytest.mark.parametrize("chunks,extra", [(32, 0), (32, 1), (64, 0), (64, 1), (80, 0), (81, 5), (128, 0), (128, 99),
                                          (272, 0), (272, 1), (300, 3101)])
def test_uniform(S, chunks, extra):
    table = W.default_nebula().table()
    table[1] = (50.0, 60.0, 1.0, 0.0)                  # long notes: no chunk is silent
    N = CHUNK * chunks + extra
    u = S.synth_sample_params(3, 9, 2)
    kw = dict(n_samples=N, first_g=9, noise_seed=3)
    whole = S.synth_render_plan(u, table, 4, 1, **kw)
    assert torch.equal(S.synth_render(u, table, **kw), whole)
    assert float(whole[:, -2000:].abs().max()) > 0.0


@pytest.mark.parametrize("rps,period,pitch", [(1, 100, 84.0), (2, 100, 84.0), (4, 100, 140.0), (1, 64, 140.0)])
def test_ragged(S, rps, period, pitch):
    table = W.default_nebula().table()
    table[1] = (50.0, 60.0, 1.0, 0.0)
    table[0] = (pitch - 10.0, pitch, 1.0, 0.0)         # 140: above half the sample rate, clamped
    c = 62 * period
    lens = np.array([c * 70 + 7, 5, c * 3, 0, c * 66, c * 90 + 1])
    offs = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)])).cuda()
    u = S.synth_sample_params(4, 0, len(lens))
    kw = dict(offsets=offs, noise_seed=4, control_rate=44100.0 / period)
    whole = S.synth_render_plan(u, table, rps, 1, **kw)
    assert torch.equal(S.synth_render_plan(u, table, rps, 7, max_samples=int(lens.max()), **kw), whole)

