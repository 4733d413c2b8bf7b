"""Split renders (chunk-start carries from one workgroup per voice, chunks and
passes spread over workgroups) are bit for bit the unsplit render, at chunk
counts around the 16 the carries kernel takes at a time and at lengths that end
inside a pass."""

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2104_12922_amd as S
    return S


@pytest.mark.parametrize("B,N", [(1, 1), (3, 6200), (5, 6201), (2, 4999), (7, 6200 * 15 + 1),
                                 (4, 6200 * 16), (3, 6200 * 17 - 3), (2, 6200 * 33 + 1777),
                                 (300, 12345), (2047, 12401)])
def test_split_is_bitwise_unsplit(S, B, N):
    table = W.default_nebula().table()
    u = S.synth_sample_params(5, 100, B)
    whole = S.synth_render_plan(u, table, 4, 1, n_samples=N, first_g=100, noise_seed=5)
    assert torch.equal(S.synth_render(u, table, n_samples=N, first_g=100, noise_seed=5), whole)
