"""The render adjoint at the edges of its chunks of 62 control samples: whole
chunks, a last chunk of one (partial) segment, whose sums share its columns of
the workspace, and a voice that is silent from its second chunk on.  Against
the oracle's exact gradient with test_gpu_adjoint's criterion and bound
(float32 amplitude-side sums, at most about 1e-4)."""
import numpy as np
import pytest
import torch

from oracle import philox
from test_gpu_adjoint import check, oracle_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 99, 6200, 6201, 6300, 12400, 12499, 24801])
def test_chunk_edges(N, nebula_table):
    import paper_2104_12922_amd as synth
    B = 3
    u = philox.sample_params(21, np.arange(B)).astype(np.float32).astype(np.float64)
    u[:, 1] = 0.9                                   # held notes,
    u[2, 1] = 0.02                                  # one short with short releases
    u[2, [5, 10, 15, 20, 25, 30]] = 1e-4
    g = np.random.default_rng(N).standard_normal((B, N)).astype(np.float32)
    ref = oracle_grad(u, g.astype(np.float64), N, nebula_table, noise_seed=5)
    ga = synth.synth_render_backward(torch.tensor(u, dtype=torch.float32).cuda(),
                                     torch.tensor(g).cuda(), nebula_table, noise_seed=5)
    torch.cuda.synchronize()
    ga = ga.cpu().numpy().astype(np.float64)
    zero = ~ref.any(axis=1)                         # a relative criterion needs a gradient
    assert not ga[zero].any()
    check(ga[~zero], ref[~zero])
