"""Bias gradients of the proposal network: the three matrices' column sums in
one pair of launches (column tiles of 128, up to 32 row slices), and one by one
where a row of odd width rules the paired reads out.  The sums are float64, so
each result is its exact sum rounded once to float32 (2^-24 relative)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split_k", [True, False])
@pytest.mark.parametrize("batch,d_h,d_out", [(1, 64, 2), (31, 128, 78), (33, 130, 128), (200, 256, 130),
                                             (1000, 192, 77)])
def test_bias_gradients(batch, d_h, d_out, split_k):
    from paper_2104_12922_amd import learned
    rng = np.random.default_rng(batch)
    w = lambda *s: (rng.standard_normal(s) / 8).astype(np.float32)
    net = learned.MLP({"w1t": w(d_h, 64), "b1": w(d_h), "w2t": w(d_h, d_h), "b2": w(d_h),
                       "w3t": w(d_out, d_h), "b3": w(d_out)}, split_k=split_k)
    x = torch.randn(batch, 64, device="cuda").bfloat16()
    net.forward(x)
    net.backward(x, torch.rand(batch, d_out, device="cuda"))
    torch.cuda.synchronize()
    for dz, b in (("dz3", "b3"), ("dh2", "b2"), ("dh1", "b1")):
        ref = net.a[dz].double().sum(0)
        assert ((net.g[b].double() - ref).abs() <= 6.1e-8 * ref.abs() + 1e-30).all(), b
