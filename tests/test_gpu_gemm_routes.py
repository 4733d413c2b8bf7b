"""The bf16 products at the lines between their kernels: a long K whose parts are
taken side by side, few rows at the line of tiles x K, few columns over a short K,
and the MLP's output layer (78 columns) where its sigmoid is not saturated.

Small-integer operands keep every float32 sum exact (|sum| <= 9 K < 2^24), so
those products must equal the integer product bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2104_12922_amd import learned
    return learned


def _ints(shape, g):
    return torch.randint(-3, 4, shape, generator=g).to(BF)


@pytest.mark.parametrize("B,d_in,d_h", [(33, 12288, 1024), (129, 12296, 264), (130, 12280, 264),
                                        (300, 20008, 200), (513, 12288, 1024), (1000, 16384, 136),
                                        (64, 16384, 1024), (65, 16384, 1024), (2049, 12320, 1024)])
def test_long_sums_are_exact(L, B, d_in, d_h):
    g = torch.Generator().manual_seed(B + d_in)
    z = lambda *s: torch.zeros(*s).numpy()
    w1 = _ints((d_h, d_in), g)
    net = L.MLP({"w1t": w1.float().numpy(), "b1": z(d_h), "w2t": z(d_h, d_h), "b2": z(d_h),
                 "w3t": z(8, d_h), "b3": z(8)})
    x = _ints((B, d_in), g)
    net.forward(x.cuda())
    ref = (x.cuda().float() @ w1.cuda().float().T).cpu()       # exact: integers below 2^24
    assert torch.equal(ref[:3].double(), x[:3].double() @ w1.double().T)
    assert torch.equal(net.a["h1pre"].cpu(), ref)


@pytest.mark.parametrize("M", [32768, 32769 + 7, 70000])
@pytest.mark.parametrize("N,K", [(8, 8), (16, 64), (24, 72), (32, 96), (32, 104), (40, 64)])
@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_few_columns_are_exact(L, M, N, K, a_layout, b_layout):
    g = torch.Generator().manual_seed(M + N + K)
    A, B = _ints((M, K), g), _ints((K, N), g)
    bias = torch.randint(-5, 6, (N,), generator=g).float()
    C = L.gemm_bf16((A if a_layout == 0 else A.T).contiguous().cuda(),
                    (B.T if b_layout == 0 else B).contiguous().cuda(), M, N, K, a_layout, b_layout,
                    bias=bias.cuda())
    assert torch.equal(C.cpu(), A.float() @ B.float() + bias)


@pytest.mark.parametrize("B", [1, 31, 33, 129, 300, 513])
def test_mlp_output_layer(L, B):
    """Logits of about 1, so that nearly every output tells of its sum: float32
    sums of 1024 terms are within 1024 x 2^-24 of the sum of magnitudes, the
    sigmoid passes at most a quarter of that on and its own arithmetic 2^-22."""
    g = torch.Generator().manual_seed(B)
    w = lambda o, i: (torch.randn(o, i, generator=g) / i ** 0.5).numpy()
    net = L.MLP({"w1t": w(1024, 8192), "b1": torch.zeros(1024).numpy(), "w2t": w(1024, 1024),
                 "b2": torch.zeros(1024).numpy(), "w3t": 2 * w(78, 1024),
                 "b3": torch.randn(78, generator=g).numpy()})
    net.forward(torch.randn(B, 8192, generator=g).to(BF).cuda())
    h = net.a["h2"][:B].double()
    w3 = net.wb["w3t"].double()
    z = h @ w3.T.contiguous() + net.w["b3"].double()
    mag = h.abs() @ w3.T.abs().contiguous() + net.w["b3"].double().abs()
    out = net.a["out"][:B].double()
    assert float((z.abs() < 4).double().mean()) > 0.95 and float(z.std()) > 0.5
    assert bool(((torch.sigmoid(z) - out).abs() <= 0.25 * 1024 * 2.0 ** -24 * mag + 2.0 ** -22).all())
