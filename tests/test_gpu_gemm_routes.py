"""The bf16 products at the lines between their kernels: a long K whose parts are
taken side by side, few rows at the line of tiles x K, few columns over a short K.

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
