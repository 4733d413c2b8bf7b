"""The GEMM kernels at the edges of their tiles: whole-K tiles of 64 x 64,
128 x 128 and 256 x 128 in every operand layout, k that ends inside a 64-wide
stage, rows that end inside a tile, an operand without 16-byte rows, and the
few-row kernel and split sums behind the MLP.

Small-integer operands keep every float32 sum exact (|sum| <= 9 K < 2^24), so
those products must equal the integer product bit for bit.  Sums of general
values are held to K 2^-24 |A| |B|, the bound of K float32 additions."""

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


@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (8, 16, 8), (72, 200, 40), (200, 136, 1000),
                                   (1088, 1096, 72), (2056, 1032, 136), (1032, 4104, 520),
                                   (1600, 8192, 584)])
@pytest.mark.parametrize("a_layout,b_layout", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_whole_tiles_are_exact(L, M, N, K, a_layout, b_layout):
    g = torch.Generator().manual_seed(M + N + K)
    A, B = _ints((M, K), g), _ints((K, N), g)
    C = L.gemm_bf16((A if a_layout == 0 else A.T).contiguous().cuda(),
                    (B.T if b_layout == 0 else B).contiguous().cuda(), M, N, K, a_layout, b_layout)
    assert torch.equal(C.cpu(), A.float() @ B.float())


@pytest.mark.parametrize("M,N,K,a_layout", [(512, 1024, 78, 0), (130, 72, 77, 0), (78, 1024, 300, 1),
                                            (1100, 1024, 78, 0), (77, 64, 65, 1)])
def test_operand_without_16_byte_rows(L, M, N, K, a_layout):
    g = torch.Generator().manual_seed(M + N + K)
    A, B = _ints((M, K), g), _ints((K, N), g)
    bias = torch.randint(-5, 6, (N,), generator=g).float()
    pre = torch.empty(M, N, device="cuda")
    C = L.gemm_bf16((A if a_layout == 0 else A.T).contiguous().cuda(), B.cuda(), M, N, K, a_layout,
                    1, bias=bias.cuda(), pre=pre)
    ref = A.float() @ B.float() + bias
    assert torch.equal(C.cpu(), ref) and torch.equal(pre.cpu(), ref)


@pytest.mark.parametrize("B", [1, 31, 33, 128, 129, 256, 300, 513, 1000])
def test_mlp_forward_sums_are_exact(L, B):
    g = torch.Generator().manual_seed(B)
    init = {"w1t": _ints((1024, 8192), g).float().numpy(), "b1": torch.zeros(1024).numpy(),
            "w2t": _ints((1024, 1024), g).float().numpy(), "b2": torch.zeros(1024).numpy(),
            "w3t": _ints((78, 1024), g).float().numpy(), "b3": torch.zeros(78).numpy()}
    net = L.MLP(init)
    x = _ints((B, 8192), g)
    net.forward(x.cuda())
    ref = x.float() @ torch.from_numpy(init["w1t"]).T
    assert torch.equal(net.a["h1pre"].cpu(), ref)
    h1, h2 = net.a["h1"].cpu().double(), net.a["h2"].cpu().double()
    for h, w, got in ((h1, "w2t", net.a["h2pre"]), (h2, "w3t", torch.logit(net.a["out"].double()))):
        w = torch.from_numpy(init[w]).double()
        z = h @ w.T
        bound = 1024 * 2.0 ** -24 * (h.abs() @ w.abs().T)
        ok = (got.cpu().double() - z).abs() <= bound
        if w.shape[0] == 78:                  # through the float32 sigmoid: where it is not saturated
            ok |= z.abs() > 4
            ok |= (torch.sigmoid(z) - net.a["out"].cpu().double()).abs() <= bound + 2.0 ** -22
        assert bool(ok.all())


@pytest.mark.parametrize("B", [256, 333, 777, 2050])
def test_mlp_weight_gradients(L, B):
    import workloads as W
    g = torch.Generator().manual_seed(B)
    net = L.MLP(W.mlp_init(3))
    x = torch.randn(B, 8192, generator=g).to(BF).cuda()
    net.forward(x)
    net.backward(x, torch.rand(B, 78, generator=g).cuda())
    a = net.a
    for k, dz, h in (("w1t", a["dh1"], x), ("w2t", a["dh2"], a["h1"]), ("w3t", a["dz3"], a["h2"])):
        d, h = dz[:B].double(), h[:B].double()
        ref, mag = d.T.contiguous() @ h, d.abs().T.contiguous() @ h.abs()
        assert bool(((net.g[k].double() - ref).abs() <= B * 2.0 ** -24 * mag + 1e-30).all()), k
