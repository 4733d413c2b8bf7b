"""The MLP backward's scratch laid out by a caller that reuses memory: dz3 and
dh2 are read by no product once the next layer's gradient is formed, so dh1 or
a weight gradient may lie over them.  Gradients are bit for bit those of
separate buffers."""
import pytest
import torch

pytestmark = pytest.mark.gpu

BATCH, D_IN, D_H, D_OUT = 300, 192, 128, 78


@pytest.mark.parametrize("over", ["dz3 = dh1", "dz3 = gw2t", "dz3 = gw1t", "dh2 = gw1t"])
@pytest.mark.parametrize("workspace", [True, False])
def test_scratch_reused(over, workspace):
    from paper_2104_12922_amd import learned as Lr
    L, s = Lr.lib(), torch.cuda.current_stream().cuda_stream
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *n: torch.randn(*n, generator=g, device="cuda")
    bf, f32 = torch.bfloat16, torch.float32
    x, h1, h2 = rnd(BATCH, D_IN).to(bf), rnd(BATCH, D_H).to(bf), rnd(BATCH, D_H).to(bf)
    h1pre, h2pre = rnd(BATCH, D_H), rnd(BATCH, D_H)
    w2t, w3t = (rnd(D_H, D_H) / 8).to(bf), (rnd(D_OUT, D_H) / 8).to(bf)
    out, target = torch.rand(BATCH, D_OUT, generator=g, device="cuda"), rnd(BATCH, D_OUT)
    n = L.synth_mlp_workspace(BATCH, D_IN, D_H, D_OUT)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")

    def gradients(alias):
        b = {k: torch.zeros(*d, dtype=f32, device="cuda") for k, d in
             (("gw1t", (D_H, D_IN)), ("gb1", (D_H,)), ("gw2t", (D_H, D_H)), ("gb2", (D_H,)),
              ("gw3t", (D_OUT, D_H)), ("gb3", (D_OUT,)))}
        b.update({k: torch.zeros(BATCH, d, dtype=bf, device="cuda") for k, d in
                  (("dz3", D_OUT), ("dh2", D_H), ("dh1", D_H))})
        b["loss"] = torch.zeros(BATCH, dtype=torch.float64, device="cuda")
        ptr = {k: v.data_ptr() for k, v in b.items()}
        if alias:                              # both in one buffer of the larger's size
            small, large = alias.split(" = ")
            size = max(b[k].numel() * b[k].element_size() for k in (small, large))
            shared = torch.zeros(size, dtype=torch.uint8, device="cuda")
            ptr[small] = ptr[large] = shared.data_ptr()
            v = b[large]
            b[large] = shared[:v.numel() * v.element_size()].view(v.dtype).view(v.shape)
        st = L.synth_mlp_backward(
            BATCH, D_IN, D_H, D_OUT, x.data_ptr(), w2t.data_ptr(), w3t.data_ptr(), h1pre.data_ptr(),
            h1.data_ptr(), h2pre.data_ptr(), h2.data_ptr(), out.data_ptr(), target.data_ptr(),
            ptr["gw1t"], ptr["gb1"], ptr["gw2t"], ptr["gb2"], ptr["gw3t"], ptr["gb3"], ptr["dz3"],
            ptr["dh2"], ptr["dh1"], ptr["loss"], ws.data_ptr() if workspace else None,
            n if workspace else 0, s)
        assert st == 0
        torch.cuda.synchronize()
        return {k: v for k, v in b.items() if k.startswith("g")}

    ref, got = gradients(None), gradients(over)
    for k, v in ref.items():
        assert torch.equal(v, got[k]), k
    assert float(ref["gb3"].abs().max()) > 0
