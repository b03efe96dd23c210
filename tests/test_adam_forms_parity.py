"""The Adam update through and past the caches: one rule on the number of parameters, the same arithmetic."""
import pytest
import torch

from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import StageConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,h,f", [("f32", 64, 250), ("bf16", 1024, 5000), ("bf16", 1024, 6500), ("f32", 1024, 8300)])
def test_adam_step_sizes(dtype, h, f):
    """fp32 arithmetic against 64 bits after one step: 1e-6, as for the mini-batch tail; the parameter is the rounded master."""
    cfg = StageConfig("adam", 1, h, 1 if h < 256 else 8, 8, 1, 1, f, True, dtype)
    n = B.query_sizes(cfg)[0] // (4 if dtype == "f32" else 2)
    g = torch.Generator(device="cuda").manual_seed(4)
    w, m, grad = (torch.empty(n, device="cuda").normal_(0, s, generator=g) for s in (0.02, 1e-3, 0.05))
    v = m.square()
    st = B.Stage(cfg, "cuda:0", params_flat=w.to(torch.float32 if dtype == "f32" else torch.bfloat16))
    st.grads.copy_(grad)
    lr, b1, b2, eps, wd, gs = 1e-3, 0.9, 0.95, 1e-8, 0.01, 0.5
    gd = grad.double() * gs
    md, vd = b1 * m.double() + (1 - b1) * gd, b2 * v.double() + (1 - b2) * gd * gd
    wd64 = w.double() - lr * (md / (1 - b1 ** 3) / ((vd / (1 - b2 ** 3)).sqrt() + eps) + wd * w.double())
    st.adam_step(w, m, v, 3, lr=lr, beta1=b1, beta2=b2, eps=eps, weight_decay=wd, grad_scale=gs)
    for got, want in ((w, wd64), (m, md), (v, vd)):
        assert float((got.double() - want).norm() / want.norm()) <= 1e-6
    assert torch.equal(st.params, w.to(st.params.dtype))
    st.close()
