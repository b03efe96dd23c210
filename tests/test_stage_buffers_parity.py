"""Where a call's tensors lie: the boundary slot itself, addresses that are not whole 16-byte pieces, one buffer for the upstream and the
input gradient, or two that overlap in part.  Every placement gives the bits of separate, aligned buffers, in the calls that recompute and
in those that keep, with and without a second stream."""
import pytest
import torch

from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import StageConfig

pytestmark = pytest.mark.gpu


def step(c, place, dropout, keep=False):
    dt = torch.float32 if c.dtype == "f32" else torch.bfloat16
    T, h = c.micro_batch * c.seq_len, c.hidden
    g = torch.Generator(device="cuda").manual_seed(3)
    n = B.Stage(c, "cuda:0").params.numel()
    st = B.Stage(c, "cuda:0", params_flat=torch.empty(n, device="cuda").normal_(0, 0.05, generator=g).to(dt))
    if place == "side":
        st.set_side_stream(torch.cuda.Stream())
    if dropout:
        st.set_dropout_seed(11)
    data = [[torch.empty(T, h, device="cuda").normal_(0, 1, generator=g).to(dt) for _ in range(2)] for _ in range(2)]
    st.grad_accum_reset()
    ys, dxs = [], []

    def at(t):
        if place != "misaligned":
            return t.clone()
        v = torch.empty(t.numel() + 1, dtype=dt, device="cuda")[1:].view(T, h)
        return v.copy_(t)

    for m, (x, dy) in enumerate(data):
        x, dy, y = at(x), at(dy), torch.empty(T, h, dtype=dt, device="cuda")
        if place == "slot":
            x = st.boundary_slot(m).copy_(x)
        (st.forward_keep if keep else st.forward)(m, x, y)
        if place != "slot":
            x.fill_(float("nan"))   # the slot holds it now
        dx = torch.empty_like(y)
        if place == "same":
            dx = dy
        elif place == "overlap":   # dx starts a token (whole 16-byte pieces in every case) after dy, or before it
            both = torch.empty((T + 1) * h, dtype=dt, device="cuda")
            dy = both[m * h:m * h + T * h].view(T, h).copy_(dy)
            dx = both[(1 - m) * h:(1 - m) * h + T * h].view(T, h)
        (st.backward_stored if keep else st.backward_recompute)(m, dy, dx)
        ys.append(y)
        dxs.append(dx.clone())
        if place not in ("same", "overlap"):
            dy.fill_(float("nan"))   # in order on the stream: the call has read it
    st.grad_flush()
    return torch.stack(ys), torch.stack(dxs), st.grads.clone()


@pytest.mark.parametrize("place", ["misaligned", "same", "side", "slot", "overlap"])
@pytest.mark.parametrize("dtype,h,heads,s,group,dropout", [("f32", 128, 2, 64, 1, 0.0), ("f32", 60, 3, 33, 1, 0.0), ("bf16", 256, 4, 128, 1, 0.0),
                                                           ("bf16", 256, 4, 128, 2, 0.0), ("bf16", 256, 4, 128, 1, 0.1), ("bf16", 200, 5, 70, 1, 0.0)])
@pytest.mark.parametrize("layers", [1, 2])
def test_placement(place, dtype, h, heads, s, group, dropout, layers):
    c = StageConfig("case", layers, h, heads, s, 2, 2, 4 * h, True, dtype, wgrad_group=group, dropout_p=dropout)
    for a, b in zip(step(c, "apart", dropout), step(c, place, dropout)):
        assert bool(torch.isfinite(a.float()).all()) and torch.equal(a, b)


@pytest.mark.parametrize("place", ["misaligned", "same", "side", "slot", "overlap"])
@pytest.mark.parametrize("dtype,h,heads,s,group,dropout", [("f32", 60, 3, 33, 1, 0.0), ("bf16", 256, 4, 128, 1, 0.1), ("bf16", 256, 4, 128, 2, 0.0), ("bf16", 200, 5, 70, 1, 0.0)])
def test_placement_of_kept_forwards(place, dtype, h, heads, s, group, dropout):
    c = StageConfig("case", 2, h, heads, s, 2, 2, 4 * h, True, dtype, wgrad_group=group, dropout_p=dropout)
    for a, b in zip(step(c, "apart", dropout), step(c, place, dropout, keep=True)):
        assert bool(torch.isfinite(a.float()).all()) and torch.equal(a, b)
