"""dL/dh written over an input of the backward call: plans with a single gradient slot, whose passes
write it themselves, and plans that reduce their slots at the end."""
import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


ONE = [(32, 2, 1, 0), (64, 1, 1, 0), (32, 2, 1, 1), (64, 2, 1, 0)]  # n, pad, n_wl, schedule
SEVERAL = [(32, 2, 5, 0)]


# a single layer and wavelength for dl_di, two layers for u_in: arrays as long as the gradient
@pytest.mark.parametrize("n,pad,n_wl,schedule,over", [c + ("dl_di",) for c in ONE] +
                         [c + (o,) for o in ("h", "u_in") for c in ONE + SEVERAL])
def test_gradient_in_place_of_an_input(n, pad, n_wl, schedule, over):
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    layers = 1 if over == "dl_di" else 2
    wl = np.linspace(450e-9, 700e-9, n_wl) if n_wl > 1 else np.array([600e-9])
    d = wk.make_design(n=n, layers=layers, wl=wl, n_mat=wk.cauchy_index(wl), dx=300e-9, z=9e-6, fov=n, pad=pad)
    plan = dpx.Plan([d], schedule=schedule)
    g = torch.Generator(device="cuda").manual_seed(n)
    h = torch.rand(plan.h_count, device="cuda", generator=g) * 1.1e-6
    u = torch.randn(2 * plan.u_count, device="cuda", generator=g)
    dl = torch.randn(plan.img_count, device="cuda", generator=g)
    plan.forward(h, u)
    ref = plan.backward(h, u, dl).clone()
    out = {"h": h, "u_in": u, "dl_di": dl}[over]
    plan.backward(h, u, dl, out=out)
    assert torch.equal(out, ref)
    plan.close()
