"""The count by which the loss launch finds its last block, after calls of one plan that overlapped."""
import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_wl,t", [(1, 8), (2, 32), (7, 32), (256, 32), (5, 96)])
def test_loss_after_overlapping_calls(n_wl, t):
    """Calls of one plan on two streams race for its per-wavelength sums (here they write the same
    values), but must not leave anything behind: later calls each write the loss again."""
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = np.linspace(450e-9, 700e-9, n_wl) if n_wl > 1 else np.array([600e-9])
    d = wk.make_design(n=96, layers=1, wl=wl, n_mat=wk.cauchy_index(wl), dx=300e-9, z=9e-6, fov=t, pad=2)
    plan = dpx.Plan([d])
    g = torch.Generator(device="cuda").manual_seed(n_wl)
    image = torch.rand(plan.img_count, device="cuda", generator=g)
    target = torch.rand(plan.img_count, device="cuda", generator=g)
    ref, _ = plan.loss(image, target)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [(torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty_like(image)) for _ in streams]
    torch.cuda.synchronize()
    for _ in range(40):
        for s, (l, dl) in zip(streams, outs):
            plan.loss(image, target, l, dl, stream=s)
    torch.cuda.synchronize()
    for _ in range(3):
        out = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda")
        plan.loss(image, target, out)
        assert torch.equal(out, ref)
    plan.close()
