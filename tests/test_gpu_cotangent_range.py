"""The backward is linear in dL/dI over the range of single precision."""
import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pad,schedule", [(32, 2, 0), (32, 2, 1), (48, 2, 1), (64, 2, 1), (96, 2, 1), (128, 2, 1), (192, 2, 1),
                                            (256, 2, 1), (512, 2, 1), (800, 2, 1), (64, 1, 0), (64, 1, 1), (96, 1, 1),
                                            (128, 1, 1), (192, 1, 1), (256, 1, 1), (384, 1, 1), (512, 1, 1)])
def test_gradients_of_scaled_cotangents(n, pad, schedule):
    """Powers of two scale every operation exactly, so the gradient scales with its bits.  At 2^96 the
    spectra reach about 2^108 and the gradients 2^121; at 2^-60 nothing comes near the denormals."""
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = np.array([450e-9, 700e-9])
    d = wk.make_design(n=n, layers=2, wl=wl, n_mat=wk.cauchy_index(wl), dx=200e-9, z=9e-6, fov=n // 2, pad=pad,
                       kappa=2e-4)
    plan = dpx.Plan([d], schedule=schedule)
    assert plan.uses_lds_path() == (schedule == 0)
    g = torch.Generator(device="cuda").manual_seed(n)
    h = torch.rand(plan.h_count, device="cuda", generator=g) * 1.1e-6
    dl = torch.randn(plan.img_count, device="cuda", generator=g)
    plan.forward(h)
    ref = plan.backward(h, None, dl)
    for e in (96, -60):
        assert torch.equal(plan.backward(h, None, dl * 2.0 ** e), ref * 2.0 ** e), e
    plan.close()
