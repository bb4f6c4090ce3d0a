"""Several wavelengths per column block in shuffled order: a long wavelength between short ones is
transformed on columns that nothing has written for it, and what those hold must not reach a result."""
import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


# split transforms with four and eight wavelengths per block, the unpadded split (one), the staged
# form with two (other radix plans; unpadded 1024 points), and the LDS-resident path beside them
@pytest.mark.parametrize("n,pad,n_wl,opts", [(64, 2, 2100, dict(schedule=1)), (64, 2, 2100, {}), (128, 2, 1100, {}),
                                             (128, 2, 2500, {}), (256, 2, 1050, {}), (256, 2, 300, dict(force_plan=1)),
                                             (512, 2, 140, dict(force_plan=1)), (256, 1, 600, {}), (1024, 1, 140, {}),
                                             (128, 2, 1100, dict(schedule=2)), (128, 2, 1100, dict(checkpoint_mode=1))])
def test_long_wavelengths_between_short_ones(n, pad, n_wl, opts):
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # 200 nm pitch: discs from every column (400 nm) down to an eighth of them (3.2 um)
    g = np.random.default_rng(n_wl)
    wl = np.where(g.random(n_wl) < 0.5, g.uniform(380e-9, 400e-9, n_wl), g.uniform(800e-9, 3.2e-6, n_wl))
    d = wk.make_design(n=n, layers=2, wl=wl, n_mat=1.5, dx=200e-9, z=9e-6, fov=16, pad=pad)
    plan = dpx.Plan([d], **opts)
    gen = torch.Generator(device="cuda").manual_seed(n)
    h = torch.rand(plan.h_count, device="cuda", generator=gen) * 1.1e-6
    dl = torch.randn(plan.img_count, device="cuda", generator=gen)
    # NaN on every column that the short wavelengths reach, then the shuffled set
    plan.set_wavelengths(0, np.full(n_wl, 390e-9), np.full(n_wl, 1.5))
    nan = torch.full_like(h, float("nan"))
    plan.forward(nan)
    plan.backward(nan, None, dl)
    plan.set_wavelengths(0, wl, d["n_mat"])
    image = plan.forward(h).reshape(n_wl, -1)
    dh = plan.backward(h, None, dl)
    assert bool(torch.isfinite(image).all()) and bool(torch.isfinite(dh).all())
    # a few wavelengths alone, on planes of their own: the same bits
    pick = [0, 1, 2, 3, n_wl // 2, n_wl // 2 + 1, n_wl - 2, n_wl - 1]
    few = dpx.Plan([wk.subset_wavelengths(d, pick)], **opts)
    assert torch.equal(few.forward(h).reshape(len(pick), -1), image[pick])
    few.close()
    plan.close()
