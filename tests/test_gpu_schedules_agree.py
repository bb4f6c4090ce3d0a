"""The promise that every schedule gives the same bits, where a schedule picks its own kernels."""
import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


def design(n, pad, n_wl, layers, fov):
    wl = np.linspace(450e-9, 700e-9, n_wl) if n_wl > 1 else np.array([600e-9])
    return wk.make_design(n=n, layers=layers, wl=wl, n_mat=wk.cauchy_index(wl), dx=300e-9, z=9e-6, fov=fov, pad=pad)


def results(torch, designs, seed, **opts):
    """Intensities, and loss, dL/dI and dL/dh of a step on random heights and targets."""
    from paper_2604_02624_amd import dpx
    plan = dpx.Plan(designs, **opts)
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.rand(plan.h_count, device="cuda", generator=g) * 1.1e-6
    tau = torch.rand(plan.img_count, device="cuda", generator=g)
    image = plan.forward(h)
    loss, dl_di = plan.loss(image, tau)
    dl_dh = plan.backward(h, None, dl_di)
    torch.cuda.synchronize()
    out = [x.cpu().numpy() for x in (image, loss, dl_di, dl_dh)]
    kind = plan.schedule(), plan.uses_lds_path()
    plan.close()
    return out, kind


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# images on both sides of the size at which the loss takes larger blocks (8192 pixels), also in one
# plan, beyond what a large block keeps in registers, and counts of wavelengths on both sides of the
# single-launch sum
@pytest.mark.parametrize("fovs,n_wl", [((90, 92), 3), ((128, 128), 2), ((32, 96, 16, 94), 5), ((192, 64), 1), ((92, 92), 300)])
def test_grouped_and_per_design_losses(torch_dev, fovs, n_wl):
    designs = [design(96 if f <= 96 else f, 2 if f <= 128 else 1, n_wl + i, 1, f) for i, f in enumerate(fovs)]
    grouped, kind2 = results(torch_dev, designs, sum(fovs), schedule=2)
    single, kind1 = results(torch_dev, designs, sum(fovs), schedule=1)
    assert (kind2[0], kind1[0]) == (2, 1)
    for a, b in zip(grouped, single):
        assert np.array_equal(a, b)


# plans that run LDS-resident by themselves or on request against the passes: slots of one
# wavelength, and of several with a short last one
@pytest.mark.parametrize("n,pad,n_wl,small", [(32, 2, 2048, 0), (64, 2, 300, 0), (64, 2, 4096, 0), (64, 2, 9001, 0), (64, 1, 4099, 0),
                                              (64, 1, 6500, 0), (32, 2, 4500, 1), (48, 2, 6145, 1), (96, 1, 2500, 1)])
def test_lds_resident_plans_and_passes(torch_dev, n, pad, n_wl, small):
    d = design(n, pad, n_wl, 2, n // 2)
    lds, kind = results(torch_dev, [d], n_wl, small_path=small)
    passes, kind1 = results(torch_dev, [d], n_wl, schedule=1)
    assert (kind[1], kind1) == (True, (1, False))
    for a, b in zip(lds, passes):
        assert np.array_equal(a, b)
