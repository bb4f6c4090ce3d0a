"""Split column transforms of 800-point halves (transform 1600): every source of the transfer function,
with wavelengths whose disc leaves columns out and a partial range of rows."""
import numpy as np
import pytest

from oracle import dpx_oracle as o
from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("option", ["mirrored", "narrow", "shift", "band", "fov"])
def test_column_halves_of_800_points(option):
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = np.array([410e-9, 633e-9, 900e-9])
    d = wk.make_design(n=800, layers=1, wl=wl, n_mat=wk.cauchy_index(wl), dx=200e-9, z=9e-6,
                       fov=6 if option == "fov" else 800, pad=2)
    d["band_limited"] = option == "band"
    if option == "shift":  # the plan takes the offsets from the design
        d["shift_x"], d["shift_y"] = np.array([35e-9]), np.array([-120e-9])
    g = np.random.default_rng(800)
    h = (g.random((1, 800, 800)) * 1.1e-6).astype(np.float32)
    plan = dpx.Plan([d], force_variant=0 if option == "narrow" else -1)
    I = plan.forward(plan.pack_heights([h]))
    torch.cuda.synchronize()
    I_ref = o.forward(d, h, None, "fft")
    I = I.cpu().numpy().reshape(I_ref.shape)
    # intensities against the FP64 oracle, relative L2 per wavelength
    for w in range(3):
        assert np.linalg.norm(I[w] - I_ref[w]) <= 1e-5 * np.linalg.norm(I_ref[w])
    plan.close()


@pytest.mark.parametrize("option", ["mirrored", "shift", "band", "fov"])
def test_one_wavelength_alone(option):
    """A launch of one wavelength runs the halves on different wavefronts: the bits of the same wavelength
    among three, and the oracle's gradient."""
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = np.array([410e-9, 633e-9, 900e-9])
    fov = 6 if option == "fov" else 800
    d = wk.make_design(n=800, layers=2, wl=wl, n_mat=wk.cauchy_index(wl), dx=200e-9, z=9e-6, fov=fov, pad=2)
    d["band_limited"] = option == "band"
    if option == "shift":
        d["shift_x"], d["shift_y"] = np.array([35e-9, 0.0]), np.array([-120e-9, 50e-9])
    g = np.random.default_rng(801)
    h = (g.random((2, 800, 800)) * 1.1e-6).astype(np.float32)
    three = dpx.Plan([d])
    I = three.forward(three.pack_heights([h])).cpu().numpy().reshape(3, fov, fov)
    three.close()
    for w in (0, 2):
        one = wk.subset_wavelengths(d, [w])
        plan = dpx.Plan([one])
        ht = plan.pack_heights([h])
        I1 = plan.forward(ht).cpu().numpy().reshape(fov, fov)
        assert np.array_equal(I1, I[w])
        dl = g.standard_normal((1, fov, fov)).astype(np.float32)
        dh = plan.backward(ht, None, plan.pack_images([dl])).cpu().numpy().reshape(h.shape)
        plan.close()
        ref = o.grad(one, h, None, dl, "fft")
        assert np.linalg.norm(dh - ref) <= 1e-4 * np.linalg.norm(ref)
