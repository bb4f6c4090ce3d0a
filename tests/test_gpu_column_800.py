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
