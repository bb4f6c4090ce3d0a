"""Row passes with too few rows to fill the chip run in blocks of 128 threads; the rows and their
binning are the same as in the larger blocks."""
import numpy as np
import pytest

from oracle import dpx_oracle as o
from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


# each wave-local length; fields of view that leave the last block short, and bins that a small block
# holds whole (several to a block, or exactly one) or does not (8 rows of 64 lanes)
@pytest.mark.parametrize("n,pad,fov,b", [(32, 2, 24, 8), (64, 2, 36, 4), (96, 2, 50, 2), (128, 2, 72, 8), (192, 2, 90, 2),
                                         (256, 2, 132, 4), (512, 2, 264, 8), (96, 1, 66, 2), (512, 1, 260, 4)])
def test_few_rows_give_the_bits_of_many(n, pad, fov, b):
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # 1 + 2 wavelengths are fewer than 256 blocks of any pass here, n_wl of them are more
    n_wl = 300 if n <= 128 else 100
    wl = np.linspace(450e-9, 700e-9, n_wl)
    d = wk.make_design(n=n, layers=2, wl=wl, n_mat=wk.cauchy_index(wl), dx=4e-6, z=0.05 * n / 400, fov=fov, bin_=b,
                       pad=pad)
    few_d = wk.subset_wavelengths(d, [0, n_wl - 1])
    g = np.random.default_rng(n + b)
    h = (g.random((2, n, n)) * 1.1e-6).astype(np.float32)
    t = fov // b
    seed = np.zeros((n_wl, t, t), np.float32)
    I_ref = o.forward(few_d, h, None, "fft")
    _, g_ref, _ = o.loss(I_ref, g.random((2, t, t)))
    seed[[0, -1]] = g_ref
    out = []
    for dd, dl in ((d, seed), (few_d, seed[[0, -1]])):
        plan = dpx.Plan([dd], schedule=1)
        assert not plan.uses_lds_path()
        ht = plan.pack_heights([h])
        I = plan.forward(ht)
        dh = plan.backward(ht, None, plan.pack_images([dl]))
        torch.cuda.synchronize()
        out.append((I.cpu().numpy().reshape(dd["wl"].size, t, t), dh.cpu().numpy().reshape(h.shape)))
        plan.close()
    I = out[1][0]
    assert np.array_equal(I, out[0][0][[0, -1]])
    for w in range(2):
        assert np.linalg.norm(I[w] - I_ref[w]) <= 1e-5 * np.linalg.norm(I_ref[w])
    dh_ref = o.grad(few_d, h, None, seed[[0, -1]], "fft")
    for _, dh in out:  # the other wavelengths' seeds are zero
        assert np.linalg.norm(dh - dh_ref) <= 1e-4 * np.linalg.norm(dh_ref)
