"""The loss on image sizes around the edges of its forms: pixels per thread kept in registers (1, 4, 16
or none) and blocks of 256 or 1024 threads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t", [1, 7, 16, 17, 32, 33, 64, 65, 90, 91, 128, 129])
def test_loss_and_gradient_against_double(t):
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n_wl = 3
    g = np.random.default_rng(t)
    image = g.random((n_wl, t, t)).astype(np.float32)
    target = g.random((n_wl, t, t)).astype(np.float32)
    dev = lambda a: torch.as_tensor(a.reshape(-1)).cuda()  # noqa: E731
    loss, dl = dpx.loss_static(dev(image), dev(target), n_wl, t)
    i, tau = image.astype(np.float64), target.astype(np.float64)
    s = i.sum((1, 2), keepdims=True)
    rel = i / s
    diff = rel - tau / tau.sum((1, 2), keepdims=True)
    ref = (diff ** 2).mean()
    grad = 2.0 / (n_wl * t * t) / s * (diff - (diff * rel).sum((1, 2), keepdims=True))
    # sums in double; the differences cancel to at worst a few ulp of the terms (2^-52 of 1 / t^2)
    assert abs(loss.item() - ref) <= 1e-12 * ref + 1e-30
    # rounded to single once
    assert np.abs(dl.cpu().numpy().reshape(grad.shape) - grad).max() <= 2.0 ** -24 * np.abs(grad).max() + 1e-22 / t ** 4
