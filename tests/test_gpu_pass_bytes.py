"""The algorithmic bytes and operations that the per-pass timers report count the spectrum columns that
carry propagating waves, which are the ones that the passes move."""
import math

import numpy as np
import pytest

from paper_2604_02624_amd import workloads as wk

pytestmark = pytest.mark.gpu


def design(n, n_wl, lo, hi, fov, bin_=1, pad=2):
    wl = np.linspace(lo, hi, n_wl)
    return wk.make_design(n=n, layers=3, wl=wl, n_mat=wk.cauchy_index(wl), dx=200e-9, z=9e-6, fov=fov, bin_=bin_, pad=pad)


def columns(d, wl):
    """Columns kx with kx^2 < (M dx n / lambda)^2, over the wavelengths."""
    m = d["n"] * d["pad"]
    kx = np.arange(m)
    kx = np.where(kx < m // 2, kx, kx - m).astype(np.float64)
    return int(sum((kx ** 2 < (m * d["dx"] * d["n_medium"] / x) ** 2).sum() for x in wl))


def read(torch, plan, wl=None):
    if wl is not None:
        for i, w in enumerate(wl):
            plan.set_wavelengths(i, w, wk.cauchy_index(w))
    h = torch.full((plan.h_count,), 5e-7, device="cuda")
    plan.timing(True)
    image = plan.forward(h)
    plan.backward(h, None, torch.ones_like(image))
    out = plan.timing_read()
    plan.timing(False)
    return {k: (v["bytes"], v["flops"]) for k, v in out.items() if v["launches"]}


def expected(d, wl):
    n, m, k, w = d["n"], d["n"] * d["pad"], d["layers"], len(wl)
    c, nn, f, t = columns(d, wl), n * n, d["fov"], d["fov"] // d["bin"]
    fft = 5.0 * m * math.log2(m)
    col = c * (2 * fft + 6.0 * m)
    full = (k - 1) * c * 8 * 2 * n
    last = c * 8 * (n + f)
    out = {"col_fwd": (full + last, k * col), "col_adj": (full + last, k * col),
           "col_fwd_full": (full, (k - 1) * col), "col_adj_full": (full, (k - 1) * col),
           "row_fwd_first": (c * 8 * n + 4 * nn, w * n * (fft + 6.0 * n)),
           "row_fwd_mid": ((k - 1) * (2 * c * 8 * n + w * 8 * nn + 4 * nn), (k - 1) * w * n * (2 * fft + 6.0 * n)),
           "row_fwd_last": (c * 8 * f + w * (8 * f * f + 4 * t * t), w * f * fft),
           "row_adj_seed": (c * 8 * f + w * (8 * f * f + 4 * t * t), w * f * fft)}
    return out


@pytest.mark.parametrize("n,n_wl,chunk", [(64, 6, 0), (128, 5, 0), (96, 7, 3), (512, 3, 0)])
def test_bytes_of_a_design(n, n_wl, chunk):
    """From wavelengths that fill every column to ones that leave most out, before and after rebinding."""
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = design(n, n_wl, 380e-9, 1200e-9, n // 2, 2)
    plan = dpx.Plan([d], schedule=1, wl_chunk=chunk)
    for wl in (d["wl"], np.linspace(500e-9, 2000e-9, n_wl)):
        got, want = read(torch, plan, None if wl is d["wl"] else [wl]), expected(d, wl)
        for k, (b, f) in want.items():
            if chunk and k in ("row_fwd_first", "row_fwd_mid"):
                continue  # each chunk reads the heights
            assert got[k][0] == b and abs(got[k][1] - f) <= 1e-12 * f, (k, got[k], (b, f))
    plan.close()


def test_bytes_of_grouped_designs():
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ds = [design(64, 5, 380e-9, 1200e-9, 32), design(64, 3, 600e-9, 900e-9, 32), design(96, 4, 450e-9, 1500e-9, 48, 2)]
    plan = dpx.Plan(ds, schedule=2)
    for wls in ([d["wl"] for d in ds], [d["wl"] * 1.4 for d in ds]):
        got = read(torch, plan, wls)
        want = [expected(d, wl) for d, wl in zip(ds, wls)]
        for k in want[0]:
            b, f = (sum(x[k][i] for x in want) for i in (0, 1))
            assert got[k][0] == b and abs(got[k][1] - f) <= 1e-12 * f, (k, got[k], (b, f))
    plan.close()


@pytest.mark.parametrize("variant,table", [(4, 0), (-1, 2)])
def test_bytes_of_other_column_passes(variant, table):
    """The matrix-core pass moves every column; a table adds the entries of the columns inside the disc."""
    import torch
    from paper_2604_02624_amd import dpx
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = design(64, 4, 380e-9, 1200e-9, 32)
    m, n, k, w = 128, 64, 3, 4
    plan = dpx.Plan([d], schedule=1, force_variant=variant, transfer_table=table)
    c = w * m if variant == 4 else columns(d, d["wl"])
    extra = (c + w) // 2 * (m // 2 + 1) * 8 if table else 0
    assert read(torch, plan)["col_fwd_full"][0] == (k - 1) * (c * 8 * 2 * n + extra)
    plan.close()
