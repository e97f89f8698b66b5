"""Rounding of the power spectra, against the same transform in extended precision.

The sequences are a few lines on weak noise, as a recorded <m_x> is: their error
sits in the lines, where every rounding of a twiddle or of a last addition arrives
undivided.  Tolerance: the root mean square over 64 sequences of |P - P_exact| /
|P_exact| stays below one unit of rounding, 2^-52.  (A radix-2 transform with every
twiddle taken from the sine, at two roundings of a product and one of a sum a level
whose contributions halve from the last level back, has 1.6e-16 to 2.3e-16;
twiddles formed as a chain of seven products have 3e-16 to 5e-16.)"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [16, 64, 256, 1024, 2048, 4096, 8192, 16384, 1 << 16])
def test_spectra_are_exact_to_a_rounding(N):
    from paper_1207_2192_amd import power_spectrum
    rng = np.random.default_rng(N)
    n = 64
    f, a, ph = (rng.uniform(lo, hi, (n, 3, 1)) for lo, hi in ((0.001, 0.4), (0.002, 0.05), (0.0, 6.28)))
    x = (a * np.sin(2.0 * np.pi * f * np.arange(N) + ph)).sum(axis=1) + 0.01 + 0.003 * rng.standard_normal((n, N))
    X = np.fft.rfft(x.astype(np.longdouble), axis=-1)
    ref = (X.real ** 2 + X.imag ** 2) / N
    assert ref.dtype == np.longdouble and np.finfo(np.longdouble).eps < 1e-18
    got = power_spectrum(torch.tensor(x, device="cuda"), False, "none").cpu().numpy().astype(np.longdouble)
    err = np.linalg.norm((got - ref).astype(np.float64), axis=1) / np.linalg.norm(ref.astype(np.float64), axis=1)
    rms = float(np.sqrt((err ** 2).mean()))
    print(f"N={N} rms {rms:.2e} max {err.max():.2e}", flush=True)
    assert rms <= 2.0 ** -52
