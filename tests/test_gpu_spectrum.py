"""Power spectra at the edges of the transform's shapes: every remainder of
log2 len modulo the radix-8 passes, the largest single-workgroup length and the
first of each split into two factors, contiguous and strided.

Tolerance: a float64 transform of N points is off by a few eps log2 N of the
sequence's norm; |X|^2 doubles it, and both sides round: 16 eps log2 N of the
largest value."""
import numpy as np
import pytest
import torch

from oracle.spectra import periodogram

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_seq", [(16, 3), (32, 1), (64, 2), (128, 5), (512, 2), (2048, 3), (4096, 97), (8192, 2),
                                     (16384, 3), (32768, 1), (1 << 19, 1), (1 << 20, 2), (1 << 22, 1), (1 << 23, 1)])
@pytest.mark.parametrize("win,strided", [("none", False), ("hann", True)])
def test_power_spectrum_shapes(N, n_seq, win, strided):
    from paper_1207_2192_amd import power_spectrum
    print(f"spectrum N={N} n_seq={n_seq} {win} strided={strided}", flush=True)
    rng = np.random.default_rng(N + n_seq)
    x = rng.standard_normal((n_seq, N)) + 0.3
    x[:, N // 3] += 2.0
    dev = torch.tensor(x, device="cuda")
    if strided:                       # samples apart by the number of sequences and a pad
        wide = torch.full((N, n_seq + 2), float("nan"), dtype=torch.float64, device="cuda")
        wide[:, :n_seq] = dev.t()
        dev = wide[:, :n_seq].t()
        assert dev.stride() == (1, n_seq + 2) and dev.reshape(-1, N).data_ptr() == dev.data_ptr()
    got = power_spectrum(dev, win == "hann", win).cpu().numpy()
    ref = periodogram(x, win == "hann", win)
    assert got.shape == (n_seq, N // 2 + 1)
    assert np.abs(got - ref).max() <= 16 * 2.2e-16 * np.log2(N) * ref.max()
