"""Rounding of the field at every transform size, against the float64 oracle.

The field is a product of spectra with most of its weight in a few of them, so its
relative error is that of the transforms' twiddles.  Bounds: what plain radix-4 and
radix-8 transforms have on these states (vortices with a random tilt of 0.1 a cell,
root mean square over eight of them), whose twiddles are products of one table entry
at most three deep, with 2 % for the states drawn."""
import numpy as np
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.demag import demag_fft

pytestmark = pytest.mark.gpu
PLAIN = {12: 1.741e-7, 24: 2.700e-7, 32: 3.450e-7, 64: 5.818e-7, 125: 7.325e-7, 150: 7.881e-7, 200: 8.886e-7,
         250: 9.826e-7}


@pytest.mark.parametrize("D", sorted(PLAIN))
def test_field_error_is_that_of_plain_transforms(D):
    from paper_1207_2192_amd import Disk
    L = round(0.2 * D, 2)
    disk, od = Disk.batch([float(D)] * 8, [L] * 8), oracle.Disk(float(D), L)
    rng = np.random.default_rng(D)
    states = []
    for _ in range(8):
        m = li.vortex_ansatz(D, *rng.uniform(-0.1 * D, 0.1 * D, 2)) + 0.1 * rng.standard_normal((3, D, D))
        states.append(torch.tensor(m / np.linalg.norm(m, axis=0), dtype=torch.float32) * od.mask)
    H = disk.demag_field(disk.pack([s.cuda() for s in states])).view(8, 3, D, D).double().cpu()
    err = []
    for s, h in zip(states, H):
        ref = demag_fft(s.double(), od) * od.mask
        err.append(float((h - ref).norm() / ref.norm()))
    rms = float(np.sqrt(np.mean(np.square(err))))
    print(f"D={D} rms {rms:.3e}", flush=True)
    assert rms <= 1.02 * PLAIN[D]
