"""Rounding of the demagnetisation energy of large boxes.  The energy sums the field
along the magnetisation, so of the field's rounding it sees the gain of the twiddles
(the part of their rounding that is no rotation), which no average over cells takes
out.  Bounds: what transforms with plain radix-8 butterflies have on such states, the
root mean square over twelve of them, and 10 % for the states drawn."""
import numpy as np
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.demag import demag_fft

pytestmark = pytest.mark.gpu
C_PY = 0.14298555


@pytest.mark.parametrize("D,L,plain", [(250, 20.0, 7.51e-8), (200, 16.0, 1.90e-7), (150, 22.5, 1.11e-7)])
def test_energy_error_is_that_of_plain_butterflies(D, L, plain):
    from paper_1207_2192_amd import Disk, LLGParams
    n = 12
    disk, od = Disk.batch([float(D)] * n, [L] * n), oracle.Disk(float(D), L)
    rng = np.random.default_rng(D)
    states = []
    for _ in range(n):
        m = li.vortex_ansatz(D, *rng.uniform(-5.0, 5.0, 2)) + 0.1 * rng.standard_normal((3, D, D))
        states.append(torch.tensor(m / np.linalg.norm(m, axis=0), dtype=torch.float32) * od.mask)
    got = disk.energy(disk.pack([s.cuda() for s in states]), LLGParams(c=C_PY))[:, 2].cpu()
    ref = torch.stack([-0.5 * C_PY * (s.double() * demag_fft(s.double(), od) * od.mask).sum() for s in states])
    rms = float((((got - ref) / ref) ** 2).mean().sqrt())
    print(f"D={D} rms {rms:.3e}", flush=True)
    assert rms <= 1.1 * plain
