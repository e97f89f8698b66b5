"""<m>, core position and energy over the shapes of their kernels: disks of one
strip and of several in one batch, the last strip partly filled, lone disks on
both sides of the row-strip threshold, and batches on both launch shapes of the
field kernels (few tiles, many tiles per CU) with odd boxes and every FFT size.

The reductions are float64 sums over at most 49080 cells of float32 values:
<m> and the core position agree with the oracle to 1e-12 and 1e-9 (as in
test_gpu_parity.py), the energy parts to 1e-6 of the total (float32 fields)."""
import numpy as np
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.demag import demag_fft
from oracle.observables import energy as o_energy, mean_m as o_mean, vortex_core_position as o_core

pytestmark = pytest.mark.gpu
C_PY, LAM_NM = 0.14298555, 5.28906


@pytest.mark.parametrize("Ds", [[96], [97], [113], [16, 97, 17, 250], [31, 33, 64, 65, 100, 129, 12, 5, 127],
                                [120] * 24 + [49], [250, 131, 40] * 6])
@pytest.mark.parametrize("hint", [False, True])
def test_observables_match_oracle(Ds, hint):
    from paper_1207_2192_amd import Disk, LLGParams
    n = len(Ds)
    disk = Disk.batch([float(D) for D in Ds], [0.2 * D for D in Ds]) if n > 1 else Disk.build(float(Ds[0]), 0.2 * Ds[0])
    print(f"observables D={Ds}", flush=True)
    states = [li.vortex_ansatz(D, 0.1 * D + 0.3, -0.07 * D) for D in Ds]
    m = disk.pack([torch.tensor(s, dtype=torch.float32, device="cuda").reshape(-1) for s in states])
    p = LLGParams(c=C_PY, hext=(0.01, -0.02, 0.03))
    mean, e = disk.mean_m(m).cpu(), disk.energy(m, p).cpu()
    H = disk.demag_field(m)
    core = disk.vortex_core_position(m, LAM_NM, [(0.2 * D, -0.1 * D) for D in Ds] if hint else None).cpu()
    disk.check()
    for k in sorted({0, 1, n // 2, n - 2, n - 1} & set(range(n))):
        od = oracle.Disk(float(Ds[k]), 0.2 * Ds[k])
        m64 = torch.tensor(states[k], dtype=torch.float32).double()
        ref = o_mean(m64, od)
        assert all(abs(float(mean[k, q]) - ref[q]) <= 1e-12 for q in range(3)), k
        rc = o_core(m64, od, LAM_NM, (0.2 * Ds[k], -0.1 * Ds[k]) if hint else None)
        assert int(core[k, 4]) == rc[4]
        # (a vortex centred on a column of cells has no +1 plaquette: r_v is NaN on both sides)
        assert np.allclose(core[k, :4].numpy(), rc[:4], rtol=1e-9, atol=1e-9, equal_nan=True), k
        eo = o_energy(m64, od, oracle.Params(c=C_PY, hext=(0.01, -0.02, 0.03)))
        assert all(abs(float(e[k, q]) - eo[q]) <= 1e-6 * abs(eo[0]) for q in range(4)), k
        ho = demag_fft(m64, od)
        assert float((disk.unpack(H, k).double().cpu() - ho).abs().max()) <= 1e-5 * float(ho.abs().max()), k
    disk.close()
