"""Small disks resident on one CU (every disk of the handle has FFT size 64 and
no explicit plan): boxes at the edges of the row tiles (one cell, one row pair,
four rows per wavefront, the full 32) against the float64 oracle and against the
persistent plan of the same handle.

Tolerances as in test_gpu_parity.py: fields and right-hand sides 1e-5 norm-wise,
energies 1e-6 of the total, states after a few steps 2e-6 absolute (5e-6 for the
thermal steps); two plans differ by float32 rounding of the transforms, within
the sum of their bounds against the oracle."""
import numpy as np
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.demag import demag_fft
from oracle.dynamics import heun_step as o_heun, llg_rhs as o_rhs, rk4_step as o_rk4
from oracle.observables import energy as o_energy, mean_m as o_mean

pytestmark = pytest.mark.gpu
C_PY = 0.14298555
BOXES = [1, 2, 3, 4, 5, 8, 15, 16, 17, 29, 30, 31, 32]


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda").reshape(-1).contiguous()


def rel(got, ref):
    return float((got - ref).abs().max() / ref.abs().max())


@pytest.mark.parametrize("D", BOXES)
def test_resident_matches_oracle(D):
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.build(float(D), 0.3 * D + 1.0)
    od = oracle.Disk(float(D), 0.3 * D + 1.0)
    print(f"resident D={D}", flush=True)
    assert disk.workgroups == [1] and disk.launch_shape()[2] == 512
    m0 = li.random_unit_field(D, 60 + D)
    m64 = torch.tensor(m0, dtype=torch.float32).double()
    junk = dev(m0).view(3, D, D)
    junk[:, ~od.mask.cuda()] = float("nan")          # cells outside the disk are never read
    m = junk.reshape(-1).contiguous()
    H = disk.demag_field(m).view(3, D, D).double().cpu()
    assert rel(H, demag_fft(m64, od)) <= 1e-5
    assert float(H[:, ~od.mask].abs().sum()) == 0.0
    kw = dict(alpha=0.1, c=C_PY, dtau=0.04, hext=(0.02, -0.01, 0.005), hac=(0.0, 0.1, 0.0), freq=0.01, phase=0.4)
    p, po = LLGParams(**kw), oracle.Params(**kw)
    assert rel(disk.rhs(m, p).view(3, D, D).double().cpu(), o_rhs(m64, od, po)) <= 1e-5
    e, eo = disk.energy(m, p).cpu()[0], o_energy(m64, od, po)
    scale = max(abs(v) for v in eo)
    for k in range(4):
        assert abs(float(e[k]) - eo[k]) <= 1e-6 * scale + 1e-12, k
    a = m.clone()
    rec = torch.full((8 * 4 * disk.state_size,), float("nan"), device="cuda")
    ser = disk.rk4_series(a, 4, p, 3).cpu()
    b, c = m.clone(), m.clone()
    disk.rk4_step(b, 4, p)
    disk.rk4_record(c, 4, p, rec)
    disk.check()
    assert torch.equal(a, b) and torch.equal(b, c) and bool(torch.isfinite(rec).all())
    assert torch.equal(rec[:3 * D * D].view(3, D, D).cpu(), (m64 * od.mask).float())
    ref = o_rk4(m64, od, po, 4)
    assert float((a.view(3, D, D).double().cpu() - ref).abs().max()) <= 2e-6
    state = m64
    for s in (0, 3):
        ps = oracle.Params(**dict(kw, tau0=s * 0.04))
        for q in range(3):
            assert abs(float(ser[s // 3, 0, q]) - o_mean(state, od)[q]) <= 2e-6
        es = o_energy(state, od, ps)
        assert abs(float(ser[s // 3, 0, 3]) - es[0]) <= 4e-6 * max(abs(v) for v in es)
        state = o_rk4(state, od, po, 3)


def test_resident_ensemble_heun_noise_and_plans_agree():
    # more disks than CUs, mixed boxes; the persistent plans of the same handle within rounding
    from paper_1207_2192_amd import Disk, LLGParams
    n = 300
    Ds = [BOXES[(5 * k) % len(BOXES)] for k in range(n)]
    batch = Disk.batch([float(D) for D in Ds], [5.0] * n)
    assert batch.workgroups == [1] * n
    kw = dict(alpha=0.1, c=C_PY, temp=0.0319, dtau=0.0266, renorm=True)
    states = [li.smooth_random_field(D, 5 + k) for k, D in enumerate(Ds)]
    m0 = batch.pack([dev(s) for s in states])
    m = m0.clone()
    batch.set_step(41)
    batch.heun_step(m, 5, LLGParams(**kw), seed=91, step0=None, replica=3)
    batch.check()
    assert batch.get_step() == 46
    for k in (0, 1, 2, 7, 150, 299):
        od = oracle.Disk(float(Ds[k]), 5.0)
        o = o_heun(torch.tensor(states[k]), od, oracle.Params(**kw), seed=91, step0=41, replica=3 + k, nsteps=5)
        assert float((batch.unpack(m, k).double().cpu() - o).abs().max()) <= 5e-6, k
    other = m0.clone()
    batch.tune(1, None, 0)
    assert batch.launch_shape()[2] == 192
    batch.heun_step(other, 5, LLGParams(**kw), seed=91, step0=41, replica=3)
    batch.check()
    assert float((other - m).abs().max()) <= 1e-5


def test_resident_graph_noalloc_and_bad_states():
    import ctypes
    from paper_1207_2192_amd import Disk, LLGParams, _lib
    disk = Disk.batch([30.0, 17.0], [10.0, 4.0])
    m0 = disk.pack([dev(li.vortex_ansatz(D, 1.0, 2.0)) for D in disk.D])
    p = LLGParams(alpha=0.1, c=C_PY, dtau=0.0266, temp=0.008, renorm=True)
    mg, me = m0.clone(), m0.clone()
    disk.set_step(7)
    g = disk.graph("heun", mg, 6, p, seed=77, replica=5)
    for rep in range(3):
        g.launch()
        float(torch.randn(1 << 18, device="cuda").sum())
        disk.heun_step(me, 6, p, seed=77, step0=7 + 6 * rep, replica=5)
        torch.cuda.synchronize()
        disk.check()
        assert torch.equal(mg, me), rep
    g.close()
    a, b = m0.clone(), m0.clone()
    disk.rk4_step(a, 9, p)
    lib = _lib.load()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert lib.llg_rk4_step_noalloc(disk._h, ctypes.c_void_p(b.data_ptr()), 9, disk._params(p), stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    b[30 * 15 + 15] = float("inf")
    disk.rk4_step(b, 2, p)
    with pytest.raises(_lib.LLGError, match="non-finite"):
        disk.check()
