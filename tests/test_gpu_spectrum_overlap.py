"""llg_power_spectrum with its result in the memory of its input, or in the
workspace: the same bits as with arrays of their own.  The results start in the
middle of the input, so that the first ones fall on sequences that are read last."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


def spectrum(x, n, N, work, out):
    from paper_1207_2192_amd import _lib
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (x, work, out)]
    _lib.check(_lib.load().llg_power_spectrum(ptr[0], n, N, N, 1, 1, 1, ptr[1], ptr[2],
                                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)), "spectrum")


@pytest.mark.parametrize("N,n", [(256, 20000), (8192, 700), (16384, 40), (32768, 17)])
@pytest.mark.parametrize("where", ["x", "work", "work behind", "x and work"])
def test_result_may_lie_in_the_input_or_the_workspace(N, n, where):
    print(f"N={N} n={n} out in {where}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + n)
    n_out = n * (N // 2 + 1)
    both = torch.zeros(2 * n * N + 4 * n * N, dtype=torch.float64, device="cuda")    # x, slack, work
    x, work = both[:n * N], both[2 * n * N:]
    x.copy_(torch.randn(n * N, dtype=torch.float64, device="cuda", generator=g))
    ref = torch.empty(n_out, dtype=torch.float64, device="cuda")
    spectrum(x.clone(), n, N, torch.empty(4 * n * N, dtype=torch.float64, device="cuda"), ref)
    at = {"x": n // 2 * N, "work": 2 * n * N, "work behind": 4 * n * N + 5 * N}.get(where)
    if where == "x and work":                   # the slack left out: the input ends where the workspace begins
        x2 = both[n * N:2 * n * N]
        x2.copy_(x)
        x, at = x2, 2 * n * N - n_out // 2
    out = both[at:at + n_out]
    spectrum(x, n, N, work, out)
    assert torch.equal(out, ref)
