"""When a trajectory's forward pass keeps stage records, on a disk that only counts its
calls (no GPU)."""
import pytest
import torch

from paper_1207_2192_amd import LLGParams, adjoint


class Counting:
    """The calls of a Disk that a trajectory makes; states pass through unchanged."""
    n, state_size = 1, 12

    def __init__(self):
        self.calls = []

    def _state(self, m):
        return m

    def vortex_core_position(self, m, lam):
        return torch.zeros(1, 5, dtype=torch.float64)

    def core_position_vjp(self, *a):
        pass

    def __getattr__(self, name):
        def call(*a, **kw):
            self.calls.append((name, kw.get("step0")))
        return call

    def count(self, name):
        return sum(n == name for n, _ in self.calls)


@pytest.fixture(autouse=True)
def memory(monkeypatch):
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (200 << 30, 288 << 30))


def run(disk, noise=None, function=None, n_seg=3, seg=2):
    m = torch.zeros(disk.state_size, requires_grad=True)
    a, c = (torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (0.1, 0.2))
    args = (m, a, c, disk, LLGParams(), n_seg, seg, 5.0)
    return (function or adjoint.core_trajectory)(*args, *([noise] if noise else []))


@pytest.mark.parametrize("function", [adjoint.core_trajectory, adjoint.CoreTrajectory.apply])
@pytest.mark.parametrize("mode", [torch.no_grad, torch.inference_mode])
def test_nothing_is_recorded_where_gradients_are_off(function, mode):
    disk = Counting()
    with mode():
        rc = run(disk, function=function)
    assert rc.shape[0] == 4 and not rc.requires_grad
    assert disk.count("rk4_record") == 0 and disk.count("rk4_step") == 3
    rc = run(disk, function=function)
    assert rc.requires_grad and disk.count("rk4_record") == 3 and disk.count("rk4_step") == 3
    rc.sum().backward()
    assert disk.count("rk4_vjp") == 3 and disk.count("rk4_record") == 3


@pytest.mark.parametrize("step0,counter", [(5, None), (-1, 0), (2 ** 64 - 1, 0), (2 ** 64 - 5, 2), (-3, 1)])
def test_a_segment_on_the_step_counter_is_stepped_plainly(step0, counter):
    disk = Counting()
    run(disk, noise=(7, step0, 0))
    want = [("heun_step" if s == counter else "heun_record", step0 + 2 * s) for s in range(3)]
    assert disk.calls == want


def test_live_trajectories_share_one_bound(monkeypatch):
    """With room for five records in all, three live trajectories of three segments keep
    three, two and none; what a backward pass or a dropped graph gives back is used again."""
    one = 4 * 8 * 2 * Counting.state_size
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (1 << 40, 16 * 5 * one + 16))
    disks = [Counting() for _ in range(3)]
    paths = [run(d) for d in disks]
    assert [d.count("rk4_record") for d in disks] == [3, 2, 0]
    assert [d.count("rk4_step") for d in disks] == [0, 1, 3]
    paths[1].sum().backward()                                  # the segment that was not kept is recorded again
    assert disks[1].count("rk4_vjp") == 3 and disks[1].count("rk4_record") == 3
    again = Counting()
    kept = run(again)
    assert again.count("rk4_record") == 2
    del paths[0], kept                                         # no backward pass: the graph's records go with it
    last = Counting()
    run(last)
    assert last.count("rk4_record") == 3


def test_little_free_memory_is_left_alone(monkeypatch):
    one = 4 * 8 * 2 * Counting.state_size
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (16 * one, 1 << 40))
    disk = Counting()
    run(disk)
    assert disk.count("rk4_record") == 2                       # an eighth of what is free


def test_records_that_cannot_be_allocated_are_recomputed(monkeypatch):
    real, given = torch.empty, []

    def empty(*a, **kw):
        if a == (8 * 2 * Counting.state_size,):
            given.append(a)
            if len(given) == 2:
                raise torch.OutOfMemoryError("none left")
        return real(*a, **kw)
    monkeypatch.setattr(torch, "empty", empty)
    before = sum(adjoint._Record.held.values())
    disk = Counting()
    rc = run(disk)
    assert disk.calls == [("rk4_step", None)] * 2 + [("rk4_record", None)]
    rc.sum().backward()
    assert disk.count("rk4_vjp") == 3
    assert sum(adjoint._Record.held.values()) == before
