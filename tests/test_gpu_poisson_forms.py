"""The forms of the Poisson solve (pic_last_poisson_form): in one launch,
continued over several, given up and started again, and in separate launches.
The field against the FFT solve of the same charge density, with the bar of
test_gpu_poisson.py."""
import threading
import time

import numpy as np
import pytest

from test_gpu_kernel_edges import _poisson_case

pytestmark = pytest.mark.gpu

SEPARATE, ONE_LAUNCH, GAVE_UP = 1, 2, 3
GRIDS = [(16, 8, 8), (41, 25, 1), (64, 64, 64), (128, 64, 64)]  # one workgroup, two, and 256 of either size


def _solve(sim, E, workgroups=-1, polls=-1, iterations=-1):
    """One solve under the limits: (iterations, form); its field is checked."""
    sim._check(sim.lib.pic_poisson_limits(sim.ctx, workgroups, polls, iterations))
    it, res = sim.solve_poisson(neutralize=True)
    assert 0 < it and res <= 1e-13
    assert np.linalg.norm(sim.fields_numpy()[:3] - E) <= 1e-9 * np.linalg.norm(E)
    return it, sim.lib.pic_last_poisson_form(sim.ctx)


@pytest.mark.parametrize("n", GRIDS)
def test_given_up_solve_starts_again(n):
    """No read of a slot allowed: every workgroup gives up at its first wait
    and ends, and separate launches solve from the start; the next solve is in
    one launch again."""
    sim, E = _poisson_case(n, 43)
    assert sim.lib.pic_last_poisson_form(sim.ctx) == 0
    assert _solve(sim, E, polls=0)[1] == GAVE_UP
    assert _solve(sim, E)[1] == ONE_LAUNCH
    assert _solve(sim, E, polls=0)[1] == GAVE_UP


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("length", [1, 7, 50])
def test_solve_over_several_launches(n, length):
    """Launches of a few iterations each continue one another: the neighbours'
    search directions from memory are those that one launch keeps.  A lost
    direction would cost conjugacy and show as more iterations (the count comes
    in whole checks of 16, and the charge density's last bits vary).  Two fields
    whose residuals are 1e-13 differ by that times the square root of the
    operator's condition at most."""
    sim, E = _poisson_case(n, 47)
    _solve(sim, E)  # neutralized by the first solve
    it, form = _solve(sim, E)
    field = sim.fields_numpy()[:3]
    it_parts, form_parts = _solve(sim, E, iterations=length)
    assert form == form_parts == ONE_LAUNCH and abs(it_parts - it) <= 16
    condition = sum(4.0 for k in n if k > 1) / (2.0 - 2.0 * np.cos(2.0 * np.pi / max(n)))
    assert np.linalg.norm(sim.fields_numpy()[:3] - field) <= 2e-13 * np.sqrt(condition) * np.linalg.norm(field)


def test_second_solve_at_a_time_takes_separate_launches():
    """While one thread solves a large grid in one launch, a solve of another
    thread takes separate launches."""
    import torch
    large, small = _poisson_case((1024, 512, 1), 53), _poisson_case((16, 8, 8), 59)
    _solve(*large), _solve(*small)
    torch.cuda.synchronize()
    forms, stop = [], threading.Event()

    def keep_solving():
        with torch.cuda.stream(torch.cuda.Stream()):
            while not stop.is_set():
                large[0].solve_poisson(neutralize=True)

    thread = threading.Thread(target=keep_solving)
    thread.start()
    try:
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(40):
                time.sleep(0.003)
                forms.append(_solve(*small)[1])
                if SEPARATE in forms:
                    break
    finally:
        stop.set()
        thread.join()
    assert SEPARATE in forms and GAVE_UP not in forms, forms


@pytest.mark.parametrize("n", GRIDS)
def test_launch_without_progress_ends_the_form(n):
    """A launch that makes no iteration (none allowed; a refused launch looks
    the same) is not repeated for ever: separate launches solve."""
    sim, E = _poisson_case(n, 61)
    assert _solve(sim, E, iterations=0)[1] == GAVE_UP


@pytest.mark.parametrize("n,needed", [((16, 8, 8), 1), ((41, 25, 1), 2), ((64, 64, 64), 256), ((128, 64, 64), 256)])
def test_one_launch_only_where_its_workgroups_fit(n, needed):
    """With fewer workgroups at once than the grid needs the solve takes separate
    launches at once, with as many one."""
    sim, E = _poisson_case(n, 67)
    assert _solve(sim, E, workgroups=needed - 1)[1] == SEPARATE
    assert _solve(sim, E, workgroups=needed)[1] == ONE_LAUNCH
