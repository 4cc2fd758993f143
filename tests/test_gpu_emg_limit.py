"""EMG solves that end at the iteration limit: a field that is not finite cannot
converge, and costs no more than its first iterations (launching all of 20000
takes 0.2 s with the diagonal preconditioner, 1.1 s with a look of the host at
each; half of the former is allowed, against milliseconds); limits of zero
to a few iterations are taken in full where the tolerance is out of reach."""
import time

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _emg(nx, ny, n, m):
    s = F.Solver(np.full(nx * ny, n, np.int32), Cm=1.0, Am=500.0, sigma=3.828, h=0.01)
    x = np.arange(nx * ny * n) % n
    vm = 90.0 * np.exp(-((x - 0.4 * n) / (0.1 * n)) ** 2)
    s.init_state(vm.astype(np.float32))
    return s, F.Emg(s, nx, ny, m, 0.05, 0.05)


def test_a_field_that_is_not_finite_ends_at_the_limit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s, e = _emg(3, 3, 101, 1)
    e.solve(1e-7, 10)
    s.state_tensor()[0][0, 5] = float("nan")
    torch.cuda.synchronize()
    t = time.perf_counter()
    it, _ = e.solve(1e-7, 20000)
    t = time.perf_counter() - t
    say(f"[emg limit] {it} iterations in {1e3 * t:.1f} ms")
    assert it == 20000 and np.isnan(e.phi()).all()
    assert t < 0.1
    e.close()


@pytest.mark.parametrize("limit", [0, 1, 2, 3, 4, 5])
def test_the_iteration_limit_counts(limit):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s, e = _emg(4, 3, 201, 2)
    it, rr = e.solve(1e-30, limit)
    say(f"[emg limit] limit {limit}: {it} iterations, residual {rr:.1e}")
    assert it == limit
    # phi_e starts at 0: the residual is b; two iterations reach 1e-7
    assert abs(rr - 1.0) < 1e-6 if limit == 0 else rr < (1e-7 if limit > 1 else 1.0)
    e.close()
