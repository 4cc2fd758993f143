"""Hodgkin-Huxley runs on windows, one split step per call: a bundle that fits
one workgroup runs it in place, a larger one through the second buffer.  Sizes
on both sides of that line, the smallest the stencil takes, and several fibers;
bit for bit one call of all steps, samples and activation times included."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("schedule", [F.FIB_SCHED_AUTO, F.FIB_SCHED_SPLIT])
@pytest.mark.parametrize("n_fibers,n", [(1, 11), (1, 300), (4, 60), (1, 1003), (1, 1004), (1, 1005),
                                        (2, 502), (2, 503)])
def test_single_steps_are_one_call(n_fibers, n, schedule):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 120
    w = I.batched_hh(n_fibers=n_fibers, n_min=n, n_max=n, t_end=0.12, onset_max=0.01)
    say(f"[window single steps] {n_fibers} x {n} schedule {schedule}")
    out = []
    for k in (steps, 1):
        s = gpu_solver(w, schedule=schedule)
        smp = torch.zeros((steps // 10, w.n_total), device="cuda")
        for n0 in range(0, steps, k):
            s.run(n0, k, 10, smp[n0 // 10:])
        s.sync()
        out.append((s.state_tensor()[0].cpu().numpy(), smp.cpu().numpy(), s.tact()))
        s.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    assert np.isfinite(out[0][2]).any()
