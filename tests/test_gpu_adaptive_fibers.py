"""Adaptive runs of the 57-state model with a fiber per workgroup, against the
form that takes a launch for each part (pcr_full keeps the partitioned solve
and with it that form), at the edges of the workgroup: fibers just long enough
for the stencil, lengths around one and two rounds of the workgroup, more
fibers than the chip has compute units, one fiber past the length the
workgroup takes; fibers with one stimulus entry and with more than it caches
(currents); both splittings.  Bundles of few fibers that take several rounds of a
workgroup run the launches in both contexts.

Bounds: the two forms' diffusions differ by FP32 rounding (1e-3 mV allowed
over an action potential, as between the solves of the plain schedules), which
may turn the verdict of a point near the threshold: the solved counts agree to
2 %, as they do with the oracle's.  At a vanishing tolerance every node-step is
solved and the counts are equal."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

torch = pytest.importorskip("torch")

SHAPES = [(1, 9), (3, 511), (2, 513), (2, 1025), (300, 40), (1, 2100)]


def _workload(n_fibers, n, entries, steps):
    w = I.st57_bundle(n_fibers=n_fibers, n_nodes=n, t_end=steps * 5e-4, onset_max=0.0)
    stims = [dict(s, step_on=0) for s in w.stims]
    if entries:
        at = np.linspace(2, n - 3, min(10, n // 4)).astype(int)
        stims = [dict(fiber=f, node=int(i), half_width=1, step_on=3 * j, n_steps=30 + j,
                      period=0, amp=-20.0 if j % 3 == 2 else 2000.0, voltage=j % 3 == 2)
                 for f in range(n_fibers) for j, i in enumerate(at)]
    return replace(w, stims=stims, rel_noise=None, vm_noise=np.zeros_like(w.vm_noise),
                   sample_every=40)


def _run(w, tol, steps, **kw):
    s = gpu_solver(w, **kw)
    s.set_adaptive(tol)
    rows = steps // w.sample_every
    smp = torch.zeros((rows, w.n_total), device="cuda")
    s.run(0, steps, w.sample_every, smp)
    s.sync()
    out = s.get_state(), smp.cpu().numpy(), s.tact(), s.adaptive_solved()
    s.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("splitting", [F.FIB_SPLIT_STRANG, F.FIB_SPLIT_GODUNOV])
@pytest.mark.parametrize("entries", [False, True])
@pytest.mark.parametrize("n_fibers,n", SHAPES)
def test_fiber_per_workgroup_is_the_launches(n_fibers, n, entries, splitting):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 240
    w = _workload(n_fibers, n, entries, steps)
    say(f"[adaptive fibers] {n_fibers} x {n} entries {entries} splitting {splitting}")
    for tol in (1e-6, 1e-30):
        a = _run(w, tol, steps, splitting=splitting)
        b = _run(w, tol, steps, splitting=splitting, pcr_full=1)
        err = max(np.max(np.abs(a[0][0] - b[0][0])), np.max(np.abs(a[1] - b[1])))
        say(f"   tol {tol}: V difference {err:.2e} mV; solved {a[3]}, {b[3]}; "
            f"{np.isfinite(a[2]).sum()} activated")
        assert err < 1e-3
        np.testing.assert_array_equal(np.isfinite(a[2]), np.isfinite(b[2]))
        fin = np.isfinite(a[2])
        assert not fin.any() or np.max(np.abs(a[2][fin] - b[2][fin])) < 1e-5
        assert abs(a[3] - b[3]) <= (0.02 * b[3] if tol > 1e-20 else 0)
