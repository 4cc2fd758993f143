"""Adaptive runs of the 57-state model: a fiber per workgroup where that is not
behind a launch for each part even with every node solved, else the launches.

* Few long fibers with every node solved are no slower than the launches, which
  a context with pcr_full keeps (a workgroup alone would take twice their
  time), and many fibers well faster (a third); a factor of 1.5 lies between.
* The workgroups' results against the launches' where a fiber takes several
  rounds of a workgroup of either size, with prescribed voltages among the
  stimulus entries, and with the wider stencils.

Bounds of the comparison as for the shorter fibers: 1e-3 mV, activation times
1e-5 ms, solved counts to 2 % and equal at a vanishing tolerance."""
import time
from dataclasses import replace

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _workload(n_fibers, n, steps, entries="one", h=0.01):
    w = I.st57_bundle(n_fibers=n_fibers, n_nodes=n, t_end=steps * 5e-4, onset_max=0.0)
    if entries == "one":
        stims = [dict(s, step_on=0) for s in w.stims]
    else:
        # currents and prescriptions, more of them than a workgroup keeps
        at = np.linspace(2, n - 3, 10).astype(int)
        stims = [dict(fiber=f, node=int(i), half_width=1, step_on=3 * j, n_steps=10 + j, period=0,
                      amp=-20.0 if j % 3 == 2 else 2000.0,
                      mode=F.FIB_STIM_VOLTAGE if j % 3 == 2 else F.FIB_STIM_CURRENT)
                 for f in range(n_fibers) for j, i in enumerate(at)]
    return replace(w, stims=stims, rel_noise=None, vm_noise=np.zeros_like(w.vm_noise), h=h,
                   sample_every=steps // 2)


def _us_per_step(w, steps, **kw):
    s = gpu_solver(w, **kw)
    s.set_adaptive(1e-30)
    s.run(0, 20)
    best = np.inf
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.run(20, steps)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / steps * 1e6)
    s.sync()
    s.close()
    return best


@pytest.mark.parametrize("n_fibers,n,workgroups", [(1, 2000, False), (4, 1481, False),
                                                   (16, 2000, False), (256, 1000, True),
                                                   (600, 1000, True)])
def test_the_faster_form_with_every_node_solved(n_fibers, n, workgroups):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = _workload(n_fibers, n, 100)
    a, b = _us_per_step(w, 80), _us_per_step(w, 80, pcr_full=1)
    say(f"[adaptive routes] {n_fibers} x {n}: {a:.1f} us per step, launches {b:.1f}")
    assert a * 1.5 < b if workgroups else a < 1.5 * b


@pytest.mark.parametrize("n_fibers,n,entries,h", [
    (100, 513, "one", 0.01), (140, 1025, "ten", 0.01), (300, 600, "ten", 0.01),
    (200, 2100, "one", 0.01),
    # stencils of 12, 16, 24 and 32 weights
    (2, 400, "ten", 0.006), (300, 60, "ten", 0.003), (2, 500, "ten", 0.0021),
    (130, 600, "ten", 0.0016), (2, 34, "one", 0.0016)])
def test_a_workgroup_of_several_rounds_is_the_launches(n_fibers, n, entries, h):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 60
    w = _workload(n_fibers, n, steps, entries, h)
    say(f"[adaptive routes] {n_fibers} x {n} entries {entries} h {h}")
    for tol in (1e-6, 1e-30):
        out = []
        for full in (0, 1):
            s = gpu_solver(w, pcr_full=full)
            s.set_adaptive(tol)
            smp = torch.zeros((2, w.n_total), device="cuda")
            s.run(0, steps, w.sample_every, smp)
            s.sync()
            out.append((s.get_state(), smp.cpu().numpy(), s.tact(), s.adaptive_solved()))
            s.close()
        a, b = out
        err = max(np.max(np.abs(a[0][0] - b[0][0])), np.max(np.abs(a[1] - b[1])))
        say(f"   tol {tol}: V difference {err:.2e} mV; solved {a[3]}, {b[3]}; "
            f"{np.isfinite(a[2]).sum()} activated")
        assert err < 1e-3
        np.testing.assert_array_equal(np.isfinite(a[2]), np.isfinite(b[2]))
        fin = np.isfinite(a[2])
        assert not fin.any() or np.max(np.abs(a[2][fin] - b[2][fin])) < 1e-5
        assert abs(a[3] - b[3]) <= (0.02 * b[3] if tol > 1e-20 else 0)
