"""What a run leaves for a surrogate step that follows it: V_m of its last split
step, which the step's activation test takes as the step before.

Every kernel that ends a run is taken: adaptive runs of both models (one launch,
and a launch for each part, which pcr_full keeps), the fused Hodgkin-Huxley
kernel, its windows, and the split schedule.  The step after the run is
compared with the same step of a context that is given the run's final state
(fib_set_state stores V_m as the previous step's; the FP32 rows are copied
over it, since offsets below 2^-53 of their rest value do not survive the FP64
form): the same nodes are activated, and a node above the threshold at the
run's end is not.  The two contexts hold the same FP32 state, so the times are
equal."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

RES = {I.MODEL_HH: [100.0, 1.0, 1.0, 1.0], I.MODEL_ST57: [100.0] + [1.0] * 56}


def _workload(model, n_fibers, n, steps):
    make = I.batched_hh if model == I.MODEL_HH else I.st57_bundle
    kw = dict(n_min=n, n_max=n) if model == I.MODEL_HH else dict(n_nodes=n)
    w = make(n_fibers=n_fibers, t_end=0.1, onset_max=0.0, **kw)
    stims = [dict(s, step_on=0, n_steps=steps, amp=2000.0) for s in w.stims]
    return replace(w, stims=stims, rel_noise=None, vm_noise=np.zeros_like(w.vm_noise))


@pytest.mark.parametrize("model,n_fibers,n,tol,kw", [
    (I.MODEL_ST57, 3, 300, 1e-6, {}),
    (I.MODEL_ST57, 3, 300, 1e-6, dict(pcr_full=1)),
    (I.MODEL_ST57, 3, 300, 0.0, {}),
    (I.MODEL_HH, 3, 1200, 1e-6, {}),
    (I.MODEL_HH, 700, 1200, 1e-6, {}),
    (I.MODEL_HH, 3, 1200, 1e-6, dict(schedule=F.FIB_SCHED_SPLIT)),
    (I.MODEL_HH, 3, 1200, 0.0, {}),
    (I.MODEL_HH, 3, 1200, 0.0, dict(threads_per_group=512, nodes_per_thread=4)),
    (I.MODEL_HH, 3, 1200, 0.0, dict(schedule=F.FIB_SCHED_SPLIT, pcr_full=1))])
def test_surrogate_step_after_a_run_knows_its_last_voltage(model, n_fibers, n, tol, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 300 if model == I.MODEL_ST57 else 500
    w = _workload(model, n_fibers, n, steps)
    say(f"[run observables] model {model} {n_fibers} x {n} tol {tol} {kw}")
    out = []
    state = None
    for fresh in (False, True):
        s = gpu_solver(w, **kw)
        if not fresh:
            s.set_adaptive(tol)
            s.run(0, steps)
            s.sync()
            state, rows = s.get_state(), s.state_tensor()[0].clone()
            s.set_adaptive(0.0)
        else:
            s.set_state(state)
            s.state_tensor()[0].copy_(rows)
        F.fib_reset_observables(s.ctx)
        s.set_predictor(F.FIB_PRED_EULER, RES[model], 1e-3)
        s.step_surrogate(steps)
        s.sync()
        out.append((s.tact(), s.state_tensor()[0].cpu().numpy()))
        s.close()
    above = state[0] >= w.v_th
    say(f"   {above.sum()} nodes above the threshold, {np.isfinite(out[0][0]).sum()} activated")
    assert above.any()
    assert not np.isfinite(out[0][0][above]).any()
    np.testing.assert_array_equal(out[0][1], out[1][1])
    np.testing.assert_array_equal(out[0][0], out[1][0])
