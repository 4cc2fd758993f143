"""The autotuner on contexts whose plain runs take whole steps on windows.

One short fiber under AUTO runs on windows at half the time of any workgroup of
whole fibers, so a tuned context stays on them: a run makes more than one
launch, and its states are bitwise those of the untuned context.  Under SPLIT
every shape runs the same windows, so the plan stays as it is.  With a
predictor attached runs take no windows, and shapes are tuned; they are back
when it is detached."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _run(s, w, steps=200):
    s.init_state(vm_noise=w.vm_noise.astype(np.float32))
    s.set_kernel_timing(True)
    s.run(0, steps)
    s.sync()
    n = s.kernel_time(F.FIB_KT_FUSED)[1] + s.kernel_time(F.FIB_KT_REACTION)[1]
    s.set_kernel_timing(False)
    return s.state_tensor()[0].cpu().numpy(), n


@pytest.mark.parametrize("schedule", [F.FIB_SCHED_AUTO, F.FIB_SCHED_SPLIT])
@pytest.mark.parametrize("predictor", [False, True])
@pytest.mark.parametrize("candidates", [1, 8])
def test_a_tuned_small_bundle_stays_on_windows(schedule, predictor, candidates):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = I.batched_hh(n_fibers=2, n_min=900, n_max=1000, t_end=0.2, onset_max=0.05)
    s = gpu_solver(w, schedule=schedule)
    plan = s.plan()
    a, na = _run(s, w)
    if predictor:
        s.set_predictor(F.FIB_PRED_EULER, [100.0, 1.0, 1.0, 1.0], 1e-3)
    info = s.autotune(trial_steps=100, max_candidates=candidates)
    if predictor:
        F.fib_clear_surrogate(s.ctx)
    b, nb = _run(s, w)
    say(f"[autotune windows] schedule {schedule} predictor {predictor}: {info}; launches {na}, {nb}")
    assert info["trial_ms_per_step"] > 0
    assert na > 2 and nb == na
    np.testing.assert_array_equal(a, b)
    if not predictor:
        assert s.plan() == plan
    s.close()
