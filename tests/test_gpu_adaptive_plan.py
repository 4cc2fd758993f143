"""Adaptive computation on automatic plans: where the plain plan's states do
not fit the adaptive fused kernel's LDS (bins near 7000 nodes at 1024 x 7),
fib_set_adaptive chooses a shape that does (fibers near 8000 nodes fit none), fib_set_adaptive(0) returns to the
plain plan, and results stay those of the split schedule: the same node-steps
solved to 1 % and V_m within 0.05 mV (the bounds the two schedules are held to
where both plans fit), on bins of one fiber and on uneven ones."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_fibers,n_min,n_max", [(2, 7100, 7900), (300, 5900, 7100),
                                                   (3, 300, 400)])
def test_automatic_plan_fits_the_adaptive_kernel(n_fibers, n_min, n_max):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = I.batched_hh(n_fibers=n_fibers, n_min=n_min, n_max=n_max, t_end=0.3, onset_max=0.1)
    w.vm_noise[:] = 0.0
    out = {}
    for sched in (F.FIB_SCHED_AUTO, F.FIB_SCHED_SPLIT):
        s = gpu_solver(w, schedule=sched)
        plain = s.plan()
        s.set_adaptive(1e-6)
        plan = s.plan()
        s.run(0, w.n_steps)
        s.sync()
        out[sched] = s.get_state(), s.adaptive_solved()
        if sched == F.FIB_SCHED_AUTO:
            say(f"[adaptive plan] {n_fibers} x {n_min}-{n_max}: {plain} -> {plan}")
            # states, list, fibers and verdicts in LDS beside the solve
            cap = plan["threads"] * plan["nodes_per_thread"]
            lds = 4 * plan["threads"] * (6 + 2 * plan["pcr_levels"]) + 19 * cap + cap // 8
            if n_max > 7500:     # a fiber of which no shape fits: the plan stays
                assert plan == plain
            else:
                assert lds < 160 * 1024
        s.set_adaptive(0.0)
        assert s.plan() == plain
        s.close()
    (ya, na), (yb, nb) = out[F.FIB_SCHED_AUTO], out[F.FIB_SCHED_SPLIT]
    assert abs(na - nb) <= 0.01 * nb
    assert np.max(np.abs(ya[0] - yb[0])) < 0.05
