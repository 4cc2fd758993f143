"""Which solve the split schedule's diffusion takes: the stencil or the
partitioned solve in place, by their cost.  fib_step_diffusion always takes the
partitioned solve, and a split step by hand (half reaction, diffusion, half
reaction) runs the same arithmetic as a run of one step.  So a run's states
are bitwise those of the steps by hand where the run takes the partitioned
solve, and differ from them by rounding where it takes the stencil.

Bound: both solves round a step's V_m of 100 mV a few times: 1e-4 mV."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HH, ST57 = F.FIB_MODEL_HH, F.FIB_MODEL_ST57
CASES = [
    # a fiber per bin: wide stencils (dt 5e-3, 2e-2) lose
    (HH, "predictor", 1, 300, 2e-2, False), (HH, "predictor", 200, 1100, 5e-3, False),
    (HH, "predictor", 1369, 1481, 5e-3, False), (HH, "predictor", 1369, 1481, 1e-3, True),
    # long fibers, and many to a bin
    (HH, "predictor", 100, 8000, 5e-3, True), (HH, "predictor", 400, 101, 5e-3, True),
    (HH, "adaptive", 1369, 1250, 1e-3, False), (HH, "adaptive", 300, 8000, 1e-3, False),
    (HH, "adaptive", 200, 600, 1e-3, True),
    (ST57, "plain", 1, 101, 4e-3, False), (ST57, "plain", 40, 600, 5e-4, True)]


@pytest.mark.parametrize("model,path,n_fibers,n,dt,stencil", CASES)
def test_run_takes_the_cheaper_solve(model, path, n_fibers, n, dt, stencil):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[diffusion route] model {model} {path} {n_fibers} x {n} dt {dt}: "
        f"{'stencil' if stencil else 'partitioned'}")
    nn = np.full(n_fibers, n, np.int32)
    vm = torch.empty(n_fibers * n, device="cuda").normal_(
        0.0, 20.0, generator=torch.Generator(device="cuda").manual_seed(3))
    stims = [dict(fiber=f, node=n // 2, half_width=1, step_on=0, n_steps=100, period=0, amp=500.0)
             for f in range(n_fibers)]
    out = []
    for by_hand in (False, True):
        s = F.Solver(nn, model=model, schedule=F.FIB_SCHED_SPLIT, Cm=1.0, Am=500.0, sigma=3.828,
                     h=0.01, dt_0D=dt / 8, dt_1D=dt, dt_split=dt)
        s.set_stimulus(stims)
        if not by_hand and path == "predictor":
            s.set_predictor(F.FIB_PRED_EULER, [100.0, 1.0, 1.0, 1.0], 1e-3)
        if not by_hand and path == "adaptive":
            s.set_adaptive(1e-30)      # every node is solved
        s.init_state(vm)
        if by_hand:
            s.step_reaction(0, 0.5 * dt)
            s.step_diffusion(dt)
            s.step_reaction(0, 0.5 * dt)
        else:
            s.run(0, 1)                # a run's only step is plain
        s.sync()
        out.append(s.state_tensor()[0].cpu().numpy())
        s.close()
    same = np.array_equal(out[0], out[1])
    err = np.max(np.abs(out[0][0] - out[1][0]))
    say(f"   {'bitwise' if same else f'V difference {err:.1e} mV'}")
    assert same != stencil
    assert err < 1e-4
