"""Turning the adaptive computation on and off on a Hodgkin-Huxley bundle whose
plain plan does not fit the adaptive kernel (two plans): a context that went
back and forth, with other stimuli set in between, runs bit for bit as a new
one; turning it off neither waits for the stream nor plans again, and turning
it on again takes milliseconds (planning 200 000 slots anew takes ten times
what is allowed; the queued sleep is 0.2 s)."""
import time

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _states(s, w, steps=60):
    s.init_state(vm_noise=w.vm_noise.astype(np.float32))
    s.run(0, steps)
    s.sync()
    return s.state_tensor()[0].cpu().numpy()


def test_back_and_forth_is_a_new_context():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = I.batched_hh(n_fibers=1369, t_end=0.2, onset_max=0.0)
    later = [dict(s, node=s["node"] + 100, step_on=5) for s in w.stims]
    want = {}
    for tol in (0.0, 1e-6):
        s = gpu_solver(w)
        s.set_stimulus(later)
        s.set_adaptive(tol)
        want[tol] = s.plan(), _states(s, w)
        s.close()
    say("[adaptive toggle]", want[0.0][0], want[1e-6][0])
    assert want[0.0][0] != want[1e-6][0]
    s = gpu_solver(w)
    s.set_adaptive(1e-6)
    _states(s, w)
    s.set_adaptive(0.0)
    s.set_stimulus(later)
    for tol in (0.0, 1e-6, 0.0, 1e-6):
        s.set_adaptive(tol)
        plan, y = s.plan(), _states(s, w)
        assert plan == want[tol][0]
        np.testing.assert_array_equal(y, want[tol][1])
    s.close()


def test_off_returns_at_once():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = I.batched_hh(n_fibers=1369, t_end=0.2, onset_max=0.0)
    s = gpu_solver(w)
    s.set_adaptive(1e-6)
    torch.cuda.synchronize()
    torch.cuda._sleep(int(5e8))
    t = time.perf_counter()
    s.set_adaptive(0.0)
    off = time.perf_counter() - t
    torch.cuda.synchronize()
    t = time.perf_counter()
    s.set_adaptive(1e-6)
    on = time.perf_counter() - t
    say(f"[adaptive toggle] off {1e3 * off:.3f} ms, on again {1e3 * on:.3f} ms")
    assert off < 1e-3 and on < 1e-3
    s.close()
