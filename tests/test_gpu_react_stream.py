"""The 57-state reaction over a resident grid: bundles of more nodes than the
grid has threads, whose nodes load their states while the node before is
solved, against the same fibers in a bundle of one fiber per thread. Fibers
are independent, so every copy of a fiber has the same states bit for bit, at
whatever node it starts: sizes one past and one short of whole rounds, a last
wave with one lane, one and several substeps, both splittings (the launches of
one phase and of two), current and voltage stimuli."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say
from test_gpu_surrogate import _random_net

torch = pytest.importorskip("torch")


def _bundle(n_fibers, n, steps):
    """n_fibers fibers of n nodes, fiber f as fiber f % 3."""
    w = I.st57_bundle(n_fibers=3, n_nodes=n, t_end=steps * 5e-4, onset_max=0.0, host_noise=False)
    vm = np.tile(w.vm_noise.reshape(3, n), (-(-n_fibers // 3), 1))[:n_fibers].reshape(-1)
    at = [n // 3, n // 2, n - 2]
    stims = [dict(fiber=f, node=at[f % 3], half_width=1, step_on=f % 3, n_steps=20, period=0,
                  amp=-40.0 if f % 3 == 2 else 2000.0, voltage=f % 3 == 2)
             for f in range(n_fibers)]
    return replace(w, n_nodes=np.full(n_fibers, n, dtype=np.int32), stims=stims, vm_noise=vm,
                   rel_noise=None)


def _states(w, steps, cuts, **kw):
    s = gpu_solver(w, **kw)
    step = 0
    for c in cuts:
        s.run(step, c)
        step += c
    assert step == steps
    s.sync()
    out = s.get_state(), s.tact()
    s.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("splitting", [F.FIB_SPLIT_STRANG, F.FIB_SPLIT_GODUNOV])
@pytest.mark.parametrize("dt_0D", [1e-4, 2.5e-4])
@pytest.mark.parametrize("n_fibers,n", [(1024, 128), (1025, 128), (1191, 331), (5, 13)])
def test_copies_of_a_fiber_are_bitwise_equal(n_fibers, n, dt_0D, splitting):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 12
    say(f"[react stream] {n_fibers} x {n} dt_0D {dt_0D} splitting {splitting}")
    kw = dict(splitting=splitting, dt_0D=dt_0D)
    y, t = _states(_bundle(n_fibers, n, steps), steps, [1, 10, 1], **kw)
    y0, t0 = _states(_bundle(3, n, steps), steps, [12], **kw)
    S = y.shape[0]
    y = y.reshape(S, n_fibers, n)
    t = t.reshape(n_fibers, n)
    y0 = y0.reshape(S, 3, n)
    t0 = t0.reshape(3, n)
    assert np.isfinite(y0).all() and not np.array_equal(y0[:, 0], y0[:, 2])
    for f in range(3):
        c = len(range(f, n_fibers, 3))
        np.testing.assert_array_equal(y[:, f::3], np.broadcast_to(y0[:, f:f + 1], (S, c, n)))
        np.testing.assert_array_equal(t[f::3], np.broadcast_to(t0[f:f + 1], (c, n)))


@pytest.mark.gpu
@pytest.mark.parametrize("path", ["plain", "euler", "zero", "network"])
@pytest.mark.parametrize("n_fibers,n", [(13800, 128), (13799, 128), (14001, 127)])
def test_streamed_states_are_the_cached_ones(n_fibers, n, path):
    """Bundles past the last-level cache whose rows start on a line (13 800 and
    13 799 fibers of 128 nodes: 403 MB, just past the rule) or not."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    steps = 5
    say(f"[streamed states] {n_fibers} x {n} {path}")
    sizes, _, net = _random_net(I.MODEL_ST57, 3)
    out = []
    for fibers in (n_fibers, 3):
        w = _bundle(fibers, n, steps)
        s = gpu_solver(w)
        if path == "network":
            s.set_surrogate(net, dict(in_shift=np.zeros(57), in_scale=np.ones(57),
                                      out_shift=np.zeros(57), out_scale=np.full(57, 1e-6),
                                      res_scale=np.ones(57), flag_scale=1.0), 1e30)
        elif path != "plain":
            s.set_predictor(F.FIB_PRED_EULER if path == "euler" else F.FIB_PRED_ZERO,
                            np.ones(57, dtype=np.float32), 1e30)
        s.run(0, steps)
        s.sync()
        y = s.get_state()
        assert np.isfinite(y).all()
        out.append(y.reshape(57, fibers, n))
        s.close()
    net.close()
    for f in range(3):
        c = len(range(f, n_fibers, 3))
        np.testing.assert_array_equal(out[0][:, f::3],
                                      np.broadcast_to(out[1][:, f:f + 1], (57, c, n)))
