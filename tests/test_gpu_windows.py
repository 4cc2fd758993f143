"""The windowed diffusion and whole split steps on windows.

* CPU: the stencil's weights, from the closed form of the inverse, against the
  dense tridiagonal solve in FP64, reflections at short fibers included;
* GPU: Hodgkin-Huxley runs on windows (schedules SPLIT and AUTO) against the
  oracle over fibers just long enough for the stencil, uneven lengths whose
  ends fall anywhere in a window, one long fiber and many nodes, with
  Godunov splitting and implicit Euler (wider stencils); calls cut at odd
  places, so that launches of every size and both buffers end a run, are
  bitwise one call; fibers too short for the stencil, and pcr_full, keep the
  partitioned solve and give the same states to FP32 rounding;
* the windowed diffusion of the split schedule at block edges (ST57 and the
  adaptive schedule) against the oracle.

Bounds: the budget of the parity tests for V_m is 0.5 mV; FP32 runs of this
length are within 1e-3 mV of the oracle (the other parity tests measure 5e-4),
so 5e-3 mV tells a wrong neighbour or a step lost from rounding."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, oracle_cfg, oracle_init, say

torch = pytest.importorskip("torch")


def _weights(w, theta):
    a = (1 + 2 * w) / w
    lam = 2 / (a + np.sqrt(a * a - 4))
    need = int(np.ceil(40 / -np.log2(lam)))
    g0 = 1 / np.sqrt(1 + 4 * w)
    return w * g0 * (1 - lam) ** 2 / theta * lam ** np.arange(need)


@pytest.mark.parametrize("w,theta,n", [(0.0383, 0.5, 11), (0.0191, 0.5, 9), (0.19, 0.5, 40),
                                       (0.0766, 1.0, 13), (0.383, 1.0, 33)])
def test_stencil_is_the_tridiagonal_solve(w, theta, n):
    L = np.zeros((n, n))
    for i in range(n):
        l, r = i > 0, i + 1 < n
        wl, wr = (w if r else 2 * w) * l, (w if l else 2 * w) * r
        if l:
            L[i, i - 1] = wl
        if r:
            L[i, i + 1] = wr
        L[i, i] = -(wl + wr)
    V = np.random.default_rng(1).standard_normal(n) * 100
    want = V + np.linalg.solve(np.eye(n) - L, (L / theta) @ V)
    h = _weights(w, theta)
    assert n > len(h) - 1 or n > 8
    period = 2 * (n - 1)

    def at(i):
        i = abs(i) % period
        return V[period - i if i >= n else i]
    got = np.array([V[i] + sum(hk * ((at(i - k - 1) - V[i]) + (at(i + k + 1) - V[i]))
                               for k, hk in enumerate(h)) for i in range(n)])
    # 2^-40 of the largest difference is dropped
    assert np.max(np.abs(got - want)) < 2.0 ** -40 * 1e3


def _check(w, kw, cuts, scheme=O.SCHEME_STRANG, theta=0.5):
    cfg = oracle_cfg(w, scheme=scheme, theta=theta)
    yo, so, to = O.run(cfg, w.n_nodes, oracle_init(w), w.stims, w.n_steps,
                       sample_every=w.sample_every)
    rows = w.n_steps // w.sample_every
    out = []
    for calls in ([w.n_steps], cuts):
        s = gpu_solver(w, **kw)
        smp = torch.zeros((rows, w.n_total), device="cuda")
        step = 0
        for n in calls:
            r0 = step // w.sample_every
            s.run(step, n, w.sample_every, smp[r0:])
            step += n
        assert step == w.n_steps
        s.sync()
        out.append((s.get_state(), smp.cpu().numpy(), s.tact()))
        s.close()
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    err = max(np.max(np.abs(out[0][0][0] - yo[0])), np.max(np.abs(out[0][1] - so)))
    fin = np.isfinite(to)
    say(f"   V err {err:.2e} mV; {fin.sum()} activated")
    assert err < 5e-3
    np.testing.assert_array_equal(np.isfinite(out[0][2]), fin)
    if fin.any():
        assert np.max(np.abs(out[0][2][fin] - to[fin])) < 1e-5
    return out[0]


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


SHAPES = [(1, 11, 11), (7, 11, 30), (3, 255, 258), (40, 60, 300), (1, 3001, 3001)]


@pytest.mark.gpu
@pytest.mark.parametrize("n_fibers,n_min,n_max", SHAPES)
@pytest.mark.parametrize("schedule", [F.FIB_SCHED_AUTO, F.FIB_SCHED_SPLIT])
def test_windows_match_the_oracle(schedule, n_fibers, n_min, n_max):
    _need_gpu()
    w = I.batched_hh(n_fibers=n_fibers, n_min=n_min, n_max=n_max, t_end=0.4, onset_max=0.1)
    w.sample_every = 25
    say(f"[windows] {n_fibers} x {n_min}-{n_max} schedule {schedule}")
    _check(w, dict(schedule=schedule), [1, 1, 2, 37, 150, 1, 208])


@pytest.mark.gpu
@pytest.mark.parametrize("splitting,time_1d,dt", [(1, 0, 1e-3), (0, 1, 1e-3), (1, 1, 5e-3),
                                                  (0, 0, 5e-3)])
def test_windows_of_other_schemes(splitting, time_1d, dt):
    _need_gpu()
    w = I.batched_hh(n_fibers=6, n_min=40, n_max=300, t_end=300 * dt, onset_max=0.1, dt=dt)
    w.dt_0D = min(w.dt_0D, 2.5e-3)
    w.sample_every = 50
    say(f"[windows] splitting {splitting} time_1d {time_1d} dt {dt}")
    _check(w, dict(schedule=F.FIB_SCHED_SPLIT, splitting=splitting, time_1d=time_1d),
           [3, 100, 1, 196], O.SCHEME_GODUNOV if splitting else O.SCHEME_STRANG,
           1.0 if time_1d else 0.5)


@pytest.mark.gpu
def test_short_fibers_and_full_pcr_keep_the_partitioned_solve():
    _need_gpu()
    w = I.batched_hh(n_fibers=9, n_min=30, n_max=90, t_end=0.3, onset_max=0.1)
    w.sample_every = 50
    a = _check(w, dict(schedule=F.FIB_SCHED_SPLIT), [300])
    b = _check(w, dict(schedule=F.FIB_SCHED_SPLIT, pcr_full=1), [300])
    # rounding of FP32 over 300 steps of an action potential's 100 mV
    assert np.max(np.abs(a[0][0] - b[0][0])) < 1e-3
    ws = I.batched_hh(n_fibers=9, n_min=2, n_max=10, t_end=0.3, onset_max=0.1)
    ws.sample_every = 50
    _check(ws, dict(schedule=F.FIB_SCHED_SPLIT), [299, 1])


@pytest.mark.gpu
@pytest.mark.parametrize("n_fibers,n", [(1, 9), (5, 205), (3, 1024), (2, 1023)])
def test_windowed_diffusion_of_the_57_state_model(n_fibers, n):
    _need_gpu()
    w = I.st57_bundle(n_fibers=n_fibers, n_nodes=n, t_end=0.06, onset_max=0.01)
    w.sample_every = 30
    say(f"[windowed diffusion st57] {n_fibers} x {n}")
    _check(w, dict(), [1, 1, 61, 57])
