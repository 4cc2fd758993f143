"""The windowed diffusion at every width it is built for (8, 10, 12, 16, 24 and
32 weights; Crank-Nicolson and implicit Euler), in each kernel that takes it.

One split step of a bundle of uneven short fibers, V_m drawn at random so that
neighbours differ by tens of mV and every weight counts: the same step by hand,
with its diffusion solved on the host in FP64 (dense tridiagonal matrix per
fiber) between the two reaction halves of the device.  Only the stencil's
rounding is left, W products of up to 100 mV in FP32 and one sum: 1e-4 mV; a
weight wrong by a thousandth shows as 1e-2 mV.  Where the by-hand diffusion of the
device (the partitioned solve) is bitwise the run's, the run did not take the
stencil, and the test would say nothing: that must not be."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIGMA, AM, CM, H = 3.828, 500.0, 1.0, 0.01
# (dt, theta scheme, the stencil's width)
WIDTHS = [(5e-4, 0, 8), (1e-3, 0, 10), (2e-3, 0, 12), (5e-3, 0, 16), (1e-2, 0, 24), (2e-2, 0, 32),
          (2.5e-4, 1, 8), (5e-4, 1, 10), (2.5e-3, 1, 16), (1e-2, 1, 32)]


def _width(dt, scheme):
    theta = 1.0 if scheme else 0.5
    w = theta * SIGMA / (AM * CM) * dt / H ** 2
    a = (1 + 2 * w) / w
    need = int(np.ceil(40 / -np.log2(2 / (a + np.sqrt(a * a - 4)))))
    return next(W for W in (8, 10, 12, 16, 24, 32) if need <= W)


def _diffuse(V, nn, dt, scheme):
    theta = 1.0 if scheme else 0.5
    r = SIGMA / (AM * CM) * dt / H ** 2
    out, at = np.empty_like(V), 0
    for n in nn:
        L = np.zeros((n, n))
        for i in range(n):
            if i > 0:
                L[i, i - 1] = r if i + 1 < n else 2 * r
            if i + 1 < n:
                L[i, i + 1] = r if i > 0 else 2 * r
            L[i, i] = -L[i].sum()
        v = V[at:at + n]
        out[at:at + n] = v + np.linalg.solve(np.eye(n) - theta * L, L @ v)
        at += n
    return out


@pytest.mark.parametrize("dt,scheme,width", WIDTHS)
@pytest.mark.parametrize("path", ["windows", "predictor", "st57"])
def test_one_step_is_the_tridiagonal_solve(path, dt, scheme, width):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _width(dt, scheme) == width
    rng = np.random.default_rng(width)
    # just longer than the stencil, and ends anywhere in a block
    nn = rng.integers(width + 1, width + 60, 300).astype(np.int32)
    nn[:3] = width + 1
    vm = rng.normal(0.0, 20.0, nn.sum()).astype(np.float32)
    model = F.FIB_MODEL_ST57 if path == "st57" else F.FIB_MODEL_HH

    def solver():
        s = F.Solver(nn, model=model, schedule=F.FIB_SCHED_SPLIT, Cm=CM, Am=AM, sigma=SIGMA, h=H,
                     dt_0D=dt / 16, dt_1D=dt, dt_split=dt, time_1d=scheme)
        s.init_state(vm)
        return s

    s = solver()
    if path == "predictor":
        s.set_predictor(F.FIB_PRED_EULER, [100.0, 1.0, 1.0, 1.0], 1e-3)
    s.run(0, 1)
    s.sync()
    got = s.state_tensor()[0].cpu().numpy()
    s.close()
    hand = []
    for on_host in (True, False):
        s = solver()
        s.step_reaction(0, 0.5 * dt)
        if on_host:
            rows, ref = s.state_tensor()
            V = _diffuse(rows[0].cpu().numpy().astype(np.float64), nn, dt, scheme)
            rows[0].copy_(torch.as_tensor(V.astype(np.float32)))
        else:
            s.step_diffusion(dt)
        s.step_reaction(0, 0.5 * dt)
        s.sync()
        hand.append(s.state_tensor()[0].cpu().numpy())
        s.close()
    err = np.max(np.abs(got[0] - hand[0][0]))
    say(f"[stencil widths] {path} dt {dt} scheme {scheme} width {width}: {err:.1e} mV")
    assert not np.array_equal(got, hand[1])
    assert err < 1e-4
