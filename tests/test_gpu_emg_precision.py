"""phi_e of the preconditioned EMG solve keeps the precision of its FP32 inputs
and results, whatever the mesh's shape: thin bundles, many layers, layers much
closer than the fibers.  The oracle solves in FP64 from the same V_m.

The bound, relative and in the 2-norm: four times what one rounding of the
right-hand side to FP32 moves the oracle's phi_e (the right-hand side is stored
so; this is the part that grows with the layers), and four roundings of
phi_e itself, 2^-24 each (x and each iteration's update are stored so).  A
residual or operator rounded to FP32 adds errors of the size of the operator's
largest terms, which the smooth modes amplify, and goes past it."""
import numpy as np
import pytest

from oracle import emg as E
from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIG = dict(sigma_i=8.93, sigma_el=6.7, sigma_et=3.35)


@pytest.mark.parametrize("nx,ny,n,m", [
    (5, 4, 121, 5), (3, 8, 737, 8), (6, 5, 471, 10), (30, 5, 336, 5), (5, 6, 1601, 25),
    (17, 18, 141, 10)])
def test_phi_keeps_single_precision(nx, ny, n, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = F.Solver(np.full(nx * ny, n, np.int32), Cm=1.0, Am=500.0, sigma=3.828, h=0.01)
    # a pulse on every fiber, each at a place of its own
    rng = np.random.default_rng(nx * ny + n)
    x = np.arange(n)[None, :] / n
    vm = 90.0 * np.exp(-((x - rng.uniform(0.2, 0.8, (nx * ny, 1))) / 0.1) ** 2)
    s.init_state(vm.reshape(-1).astype(np.float32))
    emg = F.Emg(s, nx, ny, m, 0.05, 0.04, **SIG)
    it, rel = emg.solve(tol=1e-7, max_iter=100)
    phi = emg.phi()
    V3 = E.prolongate(s.get_state()[0], nx, ny, n, m)
    g = E.Grid(nx, ny, (n - 1) // m + 1, 0.05, 0.04, m * 0.01)
    phi_o, b = E.solve(g, V3, SIG["sigma_i"], SIG["sigma_el"], SIG["sigma_et"])
    Kt = E.stiffness_3d(g, (SIG["sigma_et"], SIG["sigma_et"], SIG["sigma_el"] + SIG["sigma_i"]))
    moved = E.solve_neumann(Kt, b.astype(np.float32) - b)
    size = np.linalg.norm(phi_o)
    bound = 4 * np.linalg.norm(moved) / size + 4 * 2.0 ** -24
    err = np.linalg.norm(phi - phi_o) / size
    say(f"[emg precision] {nx}x{ny}x{g.nz}: {it} iterations to {rel:.1e}, error {err:.2e}, "
        f"bound {bound:.2e}")
    assert rel <= 1e-7 and err < bound
    emg.close()
    s.close()
