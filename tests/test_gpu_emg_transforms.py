"""The EMG solve at the edges of its transforms: axes of 2 nodes and around the
16-node tiles, more layers than two panels of a block's LDS hold, and a bundle
beyond the transforms (130 fibers along x), which keeps the diagonal
preconditioner.  phi_e against the oracle's direct solve to 1e-4 of its largest
value at a relative residual of 1e-7, the bound of the other EMG tests; with
the transforms in at most 20 iterations (each removes two to three digits of the
residual; the diagonal preconditioner takes hundreds), and to 1e-9 in at most
30."""
import numpy as np
import pytest

from oracle import emg as E
from paper_2107_07104_amd import fib as F
from paper_2107_07104_amd import inputs as I

from gpu_helpers import gpu_solver, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIG = dict(sigma_i=8.93, sigma_el=6.7, sigma_et=3.35)


@pytest.mark.parametrize("nx,ny,n,m", [(2, 2, 33, 16), (16, 17, 97, 6), (17, 15, 161, 10),
                                       (3, 2, 1481, 1), (130, 2, 61, 10)])
def test_phi_at_the_edges_of_the_transforms(nx, ny, n, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = I.batched_hh(n_fibers=nx * ny, n_min=n, n_max=n, t_end=1.0, onset_max=0.4)
    s = gpu_solver(w)
    s.run(0, 900)
    s.sync()
    emg = F.Emg(s, nx, ny, m, 0.05, 0.04, **SIG)
    it, rel = emg.solve(tol=1e-7, max_iter=5000)
    phi = emg.phi()
    V3 = E.prolongate(s.get_state()[0], nx, ny, n, m)
    g = E.Grid(nx, ny, (n - 1) // m + 1, 0.05, 0.04, m * w.h)
    phi_o, _ = E.solve(g, V3, SIG["sigma_i"], SIG["sigma_el"], SIG["sigma_et"])
    err = np.max(np.abs(phi - phi_o)) / np.max(np.abs(phi_o))
    it2, rel2 = emg.solve(tol=1e-9, max_iter=5000)
    say(f"[emg transforms] {nx}x{ny}x{g.nz}: {it} iterations to {rel:.1e}, phi err {err:.1e}; "
        f"{it2} more to {rel2:.1e}")
    assert rel <= 1e-7 and rel2 <= 1e-9 and err < 1e-4
    assert abs(phi.mean()) < 1e-6 * np.max(np.abs(phi_o))
    if nx <= 128:
        assert it <= 20 and it2 <= 30
    # a limit is kept, and reported as not reached
    s.run(900, 100)
    it3, rel3 = emg.solve(tol=1e-9, max_iter=1)
    assert it3 == 1 and rel3 > 1e-9
    emg.close()
    s.close()
