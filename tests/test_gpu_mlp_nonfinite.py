"""Infinite values in a network's forward pass reach the outputs they reach in
FP32 and no others: with positive weights an infinite input gives an infinite
output (not the NaN that a padded feature, 0 * inf, would add), and the other
samples of its chunk keep their values bit for bit."""
import numpy as np
import pytest

from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("act", ["silu", "relu"])
@pytest.mark.parametrize("sizes", [[2, 20, 1], [3, 16, 40, 2], [33, 17, 5, 3], [4, 32, 3]])
def test_infinite_input_reaches_its_own_outputs_only(sizes, act):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[mlp non-finite] {sizes} {act}")
    rng = np.random.default_rng(5)
    n = sum(a * b + b for a, b in zip(sizes, sizes[1:]))
    net = F.Mlp(sizes, act=act)
    net.set_params(rng.uniform(0.1, 1.0, n).astype(np.float32))
    X = torch.as_tensor(rng.uniform(0.1, 1.0, (37, sizes[0])).astype(np.float32), device="cuda")
    base = net.forward(X).cpu().numpy()
    X[5, 1] = float("inf")
    out = net.forward(X).cpu().numpy()
    assert np.isfinite(base).all()
    assert np.isposinf(out[5]).all()
    keep = np.arange(37) != 5
    np.testing.assert_array_equal(out[keep], base[keep])
    net.close()
