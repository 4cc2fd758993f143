"""The training loss is the sum of the squares of the differences of the
network's own FP32 outputs from the targets: within 1.2e-7 of that sum in FP64,
two roundings to FP32 (the loss itself and the differences)."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes,act", [([57, 128, 128, 57], "relu"), ([5, 64, 64, 64, 4], "silu")])
@pytest.mark.parametrize("B", [1, 33, 1000, 8192, 8191, 25408 + 33])
def test_loss_is_the_sum_of_its_squares(sizes, act, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(B)
    params = [(W, 0.1 * rng.standard_normal(b.shape)) for W, b in M.init_params(sizes, 4)]
    net = F.Mlp(sizes, act=act)
    net.set_params(M.flatten(params).astype(np.float32))
    X = rng.standard_normal((B, sizes[0])).astype(np.float32)
    T = rng.standard_normal((B, sizes[-1])).astype(np.float32)
    Xt, Tt = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    _, loss = net.gradient(Xt, Tt)
    O = net.forward(Xt).cpu().numpy()
    diff = (O - T).astype(np.float64)
    want = np.sum(diff * diff) / (2.0 * B * sizes[-1])
    err = abs(float(loss.item()) - want) / want
    say(f"[mlp loss] {sizes} B={B}: {err:.1e}")
    assert err < 1.2e-7
    net.close()
