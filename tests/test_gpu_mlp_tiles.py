"""The network kernels at the edges of their tiles: widths around 16 and 32
(the matrix-core tile and the padding), batches of one sample, one chunk of
32 samples and just beyond, and 258 chunks, more than the 128 whose operands
the gradient's contraction has in flight.

Reference: oracle/mlp.py in FP64 on bfloat16-rounded operands, which takes the
same rounding decisions as the device except where FP32 and FP64
accumulation round a value to different sides.  A flipped BF16 rounding
changes one operand by 2^-8 relative, and sums over K operands average such
flips, so a few times 2^-8 of the largest value bounds them: 2e-2 (the other
network tests' 3e-2 covers unrounded references)."""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [([1, 1], 1, "relu"), ([15, 16, 17], 31, "silu"), ([16, 33, 32, 1], 32, "relu"),
         ([57, 31, 64, 3], 33, "silu"), ([33, 17, 65, 2], 8192 + 33, "relu"),
         ([320, 320], 70, "relu")]


@pytest.mark.parametrize("sizes,B,act", CASES)
def test_forward_and_gradient_at_tile_edges(sizes, B, act):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    say(f"[mlp tiles] {sizes} B={B} {act}")
    rng = np.random.default_rng(3)
    params = [(W, 0.1 * rng.standard_normal(b.shape)) for W, b in M.init_params(sizes, 4)]
    params = [(W.astype(np.float32).astype(np.float64), b.astype(np.float32).astype(np.float64))
              for W, b in params]
    net = F.Mlp(sizes, act=act)
    net.set_params(M.flatten(params).astype(np.float32))
    X = rng.standard_normal((B, sizes[0])).astype(np.float32)
    T = rng.standard_normal((B, sizes[-1])).astype(np.float32)
    Xt, Tt = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    O = net.forward(Xt).cpu().numpy()
    ref, _ = M.forward(params, X.astype(np.float64), act, bf16=True)
    assert np.max(np.abs(O - ref)) <= 2e-2 * np.max(np.abs(ref))
    g, loss = net.gradient(Xt, Tt)
    ref_g = M.backward(params, X.astype(np.float64), T.astype(np.float64), act, bf16=True)
    for li, ((gW, gb), (rW, rb)) in enumerate(
            zip(M.unflatten(g.cpu().numpy().astype(np.float64), sizes), ref_g)):
        for name, a, r in (("W", gW, rW), ("b", gb, rb)):
            worst = np.max(np.abs(a - r)) / max(np.max(np.abs(r)), 1e-30)
            say(f"   layer {li + 1} {name}: {worst:.2e}")
            assert worst < 2e-2, (li, name)
    ref_loss = M.loss(params, X.astype(np.float64), T.astype(np.float64), act)
    assert abs(float(loss.item()) - ref_loss) < 2e-2 * ref_loss
    # the step leaves the operand fragments at the new parameters
    net.adam_step(Xt, Tt, 1e-2)
    p1 = M.unflatten(net.get_params().astype(np.float64), sizes)
    O1 = net.forward(Xt).cpu().numpy()
    ref1, _ = M.forward(p1, X.astype(np.float64), act, bf16=True)
    assert np.max(np.abs(O1 - ref1)) <= 2e-2 * np.max(np.abs(ref1))
    net.close()
