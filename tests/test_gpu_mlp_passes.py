"""Training batches around and past one pass of the gradient kernels (794 chunks
of 32 samples for one layer of 320 x 320, 1787 for the narrow network).

* Gradient and loss against oracle/mlp.py in FP64 on bfloat16-rounded operands,
  with the 2e-2 of the other batch sizes, and one Adam step against the update
  formed from that gradient: parameters below 0.5 and steps of 1e-2 round to
  less than 1e-7.
* A gradient's sums have one order, over the samples of a chunk and then the
  chunks, also across passes: the bias gradients of a batch are bitwise those of
  FP32 sums in that order, taken from each chunk's own gradient.  (A batch of
  one chunk has another 1 / B; powers of two keep every bit.)"""""
import numpy as np
import pytest

from oracle import mlp as M
from paper_2107_07104_amd import fib as F

from gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _setup(sizes, B, act, seed=3):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(seed)
    params = [(W.astype(np.float32).astype(np.float64),
               (0.1 * rng.standard_normal(b.shape)).astype(np.float32).astype(np.float64))
              for W, b in M.init_params(sizes, 4)]
    net = F.Mlp(sizes, act=act)
    net.set_params(M.flatten(params).astype(np.float32))
    X = rng.standard_normal((B, sizes[0])).astype(np.float32)
    T = rng.standard_normal((B, sizes[-1])).astype(np.float32)
    return net, params, X, T, torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")


@pytest.mark.parametrize("sizes,B", [([320, 320], 794 * 32), ([320, 320], 794 * 32 + 33),
                                     ([33, 17, 65, 2], 1787 * 32 + 1)])
def test_gradient_and_step_past_one_pass(sizes, B):
    net, params, X, T, Xt, Tt = _setup(sizes, B, "relu")
    say(f"[mlp passes] {sizes} B={B}")
    g, loss = net.gradient(Xt, Tt)
    g = g.cpu().numpy().astype(np.float64)
    ref = M.backward(params, X.astype(np.float64), T.astype(np.float64), "relu", bf16=True)
    for li, ((gW, gb), (rW, rb)) in enumerate(zip(M.unflatten(g, sizes), ref)):
        for name, a, r in (("W", gW, rW), ("b", gb, rb)):
            worst = np.max(np.abs(a - r)) / max(np.max(np.abs(r)), 1e-30)
            say(f"   layer {li + 1} {name}: {worst:.2e}")
            assert worst < 2e-2, (li, name)
    ref_loss = M.loss(params, X.astype(np.float64), T.astype(np.float64), "relu")
    assert abs(float(loss.item()) - ref_loss) < 2e-2 * ref_loss
    p0 = net.get_params().astype(np.float64)
    l2 = torch.zeros(1, device="cuda")
    net.adam_step(Xt, Tt, 1e-2, l2)
    # the first step of Adam: both moments are the gradient's own
    want = p0 - 1e-2 * g / (np.abs(g) + 1e-8)
    assert np.max(np.abs(net.get_params() - want)) < 1e-7
    assert float(l2.item()) == float(loss.item())
    net.close()


@pytest.mark.parametrize("chunks", [64, 2048])
def test_sums_keep_the_order_of_the_chunks_across_passes(chunks):
    # 2048 chunks of 320 x 320 take three passes
    sizes = [320, 320]
    net, _, _, _, Xt, Tt = _setup(sizes, 32 * chunks, "relu")
    say(f"[mlp passes] order over {chunks} chunks")
    n_w = sizes[0] * sizes[1]
    whole = net.gradient(Xt, Tt)[0][n_w:].cpu().numpy()
    want = np.zeros(sizes[1], np.float32)
    for c in range(chunks):
        rows = slice(32 * c, 32 * c + 32)
        part = net.gradient(Xt[rows], Tt[rows])[0][n_w:].cpu().numpy()
        want += part / np.float32(chunks)
    np.testing.assert_array_equal(whole, want)
    net.close()
