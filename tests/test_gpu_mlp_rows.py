"""Row counts at which the perceptron's gradient kernel changes its work: a wave's 16 rows, a pass's 128
and the grid's 256 passes.  Repeating a batch 2^k times divides every pre-activation gradient by 2^k
exactly (BF16 roundings are scale-free in powers of two), so the gradient of the repeated batch is that
of the batch up to the order of its FP32 sums, whatever waves and passes its rows fall into: 1e-5
normwise per tensor (sums of up to 40,000 terms at 6e-8, growing as the square root).  The logits of
equal rows are equal bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4  # noqa: E402
from test_gpu_mlp import BLOCKS, dev, mlp_inputs, rel  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


def gradient(prm, norm, feat, tags):
    n = feat.shape[0]
    work = torch.empty(ccz4.ccz4_mlp_workspace(n), dtype=torch.float32, device="cuda")
    grad = torch.empty(ccz4.MLP_NPARAM, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    logits = torch.empty((n, 3), dtype=torch.float32, device="cuda")
    ccz4.ccz4_mlp_grad(prm, norm, feat, tags, n, work, grad, loss)
    ccz4.ccz4_mlp_forward(prm, norm, feat, n, logits)
    return grad.cpu().numpy(), float(loss.item()), logits


@pytest.mark.parametrize("n", [1, 15, 17, 127, 129, 1025])
def test_repeated_batches_give_the_same_gradient(n):
    prm, feat, norm, tags = (dev(a) for a in mlp_inputs(n, 90 + n))
    g, loss, z = gradient(prm, norm, feat, tags)
    for k in (1, 32 if n > 1000 else 2048 if n < 20 else 256):  # the last beyond one pass of the full grid
        gk, lk, zk = gradient(prm, norm, feat.repeat(k, 1), tags.repeat(k))
        assert torch.equal(zk, z.repeat(k, 1))
        assert abs(lk - loss) <= 1e-5 * abs(loss)
        for name, (a, b) in BLOCKS.items():
            assert rel(gk[a:b], g[a:b]) <= 1e-5, (name, k, rel(gk[a:b], g[a:b]))
