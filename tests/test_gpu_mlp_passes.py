"""The perceptron's gradient where its work-groups take several passes of 128 rows: the grid is 256 work-groups,
so that 32,768 rows are one full pass.  A batch repeated 2^k times has the batch's gradient up to the order of its
FP32 sums (every pre-activation gradient is divided by 2^k exactly): normwise per tensor 1e-5 for up to 70,000
terms of 6e-8 each, growing as the square root.  The last case has eight full passes and a ragged ninth."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4  # noqa: E402
from test_gpu_mlp import BLOCKS, dev, mlp_inputs, rel  # noqa: E402
from test_gpu_mlp_rows import gradient  # noqa: E402

PASS = 256 * 128


@pytest.mark.parametrize("n,copies,passes", [(1, 1 << 17, 4), (15, 1 << 13, 3), (127, 1 << 10, 3), (129, 1 << 10, 4),
                                             (1025, 1 << 8, 8)])
def test_several_passes(n, copies, passes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()
    assert passes * PASS <= n * copies < (passes + 2) * PASS
    prm, feat, norm, tags = (dev(a) for a in mlp_inputs(n, 60 + n))
    g, loss, z = gradient(prm, norm, feat, tags)
    gk, lk, zk = gradient(prm, norm, feat.repeat(copies, 1), tags.repeat(copies))
    assert torch.equal(zk, z.repeat(copies, 1))
    assert abs(lk - loss) <= 1e-5 * abs(loss)
    for name, (a, b) in BLOCKS.items():
        assert rel(gk[a:b], g[a:b]) <= 1e-5, (name, rel(gk[a:b], g[a:b]))
