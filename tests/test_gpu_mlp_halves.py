"""The sums over the rows of a gradient pass: its two halves of 64 rows are summed apart and added at the end.
The gradient of 128 rows is then the mean of the gradients of its halves, to the last bit: the pre-activation
gradients of a half are scaled by two exactly (they carry 1/n, and BF16 roundings are scale-free in powers of
two), and the one FP32 addition rounds the same.  One chain of sums over all 128 rows rounds differently, and
further from the exact sums."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4  # noqa: E402
from test_gpu_mlp import BLOCKS, dev, mlp_inputs  # noqa: E402
from test_gpu_mlp_rows import gradient  # noqa: E402


@pytest.mark.parametrize("seed", [31, 32, 33])
def test_halves_are_summed_apart(seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()
    prm, feat, norm, tags = (dev(a) for a in mlp_inputs(128, seed))
    whole, _, _ = gradient(prm, norm, feat, tags)
    first, _, _ = gradient(prm, norm, feat[:64].contiguous(), tags[:64].contiguous())
    second, _, _ = gradient(prm, norm, feat[64:].contiguous(), tags[64:].contiguous())
    for name in ("W1", "W2", "W3"):
        a, b = BLOCKS[name]
        assert (whole[a:b] == (first[a:b] + second[a:b]) / 2).all(), name
