"""The constraint kernels' sums over the derivatives of D.  No difference of D_aaa enters H (its coefficient,
a 2 x 2 minor of the inverse metric with two equal rows, vanishes), so D_aaa of one cell, however large,
leaves H of every other cell as it is, to the last bit: an evaluation that lets the two products of the
minor cancel in rounded arithmetic leaves 1e-17 of it there.  At 1e12 the rounding of such a difference
would be about 1e-4 of H."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


@pytest.mark.parametrize("a,s", [(0, 0), (1, 3), (2, 5)])
def test_h_takes_no_difference_of_d_aaa(a, s):
    prm = scenarios.config(2).params()
    ctx = ccz4.Context((2, 1, 1), (0.0, 0.0, 0.0), (2.0, 1.0, 1.0), ccz4.BC_PERIODIC, prm)
    torch.manual_seed(5)
    Q = 0.01 * (torch.rand((2, ccz4.NV, 15, 15, 16), dtype=torch.float64, device="cuda") - 0.5)
    for v in (0, 3, 5, 6, 10):
        Q[:, v] += 1.0
    ctx.fill_halos(Q)
    H = [torch.zeros((2, 4, 729), dtype=torch.float64, device="cuda") for _ in range(2)]
    ind = [torch.zeros((2, 3), dtype=torch.float64, device="cuda") for _ in range(2)]
    tags = torch.zeros(2, dtype=torch.int8, device="cuda")
    P = Q.clone()
    z, y, x = 7, 8, 6
    P[1, 37 + 6 * a + s, z, y, x] = 1e12
    for q, h, i in zip((Q, P), H, ind):
        ctx.constraints(q, h)
        ctx.tag_refine(q, 1.0, 0.1, 1, tags, i)
    same = (H[0] == H[1])[:, 0].cpu()
    other = torch.ones((2, 9, 9, 9), dtype=torch.bool)
    other[1, z - 3, y - 3, x - 3] = False
    assert same[other.reshape(2, 729)].all()
    assert torch.equal(ind[0][0], ind[1][0])  # the criterion of the untouched leaf
