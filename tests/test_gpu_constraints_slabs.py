"""The constraint monitor by slabs of three planes (at most 85 leaves: three work-groups a leaf, one per CU)
and by whole leaves, on the same boxes: H and M of a leaf depend on its own box and spacing only, so the
first leaves of a mesh of 86 and a smaller mesh of those leaves alone must agree, and so must the norms and
the count of non-finite cells, those at the seams of the slabs among them.

Tolerance: both evaluate the same expression, whose products the compiler may fuse differently: H sums
about a hundred products of order 10 at most (fields of 0.02 around a flat metric at spacing 1/9: first
differences up to 0.3, their inverse-metric factors near 1), each rounded to 1e-15 at worst, in all 1e-13."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402

BIG = (2, 43, 1)  # 86 leaves: by whole leaves


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


def context(n):
    return ccz4.Context(n, (0.0,) * 3, tuple(float(a) for a in n), ccz4.BC_PERIODIC, scenarios.config(2).params())


def boxes():
    torch.manual_seed(7)
    Q = 0.02 * (torch.rand((86, ccz4.NV, 15, 15, 16), dtype=torch.float64, device="cuda") - 0.5)
    for v in (0, 3, 5, 6, 10):
        Q[:, v] += 1.0
    return Q


def monitor(n, Q):
    ctx = context(n)
    assert ctx.n_patches == Q.shape[0]
    HM = torch.zeros((ctx.n_patches, 4, 729), dtype=torch.float64, device="cuda")
    norms, _ = ctx.constraints(Q, HM)
    return HM, norms


@pytest.mark.parametrize("n", [(1, 1, 1), (3, 3, 1), (4, 4, 4), (5, 17, 1)])
def test_slabs_agree_with_whole_leaves(n):
    Q = boxes()
    count = n[0] * n[1] * n[2]
    whole, _ = monitor(BIG, Q)
    slabs, norms = monitor(n, Q[:count].contiguous())
    assert (whole[:count] - slabs).abs().max() <= 1e-13
    cells = count * 729
    assert norms[0] == pytest.approx(float(((whole[:count, 0] ** 2).sum() / cells).sqrt()), rel=1e-12)
    assert norms[1] == pytest.approx(float(((whole[:count, 1:] ** 2).sum() / cells).sqrt()), rel=1e-12)
    assert norms[2] == 0


@pytest.mark.parametrize("n", [(1, 1, 1), (5, 17, 1), BIG])
@pytest.mark.parametrize("slot", [7, 37, 57, 11, 17])
def test_bad_cells_at_the_seams(n, slot):
    count = n[0] * n[1] * n[2]
    Q = boxes()[:count].contiguous()
    for z in (3, 5, 6, 8, 9, 11):
        P = Q.clone()
        P[count - 1, slot, z, 7, 10] = float("nan")
        # y = 7 has two cells on either side, x = 10 two and one, z those inside the leaf
        reach = 1 + 4 + 3 + min(2, z - 3) + min(2, 11 - z) if slot != 7 else 1
        assert monitor(n, P)[1][2] == reach
