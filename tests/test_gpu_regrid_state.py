"""A regridded state made in one pass (ccz4_regrid_state) against its parts: a zeroed state, the initial
data, then ccz4_regrid_transfer.  The same kernels form the same values: equality, bit for bit, of the
whole state (halos, corners and the padding column included) and of the Sommerfeld background, seen
through the right-hand side on the evolved ghosts.

The tags refine a leaf (and with it its coarser face neighbours) or coarsen the family at a domain corner, so that copied, interpolated and
averaged leaves all lie on the outer boundary."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402

BL_BY = [0.5, 0.9, 0.1, -0.2, 0.0, 0.1, 0.0, 0.5, -0.8, 0.0, 0.1, 0.0, -0.1, 0.0]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


@pytest.mark.parametrize("bc", [ccz4.BC_SOMMERFELD, ccz4.BC_NEUMANN])
@pytest.mark.parametrize("scen,args", [(ccz4.SCEN_PUNCTURE, [1.0, 0.1, 0.2, 0.3, 0]), (ccz4.SCEN_BL_BY, BL_BY)])
@pytest.mark.parametrize("change", ["none", "refine", "coarsen"])
def test_one_pass(bc, scen, args, change):
    n = (3, 2, 3)
    old = ccz4.Context(n, (-4.0,) * 3, (8.0,) * 3, bc, ccz4.params(**scenarios.BLACK_HOLE), [(0, 0, 0, 0)])
    torch.manual_seed(3)
    Q = old.new_state()
    old.init_patches(Q, scen, args)
    Q += 1e-3 * torch.rand_like(Q)
    tags = np.zeros(old.n_patches, np.int8)
    if change == "refine":
        tags[-1] = 1
    elif change == "coarsen":
        tags[old.ids[:, 0] == 1] = -1
    refined = [tuple(int(v) for v in r) for r in ccz4.ccz4_regrid_plan(old.h, tags, 2)]
    assert np.sign(len(refined) - 1) == {"none": 0, "refine": 1, "coarsen": -1}[change]
    a = ccz4.Context(n, old.origin, old.extent, bc, old.prm, refined)
    A = a.new_state(0.0)
    a.init_patches(A, scen, args)
    ccz4.ccz4_regrid_transfer(old.h, Q, a.h, A)
    b = ccz4.Context(n, old.origin, old.extent, bc, old.prm, refined)
    B = b.new_state(float("nan"))
    ccz4.ccz4_regrid_state(old.h, Q, b.h, B, scen, args)
    assert torch.equal(A, B)
    ka, kb = a.new_state(), b.new_state()
    for c, S, k in ((a, A, ka), (b, B, kb)):
        c.fill_halos(S)
        c.rhs(S, k)
    assert torch.isfinite(ka).all() and torch.equal(ka, kb)


def test_refusals():
    a, b = (ccz4.Context((2, 1, 1), (0.0,) * 3, (2.0, 1.0, 1.0), ccz4.BC_SOMMERFELD) for _ in range(2))
    Q, R = a.new_state(), b.new_state()
    with pytest.raises(ccz4.CCZ4Error):  # unknown scenario
        ccz4.ccz4_regrid_state(a.h, Q, b.h, R, 7, [0.0] * 14)
    with pytest.raises(ccz4.CCZ4Error):  # too few parameters
        ccz4.ccz4_regrid_state(a.h, Q, b.h, R, ccz4.SCEN_BL_BY, [0.0] * 13)
    with pytest.raises(ccz4.CCZ4Error):  # one state
        ccz4.ccz4_regrid_state(a.h, Q, b.h, Q, ccz4.SCEN_PUNCTURE, [1.0, 0.0, 0.0, 0.0, 0])
    assert not R.any()
