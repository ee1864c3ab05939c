"""The refinement criterion's third indicator, dx^2 max |H| of a leaf, formed without the momentum
constraints and the norms, against H of the monitor on the same state.

Tolerance: the two kernels run the same formula; the compiler may fuse its multiplications and
additions differently, a few units of FP64 rounding of the terms, which are of the size of the curvature
terms of H (at most 1e4 here), not of H itself: 1e-12 of the largest |H| plus 1e-11.  Sizes: one leaf,
counts that are no multiple of 8 (the launch is padded to one), a refined mesh.  A non-finite value in a
slot that does not enter H leaves the indicator alone; in one that does, the cell drops out of the
maximum as it does in the maximum over the monitor's H."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


def both(n, refined, poke=()):
    ctx = ccz4.Context(n, (-3.0,) * 3, tuple(2.0 * a for a in n), ccz4.BC_SOMMERFELD,
                       ccz4.params(**scenarios.BLACK_HOLE), refined)
    Q = ctx.new_state()
    ctx.init_patches(Q, ccz4.SCEN_PUNCTURE, [1.0, 0.4, 0.3, -0.2, 0])
    torch.manual_seed(2)
    Q[..., :15] += 1e-3 * torch.rand_like(Q[..., :15])
    ctx.fill_halos(Q)
    for v in poke:
        Q[0, v, 7, 7, 7] = float("nan")
    HM = torch.zeros((ctx.n_patches, 4, 729), dtype=torch.float64, device="cuda")
    ccz4.lib().ccz4_constraints(ctx.h, Q.data_ptr(), HM.data_ptr(), 0.0, None, None)
    tags = torch.zeros(ctx.n_patches, dtype=torch.int8, device="cuda")
    ind = torch.full((ctx.n_patches, 3), -1.0, dtype=torch.float64, device="cuda")
    ctx.tag_refine(Q, 1e300, 0.0, 3, tags, ind)
    torch.cuda.synchronize()
    h = HM[:, 0].abs()
    h = torch.where(torch.isnan(h), torch.zeros_like(h), h)
    dx = torch.tensor(ctx.geom[:, 3], device="cuda")
    return ind[:, 2], dx * dx * h.amax(1), dx * dx


@pytest.mark.parametrize("n,refined", [((1, 1, 1), []), ((3, 3, 1), []), ((2, 3, 4), []),
                                       ((3, 3, 3), [(0, 1, 1, 1)])])
def test_indicator_is_the_monitors(n, refined):
    got, want, d2 = both(n, refined)
    assert (want > 0).all()
    assert ((got - want).abs() <= 1e-12 * want + 1e-11 * d2).all()


@pytest.mark.parametrize("slot", [7, 19, 22, 25, 28, 58])
def test_slots_that_do_not_enter(slot):
    got, want, d2 = both((2, 1, 1), [], (slot,))
    assert torch.isfinite(got).all()
    assert ((got - want).abs() <= 1e-12 * want + 1e-11 * d2).all()


@pytest.mark.parametrize("slot", [0, 10, 11, 17, 37, 55])
def test_non_finite_cells(slot):
    got, want, d2 = both((2, 1, 1), [], (slot,))
    assert torch.isfinite(got).all()
    assert ((got - want).abs() <= 1e-12 * want + 1e-11 * d2).all()
