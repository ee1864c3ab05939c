"""A fused step on either side of the size from which its stages stream their output past the caches (a
state of 256 MB: 157 leaves do not, 158 do): the step against the same stages with every halo filled in
between, to the rounding of the two forms of the combine (1e-13 of each slot's largest value, as for the
fused step on other meshes)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402


@pytest.mark.parametrize("precision", [ccz4.PREC_FP64, ccz4.PREC_MIXED])
@pytest.mark.parametrize("leaves", [157, 158])
def test_both_sides(leaves, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = ccz4.Context((leaves, 1, 1), (-0.5,) * 3, (1.0, 1.0 / leaves, 1.0 / leaves), ccz4.BC_PERIODIC,
                       ccz4.params(**scenarios.GAUGE))
    Q = ctx.new_state()
    ctx.init_patches(Q, ccz4.SCEN_GAUGE_WAVE, [0.01, 2.0])
    ctx.fill_halos(Q)
    R = Q.clone()
    dt = 0.1 * float(ctx.geom[:, 3:].min())
    for S, push in ((Q, True), (R, False)):
        ctx.rk4_step_fused(S, dt, tuple(ctx.new_state() for _ in range(3)), precision, push=push)
    inner = (slice(None), slice(None), slice(3, 12), slice(3, 12), slice(3, 12))
    scale = R[inner].abs().amax((0, 2, 3, 4)).clamp(min=1.0)
    err = (Q - R)[inner].abs().amax((0, 2, 3, 4)) / scale
    assert err.max() <= (1e-13 if precision == ccz4.PREC_FP64 else 1e-6), (int(err.argmax()), float(err.max()))
