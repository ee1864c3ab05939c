"""The whole fused step (ccz4_step_fused): its stages read every same-level halo of the intermediate
states from the neighbours and combine in the closed form of RK4.  It equals the same step made of
single calls (every halo filled before each stage, two-register combine) up to rounding, and depends
on nothing its work buffers held, on meshes whose leaves are their own periodic neighbours, with
coarse-fine, Sommerfeld and Neumann faces on every axis, in both formulations and precisions.

Tolerance in FP64: the two combines differ by a few roundings per stage, which a step at CFL 0.1 does
not amplify beyond the weights of its stencils: 4 stages x 50 roundings of 2.2e-16 of a slot's size,
taken as 1e-13 for the slots the step combines.  Mixed precision: a flipped rounding of an FP32 term, the 1e-6 bound of that mode."""
import math

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_helpers import INTERIOR, SLABS, parity_error, to_gpu, to_host  # noqa: E402
from seeded_inputs import box_centers, smooth_state  # noqa: E402
from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


MESHES = {
    "self-neighbours": ((1, 2, 3), ccz4.BC_PERIODIC, []),
    "one leaf": ((1, 1, 1), ccz4.BC_SOMMERFELD, []),
    "levels, sommerfeld": ((3, 3, 2), ccz4.BC_SOMMERFELD, [(0, 1, 1, 0)]),
    "levels, neumann": ((2, 3, 3), ccz4.BC_NEUMANN, [(0, 0, 1, 1), (0, 1, 1, 1)]),
}


@pytest.mark.parametrize("formulation", [ccz4.FORMULATION_FO, ccz4.FORMULATION_SO])
@pytest.mark.parametrize("precision", [ccz4.PREC_FP64, ccz4.PREC_MIXED])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_whole_step_equals_single_calls(mesh, precision, formulation):
    import numpy as np
    n0, bc, refined = MESHES[mesh]
    ctx = ccz4.Context(n0, (0.3, -0.2, 0.1), tuple(float(n) for n in n0), bc,
                       ccz4.params(**{**scenarios.BLACK_HOLE, "formulation": formulation,
                                      "advection": 1 if mesh == "levels, neumann" else 0}), refined)
    Qo = np.stack([smooth_state(box_centers(g[:3], g[3:]), 7) for g in ctx.geom])
    Q = to_gpu(Qo)
    ctx.set_background(Q)
    ctx.fill_halos(Q)
    if formulation:
        ctx.reconstruct(Q, True)
        ctx.fill_halos(Q)
    R = Q.clone()
    dt = 0.1 * float(ctx.geom[:, 3:].min())
    nan = tuple(ctx.new_state(math.nan) for _ in range(3))
    ctx.rk4_step_fused(Q, dt, nan, precision)
    ctx.rk4_step_fused(R, dt, tuple(ctx.new_state(0.0) for _ in range(3)), precision, push=False)
    ctx.fill_halos(R)
    torch.cuda.synchronize()
    # the second-order auxiliaries are not combined but reconstructed: bit for bit from the step's own
    # primaries (against the other step their differences are those of the primaries over dx)
    e = parity_error(to_host(Q), to_host(R), INTERIOR | SLABS, nslots=25 if formulation else 59)
    if formulation:
        H = Q.clone()
        ctx.reconstruct(H, False)
        ctx.fill_halos(H)
        assert torch.equal(H, Q)
    assert e.max() <= (1e-13 if precision == ccz4.PREC_FP64 else 1e-6), (int(e.argmax()), e.max())
