"""The whole fused step on refined meshes, with data in every slot and work buffers full of NaN, against the
same step made of single calls: on either side of the size from which stages 0..2 stream their output past
the caches (157 leaves), where that output shares lines with Sommerfeld ghosts and level fills and is what
the reconstruction of the second-order formulation reads, and with the higher-order coarse-fine operators.
Interiors and face halos are compared.

Tolerance as for the fused step on small meshes: four stages of at most 50 roundings of a slot's size, 1e-13,
for the slots that the step combines; in mixed precision a flipped rounding of an FP32 term, 1e-6."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from gpu_helpers import INTERIOR, SLABS, parity_error, to_gpu, to_host  # noqa: E402
from seeded_inputs import box_centers, smooth_state  # noqa: E402
from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402

STREAMED = ((6, 5, 5), [(0, 3, 0, 2)])      # 176 leaves, level faces next to boundary faces
RESIDENT = ((5, 5, 5), [(0, 2, 4, 0)])      # 151
SMALL = ((3, 3, 2), [(0, 1, 1, 0), (0, 2, 1, 0), (1, 4, 4, 1)])  # three levels


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


@pytest.mark.parametrize("formulation", [ccz4.FORMULATION_FO, ccz4.FORMULATION_SO])
@pytest.mark.parametrize("mesh,transfer,precision,bc", [
    (STREAMED, ccz4.TRANSFER_APP_E, ccz4.PREC_FP64, ccz4.BC_SOMMERFELD),
    (STREAMED, ccz4.TRANSFER_HIGHER_ORDER, ccz4.PREC_MIXED, ccz4.BC_NEUMANN),
    (RESIDENT, ccz4.TRANSFER_APP_E, ccz4.PREC_FP64, ccz4.BC_SOMMERFELD),
    (SMALL, ccz4.TRANSFER_HIGHER_ORDER, ccz4.PREC_FP64, ccz4.BC_SOMMERFELD),
    (SMALL, ccz4.TRANSFER_HIGHER_ORDER, ccz4.PREC_MIXED, ccz4.BC_PERIODIC),
    (SMALL, ccz4.TRANSFER_HIGHER_ORDER, ccz4.PREC_FP64, ccz4.BC_NEUMANN),
])
def test_whole_step_equals_single_calls(mesh, transfer, precision, bc, formulation):
    n0, refined = mesh
    ctx = ccz4.Context(n0, (0.3, -0.2, 0.1), tuple(float(n) for n in n0), bc,
                       ccz4.params(**{**scenarios.BLACK_HOLE, "formulation": formulation, "transfer": transfer}), refined)
    assert (ctx.n_patches > 157) == (mesh is STREAMED)
    Q = to_gpu(np.stack([smooth_state(box_centers(g[:3], g[3:]), 7) for g in ctx.geom]))
    Q[:, 58] = 0.1 * Q[:, 17]  # K_0, which that state leaves at zero
    assert (Q[:, :, 3:12, 3:12, 3:12].abs().amax((0, 2, 3, 4)) > 0).all()
    ctx.set_background(Q)
    ctx.fill_halos(Q)
    if formulation:
        ctx.reconstruct(Q, True)
        ctx.fill_halos(Q)
    R = Q.clone()
    dt = 0.1 * float(ctx.geom[:, 3:].min())
    ctx.rk4_step_fused(Q, dt, tuple(ctx.new_state(math.nan) for _ in range(3)), precision)
    ctx.rk4_step_fused(R, dt, tuple(ctx.new_state(0.0) for _ in range(3)), precision, push=False)
    ctx.fill_halos(R)
    torch.cuda.synchronize()
    # the second-order auxiliaries follow from the step's own primaries, bit for bit
    if formulation:
        H = Q.clone()
        ctx.reconstruct(H, False)
        ctx.fill_halos(H)
        assert torch.equal(H, Q)
    e = parity_error(to_host(Q), to_host(R), INTERIOR | SLABS, nslots=25 if formulation else 59)
    assert e.max() <= (1e-13 if precision == ccz4.PREC_FP64 else 1e-6), (int(e.argmax()), e.max())
