"""The stage combine ccz4_rk4_stage, cell for cell, against the two-register form in torch: interior
cells and the ghosts of Sommerfeld faces are combined, every other element of acc and Qnext is left
alone, and s = 3 projects the interior (det gt = 1, tr At = 0) but no ghost.

Tolerance: each value is a sum of two products rounded once or twice, so at most three units of FP64
rounding of its terms; the projection of data of order one with det gt near one adds a cube root and
products of three entries, under 100 units.  Sizes: one leaf with six boundary faces, counts that are no multiple of
8 (the launch is padded to one), no boundary at all, and a refined leaf away from the boundary."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2406_11626_amd import ccz4, scenarios  # noqa: E402

EPS = float(np.finfo(np.float64).eps)
GT, AT = slice(0, 6), slice(11, 17)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ccz4.lib()


def combined_cells(ctx, n, bc):
    """True on the cells that a stage combines: [leaf, z, y, x] of the box."""
    m = torch.zeros((ctx.n_patches, 15, 15, 16), dtype=torch.bool)
    m[:, 3:12, 3:12, 3:12] = True
    inside = m.clone()
    if bc == ccz4.BC_SOMMERFELD:
        for p, (lev, *ijk) in enumerate(ctx.ids):
            for a in range(3):
                for side in (0, 1):
                    if ijk[a] != (0 if side == 0 else n[a] * 3 ** int(lev) - 1):
                        continue
                    box = [slice(3, 12)] * 3
                    box[2 - a] = slice(0, 3) if side == 0 else slice(12, 15)
                    m[(p, *box)] = True
    return m.cuda()[:, None], inside.cuda()[:, None]


@pytest.mark.parametrize("s", [0, 1, 2, 3])
@pytest.mark.parametrize("n,bc,refined", [
    ((1, 1, 1), ccz4.BC_SOMMERFELD, []),
    ((3, 1, 1), ccz4.BC_SOMMERFELD, []),
    ((2, 1, 1), ccz4.BC_PERIODIC, []),
    ((3, 3, 3), ccz4.BC_SOMMERFELD, [(0, 1, 1, 1)]),
])
def test_combine(n, bc, refined, s):
    ctx = ccz4.Context(n, (0.0,) * 3, tuple(float(a) for a in n), bc, scenarios.config(2).params(), refined)
    torch.manual_seed(11 + s)
    shape = (ctx.n_patches, ccz4.NV, 15, 15, 16)
    Q, k, acc, Qx = (torch.rand(shape, dtype=torch.float64, device="cuda") - 0.5 for _ in range(4))
    for t in (Q, acc):
        t[:, GT] *= 0.1
        for v in (0, 3, 5):
            t[:, v] += 1.0
    dt = 0.01
    where, inside = combined_cells(ctx, n, bc)
    a0, x0 = acc.clone(), Qx.clone()
    if s == 0:
        want_a, want_x = Q + dt / 6 * k, Q + dt / 2 * k
    elif s < 3:
        want_a, want_x = acc + dt / 3 * k, Q + (dt / 2 if s == 1 else dt) * k
    else:
        want_a, want_x = acc, acc + dt / 6 * k
    want_a, want_x = torch.where(where, want_a, a0), torch.where(where, want_x, x0)
    ctx.rk4_stage(s, dt, Q, k, acc, Qx)
    assert torch.equal(acc[~where.expand(shape)], a0[~where.expand(shape)])
    assert torch.equal(Qx[~where.expand(shape)], x0[~where.expand(shape)])
    bound = 3 * EPS * (torch.maximum(Q.abs(), a0.abs()) + dt * k.abs())
    if s == 3:
        q = want_x.clone()
        g = torch.stack([q[:, v] for v in (0, 1, 2, 1, 3, 4, 2, 4, 5)], -1).reshape(ctx.n_patches, 15, 15, 16, 3, 3)
        ok = inside[:, 0]
        gi = g[ok].cpu()
        gi = gi / torch.linalg.det(gi)[:, None, None] ** (1.0 / 3.0)
        A = torch.stack([q[:, 11 + v] for v in (0, 1, 2, 1, 3, 4, 2, 4, 5)], -1).reshape(*g.shape)[ok].cpu()
        tr = (torch.linalg.inv(gi) * A).sum((1, 2))
        A = A - gi * tr[:, None, None] / 3.0
        for v, (i, j) in enumerate(((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))):
            want_x[:, v][ok] = gi[:, i, j].cuda()
            want_x[:, 11 + v][ok] = A[:, i, j].cuda()
        both = inside.expand(shape).clone()
        both[:, 6:11] = both[:, 17:] = False
        bound = torch.where(both, 100 * EPS * torch.ones_like(bound), bound)
    assert ((acc - want_a).abs() <= bound).all()
    assert ((Qx - want_x).abs() <= bound).all()
