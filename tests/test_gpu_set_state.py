"""The state a context starts with, and the populations it is set to: every
boundary kind, form and lattice, single and in a batch, against the values
written down with numpy.  Needs an MI355X."""
import numpy as np
import pytest

from gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu

CX = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1])
CY = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])
W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


def _equilibrium(lattice, rho, ux, uy):
    cx, cy, w = (CX, CY, W9) if lattice == "d2q9" else (np.array([0, 1, -1]), np.zeros(3), np.array([2 / 3, 1 / 6, 1 / 6]))
    cu = np.multiply.outer(cx, ux) + np.multiply.outer(cy, uy)
    return w.reshape(-1, *[1] * rho.ndim) * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy))


def _inside(lattice, bc, nx, ny):
    """Per direction, the nodes whose upstream node is in the lattice."""
    y, x = np.mgrid[0:ny, 0:nx]
    out = []
    for cx, cy in zip(CX, CY) if lattice == "d2q9" else ((0, 0), (1, 0), (-1, 0)):
        okx = (bc == "periodic") | ((x - cx >= 0) & (x - cx < nx))
        oky = (lattice == "d1q3") | (bc in ("periodic", "tube")) | ((y - cy >= 0) & (y - cy < ny))
        out.append(okx & oky)
    return np.array(out)


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("lattice,bc", [("d2q9", "cavity"), ("d2q9", "periodic"), ("d2q9", "tube"), ("d2q9", "box"),
                                        ("d1q3", "tube"), ("d1q3", "periodic")])
def test_initial_and_restored_populations(lattice, bc, batch):
    # FP64 values are written as computed or as given; the equilibrium's
    # few operations are rounded alike up to their order (1e-15 of the weights)
    b = B()
    q = 9 if lattice == "d2q9" else 3
    sizes = [(17, 9), (3, 3), (300, 5), (64, 70)] if batch else [(37, 21)]
    sizes = sizes if q == 9 else [(nx * ny, 1) for nx, ny in sizes]
    params = [b.make_params(lattice, "srt", bc, "fp64", nx, ny, 0.7, 0.0, 0.05, 1.0) for nx, ny in sizes]
    fields = [smooth_fields(nx, ny, seed=800 + k) for k, (nx, ny) in enumerate(sizes)]
    if q == 3:
        fields = [(r, u, np.zeros_like(v)) for r, u, v in fields]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    ctx = b.lbm_init_batch(params, rho, ux, uy) if batch else b.lbm_init(params[0], rho, ux, uy)
    try:
        got, want, ok = b.lbm_get_populations(ctx, q), [], []
        for (nx, ny), (r, u, v) in zip(sizes, fields):
            f = _equilibrium(lattice, r, u, v)
            if bc == "cavity":
                f[:, -1, :] = _equilibrium(lattice, np.ones(nx), np.full(nx, 0.05), np.zeros(nx))
            want.append(f.reshape(-1))
            ok.append(_inside(lattice, bc, nx, ny).reshape(-1))
        want, ok = np.concatenate(want), np.concatenate(ok)
        assert np.max(np.abs(got - want)[ok]) <= 1e-15
        new = np.random.default_rng(1).uniform(0.01, 0.1, got.size)
        b.lbm_set_populations(ctx, new)
        assert np.array_equal(b.lbm_get_populations(ctx, q)[ok], new[ok])
    finally:
        b.lbm_free(ctx)
