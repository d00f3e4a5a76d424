"""Host transfers: fields and populations pass through a ring of pinned slots,
in pieces when they are larger than one.

Sizes sit at the edges: one slot, a few (copied by the caller), more than the
ring holds (several host threads), pieces that cut rows and batch instances.
What goes in comes back bit for bit, for single lattices and batches.
"""
import numpy as np
import pytest

from gpu_helpers import B, orc_run, smooth_fields

pytestmark = pytest.mark.gpu


def _ctx(b, lattice, bc, prec, sizes, seed):
    rng = np.random.default_rng(seed)
    params = [b.make_params(lattice, "srt", bc, prec, nx, ny, 0.7, 0.0, 0.03, 1.0) for nx, ny in sizes]
    n = sum(nx * ny for nx, ny in sizes)
    rho = 1.0 + 0.01 * rng.uniform(-1, 1, n)
    ux, uy = 0.02 * rng.uniform(-1, 1, n), 0.02 * rng.uniform(-1, 1, n)
    uy = uy if lattice == "d2q9" else None
    if len(sizes) == 1:
        return b.lbm_init(params[0], rho, ux, uy), n, (rho, ux, uy)
    return b.lbm_init_batch(params, rho, ux, uy), n, (rho, ux, uy)


CASES = [("d2q9", "periodic", [(5, 4)]),                       # one small slot
         ("d2q9", "periodic", [(300, 211)]),                   # one slot of fields, several of populations
         ("d2q9", "periodic", [(401, 503)]),                   # a few slots
         ("d2q9", "periodic", [(1201, 1003)]),                 # more pieces than slots
         ("d1q3", "periodic", [(700001, 1)]),
         ("d2q9", "periodic", [(3, 3), (700, 301), (64, 64), (9, 1200), (811, 650)]),
         ("d1q3", "periodic", [(k * 97 + 3, 1) for k in range(200)])]


@pytest.mark.parametrize("lattice,bc,sizes", CASES)
def test_fields_and_populations_come_back(lattice, bc, sizes):
    b = B()
    ctx, n, (rho, ux, uy) = _ctx(b, lattice, bc, "fp64", sizes, seed=3)
    q = 9 if lattice == "d2q9" else 3
    try:
        r, u, v = b.lbm_moments(ctx)
        # moments of an equilibrium: the fields to round-off of the sums
        assert np.max(np.abs(r - rho)) <= 1e-14 and np.max(np.abs(u - ux)) <= 1e-14
        if uy is not None:
            assert np.max(np.abs(v - uy)) <= 1e-14
        b.lbm_step(ctx, 3)
        f = b.lbm_get_populations(ctx, q)
        m = b.lbm_moments(ctx)
        b.lbm_step(ctx, 2)
        after = b.lbm_get_populations(ctx, q)
        assert not np.array_equal(f, after)
        for _ in range(2):  # restored state: the same fields, and the same two steps
            b.lbm_set_populations(ctx, f)
            assert np.array_equal(b.lbm_get_populations(ctx, q), f)
            assert all(np.array_equal(x, y) for x, y in zip(b.lbm_moments(ctx), m))
            b.lbm_step(ctx, 2)
            assert np.array_equal(b.lbm_get_populations(ctx, q), after)
    finally:
        b.lbm_free(ctx)


@pytest.mark.parametrize("bc", ["cavity", "box", "tube", "periodic"])
def test_pieces_that_cut_rows_match_the_oracle(bc):
    # 521 x 400 nodes: four pieces of fields, cut inside rows
    nx, ny = 521, 400
    rho, ux, uy = smooth_fields(nx, ny, seed=11)
    o = orc_run("d2q9", "minxent4", bc, nx, ny, 0.6, rho, ux, uy, steps=2, u_lid=0.05)
    b = B()
    ctx = b.lbm_init(b.make_params("d2q9", "minxent4", bc, "fp64", nx, ny, 0.6, 0.0, 0.05, 1.0), rho, ux, uy)
    try:
        b.lbm_step(ctx, 2)
        r, u, v = (a.reshape(ny, nx) for a in b.lbm_moments(ctx))
    finally:
        b.lbm_free(ctx)
    sl = (slice(1, ny - 1), slice(1, nx - 1))
    for g, name in ((r, "rho"), (u, "ux"), (v, "uy")):
        ref = o[name][sl]
        assert np.max(np.abs(g[sl] - ref)) <= 1e-12 * np.max(np.abs(ref)), name
