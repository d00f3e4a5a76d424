"""The tuner leaves the state as it was, also where it times a large state from
one buffer to the other and back (32 MiB and more).  Needs an MI355X."""
import numpy as np
import pytest

from tests.gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,nx,ny,prec", [("d2q9", 1365, 1366, "fp16dev"),  # 33.6 MB, just above
                                                ("d2q9", 680, 680, "fp64"),  # 33.3 MB, just below
                                                ("d2q9", 1025, 1003, "fp64"),
                                                ("d1q3", 3000001, 1, "fp64")])
def test_tuning_leaves_the_state(lattice, nx, ny, prec):
    b = B()
    q, coll, bc = (9, "minxent4", "cavity") if lattice == "d2q9" else (3, "srt", "tube")
    rho, ux, uy = smooth_fields(nx, ny, seed=71)
    if q == 3:
        uy = np.zeros_like(ux)
    p = b.make_params(lattice, coll, bc, prec, nx, ny, 0.6, 0.0, 0.05 if q == 9 else 0.0, 1.0)
    got = []
    for tune in (False, True):
        ctx = b.lbm_init(p, rho, ux, uy)
        try:
            b.lbm_set_variant(ctx, 0)
            b.lbm_step(ctx, 3)
            if tune:
                f0 = b.lbm_get_populations(ctx, q)
                assert 0 <= b.lbm_autotune(ctx, None) < b.lbm_variant_count(ctx)
                assert np.array_equal(f0, b.lbm_get_populations(ctx, q))
            b.lbm_step(ctx, 9)
            got.append((b.lbm_get_populations(ctx, q), b.lbm_status(ctx)))
        finally:
            b.lbm_free(ctx)
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]
