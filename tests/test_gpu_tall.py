"""A lattice of more rows than a launch grid has: every shape steps it as shape
0 does, bit for bit, and it can be tuned.  Needs an MI355X."""
import numpy as np
import pytest

from gpu_helpers import B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coll,bc", [("srt", "box")])
def test_tall_lattice_in_every_shape_and_tuned(coll, bc):
    b = B()
    nx, ny = 3, 1900000  # beyond 28 rows times 65535 blocks
    y = np.arange(ny)
    rho = np.repeat(1.0 + 0.01 * np.cos(0.37 * y), nx)
    ux, uy = np.repeat(0.02 * np.sin(0.11 * y), nx), np.repeat(0.02 * np.cos(0.23 * y), nx)
    c = b.lbm_init(b.make_params("d2q9", coll, bc, "fp16dev", nx, ny, 0.6), rho, ux, uy)
    try:
        f0 = b.lbm_get_populations(c, 9)
        ref = None
        for v in range(b.lbm_variant_count(c)):
            print(b.lbm_variant_name(c, v), flush=True)
            b.lbm_set_variant(c, v)
            b.lbm_set_populations(c, f0)
            b.lbm_step(c, 5)
            m = b.lbm_moments(c)
            ref = ref or m
            assert all(np.array_equal(p, q) for p, q in zip(ref, m)), b.lbm_variant_name(c, v)
        b.lbm_set_populations(c, f0)
        assert 0 <= b.lbm_autotune(c, None) < b.lbm_variant_count(c)
        b.lbm_step(c, 5)
        assert all(np.array_equal(p, q) for p, q in zip(ref, b.lbm_moments(c)))
    finally:
        b.lbm_free(c)
