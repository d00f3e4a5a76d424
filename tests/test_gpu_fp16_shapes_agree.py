"""FP16 deviations of populations far from the reference: every launch shape
stores the same bits.

Near rest v*scale - ref*scale is exact in float and a second rounding changes
nothing; a population of less than half or more than twice its reference is where
a shape that rounds to float before it rounds to binary16 shows.  Flows of 0.45
lattice units and a lid of 0.4 hold many.  Needs an MI355X."""
import numpy as np
import pytest

from gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu


def _all_shapes(b, ctx, q, f0, steps):
    ref = None
    for v in range(b.lbm_variant_count(ctx)):
        b.lbm_set_variant(ctx, v)
        b.lbm_set_populations(ctx, f0)
        b.lbm_step(ctx, steps)
        f = b.lbm_get_populations(ctx, q)
        ref = f if ref is None else ref
        d = ~((f == ref) | (np.isnan(f) & np.isnan(ref)))
        assert not d.any(), (b.lbm_variant_name(ctx, v), steps, int(d.sum()), f[d][:3], ref[d][:3])


@pytest.mark.parametrize("bc", ["cavity", "tube", "periodic", "box"])
@pytest.mark.parametrize("coll", ["minxent4", "minxent2", "srt", "trt", "mrt"])
@pytest.mark.parametrize("steps", [1, 2, 3, 6])
def test_single_lattices(coll, bc, steps):
    b = B()
    nx, ny = 301, 231
    c = b.lbm_init(b.make_params("d2q9", coll, bc, "fp16dev", nx, ny, 0.8, 0.0, 0.4, 1.0),
                   *smooth_fields(nx, ny, seed=5, amp=0.45, rho_amp=0.3))
    try:
        _all_shapes(b, c, 9, b.lbm_get_populations(c, 9), steps)
    finally:
        b.lbm_free(c)


@pytest.mark.parametrize("coll,bc", [("minxent4", "cavity"), ("srt", "tube"), ("mrt", "box")])
def test_batches(coll, bc):
    b = B()
    sizes = [(17, 17), (65, 40), (63, 33), (41, 90)]
    fields = [smooth_fields(nx, ny, seed=40 + k, amp=0.45, rho_amp=0.3) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    c = b.lbm_init_batch([b.make_params("d2q9", coll, bc, "fp16dev", nx, ny, 0.8, 0.0, 0.4, 1.0) for nx, ny in sizes],
                         rho, ux, uy)
    try:
        f0 = b.lbm_get_populations(c, 9)
        for steps in (1, 2, 3, 6):
            _all_shapes(b, c, 9, f0, steps)
    finally:
        b.lbm_free(c)


def test_tubes():
    b = B()
    n = 20000
    x = np.arange(n)
    c = b.lbm_init(b.make_params("d1q3", "srt", "tube", "fp16dev", n, 1, 0.7),
                   1.0 + 0.8 * np.sin(0.01 * x), 0.45 * np.cos(0.03 * x))
    try:
        f0 = b.lbm_get_populations(c, 3)
        for steps in (1, 2, 5, 33):
            _all_shapes(b, c, 3, f0, steps)
    finally:
        b.lbm_free(c)
