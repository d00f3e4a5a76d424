"""The batch shape with its lattices resident in LDS takes the nodes that
collide first and the walls last; its results are those of one step per launch,
bit for bit, for every boundary, for lattices of the smallest size, of whole
waves, and of more nodes than a workgroup has threads.  Needs an MI355X."""
import numpy as np
import pytest

from tests.gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["cavity", "box", "tube", "periodic"])
@pytest.mark.parametrize("coll,prec,large", [("minxent4", "fp64", (33, 33)), ("minxent2", "fp32", (47, 48)),
                                             ("srt", "fp16dev", (67, 66)), ("mrt", "fp64", (3, 370)),
                                             ("trt", "fp32_newton64", (700, 3))])
def test_lattices_in_lds_equal_single_steps(bc, coll, prec, large):
    b = B()
    sizes = [(3, 3), (3, 40), (40, 3), (10, 10), (17, 17), (18, 9), (31, 33), (4, 5)]
    limits = [-1, 0, 1, 7, -1, 12, 30, 5, -1]
    for shapes in (sizes, sizes + [large]):  # a thread for every node, and more nodes than threads
        params = [b.make_params("d2q9", coll, bc, prec, nx, ny, 0.55 + 0.01 * k, 0.0, 0.3, 1.0)
                  for k, (nx, ny) in enumerate(shapes)]
        fields = [smooth_fields(nx, ny, seed=500 + k) for k, (nx, ny) in enumerate(shapes)]
        rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
        for limited in (False, True):
            got = []
            for lds in (False, True):
                ctx = b.lbm_init_batch(params, rho, ux, uy)
                try:
                    names = [b.lbm_variant_name(ctx, v) for v in range(b.lbm_variant_count(ctx))]
                    b.lbm_set_variant(ctx, len(names) - 1 if lds else 0)
                    assert ("LDS" in names[-1]) and names[-1].startswith("batch persistent")
                    if limited:
                        b.lbm_set_batch_steps(ctx, limits[:len(shapes)])
                    b.lbm_step(ctx, 1)
                    b.lbm_step(ctx, 20)
                    got.append((b.lbm_get_populations(ctx, 9), b.lbm_status_batch(ctx, len(shapes))))
                finally:
                    b.lbm_free(ctx)
            assert np.array_equal(got[0][0], got[1][0], equal_nan=True), (len(shapes), limited)
            for u, v in zip(got[0][1], got[1][1]):
                assert {k: u[k] for k in ("unstable", "first_step", "first_node", "guarded")} == \
                       {k: v[k] for k in ("unstable", "first_step", "first_node", "guarded")}, (len(shapes), limited)
