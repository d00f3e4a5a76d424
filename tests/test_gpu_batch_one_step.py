"""Batches stepped one at a time, and with step counts that leave a last step, in
every shape that then takes shape 0's kernel and tiles: equal to shape 0 bit for
bit, step limits and status records included.  Needs an MI355X."""
import numpy as np
import pytest

from gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,coll,prec,bc", [("d2q9", "minxent4", "fp64", "cavity"),
                                                  ("d2q9", "minxent4", "fp16dev", "periodic"),
                                                  ("d2q9", "mrt", "fp32", "box"), ("d1q3", "srt", "fp64", "tube"),
                                                  ("d1q3", "srt", "fp16dev", "periodic")])
def test_single_steps_between_launches_of_several(lattice, coll, prec, bc):
    b = B()
    q = 9 if lattice == "d2q9" else 3
    sizes = [(3, 3), (62, 17), (257, 5), (7, 150), (64, 64), (130, 70)]
    sizes = sizes if q == 9 else [(nx * ny, 1) for nx, ny in sizes]
    limits = [-1, 0, 1, 4, 6, 9]
    params = [b.make_params(lattice, coll, bc, prec, nx, ny, 0.56 + 0.01 * k, 0.0, 0.05, 1.0)
              for k, (nx, ny) in enumerate(sizes)]
    fields = [smooth_fields(nx, ny, seed=600 + k) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    ref = {}
    word = "register pipeline" if q == 9 else "nodes in registers"
    ctx = b.lbm_init_batch(params, rho, ux, uy)
    names = [b.lbm_variant_name(ctx, v) for v in range(b.lbm_variant_count(ctx))]
    b.lbm_free(ctx)
    shapes = [v for v, name in enumerate(names) if word in name]
    assert shapes
    for v in [0] + shapes:
        for steps, graph in (((1, 1, 1, 5, 1), 0), ((9,), 3), ((1, 7, 1), 4)):
            ctx = b.lbm_init_batch(params, rho, ux, uy)
            try:
                b.lbm_set_variant(ctx, v)
                b.lbm_set_batch_steps(ctx, limits)
                if graph:
                    b.lbm_set_graph_chunk(ctx, graph)
                for n in steps:
                    b.lbm_step(ctx, n)
                got = b.lbm_get_populations(ctx, q), b.lbm_status_batch(ctx, len(sizes))
            finally:
                b.lbm_free(ctx)
            want = ref.setdefault(steps, got)
            assert np.array_equal(want[0], got[0]) and want[1] == got[1], (names[v], steps, graph)
