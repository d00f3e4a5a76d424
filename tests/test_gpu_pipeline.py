"""Register-pipeline shapes: 2, 3 and 4 steps per launch with every row passed
from step to step in registers.

Every result must equal shape 0's (one step per launch) bit for bit, status
included.  Sizes sit at the edges of the tiles (62, 60 and 58 columns for 2, 3
and 4 steps; 8, 16 and 32 rows, or rows chosen by the size): one column more or
less than a tile, tiles that end ragged, lattices narrower than a wave and
shorter than the pipeline is deep, and lattices with tiles that touch no wall.
"""
import numpy as np
import pytest

from gpu_helpers import B, gpu_run, orc_run, smooth_fields

pytestmark = pytest.mark.gpu


def _shapes(b, coll):
    rho, ux, uy = smooth_fields(8, 8, seed=1)
    ctx = b.lbm_init(b.make_params("d2q9", coll, "box", "fp64", 8, 8, 0.6, 0.0, 0.0, 1.0), rho, ux, uy)
    try:
        vs = [v for v in range(b.lbm_variant_count(ctx)) if "register pipeline" in b.lbm_variant_name(ctx, v)]
        assert {b.lbm_variant_steps(ctx, v) for v in vs} == {2, 3, 4}
        return vs
    finally:
        b.lbm_free(ctx)


SIZES = [(3, 3), (4, 70), (58, 9), (61, 33), (63, 16), (121, 5), (250, 67)]


@pytest.mark.parametrize("bc", ["cavity", "periodic", "tube", "box"])
@pytest.mark.parametrize("coll,prec", [("minxent4", "fp64"), ("minxent4", "fp32_newton64"), ("minxent4", "fp32"),
                                       ("minxent4", "fp16dev"), ("minxent2", "fp16dev"), ("srt", "fp32"),
                                       ("trt", "fp64"), ("mrt", "fp32_newton64")])
def test_pipeline_shapes_equal_single_steps(bc, coll, prec):
    b = B()
    shapes = _shapes(b, coll)
    for k, (nx, ny) in enumerate(SIZES):
        rho, ux, uy = smooth_fields(nx, ny, seed=200 + k)
        kw = dict(u_lid=0.05, want_f=True)
        for steps, graph in ((13, 0), (11, 7)):  # remainders of 1, 2 and 3 steps, plain and in graphs
            ref = gpu_run("d2q9", coll, bc, prec, nx, ny, 0.6, rho, ux, uy, steps=steps, variant=0, **kw)
            for v in shapes:
                g = gpu_run("d2q9", coll, bc, prec, nx, ny, 0.6, rho, ux, uy, steps=steps, variant=v, graph=graph, **kw)
                assert np.array_equal(ref["f"], g["f"]), (nx, ny, steps, graph, v)
                assert ref["status"] == g["status"], (nx, ny, steps, graph, v)


@pytest.mark.parametrize("amp,seed,first", [(0.38, 3, 1), (0.36, 3, 2), (0.36, 0, 3)])
def test_pipeline_status_matches_oracle_wherever_the_event_falls(amp, seed, first):
    nx, ny = 40, 30
    rho, ux, uy = smooth_fields(nx, ny, seed=seed, amp=amp, rho_amp=0.2)
    o = orc_run("d2q9", "minxent4", "periodic", nx, ny, 0.501, rho, ux, uy, steps=9)
    assert o["unstable"] and o["first_step"] == first
    b = B()
    for v in _shapes(b, "minxent4"):
        for lead in (0, 1):
            ctx = b.lbm_init(b.make_params("d2q9", "minxent4", "periodic", "fp64", nx, ny, 0.501, 0.0, 0.0, 1.0),
                             rho, ux, uy)
            try:
                b.lbm_set_variant(ctx, v)
                b.lbm_step(ctx, lead)
                b.lbm_step(ctx, 9 - lead)
                s = b.lbm_status(ctx)
            finally:
                b.lbm_free(ctx)
            assert (s["first_step"], s["first_node"], s["guarded"]) == \
                (o["first_step"], o["first_node"], o["guarded"]), (v, lead)


@pytest.mark.parametrize("coll,prec,nx,ny", [("mrt", "fp64", 640, 600), ("minxent4", "fp64", 700, 600),
                                             ("srt", "fp32", 1100, 700)])
def test_contexts_and_noalloc_start_in_a_pipeline_beyond_the_windows(coll, prec, nx, ny):
    # sizes whose starting shape the estimate may take beyond the windows; the
    # result is the same whichever it takes
    import torch
    b = B()
    rho, ux, uy = smooth_fields(nx, ny, seed=5)
    ref = gpu_run("d2q9", coll, "cavity", prec, nx, ny, 0.6, rho, ux, uy, steps=7, u_lid=0.05, variant=0)
    g = gpu_run("d2q9", coll, "cavity", prec, nx, ny, 0.6, rho, ux, uy, steps=7, u_lid=0.05)
    for name in ("rho", "ux", "uy"):
        assert np.array_equal(ref[name], g[name]), name
    p = b.make_params("d2q9", coll, "cavity", prec, nx, ny, 0.6, 0.0, 0.05, 1.0)
    t = [torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).cuda() for a in (rho, ux, uy)]
    out = [torch.empty_like(a) for a in t]
    assert b.lbm_run_noalloc(p, *t, 7, *out) == ref["status"]
    for name, a in zip(("rho", "ux", "uy"), out):
        assert np.array_equal(ref[name].reshape(-1), a.cpu().numpy()), name


@pytest.mark.parametrize("bc", ["cavity", "periodic", "box"])
@pytest.mark.parametrize("coll,prec", [("minxent4", "fp64"), ("minxent4", "fp32"), ("minxent4", "fp16dev"),
                                       ("minxent2", "fp32_newton64"), ("srt", "fp64"), ("mrt", "fp16dev")])
def test_batch_pipelines_equal_single_steps(bc, coll, prec):
    # widths and heights around the tiles; step limits before, inside and after
    # launches of 2, 3 and 4 steps; plain launches and graphs
    b = B()
    sizes = [(3, 3), (58, 8), (60, 33), (62, 16), (63, 17), (125, 9), (7, 150), (250, 70), (64, 64)]
    limits = [-1, 0, 1, 2, 3, 5, 11, -1, 8]
    params = [b.make_params("d2q9", coll, bc, prec, nx, ny, 0.58 + 0.01 * k, 0.0, 0.05, 1.0)
              for k, (nx, ny) in enumerate(sizes)]
    fields = [smooth_fields(nx, ny, seed=300 + k) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))

    def run(v, steps, graph, limited):
        ctx = b.lbm_init_batch(params, rho, ux, uy)
        try:
            if v is None:
                return [v for v in range(b.lbm_variant_count(ctx)) if "register pipeline" in b.lbm_variant_name(ctx, v)]
            b.lbm_set_variant(ctx, v)
            if limited:
                b.lbm_set_batch_steps(ctx, limits)
            if graph:
                b.lbm_set_graph_chunk(ctx, graph)
            for n in steps:
                b.lbm_step(ctx, n)
            return b.lbm_get_populations(ctx, 9), b.lbm_status_batch(ctx, len(sizes))
        finally:
            b.lbm_free(ctx)

    shapes = run(None, (), 0, False)
    assert len(shapes) == 7
    for steps, graph, limited in (((12,), 0, False), ((1, 10), 0, True), ((14,), 5, True)):
        ref = run(0, steps, 0, limited)
        for v in shapes:
            got = run(v, steps, graph, limited)
            assert np.array_equal(ref[0], got[0]), (v, steps, graph, limited)
            assert ref[1] == got[1], (v, steps, graph, limited)


def test_large_batches_start_in_a_pipeline():
    b = B()
    sizes = [(300, 300)] * 30 + [(40, 500)] * 4
    params = [b.make_params("d2q9", "minxent4", "cavity", "fp32", nx, ny, 0.6, 0.0, 0.05, 1.0) for nx, ny in sizes]
    fields = [smooth_fields(nx, ny, seed=k) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    got = []
    for v in (0, None):
        ctx = b.lbm_init_batch(params, rho, ux, uy)
        try:
            if v is not None:
                b.lbm_set_variant(ctx, v)
            b.lbm_step(ctx, 7)
            got.append((b.lbm_get_populations(ctx, 9), b.lbm_status_batch(ctx, len(sizes))))
        finally:
            b.lbm_free(ctx)
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]


@pytest.mark.parametrize("coll,prec,bc,nx,ny", [("minxent4", "fp16dev", "cavity", 2500, 1301),
                                                ("minxent4", "fp16dev", "periodic", 2480, 2600),
                                                ("minxent2", "fp64", "box", 2501, 1111),
                                                ("minxent4", "fp32_newton64", "tube", 3000, 1603)])
def test_tiles_of_two_heights_equal_single_steps(coll, prec, bc, nx, ny):
    # more tiles than the chip holds at once: the last ones have half the rows
    b = B()
    rho, ux, uy = smooth_fields(nx, ny, seed=17)
    p = b.make_params("d2q9", coll, bc, prec, nx, ny, 0.6, 0.0, 0.05 if bc == "cavity" else 0.0, 1.0)
    ctx = b.lbm_init(p, rho, ux, uy)
    try:
        f0 = b.lbm_get_populations(ctx, 9)
        names = [b.lbm_variant_name(ctx, v) for v in range(b.lbm_variant_count(ctx))]
        ref = None
        for v in [0] + [v for v, nm in enumerate(names) if "register pipeline" in nm]:
            b.lbm_set_variant(ctx, v)
            b.lbm_set_populations(ctx, f0)
            b.lbm_reset_status(ctx)
            b.lbm_step(ctx, 13)
            got = (b.lbm_get_populations(ctx, 9), b.lbm_status(ctx)["flags"])
            ref = ref or got
            assert np.array_equal(ref[0], got[0]) and ref[1] == got[1], names[v]
    finally:
        b.lbm_free(ctx)
