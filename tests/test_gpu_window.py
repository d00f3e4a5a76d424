"""Shapes that take several steps per launch in on-chip windows, and the calls
they now serve (a new context, the no-allocation call).

Every result must equal shape 0's (one step per launch) bit for bit, status
included: both do the same arithmetic on every node and round to the storage
type after every step.  Sizes sit at the edges: the smallest lattice, axes a
tile covers whole, windows longer than a wrapping axis, tiles that end ragged,
and windows cut at a wall several nodes away.
"""
import numpy as np
import pytest

from gpu_helpers import B, gpu_run, orc_run, smooth_fields

pytestmark = pytest.mark.gpu


def _window_shapes(b, coll, bc, prec, nx, ny, rho, ux, uy):
    ctx = b.lbm_init(b.make_params("d2q9", coll, bc, prec, nx, ny, 0.6, 0.0, 0.05, 1.0), rho, ux, uy)
    try:
        return [v for v in range(b.lbm_variant_count(ctx)) if "window" in b.lbm_variant_name(ctx, v)]
    finally:
        b.lbm_free(ctx)


SIZES = [(3, 3), (5, 40), (33, 3), (17, 17), (31, 29), (70, 45), (130, 9), (257, 66)]


@pytest.mark.parametrize("bc", ["cavity", "periodic", "tube", "box"])
@pytest.mark.parametrize("coll,prec", [("minxent4", "fp64"), ("minxent4", "fp32_newton64"), ("minxent4", "fp16dev"),
                                       ("minxent2", "fp32"), ("srt", "fp64"), ("trt", "fp16dev"), ("mrt", "fp32")])
def test_window_shapes_equal_single_steps(bc, coll, prec):
    b = B()
    for k, (nx, ny) in enumerate(SIZES):
        rho, ux, uy = smooth_fields(nx, ny, seed=100 + k)
        kw = dict(u_lid=0.05, want_f=True)
        for steps, graph in ((37, 0), (21, 9)):
            ref = gpu_run("d2q9", coll, bc, prec, nx, ny, 0.6, rho, ux, uy, steps=steps, variant=0, **kw)
            shapes = _window_shapes(b, coll, bc, prec, nx, ny, rho, ux, uy)
            assert shapes
            for v in shapes + [None]:  # None: the shape the context starts with
                g = gpu_run("d2q9", coll, bc, prec, nx, ny, 0.6, rho, ux, uy, steps=steps, variant=v, graph=graph, **kw)
                assert np.array_equal(ref["f"], g["f"], equal_nan=True), (nx, ny, steps, graph, v)
                assert ref["status"] == g["status"], (nx, ny, steps, graph, v)


@pytest.mark.parametrize("amp,seed,first", [(0.38, 3, 1), (0.36, 3, 2), (0.36, 0, 3)])
def test_window_status_matches_oracle_wherever_the_event_falls(amp, seed, first):
    # a periodic lattice whose first unstable event falls on step 1, 2 or 3:
    # inside a launch, in several tiles' windows at once
    nx, ny = 40, 30
    rho, ux, uy = smooth_fields(nx, ny, seed=seed, amp=amp, rho_amp=0.2)
    o = orc_run("d2q9", "minxent4", "periodic", nx, ny, 0.501, rho, ux, uy, steps=9)
    assert o["unstable"] and o["first_step"] == first
    b = B()
    for v in _window_shapes(b, "minxent4", "periodic", "fp64", nx, ny, rho, ux, uy):
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
            assert s["unstable"]
            assert (s["first_step"], s["first_node"], s["guarded"]) == \
                (o["first_step"], o["first_node"], o["guarded"]), (v, lead)


@pytest.mark.parametrize("prec", ["fp64", "fp32_newton64", "fp32", "fp16dev"])
def test_noalloc_equals_single_steps_in_its_new_shapes(prec):
    import torch
    b = B()
    rng = np.random.default_rng(7)
    for coll in ("minxent4", "minxent2", "srt", "trt", "mrt"):
        for bc in ("cavity", "periodic", "tube", "box"):
            nx, ny = int(rng.integers(3, 180)), int(rng.integers(3, 120))
            steps = int(rng.integers(1, 40))
            rho, ux, uy = smooth_fields(nx, ny, seed=int(rng.integers(1000)))
            ref = gpu_run("d2q9", coll, bc, prec, nx, ny, 0.6, rho, ux, uy, steps=steps, u_lid=0.05, variant=0)
            t = [torch.from_numpy(np.ascontiguousarray(a).reshape(-1)).cuda() for a in (rho, ux, uy)]
            out = [torch.empty_like(a) for a in t]
            st = b.lbm_run_noalloc(b.make_params("d2q9", coll, bc, prec, nx, ny, 0.6, 0.0, 0.05, 1.0), *t, steps, *out)
            for name, a in zip(("rho", "ux", "uy"), out):
                assert np.array_equal(ref[name].reshape(-1), a.cpu().numpy()), (coll, bc, nx, ny, steps, name)
            assert st == ref["status"], (coll, bc, nx, ny, steps)
