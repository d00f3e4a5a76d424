"""D1Q3 shapes that keep the nodes in registers for up to 32 steps per launch,
and the calls that start in them (contexts, the no-allocation call).

Every result must equal shape 0's (one step per launch) bit for bit, status
included.  Sizes sit at the edges of what a wave owns (64, 192 and 448 nodes
with 2, 4 and 8 per lane) and of its window (128, 256, 512): one node more or
less, lattices inside one window, wrapping lattices shorter than it; step
counts below, at and above a launch's.
"""
import numpy as np
import pytest

from gpu_helpers import B, gpu_run

pytestmark = pytest.mark.gpu


def _register_shapes(b, ctx):
    vs = [v for v in range(b.lbm_variant_count(ctx)) if "nodes in registers" in b.lbm_variant_name(ctx, v)]
    assert len(vs) == 3 and all(b.lbm_variant_steps(ctx, v) == 32 for v in vs)
    return vs


def _fields(n, seed):
    rng = np.random.default_rng(seed)
    return 1.0 + 0.2 * rng.uniform(-1, 1, n), 0.1 * rng.uniform(-1, 1, n)


@pytest.mark.parametrize("bc", ["tube", "periodic", "box"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_newton64", "fp32", "fp16dev"])
def test_register_shapes_equal_single_steps(bc, prec):
    b = B()
    for n in (3, 31, 63, 64, 65, 127, 128, 129, 192, 193, 255, 257, 447, 449, 511, 513, 1000, 2049):
        rho, ux = _fields(n, n)
        ctx = b.lbm_init(b.make_params("d1q3", "srt", bc, prec, n, 1, 0.6), rho, ux)
        shapes = _register_shapes(b, ctx)
        b.lbm_free(ctx)
        for steps, graph in ((1, 0), (31, 0), (33, 0), (70, 37)):
            ref = gpu_run("d1q3", "srt", bc, prec, n, 1, 0.6, rho, ux, steps=steps, variant=0, want_f=True)
            for v in shapes + [None]:  # None: the shape the context starts with
                g = gpu_run("d1q3", "srt", bc, prec, n, 1, 0.6, rho, ux, steps=steps, variant=v, graph=graph, want_f=True)
                assert np.array_equal(ref["f"], g["f"]), (n, steps, v)
                assert ref["status"] == g["status"], (n, steps, v)


@pytest.mark.parametrize("prec", ["fp64", "fp16dev"])
def test_register_shapes_in_batches_with_limits_inside_a_launch(prec):
    b = B()
    sizes = [3, 64, 65, 448, 449, 1300, 9, 4000]
    limits = [-1, 5, 40, 0, 33, 70, 1, 64]
    params = [b.make_params("d1q3", "srt", "tube", prec, n, 1, 0.55 + 0.01 * k) for k, n in enumerate(sizes)]
    fields = [_fields(n, 50 + n) for n in sizes]
    rho, ux = (np.concatenate(a) for a in zip(*fields))
    got = []
    ctx = b.lbm_init_batch(params, rho, ux)
    shapes = _register_shapes(b, ctx)
    b.lbm_free(ctx)
    for v in [0] + shapes + [None]:
        ctx = b.lbm_init_batch(params, rho, ux)
        try:
            if v is not None:
                b.lbm_set_variant(ctx, v)
            b.lbm_set_batch_steps(ctx, limits)
            b.lbm_step(ctx, 3)
            b.lbm_step(ctx, 70)
            got.append((b.lbm_get_populations(ctx, 3), b.lbm_status_batch(ctx, len(sizes))))
        finally:
            b.lbm_free(ctx)
    for f, st in got[1:]:
        assert np.array_equal(f, got[0][0]) and st == got[0][1]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16dev"])
def test_noalloc_tubes_equal_single_steps(prec):
    import torch
    b = B()
    for n, steps in ((5, 3), (800, 100), (5000, 37)):
        rho, ux = _fields(n, n)
        ref = gpu_run("d1q3", "srt", "tube", prec, n, 1, 0.6, rho, ux, steps=steps, variant=0)
        t = [torch.from_numpy(a).cuda() for a in (rho, ux)]
        out = [torch.empty_like(t[0]) for _ in range(2)]
        st = b.lbm_run_noalloc(b.make_params("d1q3", "srt", "tube", prec, n, 1, 0.6), t[0], t[1], None, steps, out[0],
                               out[1], None)
        assert st == ref["status"]
        assert np.array_equal(out[0].cpu().numpy(), ref["rho"]) and np.array_equal(out[1].cpu().numpy(), ref["ux"])
