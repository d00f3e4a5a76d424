"""D1Q3 launches of few steps in the shapes that keep the nodes in registers:
their windows start on a whole vector, up to seven nodes before the first node
that the steps need.  Step counts around the vectors of each storage type (2, 4
and 8 values), sizes around what a wave owns; equal to shape 0 bit for bit.
Needs an MI355X."""
import numpy as np
import pytest

from gpu_helpers import B, gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["tube", "periodic"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_newton64", "fp32", "fp16dev"])
def test_few_steps_equal_single_steps(bc, prec):
    b = B()
    for n in (5, 65, 129, 193, 449, 520, 1025, 1409):
        rng = np.random.default_rng(n)
        rho, ux = 1.0 + 0.2 * rng.uniform(-1, 1, n), 0.1 * rng.uniform(-1, 1, n)
        c = b.lbm_init(b.make_params("d1q3", "srt", bc, prec, n, 1, 0.6), rho, ux)
        shapes = [v for v in range(b.lbm_variant_count(c)) if "nodes in registers" in b.lbm_variant_name(c, v)]
        b.lbm_free(c)
        for steps in (1, 2, 3, 4, 5, 7, 8, 9, 15, 17, 25, 32):
            ref = gpu_run("d1q3", "srt", bc, prec, n, 1, 0.6, rho, ux, steps=steps, variant=0, want_f=True)
            for v in shapes:
                g = gpu_run("d1q3", "srt", bc, prec, n, 1, 0.6, rho, ux, steps=steps, variant=v, want_f=True)
                assert np.array_equal(ref["f"], g["f"]) and ref["status"] == g["status"], (n, steps, v)
