"""Two host threads, each with a context of its own on its own stream, step and
read back at the same time, and free and make contexts while the other reads:
the one that finds the shared read-back slots in use takes its own, and the
slots come and go with the contexts.  What each reads is what it reads alone,
bit for bit.  Needs an MI355X."""
import threading

import numpy as np
import pytest

from gpu_helpers import B, smooth_fields

pytestmark = pytest.mark.gpu

# more values than the slots hold at once (18 MiB), and a batch
SIZES = [[(1311, 1203)], [(700, 801), (64, 64), (900, 900)]]


def _work(b, sizes, stream):
    params = [b.make_params("d2q9", "srt", "periodic", "fp32", nx, ny, 0.7) for nx, ny in sizes]
    fields = [smooth_fields(nx, ny, seed=k) for k, (nx, ny) in enumerate(sizes)]
    rho, ux, uy = (np.concatenate([f[i].reshape(-1) for f in fields]) for i in range(3))
    out = []
    for _ in range(3):
        c = b.lbm_init(params[0], rho, ux, uy, stream=stream) if len(sizes) == 1 else \
            b.lbm_init_batch(params, rho, ux, uy, stream=stream)
        try:
            for steps in (3, 4):
                b.lbm_step(c, steps)
                out += [*b.lbm_moments(c), b.lbm_get_populations(c, 9)]
        finally:
            b.lbm_free(c)
    return out


def test_two_threads_read_back_at_once():
    import torch
    b = B()
    streams = [torch.cuda.Stream() for _ in SIZES]
    alone = [_work(b, s, t) for s, t in zip(SIZES, streams)]
    got, errors = [None] * len(SIZES), []

    def body(k):
        try:
            torch.cuda.set_device(0)
            start.wait(timeout=30)
            got[k] = _work(b, SIZES[k], streams[k])
        except BaseException as e:  # noqa: BLE001 (reported by the test)
            errors.append(e)

    start = threading.Barrier(len(SIZES))
    threads = [threading.Thread(target=body, args=(k,)) for k in range(len(SIZES))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=90)
    assert not errors and all(g is not None for g in got), errors
    for a, g in zip(alone, got):
        assert len(a) == len(g) and all(np.array_equal(x, y) for x, y in zip(a, g))
