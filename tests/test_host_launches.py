"""Which kernels a call enqueues, and what it does when the runtime refuses
something, seen on the CPU through a runtime that only records (recorded.py).
Nothing here runs on a device."""
import os
import subprocess

import pytest

import recorded


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = recorded.build_recorder(tmp_path_factory.mktemp("recorder"))
    return lambda body, **kw: recorded.run(lib, body, **kw)


def test_recorder_sees_the_launches_of_a_run(run):
    run("""
    c = single("d2q9", "minxent4", "cavity", "fp64", 300, 7)
    ks = kernels()
    assert [k[0] for k in ks] == ["k_clear_status", "k_init"], ks
    B.lbm_set_variant(c, 0)
    B.lbm_step(c, 3)
    assert kernels() == [("k_d2q9", 2, 7, 256)] * 3
    B.lbm_moments(c)
    assert kernels() == [("k_gather", 9, 1, 256)]
    B.lbm_free(c)
    assert rec.rec_blocks() == 0
    """)


def test_store_offsets_of_planes_beyond_4_gib(tmp_path):
    # the offset the window kernel stores at, evaluated by the host compiler:
    # corners of the largest lattices the library takes (rows of whole 128-byte
    # lines, fewer than 2^31 elements), against Python's integers
    cases = [(nx, ny, (nx * e + 127) // 128 * 128 // e, e)
             for e, nx, ny in ((8, 24000, 24000), (8, 33, 11_300_000), (4, 32767, 32767), (2, 3, (1 << 25) - 1), (8, 9, 7))]
    src = tmp_path / "offsets.cpp"
    src.write_text('#include <cstdio>\n#include "kernels.hpp"\nint main() {\n' + "".join(
        'std::printf("%%lld\\n", (long long)lbm::plane_bytes(%d, %d, %d, %d));\n' % (nx - 1, ny - 1, p, e)
        for nx, ny, p, e in cases) + "}\n")
    csrc = os.path.join(recorded.ROOT, "paper_1801_03863_amd", "csrc")
    exe = str(tmp_path / "offsets")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + csrc, str(src), "-o", exe],
                   check=True)
    got = [int(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    assert got == [((ny - 1) * p + nx - 1) * e for nx, ny, p, e in cases]
    assert max(got) >= 1 << 32


@pytest.mark.parametrize("coll", ["minxent4", "mrt"])
def test_one_step_of_a_window_shape_is_shape_0s(run, coll):
    # small lattices, where windows of several steps exist, and lattices too
    # tall or too large for one
    run("""
    for prec, nx, ny in (("fp64", 17, 17), ("fp32", 257, 400), ("fp64", 3, 2000000), ("fp16dev", 64, 1900000),
                         ("fp64", 24000, 24000)):
        c = single("d2q9", %r, "cavity", prec, nx, ny)
        B.lbm_set_variant(c, 0)
        kernels()
        B.lbm_step(c, 1)
        one = kernels()
        assert [k[0] for k in one] == ["k_d2q9"]
        found = shapes(c, "window")
        assert found
        for v in found:
            B.lbm_set_variant(c, v)
            B.lbm_step(c, 1)
            assert kernels() == one, (nx, ny, v)
            n = B.lbm_variant_steps(c, v)
            assert (n > 1) == (nx * ny < 200000), (nx, ny, n)
            B.lbm_step(c, 2 * n + 1)
            ks = kernels()
            assert [k[0] for k in ks] == ["k_d2q9_win" if n > 1 else "k_d2q9"] * 2 + ["k_d2q9"]
        B.lbm_free(c)
    """ % coll)


@pytest.mark.parametrize("prec,nx,ny", [("fp64", 3, 2000000), ("fp16dev", 64, 1900000)])
def test_tall_lattices_can_be_tuned(run, prec, nx, ny):
    run("""
    c = single("d2q9", "srt", "box", %r, %d, %d)
    assert 0 <= B.lbm_autotune(c, None) < B.lbm_variant_count(c)
    B.lbm_step(c, 5)
    B.lbm_free(c)
    """ % (prec, nx, ny))


@pytest.mark.parametrize("refused", [0, 150, 5000])
def test_a_tuning_that_fails_leaves_the_shape(run, refused):
    # `refused` launches into the tuning the runtime refuses one: the call fails,
    # and the context goes on in the shape it had
    run("""
    for start in (None, 7):
        c = single("d2q9", "minxent4", "cavity", "fp64", 700, 900)  # planes with a pad, states set aside
        if start is not None:
            B.lbm_set_variant(c, start)
        kernels()
        B.lbm_step(c, 24)
        before, blocks = kernels(), rec.rec_blocks()
        rec.rec_refuse(%d, 0, 0, 0)
        try:
            B.lbm_autotune(c, None)
        except B.LbmError as e:
            assert e.code == B.LBM_EHIP and "recorded error" in str(e)
        else:
            raise AssertionError("tuned")
        rec.rec_refuse(-1, 0, 0, 0)
        kernels()
        B.lbm_step(c, 24)
        assert kernels() == before
        assert rec.rec_blocks() == blocks and rec.rec_events() == 0
        B.lbm_free(c)
    """ % refused)


@pytest.mark.parametrize("lattice,prec", [("d2q9", "fp32"), ("d1q3", "fp64")])
def test_a_shape_whose_tiles_find_no_memory_is_not_set(run, lattice, prec):
    run("""
    lattice = %r
    c = batch(lattice, "minxent4" if lattice == "d2q9" else "srt", "periodic", %r,
              [(300, 200 if lattice == "d2q9" else 1), (70, 90 if lattice == "d2q9" else 1)])
    for start in range(B.lbm_variant_count(c)):
        B.lbm_set_variant(c, start)
        kernels()
        B.lbm_step(c, 12)
        before, blocks = kernels(), rec.rec_blocks()
        for v in range(B.lbm_variant_count(c)):
            rec.rec_refuse(-1, 0, 0, 1)
            try:
                B.lbm_set_variant(c, v)
            except B.LbmError as e:
                assert e.code == B.LBM_EHIP
                rec.rec_refuse(-1, 0, 0, 0)
                B.lbm_step(c, 12)
                assert kernels() == before, (start, v)
            else:  # the same tiles: nothing to allocate
                rec.rec_refuse(-1, 0, 0, 0)
                B.lbm_set_variant(c, start)
                kernels()
        assert rec.rec_blocks() == blocks
    B.lbm_free(c)
    assert rec.rec_blocks() == 0
    """ % (lattice, prec))


@pytest.mark.parametrize("lattice,sizes", [("d2q9", [(40, 30)]), ("d2q9", [(1201, 1003)]),
                                           ("d2q9", [(9, 7), (700, 301), (64, 64)]), ("d1q3", [(900001, 1)])])
@pytest.mark.parametrize("refused", ["pinned", "threads", "pinned and device"])
def test_reading_back_without_pinned_memory_or_threads(run, lattice, sizes, refused):
    # neither is needed: the call reads back some other way.  Without device
    # memory for that either it fails, and leaves nothing behind for the next.
    run("""
    lattice, sizes, refused = %r, %r, %r
    prec, coll = "fp32", "srt"
    if len(sizes) == 1:
        c = single(lattice, coll, "periodic", prec, *sizes[0])
    else:
        c = batch(lattice, coll, "periodic", prec, sizes)
    blocks = rec.rec_blocks()
    rec.rec_refuse(-1, "pinned" in refused, "threads" in refused, "device" in refused)
    for read in (lambda: B.lbm_moments(c), lambda: B.lbm_get_populations(c, 9 if lattice == "d2q9" else 3)):
        try:
            read()
        except B.LbmError as e:
            assert refused == "pinned and device" and e.code == B.LBM_EHIP, e
        else:
            assert refused != "pinned and device"
        B.lbm_step(c, 3)
    rec.rec_refuse(-1, 0, 0, 0)
    assert rec.rec_events() == 0 and ("pinned" not in refused or rec.rec_blocks() == blocks)
    B.lbm_free(c)
    assert rec.rec_blocks() == 0
    """ % (lattice, sizes, refused))


@pytest.mark.parametrize("coll,prec,sizes,kernel", [
    # tiles nearly empty, or a state the caches hold: one step per launch
    ("minxent4", "fp64", [(4, 800)] * 41, "k_d2q9_batch"),
    ("minxent4", "fp64", [(17, 17)] * 1100, "k_d2q9_batch"),
    ("minxent4", "fp16dev", [(64, 64)] * 600, "k_d2q9_batch"),
    ("mrt", "fp64", [(8, 512)] * 1000, "k_d2q9_batch"),
    ("srt", "fp32", [(180, 180)] * 8, "k_d2q9_batch"),
    ("minxent4", "fp64", [(3, 3)], "k_d2q9_batch"),
    # full tiles of lattices that fill the chip: a register pipeline
    ("minxent4", "fp32", [(300, 300)] * 30 + [(40, 500)] * 4, "k_d2q9_rp"),
    ("minxent4", "fp64", [(32 + 15 * k // 4, 32 + 15 * k // 4) for k in range(128)], "k_d2q9_rp"),
    ("minxent2", "fp32_newton64", [(300, 300)] * 60, "k_d2q9_rp"),
    ("srt", "fp64", [(1000, 33)] * 150, "k_d2q9_rp")])
def test_starting_shape_of_a_batch_goes_by_its_tiles(run, coll, prec, sizes, kernel):
    run("""
    c = batch("d2q9", %r, "cavity", %r, %r)
    kernels()
    B.lbm_step(c, 2)
    ks = kernels()
    assert {k[0] for k in ks} == {%r}, ks
    B.lbm_free(c)
    """ % (coll, prec, sizes, kernel))


def test_one_step_of_a_register_shape_is_shape_0s(run):
    run("""
    for prec, n in (("fp64", 30), ("fp32", 50000), ("fp16dev", 1000003), ("fp64", 10000000)):
        c = single("d1q3", "srt", "tube", prec, n, 1)
        kernels()
        B.lbm_step(c, 33)
        assert [k[0] for k in kernels()] == ["k_d1q3_regs", "k_d1q3"], n
        for v in shapes(c, "nodes in registers"):
            B.lbm_set_variant(c, v)
            B.lbm_step(c, 1)
            assert [k[0] for k in kernels()] == ["k_d1q3"], (n, v)
            B.lbm_step(c, 34)
            assert [k[0] for k in kernels()] == ["k_d1q3_regs"] * 2, (n, v)
        B.lbm_free(c)
    """)


@pytest.mark.parametrize("lattice,coll,prec", [("d2q9", "minxent4", "fp64"), ("d2q9", "srt", "fp16dev"),
                                               ("d1q3", "srt", "fp64")])
def test_one_step_of_a_batch_is_shape_0s(run, lattice, coll, prec):
    # plain launches and the last launch of a captured chunk
    run("""
    lattice, coll, prec = %r, %r, %r
    sizes = [(k, 300 if lattice == "d2q9" else 1) for k in range(100, 400, 3)]
    c = batch(lattice, coll, "periodic", prec, sizes)
    word, kernel, many = ("register pipeline", "k_d2q9_batch", "k_d2q9_rp") if lattice == "d2q9" else \
        ("nodes in registers", "k_d1q3_batch", "k_d1q3_regs")
    blocks = rec.rec_blocks()
    B.lbm_set_variant(c, 0)
    kernels()
    B.lbm_step(c, 1)
    one = kernels()
    assert [k[0] for k in one] == [kernel]
    for v in shapes(c, word):
        B.lbm_set_variant(c, v)
        n = B.lbm_variant_steps(c, v)
        B.lbm_step(c, 1)
        assert kernels() == one, v
        B.lbm_step(c, n + 1)
        ks = kernels()
        assert [k[0] for k in ks] == [many, kernel] and ks[1:] == one, v
        B.lbm_step(c, n)
        assert kernels() == ks[:1], v
        B.lbm_set_graph_chunk(c, 2 * n + 1)
        B.lbm_step(c, 2 * n + 1)
        ks2 = kernels()
        assert [k for k in ks2 if k[0] != "k_step_base"] == [ks[0], ks[0], one[0]], v
        B.lbm_set_graph_chunk(c, 0)
    B.lbm_set_variant(c, 0)
    assert rec.rec_blocks() <= blocks
    B.lbm_free(c)
    assert rec.rec_blocks() == 0
    """ % (lattice, coll, prec))


# Rule, form, boundary, size; launches of 192 steps, kernel, grid and block of the
# first: what the search over every tile and row count finds.
STARTING_SHAPES = [
    ('srt', 'fp32_newton64', 'box', 3, 3, 3, 'k_d2q9_win', 1, 3, 64),
    ('srt', 'fp32', 'cavity', 3, 3, 3, 'k_d2q9_win', 1, 3, 64),
    ('mrt', 'fp64', 'periodic', 17, 17, 12, 'k_d2q9_win', 1, 17, 576),
    ('minxent4', 'fp16dev', 'box', 17, 17, 3, 'k_d2q9_win', 1, 17, 320),
    ('minxent4', 'fp16dev', 'box', 32, 32, 24, 'k_d2q9_win', 8, 32, 320),
    ('minxent4', 'fp32_newton64', 'periodic', 32, 32, 24, 'k_d2q9_win', 8, 32, 320),
    ('minxent4', 'fp64', 'cavity', 800, 4, 12, 'k_d2q9_win', 200, 1, 192),
    ('minxent4', 'fp16dev', 'box', 800, 4, 3, 'k_d2q9_win', 200, 1, 576),
    ('srt', 'fp32_newton64', 'box', 4, 800, 3, 'k_d2q9_win', 1, 200, 576),
    ('srt', 'fp32', 'cavity', 4, 800, 3, 'k_d2q9_win', 1, 200, 576),
    ('minxent4', 'fp32_newton64', 'periodic', 100, 100, 24, 'k_d2q9_win', 25, 10, 448),
    ('minxent4', 'fp16dev', 'box', 100, 100, 24, 'k_d2q9_win', 25, 10, 448),
    ('minxent4', 'fp64', 'cavity', 257, 257, 32, 'k_d2q9_win', 22, 11, 768),
    ('mrt', 'fp64', 'periodic', 257, 257, 32, 'k_d2q9_win', 22, 11, 768),
    ('trt', 'fp16dev', 'tube', 400, 400, 48, 'k_d2q9_win', 25, 10, 1024),
    ('minxent4', 'fp32_newton64', 'periodic', 400, 400, 48, 'k_d2q9_win', 25, 10, 1024),
    ('srt', 'fp32_newton64', 'box', 500, 300, 48, 'k_d2q9_win', 25, 10, 960),
    ('mrt', 'fp64', 'periodic', 500, 300, 32, 'k_d2q9_win', 36, 14, 768),
    ('trt', 'fp16dev', 'tube', 600, 600, 32, 'k_d2q9_win', 30, 25, 1024),
    ('minxent4', 'fp32_newton64', 'periodic', 600, 600, 192, 'k_d2q9', 3, 600, 256),
    ('minxent4', 'fp16dev', 'box', 1000, 1000, 192, 'k_d2q9', 4, 1000, 256),
    ('minxent4', 'fp32_newton64', 'periodic', 1000, 1000, 192, 'k_d2q9', 4, 1000, 256),
    ('minxent4', 'fp64', 'cavity', 2048, 64, 48, 'k_d2q9_win', 256, 1, 896),
    ('srt', 'fp32_newton64', 'box', 2048, 64, 48, 'k_d2q9_win', 256, 1, 896),
    ('minxent4', 'fp16dev', 'box', 2048, 2048, 192, 'k_d2q9', 8, 2048, 256),
    ('srt', 'fp32', 'cavity', 2048, 2048, 48, 'k_d2q9_rp', 972, 1, 256),
    ('minxent4', 'fp32_newton64', 'periodic', 61, 3001, 48, 'k_d2q9_win', 4, 126, 704),
    ('trt', 'fp16dev', 'tube', 61, 3001, 32, 'k_d2q9_win', 4, 126, 896),
]


def test_starting_shapes_are_those_of_the_whole_search(run):
    # the search leaves candidates early; it has to find what it found without
    run("""
    for coll, prec, bc, nx, ny, launches, *first in %r:
        c = single("d2q9", coll, bc, prec, nx, ny)
        kernels()
        B.lbm_step(c, 192)
        ks = kernels()
        assert len(ks) == launches and list(ks[0]) == first, (coll, prec, bc, nx, ny, len(ks), ks[0])
        B.lbm_free(c)
    """ % (STARTING_SHAPES,))


def test_cache_keys_tell_contexts_apart(run, tmp_path):
    # a lattice and a batch of it alone; batches of one first lattice and total
    run("""
    path, keys = %r, []
    for k, (sizes, many) in enumerate((([(40, 30)], 0), ([(40, 30)], 1), ([(40, 30), (20, 60), (60, 40)], 1),
                                       ([(40, 30), (40, 60), (60, 20)], 1))):
        c = batch("d2q9", "srt", "box", "fp32", sizes) if many else single("d2q9", "srt", "box", "fp32", *sizes[0])
        B.lbm_autotune(c, path)
        B.lbm_free(c)
        keys = [line.split()[0] for line in open(path)]
        assert len(keys) == k + 1, keys
    assert len(set(keys)) == len(keys)
    """ % str(tmp_path / "cache.txt"))


@pytest.mark.parametrize("coll,prec,nx,ny", [("srt", "fp32", 257, 257), ("minxent4", "fp64", 32, 32),
                                             ("mrt", "fp64", 1500, 1500), ("minxent4", "fp16dev", 3000, 2000)])
def test_tuning_times_each_launch_once(run, coll, prec, nx, ny):
    # window shapes that plan alike, or that run as shape 0, are timed once; and
    # shapes of several steps per launch take no more steps than those of two
    run("""
    nx, ny = %d, %d
    c = single("d2q9", %r, "box", %r, nx, ny)
    steps = {v: B.lbm_variant_steps(c, v) for v in range(B.lbm_variant_count(c))}
    windows = {steps[v] for v in shapes(c, "window")} - {1}
    timed = len(steps) - len(shapes(c, "window")) + len(windows)
    kernels()
    B.lbm_autotune(c, None)
    ks = kernels()
    B.lbm_free(c)
    assert len({k for k in ks if k[0] == "k_d2q9_win"}) == len(windows)
    # the first shape timed after the windows marks the end of their first trials
    reps = max(3, min(50, 200000000 // (nx * ny)))
    first = [k for k in ks[:next(i for i, k in enumerate(ks) if k[0] == "k_d2q9_rp")] if k[0] == "k_d2q9_win"]
    assert len(first) == sum(3 + 3 * max(3, 2 * reps // k) for k in windows)
    pads = 0 if nx * ny * 4 < 1 << 20 else 30
    assert len(ks) <= timed * (6 + 3 * reps) + (48 + pads) * (4 * reps + 2) + 200, len(ks)
    """ % (nx, ny, coll, prec))


@pytest.mark.parametrize("nx,ny", [(17, 17), (600, 600), (1500, 1500)])
def test_tuning_moves_the_state_as_a_run_does(run, nx, ny):
    # every timing sets the state aside and puts it back; without memory for the
    # copy the tuner still answers, and writes the other buffer only
    run("""
    c = single("d2q9", "minxent4", "box", "fp64", %d, %d)
    kernels()
    B.lbm_autotune(c, None)
    ks = [k[0] for k in kernels()]
    timings = [i for i, k in enumerate(ks) if k == "k_copy"]
    assert timings and len(timings) %% 2 == 0 and ks[0] == ks[-1] == "k_copy"
    rec.rec_refuse(-1, 0, 0, 1)
    assert 0 <= B.lbm_autotune(c, None) < B.lbm_variant_count(c)
    assert "k_copy" not in [k[0] for k in kernels()]
    B.lbm_free(c)
    """ % (nx, ny))
