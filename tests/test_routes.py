"""Which form of a kernel a call takes, and with what launch shape: the rules of the host
code, read off the arguments of its launches (no GPU needed). Each rule's reason and measured figures stand
beside it in the sources."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_12569_amd", "csrc")
F32X, F64 = 0, 1
I, II = 0, 1
RKF45, RK4, RK4_38 = 0, 1, 2
GPP = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", "-I",
       os.path.join(ROOT, "include"), "-I", CSRC]


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "route_driver")
    subprocess.check_call([*GPP, os.path.join(CSRC, "api.cpp"),
                           os.path.join(ROOT, "tests", "sanitize", "route_driver.cpp"), "-o", exe])

    def call(kind, n, seeds, precision=F32X, method=I, scheme=RKF45, in_flight=0, waves=0, height=0.0, jobs=1):
        seeds = tuple(seeds) + (1,) * (3 - len(seeds))
        args = [kind, *n, *seeds, precision, method, scheme, in_flight, waves, height, jobs]
        r = subprocess.run([exe, *(str(a) for a in args)], capture_output=True, text=True)
        assert r.returncode == 0, (args, r.stdout, r.stderr)
        return {k: int(v) for k, v in (line.split() for line in r.stdout.splitlines())}

    return call


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """(status, [(blocks, threads, kernel)]) of the launchers' host code."""
    from paper_2208_12569_amd import build

    d = tmp_path_factory.mktemp("launches")
    objs = []
    for src in ("trace", "trace_quad", "prep"):
        objs.append(str(d / f"{src}.o"))
        subprocess.check_call([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O0", "-std=c++17", "-w",
                               "-I", build.INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, f"{src}.hip"), "-o", objs[-1]])
    exe = str(d / "launch_driver")
    # (the device code these objects would carry is left out)
    subprocess.check_call([*GPP, "-no-pie", os.path.join(ROOT, "tests", "sanitize", "launch_driver.cpp"), *objs,
                           "-Wl,--unresolved-symbols=ignore-all", "-o", exe])

    def call(*args):
        r = subprocess.run([exe, *(str(int(a) if isinstance(a, bool) else a) for a in args)], capture_output=True, text=True)
        assert r.returncode == 0, (args, r.stdout, r.stderr)
        *rows, status = r.stdout.splitlines()
        return int(status.split()[1]), [(int(g), int(b), k) for g, b, k in (x.split(" ", 2) for x in rows)]

    def trace(precision=F64, store=1, twm=1, list_=0, rev=0, few=0, cyl=0, scheme=RKF45, method=I, jobs=1, tape=0,
              block=0, waves=0):
        return call("trace", precision, store, twm, list_, rev, few, cyl, scheme, method, jobs, tape, block, waves)

    call.trace = trace
    return call


# (fixed steps differentiate planes on a face only)
@pytest.mark.parametrize("kind,height,precision,scheme",
                         [("fit", 0.0, p, s) for p in (F32X, F64) for s in (RKF45, RK4, RK4_38)]
                         + [(k, z, p, RKF45) for k, z in (("fit", 0.13), ("fit3", 0.0)) for p in (F32X, F64)])
def test_gradient_layout_follows_the_reverse_kernel(route, kind, height, precision, scheme):
    """Node gradients lie side by side only for the reverse kernel whose half lines have a
    lane per component (FP64, RKF45); with one lane to a half line each component has a
    plane of its own, where neighbouring lines' additions share cache lines."""
    n = (40, 36, 30)
    r = route(kind, n, (12, 11, 5), precision=precision, scheme=scheme, height=height)
    if precision == F64 and scheme == RKF45:
        assert (r["node_step"], r["value_step"], r["grad_form"]) == (6, 1, 1)
    else:
        assert (r["node_step"], r["value_step"], r["grad_form"]) == (1, 40 * 36 * 30, 3)


@pytest.mark.parametrize("precision", [F32X, F64])
@pytest.mark.parametrize("edge", [64, 128, 256, 400])
def test_four_lanes_to_a_line_up_to_a_share_of_the_chip(route, edge, precision):
    """Up to 65536 half lines and 256 for each node of the longest axis, at most 131072; of
    that a quarter (F32X) or two fifths (F64) where other maps are in flight."""
    n = (edge, edge, edge * 3 // 4)
    most = min(131072, 65536 + 256 * edge)
    for in_flight, limit in ((0, most), (1, most // 4 if precision == F32X else most * 2 // 5)):
        for seeds in (1, 64, 1000, limit - 1, limit, limit + 1, 3 * limit):
            r = route("plane", n, (seeds, 1), precision=precision, in_flight=in_flight)
            assert r["few"] == (seeds <= limit), (seeds, limit, in_flight)
            # an interior plane traces both halves of each line
            r = route("plane", n, (seeds, 1), precision=precision, in_flight=in_flight, height=0.2)
            assert r["few"] == (2 * seeds <= limit), (seeds, limit, in_flight)


@pytest.mark.parametrize("precision,method,limit", [(F32X, I, 32768), (F32X, II, 15360), (F64, I, 15360), (F64, II, 15360)])
def test_tiles_of_a_plane_are_ordered_from_a_wave_or_two_per_simd(route, precision, method, limit):
    """A plane by itself: from about one wave of quads per SIMD on, two in F32X. A chosen
    residency (waves_per_cu) always orders."""
    n = (64, 64, 48)
    for height in (0.0, 0.2):
        lines = limit if height == 0.0 else limit // 2
        for seeds, want in ((16, 0), (lines, 0), (lines + 1, 1), (65536, 1), (300000, 1)):
            r = route("plane", n, (seeds, 1), precision=precision, method=method, height=height)
            assert r["orders"] == want, (seeds, height)
    assert route("plane", n, (16, 1), precision=precision, method=method, waves=4)["orders"] == 1


@pytest.mark.parametrize("precision", [F32X, F64])
def test_voxels_and_batches_are_ordered_above_a_wave_of_lines_per_simd(route, precision):
    n = (64, 64, 48)
    for edge, want in ((8, 0), (32, 0), (33, 1)):
        assert route("voxels", n, (edge, edge, edge), precision=precision)["orders"] == want, edge
    for jobs, seeds, want in ((16, 4096, 0), (16, 4097, 16), (2, 30000, 0), (2, 40000, 2)):
        assert route("plane", n, (seeds, 1), precision=precision, jobs=jobs)["orders"] == want, (jobs, seeds)


@pytest.mark.parametrize("block", [0, 64, 128, 192, 256])
@pytest.mark.parametrize("waves", [0, 1, 4, 6, 12, 64])
def test_every_tracer_launch_takes_the_callers_shape(launches, block, waves):
    """block threads (256 by default) and as many blocks a CU as hold waves_per_cu waves, in
    the one-lane and the four-lane kernel, of maps and of re-trace lists."""
    threads = block or 256
    per_cu = 2048 // threads
    if waves:
        per_cu = min(per_cu, -(-waves * 64 // threads))
    for kw in (dict(few=0), dict(few=1), dict(few=1, method=II), dict(list_=1, twm=2), dict(list_=1, rev=1)):
        status, rows = launches.trace(block=block, waves=waves, **kw)
        assert status == 0 and rows
        for grid, thr, kernel in rows:
            assert (grid, thr) == (256 * per_cu, threads), (kw, kernel)


@pytest.mark.parametrize("n", [(2, 65535, 65535), (2, 65535, 32768), (3, 65535, 32000), (65, 8000, 12500), (65535, 2, 49000),
                               (65535, 49000, 2), (2, 2, 65535), (2048, 2048, 1500), (64, 64, 64), (5, 9, 6)])
@pytest.mark.parametrize("tw", [0, 1])
def test_prep_launch_fits_every_grid_that_memory_holds(launches, n, tw):
    """Fewer than 2^32 threads in a launch, for grids up to what 288 GB hold (28 bytes a
    node with FP32 records, 44 with twist)."""
    assert n[0] * n[1] * n[2] * 28 < 288e9
    status, rows = launches("prep", *n, 0, F32X, tw)
    assert status == 0 and len(rows) == 1
    grid, threads, _ = rows[0]
    assert threads == 256 and 0 < grid * threads < 1 << 32


@pytest.mark.parametrize("dtype,precision", [(0, F32X), (1, F32X), (0, F64), (1, F64)])
def test_records_without_twist_are_packed_in_memory_order(launches, dtype, precision):
    """No neighbours, so no march along y with its lanes past the ends of ragged rows."""
    for n in ((2, 2, 2), (65, 400, 400), (300, 300, 5)):
        for tw, kernel in ((0, "pack_kernel"), (1, "prep_kernel")):
            status, rows = launches("prep", *n, dtype, precision, tw)
            assert status == 0 and len(rows) == 1 and kernel in rows[0][2]
            if not tw:
                assert rows[0][0] == min(4096, -(-n[0] * n[1] * n[2] // 1024))


def test_tape_kernels_on_both_sides_of_the_limit(route, launches):
    """The planes of the adjoint tests on both sides: 270 x 270 on a face and 192 x 192 inside
    a 24-node grid are traced by the one-lane kernel, what lies inside them by the other."""
    n = (24, 21, 19)
    for side, z, few in ((270, 0.0, 0), (192, 0.25, 0), (27, 0.0, 1), (27, 0.25, 1)):
        for precision in (F32X, F64):
            assert route("fit", n, (side, side), precision=precision, height=z)["few"] == few
    for few, kernel in ((0, "trace_kernel"), (1, "trace_quad_kernel")):
        for precision, store in ((F32X, 0), (F64, 1)):
            status, rows = launches.trace(precision=precision, store=store, few=few, tape=1)
            assert status == 0 and [r for r in rows if kernel in r[2]] == rows and len(rows) == 1


def test_positions_only_passes_are_fp64(launches):
    """An FP32 pass takes no positions-only form, in either kernel."""
    for few in (0, 1):
        for twm, ok in ((-1, False), (0, True), (1, True), (2, False), (3, False)):
            status, rows = launches.trace(precision=F32X, store=0, twm=twm, few=few)
            assert (status == 0) == ok and bool(rows) == ok, (few, twm)
        for twm, ok in ((0, True), (1, True), (2, True), (3, True), (4, False)):
            status, rows = launches.trace(twm=twm, few=few, list_=1)
            assert (status == 0) == ok and bool(rows) == ok, (few, twm)


def test_unfinished_half_lines_take_one_lane(launches):
    """The re-trace list goes to both kernels, one of which finds nothing to do; the list of
    half lines that the FP32 pass could not finish to the one-lane kernel alone, which
    ends a line whose trials repeat."""
    for store in (0, 1):
        status, rows = launches.trace(store=store, list_=1, twm=2)
        assert status == 0 and ["trace_quad_kernel" in r[2] for r in rows] == [True, False]
        status, rows = launches.trace(store=store, list_=1, rev=1)
        assert status == 0 and len(rows) == 1 and "trace_quad_kernel" not in rows[0][2]


def test_a_trial_that_repeats_ends_the_line(tmp_path):
    """The one-lane trial step on the host: a rejected step of the smallest length leaves
    every trial after it the same, so the line ends with all of its trials counted."""
    exe = str(tmp_path / "step_driver")
    subprocess.check_call([*GPP, "-O2", "-ffp-contract=off", "-w",
                           os.path.join(ROOT, "tests", "sanitize", "step_driver.cpp"), "-o", exe])
    for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines():
        name, out_of_trials, stood_still, _, faults = line.split()
        assert int(out_of_trials) >= int(stood_still) > 100 and int(faults) == 0, line
