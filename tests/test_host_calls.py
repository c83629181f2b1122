"""What the library's calls ask of the HIP runtime, on a runtime that runs nothing (tests/host/calls.cpp; no GPU):
the kernels launched, their limits of dynamic LDS, streams, events and captures."""

import math
import os
import subprocess

import pytest

from paper_1502_07478_amd import jpet

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PIXEL = 2.0
# the register caches of the passes on ring blocks: 1000 (one event per wavefront) + 100 rings + pixels of a row
SHAPES = [108, 112, 116, 124, 210, 214, 218, 222, 228, 314, 318, 322, 326, 1132, 1148, 1164, 1216, 1222, 1228, 1236,
          1248, 1264, 1318, 1324, 1332, 1344, 1354, 1364, 1420, 1428, 1440, 1454]
# ellipses of these sizes leave the regions of the log-likelihood (doubles) no room in LDS: the pass without binning
LOGLIK_GENERIC = (1264, 1344, 1354, 1364, 1440, 1454)


def resolution(shape, half_rows=None):
    """sigma_z and sigma_dl whose largest ellipse just fits a shape (122.4 rows: a region of 256 rows)."""
    if half_rows is None:
        half_rows = min((32 if shape >= 1000 else 16) * (shape % 1000 // 100) - 0.6, 122.4)
    return (shape % 100 - 0.5) * PIXEL * math.sqrt(2.0) / 6.0, half_rows * PIXEL / 1.5


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    lib = jpet.LIB_PATH
    if not os.path.exists(lib):
        from paper_1502_07478_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "calls")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(rocm, "include"), "-pthread", os.path.join(ROOT, "tests", "host", "calls.cpp"), "-rdynamic",
                    lib, f"-Wl,-rpath,{os.path.dirname(lib)}", f"-Wl,-rpath-link,{rocm}/lib", "-o", exe], check=True)

    def run(call, *geometries):
        """The log of a call: geometries are (sigma_z, sigma_dl, pixel, n_y, n_z, n, plan[, R, L])."""
        args = [call]
        for k, (sz, sdl, pixel, n_y, n_z, n, plan, *strips) in enumerate(geometries):
            R, L = strips or (450.0, 500.0)
            args += ([";"] if k else []) + [repr(float(v)) for v in (R, L, sz, sdl, pixel)] + [str(v) for v in (n_y, n_z, n, plan)]
        res = subprocess.run([exe, *args], capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, (res.returncode, res.stderr)
        return [line.split() for line in res.stdout.splitlines()]
    return run


def codes(log):
    return {line[1]: int(line[2]) for line in log if line[0] == "rc"}


def launches(log, name):
    """(kernel with its arguments, line) of every launch of a kernel by its name without arguments."""
    return [(line[1], line) for line in log if line[0] == "launch" and line[1].split("<")[0] == name]


def limits_hold(log):
    """Every launch has a raised limit where it needs one, of at least its dynamic LDS."""
    limit = {}
    for line in log:
        if line[0] == "limit":
            limit[line[1]] = int(line[3])
        elif line[0] == "launch":
            lds = int(line[line.index("lds") + 1])
            assert lds <= limit.get(line[1], 64 * 1024), line
            assert int(line[line.index("block") + 1]) <= 1024


@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_reach_their_kernels(calls, shape):
    """An ellipse that just fits a register cache launches the kernels compiled for it: alone and in a batch, the
    pass and the forward sums, the log-likelihood and its value."""
    sz, sdl = resolution(shape)
    n = 257
    g = jpet.geometry(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=101, n_z=83)
    plan = next(c for c, _ in jpet.plan_candidates(g, n) if c & 4 and c >> 12 == 0)
    geo = (sz, sdl, PIXEL, 101, 83, n, plan)
    for call, kernel, rest in (("iterate", "k_event_pass_rings", ",false"), ("denominators", "k_event_pass_rings", ",true"),
                               ("batch", "k_event_pass_rings_batched", "")):
        log = calls(call, geo)
        assert set(codes(log).values()) == {0}, log
        limits_hold(log)
        found = [name for name, _ in launches(log, kernel)]
        assert found, log
        for name in found:
            args = name[name.index("<") + 1:-1].split(",", 2)
            assert int(args[0]) == shape and "," + args[2] == rest if rest else len(args) == 2 and int(args[0]) == shape, name
    geo = geo[:-1] + (0,)
    log = calls("loglik", geo)
    limits_hold(log)
    assert codes(log)["loglik"] == 0
    if shape in LOGLIK_GENERIC:
        assert launches(log, "k_loglik_pass")
        return
    assert launches(log, "k_loglik_rings")[0][0].startswith(f"k_loglik_rings<{shape},")
    log = calls("value", geo)
    limits_hold(log)
    rings, solo = shape % 1000 // 100, "true" if shape >= 1000 else "false"
    assert codes(log)["loglik"] == 0 and launches(log, "k_loglik_rings_value")[0][0] == f"k_loglik_rings_value<{rings},{solo}>"


@pytest.mark.parametrize("half_rows", [95.6, 96.0, 103.0, 111.0, 118.0, 122.0, 123.0, 126.0, 126.9])
@pytest.mark.parametrize("length", [8, 20, 28])
def test_batches_of_tall_ellipses(calls, half_rows, length):
    """Regions of more than 256 rows (a pitch of 320) run in a batch as they do alone."""
    sz, sdl = resolution(1400 + length, half_rows)
    geo = (sz, sdl, PIXEL, 300, 300, 50_000, 0)
    alone, log, graph = calls("iterate", geo), calls("batch", geo), calls("graph", geo)
    for got in (alone, log, graph):
        assert set(codes(got).values()) == {0}, codes(got)
        limits_hold(got)
    kernels = {name for name, line in launches(log, "k_event_pass_rings_batched")}
    assert len(kernels) == 1 and kernels == {name for name, line in launches(graph, "k_event_pass_rings_batched")}


@pytest.mark.parametrize("shape,half_rows,pitch", [(112, 15.4, 64), (112, 15.4, 128), (218, 26.0, 64), (218, 31.4, 128),
                                                   (322, 47.4, 128), (322, 47.4, 192), (1132, 26.0, 64), (1132, 31.4, 128),
                                                   (1222, 57.0, 128), (1222, 63.4, 192), (1324, 89.0, 192), (1324, 95.4, 256),
                                                   (1428, 122.4, 256), (1428, 126.0, 320)])
def test_large_items_reach_both_pitches(calls, shape, half_rows, pitch):
    """The kernels of the plans that the GPU tests of items of 128 events and more name."""
    sz, sdl = resolution(shape, half_rows)
    n = 140_000
    g = jpet.geometry(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=33, n_z=33)
    for plan, _ in jpet.plan_candidates(g, n):
        i = jpet.launch_info(jpet.with_plan(g, plan), n)
        rows = i["tile_rows"] + 2 * i["halo_rows"]
        if (i["accumulator_bits"] == 32 and i["row_segments"] == 1 and i["events_per_batch"] == (1 if shape >= 1000 else 2) and
                i["events_per_workgroup"] >= 128 and (rows + 63) // 64 * 64 == pitch):
            break
    else:
        pytest.fail("no plan")
    log = calls("iterate", (sz, sdl, PIXEL, 33, 33, n, plan))
    limits_hold(log)
    assert {name for name, _ in launches(log, "k_event_pass_rings")} == {f"k_event_pass_rings<{shape},{pitch},false>"}


# the most events jpet_mlem_iterate_noalloc took on batches of rows, and for a named plan (R, L, sigma_z, sigma_dl,
# pixel, n_y, n_z): (events, (events, plan) or None)
NOALLOC = {
    (450, 500, 14.2, 17.2, 2.21, 344, 500): (884704, None),
    (450, 500, 19.8, 15.9, 1.79, 73, 200): (849564, (809586, 2253)),
    (450, 500, 19.2, 11.6, 1.31, 609, 609): (828252, (764740, 2061)),
    (450, 500, 8.7, 14.0, 1.05, 134, 134): (719465, (676356, 2253)),
    (450, 500, 4.2, 13.3, 4.63, 39, 300): (997184, (956800, 2253)),
    (450, 500, 13.6, 28.1, 1.89, 119, 119): (677611, (645843, 2253)),
    (450, 500, 19.4, 47.4, 0.23, 1004, 300): (4393033, None),
    (450, 500, 30, 63, 1, 400, 400): (4430692, None),
    (450, 500, 10, 63, 2, 400, 400): (403470, None),
    (450, 500, 10, 63, 4, 64, 64): (631900, None),
    (130, 300, 10, 40, 4, 64, 76): (784512, None),
}


@pytest.mark.parametrize("geo", list(NOALLOC))
def test_noalloc_takes_what_fits_on_batches_of_rows(calls, geo):
    """Its array has a fixed size: where ring blocks need more, the call takes a plan that fits, or the named plan
    on batches of rows."""
    R, L, sz, sdl, pixel, n_y, n_z = geo
    most, named = NOALLOC[geo]
    for n, plan in ((most, 0), (int(0.9 * most), 0), *([named] if named else [])):
        log = calls("noalloc", (sz, sdl, pixel, n_y, n_z, n, plan, float(R), float(L)))
        assert codes(log)["noalloc"] == 0, (n, plan)
        limits_hold(log)
    assert codes(calls("noalloc", (sz, sdl, pixel, n_y, n_z, 20_000_000, 0, float(R), float(L))))["noalloc"] == jpet.JPET_EWORKSPACE


TWO_CLASSES = ((10.0, 63.0, 2.0, 200, 200, 50_000, 0), (4.0, 20.0, 2.0, 100, 100, 4_000, 0))


def test_a_capture_has_its_streams_and_events_to_itself(calls):
    """Streams and events of a graph's capture are made for it, used by nothing else and kept until the graph is
    instantiated: work that another call enqueued on them would become part of the graph."""
    log = calls("mixed", *TWO_CLASSES)
    assert set(codes(log).values()) == {0}
    at = {key: next(k for k, line in enumerate(log) if line[0] == key) for key in ("capture+", "capture-", "instantiate")}
    start = max(k for k, line in enumerate(log[:at["capture+"]]) if line[0] == "launch") + 1  # the batch's set-up ends

    def used(lines):
        streams = {line[line.index("stream") + 1] for line in lines if "stream" in line}
        return streams, {line[1] for line in lines if line[0] in ("record", "wait")}

    inside = used(log[at["capture+"]:at["capture-"] + 1])
    made = log[start:at["capture+"]]
    assert len(inside[0]) == 2 and len(inside[1]) == 2
    assert inside[0] == {line[1] for line in made if line[0] == "stream+"}
    assert inside[1] == {line[1] for line in made if line[0] == "event+"}
    outside = used(log[:start] + log[at["capture-"] + 1:])
    assert not inside[0] & outside[0] and not inside[1] & outside[1]
    for line in log[:at["instantiate"]]:
        assert line[0] not in ("stream-", "event-")
    gone = log[at["instantiate"]:]
    assert inside[0] == {line[1] for line in gone if line[0] == "stream-"}
    assert inside[1] == {line[1] for line in gone if line[0] == "event-"}


def test_threads_do_not_mix_their_forks_and_joins(calls):
    """Eager batches of two threads share the side stream and its events: a wait takes an event's latest record, so
    between one thread's record and its wait the other records nothing."""
    log = [line for line in calls("threads", *TWO_CLASSES) if line[0] in ("record", "wait")]
    assert {line[-1] for line in log} == {"1", "2"}
    latest = {}
    for line in log:
        if line[0] == "record":
            latest[line[1]] = line[-1]
        else:
            assert latest[line[1]] == line[-1], line


def test_graphs_are_closed_after_their_launches(monkeypatch):
    """A graph that is created again (another number of iterations, or after eager iterations) replaces one whose last
    launch may still run; destroying it waits for the device first."""
    import ctypes

    import torch
    done = []

    class Library:
        def jpet_mlem_batched_graph_create(self, *a):
            done.append("create")
            return 0

        def jpet_mlem_batched_graph_destroy(self, h):
            done.append("destroy")
            return 0

    monkeypatch.setattr(jpet, "_lib", lambda: Library())
    monkeypatch.setattr(jpet, "_stream", lambda stream: None)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: done.append("wait"))
    b = jpet.BatchedMLEM.__new__(jpet.BatchedMLEM)
    b.arr, b.count, b.ws = None, 0, torch.empty(256, dtype=torch.uint8)
    b._graphs, b._table_of = {2: ctypes.c_void_p(1)}, 2
    b.graph(3)
    assert done == ["wait", "destroy", "create"]
    b.close_graphs()
    assert done == ["wait", "destroy", "create", "wait", "destroy"]


def test_denominators_of_long_lists_are_cleared_by_many_blocks(calls):
    """A list of 10M events on a 4 x 4 grid: the launch that clears its denominators (and reads the image) has blocks
    for the list, not for the 16 pixels alone."""
    for call in ("loglik", "value"):
        (name, line), = launches(calls(call, (10.0, 63.0, 4.0, 4, 4, 10_000_000, 0)), "k_loglik_begin")
        assert int(line[line.index("grid") + 1]) == 256
    (name, line), = launches(calls("loglik", (10.0, 63.0, 4.0, 4, 4, 300, 0)), "k_loglik_begin")
    assert int(line[line.index("grid") + 1]) == 2


def test_scan_of_many_bins_is_not_quadratic(calls):
    """A fine grid has millions of bins: at most 2048 blocks scan them, from sums of each block's bins."""
    geo = (1.5, 8.0, 0.2, 4096, 4096, 100_000, 0, 450.0, 1000.0)
    g = jpet.geometry(R=450.0, L=1000.0, sigma_z=1.5, sigma_dl=8.0, pixel=0.2, n_y=4096, n_z=4096)
    assert jpet.launch_info(g, 100_000)["bins"] > 2_097_152
    log = calls("iterate", geo)
    grids = [int(launches(log, name)[0][1][3]) for name in ("k_scan_sums", "k_scan")]
    assert grids[0] == grids[1] <= 2048
    # few bins: no sums
    assert not launches(calls("iterate", TWO_CLASSES[0]), "k_scan_sums")


def test_limits_do_not_depend_on_the_call(calls):
    """A kernel's limit of dynamic LDS is process-wide: were it each call's own need, two threads could lower it under
    each other's launches.  The preparation and the passes on ring blocks, small plans and large ones."""
    limits = {}
    for shape in (112, 322, 1344):
        sz, sdl = resolution(shape)
        for grid in (30, 400):
            n = 140_000
            g = jpet.geometry(R=450.0, L=500.0, sigma_z=sz, sigma_dl=sdl, pixel=PIXEL, n_y=grid, n_z=grid)
            plans = [c for c, _ in jpet.plan_candidates(g, n) if c & 4 and c >> 12 == 0]
            for plan in (plans[0], plans[-1]):
                geo = (sz, sdl, PIXEL, grid, grid, n, plan)
                for call in ("iterate", "denominators", "batch"):
                    for line in calls(call, geo):
                        if line[0] == "limit" and ("rings" in line[1] or "prepare" in line[1]):
                            limits.setdefault(line[1], set()).add(int(line[3]))
            for call in ("loglik", "value"):
                for line in calls(call, geo[:-1] + (0,)):
                    if line[0] == "limit" and ("rings" in line[1] or "prepare" in line[1]):
                        limits.setdefault(line[1], set()).add(int(line[3]))
    assert "k_prepare<true>" in limits and len(limits) > 8
    assert all(len(v) == 1 for v in limits.values()), limits
