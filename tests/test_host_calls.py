"""The library's host side on a recording HIP runtime (hip_recorder.cpp): which
kernels and copies its calls enqueue, on which threads, and what they do when
memory runs out. No GPU takes part."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, json, re, sys
sys.modules["torch"] = None  # its libraries would bind to the recorder too
R = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
R.recorder_take.restype = ctypes.c_size_t
import numpy as np
from paper_1203_6350_amd import lbm

def take():
    buf = ctypes.create_string_buffer(R.recorder_take(None, ctypes.c_size_t(0)) + 1)
    R.recorder_take(buf, ctypes.c_size_t(len(buf)))
    return [l.split() for l in buf.value.decode().splitlines()]

def steps(log=None):
    "The time steps of each launch, with the kernel: o(ne), s(trip) or t(ile)."
    out = []
    for l in take() if log is None else log:
        m = re.search(r"step_multi_strip.*?Li\\d+ELi\\d+ELi(\\d)E", l[1])
        if m:
            out.append("s" + m.group(1))
        elif "11tile_kernel" in l[1]:
            out.append("t" + l[4])
        elif re.search("lbm.{1,3}step_", l[1]):
            out.append("o1")
    return out

def lattice(nx, ny, storage="f32", **kw):
    lat = lbm.Lattice(nx, ny, storage=storage, **kw)
    take()
    return lat
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("recorder") / "recorder.so")
    cxx = shutil.which("g++") or shutil.which("c++")
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(ROOT, "tests", "hip_recorder.cpp"),
                           "-o", out, "-lpthread"])

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body, out], cwd=ROOT,
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.splitlines()[-1])
    return run


def test_copies_on_the_per_thread_stream_stay_on_its_thread(recorder):
    """hipStreamPerThread names another stream in every thread, so a large
    read-out of a handle on it must not copy from other threads."""
    got = recorder("""
out = {}
for stream in (2, 0):  # hipStreamPerThread, the default stream
    lat = lattice(2048, 2048, stream=stream)
    lat3 = lbm.Lattice3(160, 160, 160, stream=stream)
    take()
    n = []
    for call in (lat.moments, lat.populations, lat.save_state, lat3.moments, lat3.populations):
        call()
        n.append(sum(l[0] == "copy" and l[-1] == "other" for l in take()))
    out[stream] = n
print(json.dumps(out))
""")
    assert got["2"] == [0] * 5
    assert any(got["0"])  # elsewhere several threads take part


def test_read_out_without_memory_for_threads(recorder):
    """No memory for a thread's state (bad_alloc): the threads that there are
    make all the copies, and nothing leaves through the C interface."""
    got = recorder("""
lat = lattice(2048, 2048)
out = []
for left in range(4):
    R.recorder_news_left(left)
    lat.moments()
    R.recorder_news_left(-1)
    out.append(sum(l[0] == "copy" for l in take()))
print(json.dumps(out))
""")
    assert got == [48] * 4  # 96 MiB in chunks of 2


def test_a_call_of_any_length(recorder):
    """lbm_step holds nothing that grows with the number of steps: 2^62 of them begin at once
    (the sixth launch is made to fail, which ends the call)."""
    got = recorder("""
import resource
resource.setrlimit(resource.RLIMIT_AS, (8 << 30, 8 << 30))
out = []
for lat in (lattice(2048, 2048), lattice(96, 80), lattice(96, 80, s=(0.3,) * 9)):
    for every in (0, 7, 2 ** 63 - 1):
        lat.set_detector(every)
        take()
        R.recorder_launches_left(5)
        try:
            lat.step(2 ** 62)
        except lbm.LbmError as e:
            out.append([e.code, len(take())])
        R.recorder_launches_left(-1)
print(json.dumps(out))
""")
    assert got == [[-3, 5]] * 9


HANDLES = {
    "strips": "lattice(1300, 1100)",
    "strips f64": "lattice(1300, 1100, 'f64')",
    "tiles": "lattice(96, 80)",
    "tiles f64": "lattice(200, 170, 'f64')",
    "four steps": "tuned(lattice(1300, 1100), 4, 0)",
    "four steps f64": "tuned(lattice(1300, 1100, 'f64'), 4, 0)",
    "three steps": "tuned(lattice(1300, 1100), 3, 8)",
    "tiles for three": "tuned(lattice(96, 80), 3, 0)",
}


@pytest.mark.parametrize("name", list(HANDLES))
def test_launches_of_a_call(recorder, name):
    """The launches of a call take its steps, as many as the set shape's own
    launches in parity (a copy of the lattice counts as one, where the last check
    leaves a single step), and a detector's checks fall on the first multiples of
    the shape's steps, from the call's start, at or after each period."""
    per = 4 if "four" in name else 3 if "three" in name else 1
    got = recorder("""
def tuned(lat, k, rows):
    lat.set_tuning(kernel=k, block=128, rows=rows)
    return lat
out = []
for every in (0, 7, 16):
    lat = %s
    lat.set_detector(every)
    take()
    for n in list(range(1, 42)) + [100, 101]:
        lat.step(n)
        log, at, k = take(), [], 0
        for l in log:
            s = steps([l])
            k += int(s[0][1:]) if s else 0
            if "check" in l[1]:
                at.append(k)
        out.append([every, n, steps(log), at, sum("copy_kernel" in l[1] for l in log)])
print(json.dumps(out))
""" % HANDLES[name])
    done = {}
    for every, n, launches, checks, copies in got:
        assert sum(int(l[1:]) for l in launches) == n
        assert (len(launches) + copies - (-(-n // per))) % 2 == 0, (n, launches)
        assert copies == 0 or every and launches[-1][1:] == "1"
        if every:
            at, k = [], 0
            t0, due = done.get(every, (0, every))
            while k < n:  # the shape's own launches
                k = min(k + per, n)
                if t0 + k >= due:
                    at.append(k)
                    due = ((t0 + k) // every + 1) * every
            done[every] = t0 + n, due
            assert checks == at, (every, n, launches)
            # between checks no more launches than the shape's own
            assert len(launches) <= -(-n // per) + 1


@pytest.mark.parametrize("shape,n", [(None, (4, 3, 6)), ((4, 0), (9, 1, 8)), ((4, 0), (8, 5, 9)),
                                     ((3, 0), (7, 3)), ((3, 8), (4, 4))])
@pytest.mark.parametrize("size", [(96, 80), (2000, 1100)])
def test_buffer_of_a_captured_running_mean(recorder, shape, n, size):
    """Captured calls of a running mean, and the ones after them, leave it in the
    buffer in which the set shape's own launches would: each launch of several
    steps changes it, a single step and a shape that is not set do not."""
    got = recorder("""
shape, calls, size = %r, %r, %r
def where(lat):  # the buffer that the field is read from
    take()
    lat.qref_field()
    return [l[1] for l in take() if l[0] == "copy"][0]
lat = lattice(*size, stream=64)
one = np.ones(size[::-1])
lat.set_qref_field(one, 0 * one, 0 * one)
lat.set_qref_average(0.01)
if shape:
    lat.set_tuning(kernel=shape[0], block=128, rows=shape[1])
    lat.step(shape[0])  # the second buffer is there before the capture
out = []
for capturing in (1, 0, 1):
    R.recorder_capturing(capturing)
    for k in calls:
        a = where(lat)
        lat.step(k)
        out.append([k, a != where(lat)])
print(json.dumps(out))
""" % (shape, n, size))
    per = shape[0] if shape else None
    for k, changed in got:
        assert changed == (per is not None and (k // per + (k % per > 1)) % 2 == 1), got


@pytest.mark.parametrize("size", [(96, 80), (1300, 1100)])
def test_running_mean_without_room_for_a_second_buffer(recorder, size):
    """Single steps need no second buffer: a handle as created takes them where
    there is no memory for one; set strips report it."""
    got = recorder("""
size = %r
out = []
for shape in (None, 0, 4):
    lat = lattice(*size, stream=64)
    one = np.ones(size[::-1])
    lat.set_qref_field(one, 0 * one, 0 * one)
    lat.set_qref_average(0.01)
    if shape is not None:
        lat.set_tuning(kernel=shape, block=128, rows=8 if shape else 0)
    take()
    R.recorder_async_left(0)
    try:
        lat.step(9)
        out.append(steps())
    except lbm.LbmError as e:
        out.append(e.code)
    R.recorder_async_left(-1)
    take()
    lat.step(9)
    out.append(len(steps()))
print(json.dumps(out))
""" % (size,))
    assert got[0] == got[2] == ["o1"] * 9 and got[1] < 9 and got[3] == 9
    assert got[4] == -2 and got[5] == 3


def test_mixes_of_launches(recorder):
    """A set shape's longer launches are taken where there are at least two fewer of
    them, else its own; a single step always takes the one-step kernel; and two steps,
    which the parity makes two launches, are two of those."""
    got = recorder("""
out = {"own": [], "fewer": [], "single": [], "two": []}
for storage in ("f32", "f64"):
    lat = lattice(2048, 1300, storage)
    lat.set_tuning(kernel=4, block=128, rows=0)
    for n in (5, 6, 7, 9, 10, 12, 13, 14, 16, 20):
        lat.step(n)
        rest = {0: [], 1: ["o1"]}.get(n % 4, ["s%d" % (n % 4)])
        out["own"].append(steps() == ["s4"] * (n // 4) + rest)
    for n in (50, 100):
        lat.step(n)
        out["fewer"].append(-(-n // 4) - len(steps()))
for storage in ("f64", "f32", "f16"):
    for nx, ny in ((16, 16), (64, 70), (128, 128), (256, 200), (500, 500), (1000, 900)):
        for kw in ({}, dict(s=(1.7,) * 9)):
            for field in (0, 1, 2):
                lat = lattice(nx, ny, storage, **kw)
                one = np.ones((ny, nx))
                if field == 1:
                    lat.set_qref_field(one, 0 * one, 0 * one)
                if field == 2:
                    lat.set_line_source((1.0, 1e-3, 0.01, 0.0, 0.0, 0.0), True)
                take()
                for n in range(2, 18):
                    lat.step(n)
                    s = steps()
                    out["single"].append("t1" in s)
                    if n == 2:
                        out["two"].append(s == ["o1"] * 2)
print(json.dumps(out))
""")
    assert all(got["own"]) and all(k >= 2 for k in got["fewer"]), got
    assert not any(got["single"]) and all(got["two"])


def test_planes_of_the_two_step_kernel(recorder):
    """D3Q15's chunk height is the best of all, is found once, and a lattice of many
    planes pays nothing for it on each call."""
    got = recorder("""
import time
out = []
for storage in ("f32", "f64"):
    for shape in ((128, 104, 64), (129, 105, 66), (1, 500, 2000), (256, 256, 256), (64, 260, 4001), (320, 130, 999)):
        lat = lbm.Lattice3(*shape, storage=storage)
        take()
        lat.step(8)
        out.append([storage, shape, [int(l[2]) for l in take() if "step3_two" in l[1]]])
def idle(*shape):
    lat = lbm.Lattice3(*shape, storage="f32")
    best = 1.0
    for _ in range(50):
        t = time.perf_counter()
        for _ in range(10):
            lat.step(0)
        best = min(best, time.perf_counter() - t)
    return best
out.append([idle(8, 8, 8), idle(4, 4, 400000)])
print(json.dumps(out))
""")
    small, flat = got.pop()
    assert flat < 4 * small  # 400000 planes had cost 400 us a call
    for storage, (nx, ny, nz), grids in got:
        wide = storage == "f32" and 120 * nx * ny * nz > 256 << 20
        tx, ty, slots = (64 if wide else 32), 13, 256 * (1 if wide or storage == "f64" else 2)
        tiles, best = -(-nx // tx) * -(-ny // ty), (0, 0)
        for chunks in range(1, nz + 1):
            d = -(-nz // chunks)
            wgs = tiles * -(-nz // d)
            use = nx * ny * nz / (-(-wgs // slots) * slots * tx * ty * (d + 2))
            if use > best[0]:
                best = (use, wgs)
            if d <= 4:
                break
        assert grids == ([8 * -(-best[1] // 8)] * 4 if best[0] > 0.5 else []), (storage, nx, ny, nz)


BATCH = """
def kinds(log):
    return ["tile" if "batch_tile" in l[1] else "strip" if "batch_multi" in l[1] else "one"
            for l in log if l[0] == "launch" and l[1] != "graph" and "fill" not in l[1] and "check" not in l[1]]
lats = [lbm.Lattice(64 + i %% 3, 60, storage=%r) for i in range(24)]
b = lbm.Batch(lats)
take()
"""


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
def test_ticks_of_a_small_batch(recorder, storage):
    """Ticks of changing lengths cut no table twice and choose nothing again; a tick of two
    steps takes single steps; a changed member list is cut anew; without memory for
    a table the batch steps one by one."""
    got = recorder(BATCH % storage + """
out = {"kinds": {}, "copies": [], "members": []}
for n in (2, 3, 4, 9, 14, 40):
    for _ in range(4):  # a table is cut once ticks would have gained what it costs
        b.step(n)
        out["kinds"][n] = kinds(take()) or out["kinds"][n]  # (a graph is captured once)
for n in (3, 9, 2, 4, 9, 3, 40, 14, 4):
    b.step(n)
    out["copies"].append(sum(l[0] == "copy" for l in take()))
for who in (lats[:20], lats):
    b.set_members(who)
    take()
    b.step(14)
    out["members"].append(sum(l[0] == "copy" for l in take()))
    b.step(14)
    out["members"].append(sum(l[0] == "copy" for l in take()))
    b.set_members(who)
    take()
    b.step(3)
    out["members"].append(sum(l[0] == "copy" for l in take()))
b = lbm.Batch(lats)
take()
R.recorder_mallocs_left(0)
b.step(14)
R.recorder_mallocs_left(-1)
out["poor"] = kinds(take())
b.step(16)
out["later"] = kinds(take())
print(json.dumps(out))
""")
    assert got["kinds"]["2"] == ["one"] * 2
    assert all(set(got["kinds"][n]) == {"tile"} for n in ("4", "9", "14", "40")), got["kinds"]
    assert all(len(got["kinds"][n]) % 2 == int(n) % 2 for n in got["kinds"])
    assert got["copies"] == [1] * 9  # the members' descriptors
    assert got["members"] == [2, 1, 1] * 2
    assert got["poor"] == ["one"] * 14 and set(got["later"]) == {"tile"}


def test_a_tick_in_which_no_member_steps(recorder):
    """It launches nothing where several steps per launch would leave an empty graph."""
    got = recorder(BATCH % "f32" + """
out = []
for n in (14, 20):
    b.step(n)
    take()
    b.tick(n, [0] * 24)
    out.append(sum(l[:2] == ["launch", "graph"] for l in take()))
out.append([l.info().steps_done for l in lats] == [34] * 24)
print(json.dumps(out))
""")
    assert got == [0, 0, True]


@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_autotuner_fits_four_steps_by_occupancy(recorder, storage):
    """Among the candidates are four steps per launch in the height at which the
    workgroups that the device says it can hold are all resident."""
    nx, ny = 2100, 1500
    got = recorder("""
lat = lattice(%d, %d, %r)
lat.autotune(reps=1)
print(json.dumps([[int(l[2]), int(l[3])] for l in take() if re.search("step_multi_strip.*ELi4EEE", l[1])]))
""" % (nx, ny, storage))
    for block in (64, 128, 256, 512) if storage == "f32" else (64, 128, 256):
        groups = -(-(-(-nx // 56)) // (block // 64))
        chunks = max(1, 256 * (512 // block) // groups)  # what the recorder says
        rows = -(-ny // chunks)
        assert [8 * -(-(groups * -(-ny // rows)) // 8), block] in got, block


def test_strips_of_a_set_height(recorder):
    """The handles of the tests of the four-step strips reach them: a set height on
    small lattices, and large lattices of the general form as created."""
    got = recorder("""
out = []
for storage in ("f64", "f32", "f16"):
    for nx, ny, kw in ((133, 29, {}), (97, 23, dict(s=(1.7,) * 9)), (97, 23, dict(shift_n=0.3, shift_m=0.8))):
        lat = lattice(nx, ny, storage, **kw)
        lat.set_tuning(kernel=4, block=64, rows=5)
        lat.step(8)
        out.append(steps() == ["s4"] * 2)
    for kw in (dict(s=(1.7,) * 9), dict(shift_n=0.3, shift_m=0.8)):
        lat = lattice(1003, 1009, storage, **kw)
        lat.step(11)
        out.append("s4" in steps())
print(json.dumps(out))
""")
    assert got == [True] * 15


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
def test_launches_that_the_benchmark_counts(recorder, storage):
    """Its group of launches is one that the library makes, of the steps it says."""
    bench = pytest.importorskip("bench")
    shapes = [dict(kernel=4, block=128, rows=0), dict(kernel=4, block=128, rows=32),
              dict(kernel=3, block=64, rows=0), dict(kernel=1, block=256, rows=0)]
    groups = []
    for t in shapes:
        per = bench.launch_steps(t, storage)
        groups.append((per, bench.launch_group(t, per, 100)))
    got = recorder("""
out = []
for t, (per, n) in zip(%r, %r):
    lat = lattice(2048, 2048, %r)
    lat.set_tuning(**t)
    lat.step(n * per)
    out.append(steps())
print(json.dumps(out))
""" % (shapes, groups, storage))
    for log, (per, n) in zip(got, groups):
        assert n * per >= 80 and len(log) == n and {int(l[1:]) for l in log} == {per}


@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_autotuned_calls_of_four_steps_per_launch(recorder, storage):
    """Where the autotuner takes more than four steps per launch, the launches of
    up to four run in the block that was fastest for them; a shape set by hand keeps its block."""
    got = recorder("""
lat = lattice(2100, 1500, %r)
lat.autotune(reps=1)
take()
out = [lat.tuning()]
for n in (20, 18 if %r == "f32" else 100):
    lat.step(n)
    log = take()
    out.append([steps(log), [int(l[3]) for l in log]])
lat.set_tuning(kernel=4, block=128, rows=0)
lat.step(20)
log = take()
out.append([steps(log), [int(l[3]) for l in log]])
print(json.dumps(out))
""" % (storage, storage))
    big, n, most = (512, 3, "s6") if storage == "f32" else (256, 0, "s5")
    assert got[0] == dict(kernel=4, block=64, nontemporal=0, rows=0)
    assert got[1] == [["s4"] * 5, [big] * 5]
    assert all(b == (64 if s in ("s5", "s6") else big) for s, b in zip(*got[2])) and most in got[2][0]
    assert got[3] == [["s4"] * 5, [128] * 5]
