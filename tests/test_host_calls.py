"""What the library's host code asks of the HIP runtime, on a runtime that records the calls and
runs nothing (hip_recorder.cpp): which launches go where, in what order streams and events put
them, and what is left behind when a call fails half way. Each test runs in a process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, importlib.util, os
R = ctypes.CDLL({rec!r}, mode=ctypes.RTLD_GLOBAL)
spec = importlib.util.spec_from_file_location("_lib", {lib!r})
_lib = importlib.util.module_from_spec(spec)
spec.loader.exec_module(_lib)
L = _lib.lib()
P, D, I = ctypes.c_void_p, ctypes.c_double, ctypes.c_int
R.rec_log.argtypes, R.rec_log.restype = [ctypes.c_char_p, ctypes.c_long], ctypes.c_long
R.rec_unordered.argtypes, R.rec_unordered.restype = [P], ctypes.c_long
R.rec_capture.argtypes = [P, ctypes.c_ulonglong]
R.rec_end_capture.argtypes = [ctypes.c_ulonglong]
R.rec_fail.argtypes = [ctypes.c_char_p, I]
R.rec_cost.argtypes = [ctypes.c_char_p, D]
HS, HS2 = 0x10, 0x20  # the caller's streams

def log():
    buf = ctypes.create_string_buffer(R.rec_log(None, 0))
    R.rec_log(buf, len(buf))
    return buf.value.decode().splitlines()

class Plan:
    def __init__(self, shapes):
        n = len(shapes)
        self.n, self.h = n, P()
        st = L.loop_batch_create(n, (D * n)(*[22.0] * n), (I * n)(*[m for m, _ in shapes]),
                                 (I * n)(*[s for _, s in shapes]), ctypes.byref(self.h))
        assert st == 0, st
        ws, pe = ctypes.c_size_t(), ctypes.c_size_t()
        L.loop_batch_info(self.h, ctypes.byref(ws), ctypes.byref(pe), None)
        self.ws_bytes, self.pool_elems = ws.value, pe.value
    def mem(self, size):  # an address with the alignment the calls ask for; kernels do not run
        self.keep = getattr(self, "keep", []) + [ctypes.create_string_buffer(size + 512)]
        return (ctypes.addressof(self.keep[-1]) + 255) // 256 * 256
    def step(self, nsteps=2, hs=HS):
        if not hasattr(self, "T"):
            self.T, self.pool, self.ws = self.mem(8 * self.n), self.mem(16 * self.pool_elems), self.mem(64)
            ctypes.c_uint64.from_address(self.ws + 8).value = 0x4C4F4F504F524254  # a prepared work space
        return L.loop_batch_step(self.h, self.T, self.pool, 1e-4, 1, nsteps, None, self.ws, self.ws_bytes, hs)

MIXED = [(32, 32), (64, 64), (64, 128), (32, 512), (64, 256)]  # three resident block sizes and two other loops
SMALL = MIXED[:3]
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rec") / "hip_recorder.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "hip_recorder.cpp"), "-o", so], check=True)
    return so


@pytest.fixture
def run(recorder):
    def go(body):
        lib = os.path.join(ROOT, "paper_2007_06427_amd", "_lib.py")
        code = PRELUDE.format(rec=recorder, lib=lib) + textwrap.dedent(body)
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go



@pytest.mark.parametrize("streams", [0, 2, 3, 4])
@pytest.mark.parametrize("shapes", ["MIXED", "SMALL"])
def test_a_failed_step_leaves_nothing_unordered(run, shapes, streams):
    """Whichever HIP call of a step fails, and whichever time it is made: the step says so or has
    completed, and what it had queued on the plan's streams comes before the caller's next work."""
    run(f"""
    L.loop_set_resident(2)
    p = Plan({shapes})
    if {streams}:
        assert L.loop_batch_set_schedule(p.h, 2) == 0 and L.loop_batch_set_streams(p.h, {streams}) == 0
    assert p.step() == 0  # the first call also sets up the kernels
    R.rec_reset()
    assert p.step() == 0
    assert R.rec_unordered(HS) == 0
    calls = log()
    assert any("k_resident_batch" in c for c in calls)
    for i, c in enumerate(calls):
        nth = sum(c in d for d in calls[:i + 1])
        R.rec_reset()
        R.rec_fail(c.encode(), nth)
        st = p.step()
        assert st == _lib.LOOP_EHIP, (c, nth, st)
        assert R.rec_unordered(HS) == 0, (c, nth, log())
    R.rec_reset()
    assert p.step() == 0
    assert [c for c in log() if "launch" in c] == [c for c in calls if "launch" in c]
    """)


@pytest.mark.parametrize("streams", [0, 2, 3, 4])
def test_steps_during_a_capture(run, streams):
    """While a capture holds the plan's streams, a step on another stream, eager or inside another
    capture, is taken on that stream alone; steps of the same capture, and later ones, fork again."""
    run(f"""
    L.loop_set_resident(2)
    p = Plan(MIXED)
    if {streams}:
        assert L.loop_batch_set_schedule(p.h, 2) == 0 and L.loop_batch_set_streams(p.h, {streams}) == 0
    def launches(hs):  # of a step on hs: (all, off its stream)
        R.rec_reset()
        assert p.step(hs=hs) == 0
        assert R.rec_unordered(hs) == 0
        at = [c.split("@")[1].split()[0] for c in log() if c.startswith("launch")]
        return len(at), sum(a != "%x" % hs for a in at)
    eager = launches(HS)
    assert eager[1] > 0
    R.rec_capture(HS, 7)
    assert launches(HS) == eager          # recorded: the plan's streams belong to capture 7
    n, off = launches(HS2)                # eager, another stream
    assert n > 0 and off == 0
    R.rec_capture(HS2, 8)
    assert launches(HS2) == (n, 0)        # recorded into a second graph
    R.rec_end_capture(8)
    assert launches(HS) == eager          # the first capture goes on
    R.rec_end_capture(7)
    assert launches(HS2) == eager and launches(HS) == eager
    R.rec_capture(HS2, 9)
    assert launches(HS2) == eager
    """)


def test_one_launch_takes_no_stream_of_the_plan(run):
    run("""
    p = Plan([(32, 32)] * 3)
    R.rec_reset()
    assert p.step() == 0
    assert [c for c in log() if c != "func attribute"] == [c for c in log() if "k_resident_batch" in c and "@10 " in c]
    """)


def test_plan_creation_asks_little_of_the_runtime(run):
    """Neither allocations nor queries grow with the number of loops."""
    run("""
    Plan(MIXED)
    counts = []
    for k in (1, 40):
        R.rec_reset()
        p = Plan(MIXED * k)
        c = log()
        L.loop_batch_destroy(p.h)
        counts.append([sum(x == y for x in c) for y in ("malloc", "memcpy", "attribute", "free")])
    assert counts[0] == counts[1], counts
    assert counts[0][0] <= 4 and counts[0][2] <= 3, counts
    """)


TUNE = """
    def tune(p, reps=4):
        p.step()
        p.rep = (D * 25)()
        R.rec_reset()
        st = L.loop_batch_autotune(p.h, p.T, p.pool, reps, p.rep, p.ws, p.ws_bytes, HS)
        assert st == 0, st
        return log()
    def variants(p):
        v = (I * 5)()
        L.loop_batch_get_config(p.h, None, v, None)
        return list(v)
    def launches(p, nsteps=4):
        R.rec_reset()
        assert p.step(nsteps) == 0
        return [c for c in log() if c.startswith("launch")]
    R.rec_cost(b"k_rag", 100.0)
    R.rec_cost(b"k_ragILi1ELi3E", 80.0)  # row variant 3 is the fastest of passes B and D alone
    R.rec_cost(b"k_ragILi3ELi3E", 80.0)
    R.rec_cost(b"k_ragILi1ELi2E", 90.0)
"""


@pytest.mark.parametrize("mode,count", [(2, 1), (1, 60)])
def test_tuner_keeps_the_resident_form(run, mode, count):
    """Row variant 3 turns the resident form off: the tuner leaves it out where steps take that
    form, and takes it where no loop has the form, or the form is off."""
    run(TUNE + f"""
    L.loop_set_resident({mode})
    shapes = MIXED * {count}
    p = Plan(shapes)
    tune(p)
    assert variants(p)[1] == 2 and variants(p)[3] != 3 and p.rep[4 + 3] == -1
    assert any("k_resident_batch" in c for c in launches(p, 40))
    q = Plan([(64, 256), (32, 512)])
    tune(q)
    assert variants(q)[1] == 3 and variants(q)[3] == 3
    L.loop_set_resident(0)
    r = Plan(shapes)
    assert variants(r)[1] != 2  # tuned with the form on
    tune(r)
    assert variants(r)[1] == 3
    L.loop_set_resident({mode})
    assert variants(Plan(shapes))[1] == 2  # and each choice is kept for its own mode
    """)


def test_tuner_times_what_steps_launch(run):
    """Over the loops that do not take the resident form; for plans whose steps write their
    intermediates in place, within whole steps; and a plan whose variants were set by hand is the
    tuner's again."""
    run(TUNE + """
    grid = lambda c: c.split("grid")[1]
    L.loop_set_resident(2)
    p = Plan(MIXED)
    L.loop_batch_set_variant(p.h, 1, 0)
    calls = [c for c in tune(p) if "k_ragILi1ELi1E" in c]
    assert L.loop_batch_set_schedule(p.h, 0) == 0
    step = launches(p)
    assert any("k_resident_batch" in c for c in step)
    rest = {grid(c) for c in step if "k_ragILi1E" in c}
    assert len(rest) == 1 and {grid(c) for c in calls} == rest, (rest, calls)
    big = Plan([(64, 256)] * 400)  # 160 MB of intermediates
    assert big.ws_bytes > 128 << 20
    calls = "".join(c.split("k_ragILi")[1][0] for c in tune(big) if "k_ragILi" in c and "@10 " in c)
    assert "22" not in calls and "33" not in calls, calls  # no pass C or D over its own output
    """)
