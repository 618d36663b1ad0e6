"""What the library's host side enqueues and answers, without a device: a child process loads a stand-in for the HIP runtime
(fake_hip.c: launches do nothing, every launch, event and wait is logged) and runs one scenario of this file."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
MiB = 1 << 20
LAUNCH, RECORD, WAIT, HOST_WAIT, COPY = 1, 2, 3, 4, 5
STREAM_A, STREAM_B = 0xA0, 0xB0                      # never dereferenced


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2604_00368_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2604_00368_amd import build
        build.build()
    lib = tmp_path_factory.mktemp("fake_hip") / "libamdhip64.so.7"
    subprocess.check_call(["gcc", "-std=gnu11", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-shared", "-fPIC",
                           "-Wl,-soname,libamdhip64.so.7", "-o", str(lib), os.path.join(HERE, "fake_hip.c")])
    return lib


def run(fake, scenario, *args):
    env = dict(os.environ)
    env["LD_LIBRARY_PATH"] = os.pathsep.join(p for p in (str(fake.parent), env.get("LD_LIBRARY_PATH")) if p)
    code = f"import sys; sys.path[:0] = [{ROOT!r}, {HERE!r}]; import test_host_calls as t; t.{scenario}(*{args!r})"
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


class Host:
    """In the child process: the library over the stand-in, one context with a source and a destination segment."""

    def __init__(self, slice_bytes=65536, flags=0, max_rails=0, pool=1 << 40):
        from paper_2604_00368_amd import binding as T
        from paper_2604_00368_amd import workloads as W
        self.T, self.W = T, W
        T.lib()
        self.hip = C.CDLL("libamdhip64.so.7")
        self.hip.fake_kernel_name.restype = C.c_char_p
        self.hip.fake_kernel_name.argtypes = [C.c_void_p]
        self.hip.fake_capture.argtypes = [C.c_void_p]
        self.hip.fake_terms.argtypes = [C.c_void_p, C.c_int, C.c_uint]
        self.ctx = T.tent_create(slice_bytes, 1 << 52, 1 << 60, flags, max_rails)
        T.tent_register_segment(self.ctx, 1 << 44, pool)
        T.tent_register_segment(self.ctx, 1 << 46, pool)

    def extents(self, n, length, step=None):
        """n transfers of one extent each."""
        ext = np.zeros(n, dtype=self.W.EXTENT_DTYPE)
        ext["off"], ext["len"] = np.arange(n, dtype=np.uint64) * np.uint64(step or length), length
        dst = ext.copy()
        dst["seg"] = self.W.DST_SEG
        ptr = np.arange(n + 1, dtype=np.uint32)
        return ptr, ext, ptr, dst

    def log(self):
        """(kind, stream, kernel name or event) of everything since the last call."""
        out = []
        for i in range(self.hip.fake_log_size()):
            stream, what = C.c_void_p(), C.c_void_p()
            kind = self.hip.fake_log_at(i, C.byref(stream), C.byref(what))
            out.append((kind, stream.value, self.hip.fake_kernel_name(what).decode() if kind == LAUNCH else what.value))
        self.hip.fake_log_clear()
        return out


def status_of(T, f, *args):
    try:
        f(*args)
    except T.TentError as e:
        return e.status
    return T.TENT_OK


def unverified_batch(bounded):
    h = Host(flags=8 if bounded else 0)
    T = h.T
    b = T.tent_declare(h.ctx, *h.extents(8, 65536))
    rails = h.W.make_rails([50000, 25000])
    h.hip.fake_fail_host_waits(1)
    assert status_of(T, T.tent_plan, h.ctx, b, rails, False, STREAM_A) == T.TENT_ERR_HIP
    h.log()
    move = (T.tent_execute_bounded, h.ctx, b, MiB, STREAM_A) if bounded else (T.tent_execute, h.ctx, b, STREAM_A)
    assert status_of(T, *move) == T.TENT_ERR_STATE
    assert not [x for x in h.log() if x[0] == LAUNCH]
    # the next plan gets the verdict, and the batch moves
    assert T.tent_plan(h.ctx, b, rails, False, STREAM_A)[0] == T.TENT_OK
    assert status_of(T, *move) == T.TENT_OK
    assert [x for x in h.log() if x[0] == LAUNCH]
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("bounded", [False, True])
def test_nothing_moves_before_the_overlap_verdict(fake, bounded):
    """A plan that cannot read the verdict of the overlap check (the host's wait fails) leaves the batch unplanned: bytes of
    extents that may overlap are not moved in one pass."""
    run(fake, "unverified_batch", bounded)


def plan_beside_bounded(flags, slots, dispatch):
    h = Host(flags=8 | flags)
    T = h.T
    b = T.tent_declare(h.ctx, *h.extents(48, 65536))
    rails = h.W.make_rails([50000, 25000])

    def plan(stream):
        if dispatch:
            T.tent_plan_dispatch(h.ctx, b, rails, h.W.make_dispatch_params(1 << 18), None, False, stream)
        else:
            T.tent_plan(h.ctx, b, rails, False, stream)

    plan(STREAM_A)
    T.tent_execute_bounded(h.ctx, b, MiB, STREAM_A, slots=slots)
    before = h.log()
    last = max(i for i, x in enumerate(before) if x[0] == LAUNCH and x[1] == STREAM_A)
    ends = {x[2] for x in before[last:] if x[0] == RECORD and x[1] == STREAM_A}
    plan(STREAM_B)
    after = h.log()
    first = min(i for i, x in enumerate(after) if x[0] == LAUNCH and x[1] == STREAM_B)
    assert ends & {x[2] for x in after[:first] if x[0] == WAIT and x[1] == STREAM_B}
    # on the execute's own stream there is nothing to wait for, and nothing is waited for inside a capture
    T.tent_execute_bounded(h.ctx, b, MiB, STREAM_A, slots=slots)
    h.log()
    plan(STREAM_A)
    h.hip.fake_capture(STREAM_B)
    plan(STREAM_B)
    assert not [x for x in h.log() if x[0] == WAIT]
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("dispatch", [False, True])
@pytest.mark.parametrize("flags,slots", [(0, 1), (0, 2), (1, 1), (1, 2)])
def test_a_plan_on_another_stream_waits_for_a_bounded_execute(fake, flags, slots, dispatch):
    """Its range copies read the rails and staging offsets that a re-plan rewrites, and its slices are marked DONE at its end."""
    run(fake, "plan_beside_bounded", flags, slots, dispatch)


def extents_in_turn():
    h = Host(slice_bytes=4096, flags=1)
    T, W = h.T, h.W
    sizes = [1 << 40, 1 << 40, 5000, 4096]              # two more segments, short ones
    for k, n in enumerate(sizes[2:]):
        assert T.tent_register_segment(h.ctx, (1 << 47) + (k << 20), n) == 2 + k
    rng = np.random.Generator(np.random.PCG64(3))
    for side in (0, 1):
        for _ in range(200):
            n = int(rng.integers(1, 9))
            ext = np.zeros(n, dtype=W.EXTENT_DTYPE)
            ext["seg"] = rng.integers(0, 4, size=n)
            ext["len"] = rng.integers(1, 4097, size=n)
            ext["off"] = [int(rng.integers(0, sizes[s] - l + 1)) for s, l in zip(ext["seg"].tolist(), ext["len"].tolist())]
            other = ext.copy()
            ptr = np.array([0, n], dtype=np.uint32)
            at, kind = int(rng.integers(0, n)), int(rng.integers(0, 6))
            size = sizes[int(ext["seg"][at])]
            if kind == 1:
                ext["seg"][at] = 4
            elif kind == 2:
                ext["seg"][at], ext["off"][at] = 0xFFFFFFFF, 0
            elif kind == 3:
                ext["off"][at] = size - int(ext["len"][at]) + 1
            elif kind == 4:
                ext["off"][at] = 0xFFFFFFFFFFFFFFFF
            elif kind == 5:
                ext["len"][at] = other["len"][at] = 0
            lists = (ptr, ext, ptr, other) if side == 0 else (ptr, other, ptr, ext)
            st = status_of(T, T.tent_declare, h.ctx, *lists)
            assert st == (T.TENT_ERR_INVALID if kind else T.TENT_OK), (side, kind, ext, other)
    T.tent_destroy(h.ctx)


def test_extents_whose_segments_take_turns(fake):
    """Every extent is held to its own segment, whichever segment the one before it lay in."""
    run(fake, "extents_in_turn")


def payload_at(limit_log2, over):
    h = Host(slice_bytes=1 << 31, flags=1)
    T, W = h.T, h.W
    big = (1 << 32) - 1
    n = (1 << limit_log2) // big
    ext = np.zeros(n + 1, dtype=W.EXTENT_DTYPE)
    ext["len"] = big
    ext["len"][n] = (1 << limit_log2) - n * big - (0 if over else 1)
    assert int(ext["len"].astype(np.uint64).sum()) == (1 << limit_log2) - (0 if over else 1)
    dst = ext.copy()
    dst["seg"] = W.DST_SEG
    ptr = np.array([0, n + 1], dtype=np.uint32)
    b = T.tent_declare(h.ctx, ptr, ext, ptr, dst)
    rails = W.make_rails([4000000000, 2000000000])
    assert status_of(T, T.tent_plan, h.ctx, b, rails, False, STREAM_A) == (T.TENT_ERR_RANGE if over else T.TENT_OK)
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("over", [False, True])
def test_bytes_bound_to_a_rail_stay_below_2_to_53(fake, over):
    """The binding chains count a rail's bytes in doubles, which hold whole numbers below 2^53 exactly."""
    run(fake, "payload_at", 53, over)


def timed_stages():
    h = Host(slice_bytes=4096, flags=2)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    one = lambda *names: {k: int(k in names) for k in T.TENT_T_NAMES}
    for n, plan in ((2048, ("bind",)), (2049, ("extent_scan", "slice_scan", "expand", "bind"))):
        b = T.tent_declare(h.ctx, *h.extents(n, 4096))
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        assert {k: v[1] for k, v in T.tent_get_timings(h.ctx).items()} == one(*plan)
        T.tent_execute(h.ctx, b, STREAM_A)
        assert {k: v[1] for k, v in T.tent_get_timings(h.ctx).items()} == one("gather")
    T.tent_destroy(h.ctx)


def test_stages_that_one_launch_stands_for(fake):
    """A small batch's first plan is one interval under "bind", one-pass copies are one under "gather"."""
    run(fake, "timed_stages")


def figures_that_do_not_come(captured):
    h = Host(slice_bytes=4096)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(64, 4096))
    T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    asks = [lambda: T.tent_plan(h.ctx, b, rails, True, STREAM_A),
            lambda: T.tent_plan_dispatch(h.ctx, b, rails, h.W.make_dispatch_params(1 << 18), None, True, STREAM_A),
            lambda: T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), True, STREAM_A),
            lambda: T.tent_sim_advance(h.ctx, b, np.zeros(2, dtype=np.uint64), STREAM_A),
            lambda: T.tent_update_bandwidth(h.ctx, b, h.W.make_probe_params([50000, 25000]), rails, STREAM_A),
            lambda: T.tent_poll(h.ctx, b, STREAM_A)]
    h.hip.fake_capture(STREAM_A if captured else 0)
    for ask in asks:
        h.log()
        ask()
        assert [x[:2] for x in h.log()].count((HOST_WAIT, STREAM_A)) == 1
    h.hip.fake_capture(0)
    h.hip.fake_fail_host_waits(1)
    assert status_of(T, T.tent_poll, h.ctx, b, STREAM_A) == T.TENT_ERR_HIP
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("captured", [False, True])
def test_a_call_whose_figures_do_not_come_waits_for_its_stream(fake, captured):
    """Kernels store their figures to host memory; where none arrive in time (here launches do nothing), or the stream is being
    captured, the call waits for the stream and passes on what that says."""
    run(fake, "figures_that_do_not_come", captured)


def go_on_elsewhere():
    h = Host(slice_bytes=4096)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(64, 4096))
    calls = [lambda s: T.tent_plan(h.ctx, b, rails, False, s), lambda s: T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), False, s),
             lambda s: T.tent_sim_advance(h.ctx, b, np.zeros(2, dtype=np.uint64), s, False), lambda s: T.tent_execute(h.ctx, b, s),
             lambda s: T.tent_sim_latency(h.ctx, b, np.array([5, 5], dtype=np.uint32), s), lambda s: T.tent_reset(h.ctx, b, s)]
    T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    for k, call in enumerate(calls):
        h.hip.fake_answer_reports(1)
        h.log()
        T.tent_plan(h.ctx, b, rails, True, STREAM_A)
        seen = h.log()
        h.hip.fake_answer_reports(0)
        assert not [x for x in seen if x[0] == HOST_WAIT and x[1] == STREAM_A]
        mark = [x[2] for x in seen if x[0] == RECORD and x[1] == STREAM_A][-1]
        T.tent_sim_latency(h.ctx, b, np.array([5, 5], dtype=np.uint32), STREAM_A)     # more of the batch's work there
        call(STREAM_B)
        log = h.log()
        assert not [x for x in log if x[0] == HOST_WAIT], k
        waits = [i for i, x in enumerate(log) if x == (WAIT, STREAM_B, mark)]
        launches = [i for i, x in enumerate(log) if x[:2] == (LAUNCH, STREAM_B)]
        assert waits and waits[0] < launches[0], k
        T.tent_reset(h.ctx, b, STREAM_A)
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    T.tent_destroy(h.ctx)


def test_a_call_on_another_stream_waits_for_what_a_report_left(fake):
    """A call that reports returns once its figures are there; its kernel may still be writing the tables.  Who goes on elsewhere
    waits for that on the device: calls that only enqueue do not hold up the host."""
    run(fake, "go_on_elsewhere")


def capture_elsewhere():
    h = Host(slice_bytes=4096)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(64, 4096))
    reports = [lambda: T.tent_plan(h.ctx, b, rails, True, STREAM_A),
               lambda: T.tent_plan_dispatch(h.ctx, b, rails, h.W.make_dispatch_params(1 << 18), None, True, STREAM_A),
               lambda: T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), True, STREAM_A),
               lambda: T.tent_sim_advance(h.ctx, b, np.zeros(2, dtype=np.uint64), STREAM_A),
               lambda: T.tent_update_bandwidth(h.ctx, b, h.W.make_probe_params([50000, 25000]), rails, STREAM_A),
               lambda: T.tent_poll(h.ctx, b, STREAM_A)]
    for k, report in enumerate(reports):
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        h.hip.fake_answer_reports(1)
        report()
        h.hip.fake_answer_reports(0)
        h.log()
        h.hip.fake_capture(STREAM_B)
        T.tent_reset(h.ctx, b, STREAM_B)
        T.tent_plan(h.ctx, b, rails, False, STREAM_B)
        T.tent_execute(h.ctx, b, STREAM_B)
        h.hip.fake_capture(0)
        seen = h.log()
        assert {x[0] for x in seen} == {LAUNCH} and {x[1] for x in seen} == {STREAM_B}, (k, seen)
    T.tent_destroy(h.ctx)


def test_a_cycle_captured_behind_a_report_elsewhere(fake):
    """Into a stream that is being captured a cycle is kernels only, whatever reported on another stream before."""
    run(fake, "capture_elsewhere")


def streams_that_are_gone():
    h = Host(slice_bytes=4096)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(64, 4096))
    T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    reports = [lambda s: T.tent_plan(h.ctx, b, rails, True, s),
               lambda s: T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), True, s),
               lambda s: T.tent_sim_advance(h.ctx, b, np.zeros(2, dtype=np.uint64), s),
               lambda s: T.tent_update_bandwidth(h.ctx, b, h.W.make_probe_params([50000, 25000]), rails, s),
               lambda s: T.tent_poll(h.ctx, b, s)]
    goes_on = [lambda: T.tent_plan(h.ctx, b, rails, False, STREAM_A), lambda: T.tent_execute(h.ctx, b, STREAM_A),
               lambda: T.tent_reset(h.ctx, b, STREAM_A)]
    streams = iter(range(0x1000, 0x2000, 16))            # more of them than a batch has marks
    for report in reports * 2:
        for go_on in goes_on:
            T.tent_plan(h.ctx, b, rails, False, STREAM_A)
            gone = next(streams)
            h.hip.fake_answer_reports(1)
            report(gone)
            h.hip.fake_answer_reports(0)
            h.log()                                      # the caller destroys the stream here
            go_on()
            assert gone not in [x[1] for x in h.log()]
    T.tent_destroy(h.ctx)
    assert all(s not in range(0x1000, 0x2000) for _, s, _ in h.log() if s)


def test_a_stream_is_not_touched_once_a_call_has_reported_on_it(fake):
    """A call that reports has waited for its stream: the caller may destroy it and go on with the batch on another."""
    run(fake, "streams_that_are_gone")


def complete(bounded):
    h = Host(flags=8 if bounded else 0)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(8, 65536))
    host_waits = lambda: [x[1:] for x in h.log() if x[0] == HOST_WAIT]

    def move(stream):
        T.tent_plan(h.ctx, b, rails, False, stream)
        h.log()
        T.tent_execute_bounded(h.ctx, b, MiB, stream) if bounded else T.tent_execute(h.ctx, b, stream)
        log = h.log()
        return [x[2] for x in log if x[0] == RECORD][-1:]

    for stream in (STREAM_A, STREAM_B):
        ends = move(STREAM_A)
        h.hip.fake_answer_reports(2)
        assert T.tent_poll(h.ctx, b, stream) != 0 and not host_waits()
        h.hip.fake_answer_reports(1)
        assert T.tent_poll(h.ctx, b, stream) == 0 and host_waits() == [(None, e) for e in ends]
        h.hip.fake_answer_reports(0)
        assert T.tent_poll(h.ctx, b, stream) == 0 and host_waits() == [(stream, None)]
    # an execute in a graph has no mark
    h.hip.fake_capture(STREAM_B)
    assert move(STREAM_B) == []
    h.hip.fake_capture(0)
    h.hip.fake_answer_reports(1)
    assert T.tent_poll(h.ctx, b, STREAM_A) == 0 and host_waits() == [(STREAM_A, None)]
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("bounded", [False, True])
def test_complete_means_that_the_copies_have_been_waited_for(fake, bounded):
    """Nothing left over is the caller's leave to read the destination from anywhere: the copies' end, with its release to the whole
    system, is waited for.  Where slices are left over the figure is enough."""
    run(fake, "complete", bounded)


def beside_copies():
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    one, two = (T.tent_declare(h.ctx, *h.extents(3000, 65536)) for _ in range(2))
    launched = lambda log: {x[1] for x in log if x[0] == LAUNCH}
    index = lambda log, *what: [i for i, x in enumerate(log) if x[:len(what)] == what]

    def cycle(b):
        T.tent_reset(h.ctx, b, STREAM_A)
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        tables = h.log()
        T.tent_execute(h.ctx, b, STREAM_A)
        return tables, h.log()

    h.log()
    for b in (one, two, one, two):                       # nothing runs: everything on the caller's stream
        tables, copies = cycle(b)
        assert launched(tables) == launched(copies) == {STREAM_A}
    h.hip.fake_busy(1)
    end_of_one = [x[2] for x in cycle(one)[1] if x[0] == RECORD][-1]
    tables, copies = cycle(two)                          # beside the copies of the other batch
    assert launched(copies) == {STREAM_A} and len(launched(tables)) == 1 and STREAM_A not in launched(tables)
    own = launched(tables).pop()
    end = [x[2] for x in tables if x[0] == RECORD and x[1] == own][-1]
    assert index(copies, WAIT, STREAM_A, end)[0] < index(copies, LAUNCH, STREAM_A)[0]
    tables, copies = cycle(one)                          # behind its own copies, beside those of the other one
    assert launched(tables) == {own} and index(tables, WAIT, own, end_of_one)[0] < index(tables, LAUNCH, own)[0]
    for _ in range(2):                                   # nothing was enqueued behind its own copies: beside nothing
        tables, copies = cycle(one)
        assert launched(tables) == {STREAM_A}
    # on another stream than the copies', and of a batch whose calls on the caller's stream have not ended: there
    T.tent_plan(h.ctx, two, rails, False, STREAM_B)
    T.tent_plan(h.ctx, two, rails, False, STREAM_A)
    assert launched(h.log()) == {STREAM_A, STREAM_B}
    assert not [x for x in h.log() if x[0] == HOST_WAIT]
    T.tent_destroy(h.ctx)


def two_streams():
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    other = T.tent_create(1 << 20, 1 << 53, 1 << 60)
    for base in (1 << 44, 1 << 46):
        T.tent_register_segment(other, base, 1 << 40)
    one, two = T.tent_declare(h.ctx, *h.extents(3000, 65536)), T.tent_declare(other, *h.extents(3000, 65536))
    h.hip.fake_busy(1)

    def plan_streams(ctx, b, stream):
        T.tent_reset(ctx, b, stream)
        h.log()
        T.tent_plan(ctx, b, rails, False, stream)
        streams = {x[1] for x in h.log() if x[0] == LAUNCH}
        T.tent_execute(ctx, b, stream)
        return streams

    for _ in range(3):                                   # on a stream each: nothing but its own copies is ahead of a plan
        assert plan_streams(h.ctx, one, STREAM_A) == {STREAM_A}
        assert plan_streams(other, two, STREAM_B) == {STREAM_B}
    plan_streams(other, two, STREAM_A)                   # on one stream: beside the copies of the other context's batch
    for _ in range(2):
        assert STREAM_A not in plan_streams(h.ctx, one, STREAM_A)
        assert STREAM_A not in plan_streams(other, two, STREAM_A)
    T.tent_destroy(other)
    T.tent_destroy(h.ctx)


def test_copies_on_another_stream_are_none_to_run_beside(fake):
    """A plan that waits for its own copies leaves the caller's stream only where other copies have been enqueued on it since."""
    run(fake, "two_streams")


def released_copies():
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    declare = lambda: T.tent_declare(h.ctx, *h.extents(3000, 65536))
    old, other = declare(), declare()
    T.tent_plan(h.ctx, old, rails, False, STREAM_A)
    T.tent_execute(h.ctx, old, STREAM_A)
    T.tent_release(h.ctx, old)
    new = declare()                                      # in the slot of the one that has gone, with its events
    T.tent_plan(h.ctx, new, rails, False, STREAM_B)
    h.hip.fake_busy(1)                                   # what runs is on the other stream
    h.log()
    T.tent_plan(h.ctx, other, rails, False, STREAM_A)
    assert {x[1] for x in h.log() if x[0] == LAUNCH} == {STREAM_A}
    T.tent_destroy(h.ctx)


def test_copies_of_a_released_batch_are_none_to_run_beside(fake):
    """A release has waited for them; what the slot's next batch records its event behind are not the copies that it stood for."""
    run(fake, "released_copies")


def streams_with_terms(priority, mask):
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    batches = [T.tent_declare(h.ctx, *h.extents(3000, 65536)) for _ in range(3)]

    def plan(b, stream):
        h.log()
        T.tent_plan(h.ctx, b, rails, False, stream)
        log = h.log()
        return {x[1] for x in log if x[0] == LAUNCH}, log

    plan(batches[0], STREAM_A)
    T.tent_execute(h.ctx, batches[0], STREAM_A)
    h.hip.fake_busy(1)
    own, log = plan(batches[1], STREAM_A)
    assert STREAM_A not in own
    end = [x[2] for x in log if x[0] == RECORD][-1]
    h.hip.fake_terms(STREAM_A, priority, mask)
    assert plan(batches[2], STREAM_A)[0] == {STREAM_A}
    streams, log = plan(batches[1], STREAM_A)            # behind what ran beside the copies
    assert streams == {STREAM_A}
    assert log.index((WAIT, STREAM_A, end)) < [x[0] for x in log].index(LAUNCH)
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("priority,mask", [(-1, 0xFFFFFFFF), (1, 0xFFFFFFFF), (0, 0x0000FFFF)])
def test_calls_stay_on_a_stream_with_a_priority_or_a_share_of_the_device(fake, priority, mask):
    """The caller gave these terms to what is enqueued there; the context's own stream has the default ones."""
    run(fake, "streams_with_terms", priority, mask)


def dispatches_beside(n):
    h = Host(slice_bytes=1 << 20)
    T, W = h.T, h.W
    rails, dp = W.make_rails([50000, 25000]), W.make_dispatch_params(1 << 18)
    one, two = (T.tent_declare(h.ctx, *h.extents(n, 1 << 16)) for _ in range(2))
    prio = np.arange(n, dtype=np.uint8) % 3
    copied = n > 2048                                    # priorities that do not fit the kernel's arguments

    def dispatch(b, info=False):
        h.log()
        h.hip.fake_answer_reports(int(info))
        T.tent_plan_dispatch(h.ctx, b, rails, dp, prio, info, STREAM_A)
        h.hip.fake_answer_reports(0)
        log = h.log()
        streams = {x[1] for x in log if x[0] in (LAUNCH, COPY)}
        assert len(streams) == 1 and [x[0] for x in log].count(COPY) == int(copied)
        first = [i for i, x in enumerate(log) if x[0] in (LAUNCH, COPY)][0]
        return streams.pop(), {x[2] for x in log[:first] if x[0] == WAIT}

    def execute(b):
        h.log()
        T.tent_execute(h.ctx, b, STREAM_A)
        return [x[2] for x in h.log() if x[0] == RECORD]  # the bookkeeping's event, the copies' end

    dispatch(one)
    _, end = execute(one)
    h.hip.fake_busy(1)
    own, waits = dispatch(two)                           # a first plan beside another batch's copies
    assert own != STREAM_A and not waits
    execute(two)
    T.tent_reset(h.ctx, one, STREAM_A)
    stream, waits = dispatch(one)                        # rewrites what its own copies read
    assert stream == own and waits == {end}
    bookkeeping, end = execute(one)
    stream, waits = dispatch(one)                        # what was deferred, behind the bookkeeping
    assert (stream, waits) == ((own, {bookkeeping}) if n * 65536 >= 64 * MiB else (STREAM_A, set()))
    execute(one)
    assert dispatch(one, True)[0] == STREAM_A
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("n", [1023, 1024, 2048, 2049])
def test_dispatches_beside_copies(fake, n):
    """As plans: a first one waits for the batch's own copies, a repeated one for their bookkeeping; one that reports stays."""
    run(fake, "dispatches_beside", n)


def test_tables_are_worked_on_beside_earlier_copies(fake):
    """A plan and a reset move no byte: while copies that they need not wait for run on the caller's stream they run on the
    context's own, behind the batch's own copies, and the batch's next call on the caller's stream waits for them."""
    run(fake, "beside_copies")


def beside_chunks(n, chunks, kind, beside):
    h = Host(slice_bytes=1 << 16, flags=8)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    # whole slices, a short slice at the end of every transfer, or one at the end of every eighth
    short = {"whole": np.zeros(n), "dispatch": np.zeros(n), "short": np.ones(n), "some": np.arange(n) % 8 == 7}[kind].astype(np.uint32)
    ptr, src, _, dst = h.extents(n, chunks * 256 * MiB // n)
    src["len"] -= 1024 * short
    dst["len"] = src["len"]
    one, two = (T.tent_declare(h.ctx, ptr, src, ptr, dst) for _ in range(2))
    h.hip.fake_busy(1)
    streams = []
    for b in (one, two, one):
        T.tent_reset(h.ctx, b, STREAM_A)
        h.log()
        if kind == "dispatch":
            T.tent_plan_dispatch(h.ctx, b, rails, h.W.make_dispatch_params(1 << 18), None, False, STREAM_A)
        else:
            T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        streams.append({x[1] for x in h.log() if x[0] == LAUNCH})
        T.tent_execute_bounded(h.ctx, b, 256 * MiB, STREAM_A)
    assert streams[0] == {STREAM_A} and all((s != {STREAM_A}) == beside for s in streams[1:]), streams
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("n,chunks,kind,beside", [
    (64, 24, "short", True), (64, 25, "short", False), (256, 48, "short", True), (256, 49, "short", False), (256, 20, "some", True),
    (256, 21, "some", False), (4096, 16, "whole", True), (4096, 17, "whole", False), (64, 24, "dispatch", True), (64, 25, "dispatch", False)])
def test_plans_stay_behind_copies_in_many_chunks(fake, n, chunks, kind, beside):
    """Every chunk is a launch, and launches in a row lose time with another stream's beside them: only a long chain is worth it, one
    that goes through many transfers one by one."""
    run(fake, "beside_chunks", n, chunks, kind, beside)


def resets():
    h = Host(slice_bytes=4096)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b = T.tent_declare(h.ctx, *h.extents(64, 4096))

    def reset(stream=STREAM_A):
        h.log()
        T.tent_reset(h.ctx, b, stream)
        assert T.tent_poll(h.ctx, b, stream) == 64
        return h.log()

    T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    T.tent_execute(h.ctx, b, STREAM_A)
    end = [x[2] for x in h.log() if x[0] == RECORD][-1]
    assert reset() == []
    T.tent_plan(h.ctx, b, rails, False, STREAM_B)                  # rewrites what the copies read
    log = h.log()
    assert log.index((WAIT, STREAM_B, end)) < [x[0] for x in log].index(LAUNCH)
    T.tent_execute(h.ctx, b, STREAM_A)
    end = [x[2] for x in h.log() if x[0] == RECORD][-1]
    assert reset(STREAM_B) == [(WAIT, STREAM_B, end)]
    for fail in (1, 0):                                            # retry counts are cleared, once
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        if fail:
            T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), False, STREAM_A)
        assert [x[0] for x in reset()].count(LAUNCH) == fail
    T.tent_plan(h.ctx, b, rails, False, STREAM_A)                  # in a graph there may be some when it is replayed
    h.hip.fake_capture(STREAM_A)
    for _ in range(2):
        assert [x[:2] for x in reset()] == [(LAUNCH, STREAM_A)]
        T.tent_plan(h.ctx, b, rails, False, STREAM_A)
        h.hip.fake_capture(0) if _ else None
    assert [x[0] for x in reset()].count(LAUNCH) == 1
    T.tent_destroy(h.ctx)


def test_a_reset_launches_only_where_something_is_to_be_cleared(fake):
    """The next plan writes the slice table afresh; without retry counts a reset is the host's bookkeeping."""
    run(fake, "resets")


def windows_beside_copies(payload, window, others, beside):
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    b, other = (T.tent_declare(h.ctx, *h.extents(n // 65536, 65536)) for n in (payload, 4 * MiB))
    T.tent_plan(h.ctx, b, rails, False, STREAM_A)
    budget = np.array([window // 2, window // 2], dtype=np.uint64)
    if window < payload:
        T.tent_sim_advance(h.ctx, b, budget, STREAM_A, False)
    else:
        T.tent_plan_dispatch(h.ctx, b, rails, h.W.make_dispatch_params(1 << 18), None, False, STREAM_A)
    h.log()
    T.tent_execute(h.ctx, b, STREAM_A)
    log = h.log()
    bookkeeping, end = [x[2] for x in log if x[0] == RECORD][:2]
    if others:
        T.tent_plan(h.ctx, other, rails, False, STREAM_A)
        T.tent_execute(h.ctx, other, STREAM_A)
        h.log()
    h.hip.fake_busy(1)
    for call in (lambda: T.tent_plan(h.ctx, b, rails, False, STREAM_A), lambda: T.tent_sim_fail(h.ctx, b, np.ones(2, dtype=np.uint8), False, STREAM_A),
                 lambda: T.tent_sim_latency(h.ctx, b, np.array([5, 5], dtype=np.uint32), STREAM_A)):
        call()
        log = h.log()
        own = [x[1] for x in log if x[0] == LAUNCH][0]
        assert (own != STREAM_A) == beside
        assert not [x for x in log if x[0] == WAIT and x[2] == end]
        if own != STREAM_A and bookkeeping:
            first = [i for i, x in enumerate(log) if x[0] == LAUNCH][0]
            assert (WAIT, own, bookkeeping) in log[:first]
            bookkeeping = None                           # (what follows is ordered behind the plan)
    # a call that reports figures has everything behind it that was enqueued on its stream, so that is where it runs
    h.hip.fake_answer_reports(1)
    T.tent_sim_advance(h.ctx, b, budget, STREAM_A)
    h.hip.fake_answer_reports(0)
    log = h.log()
    assert {x[1] for x in log if x[0] == LAUNCH} == {STREAM_A}
    assert bool([x for x in log if x[0] == WAIT and x[1] == STREAM_A]) == (own != STREAM_A)
    T.tent_execute(h.ctx, b, STREAM_A)
    log = h.log()
    assert {x[1] for x in log if x[0] == LAUNCH} == {STREAM_A} and not [x for x in log if x[0] == WAIT]
    T.tent_plan(h.ctx, b, rails, True, STREAM_A)
    assert {x[1] for x in h.log() if x[0] == LAUNCH} == {STREAM_A}
    T.tent_destroy(h.ctx)


@pytest.mark.parametrize("payload,window,others,beside", [
    (64 * MiB, 64 * MiB, False, True), (64 * MiB - 65536, 64 * MiB - 65536, False, False), (1024 * MiB, 64 * MiB, False, True),
    (1024 * MiB, 64 * MiB - 65536, False, False), (1024 * MiB, 2 * MiB, True, True), (64 * MiB - 65536, 2 * MiB, True, False)])
def test_windows_beside_their_own_copies(fake, payload, window, others, beside):
    """A re-plan and the rail simulator behind an execute wait for its bookkeeping only, where that execute's copies are long enough, or
    those of others have been enqueued behind them."""
    run(fake, "windows_beside_copies", payload, window, others, beside)


def capture_behind_beside():
    h = Host(slice_bytes=1 << 20)
    T, rails = h.T, h.W.make_rails([50000, 25000])
    one, two = (T.tent_declare(h.ctx, *h.extents(3000, 65536)) for _ in range(2))
    T.tent_plan(h.ctx, one, rails, False, STREAM_A)
    T.tent_execute(h.ctx, one, STREAM_A)
    h.hip.fake_busy(1)
    h.log()
    T.tent_plan(h.ctx, two, rails, False, STREAM_A)
    log = h.log()
    own = [x[1] for x in log if x[0] == LAUNCH][0]
    end = [x[2] for x in log if x[0] == RECORD and x[1] == own][-1]
    assert own != STREAM_A
    h.hip.fake_capture(STREAM_B)
    T.tent_execute(h.ctx, two, STREAM_B)
    h.hip.fake_capture(0)
    log = h.log()
    assert [x[0] for x in log if x[0] != LAUNCH] == [HOST_WAIT] and log[0] == (HOST_WAIT, None, end)
    assert {x[1] for x in log if x[0] == LAUNCH} == {STREAM_B}
    # a graph holds a call of the batch now: its tables are worked on where the caller can order its replays
    T.tent_execute(h.ctx, one, STREAM_A)
    h.log()
    T.tent_reset(h.ctx, two, STREAM_A)
    T.tent_plan(h.ctx, two, rails, False, STREAM_A)
    assert {x[1] for x in h.log() if x[0] == LAUNCH} == {STREAM_A}
    T.tent_destroy(h.ctx)


def test_a_capture_behind_work_beside_copies(fake):
    """A graph can wait for nothing outside it, and its caller cannot order it behind the context's own stream: the host waits."""
    run(fake, "capture_behind_beside")


def dispatch_chains():
    h = Host(slice_bytes=1)
    T, W = h.T, h.W

    def chain(slices, rails):
        ptr, src, _, dst = h.extents(2, slices)
        b = T.tent_declare(h.ctx, ptr, src, ptr, dst)
        h.log()
        T.tent_plan_dispatch(h.ctx, b, rails, W.make_dispatch_params(1), None, False, STREAM_A)
        names = [x[2] for x in h.log() if x[0] == LAUNCH and "dispatch_chain" in x[2]]
        T.tent_release(h.ctx, b)
        return int(names[0].split("ILi")[1].split("E")[0])

    near = lambda R: W.make_rails([4000000] * R, lat_ns=0)
    assert chain(1000, near(16)) == 0 and chain(1000, near(17)) == 32
    assert chain((1 << 20) - 1, near(16)) == 0 and chain(1 << 20, near(16)) == 16
    # 4,032 slices: costs below 2^37 ps, of which the bytes make up 2,016
    at = ((1 << 37) - 1 - 2016) // 1000
    rails = lambda lat: W.make_rails([4000000] * 3, lat_ns=lat)
    assert chain(4032, rails(at)) == 0 and chain(4032, rails(at + 1)) == 16
    T.tent_destroy(h.ctx)


def test_which_chain_a_dispatch_takes(fake):
    """Up to 16 rails, below 2^20 slices a transfer, and below 2^49 for the largest cost times its slots."""
    run(fake, "dispatch_chains")


# The largest batches tent_declare_static accepts, in units of each kind: flags 0, no overlap check, bounded staging, both;
# with 16 rails and with 64 each.  Found by bisection over a library whose limit was the space its tables took.
STATIC_LIMITS = {
    ("bytes", 4096): [83791, 34360, 98560, 36608, 75935, 31137, 89323, 33178],
    ("slices", 4096): [431520, 431520, 432191, 432191, 371935, 371904, 372479, 372479],
    ("pages", 262144): [97516, 95911, 106832, 104904, 80848, 79632, 87864, 86424],
    ("pieces", 300): [240640, 151327, 422559, 207501, 218080, 137135, 382928, 188048],
}


def static_batch(W, kind, n):
    if kind == "bytes":                                  # transfers of 1001 bytes
        lens, ptr = [1001] * n, np.arange(n + 1)
    elif kind == "slices":                               # one transfer, whole slices
        lens = [MiB] * (n // 256) + ([n % 256 * 4096] if n % 256 else [])
        ptr = np.array([0, len(lens)])
    elif kind == "pages":                                # requests of 100 pages
        lens, ptr = [32768] * n, np.unique(np.append(np.arange(0, n, 100), n))
    else:                                                # transfers of seven extents
        lens, ptr = [77] * n, np.unique(np.append(np.arange(0, n, 7), n))
    src = np.zeros(len(lens), dtype=W.EXTENT_DTYPE)
    src["len"], src["off"] = lens, np.cumsum([0] + lens[:-1])
    dst = src.copy()
    dst["seg"] = W.DST_SEG
    ptr = ptr.astype(np.uint32)
    return ptr, src, ptr, dst


def static_limit(kind, slice_bytes):
    most = iter(STATIC_LIMITS[kind, slice_bytes])
    for flags in (0, 1, 8, 9):
        for max_rails in (16, 64):
            n = next(most)
            h = Host(slice_bytes, flags, max_rails)
            for k in (n, n + 1):
                st = status_of(h.T, h.T.tent_declare_static, h.ctx, *static_batch(h.W, kind, k))
                assert st == (h.T.TENT_OK if k == n else h.T.TENT_ERR_RANGE), (kind, flags, max_rails, k)
            h.T.tent_destroy(h.ctx)


@pytest.mark.parametrize("kind,slice_bytes", sorted(STATIC_LIMITS))
def test_static_limit_stays_where_it_was(fake, kind, slice_bytes):
    run(fake, "static_limit", kind, slice_bytes)
