"""Calls that only work on a batch's tables run beside copies that were enqueued on the caller's stream before.  A program that
never waits must leave what the same program leaves when it waits for the device after every call (then everything runs on the
caller's stream).  A kernel that only takes time in front of every execute keeps the copies from ending."""
import numpy as np
import pytest

from paper_2604_00368_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MiB = 1 << 20


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_00368_amd import binding
    return binding


def geometry(kind, total, g, per=7):
    """CSR pointers and extents of both sides: transfers of `per` pieces, source pieces in order, destination pieces shuffled."""
    piece = 65536 if kind == "tiled" else 65000
    n = total // piece
    sizes = np.full(n, piece, dtype=np.int64)
    if kind == "ragged":
        sizes -= g.integers(0, 3000, size=n)
    ptr = np.unique(np.concatenate([np.arange(0, n, per), [n]])).astype(np.uint32)
    src = np.zeros(n, dtype=W.EXTENT_DTYPE)
    src["len"], src["off"] = sizes, np.concatenate([[0], np.cumsum(sizes)[:-1]])
    order = g.permutation(n)
    dst = src.copy()
    dst["seg"] = W.DST_SEG
    dst["off"][order] = np.concatenate([[0], np.cumsum(sizes[order])[:-1]])
    return ptr, src, ptr, dst, int(sizes.sum())


class Pools:
    def __init__(self, T, lists, slice_bytes, flags, R):
        self.T, self.dev = T, torch.device("cuda:0")
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        self.n = lists[4]
        self.src = torch.empty(self.n + 8, dtype=torch.uint8, device=self.dev).random_(generator=g)
        self.dst = torch.zeros(self.n + 8, dtype=torch.uint8, device=self.dev)
        self.arena = torch.zeros(self.n + 256 * 64, dtype=torch.uint8, device=self.dev)
        self.stream = torch.cuda.current_stream(self.dev)
        self.ctx = T.tent_create(slice_bytes, self.arena.data_ptr(), self.arena.numel(), flags, R)
        T.tent_register_segment(self.ctx, self.src.data_ptr(), self.src.numel())
        T.tent_register_segment(self.ctx, self.dst.data_ptr(), self.dst.numel())
        self.lists = lists[:4]

    def declare(self):
        return self.T.tent_declare(self.ctx, *self.lists)

    def keep(self):
        return [self.dst.clone(), self.arena.clone()]


def slow_execute(T, p, batch, bounded=False):
    torch.cuda._sleep(1 << 21)
    T.tent_execute_bounded(p.ctx, batch, 4 * MiB, p.stream) if bounded else T.tent_execute(p.ctx, batch, p.stream)


def in_turn(T, kind, flags, wait):
    g = np.random.Generator(np.random.PCG64(3))
    bounded = bool(flags & T.TENT_FLAG_BOUNDED_STAGING)
    pools = [Pools(T, geometry(kind, (12 + 8 * k) * MiB, g), 100 * 1024 if k else 65536, flags, 8) for k in range(3)]
    pause = torch.cuda.synchronize if wait else (lambda: None)
    kept, told = [], []
    try:
        batches = [(p, p.declare()) for p in pools] + [(pools[0], pools[0].declare())]
        for turn in range(14):
            p, b = batches[turn % len(batches)]
            rails = W.make_rails(g.integers(10000, 90000, size=8), queued=g.integers(0, 1 << 20, size=8))
            p.src.add_(turn + 1)                              # the program's own work on the stream, behind the copies of before
            T.tent_reset(p.ctx, b, p.stream); pause()
            if turn % 3 == 2:
                st, info = T.tent_plan_dispatch(p.ctx, b, rails, W.make_dispatch_params(1 << 18, window=turn), None, turn % 2 == 0, p.stream)
                told.append([info.n_mice, info.n_elephant, info.n_deferred] + list(info.plan.rail_bytes) if info else [])
            else:
                st, info = T.tent_plan(p.ctx, b, rails, turn % 3 == 1, p.stream)
                told.append(list(info.rail_bytes) if info else [])
            assert st == 0
            pause()
            slow_execute(T, p, b, bounded); pause()
            kept += p.keep()
            if turn == 8:                                     # a batch goes and another takes its tables while copies run
                T.tent_release(p.ctx, b); pause()
                batches[turn % len(batches)] = (p, p.declare()); pause()
        left = [T.tent_poll(p.ctx, b, p.stream) for p, b in batches]
        tables = [T.tent_get_plan(p.ctx, b).tobytes() for p, b in batches if T.tent_poll(p.ctx, b, p.stream) == 0]
        return kept, told, left, tables
    finally:
        torch.cuda.synchronize()
        for p in pools:
            T.tent_destroy(p.ctx)


@pytest.mark.parametrize("flags", [0, 1, 8])
@pytest.mark.parametrize("kind", ["tiled", "ragged"])
def test_batches_in_turn(T, kind, flags):
    with_waits, without = in_turn(T, kind, flags, True), in_turn(T, kind, flags, False)
    assert with_waits[1:] == without[1:]
    for k, (a, b) in enumerate(zip(with_waits[0], without[0])):
        assert torch.equal(a, b), k


def windows(T, kind, flags, wait):
    g = np.random.Generator(np.random.PCG64(4))
    p = Pools(T, geometry(kind, 320 * MiB, g), 65536, flags, 6)
    pause = torch.cuda.synchronize if wait else (lambda: None)
    told = []
    try:
        b = p.declare()
        for turn in range(2):
            T.tent_reset(p.ctx, b, p.stream); pause()
            for e in range(5):
                rails = W.make_rails(g.integers(10000, 90000, size=6), queued=g.integers(0, 1 << 18, size=6))
                st, _ = T.tent_plan(p.ctx, b, rails, False, p.stream); pause()
                if st != 0:
                    continue
                told.append(T.tent_sim_fail(p.ctx, b, (g.random(6) < 0.2).astype(np.uint8), e % 2 == 0, p.stream)); pause()
                budget = rails["queued_bytes"] + np.uint64((3 if e == 2 else 11) * MiB)      # 66 MiB a window: beside; 18: not
                told.append(T.tent_sim_advance(p.ctx, b, budget, p.stream, e % 2 == 1)); pause()
                T.tent_sim_latency(p.ctx, b, rails["bw_MBps"], p.stream); pause()
                if e == 3:
                    told.append(T.tent_update_bandwidth(p.ctx, b, W.make_probe_params([50000] * 6), rails, p.stream)[1]); pause()
                slow_execute(T, p, b); pause()
        told += [T.tent_poll(p.ctx, b, p.stream), T.tent_get_plan(p.ctx, b).tobytes(), T.tent_get_retries(p.ctx, b).tobytes()]
        return p.keep(), told
    finally:
        torch.cuda.synchronize()
        T.tent_destroy(p.ctx)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("kind", ["tiled", "ragged"])
def test_windows_beside_their_own_copies(T, kind, flags):
    with_waits, without = windows(T, kind, flags, True), windows(T, kind, flags, False)
    for a, b in zip(with_waits[1], without[1]):
        assert np.array_equal(a, b)
    for a, b in zip(with_waits[0], without[0]):
        assert torch.equal(a, b)


def dispatches(T, flags, wait):
    g = np.random.Generator(np.random.PCG64(6))
    # 2,560 transfers, whose priorities travel by a copy, and 366, whose priorities travel with the kernel's arguments
    pools = [Pools(T, geometry("tiled", 160 * MiB, g, per), 65536, flags, 6) for per in (1, 7)]
    pause = torch.cuda.synchronize if wait else (lambda: None)
    kept, told = [], []
    try:
        batches = [p.declare() for p in pools]
        for turn in range(3):
            for p, b in zip(pools, batches):
                p.src.add_(1)
                T.tent_reset(p.ctx, b, p.stream); pause()
            for window in range(3):                               # what no slot takes is deferred, and planned again behind the copies
                for p, b in zip(pools, batches) if turn != 1 else [(pools[0], batches[0])]:
                    n = p.lists[0].shape[0] - 1
                    rails = W.make_rails(g.integers(10000, 90000, size=6), queued=g.integers(0, 1 << 18, size=6), health=[0, 0, 2, 2, 2, 2])
                    dp = W.make_dispatch_params(1 << 17, window=window + turn)
                    st, info = T.tent_plan_dispatch(p.ctx, b, rails, dp, g.integers(0, 3, size=n).astype(np.uint8), (turn, window) == (2, 1), p.stream); pause()
                    assert st == 0
                    if info:
                        told.append([info.n_mice, info.n_elephant, info.n_deferred] + list(info.plan.rail_bytes))
                    slow_execute(T, p, b); pause()
            told += [T.tent_poll(p.ctx, b, p.stream) for p, b in zip(pools, batches)] if turn else []
            for p in pools:
                kept += p.keep()
        told += [T.tent_get_plan(p.ctx, b).tobytes() for p, b in zip(pools, batches)]
        told += [T.tent_get_modes(p.ctx, b, p.lists[0].shape[0] - 1).tobytes() for p, b in zip(pools, batches)]
        return kept, told
    finally:
        torch.cuda.synchronize()
        for p in pools:
            T.tent_destroy(p.ctx)


@pytest.mark.parametrize("flags", [0, 1])
def test_dispatches_beside_copies(T, flags):
    with_waits, without = dispatches(T, flags, True), dispatches(T, flags, False)
    assert with_waits[1] == without[1]
    for k, (a, b) in enumerate(zip(with_waits[0], without[0])):
        assert torch.equal(a, b), k


def test_an_execute_recorded_behind_a_plan_beside_copies(T):
    g = np.random.Generator(np.random.PCG64(5))
    rails = W.make_rails([50000, 25000, 40000])
    p = Pools(T, geometry("tiled", 20 * MiB, g), 65536, 0, 4)
    try:
        one, two = p.declare(), p.declare()
        T.tent_plan(p.ctx, one, rails, False, p.stream)
        T.tent_execute(p.ctx, one, p.stream)
        torch.cuda.synchronize()
        want, p_want = p.dst.clone(), p.arena.clone()
        T.tent_reset(p.ctx, one, p.stream)
        T.tent_plan(p.ctx, one, rails, False, p.stream)
        slow_execute(T, p, one)
        T.tent_plan(p.ctx, two, rails, False, p.stream)       # beside the copies of `one`
        side, graph = torch.cuda.Stream(p.dev), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            T.tent_execute(p.ctx, two, torch.cuda.current_stream(p.dev))
        torch.cuda.synchronize()
        p.dst.zero_()
        p.arena.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(p.dst, want) and torch.equal(p.arena, p_want)
        # the batch is in a graph now: its plans stay on the caller's stream, which orders them before a replay
        for turn in range(3):
            T.tent_reset(p.ctx, one, p.stream)
            T.tent_plan(p.ctx, one, rails, False, p.stream)
            slow_execute(T, p, one)
            T.tent_reset(p.ctx, two, p.stream)
            T.tent_plan(p.ctx, two, rails, False, p.stream)
            p.dst.zero_()
            p.arena.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(p.dst, want) and torch.equal(p.arena, p_want), turn
    finally:
        torch.cuda.synchronize()
        T.tent_destroy(p.ctx)
