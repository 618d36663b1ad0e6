"""Declarations at the sizes where the address order changes its method (one workgroup up to 4096 extents, a device-wide sort
above), address bits that differ in few or many places, and overlaps wherever they can hide."""
import numpy as np
import pytest

from paper_2604_00368_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_00368_amd import binding
    return binding


class Pools:
    """Source and destination pools of `n` extents of `size` bytes (destination `gap` bytes apart) in shuffled order."""

    def __init__(self, T, n, size, gap=0, per_desc=3, seed=1, flags=0, dst_base=0):
        g = np.random.Generator(np.random.PCG64([n, size, seed]))
        self.T, self.n, self.size = T, n, size
        pitch = size + gap
        self.src = torch.from_numpy(g.integers(0, 256, size=n * size + 64, dtype=np.uint8)).cuda()
        self.dst = torch.zeros(dst_base + n * pitch + 64, dtype=torch.uint8, device="cuda")
        self.arena = torch.zeros(n * size + 1024, dtype=torch.uint8, device="cuda")
        self.ctx = T.tent_create(4 * size, self.arena.data_ptr(), self.arena.numel(), flags)
        T.tent_register_segment(self.ctx, self.src.data_ptr(), self.src.numel())
        T.tent_register_segment(self.ctx, self.dst.data_ptr(), self.dst.numel())
        self.se, self.de = np.zeros(n, dtype=W.EXTENT_DTYPE), np.zeros(n, dtype=W.EXTENT_DTYPE)
        self.se["off"], self.se["len"] = g.permutation(n) * size, size
        self.de["seg"], self.de["off"], self.de["len"] = W.DST_SEG, dst_base + g.permutation(n) * pitch, size
        self.ptr = np.append(np.arange(0, n, per_desc), n).astype(np.uint32)
        self.rails = W.make_rails([50000, 20000, 70000])

    def declare(self, se=None, de=None):
        return self.T.tent_declare(self.ctx, self.ptr, self.se if se is None else se, self.ptr, self.de if de is None else de)

    def move(self, h, info=False):
        stream = torch.cuda.current_stream()
        self.T.tent_plan(self.ctx, h, self.rails, info, stream)
        self.T.tent_execute(self.ctx, h, stream)
        assert self.T.tent_poll(self.ctx, h, stream) == 0

    def check(self):
        src, dst = self.src.cpu().numpy(), self.dst.cpu().numpy()
        want = np.zeros_like(dst)
        for a, b in zip(self.se["off"].tolist(), self.de["off"].tolist()):
            want[b:b + self.size] = src[a:a + self.size]
        assert np.array_equal(dst, want)

    def close(self):
        self.T.tent_destroy(self.ctx)


@pytest.mark.parametrize("n", [1, 2, 3, 1023, 1024, 1025, 2047, 2048, 2049, 5000])
@pytest.mark.parametrize("size,gap", [(64, 0), (61, 0), (1024, 3072)])
def test_address_order_at_the_edges(T, n, size, gap):
    p = Pools(T, n, size, gap)
    h = p.declare()
    p.move(h, info=n % 2 == 0)
    p.check()
    p.close()


def test_order_without_the_check(T):
    for n in (2048, 4096, 4097):                             # destinations only
        p = Pools(T, n, 1024, 0, flags=T.TENT_FLAG_SKIP_OVERLAP_CHECK)
        p.move(p.declare())
        p.check()
        p.close()


@pytest.mark.parametrize("n", [2, 40, 2048, 2049, 4000])
@pytest.mark.parametrize("where", ["first_two", "last_two", "inside_a_longer_one", "source_under_destination", "same_place"])
def test_overlaps_are_found(T, n, where):
    p = Pools(T, n, 64, 0)
    se, de = p.se.copy(), p.de.copy()
    order = np.argsort(de["off"])
    if where == "first_two":
        de["off"][order[1]] -= 1
    elif where == "last_two":
        de["off"][order[-1]] -= 63
    elif where == "same_place":
        de["off"][order[n // 2]] = de["off"][order[n // 2 - 1]]
    elif where == "inside_a_longer_one":                     # a long extent covers several that do not touch each other
        se, de = np.append(se, se[:1]), np.append(de, de[:1])
        se["len"][-1] = de["len"][-1] = 2 * 64 if n > 1 else 64
        se["off"][-1], de["off"][-1] = 0, 0
    else:                                                    # a source extent lies where a destination is
        se["seg"][0], se["off"][0] = W.DST_SEG, de["off"][order[n // 2]] + 60
    ptr = p.ptr.copy()
    ptr[-1] = se.shape[0]
    for info in (False, True):
        h = T.tent_declare(p.ctx, ptr, se, ptr, de)
        with pytest.raises(T.TentError) as err:
            T.tent_plan(p.ctx, h, p.rails, info, torch.cuda.current_stream())
        assert err.value.status == T.TENT_ERR_INVALID
        with pytest.raises(T.TentError) as err:              # the batch is gone
            T.tent_slice_count(p.ctx, h)
        assert err.value.status == T.TENT_ERR_INVALID
    # the verdict comes before "no rail" and "arena too small", and the context goes on
    h = T.tent_declare(p.ctx, ptr, se, ptr, de)
    none = p.rails.copy()
    none["health"] = 2
    with pytest.raises(T.TentError) as err:
        T.tent_plan(p.ctx, h, none, True, torch.cuda.current_stream())
    assert err.value.status == T.TENT_ERR_INVALID
    p.move(p.declare())
    p.check()
    p.close()


def test_extents_that_touch_do_not_overlap(T):
    p = Pools(T, 500, 33, 0)
    p.move(p.declare())
    p.check()
    p.close()


def test_counters_start_afresh_every_time(T):
    """Calls that report counts, repeated and interleaved: every one counts from zero."""
    p = Pools(T, 3000, 64, 0)
    stream = torch.cuda.current_stream()
    h = p.declare()
    n = T.tent_slice_count(p.ctx, h)
    for _ in range(3):
        T.tent_reset(p.ctx, h, stream)
        _, info = T.tent_plan(p.ctx, h, p.rails, True, stream)
        assert info.n_slices == n and sum(info.rail_slices) == n
        assert T.tent_poll(p.ctx, h, stream) == n
        failed = T.tent_sim_fail(p.ctx, h, [0, 1, 0], True, stream)
        assert failed[1] == info.rail_slices[1] and failed[0] == failed[2] == 0
        assert T.tent_sim_advance(p.ctx, h, [1 << 40] * 3, stream) == n - failed[1]
        T.tent_sim_latency(p.ctx, h, [50000, 20000, 70000], stream)
        for _ in range(2):
            rails, probe = T.tent_update_bandwidth(p.ctx, h, W.make_probe_params([100000] * 3), p.rails, stream)
            assert probe[1] == 0 and probe[0] > 0 and rails["bw_MBps"][1] == 20000
        T.tent_execute(p.ctx, h, stream)
        assert T.tent_poll(p.ctx, h, stream) == failed[1]
        T.tent_plan(p.ctx, h, p.rails, False, stream)
        T.tent_execute(p.ctx, h, stream)
        assert T.tent_poll(p.ctx, h, stream) == 0
    p.check()
    p.close()


@pytest.mark.parametrize("max_rails", [16, 64])
def test_static_limit_counts_entries_not_layout(T, max_rails):
    """The largest batch that the 64 MiB limit accepts is declared, planned and moved; one transfer more than fits is
    refused.  Geometry without a tile size and without the address order, whose tables take most per counted byte."""
    S, length = 4096, 1001
    n = {16: 98560, 64: 36608}[max_rails]                    # (test_host_calls.py has the limit for more kinds of batch)
    rails = W.tiny().rails
    pool = (n + 1) * 1024
    src = torch.randint(0, 256, (pool,), dtype=torch.uint8, device="cuda:0")
    dst = torch.zeros_like(src)
    arena = torch.empty((n + 1) * length + 256 * 64, dtype=torch.uint8, device="cuda:0")
    ctx = T.tent_create(S, arena.data_ptr(), arena.numel(), T.TENT_FLAG_SKIP_OVERLAP_CHECK, max_rails)
    try:
        T.tent_register_segment(ctx, src.data_ptr(), pool)
        T.tent_register_segment(ctx, dst.data_ptr(), pool)

        def batch(n):
            ptr = np.arange(n + 1, dtype=np.uint32)
            se = np.zeros(n, dtype=W.tiny().src_ext.dtype)
            se["off"], se["len"], se["seg"] = np.arange(n, dtype=np.uint64) * 1024, length, W.SRC_SEG
            de = se.copy()
            de["seg"] = W.DST_SEG
            return ptr, se, ptr, de

        stream = torch.cuda.current_stream()
        h = T.tent_declare_static(ctx, *batch(n))
        st, _ = T.tent_plan(ctx, h, rails, True, stream)
        assert st == 0
        T.tent_execute(ctx, h, stream)
        assert T.tent_poll(ctx, h, stream) == 0
        rows = torch.arange(pool, device="cuda:0") % 1024 < length
        rows[n * 1024:] = False
        assert torch.equal(dst, torch.where(rows, src, torch.zeros_like(src)))
        with pytest.raises(T.TentError) as ei:
            T.tent_declare_static(ctx, *batch(n + 1))
        assert ei.value.status == T.TENT_ERR_RANGE
    finally:
        T.tent_destroy(ctx)


@pytest.mark.parametrize("n", [1, 3, 700, 1025, 2600, 4096, 4097, 6000])
@pytest.mark.parametrize("n_src", ["half", "same", "double"])
@pytest.mark.parametrize("grid", ["dense", "sparse", "any"])
def test_every_way_to_the_order(T, n, n_src, grid):
    # sources and destinations side by side in one pool, at multiples of 256 bytes that fill the pool or leave most of it, or at any
    # address: places in LDS, a sort in LDS, places in device memory, a device-wide sort; then one extent is moved by a byte
    g = np.random.Generator(np.random.PCG64([n, len(n_src), len(grid)]))
    L = 64
    k = {"half": 1, "same": 2, "double": 4}[n_src]               # sources: n k / 2 of 2 L / k bytes each
    n = n + n % 2
    ns, ls = n * k // 2, 2 * L // k
    pitch = {"dense": 256, "sparse": 256, "any": 139}[grid]
    room = (n + ns) * (40 if grid == "sparse" else 1)
    at = g.choice(room, size=n + ns, replace=False).astype(np.uint64) * np.uint64(pitch)
    if grid == "any":
        at += g.integers(0, 10, size=n + ns).astype(np.uint64)
    pool = torch.from_numpy(g.integers(0, 256, size=room * pitch + 256, dtype=np.uint8)).cuda()
    before = pool.cpu().numpy()
    arena = torch.zeros(n * L + 4096, dtype=torch.uint8, device="cuda")
    ctx = T.tent_create(1000, arena.data_ptr(), arena.numel())
    T.tent_register_segment(ctx, pool.data_ptr(), pool.numel())
    se, de = np.zeros(ns, dtype=W.EXTENT_DTYPE), np.zeros(n, dtype=W.EXTENT_DTYPE)
    se["off"], se["len"] = at[:ns], ls
    de["off"], de["len"] = at[ns:], L
    rails, stream = W.make_rails([50000, 20000, 70000]), torch.cuda.current_stream()
    sp, dp = np.array([0, ns], dtype=np.uint32), np.array([0, n], dtype=np.uint32)

    def overlaps(se, de):
        starts = np.concatenate([de["off"], se["off"]])
        order = np.lexsort((np.arange(starts.shape[0]), starts))
        far_any = far_dst = 0
        for v in order.tolist():
            a = int(starts[v])
            if a < (far_any if v < n else far_dst):
                return True
            end = a + (L if v < n else ls)
            far_any = max(far_any, end)
            far_dst = max(far_dst, end) if v < n else far_dst
        return False

    assert not overlaps(se, de)
    h = T.tent_declare(ctx, sp, se, dp, de)
    T.tent_plan(ctx, h, rails, False, stream)
    T.tent_execute(ctx, h, stream)
    assert T.tent_poll(ctx, h, stream) == 0
    want = before.copy()
    data = np.concatenate([before[a:a + ls] for a in se["off"].tolist()])
    for j, a in enumerate(de["off"].tolist()):
        want[a:a + L] = data[j * L:(j + 1) * L]
    assert np.array_equal(pool.cpu().numpy(), want)
    T.tent_release(ctx, h)
    for _ in range(12):
        s2, d2 = se.copy(), de.copy()
        i, j = int(g.integers(0, n)), int(g.integers(0, ns))
        what = int(g.integers(0, 6))
        if what == 0:
            d2["off"][i] = d2["off"][(i + 1) % n]                # two at one place
        elif what == 1:
            d2["off"][i] = s2["off"][j] + (ls - 1)               # the source's last byte
        elif what == 2:
            s2["off"][j] = d2["off"][i] + (L - 1)
        elif what == 3:
            s2["off"][j] = max(0, int(d2["off"][i]) - (ls - 1))
        elif what == 4:
            s2["off"][j] = s2["off"][(j + 1) % ns]               # two sources may share their bytes
        else:
            d2["off"][i] = max(0, int(d2["off"][(i + 1) % n]) - (L - 1))
        h = T.tent_declare(ctx, sp, s2, dp, d2)
        if overlaps(s2, d2):
            with pytest.raises(T.TentError) as err:
                T.tent_plan(ctx, h, rails, False, stream)
            assert err.value.status == T.TENT_ERR_INVALID
        else:
            T.tent_plan(ctx, h, rails, True, stream)
            T.tent_release(ctx, h)
    T.tent_destroy(ctx)
