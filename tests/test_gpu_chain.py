"""The binding chain where its short path gives way: rails far from the cost level, slots and runs that lift the level
by more than the relative state spans, slices outside the key window, more records than the ring holds, runs of a few
slices.  Rails, staging offsets and totals against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_2604_00368_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


def transfers(lens, S, rails):
    """Contiguous transfers of the given byte lengths, destinations in the same order."""
    lens = np.asarray(lens, dtype=np.uint64)
    D = lens.shape[0]
    ext = np.zeros(D, dtype=W.EXTENT_DTYPE)
    ext["len"], ext["off"] = lens, np.concatenate([[0], np.cumsum(lens)[:-1]])
    ptr = np.arange(D + 1, dtype=np.uint32)
    dst = ext.copy()
    dst["seg"] = W.DST_SEG
    total = int(lens.sum())
    return W.Workload("transfers", 0, S, [total, total], ptr, ext, ptr.copy(), dst, rails, "u8")


def check_binding(H, oracle, w):
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    b = oracle.bind(s.len, w.rails)
    assert b.status == 0
    with H.Engine(w) as eng:
        eng.declare()
        st, info = eng.plan()
        assert st == 0
        H.assert_plan_equal(eng.table(), s, b, info)
        st, info = eng.plan()                                  # the same again over a used run table
        H.assert_plan_equal(eng.table(), s, b, info)


def mixed_lengths(rng, n, S, most):
    """Whole multiples, tails of every length, transfers shorter than a slice, equal neighbours."""
    lens = rng.integers(1, most * S, size=n)
    lens[rng.random(n) < 0.15] = S * int(rng.integers(1, most))
    lens[rng.random(n) < 0.1] = int(rng.integers(1, S))
    return lens


KINDS = {
    # queues 0 .. 0.25 s apart: rails are infinitely far (2^36 ps) at first and join while the plan runs
    "queues_that_are_reached": lambda g, R: W.make_rails(g.integers(16, 40, size=R), queued=g.integers(0, 1 << 22, size=R)),
    "queues_never_reached": lambda g, R: W.make_rails(g.integers(20000, 90000, size=R),
                                                      queued=np.where(np.arange(R) % 3 == 1, 1 << 36, 0)),
    # one slice of 512 KiB costs 2^34 ps and more on some rails: no level serves
    "slots_beyond_a_step": lambda g, R: W.make_rails(np.where(np.arange(R) % 2 == 0, 16, 90)),
    # tails and single slices far outside the window of the 32-bit keys
    "wide_spread": lambda g, R: W.make_rails(np.where(np.arange(R) % 2 == 0, 400000, 20), lat_ns=g.integers(0, 1 << 20, size=R)),
    "one_fast_rail": lambda g, R: W.make_rails(np.where(np.arange(R) == R - 1, 4000000, 1000)),
    "identical": lambda g, R: W.make_rails([50000] * R),
    "degraded_and_excluded": lambda g, R: W.make_rails(g.integers(1000, 90000, size=R), queued=g.integers(0, 1 << 16, size=R),
                                                       health=np.where(np.arange(R) % 4 == 0, 0, np.arange(R) % 3)),
    "free_of_cost": lambda g, R: W.make_rails([4000000] * R, lat_ns=0, beta1_q8=1, penalty_q8=256),
}


@pytest.mark.parametrize("R", [1, 2, 9, 16, 17, 40])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_chain_against_oracle(H, oracle, kind, R):
    g = np.random.Generator(np.random.PCG64([R, len(kind)]))
    S, n = {"slots_beyond_a_step": (1 << 19, 60), "queues_that_are_reached": (4096, 700)}.get(kind, (192, 700))
    check_binding(H, oracle, transfers(mixed_lengths(g, n, S, 12), S, KINDS[kind](g, R)))


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 127, 128, 129, 300, 3000])
def test_record_ring_and_feeder_blocks(H, oracle, n):
    # two runs per transfer, 64 runs to a feeder block, 256 records to the ring
    g = np.random.Generator(np.random.PCG64(n))
    rails = W.make_rails([25000, 50000] * 8, queued=g.integers(0, 5000, size=16))
    check_binding(H, oracle, transfers(g.integers(40, 90, size=n) * 100, 1600, rails))


@pytest.mark.parametrize("case", ["singles_only", "whole_slices_only", "pairs", "alternating_slice_of_one_byte", "one_long_run"])
def test_run_shapes(H, oracle, case):
    g = np.random.Generator(np.random.PCG64(17))
    S, n = 500, 400
    lens = {"singles_only": g.integers(1, S, size=n), "whole_slices_only": S * g.integers(1, 9, size=n),
            "pairs": np.full(n, 2 * S), "alternating_slice_of_one_byte": np.where(np.arange(n) % 2 == 0, 1, 3 * S + 1),
            "one_long_run": np.array([S * 60000 + 7])}[case]
    for rails in (W.make_rails([50000] * 8 + [400000]), W.make_rails([12000, 31000, 77000], queued=[0, 40000, 9])):
        check_binding(H, oracle, transfers(lens, S, rails))


@pytest.mark.parametrize("n", [1, 2, 3, 2046, 2047, 2048, 2049])
@pytest.mark.parametrize("what", ["transfers", "slices", "tiles"])
def test_plan_in_one_workgroup_and_beyond(H, oracle, n, what):
    # one workgroup plans up to 2048 extents a side, 2048 slices and 16384 tiles
    g = np.random.Generator(np.random.PCG64([n, len(what)]))
    rails = W.make_rails([25000, 50000, 40000, 10000], queued=g.integers(0, 5000, size=4))
    if what == "transfers":
        check_binding(H, oracle, transfers(g.integers(1, 900, size=n), 1 << 20, rails))      # a slice each
    elif what == "slices":
        check_binding(H, oracle, transfers([700 * (n // 2) + 1] * (2 if n > 1 else 1), 700, rails))
    else:
        check_binding(H, oracle, transfers([8 * 1024 * n - 1024 * (n > 2)], 8 * 1024, rails))


@pytest.mark.parametrize("n", [2049, 3071, 3072, 3073, 4095, 4096, 4097])
@pytest.mark.parametrize("what", ["extents", "slices", "transfers", "dispatch"])
def test_front_part_in_one_workgroup_and_beyond(H, oracle, n, what):
    # one workgroup writes the slice table of up to 4096 extents a side, 2048 transfers and 2048 slices (3072 with up to 2048 extents)
    from paper_2604_00368_amd import binding as T
    g = np.random.Generator(np.random.PCG64([n, len(what)]))
    rails = W.make_rails([25000, 50000, 40000, 10000], queued=g.integers(0, 5000, size=4))
    if what == "slices":
        return check_binding(H, oracle, transfers([1024 * (n // 3) - 5, 1024 * (n // 3), 1024 * (n - 2 * (n // 3))], 1024, rails))
    if what == "transfers":
        return check_binding(H, oracle, transfers(g.integers(1, 5000, size=n // 2), 4096, rails))
    # transfers of several extents, cut differently on either side; whole tiles or not
    for unit in (1024, 1000):
        sizes = unit * g.integers(1, 9, size=n)
        starts = np.unique(np.concatenate([[0], g.integers(1, n, size=60)]))
        w = transfers(sizes, 16384, rails)
        w.src_ptr = np.append(starts, n).astype(np.uint32)
        merged = np.add.reduceat(sizes, starts)
        w.dst_ext = w.dst_ext[:len(starts)].copy()
        w.dst_ext["len"], w.dst_ext["off"] = merged, np.concatenate([[0], np.cumsum(merged)[:-1]])
        w.dst_ptr = np.arange(len(starts) + 1, dtype=np.uint32)
        if what == "extents":
            check_binding(H, oracle, w)
            continue
        s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
        dp = W.make_dispatch_params(1 << 15)
        r = oracle.dispatch(s, w.rails, dp)
        with H.Engine(w) as eng:
            eng.declare()
            assert T.tent_plan_dispatch(eng.ctx, eng.batch, w.rails, dp, None, True, eng.stream)[0] == 0
            H.assert_plan_equal(eng.table(), s, r.binding)


def stretches(g, S, n, singles, equal):
    """Stretches of `equal` transfers of whole slices and a tail, `singles` transfers shorter than a slice, and one whose
    slices are short (a run of its own slice length when repeated) in turn."""
    lens = []
    while len(lens) < n:
        lens += (S * g.integers(1, 60, size=equal) + g.integers(1, S, size=equal)).tolist()
        lens += g.integers(1, S, size=singles).tolist()
        lens += [int(g.integers(1, S))] * int(g.integers(0, 6))
    return np.array(lens[:n])


@pytest.mark.parametrize("singles,equal", [(0, 70), (1, 3), (1, 4), (3, 5), (4, 2), (40, 9), (70, 1)])
@pytest.mark.parametrize("kind", ["two_speeds", "one_rail_of_half", "equal_idle", "around_the_window", "five_live"])
def test_ways_of_taking_a_record(H, oracle, kind, singles, equal):
    # up to 16 rails the chain takes stretches of equal slices four at a time, other runs and single slices one by one, and
    # changes the way at the ends of stretches; keys cover 134 us on either side of the level
    g = np.random.Generator(np.random.PCG64([singles, equal, len(kind)]))
    S = 1 << 20 if kind == "around_the_window" else 16384
    rails = {"two_speeds": lambda: W.make_rails([25000, 50000] * 8, queued=g.integers(0, 1 << 18, size=16)),
             "one_rail_of_half": lambda: W.make_rails([50000] * 8 + [400000], queued=g.integers(0, 1 << 18, size=9)),
             "equal_idle": lambda: W.make_rails([65536] * 16),
             # a slice costs 52, 84, 105, 131, 140 us: some runs fit the window and some do not
             "around_the_window": lambda: W.make_rails([20000, 12500, 10000, 8000, 7500][:2 + (singles + equal) % 4]),
             "five_live": lambda: W.make_rails(g.integers(10000, 400000, size=6), lat_ns=g.integers(0, 20000, size=6),
                                               health=[0, 1, 2, 0, 0, 0])}[kind]()
    check_binding(H, oracle, transfers(stretches(g, S, 500 if S < 1 << 20 else 60, singles, equal), S, rails))


# A run of slices much shorter than the last one meets rails that the longer one has left far apart: the guess of its split is
# too high, the dearest slots are dropped again and some rail's next slot ends more than 134 us below the level.  The
# slice behind the run must still go where it costs least.
DROPPED = {
    # three rails of 25 GB/s: 451 us on one of them, two slices of 35 us, one of 40 ns, which belongs on rail 2
    "behind_one_slice": (16 << 20, [11287500, 875000, 875000, 1000], dict(bw_MBps=[25000] * 3, queued=[0, 1000, 0]), [0, 2, 1, 2]),
    "behind_a_run": (5600000, [5600000] * 2 + [440000] * 2 + [10000],
                     dict(bw_MBps=[10000] * 3, lat_ns=0, queued=[0, 5700000, 5605000]), [0, 0, 2, 1, 2]),
    # three slots to drop, of which the second ends beyond the window too, where the rail without a slot looks alike
    "beyond_the_window": (8000000, [3000000] + [50000] * 3, dict(bw_MBps=[2000, 10000], lat_ns=0, queued=[500000, 2700000]), [1, 0, 0, 0]),
}


@pytest.mark.parametrize("case", sorted(DROPPED))
def test_slice_behind_dropped_slots(H, oracle, case):
    S, lens, rails, want = DROPPED[case]
    w = transfers(lens, S, W.make_rails(**rails))
    assert oracle.bind(oracle.split(w.src_ptr, w.src_ext, S).len, w.rails).rail.tolist() == want
    check_binding(H, oracle, w)


@pytest.mark.parametrize("R", [2, 3, 5, 8])
@pytest.mark.parametrize("singles", [1, 3, 4])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_slices_behind_runs_of_dropped_slots(H, oracle, R, singles, seed):
    # the same at random, over and over: a long slice or two, 2 - 8 equal ones of 20 - 60 us, then a few short ones, of which the
    # first goes with the run and up to three more as runs of none
    g = np.random.Generator(np.random.PCG64([R, singles, seed]))
    S, bw = 16 << 20, g.integers(12500, 50001, size=R) if seed else np.full(R, 25000)
    lens = []
    for _ in range(24):
        lens += [int(g.integers(1 << 20, S))] * int(g.integers(1, 3))
        lens += [int(g.integers(20, 61) * bw.mean())] * int(g.integers(2, 9))
        lens += g.permutation(np.arange(1, 40))[:singles].tolist()
    check_binding(H, oracle, transfers(lens, S, W.make_rails(bw, queued=g.integers(0, 1 << 20, size=R))))


@pytest.mark.parametrize("row", [1, 3, 5, 6, 7])
@pytest.mark.parametrize("longest", [1.0, 2.0, 9.0])
@pytest.mark.parametrize("runs", ["first", "alike"])
def test_rows_of_single_slices_behind_short_runs(H, oracle, row, longest, runs):
    # rows of up to six go as runs of none where runs of one slice length stand around them; not behind the first run of a length, and
    # not if they are longer than two of its slices
    g = np.random.Generator(np.random.PCG64([row, int(longest), len(runs)]))
    S, lens = 400000, []
    for _ in range(40):
        if runs == "first":
            lens += (S * g.integers(1, 4, size=2)).tolist()
        l = 7000 if runs == "alike" else int(g.integers(5000, 9001))
        lens += [l] * int(g.integers(2, 5)) + g.integers(1, int(longest * l) + 1, size=row).tolist()
    rails = W.make_rails(g.integers(10000, 90000, size=8), queued=g.integers(0, 1 << 18, size=8))
    check_binding(H, oracle, transfers(lens, S, rails))


@pytest.mark.parametrize("at", [1, 2, 3, 4, 5, 60, 61, 62, 63, 64])
@pytest.mark.parametrize("n", [6, 65, 131])
def test_a_slice_outside_the_window_among_single_slices(H, oracle, at, n):
    # single slices are bound four to a check: one that costs 160 us and more lies outside the keys' window wherever it stands among them
    g = np.random.Generator(np.random.PCG64([at, n]))
    rails = W.make_rails([25000, 12500, 20000], queued=g.integers(0, 1 << 16, size=3))
    lens = g.integers(1, 200000, size=n)
    lens[at % n::64] = 4000000 + at
    check_binding(H, oracle, transfers(lens, 1 << 22, rails))


@pytest.mark.parametrize("row", [1, 2, 3, 5, 64])
@pytest.mark.parametrize("between", [0, 1, 4, 5])
def test_slices_outside_the_window_in_a_row(H, oracle, row, between):
    # the first of a row of single slices has a check of its own, the next four share one; each row here begins with slices outside
    g = np.random.Generator(np.random.PCG64([row, between]))
    rails = W.make_rails([25000, 12500, 20000], queued=g.integers(0, 1 << 16, size=3))
    lens = []
    while len(lens) < 200:
        lens += g.integers(3500000, 4100000, size=row).tolist() + g.integers(1, 200000, size=between).tolist()
    check_binding(H, oracle, transfers(lens, 1 << 22, rails))
