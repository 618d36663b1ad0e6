"""GPU parity for the request-level dispatch (Algorithm 1: QoS admission, mice round robin, weighted
spraying of elephants) against the CPU oracle, bit for bit."""
import numpy as np
import pytest

from paper_2604_00368_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KiB = 1 << 10


@pytest.fixture(scope="module")
def H():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


def contiguous_requests(lens, S, rails, seed):
    """Contiguous transfers of the given lengths; destination order shuffled."""
    lens = np.asarray(lens, dtype=np.uint64)
    D = lens.shape[0]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    ptr = np.arange(D + 1, dtype=np.uint32)
    se = np.zeros(D, dtype=W.EXTENT_DTYPE)
    se["seg"], se["len"], se["off"] = W.SRC_SEG, lens, off[:-1]
    order = np.random.Generator(np.random.PCG64(seed)).permutation(D)
    doff = np.zeros(D, dtype=np.uint64)
    doff[order] = np.concatenate([[0], np.cumsum(lens[order])])[:-1]
    de = se.copy()
    de["seg"], de["off"] = W.DST_SEG, doff
    total = int(off[-1])
    return W.Workload("requests", seed, S, [total, total], ptr, se, ptr.copy(), de, rails, "u8")


def dispatch_windows_and_compare(H, oracle, w, theta, gamma_q8, prio, windows, flags=0, bytes_too=True, rr_start=0,
                                 final_check=None):
    """Dispatch the batch window after window (deferred transfers wait for a window that admits them), moving
    what was dealt after every window; everything is compared with the oracle."""
    from paper_2604_00368_amd import binding as T
    R = w.rails.shape[0]
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    src = W.fill_numpy(w, 0) if bytes_too else None
    dst0 = W.fill_numpy(w, 1) if bytes_too else None
    dst_want = dst0.copy() if bytes_too else None
    staging_want = np.zeros(w.staging_bytes, dtype=np.uint8) if bytes_too else None
    eng = H.Engine(w, src, dst0, flags=flags) if bytes_too else H.Engine(w, flags=flags)
    try:
        eng.declare()
        done = np.zeros(s.n, dtype=np.uint8)
        rr = rr_start
        seen_modes = set()
        for window in windows:
            dp = W.make_dispatch_params(theta, gamma_q8=gamma_q8, window=window, rr_start=rr)
            r = oracle.dispatch(s, w.rails, dp, priority=prio, done=done)
            print("dispatch window", window, "pending", int((done == 0).sum()), "dealt", int(r.bound.sum()),
                  "modes", np.bincount(r.mode, minlength=4).tolist(), flush=True)
            st, info = T.tent_plan_dispatch(eng.ctx, eng.batch, w.rails, dp, prio, True, eng.stream)
            assert st == r.binding.status == 0
            tab = eng.table()
            assert np.array_equal(tab["desc"], s.desc) and np.array_equal(tab["len"], s.len)
            ids = np.flatnonzero(r.bound)
            assert np.array_equal(np.flatnonzero(tab["state"] == 1), ids)
            assert np.array_equal(np.flatnonzero(tab["state"] == 2), np.flatnonzero(done))
            assert np.array_equal(tab["rail"][ids], r.binding.rail[ids])
            assert np.array_equal(tab["stage_off"][ids], r.binding.stage_off[ids])
            assert np.array_equal(T.tent_get_modes(eng.ctx, eng.batch, w.n_desc), r.mode)
            b = r.binding
            assert list(info.plan.rail_bytes)[:R] == b.T.tolist()
            assert list(info.plan.rail_slices)[:R] == b.n_slices.tolist()
            assert list(info.plan.queued_after)[:R] == b.A_after.tolist()
            assert list(info.plan.stage_base)[:R] == b.base.tolist()
            assert info.plan.n_slices == ids.shape[0]
            assert (info.n_mice, info.n_elephant, info.n_deferred) == tuple(int((r.mode == k).sum()) for k in (1, 2, 3))
            assert info.rr_next == r.rr_end
            rr = r.rr_end
            seen_modes.update(np.unique(r.mode).tolist())
            if bytes_too and ids.shape[0]:
                oracle.execute(w, s, b, [src, dst_want], staging_want, ids=np.ascontiguousarray(ids.astype(np.uint32)))
            eng.execute()
            done[ids] = 1
            assert T.tent_poll(eng.ctx, eng.batch, eng.stream) == int((done == 0).sum())
            if bytes_too:
                assert np.array_equal(eng.dst.cpu().numpy(), dst_want)
                assert np.array_equal(eng.arena.cpu().numpy(), staging_want)
        if final_check is not None:
            final_check(eng, done)
        return done, seen_modes
    finally:
        eng.close()


@pytest.mark.parametrize("seed", range(6))
def test_random_requests_bit_exact(H, oracle, seed):
    rng = np.random.Generator(np.random.PCG64(700 + seed))
    R = int(rng.choice([1, 3, 9, 16, 40, 64]))
    S = int(rng.choice([4 * KiB, 64 * KiB]))
    D = int(rng.integers(20, 200))
    lens = np.where(rng.random(D) < 0.5, rng.integers(1, 3 * S, D), rng.integers(1, 120 * S, D))
    rails = W.make_rails(rng.integers(1000, 400000, R), lat_ns=rng.integers(0, 20000, R),
                         queued=rng.integers(0, 1 << 22, R), health=rng.choice([0, 0, 0, 1, 2], R),
                         penalty_q8=rng.choice([256, 256, 384], R))
    rails["health"][int(rng.integers(0, R))] = 0
    if seed == 3:                                              # identical idle rails: every cost ties
        rails = W.make_rails([50000] * R)
    w = contiguous_requests(lens, S, rails, seed)
    prio = W.make_priorities(seed, D)
    done, modes = dispatch_windows_and_compare(H, oracle, w, theta=int(rng.choice([S, 2 * S, 8 * S])),
                                               gamma_q8=int(rng.choice([0, 26, 128, 1000])), prio=prio,
                                               windows=[5, 6, 7, 8, 9, 10], rr_start=int(rng.integers(0, 5)))
    assert {1, 2} <= modes
    if R >= 3 and (rails["health"][:3] != 2).all():
        assert done.all()


@pytest.mark.parametrize("name", ["tiny", "kv_migration", "rl_params", "many_small"])
def test_small_configs_dispatch_bit_exact(H, oracle, name):
    w = W.small_variant(name)
    prio = W.make_priorities(11, w.n_desc)
    done, modes = dispatch_windows_and_compare(H, oracle, w, theta=4 * w.slice_bytes, gamma_q8=26, prio=prio,
                                               windows=[0, 1, 2])
    assert done.all()


@pytest.mark.parametrize("D", [1, 63, 64, 65, 129])
@pytest.mark.parametrize("kind", ["mixed", "alike", "one fast", "far"])
def test_request_chain_at_its_block_edges(H, oracle, D, kind):
    # blocks of 64 requests; rails that move in step (exact ties), one that takes several slots while the others take one, and costs
    # too large for the chain of up to 16 rails, which go through that of any width
    rng = np.random.Generator(np.random.PCG64(D))
    S = 64 * KiB
    if kind == "mixed":
        rails = W.make_rails(rng.integers(10000, 400000, 5), queued=rng.integers(0, 1 << 22, 5))
    elif kind == "alike":
        rails = W.make_rails([50000] * 16)
    elif kind == "one fast":
        rails = W.make_rails([50000] * 8 + [400000], queued=rng.integers(0, 1 << 18, 9))
    else:
        rails = W.make_rails(rng.integers(10000, 400000, 5), lat_ns=[1 << 31, 5000, 1 << 30, 1 << 31, 0], penalty_q8=[65535, 256, 65535, 65535, 256])
    lens = np.where(rng.random(D) < 0.3, rng.integers(1, 4 * S, D), rng.integers(1, 80 * S, D))
    w = contiguous_requests(lens, S, rails, D)
    dispatch_windows_and_compare(H, oracle, w, theta=4 * S, gamma_q8=64, prio=W.make_priorities(D, D), windows=[0, 1, 2],
                                 bytes_too=False, rr_start=(1 << 40) + 5)


def largest_cost(rails, payload):
    """What a rail's cost can reach in a plan of `payload` bytes, ps."""
    c1 = [10**6 * int(r["beta1_q8"]) * int(r["penalty_q8"]) // int(r["bw_MBps"]) for r in rails]
    return max((int(r["lat_ns"]) * 1000 * int(r["penalty_q8"]) >> 8) + ((int(r["queued_bytes"]) + payload) * c >> 16) for r, c in zip(rails, c1))


def dispatch_and_compare(H, oracle, w, dp):
    from paper_2604_00368_amd import binding as T
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    r = oracle.dispatch(s, w.rails, dp)
    with H.Engine(w) as eng:
        eng.declare()
        st, info = T.tent_plan_dispatch(eng.ctx, eng.batch, w.rails, dp, None, True, eng.stream)
        assert st == r.binding.status == 0
        tab = eng.table()
        assert np.array_equal(tab["rail"], r.binding.rail) and np.array_equal(tab["stage_off"], r.binding.stage_off)
        assert list(info.plan.rail_slices)[:w.rails.shape[0]] == r.binding.n_slices.tolist()
        assert info.rr_next == r.rr_end


@pytest.mark.parametrize("most", [(1 << 20) - 1, 1 << 20])
@pytest.mark.parametrize("kind", ["one", "alike", "wide"])
def test_requests_of_as_many_slices_as_the_chain_takes(H, oracle, most, kind):
    # the chain of up to 16 rails guesses a rail's slots in 32-bit floats, right to within one below 2^20 slices; rails whose costs
    # are the same, and those of 370 ps and of none at all
    rails = {"one": lambda: W.make_rails([2700], lat_ns=0), "alike": lambda: W.make_rails([65536] * 16, lat_ns=300),
             "wide": lambda: W.make_rails(np.geomspace(2700, 4e6, 16).astype(np.int64), lat_ns=0)}[kind]()
    w = contiguous_requests([5, most, 1000, 3, most // 3], 1, rails, 1)
    assert largest_cost(rails, w.payload) * (most + 64) < 1 << 49
    dispatch_and_compare(H, oracle, w, W.make_dispatch_params(4, gamma_q8=64, rr_start=(1 << 64) - 1))


@pytest.mark.parametrize("over", [False, True])
@pytest.mark.parametrize("kind", ["one", "alike", "apart"])
def test_costs_as_large_as_the_chain_takes(H, oracle, over, kind):
    # ... and holds a slot's key, slots x cost x 16 + rail, in a double: up to 2^53, which the largest costs here reach but for 2 %
    bw = {"one": [50000], "alike": [50000] * 16, "apart": [50000] * 8 + [400000]}[kind]
    lens = [5, 65536, 1000, 3, 20000]
    lat = 0
    for bit in reversed(range(32)):
        if largest_cost(W.make_rails(bw, lat_ns=lat | 1 << bit), sum(lens)) * (65536 + 64) < 1 << 49:
            lat |= 1 << bit
    rails = W.make_rails(bw, lat_ns=lat + over)
    if kind == "apart":
        rails["lat_ns"][:4] //= 1000
    assert (largest_cost(rails, sum(lens)) * (65536 + 64) < 1 << 49) != over
    dispatch_and_compare(H, oracle, contiguous_requests(lens, 1, rails, 2), W.make_dispatch_params(4, gamma_q8=64, rr_start=7))


@pytest.mark.parametrize("R", [4, 20])
@pytest.mark.parametrize("D", [15, 16, 17, 2047, 2048, 2049])
def test_priorities_with_the_arguments_and_in_memory(H, oracle, D, R):
    # two bits each, sixteen to a word, for up to 2048 transfers
    rng = np.random.Generator(np.random.PCG64(D))
    S = 4 * KiB
    w = contiguous_requests(rng.integers(1, 6 * S, D), S, W.make_rails(rng.integers(10000, 400000, R)), D)
    dispatch_windows_and_compare(H, oracle, w, theta=2 * S, gamma_q8=64, prio=W.make_priorities(D, D), windows=[0, 1, 2], bytes_too=False)


def test_dispatch_then_cost_model_replan(H, oracle):
    # a window of request-level dispatch, then the per-slice planner finishes what was deferred
    from paper_2604_00368_amd import binding as T
    w = W.small_variant("kv_migration")
    w.rails = w.rails[:2].copy()                               # two rails: in window 0 nothing admits LOW
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    prio = W.make_priorities(4, w.n_desc)
    src, dst0 = W.fill_numpy(w, 0), W.fill_numpy(w, 1)
    dst_want, staging_want = dst0.copy(), np.zeros(w.staging_bytes, dtype=np.uint8)
    dp = W.make_dispatch_params(2 * w.slice_bytes, window=0)
    r = oracle.dispatch(s, w.rails, dp, priority=prio)
    assert (r.mode == 3).any()
    ids = np.flatnonzero(r.bound).astype(np.uint32)
    oracle.execute(w, s, r.binding, [src, dst_want], staging_want, ids=ids)
    rest = np.flatnonzero(r.bound == 0).astype(np.uint32)
    b2 = oracle.bind(s.len, w.rails, ids=rest)
    oracle.execute(w, s, b2, [src, dst_want], staging_want, ids=rest)
    with H.Engine(w, src, dst0) as eng:
        eng.declare()
        st, info = T.tent_plan_dispatch(eng.ctx, eng.batch, w.rails, dp, prio, True, eng.stream)
        assert st == 0 and info.n_deferred == int((r.mode == 3).sum())
        eng.execute()
        st, info2 = eng.plan()
        assert st == 0 and info2.n_slices == rest.shape[0]
        tab = eng.table()
        assert np.array_equal(tab["rail"][rest], b2.rail[rest]) and np.array_equal(tab["stage_off"][rest], b2.stage_off[rest])
        eng.execute()
        assert np.array_equal(eng.dst.cpu().numpy(), dst_want)
        assert np.array_equal(eng.arena.cpu().numpy(), staging_want)


def test_dispatch_argument_errors(H, oracle):
    from paper_2604_00368_amd import binding as T
    w = W.tiny()
    with H.Engine(w, W.fill_numpy(w, 0), W.fill_numpy(w, 1)) as eng:
        h = eng.declare()
        dp = W.make_dispatch_params(4 * w.slice_bytes)
        bad = np.zeros(w.n_desc, dtype=np.uint8); bad[3] = 3
        with pytest.raises(T.TentError) as ei:
            T.tent_plan_dispatch(eng.ctx, h, w.rails, dp, bad)
        assert ei.value.status == T.TENT_ERR_INVALID
        with pytest.raises(T.TentError) as ei:
            T.tent_plan_dispatch(eng.ctx, h, w.rails, W.make_dispatch_params(1, gamma_q8=70000))
        assert ei.value.status == T.TENT_ERR_RANGE
        huge = w.rails.copy(); huge["lat_ns"] = 0xFFFFFFFF; huge["penalty_q8"] = 65535
        with pytest.raises(T.TentError) as ei:
            T.tent_plan_dispatch(eng.ctx, h, huge, W.make_dispatch_params(1, gamma_q8=65535))
        assert ei.value.status == T.TENT_ERR_RANGE
        off = w.rails.copy(); off["health"] = 2
        st, _ = T.tent_plan_dispatch(eng.ctx, h, off, dp)
        assert st == T.TENT_DEFER
        # still usable afterwards, without priorities every transfer is HIGH
        s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
        r = oracle.dispatch(s, w.rails, dp)
        st, info = T.tent_plan_dispatch(eng.ctx, h, w.rails, dp)
        assert st == 0 and info.n_deferred == 0
        tab = eng.table()
        assert np.array_equal(tab["rail"], r.binding.rail) and np.array_equal(tab["stage_off"], r.binding.stage_off)
