"""GPU parity for the resilience path (Section 4.3): failure marking, retry rotation ahead of the cost
model, and the rail health monitor, against the CPU oracle, bit for bit."""
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


def run_resilient_and_compare(H, oracle, w, params, mp, fails, cong, flags=0, bytes_too=True, final_check=None):
    from paper_2604_00368_amd import binding as T
    R = w.rails.shape[0]
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    src = W.fill_numpy(w, 0) if bytes_too else None
    dst0 = W.fill_numpy(w, 1) if bytes_too else None
    dst_want = dst0.copy() if bytes_too else None
    staging_want = np.zeros(w.staging_bytes, dtype=np.uint8) if bytes_too else None
    recs = oracle.run_epochs_resilient(w, s, params, mp, fails, cong, [src, dst_want] if bytes_too else None,
                                       staging_want)
    eng = H.Engine(w, src, dst0, flags=flags) if bytes_too else H.Engine(w, flags=flags)
    try:
        eng.declare()
        mon = T.tent_monitor_init(mp, R)
        est = w.rails["bw_MBps"].astype(np.uint32).copy()
        health = np.zeros(R, dtype=np.uint8)
        for e, rec in enumerate(recs):
            ep = rec["epoch"]
            print("resilient window", e, "pending", rec["pending"].shape[0], "retried",
                  int((rec["retry"][rec["pending"]] > 0).sum()), "health", rec["rails"]["health"].tolist(), flush=True)
            rails = ep.rails.copy()
            rails["bw_MBps"] = est
            rails["health"] = np.where(ep.rails["health"] == 2, 2, health).astype(np.uint8)
            assert np.array_equal(rails, rec["rails"])
            assert np.array_equal(T.tent_get_retries(eng.ctx, eng.batch), rec["retry"])
            hard = np.zeros(R, dtype=np.uint32)
            probe = np.zeros(R, dtype=np.uint32)
            if rec["pending"].shape[0]:
                st, info = eng.plan(rails=rails)
                assert st == rec["status"]
            else:
                st = -99
            if st == 0:
                pend = rec["pending"]
                assert info.n_slices == pend.shape[0]
                tab = eng.table()
                assert np.array_equal(np.nonzero(tab["state"] != 2)[0], pend)
                assert np.array_equal(tab["rail"][pend], rec["rail"])
                assert np.array_equal(tab["stage_off"][pend], rec["stage_off"])
                assert list(info.rail_bytes)[:R] == rec["T"].tolist()
                assert list(info.rail_slices)[:R] == rec["n_slices"].tolist()
                assert list(info.queued_after)[:R] == rec["A_after"].tolist()
                assert list(info.stage_base)[:R] == rec["base"].tolist()
                fl = fails[e] if e < len(fails) else np.zeros(R, dtype=np.uint8)
                per_rail = T.tent_sim_fail(eng.ctx, eng.batch, fl, True, eng.stream)
                assert np.array_equal(per_rail, rec["failed_per_rail"])
                hard = np.minimum(per_rail, 0xFFFFFFFF).astype(np.uint32)
                n_done = T.tent_sim_advance(eng.ctx, eng.batch, ep.budget, eng.stream)
                assert n_done == rec["done_ids"].shape[0]
                tab = eng.table()
                assert np.array_equal(np.nonzero(tab["state"] == 1)[0], rec["done_ids"])
                T.tent_sim_latency(eng.ctx, eng.batch, ep.rails["bw_MBps"], eng.stream)
                new_rails, probe = T.tent_update_bandwidth(eng.ctx, eng.batch, params, rails, eng.stream)
                assert np.array_equal(probe, rec["probe"])
                tau = T.tent_get_latencies(eng.ctx, eng.batch)
                assert np.array_equal(tau[rec["done_ids"]], rec["tau"])
                eng.execute()
                est_before = est
                est = new_rails["bw_MBps"].astype(np.uint32)
            else:
                est_before = est
            assert np.array_equal(est, rec["est_after"])
            cg = cong[e] if e < len(cong) else np.zeros(R, dtype=np.uint32)
            out = T.tent_monitor_update(mp, mon, rails, hard, cg, probe, est_before)
            for f in mon.dtype.names:
                assert np.array_equal(mon[f], rec["mon_after"][f]), f
            health = out["health"].copy()
            assert np.array_equal(health, rec["mon_after"]["state"].astype(np.uint8))
            assert np.array_equal(T.tent_get_retries(eng.ctx, eng.batch), rec["retry_after"])
        assert T.tent_poll(eng.ctx, eng.batch, eng.stream) == 0
        if bytes_too:
            assert np.array_equal(eng.dst.cpu().numpy(), dst_want)
            assert np.array_equal(eng.arena.cpu().numpy(), staging_want)
        if final_check is not None:
            final_check(eng)
    finally:
        eng.close()
    return recs


@pytest.mark.parametrize("seed", [5, 6])
def test_faulty_rails_closed_loop_bit_exact(H, oracle, seed):
    from paper_2604_00368_amd import binding as T
    w = W.replanning(n_req=6, layers=4, ctx_lo=400, ctx_hi=2000, queued_hi=1 << 20)
    R = w.rails.shape[0]
    params = W.make_probe_params(2 * w.rails["bw_MBps"].astype(np.uint64), ewma_q8=128)
    fails, cong = W.failure_schedule(seed, len(w.epochs), R)
    recs = run_resilient_and_compare(H, oracle, w, params, W.make_monitor_params(), fails, cong)
    assert any((r["retry"][r["pending"]] > 0).any() for r in recs)
    if seed == 5:
        run_resilient_and_compare(H, oracle, w, params, W.make_monitor_params(), fails, cong,
                                  flags=T.TENT_FLAG_SERIAL_BINDING)


def test_everything_fails_at_once(H, oracle):
    # every rail reports a hard error in the first window: the whole batch is retried by rotation, the
    # cost-model pass has nothing left to bind, and the rails are paused for a window
    w = W.small_variant("kv_migration")
    R = w.rails.shape[0]
    w.epochs = [W.Epoch(w.rails.copy(), np.full(R, np.iinfo(np.uint64).max, dtype=np.uint64)) for _ in range(2)]
    w.drain = w.epochs[0]
    params = W.make_probe_params(2 * w.rails["bw_MBps"].astype(np.uint64))
    fails = np.zeros((2, R), dtype=np.uint8)
    fails[0, :] = 1
    cong = np.zeros((2, R), dtype=np.uint32)
    mp = W.make_monitor_params(err_threshold=2, cooldown_windows=0)       # zero-length pause: straight to DEGRADED
    recs = run_resilient_and_compare(H, oracle, w, params, mp, fails, cong)
    assert (recs[1]["retry"] == 1).all() and (recs[1]["rails"]["health"] == 1).all()
    mp = W.make_monitor_params(err_threshold=2, cooldown_windows=1)       # one window with every rail paused: deferred
    recs = run_resilient_and_compare(H, oracle, w, params, mp, fails, cong)
    assert recs[1]["status"] == 1


def test_many_small_retries_span_rotation_chunks(H, oracle):
    # enough retried slices of mixed lengths for several rotation workgroups, 16 rails, no byte movement
    w = W.many_small(n_req=640)
    R = w.rails.shape[0]
    rng = np.random.Generator(np.random.PCG64(31))
    epochs = []
    t_us = -(-w.payload // int(4 * int(w.rails["bw_MBps"].astype(np.uint64).sum())))
    for e in range(5):
        bw = np.maximum(1, np.rint(w.rails["bw_MBps"] * np.exp(0.3 * rng.standard_normal(R)))).astype(np.uint64)
        rails = W.make_rails(bw, queued=rng.integers(0, 1 << 20, size=R),
                             penalty_q8=rng.choice([256, 256, 320], size=R))
        epochs.append(W.Epoch(rails, bw * np.uint64(t_us)))
    w.epochs = epochs
    w.drain = W.Epoch(epochs[-1].rails.copy(), np.full(R, np.iinfo(np.uint64).max, dtype=np.uint64))
    params = W.make_probe_params(2 * w.rails["bw_MBps"].astype(np.uint64), ewma_q8=64)
    fails, cong = W.failure_schedule(9, len(epochs), R, p_fail=0.3)
    recs = run_resilient_and_compare(H, oracle, w, params, W.make_monitor_params(err_threshold=4), fails, cong,
                                     bytes_too=False)
    assert max(int((r["retry"][r["pending"]] > 0).sum()) for r in recs) > 2 * 1024


def test_fail_argument_errors(H, oracle):
    from paper_2604_00368_amd import binding as T
    w = W.tiny()
    with H.Engine(w, W.fill_numpy(w, 0), W.fill_numpy(w, 1)) as eng:
        h = eng.declare()
        with pytest.raises(T.TentError) as ei:
            T.tent_sim_fail(eng.ctx, h, np.zeros(4, dtype=np.uint8))
        assert ei.value.status == T.TENT_ERR_STATE
        assert not T.tent_get_retries(eng.ctx, h).any()
        eng.plan()
        assert T.tent_sim_fail(eng.ctx, h, np.zeros(4, dtype=np.uint8)).tolist() == [0, 0, 0, 0]
        counts = T.tent_sim_fail(eng.ctx, h, np.array([0, 0, 1, 0], dtype=np.uint8))
        tab = eng.table()
        assert counts.tolist() == [0, 0, int(((tab["rail"] == 2)).sum()), 0]
        assert np.array_equal(T.tent_get_retries(eng.ctx, h), (tab["rail"] == 2).astype(np.uint8))
        T.tent_reset(eng.ctx, h, eng.stream)                      # reset forgets the retry counts
        assert not T.tent_get_retries(eng.ctx, h).any()
        s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
        st, info = eng.plan()
        H.assert_plan_equal(eng.table(), s, oracle.bind(s.len, w.rails), info)


@pytest.mark.parametrize("kind", range(6))
def test_randomized_rotation_and_dispatch_plans(H, oracle, kind):
    # plan-only, degenerate telemetry (ties, sub-picosecond cost steps, huge latencies and queues, 1-byte slices):
    # request-level dispatch over three windows, then rounds of failures re-planned by rotation + cost model
    from paper_2604_00368_amd import binding as T
    from test_gpu_parity import _runs_workload
    rng = np.random.Generator(np.random.PCG64(5000 + kind))
    for trial in range(15):
        w = _runs_workload(rng, kind)
        R = w.rails.shape[0]
        s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
        print("random plans kind", kind, "trial", trial, "S", w.slice_bytes, "D", w.n_desc, "N", s.n, "R", R, flush=True)
        zeros = (np.zeros(w.seg_bytes[0], np.uint8), np.zeros(w.seg_bytes[1], np.uint8))
        with H.Engine(w, *zeros) as eng:
            eng.declare()
            prio = W.make_priorities(int(rng.integers(0, 1 << 30)), w.n_desc)
            done = np.zeros(s.n, dtype=np.uint8)
            rr = int(rng.integers(0, 7))
            theta = int(rng.choice([1, w.slice_bytes, 3 * w.slice_bytes + 1, 50 * w.slice_bytes]))
            gamma = int(rng.choice([0, 3, 26, 256, 5000]))
            w0 = int(rng.integers(0, 9))
            for window in range(w0, w0 + 3):
                dp = W.make_dispatch_params(theta, gamma_q8=gamma, window=window, rr_start=rr)
                st, info = T.tent_plan_dispatch(eng.ctx, eng.batch, w.rails, dp, prio, True, eng.stream)
                r = oracle.dispatch(s, w.rails, dp, priority=prio, done=done)
                tab = eng.table()
                ids = np.flatnonzero(r.bound)
                assert np.array_equal(np.flatnonzero(tab["state"] == 1), ids)
                assert np.array_equal(tab["rail"][ids], r.binding.rail[ids])
                assert np.array_equal(tab["stage_off"][ids], r.binding.stage_off[ids])
                assert list(info.plan.rail_bytes)[:R] == r.binding.T.tolist()
                assert np.array_equal(T.tent_get_modes(eng.ctx, eng.batch, w.n_desc), r.mode)
                assert info.rr_next == r.rr_end
                rr = r.rr_end
                eng.execute()
                done[ids] = 1
        with H.Engine(w, *zeros) as eng:
            eng.declare()
            eng.plan()
            b = oracle.bind(s.len, w.rails)
            retry = np.zeros(s.n, dtype=np.uint8)
            pending = np.arange(s.n, dtype=np.uint32)
            rails = w.rails.copy()
            for rnd in range(3):
                fl = (rng.random(R) < 0.4).astype(np.uint8)
                failed, per = oracle.fail(b, fl, retry, ids=pending)
                assert np.array_equal(T.tent_sim_fail(eng.ctx, eng.batch, fl, True, eng.stream), per)
                eng.execute()                                  # the survivors complete
                pending = np.ascontiguousarray(pending[failed.astype(bool)])
                if pending.shape[0] == 0:
                    break
                u = rng.random(R)
                rails["health"] = np.where(u < 0.25, 2, np.where(u < 0.5, 1, 0)).astype(np.uint8)
                if (rails["health"] == 2).all():
                    rails["health"][int(rng.integers(0, R))] = int(rng.integers(0, 2))
                if kind == 3:
                    rails["penalty_q8"] = np.minimum(rails["penalty_q8"], 500)
                b = oracle.plan(s.len, retry, rails, ids=pending)
                st, info = eng.plan(rails=rails)
                tab = eng.table()
                assert st == b.status == 0
                assert np.array_equal(np.flatnonzero(tab["state"] != 2), pending)
                assert np.array_equal(tab["rail"][pending], b.rail[pending])
                assert np.array_equal(tab["stage_off"][pending], b.stage_off[pending])
                assert list(info.rail_bytes)[:R] == b.T.tolist()
                assert np.array_equal(T.tent_get_retries(eng.ctx, eng.batch), retry)


@pytest.mark.parametrize("R", [1, 17, 33, 64])
def test_rotation_with_many_rails(H, oracle, R):
    # every reduction width of the binders (16 / 32 / 64 lanes) behind a rotation pass; rail R-1 stays healthy
    from paper_2604_00368_amd import binding as T
    rng = np.random.Generator(np.random.PCG64(40 + R))
    w = W.small_variant("many_small")
    w.rails = W.make_rails(rng.integers(5000, 100000, R), queued=rng.integers(0, 1 << 20, R))
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    zeros = (np.zeros(w.seg_bytes[0], np.uint8), np.zeros(w.seg_bytes[1], np.uint8))
    with H.Engine(w, *zeros) as eng:
        eng.declare()
        st, _ = eng.plan()
        b = oracle.bind(s.len, w.rails)
        retry = np.zeros(s.n, dtype=np.uint8)
        fl = (rng.random(R) < 0.5).astype(np.uint8)
        fl[0] = 1
        failed, per = oracle.fail(b, fl, retry)
        assert np.array_equal(T.tent_sim_fail(eng.ctx, eng.batch, fl, True, eng.stream), per)
        rails = w.rails.copy()
        rails["health"] = np.where(fl == 1, rng.choice([1, 2], R), 0).astype(np.uint8)
        rails["health"][R - 1] = 0 if R > 1 else 1
        pending = np.arange(s.n, dtype=np.uint32)               # nothing was executed: everything is re-planned
        b2 = oracle.plan(s.len, retry, rails, ids=pending)
        st, info = eng.plan(rails=rails)
        assert st == b2.status == 0 and info.n_slices == s.n
        tab = eng.table()
        assert np.array_equal(tab["rail"], b2.rail) and np.array_equal(tab["stage_off"], b2.stage_off)
        assert list(info.rail_bytes)[:R] == b2.T.tolist() and list(info.stage_base)[:R] == b2.base.tolist()
        assert list(info.rail_slices)[:R] == b2.n_slices.tolist()
        assert int((retry > 0).sum()) == int(per.sum()) > 0


@pytest.mark.parametrize("n", [1, 8, 2047, 2048, 2049, 6145, 256 * 2048 + 2049, 2048 * 2048, 2048 * 2048 + 2049])
def test_lists_of_a_replan_at_the_edges_of_their_tiles(H, oracle, n):
    # 8 slices to a thread, 2048 to a tile, 256 tiles to a row, a spine beyond 2048 tiles: what every rail drained in half its bytes is
    # done, which empties the first tiles; one rail's slices are retried; equal and unequal lengths meet across tiles
    from paper_2604_00368_amd import binding as T
    from test_gpu_chain import transfers
    S = 64
    rng = np.random.Generator(np.random.PCG64(n))
    count = np.minimum(rng.integers(1, 80, size=n), 1 + rng.integers(0, 4000, size=n) // 40)
    count = count[:np.searchsorted(np.cumsum(count), n) + 1]
    count[-1] -= int(count.sum()) - n
    lens = count * S - np.where(rng.random(count.shape[0]) < 0.5, 0, rng.integers(0, S, size=count.shape[0]))
    w = transfers(lens, S, W.make_rails([20000, 50000, 35000, 80000, 50000], queued=rng.integers(0, 4096, 5)))
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    assert s.n == n
    with H.Engine(w) as eng:
        eng.declare()
        st, info = eng.plan()
        for rnd in range(4):
            T.tent_sim_fail(eng.ctx, eng.batch, np.array([0, rnd == 1, rnd == 0, 0, rnd < 2], dtype=np.uint8), True, eng.stream)
            half = np.array(list(info.rail_bytes)[:5], dtype=np.uint64) // np.uint64(2)
            T.tent_sim_advance(eng.ctx, eng.batch, w.rails["queued_bytes"] + half, eng.stream)
            eng.execute()
            pending = np.flatnonzero(eng.table()["state"] != 2).astype(np.uint32)
            assert 0 < pending.shape[0] and (n < 2047 or pending.shape[0] < n)
            b = oracle.plan(s.len, T.tent_get_retries(eng.ctx, eng.batch), w.rails, ids=pending)
            st, info = eng.plan()
            tab = eng.table()
            assert info.n_slices == pending.shape[0]
            assert np.array_equal(tab["rail"][pending], b.rail[pending])
            assert np.array_equal(tab["stage_off"][pending], b.stage_off[pending])
            assert list(info.rail_bytes)[:5] == b.T.tolist()
            assert list(info.rail_slices)[:5] == b.n_slices.tolist()


@pytest.mark.parametrize("n", [1, 255, 256, 257, 2047, 2048, 2049])
@pytest.mark.parametrize("R", [3, 64])
def test_rotation_of_everything_in_one_launch_and_beyond(H, oracle, n, R):
    # chunks of 256 retried slices; up to 2048 slices one workgroup takes them all
    from paper_2604_00368_amd import binding as T
    from test_gpu_chain import transfers
    S = 64
    rng = np.random.Generator(np.random.PCG64([n, R]))
    w = transfers([S * (n // 2) + 1, S * (n - n // 2 - 1) - 3] if n > 2 else [S * n], S, W.make_rails(rng.integers(20000, 90000, R)))
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    assert s.n == n
    with H.Engine(w) as eng:
        eng.declare()
        assert eng.plan()[0] == 0
        for _ in range(2):
            T.tent_sim_fail(eng.ctx, eng.batch, np.ones(R, dtype=np.uint8), True, eng.stream)
            b = oracle.plan(s.len, T.tent_get_retries(eng.ctx, eng.batch), w.rails, ids=np.arange(n, dtype=np.uint32))
            st, info = eng.plan()
            assert st == 0
            H.assert_plan_equal(eng.table(), s, b, info)
