"""The one-pass copies (source -> staging and destination in one launch) against the two passes they stand in for, and
the batches that must keep two passes: destinations that reuse source bytes, an arena inside a segment."""
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


def cut_tails(w, seed, most):
    """The last extent of every transfer loses up to `most` bytes on both sides."""
    rng = np.random.Generator(np.random.PCG64(seed))
    cut = rng.integers(0, most + 1, size=w.n_desc).astype(np.uint32)
    w.src_ext["len"][w.src_ptr[1:] - 1] -= cut
    w.dst_ext["len"][w.dst_ptr[1:] - 1] -= cut
    return w


LAYOUTS = {
    "tiles_4KiB": lambda: W.kv_migration(n_req=3, layers=1, ctx_lo=40, ctx_hi=400, page_tokens=16, slice_bytes=256 * KiB),
    "tiles_2KiB": lambda: W.many_small(n_req=24),
    "slice_of_many_tiles": lambda: W.sweep(8 << 20, True, payload=32 << 20, n_desc=2),
    "one_tile_slices": lambda: W.tiny(n_desc=5, slice_bytes=4 * KiB),
    "ragged_tails": lambda: cut_tails(W.many_small(n_req=24), 1, 1500),
    "tails_of_single_bytes": lambda: cut_tails(W.tiny(n_desc=9), 2, 17),
    "cut_anywhere": lambda: W.ragged(3, n_desc=20, max_len=90_000, max_ext=700, slice_bytes=16 * KiB),
    "tiny_extents": lambda: W.ragged(4, n_desc=9, max_len=4000, max_ext=3, slice_bytes=1500),
    "pieces_of_4096": lambda: W.ragged(5, n_desc=12, max_len=60_000, max_ext=40_000, slice_bytes=4 * KiB),
}


@pytest.mark.parametrize("name", sorted(LAYOUTS))
@pytest.mark.parametrize("partial", [False, True])
def test_one_pass_equals_two_passes(H, name, partial):
    from paper_2604_00368_amd import binding as T
    w = LAYOUTS[name]()
    src, dst0 = W.fill_numpy(w, 0), W.fill_numpy(w, 1)
    R = w.rails.shape[0]
    results = []
    for flags in (0, T.TENT_FLAG_SKIP_OVERLAP_CHECK):
        with H.Engine(w, src, dst0, flags=flags, arena_skew=3) as eng:
            eng.declare()
            moved = []
            for window in range(3 if partial else 1):
                st, info = eng.plan()
                assert st == 0
                if partial and window < 2:                   # a third of what is bound, then the rest
                    share = np.array(list(info.rail_bytes)[:R], dtype=np.uint64) // np.uint64(3 - window)
                    moved.append(T.tent_sim_advance(eng.ctx, eng.batch, w.rails["queued_bytes"] + share, eng.stream))
                eng.execute()
                moved.append(T.tent_poll(eng.ctx, eng.batch, eng.stream))
            assert moved[-1] == 0
            results.append((eng.dst.cpu().numpy(), eng.arena.cpu().numpy(), eng.table(), moved))
    one, two = results
    assert np.array_equal(one[0], two[0])
    assert np.array_equal(one[1], two[1])
    assert np.array_equal(one[2], two[2]) and one[3] == two[3]


@pytest.mark.parametrize("size", [32 * KiB, 1000])
def test_destinations_that_reuse_source_bytes_keep_two_passes(H, size):
    """Pages permuted in place: every source byte must be in staging before the first destination byte is written."""
    from paper_2604_00368_amd import binding as T
    dev, n = "cuda:0", 64
    perm = np.random.Generator(np.random.PCG64(7)).permutation(n)
    pool0 = np.random.Generator(np.random.PCG64(8)).integers(0, 256, size=n * size, dtype=np.uint8)
    pool = torch.from_numpy(pool0).to(dev)
    arena = torch.zeros(n * size + 256 * 4, dtype=torch.uint8, device=dev)
    src = np.zeros(n, dtype=W.EXTENT_DTYPE)
    src["off"], src["len"] = np.arange(n) * size, size
    dst = src.copy()
    dst["off"] = perm * size
    ptr = np.arange(0, n + 1, 8, dtype=np.uint32)
    ctx = T.tent_create(16 * KiB, arena.data_ptr(), arena.numel(), T.TENT_FLAG_SKIP_OVERLAP_CHECK)
    T.tent_register_segment(ctx, pool.data_ptr(), pool.numel())
    stream = torch.cuda.current_stream()
    h = T.tent_declare(ctx, ptr, src, ptr, dst)
    T.tent_plan(ctx, h, W.make_rails([50000, 25000, 40000]), False, stream)
    T.tent_execute(ctx, h, stream)
    torch.cuda.synchronize()
    want = np.empty_like(pool0)
    want.reshape(n, size)[perm] = pool0.reshape(n, size)
    assert np.array_equal(pool.cpu().numpy(), want)
    T.tent_destroy(ctx)


@pytest.mark.parametrize("chunk", [0, 1 << 20])
def test_arena_inside_a_segment(H, oracle, chunk):
    """The arena may be part of a registered range; the result is the same, in one piece and in chunks."""
    from paper_2604_00368_amd import binding as T
    w = W.small_variant("many_small")
    src_h, dst_h = W.fill_numpy(w, 0), W.fill_numpy(w, 1)
    n_arena = chunk + 256 * w.rails.shape[0] if chunk else w.staging_bytes
    whole = torch.zeros(src_h.size + n_arena + 512, dtype=torch.uint8, device="cuda:0")
    at = -(-src_h.size // 256) * 256
    whole[:src_h.size] = torch.from_numpy(src_h).to(whole.device)
    dst = torch.from_numpy(dst_h).to(whole.device)
    ctx = T.tent_create(w.slice_bytes, whole.data_ptr() + at, n_arena, T.TENT_FLAG_BOUNDED_STAGING if chunk else 0)
    T.tent_register_segment(ctx, whole.data_ptr(), whole.numel())
    T.tent_register_segment(ctx, dst.data_ptr(), dst.numel())
    stream = torch.cuda.current_stream()
    h = T.tent_declare(ctx, w.src_ptr, w.src_ext, w.dst_ptr, w.dst_ext)
    T.tent_plan(ctx, h, w.rails, False, stream)
    if chunk:
        T.tent_execute_bounded(ctx, h, chunk, stream)
    else:
        T.tent_execute(ctx, h, stream)
    torch.cuda.synchronize()
    s = oracle.split(w.src_ptr, w.src_ext, w.slice_bytes)
    b = oracle.bind(s.len, w.rails)
    want, staging = dst_h.copy(), np.zeros(n_arena, dtype=np.uint8)
    if chunk:
        assert chunk < w.payload and oracle.execute_bounded(w, s, b, [src_h, want], staging, chunk) == 0
    else:
        oracle.execute(w, s, b, [src_h, want], staging)
    assert np.array_equal(dst.cpu().numpy(), want)
    assert np.array_equal(whole[at:at + n_arena].cpu().numpy(), staging)
    T.tent_destroy(ctx)


@pytest.mark.parametrize("partial", [False, True])
def test_a_replan_on_another_stream_than_the_execute(H, partial):
    """After an execute that leaves slices over and after one that cannot, a plan on another stream comes after the
    bookkeeping: it finds exactly what is left, and the batch ends as on one stream."""
    from paper_2604_00368_amd import binding as T
    w = LAYOUTS["tiles_4KiB"]()
    src, dst0 = W.fill_numpy(w, 0), W.fill_numpy(w, 1)
    R = w.rails.shape[0]
    results = []
    for two_streams in (False, True):
        with H.Engine(w, src, dst0) as eng:
            eng.declare()
            torch.cuda.synchronize(eng.dev)
            side = torch.cuda.Stream(eng.dev) if two_streams else None
            s = side.cuda_stream if two_streams else eng.stream
            st, info = T.tent_plan(eng.ctx, eng.batch, w.rails, stream=s)
            assert st == 0
            if partial:
                share = np.array(list(info.rail_bytes)[:R], dtype=np.uint64) // np.uint64(2)
                T.tent_sim_advance(eng.ctx, eng.batch, w.rails["queued_bytes"] + share, s)
            T.tent_execute(eng.ctx, eng.batch, s)
            st, info = eng.plan()                                # on the engine's stream
            left = (st, info.n_slices)
            if two_streams:
                side.synchronize()
            eng.execute()
            assert T.tent_poll(eng.ctx, eng.batch, eng.stream) == 0
            results.append((left, eng.dst.cpu().numpy(), eng.table()))
    assert (results[0][0][1] > 0) == partial
    assert results[0][0] == results[1][0]
    assert np.array_equal(results[0][1], results[1][1])
    assert np.array_equal(results[0][2], results[1][2])


@pytest.mark.parametrize("two_passes", [False, True])
def test_a_list_too_short_for_what_is_bound(H, two_passes):
    """A partial execute recorded into a graph and replayed when far more is BOUND than its tile list holds: in one pass the
    workgroups that fit move theirs, in two passes nothing counts as moved.  A slice is DONE only if its bytes have arrived,
    the rest stays BOUND, and a later plan and execute complete the batch."""
    from helpers import expected_destination
    from paper_2604_00368_amd import binding as T
    w = W.kv_migration(n_req=12, layers=2, ctx_lo=200, ctx_hi=400, page_tokens=16, slice_bytes=256 * KiB)
    src, dst0 = W.fill_numpy(w, 0), W.fill_numpy(w, 1)
    dst_want = expected_destination(w, src, dst0)
    R = w.rails.shape[0]
    with H.Engine(w, src, dst0, flags=T.TENT_FLAG_SKIP_OVERLAP_CHECK if two_passes else 0) as eng:
        eng.declare()
        _, info = eng.plan()
        quarter = np.array(list(info.rail_bytes)[:R], dtype=np.uint64) // np.uint64(4)
        stayed = T.tent_sim_advance(eng.ctx, eng.batch, w.rails["queued_bytes"] + quarter, eng.stream)
        assert 0 < stayed < info.n_slices
        side = torch.cuda.Stream(eng.dev)
        side.wait_stream(torch.cuda.current_stream(eng.dev))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                T.tent_execute(eng.ctx, eng.batch, torch.cuda.current_stream(eng.dev))
        torch.cuda.synchronize(eng.dev)
        _, info = eng.plan()                                       # nothing has moved: every slice is BOUND now
        assert info.n_slices == info.n_pending_before == eng.table().shape[0]
        graph.replay()
        torch.cuda.synchronize(eng.dev)
        tab, dst = eng.table(), eng.dst.cpu().numpy()
        done = tab["state"] == T.TENT_SLICE_DONE
        assert (tab["state"][~done] == T.TENT_SLICE_BOUND).all()
        assert T.tent_poll(eng.ctx, eng.batch, eng.stream) == int((~done).sum())
        moved = int(tab["len"][done].astype(np.uint64).sum())
        if two_passes:
            assert moved == 0
        else:
            assert 0 < moved <= int(quarter.sum())
        print("listed", int(done.sum()), "of", done.shape[0], "slices", flush=True)
        # the bytes of every DONE slice are where they belong
        first = np.zeros(w.n_desc + 1, dtype=np.int64)             # payload position of every transfer
        for j in range(w.n_desc):
            first[j + 1] = first[j] + int(w.src_ext["len"][w.src_ptr[j]:w.src_ptr[j + 1]].sum())
        def payload(pool, ext, keep):
            return np.concatenate([pool[int(e["off"]):int(e["off"]) + int(e["len"])] for e in ext])[keep]
        keep = np.zeros(int(first[-1]), dtype=bool)
        for row in tab[done]:
            at = int(first[row["desc"]]) + int(row["off"])
            keep[at:at + int(row["len"])] = True
        assert np.array_equal(payload(dst, w.dst_ext, keep), payload(src, w.src_ext, keep))
        st, info = eng.plan()
        assert st == 0 and info.n_slices == int((~done).sum())
        eng.execute()
        assert T.tent_poll(eng.ctx, eng.batch, eng.stream) == 0
        assert np.array_equal(eng.dst.cpu().numpy(), dst_want)
