"""Performance cases of the slice-spraying engine, each one pass of a caller's program through the C ABI.

A case names a *layout* (which transfers exist: paged KV blocks, whole tensors, ragged byte ranges) and a *flow* (the
calls a program makes on them).  Everything that decides how much moves -- context lengths, tensor shapes, extent
lengths -- follows from the case alone; page tables, pool contents and rail telemetry are drawn from the seed.

Layouts
  paged    requests x planes (layers, K and V) of fixed-size pages, page tables randomly permuted on both sides; with
           `token_bytes` the last page of every transfer carries only the tokens that are there; `skew_src` and
           `skew_dst` shift every page to an odd address
  tensors  the contiguous tensors of a transformer, destination order shuffled
  ragged   transfers of any byte length, source and destination cut independently into extents of any length

Flows
  life      a serving request: declare, plan, execute, poll until complete, release -- what a batch costs that moves once
  cycle     reset, plan, execute on one stream: a recurring transfer whose descriptors stay declared
  graph     the same cycle recorded once into a HIP graph and replayed
  epochs    a transfer that spans telemetry windows: re-plan what is unfinished, rails fail, bandwidth probes feed the next
            plan, the monitor pauses and re-admits rails, a last window drains
  dispatch  request-level planning with priorities (mice round robin, elephants sprayed by weight), then execute
  bounded   plan, then execute through a staging arena much smaller than the payload

The outputs are the destination pool and the staging arena as they stand after the pass and whatever the calls hand
back.  They are bytes and whole numbers, so two correct implementations agree exactly.
"""
import math

import numpy as np
import torch

from paper_2604_00368_amd import binding as T
from paper_2604_00368_amd import workloads as W

KiB, MiB = 1 << 10, 1 << 20

_KV = dict(layout="paged", planes=64, page_bytes=32 * KiB, pages_lo=128, pages_hi=512, slice_bytes=256 * KiB,
           rails="eight_and_one")
_LATENT = dict(layout="paged", planes=1, page_bytes=18 * KiB, pages_lo=8, pages_hi=64, slice_bytes=16 * KiB,
               rails="alternating16")
_SMALL = dict(layout="paged", n_req=64, planes=1, page_bytes=16 * KiB, pages_lo=4, pages_hi=16, slice_bytes=64 * KiB,
              rails="four_one_down")


def listed():
    return [
        # 64 short transfers of shuffled 16 KiB blocks (10 MB): the smallest serving call, declared, planned, moved,
        # polled and released; latency and launches decide it
        dict(_SMALL, name="tiny_life", flow="life", shape=1),
        # the same batch as a recurring transfer replayed from a HIP graph: what is left when no host work is
        dict(_SMALL, name="tiny_graph", flow="graph", shape=1),
        # prefill -> decode migration of two requests of an 8B-class model (32 layers, K and V pages of 32 KiB,
        # 2k-8k tokens), as a serving engine issues it: one batch, used once
        dict(_KV, name="kv_two_requests_life", flow="life", shape=2, n_req=2),
        # the whole KV migration of 32 requests (about 20 GiB, 82 k slices, 9 rails): the benchmark's step
        dict(_KV, name="kv_migration_cycle", flow="cycle", shape=2, n_req=32),
        # RL parameter update: the 7.5 B bf16 parameters of a 32-layer transformer as contiguous tensors, 1 MiB slices
        dict(name="rl_params_cycle", layout="tensors", flow="cycle", shape=3, layers=32, hidden=4096, ffn=14336,
             vocab=128256, kv_dim=1024, slice_bytes=1 * MiB, rails="loguniform8"),
        # many small flows: 4096 requests of 8-64 latent-KV pages of 18 KiB, 16 KiB slices that straddle pages
        dict(_LATENT, name="many_small_cycle", flow="cycle", shape=5, n_req=4096),
        # the same over six layers: about a million slices planned per call
        dict(_LATENT, name="many_small_x6_cycle", flow="cycle", shape=5, n_req=4096, planes=6),
        # a KV migration that spans sixteen telemetry windows with failing rails
        dict(_KV, name="kv_failures_epochs", flow="epochs", shape=4, n_req=8, epochs=16),
        # Algorithm 1 request by request: three priorities, transfers shorter than theta go out whole
        dict(_KV, name="kv_priorities_dispatch", flow="dispatch", shape=6, n_req=8, theta_slices=24),
        # staging buffer of 256 MiB for a payload of gigabytes
        dict(_KV, name="kv_bounded_256MiB", flow="bounded", shape=7, n_req=8, chunk_MiB=256),
        # latent KV whose last page holds only the tokens that are there (1152 bytes each)
        dict(_LATENT, name="latent_partial_pages_cycle", flow="cycle", shape=8, n_req=1024, planes=2,
             token_bytes=1152),
        # byte ranges of any length on both sides, as a checkpoint shard or an object store hands them out
        dict(name="ragged_cycle", layout="ragged", flow="cycle", shape=9, n_req=256, max_len=2 * MiB, max_ext=48 * KiB,
             slice_bytes=64 * KiB, rails="mixed5"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    flow = rng.choice(["life", "life", "cycle", "cycle", "cycle", "graph", "epochs", "dispatch", "bounded"])
    shape = rng.randrange(1 << 20)
    rails = rng.choice(["four_one_down", "eight_and_one", "loguniform8", "alternating16", "mixed5"])
    layout = rng.choice(["paged", "paged", "paged", "paged", "tensors", "ragged"])
    if layout == "paged":
        page = rng.choice([4, 16, 18, 32, 36, 64, 128]) * KiB
        lo = rng.randint(2, 32)
        hi = lo + _log(rng, 4, 256)
        planes = rng.choice([1, 1, 2, 6, 16, 64, 120])
        budget = _log(rng, 4 * MiB, 1536 * MiB if flow == "graph" else 6144 * MiB)
        n_req = max(1, min(4096, budget // (planes * page * (lo + hi) // 2)))
        case = dict(layout=layout, n_req=n_req, planes=planes, page_bytes=page, pages_lo=lo, pages_hi=hi,
                    slice_bytes=rng.choice([16, 48, 64, 100, 256, 1024]) * KiB)
        option = rng.randrange(6)
        if option == 0:
            case["token_bytes"] = page // 16
        elif option == 1:
            case["skew_src"], case["skew_dst"] = rng.randint(1, 15), rng.randint(0, 15)
    elif layout == "tensors":
        hidden = rng.choice([512, 768, 1024, 2048, 4096])
        case = dict(layout=layout, layers=rng.randint(1, 12), hidden=hidden, ffn=hidden * rng.randint(5, 14) // 4,
                    vocab=rng.randint(4001, 128256), kv_dim=hidden // rng.choice([1, 4]),
                    slice_bytes=rng.choice([256 * KiB, 1 * MiB, 4 * MiB]))
    else:
        case = dict(layout=layout, n_req=rng.randint(24, 256), max_len=_log(rng, 64 * KiB, 2 * MiB),
                    max_ext=_log(rng, 4 * KiB, 96 * KiB), slice_bytes=rng.choice([4096 + 7, 16 * KiB, 64 * KiB, 100_000]))
    case.update(flow=flow, shape=shape, rails=rails)
    if flow == "epochs":
        case["epochs"] = rng.randint(3, 16)
    elif flow == "dispatch":
        case["theta_slices"] = rng.choice([1, 2, 8, 32])
    elif flow == "bounded":
        case["chunk_MiB"] = rng.choice([16, 64, 128, 256])
    return case


# ---- what follows from the case alone -----------------------------------------------------------
def _rng(*key):
    return np.random.Generator(np.random.PCG64(list(key)))


def _transfer_bytes(case):
    """Byte length of every transfer."""
    g = _rng(case["shape"], 11)
    if case["layout"] == "paged":
        pages = g.integers(case["pages_lo"], case["pages_hi"] + 1, size=case["n_req"]).astype(np.int64)
        size = pages * case["page_bytes"]
        if case.get("token_bytes"):
            per_page = case["page_bytes"] // case["token_bytes"]
            size -= g.integers(0, per_page, size=case["n_req"]) * case["token_bytes"]
        return np.repeat(size, case["planes"])
    if case["layout"] == "tensors":
        h, f, kv = case["hidden"], case["ffn"], case["kv_dim"]
        one = [h, h * h, kv * h, kv * h, h * h, h, f * h, f * h, h * f]
        return 2 * np.array([case["vocab"] * h] + one * case["layers"] + [h], dtype=np.int64)
    return g.integers(1, case["max_len"] + 1, size=case["n_req"]).astype(np.int64)


def _ragged_extents(case, lengths, side):
    """Extent lengths of all transfers (any byte length up to max_ext) and how many each transfer has."""
    g = _rng(case["shape"], 12, side)
    counts, sizes = [], []
    for total in lengths.tolist():
        cuts = np.cumsum(g.integers(1, case["max_ext"] + 1, size=2 * total // case["max_ext"] + 8))
        while cuts[-1] < total:
            cuts = np.concatenate([cuts, cuts[-1] + np.cumsum(g.integers(1, case["max_ext"] + 1, size=64))])
        ends = np.concatenate([cuts[cuts < total], [total]])
        sizes.append(np.diff(ends, prepend=0))
        counts.append(ends.shape[0])
    return np.array(counts, dtype=np.int64), np.concatenate(sizes)


def _extent_count(case):
    lengths = _transfer_bytes(case)
    if case["layout"] == "paged":
        return 2 * int((-(-lengths // case["page_bytes"])).sum())
    if case["layout"] == "tensors":
        return 2 * lengths.shape[0]
    return sum(int(_ragged_extents(case, lengths, side)[0].sum()) for side in (0, 1))


def work(case):
    lengths = _transfer_bytes(case)
    payload = int(lengths.sum())
    n_slices = int((-(-lengths // case["slice_bytes"])).sum())
    # source bytes read, staging and destination bytes written, 16-byte extents read, a 32-byte row per slice written
    # (in every telemetry window rows of what is unfinished, about half of the batch on average)
    rows = n_slices * (case["epochs"] // 2 + 1 if case["flow"] == "epochs" else 1)
    return {"bytes": 3 * payload + 16 * _extent_count(case) + 32 * rows, "flops": 0}


def tolerance(case):
    return "exact"


# ---- inputs -------------------------------------------------------------------------------------
def _csr(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)


def _extents(seg, off, length):
    e = np.zeros(off.shape[0], dtype=W.EXTENT_DTYPE)
    e["seg"], e["off"], e["len"] = seg, off, length
    return e


def _side(case, lengths, side, g):
    """CSR pointers, extents and pool size of one side."""
    if case["layout"] == "paged":
        page, planes, n_req = case["page_bytes"], case["planes"], case["n_req"]
        per_req = -(-lengths[::planes] // page)
        total = int(per_req.sum())
        perm = g.permutation(total).astype(np.int64)                    # one page table, shared by the planes
        starts = np.concatenate([[0], np.cumsum(per_req)])
        plane_base = (np.arange(planes, dtype=np.int64) * total)[:, None]
        off = np.concatenate([((plane_base + perm[starts[r]:starts[r + 1]][None, :]) * page).ravel() for r in range(n_req)])
        counts = np.repeat(per_req, planes)
        ext = _extents(side, off, page)
        ext["len"][np.cumsum(counts) - 1] = lengths - (counts - 1) * page
        skew = case.get("skew_dst" if side else "skew_src", 0)
        ext["off"] += np.uint64(skew)
        return _csr(counts), ext, planes * total * page + 16
    if case["layout"] == "tensors":
        n = lengths.shape[0]
        order = np.arange(n) if side == 0 else g.permutation(n)
        off = np.zeros(n, dtype=np.int64)
        off[order] = np.concatenate([[0], np.cumsum(lengths[order])[:-1]])
        return np.arange(n + 1, dtype=np.uint32), _extents(side, off, lengths), int(lengths.sum())
    counts, sizes = _ragged_extents(case, lengths, side)
    order = g.permutation(sizes.shape[0])                               # shuffled over the pool, with gaps
    run = np.cumsum(sizes[order] + g.integers(0, 64, size=sizes.shape[0]))
    off = np.zeros(sizes.shape[0], dtype=np.int64)
    off[order] = run - sizes[order]
    return _csr(counts), _extents(side, off, sizes), int(sizes.sum()) + 64 * sizes.shape[0]


def _rails(case, g):
    kind = case["rails"]
    if kind == "four_one_down":
        return W.make_rails([25000, 25000, 50000, 100000], queued=g.integers(0, MiB + 1, size=4),
                            health=[W.HEALTHY, W.EXCLUDED, W.HEALTHY, W.HEALTHY])
    if kind == "eight_and_one":
        return W.make_rails([50000] * 8 + [400000], queued=g.integers(0, 256 * KiB, size=9))
    if kind == "loguniform8":
        return W.make_rails(np.rint(np.exp(g.uniform(np.log(12500.0), np.log(100000.0), size=8))).astype(np.uint64))
    if kind == "alternating16":
        return W.make_rails([25000, 50000] * 8, queued=g.integers(0, 256 * KiB, size=16))
    return W.make_rails(g.integers(10000, 400000, size=5), lat_ns=g.integers(0, 20000, size=5),
                        queued=g.integers(0, 1 << 22, size=5), health=[0, 1, 0, 0, 0],
                        beta1_q8=g.integers(128, 512, size=5), penalty_q8=g.integers(128, 512, size=5))


def _source_pool(case, nbytes, seed):
    """Seeded contents: bf16 normal values for KV pages and tensors, uniform bytes otherwise."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pool = torch.empty(-(-nbytes // 8), dtype=torch.int64, device="cuda")
    if case["layout"] == "ragged":
        return pool.random_(generator=g)
    flat = pool.view(torch.bfloat16)
    for lo in range(0, flat.numel(), 1 << 29):
        flat[lo:lo + (1 << 29)].normal_(generator=g)
    return pool


class State:
    """Pools, engine context and declared batch of one caller."""

    ctx = None

    def __init__(self, case, seed):
        self.case = case
        g = _rng(case["shape"], 13, seed)
        lengths = _transfer_bytes(case)
        self.src_ptr, self.src_ext, src_bytes = _side(case, lengths, W.SRC_SEG, g)
        self.dst_ptr, self.dst_ext, dst_bytes = _side(case, lengths, W.DST_SEG, g)
        self.rails = _rails(case, g)
        payload = int(lengths.sum())
        R = self.rails.shape[0]
        flags, arena_bytes = 0, payload + 64 * 256
        if case["flow"] == "bounded":
            flags, arena_bytes = T.TENT_FLAG_BOUNDED_STAGING, case["chunk_MiB"] * MiB + 64 * 256
        self.src = _source_pool(case, src_bytes, seed)
        self.dst = torch.zeros(-(-dst_bytes // 8), dtype=torch.int64, device="cuda")
        self.arena = torch.zeros(-(-arena_bytes // 8), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        self.stream = torch.cuda.current_stream()
        self.ctx = T.tent_create(case["slice_bytes"], self.arena.data_ptr(), self.arena.numel() * 8, flags, R)
        T.tent_register_segment(self.ctx, self.src.data_ptr(), self.src.numel() * 8)
        T.tent_register_segment(self.ctx, self.dst.data_ptr(), self.dst.numel() * 8)
        if case["flow"] == "life":
            return
        self.batch = T.tent_declare(self.ctx, self.src_ptr, self.src_ext, self.dst_ptr, self.dst_ext)
        if case["flow"] == "graph":
            _cycle(self, self.stream)                                   # the batch's first plan checks the declaration
            torch.cuda.synchronize()
            self.graph = torch.cuda.CUDAGraph()
            side = torch.cuda.Stream()
            with torch.cuda.stream(side), torch.cuda.graph(self.graph, stream=side):
                _cycle(self, torch.cuda.current_stream())
            torch.cuda.synchronize()
        elif case["flow"] == "epochs":
            self._telemetry(g, payload)
        elif case["flow"] == "dispatch":
            self.priority = g.integers(0, 3, size=lengths.shape[0]).astype(np.uint8)

    def _telemetry(self, g, payload):
        """Per window: queued bytes, true bandwidths, how much each rail drains, which rails fail."""
        n, R = self.case["epochs"], self.rails.shape[0]
        nominal = self.rails["bw_MBps"].astype(np.float64)
        up = self.rails["health"] != W.EXCLUDED
        t_us = -(-payload // int(n * nominal[up].sum()))
        self.true_bw = np.maximum(1, np.rint(nominal * np.exp(0.5 * g.standard_normal((n, R))))).astype(np.uint32)
        self.queued = g.integers(0, 4 * MiB + 1, size=(n, R)).astype(np.uint64)
        self.budget = self.true_bw.astype(np.uint64) * np.uint64(t_us)
        self.fails = (g.random((n, R)) < 0.03).astype(np.uint8)
        self.congestion = (g.integers(1, 9, size=(n, R)) * (g.random((n, R)) < 0.15)).astype(np.uint32)
        self.probe_params = W.make_probe_params(2 * self.rails["bw_MBps"].astype(np.uint64), ewma_q8=128)
        self.monitor_params = W.make_monitor_params()

    def __del__(self):
        if self.ctx is not None:
            T.tent_destroy(self.ctx)
            self.ctx = None


def prepare(case, seed):
    return State(case, seed)


# ---- one pass -----------------------------------------------------------------------------------
def _plan(s, rails, stream):
    st, _ = T.tent_plan(s.ctx, s.batch, rails, False, stream)
    return st


def _cycle(s, stream):
    T.tent_reset(s.ctx, s.batch, stream)
    _plan(s, s.rails, stream)
    T.tent_execute(s.ctx, s.batch, stream)


def _life(s):
    batch = T.tent_declare(s.ctx, s.src_ptr, s.src_ext, s.dst_ptr, s.dst_ext)
    _, info = T.tent_plan(s.ctx, batch, s.rails, True, s.stream)
    T.tent_execute(s.ctx, batch, s.stream)
    remaining = T.tent_poll(s.ctx, batch, s.stream)
    T.tent_release(s.ctx, batch)
    return {"remaining": remaining, "rail_bytes": np.array(info.rail_bytes, dtype=np.int64),
            "queued_after": np.array(info.queued_after, dtype=np.int64)}


def _epochs(s):
    R = s.rails.shape[0]
    monitor = T.tent_monitor_init(s.monitor_params, R)
    rails = s.rails.copy()
    base_health = s.rails["health"].copy()
    zero = np.zeros(R, dtype=np.uint32)
    done = []
    T.tent_reset(s.ctx, s.batch, s.stream)
    for e in range(s.case["epochs"]):
        rails["queued_bytes"] = s.queued[e]
        before = rails["bw_MBps"].copy()
        hard, probe = zero, zero
        if _plan(s, rails, s.stream) == T.TENT_OK:
            hard = T.tent_sim_fail(s.ctx, s.batch, s.fails[e], True, s.stream).astype(np.uint32)
            done.append(T.tent_sim_advance(s.ctx, s.batch, s.budget[e], s.stream))
            T.tent_sim_latency(s.ctx, s.batch, s.true_bw[e], s.stream)
            rails, probe = T.tent_update_bandwidth(s.ctx, s.batch, s.probe_params, rails, s.stream)
            T.tent_execute(s.ctx, s.batch, s.stream)
        rails = T.tent_monitor_update(s.monitor_params, monitor, rails, hard, s.congestion[e], probe, before)
        rails["health"] = np.where(base_health == W.EXCLUDED, W.EXCLUDED, rails["health"])
    _plan(s, s.rails, s.stream)                                          # the rest drains on the nominal rails
    T.tent_execute(s.ctx, s.batch, s.stream)
    remaining = T.tent_poll(s.ctx, s.batch, s.stream)
    return {"remaining": remaining, "done": np.array(done, dtype=np.int64),
            "estimates": rails["bw_MBps"].astype(np.int64), "health": rails["health"].astype(np.int64)}


def _dispatch(s):
    T.tent_reset(s.ctx, s.batch, s.stream)
    params = W.make_dispatch_params(s.case["theta_slices"] * s.case["slice_bytes"])
    told = []
    for window in range(3):                          # every priority meets a slot that takes it within three windows
        params["window"] = window
        st, info = T.tent_plan_dispatch(s.ctx, s.batch, s.rails, params, s.priority, True, s.stream)
        params["rr_start"] = info.rr_next
        told.append([info.plan.n_slices, info.n_mice, info.n_elephant, info.n_deferred, info.rr_next])
        T.tent_execute(s.ctx, s.batch, s.stream)
        if info.n_deferred == 0:
            break
    return {"windows": np.array(told, dtype=np.int64)}


def _bounded(s):
    T.tent_reset(s.ctx, s.batch, s.stream)
    _plan(s, s.rails, s.stream)
    T.tent_execute_bounded(s.ctx, s.batch, s.case["chunk_MiB"] * MiB, s.stream)
    return {}


def run(state):
    flow = state.case["flow"]
    told = {}
    if flow == "life":
        told = _life(state)
    elif flow == "cycle":
        _cycle(state, state.stream)
    elif flow == "graph":
        state.graph.replay()
    elif flow == "epochs":
        told = _epochs(state)
    elif flow == "dispatch":
        told = _dispatch(state)
    else:
        told = _bounded(state)
    return {"destination": state.dst, "staging": state.arena, "told": told}


# ---- the destination by its definition ----------------------------------------------------------
def exact(case, seed):
    """DST_j[x] = SRC_j[x]: the destination pool from the descriptors and the source pool alone, whatever the slices
    and rails were.  What depends on the binding (staging bytes, counts) is left out."""
    g = _rng(case["shape"], 13, seed)
    lengths = _transfer_bytes(case)
    src_ptr, src_ext, src_bytes = _side(case, lengths, W.SRC_SEG, g)
    dst_ptr, dst_ext, dst_bytes = _side(case, lengths, W.DST_SEG, g)
    src = _source_pool(case, src_bytes, seed).view(torch.uint8)
    out = torch.zeros(-(-dst_bytes // 8), dtype=torch.int64, device="cuda")
    dst = out.view(torch.uint8)
    if case["layout"] == "paged":
        page = case["page_bytes"]
        a, b = case.get("skew_src", 0), case.get("skew_dst", 0)
        n = (src_bytes - 16) // page
        rows_in = src[a:a + n * page].view(n, page)
        rows_out = dst[b:b + n * page].view(n, page)
        at_in = torch.from_numpy((src_ext["off"] // page).astype(np.int64)).cuda()
        at_out = torch.from_numpy((dst_ext["off"] // page).astype(np.int64)).cuda()
        held = torch.from_numpy(src_ext["len"].astype(np.int64)).cuda()
        column = torch.arange(page, device="cuda")
        for lo in range(0, at_in.numel(), 1 << 14):
            part = rows_in[at_in[lo:lo + (1 << 14)]]
            if case.get("token_bytes"):
                part[column[None, :] >= held[lo:lo + (1 << 14), None]] = 0
            rows_out[at_out[lo:lo + (1 << 14)]] = part
    else:
        host = case["layout"] == "ragged"                              # many short pieces: on the host
        a = src.cpu().numpy() if host else src
        b = np.zeros(dst.numel(), dtype=np.uint8) if host else dst
        join = np.concatenate if host else torch.cat
        for j in range(lengths.shape[0]):
            data = join([a[int(e["off"]):int(e["off"]) + int(e["len"])] for e in src_ext[src_ptr[j]:src_ptr[j + 1]]])
            at = 0
            for e in dst_ext[dst_ptr[j]:dst_ptr[j + 1]]:
                b[int(e["off"]):int(e["off"]) + int(e["len"])] = data[at:at + int(e["len"])]
                at += int(e["len"])
        if host:
            out = torch.from_numpy(b).cuda().view(torch.int64)
    return {"destination": out, "staging": None, "told": None}
