"""Host logic of libcocktail.so (no GPU): symbols, argument validation, planner vs oracle, work split."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import workloads
from oracle import cocktail_oracle as O
import paper_2503_23294_amd as ck
from paper_2503_23294_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "cocktail.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(cocktail_[a-z0-9_]+)\s*\(", hdr))
    assert declared == set(_lib.EXPORTS), declared ^ set(_lib.EXPORTS)
    handle = _lib.lib()
    for name in declared:
        assert getattr(handle, name) is not None
    assert handle.cocktail_version() >= 1


def _plan(w, workers):
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = workloads.chunk_bits(w)
    flat = np.concatenate(bits) if bits else np.zeros(0, np.uint8)
    return ck.cocktail_plan(sh, w.seq_lens, flat, workers), bits


def _parse(plan):
    """The fields of the plan's internal header that these tests look at, read by name through the library's
    accessor, so that a change of the header layout cannot be misread here."""
    f = lambda name, i=0: ck.cocktail_plan_field(plan, name, i)
    h = {"rep": f("rep"), "workers": f("num_workers"), "segments": f("num_segments"), "partials": f("num_partials"),
         "gblocks": f("total_gblocks"), "v_layout": f("v_layout"), "plan_bytes": f("plan_bytes"),
         "work_heads": f("work_heads"), "work_rep": f("work_rep"),
         "groups": f("num_groups"), "pool_segs": f("num_pool_segs"), "ws_status_off": f("ws_status_off"),
         "block_bytes": [f("block_bytes", c) for c in range(_lib.NUM_CLASSES)]}
    h["off"] = {k: f("off_" + k) for k in ("segments", "worker_rec", "group_rec", "pool_seg", "counters", "bh_off")}
    assert f("sizeof_segment") == 32 and f("sizeof_worker_rec") == 64 and f("sizeof_group_rec") == 32
    assert f("sizeof_pool_seg") == 32
    return h


def _consts(plan):
    return ([ck.cocktail_plan_field(plan, "iter_units", c) for c in range(_lib.NUM_CLASSES)],
            ck.cocktail_plan_field(plan, "counter_stride_bytes") // 4, ck.cocktail_plan_field(plan, "partial_header_floats"))


def _arr(blob, off, dtype, n):
    return np.frombuffer(blob.tobytes(), dtype=dtype, count=n, offset=off)


def _check_work_split(plan, w, workers, seed=0):
    """Replays the decode kernel's walk over the plan (own ranges, then pool tickets in a random
    hand-out order) and checks that every unit is read exactly once and every partial id is sound."""
    h = _parse(plan)
    ITER_UNITS, COUNTER_STRIDE, header_floats = _consts(plan)
    # the requested number of workers is an upper bound: never more workers than units of work (multiples of 64)
    share = h["work_heads"] // w.num_kv_heads
    nc = _lib.NUM_CLASSES
    f = ck.cocktail_plan_field
    # blocks per head that hold tokens, blocks per head the run is laid out with (room to grow), first block per sequence
    used_blk = _arr(plan.blob, f(plan, "off_nblk"), np.int32, nc * w.batch).reshape(w.batch, nc)
    run_blk = _arr(plan.blob, f(plan, "off_run_blocks"), np.int32, nc * w.batch).reshape(w.batch, nc)
    base_blk = _arr(plan.blob, f(plan, "off_blk_base"), np.int32, nc * (w.batch + 1)).reshape(w.batch + 1, nc)
    work_blocks = int(used_blk.sum()) * w.num_kv_heads
    units = work_blocks * share * (1 if w.head_dim == 64 else 2)
    assert h["plan_bytes"] == plan.blob.size
    assert h["workers"] == plan.sizes.num_workers == min(workers, max((units + 63) // 64 * 64, 64))
    workers = h["workers"]
    S, P, NG, NPS = h["segments"], workers, h["groups"], h["pool_segs"]
    segs = _arr(plan.blob, h["off"]["segments"], np.int32, 8 * S).reshape(S, 8)
    BH = w.batch * h["work_heads"]
    bh_off = _arr(plan.blob, h["off"]["bh_off"], np.int32, BH + 1)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * P).reshape(P, 16)
    groups = _arr(plan.blob, h["off"]["group_rec"], np.int32, 8 * NG).reshape(NG, 8)
    psegs = _arr(plan.blob, h["off"]["pool_seg"], np.int32, 8 * NPS).reshape(NPS, 8)
    counters = _arr(plan.blob, h["off"]["counters"], np.uint32, COUNTER_STRIDE * NG)
    assert (counters == 0).all() and h["off"]["counters"] % 128 == 0
    share = h["work_heads"] // w.num_kv_heads              # work heads that walk the blocks of one kv head
    assert h["gblocks"] == work_blocks * share
    # segments tile the class buffers: every physical block of every (class, b, h) exactly once per work head
    phys = [np.zeros(int(plan.sizes.class_blocks[c]), dtype=np.int32) for c in range(_lib.NUM_CLASSES)]
    g = 0
    for b_, h_, cls, ntok, blk0, nblk, gblk0, spid in segs:
        assert gblk0 == g and nblk > 0 and (nblk - 1) * 64 < ntok
        phys[cls][blk0:blk0 + nblk] += 1
        g += nblk
    for c in range(nc):
        want = np.zeros_like(phys[c])
        for b_ in range(w.batch):
            for h_ in range(w.num_kv_heads):
                first = base_blk[b_, c] + h_ * run_blk[b_, c]
                want[first:first + used_blk[b_, c]] = share       # blocks that are only room to grow belong to nobody
        assert np.array_equal(phys[c], want)

    rng = np.random.default_rng(seed)
    seen = np.zeros(2 * h["gblocks"], dtype=np.int32)       # per unit
    pid_owner = {}
    members = {}
    for it in range(P):
        members.setdefault(int(recs[it, 12]), []).append(it)
    cost = np.zeros(P, dtype=np.int64)
    pool_cost = 0
    for gi in range(NG):
        ngran, pseg0, nps, nworkers, counter = groups[gi, :5]
        ws = sorted(members.get(gi, []), key=lambda x: int(recs[x, 13]) & 0xffff)
        assert len(ws) == nworkers and [int(recs[x, 13]) & 0xffff for x in ws] == list(range(nworkers))
        assert all(recs[x, 13] >> 16 == nps and recs[x, 14] == ngran and recs[x, 15] == pseg0 for x in ws)
        assert 0 <= nps <= 32 and counter == gi
        if h["work_rep"] > 4:
            assert ngran == 0                                # five to eight heads per workgroup: static split only
        # tickets are handed out in ascending order to whichever worker asks next
        hand = sorted(rng.integers(0, nworkers, size=ngran).tolist()) if ngran else []
        tickets = {r: [] for r in range(nworkers)}
        for t, r in zip(range(ngran), rng.permutation(hand) if ngran else []):
            tickets[int(r)].append(t)
        if nps:
            assert psegs[pseg0, 3] == 0
            last = psegs[pseg0 + nps - 1]
            J = ITER_UNITS[segs[last[0], 2]]
            assert last[3] + (last[2] + J - 1) // J == ngran
        for r, it in enumerate(ws):
            g0, g1, s, pid = recs[it, :4]
            if g0 < g1:
                assert recs[it, 4:12].tolist() == segs[s].tolist()
            last_seg, used = -1, set()
            u, u1 = 2 * g0, 2 * g1
            while u < u1:                                    # own range
                b_, h_, cls, ntok, blk0, nblk, gblk0, spid = segs[s]
                bh = b_ * h["work_heads"] + h_
                if u >= 2 * (gblk0 + nblk):
                    s += 1
                    pid = segs[s, 7]                         # enters the next segment as its first visitor
                    continue
                assert 2 * gblk0 <= u
                if s != last_seg:
                    assert pid not in pid_owner
                    pid_owner[pid] = (cls, bh, 0)
                    last_seg = s
                end = min(u1, 2 * (gblk0 + nblk))
                nu = min(ITER_UNITS[cls], end - u)
                seen[u:u + nu] += 1
                cost[it] += nu * h["block_bytes"][cls]
                u += nu
            for t in tickets[r]:                             # pool
                pi = max(i for i in range(nps) if psegs[pseg0 + i, 3] <= t)
                seg, unit0, nunits, gran0, slot0 = psegs[pseg0 + pi, :5]
                b_, h_, cls, ntok, blk0, nblk, gblk0, spid = segs[seg]
                bh = b_ * h["work_heads"] + h_
                J = ITER_UNITS[cls]
                us = unit0 + (t - gran0) * J
                nu = min(J, unit0 + nunits - us)
                assert 0 < nu and us + nu <= 2 * nblk and seg >= last_seg
                if seg != last_seg:
                    slot = slot0 + r
                    assert r < psegs[pseg0 + pi, 5], "a rank that can enter this part from outside has a slot"
                    assert slot not in pid_owner
                    pid_owner[slot] = (cls, bh, 1)
                    used.add(pi)
                    last_seg = seg
                seen[2 * gblk0 + us:2 * gblk0 + us + nu] += 1
                pool_cost += nu * h["block_bytes"][cls]
            for pi in range(nps):                            # slots the worker fills with the neutral state
                if pi not in used and r < psegs[pseg0 + pi, 5]:
                    seg, slot0 = psegs[pseg0 + pi, 0], psegs[pseg0 + pi, 4]
                    assert slot0 + r not in pid_owner
                    pid_owner[slot0 + r] = (segs[seg, 2], segs[seg, 0] * h["work_heads"] + segs[seg, 1], 1)
    # the appended tokens of a (sequence, work head): the last ids of its range, one per slice
    for bh in range(BH):
        for pid in range(bh_off[bh + 1] - f(plan, "append_slices"), bh_off[bh + 1]):
            assert pid not in pid_owner
            pid_owner[pid] = (_lib.NUM_CLASSES - 1, bh, 2)
    assert (seen == 1).all()
    assert sorted(pid_owner) == list(range(h["partials"])) and h["partials"] == plan.sizes.num_partials
    assert bh_off[0] == 0 and bh_off[BH] == h["partials"] and (np.diff(bh_off) >= 0).all()
    for bh in range(BH):
        assert all(pid_owner[p][1] == bh for p in range(bh_off[bh], bh_off[bh + 1]))
    # workspace: the partial states (header + head_dim floats each), then one status word per (sequence, query head)
    assert h["ws_status_off"] == max(h["partials"], 1) * h["work_rep"] * (w.head_dim + header_floats) * 4
    assert plan.sizes.workspace_bytes == h["ws_status_off"] + (4 * w.batch * w.num_q_heads + 15) // 16 * 16
    return h, cost, pool_cost


@pytest.mark.parametrize("cfg,workers", [(1, 64), (1, 2048), (2, 2048), (3, 512), (4, 2048), (5, 512), (5, 7)])
def test_planner_matches_oracle_and_splits_work_exactly_once(cfg, workers):
    w = workloads.config(cfg)
    plan, bits = _plan(w, workers)
    pos = 0
    packed = 0
    for b, t in enumerate(w.seq_lens):
        sp = O.plan_sequence(t, w.chunk_size, bits[b])
        n = t // w.chunk_size
        assert plan.perm[pos:pos + n].tolist() == sp.perm.tolist()
        assert tuple(plan.class_tokens[b]) == sp.class_tokens
        packed += O.packed_bytes(sp.class_tokens, w.num_kv_heads, w.head_dim, w.group_size)
        pos += n
    assert plan.sizes.packed_bytes == packed
    for c in range(_lib.NUM_CLASSES):
        blocks = sum(((int(plan.class_tokens[b, c]) + 63) // 64) * w.num_kv_heads for b in range(w.batch))
        assert plan.sizes.class_blocks[c] == blocks
        assert plan.sizes.class_bytes[c] == blocks * O.block_bytes(c, w.head_dim, w.group_size)
    h, cost, pool_cost = _check_work_split(plan, w, workers)
    if cfg == 4:
        # the headline shape has pools: a fifth of the bytes, the rest in near-equal own ranges
        total = cost.sum() + pool_cost
        assert 0.15 * total <= pool_cost <= 0.25 * total and h["groups"] == 256   # long ranges: groups of eight


@pytest.mark.parametrize("env", [{"COCKTAIL_POOL_PERCENT": "100"}, {"COCKTAIL_POOL_PERCENT": "0"},
                                 {"COCKTAIL_GROUP_WORKERS": "3", "COCKTAIL_POOL_PERCENT": "50"},
                                 {"COCKTAIL_LAYOUT": "1"}, {"COCKTAIL_LAYOUT": "1", "COCKTAIL_PAIR_MODE": "2"},
                                 {"COCKTAIL_PAIR_MODE": "3", "COCKTAIL_GROUP_WORKERS": "4"}])
def test_work_split_under_tuning_knobs(env, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    for cfg, workers in ((2, 2048), (4, 2048), (1, 64)):
        w = workloads.config(cfg)
        plan, _ = _plan(w, workers)
        _check_work_split(plan, w, workers)


@pytest.mark.parametrize("seed", range(6))
def test_work_split_of_random_small_shapes(seed, monkeypatch):
    rng = np.random.default_rng(1000 + seed)
    batch = int(rng.integers(1, 5))
    hkv = int(rng.integers(1, 4))
    chunk = int(rng.choice([8, 16, 64, 128]))
    lens = [int(x) for x in rng.integers(0, 6000, size=batch)]
    w = workloads.small(f"rand{seed}", batch, hkv, hkv, lens, chunk, int(rng.choice([32, 64, 128])), seed_offset=seed)
    with_pools = 0
    for percent in (None, "25"):                             # with ranges that end where runs end, and never
        if percent:
            monkeypatch.setenv("COCKTAIL_POOL_PERCENT", percent)
        for workers in (1, 3, 16, 40):
            plan, _ = _plan(w, workers)
            h, _, _ = _check_work_split(plan, w, workers, seed)
            with_pools += percent is not None and h["pool_segs"] > 0
    assert with_pools >= 2


@pytest.mark.parametrize("mix,workers,trades", [((0.0, 0.0, 1.0), 64, True), ((0.0, 0.0, 1.0), 192, True), ((0.1, 0.1, 0.8), 128, True),
                                                ((0.3, 0.35, 0.35), 128, False), ((0.0, 0.0, 1.0), 65, False)])
def test_workers_next_to_one_of_their_own_class_trade_places(mix, workers, trades):
    """One head per wave: where worker w and its mate w + P/2 stream the same class, every other rank runs in the place of its mate, so
    that the pools of such groups are shared by both kinds; whatever runs where, every unit is read once."""
    w = workloads.small(f"trade{workers}", 1, 4, 4, [64 * 600], 64, 32, mix=mix, seed_offset=901)
    plan, _ = _plan(w, workers)
    _check_work_split(plan, w, workers)
    h, p = _parse(plan), int(plan.sizes.num_workers)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * p).reshape(p, 16)
    order = recs[:, 0]                                        # first block of a worker's own range, by worker id
    moved = [i for i in range(p) if order[i] != np.sort(order)[i]]
    assert bool(moved) == trades
    if trades:
        assert all(recs[i, 6] == recs[(i + p // 2) % p, 6] for i in moved)
        groups = [{i < p // 2 for i in range(p) if recs[i, 12] == g} for g in set(recs[moved, 12].tolist())]
        assert all(len(g) == 2 for g in groups)


@pytest.mark.parametrize("rep,lens,workers,aligned", [
    (1, [64 * 128], 64, True), (1, [64 * 129 + 64], 64, False), (4, [64 * 128], 64, True), (4, [64 * 1280], 2048, True), (4, [64 * 10300], 2048, False),
    (8, [64 * 6000, 64 * 77 + 5], 2048, True), (16, [64 * 300], 256, True), (6, [64, 65, 1, 0, 640], 2048, True), (8, [40, 0, 3], 4, False)])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_ranges_that_end_where_runs_end(rep, lens, workers, aligned, head_dim):
    """Few blocks per worker, and five to eight heads per wave: every worker stays in one run, ranges of a run differ by a
    block at most, at least 95 % of the workers have work, and there are no pools.  More runs than workers: the plain split."""
    w = workloads.small(f"aligned{rep}", len(lens), 4 * rep, 4, lens, 64, 32, mix=(0.2, 0.3, 0.3, 0.2), head_dim=head_dim, seed_offset=903)
    plan, _ = _plan(w, workers)
    if aligned or head_dim == 128:
        _check_work_split(plan, w, workers)                  # (it replays pools in units of half a block)
    h, p = _parse(plan), int(plan.sizes.num_workers)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * p).reshape(p, 16)
    segs = _arr(plan.blob, h["off"]["segments"], np.int32, 8 * h["segments"]).reshape(-1, 8)
    busy = recs[recs[:, 0] < recs[:, 1]]
    run = np.searchsorted(segs[:, 6], busy[:, 0], side="right") - 1
    inside = busy[:, 1] <= segs[run, 6] + segs[run, 5]
    assert (inside.all() and (recs[:, 14] == 0).all()) == aligned
    if aligned:
        size = {}
        for r, s in zip(busy, segs[run]):
            size.setdefault(tuple(s[:3]), []).append(int(r[1] - r[0]))
        assert all(max(v) - min(v) <= 1 for v in size.values())
        assert len(busy) >= 0.95 * min(p, h["gblocks"])


_WEIGHTS = {1: (1150, 1300, 1100, 530), 4: (1300, 1250, 950, 450), 8: (1300, 1250, 950, 390), 16: (1300, 1250, 950, 330)}


def _ranges(plan):
    """Class and cost of the own range of every worker that has one (a range in one run, else the classes' costs added up), and the
    mean cost per worker.  The cost of a block: its bytes times the planner's weight of its class."""
    h, f = _parse(plan), ck.cocktail_plan_field
    p = int(plan.sizes.num_workers)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * p).reshape(p, 16)
    segs = _arr(plan.blob, h["off"]["segments"], np.int32, 8 * h["segments"]).reshape(-1, 8)
    key = 1 if h["v_layout"] == 0 else 4 if h["work_rep"] <= 4 else 8 if h["work_rep"] == h["rep"] else 16
    block = np.array(h["block_bytes"], float) * np.array(_WEIGHTS[key], float)
    ends = np.concatenate([[0.0], np.cumsum(segs[:, 5] * block[segs[:, 2]])])

    def at(g):
        s = np.searchsorted(segs[:, 6], g, side="right") - 1
        return ends[s] + (g - segs[s, 6]) * block[segs[s, 2]]
    busy = recs[recs[:, 0] < recs[:, 1]]
    return busy[:, 6], at(busy[:, 1]) - at(busy[:, 0]), ends[-1] / p, block


@pytest.mark.parametrize("rep,lens,mix,workers,held", [
    (1, [64 * 4000], (0.05, 0.25, 0.0, 0.7), 2048, True), (8, [64 * 3000, 64 * 2500 + 7], (0.05, 0.25, 0.0, 0.7), 2048, True),
    (4, [64 * 9000], (0.05, 0.25, 0.0, 0.7), 2048, True), (16, [64 * 2500] * 2, (0.05, 0.25, 0.0, 0.7), 2048, True),
    (8, [64 * 3000], (0.0, 0.0, 0.0, 1.0), 2048, False), (8, [64 * 3000], (0.0, 0.1, 0.0, 0.9), 2048, False)])
def test_no_two_workers_of_a_simd_on_int2(rep, lens, mix, workers, held):
    """INT2 has more than half of the cost: it gets no more workers than there are SIMDs, where that does not make its ranges much
    longer than the others; every block is still read once."""
    w = workloads.small(f"held{rep}", len(lens), 4 * rep, 4, lens, 64, 32, mix=mix, seed_offset=905)
    plan, _ = _plan(w, workers)
    _check_work_split(plan, w, workers)
    cls, cost, _, _ = _ranges(plan)
    assert ((cls == 0).sum() <= 1024) == held
    assert cls.size >= 0.95 * int(plan.sizes.num_workers)


@pytest.mark.parametrize("rep,blocks", [(4, 8000), (8, 20000), (16, 10000)])
@pytest.mark.parametrize("workers,capacity,mix", [(2048, 300, (0.05, 0.2, 0.0, 0.75)), (3072, 0, (0.2, 0.35, 0.45)), (1536, 0, (0.0, 0.15, 0.85)),
                                                  (1000, 0, (0.05, 0.2, 0.75))])
def test_int2_ranges_are_as_long_as_the_others_where_simd_mates_are_not_known(rep, blocks, workers, capacity, mix):
    """Waves launched one by one (append slices, another number of workers than the chip's slots): worker w and w + 1024 need not share
    a SIMD, and longer INT2 ranges only make the call longer."""
    w = workloads.small(f"free{rep}", 1, 4 * rep, 4, [64 * blocks], 64, 32, mix=mix, seed_offset=905)
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = np.concatenate(workloads.chunk_bits(w))
    cls, cost, mean, block = _ranges(ck.cocktail_plan(sh, w.seq_lens, bits, workers, append_capacity=capacity))
    # equal parts of a run differ by a block, and up to 1 in 40 workers may be left over
    assert cost[cls == 0].max() <= 1.03 * mean + 1.5 * block[0]
    if (workers, capacity) == (2048, 300):                    # the same without slices: held, by more than that
        cls, cost, mean, block = _ranges(ck.cocktail_plan(sh, w.seq_lens, bits, 2048))
        assert (cls == 0).sum() <= 1024 and cost[cls == 0].max() > 1.03 * mean + 1.5 * block[0]


@pytest.mark.parametrize("hq,hkv,long,short,n,mix", [
    (64, 8, 131072, 1024, 83, (0.15, 0.35, 0.5)), (64, 8, 131072, 4096, 62, (0.05, 0.15, 0.3, 0.5)), (64, 8, 16384, 16384, 63, (0.15, 0.35, 0.5)),
    (64, 8, 131072, 4096, 85, (0.15, 0.35, 0.5)), (32, 8, 131072, 1024, 79, (0.15, 0.35, 0.5)), (32, 8, 32768, 2048, 79, (0.05, 0.15, 0.3, 0.5)),
    (40, 40, 16384, 1024, 15, (0.15, 0.35, 0.5)), (64, 4, 131072, 1024, 84, (0.15, 0.35, 0.5)), (128, 8, 131072, 2048, 41, (0.1, 0.3, 0.6)),
    (8, 8, 131072, 500, 200, (0.1, 0.3, 0.6)), (64, 8, 65536, 2048, 24, (0.15, 0.35, 0.5)), (32, 8, 65536, 65536, 3, (0.05, 0.15, 0.3, 0.5))])
@pytest.mark.parametrize("workers", [2048, 1000])
def test_no_worker_holds_up_the_call(hq, hkv, long, short, n, mix, workers):
    """One long context among many short ones, up to as many runs as workers: no own range is much longer than the mean one,
    whichever split is taken."""
    w = workloads.small(f"long{hq}", n + 1, hq, hkv, [long] + [short] * n, 256, 32, mix=mix, seed_offset=909)
    cls, cost, mean, block = _ranges(_plan(w, workers)[0])
    # ends on runs: at most 1.25 of the mean and two blocks of the dearest class, 1.8 with up to four heads per wave; by cost: to the
    # nearest block, and with one head per wave up to 1.27 / 0.9 of the mean by the speed of the SIMD mate
    assert cost.max() <= (1.25 if hq > 4 * hkv else 1.8) * mean + 2 * block.max()


@pytest.mark.parametrize("hq,hkv,n,tokens,workers,cut_by_cost", [(64, 8, 160, 1200, 4096, False), (128, 8, 85, 1200, 4096, False),
                                                                 (40, 8, 160, 1200, 4096, True), (64, 8, 80, 1200, 2048, True)])
def test_uneven_ranges_rather_than_a_plan_the_built_in_workspace_cannot_hold(hq, hkv, n, tokens, workers, cut_by_cost):
    """So many runs that the longest range is too long.  The split by cost has a partial state for nearly each worker and run; where
    only that makes a plan outgrow the built-in workspace, each worker stays in one run all the same.  Sizes asked for alone,
    a buffer that is too small and the plan itself say the same."""
    import ctypes as C
    w = workloads.small("many", n, hq, hkv, [40000] + [tokens + 32 * (i % 7) for i in range(n - 1)], 32, 32, mix=(0.3, 0.3, 0.4), seed_offset=923)
    plan, bits = _plan(w, workers)
    _check_work_split(plan, w, workers)
    h, (cls, cost, mean, block) = _parse(plan), _ranges(plan)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * workers).reshape(workers, 16)
    segs = _arr(plan.blob, h["off"]["segments"], np.int32, 8 * h["segments"]).reshape(-1, 8)
    run = np.searchsorted(segs[:, 6], recs[:, 0], side="right") - 1
    one_run = (recs[:, 1] <= segs[run, 6] + segs[run, 5]) | (recs[:, 0] == recs[:, 1])
    assert one_run.all() != cut_by_cost
    assert plan.sizes.workspace_bytes <= 24 << 20
    assert (cost.max() > 1.25 * mean + 2 * block.max()) != cut_by_cost
    sl, flat, sizes = np.asarray(w.seq_lens, np.int32), np.concatenate(bits), _lib.Sizes()
    args = (C.byref(plan.shape), sl.ctypes.data, flat.ctypes.data, workers, None, C.byref(sizes))
    assert _lib.lib().cocktail_plan_ex(*args, None, 0, None, None) == 0 and bytes(sizes) == bytes(plan.sizes)
    blob = np.full(plan.blob.size, 0xAB, np.uint8)
    assert _lib.lib().cocktail_plan_ex(*args, blob.ctypes.data, blob.size - 1, None, None) == _lib.ENOSPACE
    assert bytes(sizes) == bytes(plan.sizes) and b"plan buffer holds" in _lib.lib().cocktail_last_error()
    assert _lib.lib().cocktail_plan_ex(*args, blob.ctypes.data, blob.size, None, None) == 0
    assert np.array_equal(blob, plan.blob)


@pytest.mark.parametrize("hq,workers,twins", [(96, 64, False), (96, 720, True), (64, 512, True), (128, 24, False)])
def test_weights_of_twins_are_for_plans_with_twins(hq, workers, twins):
    """More than eight heads per kv head: sets that are not laid out as twins fetch every block themselves, and FP16 bytes count as much
    as with one set."""
    w = workloads.small(f"sets{hq}", 1, hq, 4, [64 * 4000], 64, 32, mix=(0.3, 0.3, 0.4), seed_offset=913)
    plan, _ = _plan(w, workers)
    cls, cost, _, block = _ranges(plan)                       # by the weights of twins
    f16 = cost[cls == 3].mean() / cost[cls == 0].mean()
    f16 *= 1.0 if twins else _WEIGHTS[8][3] / _WEIGHTS[16][3]
    assert abs(f16 - 1) < 0.05


_FOUR = (0.1, 0.2, 0.3, 0.4)


@pytest.mark.parametrize("rep,blocks,workers,mix,pools", [
    (1, 5000, 2048, _FOUR, False), (1, 5000, 1536, _FOUR, True), (1, 3000, 1024, _FOUR, True), (1, 2000, 1024, _FOUR, False), (1, 9000, 3072, _FOUR, False),
    (4, 9000, 2048, _FOUR, False), (4, 6000, 1536, _FOUR, True), (4, 5000, 1024, _FOUR, True), (4, 2000, 1024, _FOUR, False),
    (4, 11000, 3072, _FOUR, False), (4, 11000, 2048, _FOUR, True),
    # INT2 on a few more workers than there are SIMDs; held to one per SIMD; on nearly all; not more than eight blocks per worker
    (1, 5000, 2048, (0.05, 0.15, 0.8), True), (1, 5000, 2048, (0.05, 0.25, 0.7), False), (1, 5000, 2048, (0.0, 0.05, 0.95), False),
    (1, 4000, 2048, (0.05, 0.15, 0.8), False),
    # a cache of FP16 alone
    (4, 9000, 2048, (1.0, 0.0, 0.0), False), (1, 5000, 2048, (1.0, 0.0, 0.0), False), (4, 11000, 2048, (1.0, 0.0, 0.0), True)])
def test_limits_up_to_which_plans_have_no_pools(rep, blocks, workers, mix, pools):
    """Four kv heads of `blocks` blocks: up to 12 per worker with one head per wave, 20 with two to four; 8 while the chip is not full,
    and where few runs of INT2 share only a few SIMDs with one another."""
    w = workloads.small(f"limits{rep}", 1, 4 * rep, 4, [64 * blocks], 64, 32, mix=mix, seed_offset=907)
    plan, _ = _plan(w, workers)
    assert (int(_parse(plan)["pool_segs"]) > 0) == pools
    _check_work_split(plan, w, workers)
    if rep == 1 and mix == (0.05, 0.15, 0.8) and pools:       # launched one by one: no such SIMDs
        sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
        bits = np.concatenate(workloads.chunk_bits(w))
        assert _parse(ck.cocktail_plan(sh, w.seq_lens, bits, workers, append_capacity=64))["pool_segs"] == 0
        many = workloads.small("limits_runs", 24, 4, 4, [64 * 210] * 24, 64, 32, mix=mix, seed_offset=907)
        assert _parse(_plan(many, workers)[0])["pool_segs"] == 0


@pytest.mark.parametrize("workers,capacity,waves", [(2048, 0, 8), (2048, 1, 1), (2047, 0, 1), (1024, 0, 1), (4096, 0, 1), (6144, 0, 1)])
def test_workgroups_of_a_compute_unit_where_the_workers_fill_the_chip_once(workers, capacity, waves):
    """Twice as many workers go out one by one again (a unit's next workgroup would wait for its slowest wave), and so do calls
    with append slices."""
    for rep in (1, 4, 8):
        w = workloads.small(f"waves{rep}", 1, 8 * rep, 8, [64 * 900], 64, 32, seed_offset=921)
        sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
        plan = ck.cocktail_plan(sh, w.seq_lens, np.concatenate(workloads.chunk_bits(w)), workers, append_capacity=capacity)
        assert int(plan.sizes.num_workers) == workers
        assert ck.cocktail_plan_field(plan, "workgroup_waves") == waves


def test_plan_is_the_same_whatever_the_buffer_it_is_written_to():
    """One pass into a buffer of any content and spare room gives the bytes of a size query followed by an exact fit."""
    import ctypes as C
    for w, workers in ((workloads.config(1), 2048), (workloads.small("b", 3, 16, 2, [700, 0, 65], 32, 32, seed_offset=4), 33)):
        plan, bits = _plan(w, workers)
        sl, flat = np.asarray(w.seq_lens, np.int32), np.concatenate(bits)
        args = (C.byref(plan.shape), sl.ctypes.data_as(C.POINTER(C.c_int32)), flat.ctypes.data_as(C.POINTER(C.c_uint8)), workers)
        sizes = _lib.Sizes()
        assert _lib.lib().cocktail_plan(*args, C.byref(sizes), None, 0, None, None) == 0
        exact = np.full(int(sizes.plan_bytes), 0xAB, np.uint8)
        assert _lib.lib().cocktail_plan(*args, C.byref(sizes), exact.ctypes.data, exact.size, None, None) == 0
        assert np.array_equal(plan.blob, exact)
        assert _lib.lib().cocktail_plan(*args, C.byref(sizes), exact.ctypes.data, exact.size - 1, None, None) == _lib.ENOSPACE


def test_plan_handles_empty_sequences_and_tail_only():
    sh = ck.make_shape(3, 2, 2, 128, 16, 32)
    plan = ck.cocktail_plan(sh, [0, 5, 16], [4], 8)
    assert plan.class_tokens.tolist() == [[0, 0, 0, 0], [0, 0, 0, 5], [0, 16, 0, 0]]
    assert list(plan.sizes.class_blocks) == [0, 2, 0, 2] and plan.sizes.num_partials >= 4


@pytest.mark.parametrize("kwargs,code", [
    (dict(hq=3, hkv=2), _lib.EINVAL), (dict(d=96), _lib.EINVAL), (dict(g=48), _lib.EINVAL),
    (dict(d=64, g=128), _lib.EINVAL), (dict(chunk=0), _lib.EINVAL), (dict(workers=0), _lib.EINVAL),
    (dict(bits=[2, 3]), _lib.EINVAL), (dict(lens=[-1]), _lib.EINVAL),
])
def test_plan_rejects_bad_arguments(kwargs, code):
    sh = ck.make_shape(1, kwargs.get("hq", 2), kwargs.get("hkv", 2), kwargs.get("d", 128), kwargs.get("chunk", 8),
                       kwargs.get("g", 32))
    lens = np.asarray(kwargs.get("lens", [16]), dtype=np.int32)
    bits = np.asarray(kwargs.get("bits", [2, 4]), dtype=np.uint8)
    sizes = _lib.Sizes()
    rc = _lib.lib().cocktail_plan(C.byref(sh), lens.ctypes.data_as(C.POINTER(C.c_int32)),
                                  bits.ctypes.data_as(C.POINTER(C.c_uint8)), kwargs.get("workers", 4),
                                  C.byref(sizes), None, 0, None, None)
    assert rc == code
    assert _lib.lib().cocktail_last_error() != b""


@pytest.mark.parametrize("lens,shape,workers,code,text", [
    ([-10**6], (1, 2, 2, 128, 8, 32), 2048, _lib.EINVAL, "negative"),
    ([64, -10**5], (2, 2, 2, 128, 64, 32), 2048, _lib.EINVAL, "negative"),
    ([2**31 - 1], (1, 64, 64, 128, 1 << 20, 32), 2048, _lib.EUNSUPPORTED, "4 GiB"),
    ([2**31 - 1], (1, 256, 256, 64, 1 << 20, 32), 2048, _lib.EUNSUPPORTED, "4 GiB"),
    ([16], (1, 2, 2, 128, 8, 32), -10**6, _lib.EINVAL, "num_workers"),
    ([16], (1, 2, 2, 128, 8, 32), 2**31 - 1, _lib.EINVAL, "num_workers"),
    ([16], (1, 2, 0, 128, 8, 32), 64, _lib.EINVAL, ">= 1"),
    ([16], (1, -2**31, 2, 128, 8, 32), 64, _lib.EINVAL, ">= 1"),
])
def test_plan_binding_hands_on_what_the_library_says(lens, shape, workers, code, text):
    """The buffer the binding makes before the library has looked at the arguments neither fails nor hides the error."""
    bits = np.full(sum(t // shape[4] for t in lens if t >= 0), 4, np.uint8)
    with pytest.raises(ck.CocktailError, match=text) as e:
        ck.cocktail_plan(ck.make_shape(*shape), lens, bits, workers)
    assert e.value.code == code


def test_plan_that_is_larger_than_the_first_buffer(monkeypatch):
    """A plan that does not fit the buffer made for it is written to one of its size."""
    w = workloads.small("large", 3, 16, 2, [700, 0, 65], 32, 32, seed_offset=4)
    want, _ = _plan(w, 33)
    monkeypatch.setattr(ck.api, "_plan_bytes_bound", lambda *a: 4096)
    got, _ = _plan(w, 33)
    assert want.blob.size > 4096 and np.array_equal(got.blob, want.blob) and np.array_equal(got.perm, want.perm)
    assert np.array_equal(got.class_tokens, want.class_tokens)


def test_plan_capacity_and_null_checks():
    sh = ck.make_shape(1, 2, 2, 128, 8, 32)
    lens = np.array([16], dtype=np.int32)
    bits = np.array([2, 4], dtype=np.uint8)
    sizes = _lib.Sizes()
    L = _lib.lib()
    lp, bp = lens.ctypes.data_as(C.POINTER(C.c_int32)), bits.ctypes.data_as(C.POINTER(C.c_uint8))
    assert L.cocktail_plan(C.byref(sh), lp, bp, 4, C.byref(sizes), None, 0, None, None) == _lib.OK
    small = np.zeros(16, dtype=np.uint8)
    assert L.cocktail_plan(C.byref(sh), lp, bp, 4, C.byref(sizes), small.ctypes.data, 16, None, None) == _lib.ENOSPACE
    assert L.cocktail_plan(C.byref(sh), None, bp, 4, C.byref(sizes), None, 0, None, None) == _lib.EINVAL
    assert L.cocktail_plan(C.byref(sh), lp, None, 4, C.byref(sizes), None, 0, None, None) == _lib.EINVAL
    assert L.cocktail_plan(None, lp, bp, 4, C.byref(sizes), None, 0, None, None) == _lib.EINVAL


def test_gpu_entry_points_validate_on_host_before_launching():
    """Bad arguments are rejected before any HIP call, so this runs without a GPU."""
    sh = ck.make_shape(1, 2, 2, 128, 8, 32)
    plan = ck.cocktail_plan(sh, [16], [2, 4], 4)
    L = _lib.lib()
    cache = _lib.Cache()
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 0, 0, 0, 128, None, None) == _lib.EINVAL
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 0, 0, 0, 128, C.byref(cache), None) == _lib.EINVAL
    cache.plan_host = plan.blob.ctypes.data
    cache.plan_dev = 4096
    assert L.cocktail_reorder_quantize(C.byref(sh), 8, 16, 0, 0, 0, 128, C.byref(cache), None) == _lib.EALIGN
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 7, 0, 0, 128, C.byref(cache), None) == _lib.EINVAL
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 0, 0, 0, 100, C.byref(cache), None) == _lib.EINVAL
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 0, 0, 0, 128, C.byref(cache), None) == _lib.EINVAL  # NULL class buffers
    other = ck.make_shape(1, 2, 2, 128, 16, 32)
    assert L.cocktail_reorder_quantize(C.byref(other), 16, 16, 0, 0, 0, 128, C.byref(cache), None) == _lib.EINVAL
    assert b"different shape" in L.cocktail_last_error()
    assert L.cocktail_decode_attention(C.byref(sh), None, C.byref(cache), 0.0, 16, None, 16, 0, None) == _lib.EINVAL
    assert L.cocktail_decode_attention(C.byref(sh), 16, C.byref(cache), 0.0, 16, None, 16, 0, None) == _lib.ENOSPACE
    assert L.cocktail_decode_attention(C.byref(sh), 16, C.byref(cache), 0.0, 24, None, 16, 1 << 20, None) == _lib.EALIGN
    sh192 = ck.make_shape(1, 2, 2, 192, 8, 32)        # the planner takes any multiple of 64, the kernels 64 and 128
    p192 = ck.cocktail_plan(sh192, [16], [2, 4], 4)
    cache.plan_host = p192.blob.ctypes.data
    assert L.cocktail_decode_attention(C.byref(sh192), 16, C.byref(cache), 0.0, 16, None, 16, 1 << 20, None) == _lib.EUNSUPPORTED
    assert L.cocktail_reorder_quantize(C.byref(sh192), 16, 16, 0, 0, 0, 192, C.byref(cache), None) == _lib.EUNSUPPORTED
    sh_wide = ck.make_shape(1, 128, 1, 128, 8, 32)        # 128 query heads on one kv head: beyond COCKTAIL_MAX_Q_PER_KV
    p_wide = ck.cocktail_plan(sh_wide, [16], [2, 4], 4)
    cache.plan_host = p_wide.blob.ctypes.data
    assert L.cocktail_decode_attention(C.byref(sh_wide), 16, C.byref(cache), 0.0, 16, None, 16, 1 << 20, None) == _lib.EUNSUPPORTED
    n = C.c_size_t(0)
    assert L.cocktail_stream_read_probe(None, 1 << 30, 16, C.byref(n), None) == _lib.EINVAL
    assert L.cocktail_stream_read_probe(8, 1 << 30, 16, C.byref(n), None) == _lib.EALIGN
    assert L.cocktail_stream_read_probe(16, 1 << 20, 16, C.byref(n), None) == _lib.EINVAL


def test_paged_source_is_validated_on_the_host():
    sh = ck.make_shape(2, 2, 2, 128, 8, 32)
    plan = ck.cocktail_plan(sh, [100, 40], [2, 4] * 6 + [16] * 5, 4)
    L = _lib.lib()
    cache = _lib.Cache()
    cache.plan_host = plan.blob.ctypes.data
    cache.plan_dev = 4096
    ok = dict(k_pages=4096, v_pages=4096, page_table=4096, table_stride=7, page_size=16, num_pages=20, reserved=0,
              stride_page=2 * 16 * 128, stride_h=16 * 128, stride_t=128)

    def call(**kw):
        src = _lib.PagedSource(**{**ok, **kw})
        return L.cocktail_reorder_quantize_paged(C.byref(sh), C.byref(src), C.byref(cache), None)

    assert call(table_stride=6) == _lib.EINVAL and b"page table row" in L.cocktail_last_error()   # 100 tokens = 7 pages
    assert call(page_size=0) == _lib.EINVAL
    assert call(num_pages=0) == _lib.EINVAL
    assert call(k_pages=None) == _lib.EINVAL
    assert call(page_table=None) == _lib.EINVAL
    assert call(v_pages=4104) == _lib.EALIGN
    assert call(stride_t=100) == _lib.EINVAL
    assert call(stride_h=4) == _lib.EINVAL
    assert call(reserved=1) == _lib.EINVAL
    assert call() == _lib.EINVAL and b"cache buffer" in L.cocktail_last_error()      # geometry accepted, class buffers are NULL
    assert L.cocktail_reorder_quantize_paged(C.byref(sh), None, C.byref(cache), None) == _lib.EINVAL
    assert L.cocktail_reorder_quantize(C.byref(sh), 16, 16, 2, 0, 0, 128, C.byref(cache), None) == _lib.EINVAL


def test_append_capacity_sizes_and_validation():
    w = workloads.config(1)
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = np.concatenate(workloads.chunk_bits(w))
    p0 = ck.cocktail_plan(sh, w.seq_lens, bits, 64)
    p1 = ck.cocktail_plan(sh, w.seq_lens, bits, 64, append_capacity=130)
    assert p0.sizes.append_capacity == 0 and p0.sizes.append_bytes == 0
    assert p1.sizes.append_capacity == 130
    assert p1.sizes.append_bytes == w.batch * w.num_kv_heads * 3 * 64 * 256     # 3 blocks of 64 fp16 rows per head
    # one more partial per (sequence, kv head), at the end of its range
    assert p1.sizes.num_partials == p0.sizes.num_partials + w.batch * w.num_kv_heads
    _check_work_split(p0, w, 64)
    h = _parse(p1)
    bh_off = _arr(p1.blob, h["off"]["bh_off"], np.int32, w.batch * w.num_kv_heads + 1)
    bh_off0 = _arr(p0.blob, _parse(p0)["off"]["bh_off"], np.int32, w.batch * w.num_kv_heads + 1)
    assert (np.diff(bh_off) == np.diff(bh_off0) + 1).all()
    L = _lib.lib()
    sizes = _lib.Sizes()
    lp = np.asarray(w.seq_lens, np.int32).ctypes.data_as(C.POINTER(C.c_int32))
    bp = bits.ctypes.data_as(C.POINTER(C.c_uint8))
    bad = _lib.PlanOptions(-1, 0)
    assert L.cocktail_plan_ex(C.byref(sh), lp, bp, 4, C.byref(bad), C.byref(sizes), None, 0, None, None) == _lib.EINVAL
    for field in (0, 1, "reserved0"):
        bad = _lib.PlanOptions(0, 0)
        if field == "reserved0":
            bad.reserved0 = 1
        else:
            bad.reserved[field] = 1
        assert L.cocktail_plan_ex(C.byref(sh), lp, bp, 4, C.byref(bad), C.byref(sizes), None, 0, None, None) == _lib.EINVAL
    assert L.cocktail_plan_ex(C.byref(sh), lp, bp, 4, None, C.byref(sizes), None, 0, None, None) == _lib.OK
    w4 = workloads.config(4)
    sh4 = ck.make_shape(w4.batch, w4.num_q_heads, w4.num_kv_heads, w4.head_dim, w4.chunk_size, w4.group_size)
    bits4 = np.concatenate(workloads.chunk_bits(w4))
    assert _parse(ck.cocktail_plan(sh4, w4.seq_lens, bits4, 2048))["pool_segs"] > 0
    assert _parse(ck.cocktail_plan(sh4, w4.seq_lens, bits4, 2048, reproducible=True))["pool_segs"] == 0
    cache = _lib.Cache()
    cache.plan_host = p0.blob.ctypes.data
    assert L.cocktail_append_fp16(C.byref(sh), 16, 16, C.byref(cache), 0, None) == _lib.EINVAL   # no append buffers
    cache.plan_host = p1.blob.ctypes.data
    assert L.cocktail_append_fp16(C.byref(sh), 16, 16, C.byref(cache), 0, None) == _lib.EINVAL   # NULL buffers
    cache.k_app, cache.v_app = 4096, 4096
    assert L.cocktail_append_fp16(C.byref(sh), 16, 16, C.byref(cache), 130, None) == _lib.EINVAL
    assert L.cocktail_append_fp16(C.byref(sh), 16, 16, C.byref(cache), -1, None) == _lib.EINVAL
    assert L.cocktail_append_fp16(C.byref(sh), 8, 16, C.byref(cache), 0, None) == _lib.EALIGN
    assert L.cocktail_append_fp16(C.byref(sh), None, 16, C.byref(cache), 0, None) == _lib.EINVAL
    # decode: num_appended must fit the plan
    cache.plan_dev = 4096
    cache.num_appended = 131
    assert L.cocktail_decode_attention(C.byref(sh), 16, C.byref(cache), 0.0, 16, None, 16, 1 << 30, None) == _lib.EINVAL
    cache.plan_host = p0.blob.ctypes.data
    cache.num_appended = 1
    assert L.cocktail_decode_attention(C.byref(sh), 16, C.byref(cache), 0.0, 16, None, 16, 1 << 30, None) == _lib.EINVAL
    big = ck.make_shape(1, 1, 1, 128, 64, 32)
    with pytest.raises(ck.CocktailError) as e:
        ck.cocktail_plan(big, [1 << 24], np.full((1 << 24) // 64, 2, np.uint8), 4)
    assert e.value.code == _lib.EUNSUPPORTED


def test_chunk_bitwidths_validates_on_host():
    L = _lib.lib()
    args = (4096, 4096, 4096, 0.6, 0.1, 4096, 4096, None)   # chunk_off, query, chunks, alpha, beta, scores, bits, stream
    assert L.cocktail_chunk_bitwidths(0, 768, 10, *args) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 0, 10, *args) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, -1, *args) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, 10, 4096, 4096, 4096, 1.5, 0.1, 4096, 4096, None) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, 10, 4096, 4096, 4096, 0.6, -0.1, 4096, 4096, None) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, 10, None, 4096, 4096, 0.6, 0.1, 4096, 4096, None) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, 10, 4096, 4096, None, 0.6, 0.1, 4096, 4096, None) == _lib.EINVAL
    assert L.cocktail_chunk_bitwidths(1, 768, 10, 4096, 4098, 4096, 0.6, 0.1, 4096, 4096, None) == _lib.EALIGN
    assert L.cocktail_chunk_bitwidths(1, 768, 0, 4096, 4096, None, 0.6, 0.1, None, None, None) == _lib.OK   # nothing to do
    assert L.cocktail_selftest_arithmetic(None, None) == _lib.EINVAL
    assert L.cocktail_selftest_arithmetic(4, None) == _lib.EALIGN


@pytest.mark.parametrize("rep,quads,valu", [(1, False, False), (2, True, False), (3, True, False), (4, True, False), (5, True, False),
                                            (8, True, False), (12, True, False), (16, True, False), (11, False, False), (4, False, True), (8, False, True)])
def test_v_layout_follows_the_query_to_kv_head_ratio(rep, quads, valu):
    """Token quads where a wave serves four query heads of a kv head (ratios 2 to 8); one-wave workgroups get pools.
    Vector-ALU-only plans and ratios beyond 8 run one query head per wave: token rows, a work head per query head."""
    shape = ck.make_shape(2, 2 * rep, 2, 128, 64, 32)
    bits = np.array([2, 4, 16, 2] * 16 + [4, 2] * 16, dtype=np.uint8)
    plan = ck.cocktail_plan(shape, [64 * 64, 32 * 64], bits, 16, vector_alu_only=valu)
    assert int(plan.sizes.v_layout) == int(quads)
    h = _parse(plan)
    assert h["rep"] == rep and h["v_layout"] == int(quads)
    work_rep = {12: 6, 16: 8}.get(rep, rep) if quads else 1      # sets of query heads that read a kv head's blocks together
    assert h["work_heads"] == 2 * rep // work_rep and h["work_rep"] == work_rep
    groups = _arr(plan.blob, h["off"]["group_rec"], np.int32, 8 * h["groups"]).reshape(-1, 8)
    assert (groups[:, 0] > 0).any() == (h["work_rep"] <= 4)
    w = workloads.small("vl", 2, 2 * rep, 2, [64 * 64, 32 * 64], 64, 32)
    _check_work_split(plan, w, 16)


@pytest.mark.parametrize("rep", list(range(1, 17)) + [18, 20, 22, 27, 33, 62, 64])
def test_which_plans_have_no_pools(rep):
    """The header promises calls that repeat bit for bit, hence no pools, for plans whose workgroups serve five to eight query
    heads and for reproducible ones; all others have pools where the context is long enough."""
    sh = ck.make_shape(1, 8 * rep, 8, 128, 64, 32)
    bits = np.tile(np.array([2, 4, 16, 2], np.uint8), 256)
    per_group = max([d for d in range(1, 9) if rep % d == 0])
    assert (per_group >= 5) == (rep in (5, 6, 7, 8, 10, 12, 14, 15, 16, 18, 20, 64))
    for kw, static in ((dict(), per_group >= 5), (dict(reproducible=True), True), (dict(vector_alu_only=True), False)):
        plan = ck.cocktail_plan(sh, [65536], bits, 256, **kw)
        h = _parse(plan)
        assert h["work_rep"] == (1 if kw.get("vector_alu_only") else per_group)
        groups = _arr(plan.blob, h["off"]["group_rec"], np.int32, 8 * h["groups"]).reshape(-1, 8)
        recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * h["workers"]).reshape(-1, 16)
        assert (groups[:, 0] == 0).all() == static and (recs[:, 14] == 0).all() == static


@pytest.mark.parametrize("hq,hkv,lens,workers,mix", [
    (8, 8, [12800], 128, (0.1, 0.3, 0.6)), (32, 8, [12800], 128, (0.1, 0.3, 0.6)), (32, 32, [1024] * 32, 2048, (0.25, 0.25, 0.5)),
    (128, 32, [512] * 32, 2048, (0.25, 0.25, 0.5))])
def test_few_blocks_per_worker_are_no_promise_of_plans_without_pools(hq, hkv, lens, workers, mix):
    """Fewer than 13 blocks per worker, and pools: calls may differ in their last bits unless `reproducible` is set.  The plan says which
    it is, and the header makes no promise by the number of blocks."""
    w = workloads.small("few", len(lens), hq, hkv, lens, 64, 32, mix=mix, seed_offset=919)
    plan, bits = _plan(w, workers)
    h = _parse(plan)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * h["workers"]).reshape(-1, 16)
    assert h["gblocks"] < 13 * h["workers"] and h["pool_segs"] > 0 and (recs[:, 14] > 0).any()
    fixed = _parse(ck.cocktail_plan(plan.shape, w.seq_lens, np.concatenate(bits), workers, reproducible=True))
    assert fixed["pool_segs"] == 0
    assert "blocks per worker" not in open(os.path.join(ROOT, "include", "cocktail.h")).read()


def test_room_to_grow_keeps_the_cache_layout_from_plan_to_plan():
    """cocktail_plan_options::max_seq_lens: FP16 runs are laid out for the length a sequence may reach, so the plan
    of a longer context (more FP16 tokens at the end, Sec. III-A) describes the same buffers."""
    w = workloads.small("grow", 3, 4, 2, [300, 64, 1000], 32, 32, mix=(0.2, 0.4, 0.4), seed_offset=41)
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = workloads.chunk_bits(w)
    flat = np.concatenate(bits)
    most = [300 + 500, 64, 1000 + 70]
    plain = ck.cocktail_plan(sh, w.seq_lens, flat, 64, append_capacity=512)
    p0 = ck.cocktail_plan(sh, w.seq_lens, flat, 64, append_capacity=512, max_seq_lens=most)
    nc = _lib.NUM_CLASSES
    f = ck.cocktail_plan_field

    def layout(plan):
        base = _arr(plan.blob, f(plan, "off_blk_base"), np.int32, nc * (w.batch + 1)).reshape(w.batch + 1, nc)
        run = _arr(plan.blob, f(plan, "off_run_blocks"), np.int32, nc * w.batch).reshape(w.batch, nc)
        used = _arr(plan.blob, f(plan, "off_nblk"), np.int32, nc * w.batch).reshape(w.batch, nc)
        return base, run, used

    base, run, used = layout(p0)
    base_plain, run_plain, used_plain = layout(plain)
    assert np.array_equal(used, used_plain) and np.array_equal(run_plain, used_plain)      # without room: run = used blocks
    assert np.array_equal(run[:, :3], used[:, :3])                                          # only FP16 runs get room
    for b in range(w.batch):
        n16 = int(p0.class_tokens[b, 3])
        assert run[b, 3] == -(-(n16 + most[b] - w.seq_lens[b]) // 64)
    assert np.array_equal(np.diff(base, axis=0), run * w.num_kv_heads)
    assert [int(x) for x in p0.sizes.class_blocks] == [int(x) for x in base[-1]]
    assert int(p0.sizes.packed_bytes) == int(plain.sizes.packed_bytes)                      # algorithmic bytes: tokens only
    # (the replay of the work split does not know the partial ids of the append workgroups: plans without them)
    _check_work_split(ck.cocktail_plan(sh, w.seq_lens, flat, 64, max_seq_lens=most), w, 64)
    # a later plan: sequence 0 grew by 200 tokens (6 chunks completed, all FP16), sequence 2 by 70
    longer = [500, 64, 1070]
    bits1 = [np.concatenate([bits[b], np.full(longer[b] // 32 - len(bits[b]), 16, np.uint8)]) for b in range(3)]
    p1 = ck.cocktail_plan(sh, longer, np.concatenate(bits1), 64, append_capacity=512, max_seq_lens=most)
    base1, run1, used1 = layout(p1)
    assert np.array_equal(base1, base) and np.array_equal(run1, run)
    assert [int(x) for x in p1.sizes.class_bytes] == [int(x) for x in p0.sizes.class_bytes]
    assert np.array_equal(p1.class_tokens[:, :3], p0.class_tokens[:, :3])
    assert (p1.class_tokens[:, 3] - p0.class_tokens[:, 3]).tolist() == [200, 0, 70]
    _check_work_split(ck.cocktail_plan(sh, longer, np.concatenate(bits1), 64, max_seq_lens=most),
                      w.__class__(**{**w.__dict__, "seq_lens": tuple(longer)}), 64)
    # validation
    with pytest.raises(ck.CocktailError, match="below seq_lens"):
        ck.cocktail_plan(sh, w.seq_lens, flat, 64, max_seq_lens=[299, 64, 1000])
    with pytest.raises(ValueError):
        ck.cocktail_plan(sh, w.seq_lens, flat, 64, max_seq_lens=[300, 64])


def test_fold_rejects_plans_that_do_not_belong_together():
    """Host-side checks of cocktail_fold_appended (no kernel is launched on any of these paths)."""
    w = workloads.small("foldv", 2, 2, 2, [100, 40], 16, 32, mix=(0.2, 0.4, 0.4), seed_offset=43)
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = [np.array([4, 2, 2, 16, 2, 2], np.uint8), np.array([2, 16], np.uint8)]   # 16 INT4 tokens: one more chunk fits its block
    most = [200, 140]
    L = _lib.lib()

    def plan(lens, bit_lists, **kw):
        return ck.cocktail_plan(sh, lens, np.concatenate(bit_lists), 16, **kw)

    def grown(lens):
        return [np.concatenate([bits[b], np.full(lens[b] // 16 - len(bits[b]), 16, np.uint8)]) for b in range(2)]

    p0 = plan(w.seq_lens, bits, append_capacity=64, max_seq_lens=most)
    good = plan([110, 50], grown([110, 50]), append_capacity=64, max_seq_lens=most)
    desc = _lib.Cache()
    desc.plan_host = p0.blob.ctypes.data
    fake = 1 << 20                               # never dereferenced: every call below fails validation first
    desc.plan_dev = fake
    desc.k_app = desc.v_app = fake
    desc.k[3] = desc.v[3] = fake
    desc.num_appended = 10

    def fold(new_plan, new_dev=fake):
        return L.cocktail_fold_appended(C.byref(sh), C.byref(desc), new_plan.blob.ctypes.data if new_plan else None, new_dev, None)

    assert fold(None) == _lib.EINVAL
    assert fold(good, None) == _lib.EINVAL
    assert fold(good, fake + 4) == _lib.EALIGN
    # a different layout (planned without room to grow), fewer tokens than before, more than the append buffers hold
    assert fold(plan([110, 50], grown([110, 50]), append_capacity=64)) == _lib.EINVAL
    assert b"lays the cache out differently" in L.cocktail_last_error()
    assert fold(plan([90, 40], [bits[0][:5], bits[1]], append_capacity=64, max_seq_lens=most)) == _lib.EINVAL
    assert fold(plan([180, 50], grown([180, 50]), append_capacity=64, max_seq_lens=most)) == _lib.EINVAL
    assert b"append buffers hold" in L.cocktail_last_error()
    # a completed chunk that is not FP16: the new plan differs in more than FP16 tokens at the end
    wrong = grown([116, 50])
    wrong[0][-1] = 4
    assert fold(plan([116, 50], wrong, append_capacity=64, max_seq_lens=most)) == _lib.EINVAL
    assert b"more than FP16 tokens" in L.cocktail_last_error()
    # lockstep counting: every sequence must have grown by num_appended
    assert fold(plan([110, 45], grown([110, 45]), append_capacity=64, max_seq_lens=most)) == _lib.EINVAL
    # a plan without append buffers cannot be folded from
    desc.plan_host = plan(w.seq_lens, bits, max_seq_lens=most).blob.ctypes.data
    assert fold(good) == _lib.EINVAL


@pytest.mark.parametrize("rep,sets", [(9, 3), (10, 2), (16, 2), (24, 3), (32, 4), (64, 8), (8, 1), (11, 1)])
@pytest.mark.parametrize("workers,capacity", [(2048, 0), (2048, 1500), (64, 0), (96, 70), (100, 70), (100, 0)])
def test_the_sets_of_a_kv_head_have_twin_workers(rep, sets, workers, capacity):
    """Sets of query heads that walk the blocks of one kv head: the workers of the sets take the same blocks, segment by
    segment, and their workgroup ids differ by multiples of eight (one XCD); no partial state is shared.  Where that would leave
    more than 1/32 of the workers without work (100 workers), and without sets, the split is the plain one: every block of
    every work head once, by workers that all have some."""
    w = workloads.small(f"twin{rep}", 3, 2 * rep, 2, (40 * 64 + 17, 0, 12345), 64, 32, mix=(0.2, 0.4, 0.4), seed_offset=rep)
    sh = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    plan = ck.cocktail_plan(sh, w.seq_lens, np.concatenate(workloads.chunk_bits(w)), workers, append_capacity=capacity)
    h = _parse(plan)
    _check_work_split(plan, w, workers)
    workers = h["workers"]                                  # at most one per unit of work: 960 for two sets of this context
    whole = workers - workers % (8 * sets)
    twins = sets > 1 and whole and (workers - whole) * 32 <= workers
    assert twins == (sets > 1 and (workers >= 960 or workers == 64 and sets != 3 or workers == 96 and sets != 8))
    segs = _arr(plan.blob, h["off"]["segments"], np.int32, 8 * h["segments"]).reshape(-1, 8)
    recs = _arr(plan.blob, h["off"]["worker_rec"], np.int32, 16 * h["workers"]).reshape(-1, 16)

    if not twins:
        assert (recs[:, 0] < recs[:, 1]).sum() > 0.95 * min(workers, h["gblocks"])
        return

    def pieces(rec):   # (segment without its set, blocks) and the set of every segment of a worker's own range
        g, g1, s = rec[:3]
        out = []
        while g < g1:
            sg = segs[s]
            end = min(sg[6] + sg[5], g1)
            out.append(((sg[0], sg[1] // sets, sg[2], sg[3], sg[4] + g - sg[6], end - g), sg[1] % sets))
            g, s = end, s + 1
        return out
    work = 0
    assert all(r[0] == r[1] for r in recs[whole:])
    for i in range(whole):
        if i // 8 % sets:
            continue
        first = pieces(recs[i])
        work += len(first)
        for k in range(sets):
            other = pieces(recs[i + 8 * k])
            assert [x[0] for x in other] == [x[0] for x in first] and all(x[1] == k for x in other)
    assert work > 0


@pytest.mark.parametrize("rep,head_dim", [(1, 128), (1, 64), (3, 128), (8, 128), (8, 64), (16, 128), (11, 64)])
@pytest.mark.parametrize("lens,capacity,workers", [([1437, 888, 1], 0, 2048), ([0, 64, 63], 0, 2048), ([5000], 70, 2048), ([2049, 0], 600, 2048), ([15251, 300], 0, 1600), ([20000, 20011], 0, 288)])
def test_the_split_for_short_contexts_covers_every_unit_once(rep, head_dim, lens, capacity, workers):
    """Workgroups of eight waves on one row each: together the waves of a row's workgroups have every unit of its runs, whole blocks where
    the kernel stages those, and every part of its appended tokens; no more waves than were asked for."""
    w = workloads.small(f"short{rep}", len(lens), 2 * rep, 2, lens, 32, 32, mix=(0.2, 0.2, 0.3, 0.3), head_dim=head_dim, seed_offset=930 + rep)
    shape = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    plan = ck.cocktail_plan(shape, w.seq_lens, np.concatenate(workloads.chunk_bits(w)), workers, append_capacity=capacity)
    f = lambda n, i=0: ck.cocktail_plan_field(plan, n, i)
    h, groups = _parse(plan), f("short_groups")
    blocks_of_a_wave = h["work_rep"] > 4 and lens[0] > 15000 and (rep, head_dim, workers) != (8, 64, 288)
    if blocks_of_a_wave or rep == 11 and workers == 288:   # more staged blocks per wave than allowed; too many rows
        assert groups == 0
        return
    assert 0 < 8 * groups <= workers and f("short_units") == (0 if workers == 288 and head_dim == 128 else 1)
    recs = _arr(plan.blob, f("off_short"), np.int32, 4 * 8 * groups).reshape(groups, 8, 4)
    recs = np.stack([recs[..., 0], recs[..., 1] & 0xffff, recs[..., 1].view(np.uint32) >> 16, recs[..., 2], recs[..., 3]], axis=2).astype(np.int64)
    place = _arr(plan.blob, f("off_short_place"), np.int32, 4 * groups).reshape(groups, 4)
    rows = w.batch * h["work_heads"]
    counters = plan.blob[f("off_short_counters"):f("off_short_counters") + f("short_counter_stride_bytes") * rows]
    assert counters.size == f("short_counter_stride_bytes") * rows and not counters.any()
    assert f("off_short_counters") % 128 == 0 and f("off_short_place") == f("off_short") + 128 * groups
    upb, heads, share = 1 if head_dim == 64 else 2, h["work_heads"], h["work_heads"] // 2
    blk_base = _arr(plan.blob, f("off_blk_base"), np.int32, 4 * (w.batch + 1)).reshape(-1, 4)
    g = 0
    for b in range(w.batch):
        for hd in range(heads):
            n = place[g, 3] >> 8 & 0xfff
            assert n >= 1 and g + n <= groups and (n == 1 or groups <= max(h["partials"], 1))
            for k in range(n):
                assert place[g + k].tolist() == [b, (b * heads + hd) * h["work_rep"], w.seq_lens[b], k | n << 8 | (b * heads + hd) << 20]
            own = recs[g:g + n].reshape(-1, 5)
            for c in range(4):
                tokens = int(plan.class_tokens[b, c])
                mine = sorted((int(x[1]), int(x[2])) for x in own if x[0] == c and x[1] < x[2])
                blocks = -(-tokens // 64)
                end = blocks * upb if h["work_rep"] > 4 and c < 2 else -(-tokens * upb // 64)
                assert [x for r in mine for x in r] == ([0] + [x for r in mine[:-1] for x in (r[1], r[1])] + [end] if tokens else [])
                for x in own:
                    if x[0] == c and x[1] < x[2]:
                        assert x[3] == tokens and x[4] == blk_base[b, c] + (hd // share) * blocks
                        assert not (h["work_rep"] > 4 and c < 2) or (x[1] % upb == 0 and x[2] % upb == 0)
            app = [x for x in own if x[0] == 4]
            if capacity:
                m = len(app)
                assert sorted(int(x[1]) for x in app) == list(range(m)) and all(x[2] == m and x[4] == (2 * b + hd // share) * f("append_blocks") for x in app)
                for units in (0, 1, 2, m, -(-capacity * upb // 64)):          # the kernel's division by multiplication
                    each = units if m == 1 else ((units + m - 1) * (int(app[0][3]) & 0xffffffff)) >> 32
                    assert each == -(-units // m)
            else:
                assert not app
            g += n
    assert g == groups


def test_contexts_without_a_split_for_short_ones():
    """Long contexts, more rows than workgroups, fewer than eight workers: the plan has only the split by workers."""
    for w, workers in ((workloads.config(2), 2048), (workloads.small("rows", 40, 8, 8, [64] * 40, 64, 32), 2048), (workloads.config(1), 7)):
        plan, _ = _plan(w, workers)
        assert ck.cocktail_plan_field(plan, "short_groups") == 0


@pytest.mark.parametrize("name,refused,taken", [
    ("COST_WEIGHTS", "64,0,64,64", "64,64,64,64"), ("POOL_PERCENT", "101", "10"), ("GROUP_WORKERS", "0", "4"), ("PAIR_SPEED", "2", "0"),
    ("LAYOUT", "-1", "1"), ("PAIR_MODE", "4", "2"), ("MIN_POOL_BLOCKS", "0", "2"), ("PAIR_TABLE", "1,1", ",".join(["1.1"] * 16))])
def test_a_tuning_value_that_is_refused_leaves_the_split_for_short_contexts(name, refused, taken, monkeypatch):
    """The split knows none of the tuning variables and makes way for the one by workers where one is set, not where its value is refused."""
    w = workloads.config(1)
    groups = ck.cocktail_plan_field(_plan(w, 2048)[0], "short_groups")
    assert groups > 0
    for value, expected in ((refused, groups), (taken, 0)):
        monkeypatch.setenv("COCKTAIL_" + name, value)
        assert ck.cocktail_plan_field(_plan(w, 2048)[0], "short_groups") == expected


def test_plans_without_pools_carry_no_lines_of_counters_and_older_ones_are_taken():
    """Counters nobody draws from take little of what a request uploads; a plan written with a line for each (version 15) is still one."""
    for w, pools in ((workloads.config(1), False), (workloads.config(5), True)):
        plan, _ = _plan(w, 2048)
        f = lambda n: ck.cocktail_plan_field(plan, n)
        assert (f("num_pool_segs") > 0) == pools and f("counter_stride_bytes") == (128 if pools else 16)
        head = plan.blob[:8].view(np.uint32)
        assert head[1] == 16
        for version, known in ((15, True), (14, False), (17, False), (16, True)):
            head[1] = version
            if known:
                assert f("batch") == w.batch
            else:
                with pytest.raises(ck.CocktailError):
                    f("batch")


@pytest.mark.parametrize("rep,head_dim,lens,capacity,taken", [
    (16, 128, [15584], 0, False), (16, 128, [14346, 896], 0, False), (12, 128, [11113], 0, False), (10, 128, [9891, 2875, 11508], 0, False),
    (16, 128, [10250, 3416], 0, True), (16, 128, [6000], 0, True), (16, 128, [14586], 362, True), (16, 64, [11181], 0, True), (8, 128, [9600, 9600], 0, True), (10, 128, [5000, 5000, 5000], 0, True)])
def test_long_rows_of_sets_of_heads_keep_two_launches(rep, head_dim, lens, capacity, taken):
    """Sets of heads at head_dim 128: more than eight workgroups per row whose waves have two staged blocks and more lose by one launch while they do not fill the chip.  One block per
    wave, appended tokens, head_dim 64, no sets, shorter rows gain."""
    w = workloads.small(f"sets{rep}", len(lens), 8 * rep, 8, lens, 32, 64, mix=(0.15, 0.35, 0.5), head_dim=head_dim, seed_offset=970 + rep)
    shape = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    plan = ck.cocktail_plan(shape, w.seq_lens, np.concatenate(workloads.chunk_bits(w)), 2048, append_capacity=capacity)
    assert (ck.cocktail_plan_field(plan, "short_groups") > 0) == taken
