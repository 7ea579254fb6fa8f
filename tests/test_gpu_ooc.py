"""Out-of-core mode on the GPU (qw_set_out_of_core): results against the
oracle's top K, and the reads of index files and data objects against the
oracle's cache model (oracle/ooc.py: the C_I / C_D caches of Section 4, with
Strategies 1 and 2 and MRU eviction of Section 5.1, answered in batches)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import ooc
from paper_1907_11803_amd import lib, synth

pytestmark = pytest.mark.gpu

I32MAX = np.iinfo(np.int32).max


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def check_topk(ids_g, dist_g, ids_o, dist_o, is_u8):
    ids_g = ids_g.cpu().numpy()
    dist_g = dist_g.cpu().numpy()
    assert np.array_equal(ids_g, ids_o), np.argwhere(ids_g != ids_o)[:5]
    if is_u8:
        want = np.where(dist_o == np.iinfo(np.int64).max, I32MAX, dist_o).astype(np.int64)
        assert np.array_equal(dist_g.astype(np.int64), want)
    else:
        fin = np.isfinite(dist_o)
        assert np.array_equal(np.isfinite(dist_g), fin)
        assert np.array_equal(dist_g[fin], dist_o[fin].astype(np.float32))


class Case:
    """A workload with its oracle answer, per-query needs and cache sizes."""

    def __init__(self, wl, w):
        p = wl.params
        self.wl, self.w = wl, w
        self.a, self.b = p.a, p.b(w)
        self.is_u8 = wl.data.dtype == np.uint8
        self.dp = (wl.d + 15) // 16 * 16
        self.row_bytes = self.dp * (1 if self.is_u8 else 4)
        self.ids, self.dist, _ = oracle.lsh_query(wl.data, wl.queries, self.a, self.b, w, wl.K)
        self.ineeds = ooc.workload_needs(wl.data, wl.queries, self.a, self.b, w)
        self.cands = oracle.lsh_candidates(wl.data, wl.queries, self.a, self.b, w)
        self.L = p.L
        self.distinct = ooc.distinct_reads(self.ineeds, self.cands, self.row_bytes)
        # the largest single query's needs (a cache must hold one query)
        self.q_ids = max(sum(s for (_, _, s) in nd) for nd in self.ineeds)
        self.q_ids_layer = max((s for nd in self.ineeds for (_, _, s) in nd), default=1)
        self.q_rows = max(len(c) for c in self.cands)

    def cache(self, frac_i, frac_d, strategy):
        """Cache bytes and index share so that C_I holds about frac_i of the
        workload's distinct index bytes and C_D frac_d of its distinct rows,
        never less than one query needs."""
        ids_need = max(int(frac_i * self.distinct["index_bytes"] / 4),
                       self.q_ids_layer * self.L + self.L if strategy == 1 else self.q_ids + 1)
        rows_need = max(int(frac_d * self.distinct["data_objects"]), self.q_rows + 1)
        ci = 4 * ids_need
        cd = rows_need * self.row_bytes
        pct = max(1, min(99, int(np.ceil(100.0 * ci / (ci + cd)))))
        total = max(-(-ci * 100 // pct), -(-cd * 100 // (100 - pct)))
        return int(total) + 64, pct

    def expected_io(self, cache_bytes, pct, strategy, policy, batch):
        return ooc.simulate(self.ineeds, self.cands, self.L, self.row_bytes, cache_bytes, pct,
                            strategy, policy, batch)


@pytest.fixture(scope="module")
def u8case():
    return Case(synth.make_config(1, Q=300), 800.0)


@pytest.fixture(scope="module")
def f32case():
    return Case(synth.make_config(3, n=20000, Q=120, L=8, k=8), 10.0)


def run_ooc(case, form, cache_bytes, pct, strategy, policy, batch, keep=0):
    wl = case.wl
    ix = lib.Index(dev(wl.data), dev(case.a), dev(case.b), case.w)
    try:
        ix.set_out_of_core(cache_bytes, index_percent=pct, strategy=strategy, policy=policy,
                           batch=batch, keep=keep)
        info = ix.info()
        assert info["out_of_core"] == 1 and info["host_bytes"] >= wl.n * case.row_bytes
        ids, dist, st = ix.query(dev(wl.queries), wl.K, lib.make_opts(form=form), stats=True)
        torch.cuda.synchronize()
        return ids, dist, st
    finally:
        ix.close()


def io_of(st):
    return {"index_files": st["ooc_index_files"], "index_bytes": st["ooc_index_bytes"],
            "data_objects": st["ooc_data_objects"], "data_bytes": st["ooc_data_bytes"],
            "batches": st["ooc_batches"], "splits": st["ooc_splits"]}


@pytest.mark.parametrize("form", [lib.QW_FORM_PLAIN_FP32, lib.QW_FORM_FAST])
def test_unbounded_cache_reads_each_item_once(u8case, form):
    c = u8case
    ids, dist, st = run_ooc(c, form, 1 << 30, 50, 2, lib.QW_OOC_MRU, 37)
    check_topk(ids, dist, c.ids, c.dist, True)
    want = dict(c.distinct, batches=-(-c.wl.Q // 37), splits=0)
    assert io_of(st) == want
    assert st["cand_unique"] == sum(len(x) for x in c.cands)


@pytest.mark.parametrize("strategy,policy,batch,frac", [
    (1, lib.QW_OOC_MRU, 1, 0.3),    # the paper's setting: one query at a time, Strategy 1, MRU
    (2, lib.QW_OOC_MRU, 1, 0.3),    # Strategy 2
    (2, lib.QW_OOC_LRU, 16, 0.3),
    (1, lib.QW_OOC_MRU, 64, 0.25),  # batches that must split
    (2, lib.QW_OOC_MRU, 300, 0.1),  # one batch of the whole workload, split down
])
def test_tight_cache_matches_oracle(u8case, strategy, policy, batch, frac):
    c = u8case
    cache_bytes, pct = c.cache(frac, frac, strategy)
    want = c.expected_io(cache_bytes, pct, strategy, policy, batch)
    # the cache is small enough that something is read twice
    assert (want["index_files"] > c.distinct["index_files"] or
            want["data_objects"] > c.distinct["data_objects"])
    ids, dist, st = run_ooc(c, lib.QW_FORM_FAST, cache_bytes, pct, strategy, policy, batch)
    check_topk(ids, dist, c.ids, c.dist, True)
    assert io_of(st) == want, (io_of(st), want)


@pytest.mark.parametrize("strategy,policy,batch", [(1, lib.QW_OOC_MRU, 8), (2, lib.QW_OOC_LRU, 1)])
def test_float_rows_match_oracle(f32case, strategy, policy, batch):
    c = f32case
    cache_bytes, pct = c.cache(0.3, 0.3, strategy)
    want = c.expected_io(cache_bytes, pct, strategy, policy, batch)
    ids, dist, st = run_ooc(c, lib.QW_FORM_FAST, cache_bytes, pct, strategy, policy, batch)
    check_topk(ids, dist, c.ids, c.dist, False)
    assert io_of(st) == want, (io_of(st), want)


def test_split_sweep_at_fixed_cache(u8case):
    """The paper's evaluation sweeps C_I's share of a fixed cache: every share
    gives the oracle's results and the oracle's reads."""
    c = u8case
    cache_bytes, _ = c.cache(0.4, 0.4, 2)
    for pct in (10, 50, 90):
        try:
            want = c.expected_io(cache_bytes, pct, 2, lib.QW_OOC_MRU, 32)
        except ooc.CacheTooSmall:
            want = None
        wl = c.wl
        ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
        try:
            ix.set_out_of_core(cache_bytes, index_percent=pct, strategy=2, batch=32)
            if want is None:
                with pytest.raises(lib.QwError) as e:
                    ix.query(dev(wl.queries), wl.K)
                assert e.value.status == lib.QW_EUNSUPPORTED
                continue
            ids, dist, st = ix.query(dev(wl.queries), wl.K, stats=True)
            check_topk(ids, dist, c.ids, c.dist, True)
            assert io_of(st) == want
        finally:
            ix.close()


def test_keep_and_round_trip(u8case):
    c = u8case
    wl = c.wl
    q = dev(wl.queries)
    ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
    try:
        dev_bytes = ix.info()["device_bytes"]
        ix.set_out_of_core(1 << 28, index_percent=30, strategy=1, batch=50, keep=1)
        _, _, st1 = ix.query(q, wl.K, stats=True)
        assert io_of(st1)["data_objects"] == c.distinct["data_objects"]
        ids, dist, st2 = ix.query(q, wl.K, stats=True)  # everything is resident
        check_topk(ids, dist, c.ids, c.dist, True)
        assert st2["ooc_index_files"] == 0 and st2["ooc_data_objects"] == 0
        # new options: empty caches, host copies kept
        ix.set_out_of_core(1 << 28, index_percent=70, strategy=2, batch=300)
        ids, dist, st3 = ix.query(q, wl.K, stats=True)
        check_topk(ids, dist, c.ids, c.dist, True)
        assert io_of(st3)["index_files"] == c.distinct["index_files"]
        # back in core: same results, the data and lists on the device again
        ix.set_out_of_core(None)
        info = ix.info()
        assert info["out_of_core"] == 0 and info["host_bytes"] == 0
        assert info["device_bytes"] == dev_bytes
        for form in (lib.QW_FORM_PLAIN_FP32, lib.QW_FORM_FAST):
            ids, dist = ix.query(q, wl.K, lib.make_opts(form=form))
            check_topk(ids, dist, c.ids, c.dist, True)
        cnt = ix.candidate_counts(q).cpu().numpy()
        assert np.array_equal(cnt, [len(x) for x in c.cands])
    finally:
        ix.close()


def test_refusals_and_limits(u8case):
    c = u8case
    wl = c.wl
    q = dev(wl.queries)
    ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
    try:
        def status(fn, *a, **kw):
            try:
                fn(*a, **kw)
            except lib.QwError as e:
                return e.status
            return lib.QW_OK

        # bad options
        for kw in (dict(cache_bytes=0), dict(cache_bytes=1 << 20, index_percent=0),
                   dict(cache_bytes=1 << 20, index_percent=100), dict(cache_bytes=1 << 20, strategy=3),
                   dict(cache_bytes=1 << 20, policy=2), dict(cache_bytes=1 << 20, batch=0),
                   dict(cache_bytes=1 << 20, keep=2)):
            cb = kw.pop("cache_bytes")
            assert status(ix.set_out_of_core, cb, **kw) == lib.QW_EINVAL, kw
        # probing or counting on: refused
        ix.set_probing(1)
        assert status(ix.set_out_of_core, 1 << 28) == lib.QW_EUNSUPPORTED
        ix.set_probing(0)
        ix.set_counting(2, 10)
        assert status(ix.set_out_of_core, 1 << 28) == lib.QW_EUNSUPPORTED
        ix.set_counting(0, 0)
        ix.set_out_of_core(1 << 28)
        assert status(ix.candidate_counts, q) == lib.QW_EUNSUPPORTED
        assert status(ix.candidate_lists, q) == lib.QW_EUNSUPPORTED
        assert status(ix.bruteforce, q, 10) == lib.QW_EUNSUPPORTED
        assert status(ix.set_probing, 2, 2) == lib.QW_EUNSUPPORTED
        assert status(ix.set_counting, 2, 10) == lib.QW_EUNSUPPORTED
        assert status(ix.train_count_model, q, epochs=1) == lib.QW_EUNSUPPORTED
        assert status(ix.query, q, 10, lib.make_opts(stage_split=50)) == lib.QW_EUNSUPPORTED
        oi = torch.empty((wl.Q, 10), dtype=torch.int32, device=q.device)
        od = torch.empty((wl.Q, 10), dtype=torch.int32, device=q.device)
        assert status(lib.qw_query_workload_noalloc, ix.handle, q, 10, oi, od) == lib.QW_EUNSUPPORTED
        # hashing and bucket sizes still work
        h, _ = ix.hash(q)
        assert np.array_equal(h.cpu().numpy(), oracle.hash_points(wl.queries, c.a, c.b, c.w))
        # a cache that cannot hold one query's rows (the oracle's model agrees)
        cb = c.q_ids * 4 * 100 + 64 * 100
        assert (cb - cb * 99 // 100) // c.row_bytes < c.q_rows
        with pytest.raises(ooc.CacheTooSmall):
            c.expected_io(cb, 99, 2, lib.QW_OOC_MRU, 4)
        ix.set_out_of_core(cb, index_percent=99, strategy=2, batch=4)
        assert status(ix.query, q, 10) == lib.QW_EUNSUPPORTED
    finally:
        ix.close()


def test_kept_caches_continue_the_workload(u8case):
    """keep = 1: two calls of 150 queries read what one workload of 300 reads
    in batches of 50 (recency continues across the calls), each call's share
    as the oracle's model gives it."""
    c = u8case
    wl = c.wl
    cache_bytes, pct = c.cache(0.3, 0.3, 1)
    want_all = c.expected_io(cache_bytes, pct, 1, lib.QW_OOC_MRU, 50)
    want_first = ooc.simulate(c.ineeds[:150], c.cands[:150], c.L, c.row_bytes, cache_bytes, pct,
                              1, lib.QW_OOC_MRU, 50)
    ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
    try:
        ix.set_out_of_core(cache_bytes, index_percent=pct, strategy=1, batch=50, keep=1)
        got = []
        for lo, hi in ((0, 150), (150, 300)):
            ids, dist, st = ix.query(dev(wl.queries[lo:hi]), wl.K, stats=True)
            check_topk(ids, dist, c.ids[lo:hi], c.dist[lo:hi], True)
            got.append(io_of(st))
        assert got[0] == want_first
        assert {k: got[0][k] + got[1][k] for k in got[0]} == want_all
    finally:
        ix.close()


def test_large_k_and_ragged_batches(f32case, u8case):
    """K beyond the in-kernel top K (64: the FP64 re-rank of the float band
    through the slot directory), a batch size that does not divide Q, and a
    batch larger than Q: results and reads as the oracle gives them."""
    c = f32case
    wl = c.wl
    ids_o, dist_o, _ = oracle.lsh_query(wl.data, wl.queries, c.a, c.b, c.w, 64)
    cache_bytes, pct = c.cache(0.3, 0.3, 2)
    want = c.expected_io(cache_bytes, pct, 2, lib.QW_OOC_MRU, 7)
    ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
    try:
        ix.set_out_of_core(cache_bytes, index_percent=pct, strategy=2, batch=7)
        ids, dist, st = ix.query(dev(wl.queries), 64, stats=True)
        check_topk(ids, dist, ids_o, dist_o, False)
        assert io_of(st) == want
    finally:
        ix.close()
    c = u8case
    wl = c.wl
    want = c.expected_io(1 << 30, 50, 1, lib.QW_OOC_LRU, 1000)
    assert want["batches"] == 1
    ids, dist, st = run_ooc(c, lib.QW_FORM_PLAIN_FP32, 1 << 30, 50, 1, lib.QW_OOC_LRU, 1000)
    check_topk(ids, dist, c.ids, c.dist, True)
    assert io_of(st) == want


def test_autotune_picks_the_fastest_share(u8case):
    """qw_autotune_ooc times the eleven index shares of a fixed cache: each
    share's reads are the oracle's for that share (or the share is refused
    where the oracle's model cannot hold one query), the fastest is chosen and
    the index is left out of core at it, with the oracle's results."""
    c = u8case
    wl = c.wl
    cache_bytes, _ = c.cache(0.3, 0.3, 2)
    ix = lib.Index(dev(wl.data), dev(c.a), dev(c.b), c.w)
    try:
        r = ix.autotune_ooc(dev(wl.queries), wl.K, cache_bytes, strategy=2, batch=25)
        fits = []
        for sh in r["shares"]:
            try:
                want = c.expected_io(cache_bytes, sh["index_percent"], 2, lib.QW_OOC_MRU, 25)
            except ooc.CacheTooSmall:
                assert sh["ms"] < 0, sh
                continue
            assert sh["ms"] > 0
            got = {"index_bytes": sh["index_bytes"], "data_bytes": sh["data_bytes"],
                   "batches": sh["batches"], "splits": sh["splits"]}
            assert got == {k: want[k] for k in got}, (sh["index_percent"], got, want)
            fits.append(sh)
        assert len(fits) >= 3
        assert r["index_percent"] == min(fits, key=lambda x: x["ms"])["index_percent"]
        info = ix.info()
        assert info["out_of_core"] == 1 and info["ooc_index_percent"] == r["index_percent"]
        ids, dist = ix.query(dev(wl.queries), wl.K)
        check_topk(ids, dist, c.ids, c.dist, True)
    finally:
        ix.close()


@pytest.mark.parametrize("batch,cache_mb", [(64, 256), (64, 24), (200, 16), (200, 12)])
def test_reads_in_flight(batch, cache_mb):
    """Batches of several MB of rows, whose reads outlast the next batches'
    planning: without evictions, with some, and with splits."""
    rng = np.random.default_rng(batch + cache_mb)
    n, d, Q = 60000, 512, 1000
    centres = rng.integers(40, 216, (60, d))
    data = np.clip(centres[rng.integers(0, 60, n)] + rng.normal(0, 20, (n, d)), 0, 255).astype(np.uint8)
    q = np.clip(centres[rng.integers(0, 60, Q)] + rng.normal(0, 20, (Q, d)), 0, 255).astype(np.uint8)
    p = synth.hash_params(3, 8, 6, d, 2500.0)
    ids_o, dist_o, _ = oracle.lsh_query(data, q, p.a, p.b(), 2500.0, 10)
    ix = lib.Index(dev(data), dev(p.a), dev(p.b()), 2500.0)
    ix.set_out_of_core(cache_mb << 20, index_percent=30, strategy=2, batch=batch)
    if cache_mb == 12:  # one query's 16,000 rows do not fit
        with pytest.raises(lib.QwError):
            ix.query(dev(q), 10)
        ix.set_out_of_core(24 << 20, index_percent=30, strategy=2, batch=batch)
    for _ in range(2):
        ids, dist, st = ix.query(dev(q), 10, stats=True)
        check_topk(ids, dist, ids_o, dist_o, True)
    assert st["ooc_data_bytes"] > 20 << 20
    ix.close()
