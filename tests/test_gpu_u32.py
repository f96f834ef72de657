"""GPU parity of integer-key jobs (all four containers x all reduce ops) against the CPU oracle, bit-exact."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

STRATS = {"lds_array": 2, "global_array": 3, "hash": 4, "sort": 5}
OPS = {"count": 0, "sum": 1, "min": 2, "max": 3}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


_jobs = {}


def _job(strategy, **kw):
    from paper_1309_0215_amd import Job
    key = (strategy, tuple(sorted(kw.items())))
    if key not in _jobs:
        _jobs[key] = Job(device=0, strategy=strategy, **kw)
    return _jobs[key]


def _run(torch, job, keys, vals, op, R):
    kt = torch.from_numpy(keys.view(np.int32)).to("cuda:0")
    vt = None if vals is None else torch.from_numpy(vals.view(np.int32)).to("cuda:0")
    return job.u32(kt, vt, op=OPS[op], key_range=R)


def _check(res, keys, vals, op):
    ek, ev = oracle.u32(keys, vals, op)
    gk = res.keys.cpu().numpy().view(np.uint32)
    gv = res.values.cpu().numpy()
    gv = gv.view(np.uint64) if op == "sum" else gv.view(np.uint32).astype(np.uint64)
    assert np.array_equal(gk, ek), (len(gk), len(ek))
    assert np.array_equal(gv, ev)


@pytest.mark.parametrize("strat", list(STRATS))
@pytest.mark.parametrize("op", list(OPS))
def test_strategies_ops(torch, strat, op):
    R = 3000
    n = 200_001
    keys, vals = gen.u32_keys(11, n, R, 1.1, with_values=True)
    if op == "count":
        vals = None
    res = _run(torch, _job(STRATS[strat]), keys, vals, op, R)
    _check(res, keys, vals, op)
    assert res.stats["strategy_used"] == STRATS[strat]


@pytest.mark.parametrize("strat", ["hash", "sort"])
def test_no_range_high_cardinality(torch, strat):
    rng = np.random.default_rng(5)
    keys = rng.integers(0, 2**32, size=300_000, dtype=np.uint64).astype(np.uint32)
    keys[:100] = 0xFFFFFFFF
    keys[100:200] = 0
    vals = rng.integers(0, 2**32, size=len(keys), dtype=np.uint64).astype(np.uint32)
    for op in OPS:
        v = None if op == "count" else vals
        _check(_run(torch, _job(STRATS[strat]), keys, v, op, 0), keys, v, op)


def test_rule_picks_by_range(torch):
    j = _job(0)
    keys, _ = gen.u32_keys(3, 100_000, 1000, 1.0)
    r = _run(torch, j, keys, None, "count", 1000)
    assert r.stats["strategy_used"] == STRATS["lds_array"]
    _check(r, keys, None, "count")
    keys2, _ = gen.u32_keys(4, 100_000, 1 << 20, 1.0)
    r = _run(torch, j, keys2, None, "count", 1 << 20)
    assert r.stats["strategy_used"] == STRATS["global_array"]
    _check(r, keys2, None, "count")
    r = _run(torch, j, keys2, None, "count", 0)
    assert r.stats["strategy_used"] == STRATS["hash"]
    _check(r, keys2, None, "count")


def test_empty_input(torch):
    for s in STRATS.values():
        j = _job(s)
        e = np.zeros(0, np.uint32)
        r = _run(torch, j, e, None, "count", 100)
        assert len(r.keys) == 0


def test_key_outside_range_is_rejected(torch):
    from paper_1309_0215_amd import MRError
    keys = np.arange(1000, dtype=np.uint32)
    for s in STRATS.values():
        with pytest.raises(MRError) as e:
            _run(torch, _job(s), keys, None, "count", 500)
        assert e.value.status == -1
    # the containers stay clean after the rejected runs
    for s in STRATS.values():
        k2 = (np.arange(5000) % 400).astype(np.uint32)
        _check(_run(torch, _job(s), k2, None, "count", 500), k2, None, "count")


def test_sum_wide_values(torch):
    keys = np.repeat(np.arange(50, dtype=np.uint32), 40_000)
    vals = np.full(len(keys), 0xFFFFFFFF, np.uint32)
    for s in STRATS.values():
        _check(_run(torch, _job(s), keys, vals, "sum", 50), keys, vals, "sum")


def test_hash_forced_collisions_and_regrowth(torch):
    keys, _ = gen.u32_keys(8, 60_000, 5000, 0.5)
    _check(_run(torch, _job(4, debug_hash=1), keys, None, "count", 0), keys, None, "count")
    keys2, _ = gen.u32_keys(9, 400_000, 200_000, 0.3)
    r = _run(torch, _job(4, table_slots=4096), keys2, None, "count", 0)
    _check(r, keys2, None, "count")
    assert r.stats["retries"] >= 1


def test_capacity_error(torch):
    import ctypes as C
    from paper_1309_0215_amd import _lib as L
    j = _job(4)
    keys = np.arange(1000, dtype=np.uint32)
    kt = torch.from_numpy(keys.view(np.int32)).to("cuda:0")
    ko = torch.empty(10, dtype=torch.int32, device="cuda:0")
    vo = torch.empty(10, dtype=torch.int32, device="cuda:0")
    o = L.Output()
    o.keys, o.values, o.cap_keys = ko.data_ptr(), vo.data_ptr(), 10
    st = j.lib.mr_run(j.h, L.MAP_U32_KEYS, L.REDUCE_COUNT, kt.data_ptr(), 4000, None, 0, 0, C.byref(o))
    assert st == L.MR_ERR_CAPACITY and o.n_keys == 1000


@pytest.mark.parametrize("strat", list(STRATS))
def test_large_zipf(torch, strat):
    R = 1 << 16 if strat != "lds_array" else 4096
    keys, vals = gen.u32_keys(21, 4_000_000, R, 1.0, with_values=True)
    _check(_run(torch, _job(STRATS[strat]), keys, vals, "sum", R), keys, vals, "sum")


def test_mixed_kinds_on_one_job(torch):
    # One job alternating integer keys, word count, histogram and k-means:
    # every kind keeps its own buffers valid across the others' runs.
    from paper_1309_0215_amd import Job
    j = Job(device=0, strategy=4, km_centroids=torch.from_numpy(gen.kmeans(3, n=64)[1]).cuda())
    keys, vals = gen.u32_keys(12, 100_000, 5000, 1.0, with_values=True)
    txt = gen.text(13, 200_000, V=3000)
    rgb = gen.rgb(14, 3 * 10_000)
    X, _ = gen.kmeans(3, n=5000)
    for rep in range(3):
        _check(_run(torch, j, keys, vals, "sum", 0), keys, vals, "sum")
        w = j.words(torch.from_numpy(txt).cuda())
        assert w.items() == oracle.words(txt).items()
        _check(_run(torch, j, keys, None, "count", 0), keys, None, "count")
        h, _ = j.rgb_hist(torch.from_numpy(rgb).cuda())
        assert np.array_equal(h.cpu().numpy().astype(np.uint64), oracle.rgb(rgb))
        a, s, c, cent, st = j.kmeans(torch.from_numpy(X).cuda())
        assert int(c.sum()) == len(X)


@pytest.mark.parametrize("n", [524_288, 524_289])
def test_sort_at_the_one_workgroup_scan_limit(torch, n):
    """The sort's digit histograms (256 digits x 2048-element tiles) are
    scanned by one workgroup up to 65,536 entries: 524,288 pairs fill that
    exactly (64 steps of 64 entries per wave), one more pair takes the
    three-kernel scan."""
    keys, vals = gen.u32_keys(31, n, 1 << 20, 1.0, with_values=True)
    res = _run(torch, _job(STRATS["sort"]), keys, vals, "sum", 1 << 20)
    assert res.stats["strategy_used"] == STRATS["sort"]
    _check(res, keys, vals, "sum")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 8191, 8192, 8193, 16_385, 131_073])
@pytest.mark.parametrize("strat", ["hash", "sort"])
def test_sorted_runs_at_tile_and_chunk_edges(torch, strat, n):
    """The radix sort takes tiles of 8192 elements and the reduce chunks of
    1024 in rows of 64: sizes at those edges, with runs of one key (longer
    than chunks and tiles), of every element its own key, and keys that differ
    in their top byte, their middle bytes or one bit only (passes skipped)."""
    rng = np.random.default_rng(n)
    i = np.arange(n, dtype=np.uint64)
    inputs = [np.full(n, 0xFFFFFFFF), i * 2654435761 % 2**32, (i % 3) << 24, (i % 700) << 8, (i // 1500) & 1,
              rng.integers(0, 50, n) ** 4 % 2**32]
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    for x in inputs:
        keys = np.asarray(x).astype(np.uint32)
        for op in OPS:
            _check(_run(torch, _job(STRATS[strat]), keys, None if op == "count" else vals, op, 0), keys,
                   None if op == "count" else vals, op)


def test_sort_of_keys_4_bytes_past_a_16_byte_boundary(torch):
    keys, _ = gen.u32_keys(41, 20_001, 5000, 0.5)
    kt = torch.from_numpy(keys.view(np.int32)).to("cuda:0")[1:]
    assert kt.data_ptr() % 16 == 4
    for strat in ("hash", "sort"):
        _check(_job(STRATS[strat]).u32(kt), keys[1:], None, "count")


# rare keys beside one frequent key, so that a sample of 8192 elements holds
# few distinct keys: as many claimed slots as one workgroup orders (4096) and
# one more, and more keys than the small table holds (2^18 slots)
@pytest.mark.parametrize("n,rare", [((1 << 20) - 1, 4095), (1 << 20, 4095), (1 << 20, 4096), (6_000_000, 300_000)])
def test_hash_of_few_frequent_keys(torch, n, rare):
    rng = np.random.default_rng(rare)
    keys = np.full(n, 77, np.uint32)
    at = rng.permutation(n)[:rare]
    keys[at] = 1000 + np.arange(rare, dtype=np.uint32) * 13
    keys[at[0]] = 0xFFFFFFFF  # kept beside the table
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    for op in OPS if rare < 10_000 else ["sum"]:
        r = _run(torch, _job(STRATS["hash"]), keys, None if op == "count" else vals, op, 0)
        assert r.stats["strategy_used"] == STRATS["hash"]
        _check(r, keys, None if op == "count" else vals, op)
    # the table is clean for the next job
    _check(_run(torch, _job(STRATS["hash"]), keys[: 1 << 20], vals[: 1 << 20], "max", 0), keys[: 1 << 20], vals[: 1 << 20], "max")


# the global array filled by key-range partitions: element counts at its
# smallest input (2^18; one less takes atomics) and around its tiles (8192
# pairs, 16,384 counted elements); ranges just past the LDS array's budget, at
# whole partitions of 2^12 keys, and at the last range of each partition size
# (2^21, 2^24, 2^25 for values, 2^22, 2^23, 2^26 for counts) and past it
@pytest.mark.parametrize("n,R", [((1 << 18) - 1, 20_000), (1 << 18, 20_000), ((1 << 18) + 8191, 16_385),
                                 ((1 << 18) + 8192, 16_384 + 8192), ((1 << 18) + 8193, 1 << 20), (300_000, 1 << 21),
                                 (300_000, (1 << 21) + 1), (300_000, (1 << 22) + 1), (300_000, (1 << 24) - 1),
                                 (300_000, (1 << 24) + 1), (280_000, 1 << 25), (280_000, (1 << 25) + 1),
                                 (280_000, (1 << 26) + 1)])
@pytest.mark.parametrize("share", [0.0, 0.95])
def test_global_array_partitions_with_values(torch, n, R, share):
    """`share` of the elements hold one key, which splits its partition over
    many workgroups; the others are uniform, both ends of the range present."""
    rng = np.random.default_rng(n + R)
    keys = rng.integers(0, R, n).astype(np.uint32)
    keys[rng.random(n) < share] = R // 3
    keys[:2] = 0, R - 1
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    j = _job(STRATS["global_array"])
    for op in OPS:
        r = _run(torch, j, keys, vals, op, R)
        assert r.stats["strategy_used"] == STRATS["global_array"]
        _check(r, keys, vals, op)
    _check(_run(torch, j, keys, None, "count", R), keys, None, "count")


# the LDS array: one workgroup's elements and one more, 32 partial rows (added
# by the output kernel) and 33 (by the reduce kernel); arrays of 1 to 32
# copies, and the last sizes of the output kernel's 1, 4 and most keys per thread
@pytest.mark.parametrize("n", [1, 4096, 4097, 32 * 4096, 32 * 4096 + 1])
@pytest.mark.parametrize("R", [1, 2, 16, 1024, 1025, 4096, 4097, 5461])
def test_lds_array_edges(torch, n, R):
    rng = np.random.default_rng(n + R)
    keys = rng.integers(0, R, n).astype(np.uint32)
    keys[rng.random(n) < 0.5] = R - 1
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    j = _job(STRATS["lds_array"])
    for op in OPS:
        if op == "sum" and R > 5460:
            continue
        r = _run(torch, j, keys, None if op == "count" else vals, op, R)
        assert r.stats["strategy_used"] == STRATS["lds_array"]
        _check(r, keys, None if op == "count" else vals, op)


@pytest.mark.parametrize("op,R", [("count", 16_384), ("min", 8192), ("max", 8192), ("sum", 5460)])
def test_lds_array_largest_ranges(torch, op, R):
    keys, vals = gen.u32_keys(51, 300_000, R, 0.3, with_values=True)
    r = _run(torch, _job(STRATS["lds_array"]), keys, None if op == "count" else vals, op, R)
    _check(r, keys, None if op == "count" else vals, op)


def test_states_after_rejected_and_short_calls(torch):
    """A job clears its next state as it ends: calls that end in an error, or
    whose outputs are too small, leave the next call's state clean."""
    from paper_1309_0215_amd import Job, MRError
    keys, vals = gen.u32_keys(61, 300_000, 3000, 0.5, with_values=True)
    for strat in STRATS.values():
        j = Job(device=0, strategy=strat)
        for _ in range(3):
            with pytest.raises(MRError):
                _run(torch, j, keys, None, "count", 100)
            _check(_run(torch, j, keys, vals, "sum", 3000), keys, vals, "sum")
            kt = torch.from_numpy(keys.view(np.int32)).to("cuda:0")
            _check(j.u32(kt, key_range=3000, cap_keys=5), keys, None, "count")  # retried at the size needed


@pytest.mark.parametrize("strat", list(STRATS))
def test_separate_and_interleaved_pairs_agree(torch, strat):
    """mr_run_pairs (keys and values in two arrays, 4 bytes past a 16-byte
    boundary) against mr_run on interleaved pairs and the oracle; the binding
    interleaves what is not one-dimensional, and strided input."""
    import ctypes as C
    from paper_1309_0215_amd import _lib as L
    R = 3000
    keys, vals = gen.u32_keys(71, 300_002, R, 0.8, with_values=True)
    kt, vt = (torch.from_numpy(x.view(np.int32)).to("cuda:0") for x in (keys, vals))
    j = _job(STRATS[strat])
    inter = torch.stack([kt, vt], dim=1).contiguous()
    for op in OPS:
        r = j.u32(kt[1:], vt[1:], op=OPS[op], key_range=R)
        _check(r, keys[1:], vals[1:], op)
        ko = torch.empty(R, dtype=torch.int32, device="cuda:0")
        vo = torch.empty(R, dtype=torch.int64 if op == "sum" else torch.int32, device="cuda:0")
        o = L.Output()
        o.keys, o.values, o.cap_keys = ko.data_ptr(), vo.data_ptr(), R
        L.check(j.lib.mr_run(j.h, L.MAP_U32_KV, OPS[op], inter.data_ptr(), inter.numel() * 4, None, 0, R, C.byref(o)))
        nk = int(o.n_keys)
        _check(type(r)(ko[:nk], vo[:nk], {}), keys, vals, op)
    _check(j.u32(kt[::2], vt[::2], op=OPS["sum"], key_range=R), keys[::2], vals[::2], "sum")
    half = len(keys) // 2
    a = j.u32(kt.view(half, 2), vt.view(half, 2), op=OPS["max"], key_range=1 << 32 if strat in ("hash", "sort") else 0) \
        if strat in ("hash", "sort") else None
    if a is not None:  # stacked along dim 1: (k0, k1), (v0, v1) per row
        two = np.stack([keys.reshape(half, 2), vals.reshape(half, 2)], axis=1).reshape(-1, 2)
        _check(a, np.ascontiguousarray(two[:, 0]), np.ascontiguousarray(two[:, 1]), "max")


def test_pairs_entry_rejects_what_mr_run_rejects(torch):
    import ctypes as C
    from paper_1309_0215_amd import Job, _lib as L
    j = _job(STRATS["sort"])
    k = torch.zeros(16, dtype=torch.int32, device="cuda:0")
    o = L.Output()
    o.keys, o.values, o.cap_keys = k.data_ptr(), k.data_ptr(), 16
    run = j.lib.mr_run_pairs
    assert run(None, 1, k.data_ptr(), k.data_ptr(), 4, 0, C.byref(o)) == L.MR_ERR_INVALID_ARG
    assert run(j.h, 1, None, k.data_ptr(), 4, 0, C.byref(o)) == L.MR_ERR_INVALID_ARG
    assert run(j.h, 1, k.data_ptr() + 2, k.data_ptr(), 4, 0, C.byref(o)) == L.MR_ERR_INVALID_ARG
    assert run(j.h, 1, k.data_ptr(), k.data_ptr() + 1, 4, 0, C.byref(o)) == L.MR_ERR_INVALID_ARG
    assert run(j.h, 9, k.data_ptr(), k.data_ptr(), 4, 0, C.byref(o)) == L.MR_ERR_INVALID_ARG
    assert run(j.h, 1, k.data_ptr(), k.data_ptr(), 1 << 32, 0, C.byref(o)) == L.MR_ERR_UNSUPPORTED
    assert run(Job(device=0, strategy=1).h, 1, k.data_ptr(), k.data_ptr(), 4, 0, C.byref(o)) == L.MR_ERR_UNSUPPORTED
    assert run(j.h, 1, None, None, 0, 0, C.byref(o)) == L.MR_OK and o.n_keys == 0


# a caller workspace that holds a table for the declared range but not the
# sort of all elements
@pytest.mark.parametrize("n,R,op", [(20_011, 1_000, "count"), (300_000, 1_000, "sum"), (1 << 20, 20_000, "count"), (1_200_007, 300, "max")])
def test_hash_table_in_a_small_workspace(torch, n, R, op):
    from paper_1309_0215_amd import Job, _lib as L
    rng = np.random.default_rng(n)
    keys = torch.from_numpy(rng.integers(0, R, n).astype(np.int32)).to("cuda:0")
    vals = torch.from_numpy(rng.integers(0, 1 << 31, n).astype(np.int32)).to("cuda:0") if op != "count" else None
    code = {"count": L.REDUCE_COUNT, "sum": L.REDUCE_SUM, "max": L.REDUCE_MAX}[op]
    want = Job(device=0, strategy=L.STRAT_SORT).u32(keys, vals, op=code, key_range=R)
    slots = max(4096, 1 << (2 * R - 1).bit_length())
    ws = torch.empty(4096 + 20 * slots + 128 * R + 8192, dtype=torch.uint8, device="cuda:0")
    assert ws.numel() < 4 * n + 20 * slots or n < 100_000
    job = Job(device=0, strategy=L.STRAT_HASH, workspace=ws)
    for _ in range(2):
        r = job.u32(keys, vals, op=code, key_range=R)
        assert r.stats["device_allocs"] == 0 and r.stats["strategy_used"] == L.STRAT_HASH
        assert torch.equal(r.keys, want.keys) and torch.equal(r.values, want.values)


def test_global_array_of_nearly_2_32_keys_in_one_range(torch):
    """The most elements an input may have (16 GiB of keys), all but one in one
    key range: its share over the elements of a workgroup is rounded up."""
    n, R = (1 << 32) - 1, 20_000
    keys = torch.full((n,), 3, dtype=torch.int32, device="cuda:0")
    keys[-1] = R - 1
    r = _job(STRATS["global_array"]).u32(keys, key_range=R)
    assert r.keys.tolist() == [3, R - 1]
    assert [x & 0xFFFFFFFF for x in r.values.tolist()] == [n - 1, 1]


def _frequent_and_rare(torch, n, rare):
    """n keys: 500 frequent ones, and `rare` others once each; (keys, counts of the frequent)."""
    g = torch.Generator(device="cuda:0").manual_seed(n + rare)
    k = torch.randint(0, 500, (n,), generator=g, device="cuda:0")
    at = torch.randperm(n, generator=g, device="cuda:0")[:rare]
    k[at] = 1000 + torch.arange(rare, device="cuda:0") * 13
    return k.int(), torch.bincount(k[k < 500], minlength=500)


# Few frequent keys and rare ones: as many as the table has room for, far more
# than the small table of short inputs (its slots follow the input's length),
# and so many that the sample's estimate sends the input to the sort.
@pytest.mark.parametrize("n,rare,slots", [(1 << 26, 400_000, 1 << 21), (1 << 24, 80_000, 1 << 19), ((1 << 24) + 1, 80_000, 1 << 20),
                                          (1 << 24, 600_000, 0)])
def test_hash_of_frequent_and_rare_keys(torch, n, rare, slots):
    keys, freq = _frequent_and_rare(torch, n, rare)
    r = _job(STRATS["hash"]).u32(keys, cap_keys=rare + 1000)
    assert r.stats["table_slots"] == slots
    assert torch.equal(r.keys[:500], torch.arange(500, device="cuda:0").int())
    assert torch.equal(r.keys[500:], (1000 + torch.arange(rare, device="cuda:0") * 13).int())
    assert torch.equal(r.values[:500].long(), freq)
    assert (r.values[500:] == 1).all()


def test_hash_table_that_fills(torch):
    """Keys met twice in the sample lower its estimate: the input takes the
    table, more than half its slots are claimed, and it is sorted after all;
    the table is clean for the next job."""
    rng = np.random.default_rng(3)
    n, rare = 6_000_000, 250_000
    keys = rng.integers(0, 250, n).astype(np.uint32)
    some = rng.permutation(n)
    keys[some[:1_300_000]] = 1000 + rng.integers(0, 800, 1_300_000)
    keys[some[-rare:]] = 5000 + np.arange(rare, dtype=np.uint32) * 13
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    j = _job(STRATS["hash"])
    for op in OPS:
        r = _run(torch, j, keys, None if op == "count" else vals, op, 0)
        _check(r, keys, None if op == "count" else vals, op)
        few = keys[:1 << 20] % 250
        r = _run(torch, j, few, vals[:1 << 20], "sum", 0)
        assert r.stats["table_slots"] == 1 << 18
        _check(r, few, vals[:1 << 20], "sum")


def test_hash_of_keys_that_recur_with_a_sample(torch):
    """One key at every 2048th place of 2^24, every other element its own key."""
    n = 1 << 24
    keys = torch.arange(n, device="cuda:0").int()
    keys[::2048] = 5
    r = _job(STRATS["hash"]).u32(keys, cap_keys=n)
    k, c = torch.unique(keys, return_counts=True)
    assert torch.equal(r.keys, k) and torch.equal(r.values.long(), c)


# key ranges that the tiles of the input share unevenly: all of a range in a
# few whole tiles (sorted keys), in some tiles and not in others, or in a stretch
# of the input beside uniform keys; ranges of one workgroup and of several
@pytest.mark.parametrize("n", [300_000, 1_100_000, 2_200_000])
@pytest.mark.parametrize("R", [1 << 15, 1 << 20, 1 << 24])
@pytest.mark.parametrize("kind", ["sorted", "blocks", "stretch", "one"])
def test_global_array_of_unevenly_spread_keys(torch, n, R, kind):
    rng = np.random.default_rng(n + R)
    keys = rng.integers(0, R, n)
    if kind == "sorted":
        keys.sort()
    elif kind == "blocks":
        at = np.arange(n) // 16_384 % 8  # one eighth of the tiles holds the first keys alone
        keys[at == 3] %= 3000
    elif kind == "stretch":
        keys[n // 2: n // 2 + n // 4] = R // 2 + rng.integers(0, 50, n // 4)
    else:
        keys[:] = R - 1
    keys = keys.astype(np.uint32)
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    j = _job(STRATS["global_array"])
    for op in OPS:
        _check(_run(torch, j, keys, None if op == "count" else vals, op, R), keys, None if op == "count" else vals, op)


# pairs on 64 times as many keys, where atomics on the array take the
# partitions' place, and one pair more; the last range of the largest
# partitions of values (2^25 keys) and past it
@pytest.mark.parametrize("n,R", [(1 << 18, 1 << 24), ((1 << 18) + 1, 1 << 24), (600_000, 1 << 25), (600_000, (1 << 25) + 1)])
def test_global_array_of_few_pairs_on_many_keys(torch, n, R):
    rng = np.random.default_rng(n)
    keys = rng.integers(0, R, n).astype(np.uint32)
    keys[:2] = 0, R - 1
    vals = rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)
    j = _job(STRATS["global_array"])
    for op in OPS:
        for _ in range(2):  # the arrays are clean for the next job
            _check(_run(torch, j, keys, vals, op, R), keys, vals, op)


def _reduced(torch, keys, vals, op):
    """Distinct keys ascending and their reduced values, in 64 bits."""
    k, inv, n = torch.unique(keys.long() & 0xFFFFFFFF, return_inverse=True, return_counts=True)
    if op == "count":
        return k, n
    v = vals.long() & 0xFFFFFFFF
    if op == "sum":
        return k, torch.zeros_like(k).index_add_(0, inv, v)
    return k, torch.zeros_like(k).scatter_reduce_(0, inv, v, "a" + op, include_self=False)


# Inputs past 2^20 elements take tiles of 8192 (one whole tile more, one element
# of the next, one short of it) and chunks of 1024; 2^26 and one more fill the
# chunk counts' scan by one workgroup (65,536) and pass it.
@pytest.mark.parametrize("n,kinds", [((1 << 20) + d, ("one", "own", "some")) for d in (1, 1023, 1024, 1025, 8191, 8192, 8193)]
                         + [((1 << 26) + d, ("runs",)) for d in (0, 1)])
def test_sort_of_large_inputs_at_tile_and_chunk_edges(torch, n, kinds):
    g = torch.Generator(device="cuda:0").manual_seed(n)
    i = torch.arange(n, device="cuda:0")
    vals = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda:0").int()
    for kind in kinds:
        if kind == "one":
            k = torch.full_like(i, 0xFFFFFFFF)
        elif kind == "own":
            k = i * 2654435761 % (1 << 32)
        elif kind == "some":
            k = torch.randint(0, 50, (n,), generator=g, device="cuda:0") ** 4
        else:  # runs of 1500, longer than a chunk, out of order
            k = (i // 1500 * 7919) % 65_536
        keys = torch.where(k >= 1 << 31, k - (1 << 32), k).int()
        for op in OPS if n < 1 << 26 else ("count", "sum"):
            r = _job(STRATS["sort"]).u32(keys, None if op == "count" else vals, op=OPS[op], cap_keys=n if kind == "own" else 65_536)
            k, v = _reduced(torch, keys, vals, op)
            assert torch.equal(r.keys.long() & 0xFFFFFFFF, k)
            assert torch.equal(r.values.long() if op == "sum" else r.values.long() & 0xFFFFFFFF, v)


def test_global_array_in_workspaces_around_its_need(torch):
    """The partitions with all their slices, with one slice where those do not
    fit, and atomics where nothing more fits."""
    from paper_1309_0215_amd import Job, _lib as L, workspace_bytes
    n, R = 2_200_000, 1 << 16
    keys, vals = gen.u32_keys(81, n, R, 0.6, with_values=True)
    keys.sort()
    need = workspace_bytes(L.MAP_U32_KV, 8 * n, R, strategy=STRATS["global_array"])
    for less in (0, 256, 1 << 20):
        ws = torch.empty(need - less, dtype=torch.uint8, device="cuda:0")
        j = Job(device=0, strategy=STRATS["global_array"], workspace=ws)
        for _ in range(2):
            r = _run(torch, j, keys, vals, "sum", R)
            assert r.stats["device_allocs"] == 0
            _check(r, keys, vals, "sum")
