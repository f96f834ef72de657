"""GPU parity of word count (MR_MAP_WORDS) against the CPU oracle, element by element.

Cases: hand-worked inputs, random bytes with every separator, NUL and high
bytes, words that straddle 16-byte chunks and 16 KiB tiles, words longer than
16 and 32 bytes, unaligned input pointers, record offsets, forced hash
collisions, a table too small at the start (regrowth), output buffers too
small (capacity error), malformed offsets, and the full 8 MiB Zipf text.
"""
import json
import os

import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


@pytest.fixture(scope="module")
def job(torch):
    from paper_1309_0215_amd import Job
    return Job(device=0)


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _check(res, buf, offs=None):
    exp = oracle.words(buf, offs)
    kb = res.key_bytes.cpu().numpy()
    ko = res.key_offsets.cpu().numpy().astype(np.uint64)
    v = res.values.cpu().numpy().astype(np.uint32).astype(np.uint64)
    assert len(v) == len(exp.values), (len(v), len(exp.values))
    assert np.array_equal(ko, exp.key_offsets)
    assert np.array_equal(kb, exp.key_bytes)
    assert np.array_equal(v, exp.values)


def test_golden_hand_cases(torch, job):
    cases = json.load(open(os.path.join(GOLDEN, "words_hand.json")))["cases"]
    for c in cases:
        buf = np.frombuffer(c["input"].encode("latin-1"), np.uint8)
        offs = None if c["offsets"] is None else np.array(c["offsets"], np.uint64)
        d = _dev(torch, buf) if len(buf) else torch.empty(0, dtype=torch.uint8, device="cuda:0")
        ro = None if offs is None else _dev(torch, offs.astype(np.int64))
        res = job.words(d, ro)
        got = res.items()
        exp = [(k.encode("latin-1"), v) for k, v in c["expect"]]
        assert got == exp, (c["input"], got, exp)


WS = list(b" \t\n\x0b\x0c\r")


@pytest.mark.parametrize("seed", range(6))
def test_random_bytes(torch, job, seed):
    rng = np.random.default_rng(seed)
    alphabet = np.array(list(b"abc") + WS + [0, 0x80, 0xFF])
    n = int(rng.integers(1, 200_000))
    buf = rng.choice(alphabet, size=n).astype(np.uint8)
    _check(job.words(_dev(torch, buf)), buf)


@pytest.mark.parametrize("maxlen", [15, 16, 17, 31, 32, 33, 70, 300])
def test_word_lengths_across_chunks(torch, job, maxlen):
    rng = np.random.default_rng(maxlen)
    parts = []
    total = 0
    while total < 150_000:
        L = int(rng.integers(1, maxlen + 1))
        w = bytes(rng.integers(97, 100, size=L).astype(np.uint8))
        parts.append(w + (b" " if rng.random() < 0.8 else b"\n\t"))
        total += L + 1
    buf = np.frombuffer(b"".join(parts), np.uint8)
    _check(job.words(_dev(torch, buf)), buf)


@pytest.mark.parametrize("shift", [1, 3, 7, 15])
def test_unaligned_input(torch, job, shift):
    buf = gen.text(3, 100_003, V=3000, s=1.0)
    big = torch.zeros(len(buf) + 64, dtype=torch.uint8, device="cuda:0")
    big[shift:shift + len(buf)] = _dev(torch, buf)
    _check(job.words(big[shift:shift + len(buf)]), buf)


def test_no_separators_and_all_separators(torch, job):
    one = np.full(1 << 20, ord("x"), np.uint8)  # one 1 MiB word
    _check(job.words(_dev(torch, one)), one)
    sp = np.full(300_000, ord(" "), np.uint8)
    _check(job.words(_dev(torch, sp)), sp)


@pytest.mark.parametrize("seed", range(4))
def test_records(torch, job, seed):
    rng = np.random.default_rng(50 + seed)
    buf = gen.text(7 + seed, 200_000, V=500, s=0.8)
    cuts = np.sort(rng.integers(0, len(buf) + 1, size=int(rng.integers(1, 3000)))).astype(np.uint64)
    if seed == 0:
        cuts = np.concatenate([[0], cuts, [len(buf)]]).astype(np.uint64)
    _check(job.words(_dev(torch, buf), _dev(torch, cuts.astype(np.int64))), buf, cuts)


def test_records_every_line(torch, job):
    buf = gen.text(9, 1 << 20)
    nl = np.flatnonzero(buf == ord("\n")) + 1
    offs = np.concatenate([[0], nl[nl < len(buf)], [len(buf)]]).astype(np.uint64)
    _check(job.words(_dev(torch, buf), _dev(torch, offs.astype(np.int64))), buf, offs)


def test_malformed_offsets(torch, job):
    from paper_1309_0215_amd import MRError
    buf = gen.text(1, 10_000, V=100)
    for bad in ([0, 5000, 4000, 10_000], [0, 20_000]):
        with pytest.raises(MRError) as e:
            job.words(_dev(torch, buf), _dev(torch, np.array(bad, np.int64)))
        assert e.value.status == -1


def test_forced_hash_collisions(torch):
    from paper_1309_0215_amd import Job
    j = Job(device=0, debug_hash=1)
    buf = gen.text(5, 60_000, V=800, s=0.7, lmin=3, lmax=20)
    _check(j.words(_dev(torch, buf)), buf)


def test_table_regrowth(torch):
    from paper_1309_0215_amd import Job
    j = Job(device=0, table_slots=4096, lds_slots=256)
    buf = gen.text(6, 1 << 20, V=20_000, s=0.5)
    res = j.words(_dev(torch, buf))
    _check(res, buf)
    assert res.stats["retries"] >= 1 and res.stats["table_slots"] > 4096


@pytest.mark.parametrize("lds", [256, 1024, 2048, 4096])
def test_lds_sizes(torch, lds):
    from paper_1309_0215_amd import Job
    j = Job(device=0, lds_slots=lds)
    buf = gen.text(8, 600_000, V=10_000, s=1.0)
    _check(j.words(_dev(torch, buf)), buf)


def test_capacity_error_reports_sizes(torch, job):
    import ctypes as C
    from paper_1309_0215_amd import _lib as L
    buf = gen.text(2, 50_000, V=300)
    exp = oracle.words(buf)
    o, keep = job._word_out(10, 20)
    st = job.words_raw(_dev(torch, buf), o)
    assert st == L.MR_ERR_CAPACITY
    assert o.n_keys == len(exp) and o.key_bytes_used == len(exp.key_bytes)


def test_repeat_runs_identical(torch, job):
    buf = gen.text(4, 2 << 20, V=30_000)
    d = _dev(torch, buf)
    a = job.words(d)
    for _ in range(3):
        b = job.words(d)
        assert torch.equal(a.key_bytes, b.key_bytes) and torch.equal(a.values, b.values)


def test_full_config_8mib(torch, job):
    buf = gen.text(1, 8 << 20)  # 8 MiB, V = 50,000, Zipf s = 1.0, lengths 3..12
    res = job.words(_dev(torch, buf))
    _check(res, buf)
    v = res.values.cpu().numpy().astype(np.uint64)
    assert int(v.sum()) == len(buf.tobytes().split())


def test_full_512mib_against_oracle(torch):
    """The 512 MiB text the benchmark times (same generator, the paper's scale),
    launched as the benchmark launches it: fixed output buffers, so the repeat
    replays the captured graph. Every key of both runs against the oracle."""
    from paper_1309_0215_amd import Job, _lib as L
    buf = gen.text(1, 512 << 20)
    d = _dev(torch, buf)
    exp = oracle.words(buf)
    job = Job(device=0)
    o, (kb, ko, vals) = job._word_out(len(exp) + 16, len(exp.key_bytes) + 64)
    for rep in range(3):
        L.check(job.words_raw(d, o), "words")
        torch.cuda.synchronize()
        nk = int(o.n_keys)
        assert nk == len(exp), rep
        assert np.array_equal(ko[:nk + 1].cpu().numpy().astype(np.uint64), exp.key_offsets), rep
        assert np.array_equal(kb[:int(o.key_bytes_used)].cpu().numpy(), exp.key_bytes), rep
        assert np.array_equal(vals[:nk].cpu().numpy().astype(np.uint32).astype(np.uint64), exp.values), rep
        kb.fill_(0)
        vals.fill_(0)
    del d


def test_workspace_reuse_across_sizes_and_kinds(torch):
    # One job alternating small and large inputs and the histogram, which
    # reuses the same workspace: every run must see a clean hash table.
    from paper_1309_0215_amd import Job
    j = Job(device=0)
    rgb = gen.rgb(9, 3 * 200_000)
    sizes = [150_000, 90_000, 170_000, 5_000, 400_000, 120_000]
    for i, n in enumerate(sizes):
        buf = gen.text(20 + i, n, V=4000, s=0.9)
        _check(j.words(_dev(torch, buf)), buf)
        if i % 2:
            h, _ = j.rgb_hist(_dev(torch, rgb))
            assert np.array_equal(h.cpu().numpy().astype(np.uint64), oracle.rgb(rgb))


def test_repeated_calls_replay_and_follow_content(torch):
    """The third identical call replays a captured graph; results track the bytes in place."""
    from paper_1309_0215_amd import Job, WordsResult, _lib as L
    j = Job(device=0)
    bufs = [gen.text(40 + i, 300_000, V=3000, s=1.0) for i in range(3)]
    bufs.append(gen.text(50, 300_000, V=200_000, s=0.3))  # many distinct words: needs a larger table
    d = _dev(torch, bufs[0])
    o, keep = j._word_out(200_000, 1 << 21)
    for i, b in enumerate(bufs + bufs[:2]):
        d.copy_(_dev(torch, b))
        L.check(j.words_raw(d, o), "words")
        kb, ko, vals = keep
        nk = int(o.n_keys)
        _check(WordsResult(kb[:o.key_bytes_used], ko[:nk + 1], vals[:nk], {}), b)


def _uneven_parts(seed: int, n_tiles: int) -> np.ndarray:
    # 16 KiB tiles of sixteen 1 KiB parts: even parts hold words of 17-60
    # bytes (measured and inserted globally by their own lane), odd parts
    # short words from a small vocabulary (LDS cache hits), so that the waves
    # of a workgroup take very different times over the same tiles; words
    # also run across part and tile boundaries
    rng = np.random.default_rng(seed)
    vocab = [bytes(rng.integers(97, 123, size=int(rng.integers(2, 9)), dtype=np.uint8)) for _ in range(300)]
    out = bytearray()
    for _ in range(n_tiles * 16):
        part = bytearray()
        long_part = (len(out) // 1024) % 2 == 0
        while len(part) < 1024:
            if long_part:
                part += bytes(rng.integers(97, 123, size=int(rng.integers(17, 61)), dtype=np.uint8)) + b" "
            else:
                part += vocab[int(rng.integers(0, len(vocab)))] + b" \n"[int(rng.integers(0, 2)):][:1]
        out += part
    return np.frombuffer(bytes(out), np.uint8).copy()


def test_uneven_parts_alone_and_in_a_batch(torch):
    from paper_1309_0215_amd import Job
    bufs = [_uneven_parts(80 + i, n) for i, n in enumerate((3, 17, 40))]
    job = Job(device=0)
    for b in bufs:
        _check(job.words(_dev(torch, b)), b)
    res = job.words_batch([_dev(torch, b) for b in bufs])
    for r, b in zip(res, bufs):
        _check(r, b)


@pytest.mark.parametrize("combine", [0, 1])
def test_wave_combiner_and_cache_misses(torch, combine):
    """The wave-level combiner on and off, on text whose vocabulary is far
    larger than the LDS caches: most words miss them, so the per-workgroup
    miss sub-queues overflow and the overflow goes to the global table."""
    from paper_1309_0215_amd import Job
    job = Job(device=0, wave_combine=combine)
    for seed, size, V, s in ((81, 16 << 20, 2_000_000, 0.3), (82, 3 << 20, 50_000, 1.0), (83, 100_003, 300, 1.2)):
        buf = gen.text(seed, size, V=V, s=s, lmin=1, lmax=16)
        _check(job.words(_dev(torch, buf)), buf)


def test_wave_combiner_records_and_hand_cases(torch):
    from paper_1309_0215_amd import Job
    job = Job(device=0, wave_combine=1)
    cases = json.load(open(os.path.join(GOLDEN, "words_hand.json")))["cases"]
    for c in cases:
        buf = np.frombuffer(c["input"].encode("latin-1"), np.uint8)
        offs = None if c["offsets"] is None else np.array(c["offsets"], np.int64)
        d = _dev(torch, buf) if len(buf) else torch.empty(0, dtype=torch.uint8, device="cuda:0")
        got = job.words(d, None if offs is None else _dev(torch, offs)).items()
        assert got == [(k.encode("latin-1"), v) for k, v in c["expect"]], c["input"]
    buf = gen.text(84, 1 << 20, V=5000, s=1.0)
    rng = np.random.default_rng(5)
    offs = np.concatenate([[0], np.sort(rng.integers(0, len(buf) + 1, 999)), [len(buf)]]).astype(np.int64)
    _check(job.words(_dev(torch, buf), _dev(torch, offs)), buf, offs.astype(np.uint64))


def _shared_prefix_text(seed: int, n_long: int, n_short: int, n_tokens: int) -> np.ndarray:
    # n_long distinct words of 17-40 bytes that all begin with the same 16
    # bytes (their order is decided past the prefix, by the bytes in the
    # input) and n_short distinct words of 1-12 bytes, in random order
    rng = np.random.default_rng(seed)
    pre = b"q" * 16
    longs = {pre + bytes(rng.integers(97, 123, size=int(rng.integers(1, 25)), dtype=np.uint8)) for _ in range(n_long)}
    shorts = {bytes(rng.integers(97, 123, size=int(rng.integers(1, 13)), dtype=np.uint8)) for _ in range(n_short)}
    vocab = sorted(longs) + sorted(shorts)
    pick = rng.integers(0, len(vocab), size=n_tokens)
    return np.frombuffer(b" ".join(vocab[i] for i in pick) + b"\n", np.uint8).copy()


@pytest.mark.parametrize("n_long,n_short", [(3_000, 30_000), (30_000, 70_000), (200_000, 400_000)])
def test_long_keys_with_one_prefix(torch, n_long, n_short):
    """Long keys that share their first 16 bytes are ordered by their input
    bytes inside the register sorts of the splitter sample and of the buckets.
    The sizes give sample sorts of one, two and four entries per thread and
    buckets of more than 1024 records."""
    from paper_1309_0215_amd import Job
    buf = _shared_prefix_text(95, n_long, n_short, 3 * (n_long + n_short))
    _check(Job(device=0).words(_dev(torch, buf)), buf)


def test_long_keys_with_one_prefix_in_a_batch(torch):
    """The same inputs as a batch of six jobs: batches of more than a few jobs
    take their splitters from a merge sort of each job's sample (one
    workgroup per job) instead of ranks, with the same order of long keys."""
    from paper_1309_0215_amd import Job
    sizes = [(3_000, 30_000), (30_000, 70_000), (200_000, 400_000), (100, 2_000), (20_000, 0), (1, 1)]
    bufs = [_shared_prefix_text(96 + i, nl, ns, 3 * (nl + ns)) for i, (nl, ns) in enumerate(sizes)]
    res = Job(device=0).words_batch([_dev(torch, b) for b in bufs])
    for r, b in zip(res, bufs):
        _check(r, b)


def test_small_batch_of_multi_bucket_jobs(torch):
    """Four jobs of 3,000 to 60,000 distinct words each: a batch this small
    takes its splitters from sample ranks spread over all CUs, with the sort
    planned inside that kernel, and its work items belong to several jobs."""
    from paper_1309_0215_amd import Job
    bufs = [gen.text(110 + i, size, V=V, s=0.8) for i, (size, V) in
            enumerate(((1 << 20, 3_000), (3 << 20, 60_000), (2 << 20, 20_000), (1 << 19, 8_000)))]
    res = Job(device=0).words_batch([_dev(torch, b) for b in bufs])
    for r, b in zip(res, bufs):
        _check(r, b)


def test_words_past_the_length_tag(torch):
    """Words of 65,535 bytes and more: the table's 16-bit length tag
    saturates, so equality needs the true lengths, and keys that share their
    first 16 bytes are ordered by their bytes in the input (here words of one
    letter repeated, differing only at the end or in length)."""
    from paper_1309_0215_amd import Job
    a = b"a"
    words = [a * 70_000, a * 70_000, a * 69_999 + b"b", a * 100_000, a * 65_535, a * 65_536, a * 65_534,
             a * 65_536, b"short", b"a", a * 17, a * 70_000]
    rng = np.random.default_rng(9)
    rng.shuffle(words)
    buf = np.frombuffer(b" ".join(words) + b"\n", np.uint8).copy()
    _check(Job(device=0).words(_dev(torch, buf)), buf)


def test_sort_spill_path(torch):
    """About 2.7 M distinct words: more than the 1024 sort buckets of 2048
    records hold in LDS, so buckets are sorted in global memory (counted in
    stats.sort_spills); the output still equals the oracle's."""
    from paper_1309_0215_amd import Job
    buf = gen.text(91, 48 << 20, V=4_000_000, s=0.0, lmin=4, lmax=16)
    res = Job(device=0).words(_dev(torch, buf))
    assert res.stats["sort_spills"] > 0
    _check(res, buf)


def _distinct(rng, n, lens, sep=32):
    """n distinct words of lengths drawn from lens, each once and some again, in random order."""
    letters = rng.integers(97, 123, (n, max(lens))).astype(np.uint8)
    words = list({letters[i, :int(rng.choice(lens))].tobytes() for i in range(n)})
    words += [words[i] for i in rng.integers(0, len(words), n // 2)]
    order = rng.permutation(len(words))
    return np.frombuffer(bytes([sep]).join(words[i] for i in order) + bytes([sep]), np.uint8)


# The partitions stage their sums' records where no key of theirs is in the
# table: few words (most partitions empty); more of one partition than its
# stretch of a small table's staging area; staged and table records that fill
# the record arrays or pass them (a larger table); words longer than 16 bytes
# beside staged ones; queues that overflow in the map; partitions flushed while
# they sum.
@pytest.mark.parametrize("n,lens,slots,lds", [
    (1, [3], 0, 4096), (40, [1, 2, 16], 4096, 256), (2_100, [9], 4096, 4096), (3_900, [6, 12], 4096, 4096),
    (4_090, [7], 4096, 256), (4_300, [7], 4096, 4096), (20_000, [5, 16, 17, 40], 0, 1024), (3_000, [17, 33, 8], 4096, 4096),
    (150_000, [3], 0, 256), (900_000, [8, 9], 1 << 22, 4096),
])
def test_staged_records_and_table_records(torch, n, lens, slots, lds):
    from paper_1309_0215_amd import Job
    rng = np.random.default_rng(n)
    buf = _distinct(rng, n, lens)
    if lens == [3]:
        buf = np.concatenate([buf] * (1 if n == 1 else 8))
    d = _dev(torch, buf)
    j = Job(device=0, table_slots=slots, lds_slots=lds)
    for _ in range(3):  # the later calls find the first one's table and scratch, and replay its launches
        _check(j.words(d), buf)
    _check(Job(device=0, table_slots=slots, lds_slots=lds).words_batch([d, d[: len(buf) // 2]])[0], buf)


@pytest.mark.parametrize("n_jobs", [1024, 1025])
def test_batches_around_the_most_jobs_that_stage(torch, n_jobs):
    from paper_1309_0215_amd import Job
    bufs = [gen.text(500 + i, 200 + i % 700, V=20 + i % 60, s=0.8) for i in range(n_jobs)]
    res = Job(device=0).words_batch([_dev(torch, b) for b in bufs])
    for r, b in zip(res, bufs):
        _check(r, b)
