"""Workloads timed through the public Python entry points.

Each case is one pass of a MapReduce job on inputs drawn on the GPU from a
seed: word count (single jobs and a batch), the RGB histogram, uint32 keys and
(key, value) pairs in each reduce container, the k-means step, the Bloom
filter build and the Reverse Index. The input recipes are those of `gen/`
(Zipf text, clipped Gaussian pixels, Zipf or uniform keys, Gaussian clusters,
DNA with runs of N, HTML with planted links), drawn with torch, with every key
of a vocabulary occurring at least once, so that the sizes of the results
follow from the case.

    listed()             the cases timed by name
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs and the Job a caller keeps between passes
    run(state)           one pass; its outputs
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the outputs in 64-bit arithmetic without the library
"""
from __future__ import annotations

import math

import torch

from paper_1309_0215_amd import Job, _lib as L

DEV = "cuda:0"
STRATS = {"rule": L.STRAT_RULE, "sort": L.STRAT_SORT}
OPS = {"count": L.REDUCE_COUNT, "sum": L.REDUCE_SUM, "min": L.REDUCE_MIN, "max": L.REDUCE_MAX}

BATCH_JOBS = 16
MIB = 1 << 20


def listed() -> list[dict]:
    return [
        # the smallest call: a few thousand records summed into a small declared range; launches and the
        # host round trip are most of it
        {"name": "kv_sum_20K_range1000", "kind": "u32", "n": 20_011, "card": 1000, "s": 1.0, "op": "sum", "pairs": True,
         "declared": True, "spread": False, "strategy": "rule"},
        # the configured word count, and the same text at the paper's 500 MB scale
        {"name": "words_8MiB", "kind": "words", "size": 8 * MIB, "vocab": 50_000, "s": 1.0, "lmax": 12},
        {"name": "words_512MiB", "kind": "words", "size": 512 * MIB, "vocab": 50_000, "s": 1.0, "lmax": 12},
        # many word jobs of mixed sizes (64 KiB to 16 MiB) and vocabularies in one call
        {"name": "words_batch16", "kind": "batch", "size_lo": 64 << 10, "size_hi": 16 * MIB, "vocab_lo": 1000,
         "vocab_hi": 1_000_000},
        # the headline histogram: 1 GiB of pixels (a length that is no multiple of 16)
        {"name": "rgb_1GiB", "kind": "rgb", "size": (1 << 30) // 3 * 3},
        # the paper's Histogram: 256 M elements over 16 M possible keys
        {"name": "hist_2p28_keys2p24", "kind": "u32", "n": 1 << 28, "card": 1 << 24, "s": 0.0, "op": "count", "pairs": False,
         "declared": True, "spread": False, "strategy": "rule"},
        # counting identifiers that have no declared range: the hash table
        {"name": "ids_count_16M_card1M", "kind": "u32", "n": 16_000_003, "card": 1_000_000, "s": 0.75, "op": "count",
         "pairs": False, "declared": False, "spread": True, "strategy": "rule"},
        # summing values over a declared range too large for a workgroup's LDS: the global array
        {"name": "kv_sum_8M_range1M", "kind": "u32", "n": 8_000_003, "card": 1 << 20, "s": 0.75, "op": "sum", "pairs": True,
         "declared": True, "spread": False, "strategy": "rule"},
        # the configured k-means step: 16 M points
        {"name": "kmeans_16M_d32_k64", "kind": "kmeans", "n": 1 << 24, "d": 32, "k": 64},
        # k-means at other dimensions and cluster counts than the configured ones
        {"name": "kmeans_500K_d64_k100", "kind": "kmeans", "n": 500_003, "d": 64, "k": 100},
        # the paper's Bloom Filter: 30 million k-mers, 300 million bits
        {"name": "bloom_30M_300Mbit", "kind": "bloom", "n": 30_000_019, "bits": 300_000_000, "k": 20, "hashes": 7},
        # the paper's Reverse Index: 78,355 files, 307,921 links, 1 GiB
        {"name": "links_1GiB_78Kfiles", "kind": "links", "size": 1 << 30, "files": 78_355, "links": 307_921,
         "urls": 48_755},
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["u32"] * 6 + ["words"] * 3 + ["batch", "rgb", "rgb", "kmeans", "kmeans", "kmeans", "bloom", "links"])
    if kind == "u32":
        n, pairs, declared = _log_int(rng, 10_000, 16_000_000), rng.random() < 0.6, rng.random() < 0.5
        return {"kind": kind, "n": n, "card": _log_int(rng, 16, min(1 << 24, n // 2)), "s": round(rng.uniform(0.0, 1.5), 3),
                "op": rng.choice(list(OPS)) if pairs else "count", "pairs": pairs, "declared": declared,
                "spread": not declared and rng.random() < 0.5, "strategy": rng.choice(["rule", "rule", "rule", "sort"])}
    if kind == "words":
        size = _log_int(rng, 64 << 10, 256 * MIB)
        return {"kind": kind, "size": size, "vocab": _log_int(rng, 500, min(1_000_000, size // 64)),
                "s": round(rng.uniform(0.6, 1.4), 3), "lmax": rng.choice([12, 16])}
    if kind == "batch":
        lo = _log_int(rng, 64 << 10, MIB)
        return {"kind": kind, "size_lo": lo, "size_hi": _log_int(rng, 2 * MIB, 16 * MIB), "vocab_lo": 1000,
                "vocab_hi": _log_int(rng, 20_000, 1_000_000)}
    if kind == "rgb":
        return {"kind": kind, "size": 3 * _log_int(rng, 10_000, (1 << 30) // 3)}
    if kind == "kmeans":
        if rng.random() < 0.4:  # the configured dimensions, fewer points
            return {"kind": kind, "n": _log_int(rng, 10_000, 1 << 24), "d": 32, "k": 64}
        return {"kind": kind, "n": _log_int(rng, 10_000, 500_000), "d": _log_int(rng, 2, 64), "k": _log_int(rng, 2, 100)}
    if kind == "bloom":
        n = _log_int(rng, 100_000, 30_000_000)
        return {"kind": kind, "n": n, "bits": 10 * n + rng.randrange(64), "k": rng.randrange(11, 33),
                "hashes": rng.randrange(2, 9)}
    size = _log_int(rng, MIB, 1 << 30)
    files = max(1, size // _log_int(rng, 4_000, 40_000))
    links = min(max(200, size // _log_int(rng, 2_000, 20_000)), 5 * files)
    return {"kind": kind, "size": size, "files": files, "links": links, "urls": max(1, links // rng.randrange(2, 20))}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


def _ints(g, lo: int, hi: int, size) -> torch.Tensor:
    return torch.randint(lo, hi, size if isinstance(size, tuple) else (size,), generator=g, device=DEV)


def _zipf(g, card: int, s: float, n: int) -> torch.Tensor:
    """n ranks in [0, card) with P(r) ~ (r + 1)^-s."""
    if s == 0.0:
        return _ints(g, 0, card, n)
    cdf = torch.cumsum(torch.arange(1, card + 1, device=DEV, dtype=torch.float64) ** -s, 0)
    cdf /= cdf[-1].clone()
    r = torch.searchsorted(cdf, torch.rand(n, generator=g, device=DEV, dtype=torch.float64), right=True)
    return r.clamp_(max=card - 1)


def _fill_tokens(out: torch.Tensor, rows: torch.Tensor, lens: torch.Tensor, pick) -> None:
    """Fills `out` with whole rows (bytes [0, lens[i]) of rows[i], i from pick(n)); newlines after the last that fits."""
    out.fill_(10)
    mean = float(lens.double().mean())
    at = torch.arange(rows.shape[1], device=DEV)
    pos, size = 0, out.numel()
    while True:
        want = int(min(4 * MIB, (size - pos) / mean * 1.05 + 64))
        ids = pick(want)
        ends = torch.cumsum(lens[ids], 0)
        fit = int(torch.searchsorted(ends, size - pos, right=True))
        ids = ids[:fit]
        b = rows[ids][at[None, :] < lens[ids][:, None]]
        out[pos:pos + b.numel()] = b
        pos += b.numel()
        if fit < want:
            return


def _words(g, vocab: int, lmax: int) -> tuple[torch.Tensor, torch.Tensor]:
    """`vocab` distinct words, the same number of each length from 3 (4 above 100,000 words) to lmax."""
    lmin = 3 if vocab <= 100_000 else 4
    i = torch.arange(vocab, device=DEV)
    lens = lmin + i % (lmax - lmin + 1)
    words = _ints(g, 97, 123, (vocab, lmax + 1))
    # the first letters number the words of one length: a bijection modulo 26^m, its multiplier coprime to 26
    m = lens.clamp(max=5)
    mult = 26 * int(_ints(g, 1, 10_000, 1)) + 3
    number = (i // (lmax - lmin + 1) * mult + int(_ints(g, 0, 10_000, 1))) % (26 ** m)
    for c in range(5):
        words[:, c] = torch.where(c < m, 97 + number % 26, words[:, c])
        number = number // 26
    return words.to(torch.uint8), lens


def _text(g, size: int, vocab: int, s: float, lmax: int) -> torch.Tensor:
    """Zipf text, each word followed by a newline (1 in 12) or a space; every word of the vocabulary occurs."""
    words, lens = _words(g, vocab, lmax)
    ends = torch.arange(vocab, device=DEV)
    # rows 0..vocab-1 end in a space, rows vocab..2*vocab-1 are the same words ending in a newline
    rows = words.repeat(2, 1)
    rows[ends, lens] = 32
    rows[ends + vocab, lens] = 10
    lens = (lens + 1).repeat(2)
    perm, each = torch.randperm(vocab, generator=g, device=DEV), torch.randperm(vocab, generator=g, device=DEV)
    every = max(1, size // ((lmax + 2) * vocab))  # token i * every is the i-th of `each`
    at = 0

    def pick(n):
        nonlocal at
        ids = perm[_zipf(g, vocab, s, n)]
        first = -(-at // every)
        some = each[first:max(first, min(vocab, -(-(at + n) // every)))]
        ids[first * every - at:][:some.numel() * every:every] = some
        at += n
        return ids + vocab * (torch.rand(n, generator=g, device=DEV) < 1 / 12).long()

    out = torch.empty(size, dtype=torch.uint8, device=DEV)
    _fill_tokens(out, rows, lens, pick)
    return out


def _pixels(g, size: int) -> torch.Tensor:
    """Bytes of three Gaussians (means 40, 128, 210, sd 25), rounded and clipped."""
    out = torch.empty(size, dtype=torch.uint8, device=DEV)
    means = torch.tensor([40.0, 128.0, 210.0], device=DEV)
    for a in range(0, size, 64 * MIB):
        m = min(64 * MIB, size - a)
        v = torch.randn(m, generator=g, device=DEV) * 25 + means[_ints(g, 0, 3, m)]
        out[a:a + m] = v.round_().clamp_(0, 255).to(torch.uint8)
    return out


def _keys(case: dict, g) -> torch.Tensor:
    """Zipf keys; every one of the `card` keys occurs."""
    n, card = case["n"], case["card"]
    keys = torch.empty(n, dtype=torch.int32, device=DEV)
    perm = torch.randperm(card, generator=g, device=DEV)
    if case["spread"]:  # identifiers anywhere in 32 bits (an odd multiplier is a bijection)
        perm = (perm * 2654435761) & 0xFFFFFFFF
    perm = torch.where(perm >= 1 << 31, perm - (1 << 32), perm).to(torch.int32)
    for a in range(0, n, 32 * MIB):
        m = min(32 * MIB, n - a)
        keys[a:a + m] = perm[_zipf(g, card, case["s"], m)]
    keys[:card * (n // card):n // card] = perm[torch.randperm(card, generator=g, device=DEV)]
    return keys


def _dna(g, n: int) -> torch.Tensor:
    """Uniform bases; a run of 1..200 N starts at about one base in 100,000."""
    out = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device=DEV)[_ints(g, 0, 4, n)]
    starts = _ints(g, 0, n, max(1, n // 100_000))
    lens = _ints(g, 1, 201, starts.numel())
    at = torch.arange(200, device=DEV)
    runs = (starts[:, None] + at)[at < lens[:, None]]
    out[runs[runs < n]] = 78
    return out


_TAGS = [b"<p>", b"</p>", b'<div class="c">', b"</div>", b"<b>", b"</b>", b'<a name="n">', b"</a>", b'<img src="i.png">',
         b"\n", b"<li>", b'<A HREF="X">', b"<a href='y'>", b"<a href=z>", b'<a  href="w">']


def _rows_of(texts: list[bytes], width: int) -> tuple[torch.Tensor, torch.Tensor]:
    flat = torch.frombuffer(bytearray(b"".join(t.ljust(width, b" ") for t in texts)), dtype=torch.uint8)
    return flat.view(len(texts), width).to(DEV), torch.tensor([len(t) for t in texts], device=DEV)


def _html(case: dict, g) -> tuple[torch.Tensor, torch.Tensor]:
    """Files of words and tags (near-misses of the link marker among them) with links at random places; file offsets."""
    width = 17
    tags, tag_lens = _rows_of(_TAGS, width)
    words, word_lens = _ints(g, 97, 123, (4096, width)).to(torch.uint8), _ints(g, 3, 12, 4096)
    words[torch.arange(4096, device=DEV), word_lens - 1] = 32
    rows, lens = torch.cat([words, tags]), torch.cat([word_lens, tag_lens])
    filler = torch.empty(case["size"], dtype=torch.uint8, device=DEV)

    def pick(n):
        tag = torch.rand(n, generator=g, device=DEV) < 0.25
        return torch.where(tag, 4096 + _ints(g, 0, len(_TAGS), n), _ints(g, 0, 4096, n))

    _fill_tokens(filler, rows, lens, pick)
    # file sizes uniform in [mean / 2, 3 mean / 2], scaled to the filler
    w = torch.cumsum(torch.rand(case["files"], generator=g, device=DEV, dtype=torch.float64) + 0.5, 0)
    edges = torch.cat([torch.zeros(1, device=DEV, dtype=torch.int64), (w / w[-1] * case["size"]).long()])
    edges[-1] = case["size"]
    # URLs <a href="http://HOST.com/PATH.html">w</a>
    V, n = case["urls"], case["links"]
    head, mid, tail = b'<a href="http://', b".com/", b'.html">w</a>'
    i = torch.arange(V, device=DEV)
    host, path = 5 + i % 10, 1 + i // 10 % 40
    url_w = len(head) + 14 + len(mid) + 40 + len(tail)
    at = torch.arange(url_w, device=DEV)[None, :]
    link = _ints(g, 97, 123, (V, url_w)).to(torch.uint8)
    o = torch.zeros(V, 1, dtype=torch.int64, device=DEV)
    for text, gap in ((head, host), (mid, path), (tail, None)):
        t = torch.frombuffer(bytearray(text), dtype=torch.uint8).to(DEV)
        inside = (at >= o) & (at < o + len(text))
        link = torch.where(inside, t[(at - o).clamp(0, len(text) - 1)], link)
        o = o + len(text) + (gap[:, None] if gap is not None else 0)
    link_len = o[:, 0]
    # links: every URL once, the others by Zipf(1); a URL's links go to different files, but for one link in 50,
    # which repeats another link of its file
    again = n // 50 if n // 50 <= n - V else 0
    ids = torch.randperm(V, generator=g, device=DEV)[torch.cat([torch.arange(V, device=DEV), _zipf(g, V, 1.0, n - V - again)])]
    ids = torch.sort(ids).values
    nth = torch.arange(ids.numel(), device=DEV) - torch.searchsorted(ids, ids)
    file = (_ints(g, 0, case["files"], V)[ids] + nth) % case["files"]
    twice = torch.randperm(ids.numel(), generator=g, device=DEV)[:again]
    ids, file = torch.cat([ids, ids[twice]]), torch.cat([file, file[twice]])
    spot = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    cuts, order = torch.sort(edges[file] + (spot * (edges[file + 1] - edges[file])).long())
    ids = ids[order]
    ends = torch.cumsum(link_len[ids], 0)
    starts = cuts + ends - link_len[ids]
    places = (starts[:, None] + at)[at < link_len[ids][:, None]]
    total = case["size"] + int(ends[-1])
    buf = torch.empty(total, dtype=torch.uint8, device=DEV)
    free = torch.ones(total, dtype=torch.bool, device=DEV)
    free[places] = False
    buf.masked_scatter_(free, filler)
    buf[places] = link[ids][at < link_len[ids][:, None]]
    before = torch.searchsorted(cuts, edges, right=False)
    before[-1] = n
    rec = edges + torch.cat([torch.zeros(1, device=DEV, dtype=torch.int64), ends])[before]
    return buf, rec


def _points(case: dict, g) -> torch.Tensor:
    n, d, k = case["n"], case["d"], case["k"]
    centres = torch.rand(k, d, generator=g, device=DEV) * 20 - 10
    return centres[_ints(g, 0, k, n)] + 0.5 * torch.randn(n, d, generator=g, device=DEV)


def _inputs(case: dict, seed: int) -> dict:
    g, kind = _gen(seed), case["kind"]
    if kind == "words":
        return {"data": _text(g, case["size"], case["vocab"], case["s"], case["lmax"])}
    if kind == "batch":
        jobs = []
        for i in range(BATCH_JOBS):  # sizes and vocabularies spread evenly over the logarithm of their ranges
            f = (i + 0.5) / BATCH_JOBS
            h = (i * 7 % BATCH_JOBS + 0.5) / BATCH_JOBS
            size = int(case["size_lo"] * (case["size_hi"] / case["size_lo"]) ** f)
            vocab = min(size // 64, int(case["vocab_lo"] * (case["vocab_hi"] / case["vocab_lo"]) ** h))
            jobs.append(_text(g, size, vocab, 0.6 + 0.8 * (i * 5 % BATCH_JOBS) / BATCH_JOBS, 16))
        return {"jobs": jobs}
    if kind == "rgb":
        return {"data": _pixels(g, case["size"])}
    if kind == "u32":
        keys = _keys(case, g)
        vals = _ints(g, -(1 << 31), 1 << 31, case["n"]).to(torch.int32) if case["pairs"] else None
        return {"keys": keys, "vals": vals}
    if kind == "kmeans":
        x = _points(case, g)
        return {"x": x, "c": x[:case["k"]].clone()}
    if kind == "bloom":
        return {"data": _dna(g, case["n"])}
    buf, rec = _html(case, g)
    return {"data": buf, "rec": rec}


def prepare(case: dict, seed: int) -> dict:
    s = {"case": case, **_inputs(case, seed)}
    kind = case["kind"]
    if kind == "u32":
        s["job"] = Job(device=0, strategy=STRATS[case["strategy"]])
    elif kind == "kmeans":
        s["job"] = Job(device=0, km_centroids=s["c"])
    elif kind == "bloom":
        s["job"] = Job(device=0, bloom_k=case["k"], bloom_hashes=case["hashes"])
    else:
        s["job"] = Job(device=0)
    if kind == "batch":
        s["prepared"] = s["job"].batch_prepare(s["jobs"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s: dict):
    job, case = s["job"], s["case"]
    kind = case["kind"]
    if kind == "words":
        r = job.words(s["data"])
        return [r.key_bytes, r.key_offsets, r.values]
    if kind == "batch":
        out = job.words_batch(s["jobs"], prepared=s["prepared"])
        return [[r.key_bytes, r.key_offsets, r.values] for r in out]
    if kind == "rgb":
        return job.rgb_hist(s["data"])[0]
    if kind == "u32":
        r = job.u32(s["keys"], s["vals"], op=OPS[case["op"]], key_range=case["card"] if case["declared"] else 0)
        return [r.keys, r.values]
    if kind == "kmeans":
        return list(job.kmeans(s["x"])[:4])
    if kind == "bloom":
        return job.bloom(s["data"], case["bits"])[0]
    r = job.links(s["data"], s["rec"])
    return [r.key_bytes, r.key_offsets, r.counts, r.list_offsets, r.list_ids]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case: dict) -> dict:
    kind = case["kind"]
    if kind == "words":
        mean = (3 + case["lmax"]) / 2
        return {"bytes": case["size"] + case["vocab"] * (mean + 12.0), "flops": 0.0}
    if kind == "batch":
        sizes = [case["size_lo"] * (case["size_hi"] / case["size_lo"]) ** ((i + 0.5) / BATCH_JOBS) for i in range(BATCH_JOBS)]
        return {"bytes": float(sum(sizes)), "flops": 0.0}
    if kind == "rgb":
        return {"bytes": case["size"] + 768 * 8.0, "flops": 0.0}
    if kind == "u32":
        return {"bytes": case["n"] * (8.0 if case["pairs"] else 4.0) + case["card"] * (12.0 if case["op"] == "sum" else 8.0),
                "flops": 0.0}
    if kind == "kmeans":
        n, d, k = case["n"], case["d"], case["k"]
        return {"bytes": 4.0 * n * d + 4.0 * n, "flops": 2.0 * n * k * d}
    if kind == "bloom":
        return {"bytes": case["n"] + case["bits"] / 8, "flops": 0.0}
    return {"bytes": case["size"] + case["links"] * 85.0 + case["urls"] * 75.0 + case["files"] * 8.0, "flops": 0.0}


# ---------------------------------------------------------------------------
# 64-bit values
# ---------------------------------------------------------------------------

def _exact_u32(case: dict, seed: int):
    x = _inputs(case, seed)
    keys, inv, counts = torch.unique(x["keys"].long() & 0xFFFFFFFF, return_inverse=True, return_counts=True)
    if case["op"] == "count":
        values = counts
    else:
        v = x["vals"].long() & 0xFFFFFFFF
        if case["op"] == "sum":
            values = torch.zeros_like(keys).index_add_(0, inv, v)
        else:
            values = torch.zeros_like(keys).scatter_reduce_(0, inv, v, "a" + case["op"], include_self=False)
    as_i32 = lambda t: torch.where(t >= 1 << 31, t - (1 << 32), t).to(torch.int32)  # noqa: E731
    return [as_i32(keys), values if case["op"] == "sum" else as_i32(values)]


def _exact_kmeans(case: dict, seed: int):
    i = _inputs(case, seed)
    x, c = i["x"], i["c"].double()
    k, d, n = case["k"], case["d"], case["n"]
    norm = (c * c).sum(1)
    assign = torch.empty(n, dtype=torch.int32, device=DEV)
    sums = torch.zeros(k, d, dtype=torch.float64, device=DEV)
    counts = torch.zeros(k, dtype=torch.int64, device=DEV)
    for a in range(0, n, MIB):
        xb = x[a:a + MIB].double()
        j = torch.argmin(norm[None, :] - 2 * (xb @ c.t().contiguous()), 1)
        assign[a:a + MIB] = j.to(torch.int32)
        sums.index_add_(0, j, xb)
        counts += torch.bincount(j, minlength=k)
    cent = torch.where(counts[:, None] > 0, sums / counts.clamp(min=1)[:, None], c)
    return [assign, sums, counts.to(torch.int32), cent]


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind == "u32" and case["n"] <= 64 * MIB:
        return _exact_u32(case, seed)
    if kind == "kmeans":
        return _exact_kmeans(case, seed)
    if kind == "rgb":
        b = _inputs(case, seed)["data"].view(-1, 3)
        return torch.stack([torch.bincount(b[:, c].contiguous(), minlength=256) for c in range(3)])
    return None
