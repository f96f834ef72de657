// Bloom filter build on gfx950 (benchmark application "Bloom Filter": large
// array container, Section III-E "eliminating local arrays").
//
// map: every k-mer (k consecutive bases of A, C, G, T; a k-mer holding any
// other byte is skipped) emits the h bit positions of the filter; reduce: OR
// into one array of m bits.
//   code  v = 2-bit packed k-mer (A 0, C 1, G 2, T 3, first base highest)
//   x     = fmix64(v) (the 64-bit finaliser of MurmurHash3)
//   g_i   = (lo32(x) + i * (hi32(x) | 1)) mod 2^32   (double hashing, i < h)
//   pos_i = floor(g_i * m / 2^32)                     (multiply-shift into [0, m))
//
// Device atomics on a 37.5 MB array would be the bottleneck, so the array is
// filled by position ranges. A tile of up to 32768 positions is ordered in LDS
// by sub-ranges of 2^sb bits (sb <= 16) and written where the tile stands, two
// bytes a position, with a row of the sub-ranges' starts; then one workgroup
// per range of up to nine neighbouring sub-ranges reads its run of every tile,
// ORs it into an LDS bit array and writes the range's words once. A position's
// sub-range is found from the row's starts, so it needs no bits of its own.
// 30 M k-mers, 7 hashes, 300 Mbit: 375 us. (A count of the positions per range
// of 2^19 bits, its scan, a scatter of four-byte positions to one segment per
// range and a fill from it took 930 us: 117 + 24 + 508 + 267.)
// Few positions go to the array by device atomics (kBloomDirectMax).
#include "common.h"
#include "launch.h"

#include <cmath>

namespace mr {

constexpr uint32_t kBloomSubBits = 16;        // bits of a sub-range at most: a position in it is two bytes
constexpr uint32_t kBloomSubBitsMin = 5;      // a sub-range is whole words
constexpr uint32_t kBloomSubsWanted = 1024;   // smaller sub-ranges up to this many: counters that seldom meet
constexpr uint32_t kBloomMaxSubs = 8192;      // m up to 2^29 bits
constexpr uint32_t kBloomMaxPer = 9;          // sub-ranges per range: 72 KB of LDS, two workgroups per CU
constexpr uint32_t kBloomFillPerCu = 2;       // fill workgroups resident at once on a CU
constexpr uint32_t kBloomThreads = 1024;
constexpr uint32_t kBloomBatch = 4 * kBloomThreads;  // k-mers staged at once, four per thread
constexpr uint32_t kBloomMaxK = 32;
constexpr uint32_t kBloomMaxH = 8;            // hashes per k-mer
constexpr uint32_t kBloomFillThreads = 1024;
constexpr uint32_t kBloomPartPad = 16;        // readable and writable past the last position
constexpr uint32_t kBloomRowPad = 12;         // sub-range starts readable past the last one
constexpr uint32_t kBloomDirectThreads = 256;
// Fewer positions than this go to the array by device atomics, without
// scratch: a tile would be mostly its row of starts, and more scratch than
// four bytes a position. (35,000 positions: 54 us by atomics, 33 us by tiles;
// 260,000: 96 and 33 us.)
constexpr uint64_t kBloomDirectMax = 1ull << 14;

// Batches of a tile: a tile holds up to 32768 positions (64 KB of LDS), so
// that its row of starts (16 KB for the largest filter) stays below half of
// its positions, whatever the hash count.
constexpr uint32_t bloom_batches(uint32_t h) { return h >= 8 ? 1 : 8 / h; }

struct BloomStage {
  uint32_t code[kBloomBatch / 16 + 2];  // 2-bit codes, 16 bases per word, the first highest
  uint32_t bad[kBloomBatch / 32 + 1];   // one bit per byte that is no base, the first highest
};

// Stages the bytes of a batch at e0 (a multiple of 4) and the 31 after it.
// Bytes past the input are no bases.
MR_DEV void bloom_stage(const uint8_t* __restrict__ in, uint64_t n_bytes, uint64_t e0, BloomStage& st) {
  for (uint32_t g = threadIdx.x; g < kBloomBatch / 4 + 8; g += blockDim.x) {
    const uint64_t p = e0 + 4ull * g;
    uint32_t x = 0;
    if (p + 4 <= n_bytes && ((uintptr_t)in & 3u) == 0) {
      x = gp(reinterpret_cast<const uint32_t*>(in + p))[0];
    } else {
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q)
        if (p + q < n_bytes) x |= (uint32_t)gp(in + p)[q] << (8 * q);
    }
    // bits 1 and 2 of a base's byte: A 0, C 1, T 2, G 3
    uint32_t c = (x >> 1) & 0x03030303u;
    c ^= (c >> 1) & 0x01010101u;
    const uint32_t d = x ^ __builtin_amdgcn_perm(0u, 0x54474341u, c);  // bytes that are not "ACGT"[code] stay nonzero
    const uint32_t nz = ((((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | d) & 0x80808080u) >> 7;
    reinterpret_cast<uint8_t*>(st.code)[g ^ 3u] = (uint8_t)((c * 0x40100401u) >> 24);
    uint32_t b = ((nz * 0x08040201u) >> 24) << (28 - 4 * (g & 7u));
    b |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    b |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0x4E, 0xF, 0xF, false);   // lane ^ 2
    b |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, 0x141, 0xF, 0xF, false);  // 7 - lane: the other four
    if ((g & 7u) == 0) st.bad[g >> 3] = b;
  }
}

// Hash halves of this thread's four k-mers of the staged batch: a = low32(x),
// b = high32(x) | 1. Bit j of the result is set when k-mer j exists and holds
// only bases.
MR_DEV uint32_t bloom_hashes(const BloomStage& st, uint64_t e0, uint64_t n_kmers, uint32_t k, uint32_t (&a)[4],
                             uint32_t (&b)[4]) {
  const uint32_t g = threadIdx.x, w = g >> 2;
  const uint64_t hi = (uint64_t)st.code[w] << 32 | st.code[w + 1], lo = st.code[w + 2];
  const uint64_t bad = ((uint64_t)st.bad[g >> 3] << 32 | st.bad[(g >> 3) + 1]) << (4 * (g & 7u));
  uint32_t valid = 0;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) {
    const uint32_t at = 8 * (g & 3u) + 2 * j;
    const uint64_t x = fmix64(((hi << at) | ((lo << at) >> 32)) >> (64 - 2 * k));
    a[j] = (uint32_t)x;
    b[j] = (uint32_t)(x >> 32) | 1u;
    if (((bad << j) >> (64 - k)) == 0 && e0 + 4 * g + j < n_kmers) valid |= 1u << j;
  }
  return valid;
}

// One workgroup per tile: counts the tile's positions per sub-range, scans the
// counts, places each position's low sb bits by a second atomic on its
// sub-range's next slot, and writes the ordered tile and its row of starts.
// LDS: the counters, then the positions. Bound by LDS: two atomics and a
// two-byte store at random addresses per position (the LDS is busy for 132 of
// 194 us on 210 M positions, the vector units for 125). Keeping the first
// atomic's rank instead of the second atomic costs a random read in its place,
// and registers.
template <uint32_t H>
__global__ __launch_bounds__(kBloomThreads, 8) void k_bloom_tile(const uint8_t* __restrict__ in, uint64_t n_bytes,
                                                                 uint64_t n_kmers, uint32_t k, uint32_t m, uint32_t sb,
                                                                 uint32_t S, uint32_t row_words,
                                                                 uint32_t* __restrict__ rows, uint16_t* __restrict__ part) {
  constexpr uint32_t kBatches = bloom_batches(H), kCap = kBatches * kBloomBatch * H;
  extern __shared__ __attribute__((aligned(16))) uint32_t bloom_lds[];
  uint16_t* const sk = reinterpret_cast<uint16_t*>(bloom_lds);  // [kCap]
  uint32_t* const cnt = bloom_lds + kCap / 2;                   // [S]
  __shared__ BloomStage st;
  __shared__ uint32_t wsum[kBloomThreads / kWave];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  const uint64_t t0 = (uint64_t)blockIdx.x * (kBatches * kBloomBatch);
  for (uint32_t s = threadIdx.x; s < S; s += kBloomThreads) cnt[s] = 0;
  uint32_t a[4], b[4], valid = 0;
  for (uint32_t q = 0; q < kBatches; ++q) {
    const uint64_t e0 = t0 + q * kBloomBatch;
    if (e0 >= n_kmers) break;
    if (q) __syncthreads();  // the previous batch is no longer read
    bloom_stage(in, n_bytes, e0, st);
    __syncthreads();
    valid = bloom_hashes(st, e0, n_kmers, k, a, b);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j)
      if (valid >> j & 1u)
#pragma unroll
        for (uint32_t i = 0; i < H; ++i) atomicAdd(&cnt[__umulhi(a[j] + i * b[j], m) >> sb], 1u);
  }
  __syncthreads();
  // exclusive scan of the counts; an odd number of them per thread keeps the reads off each other's banks
  const uint32_t each = ((S + kBloomThreads - 1) / kBloomThreads) | 1u;
  const uint32_t s0 = threadIdx.x * each, s1 = s0 + each < S ? s0 + each : S;
  uint32_t sum = 0;
  for (uint32_t s = s0; s < s1; ++s) sum += cnt[s];
  const uint32_t incl = wave_incl_scan(sum);
  if (lane == kWave - 1) wsum[wv] = incl;
  __syncthreads();
  uint32_t run = incl - sum, total = 0;
#pragma unroll
  for (uint32_t w = 0; w < kBloomThreads / kWave; ++w) {
    if (w < wv) run += wsum[w];
    total += wsum[w];
  }
  for (uint32_t s = s0; s < s1; ++s) {
    const uint32_t c = cnt[s];
    cnt[s] = run;
    run += c;
  }
  __syncthreads();
  const uint32_t mask = (1u << sb) - 1u;
  for (uint32_t q = 0; q < kBatches; ++q) {
    if (kBatches > 1) {
      const uint64_t e0 = t0 + q * kBloomBatch;
      if (e0 >= n_kmers) break;
      if (q) __syncthreads();
      bloom_stage(in, n_bytes, e0, st);
      __syncthreads();
      valid = bloom_hashes(st, e0, n_kmers, k, a, b);
    }
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      if (valid >> j & 1u) {
        uint32_t slot[H];
#pragma unroll
        for (uint32_t i = 0; i < H; ++i) slot[i] = atomicAdd(&cnt[__umulhi(a[j] + i * b[j], m) >> sb], 1u);
#pragma unroll
        for (uint32_t i = 0; i < H; ++i) sk[slot[i]] = (uint16_t)(__umulhi(a[j] + i * b[j], m) & mask);
      }
    }
  }
  __syncthreads();
  // a sub-range's counter now holds the start of the next one
  MR_GLOBAL uint32_t* const row = gp(rows + (uint64_t)blockIdx.x * row_words);
  for (uint32_t w = threadIdx.x; w < row_words; w += kBloomThreads) {
    const uint32_t lo = w == 0 ? 0u : 2 * w - 1 < S ? cnt[2 * w - 1] : total;
    const uint32_t hi = 2 * w < S ? cnt[2 * w] : total;
    row[w] = lo | hi << 16;
  }
  uint16_t* const out = part + (uint64_t)blockIdx.x * kCap;
  for (uint32_t i = threadIdx.x * 8; i < total; i += kBloomThreads * 8)
    gstore16(out + i, *reinterpret_cast<const uint4*>(sk + i));
}

// One workgroup per range of `per` sub-ranges: lpg neighbouring lanes take a
// tile's run together, a piece of eight positions (one 16-byte load) each. A
// piece's sub-ranges come from the run's inner starts: each adds one to the
// 4-bit fields of the piece's elements at or after it. Elements of a piece
// outside the run OR nothing. Bound by vector instructions, about 120 a piece
// (154 of 199 us on 210 M positions): long runs waste the fewest lanes, so a
// range is as large as two workgroups per CU allow (runs of 56 positions on
// ten lanes; ranges of five sub-ranges 226 us, of three 270). Loading a run's
// pieces, or the next tile's, ahead of their use was slower (250, 257 us).
__global__ __launch_bounds__(kBloomFillThreads, 8) void k_bloom_fill(const uint16_t* __restrict__ part,
                                                                  const uint32_t* __restrict__ rows, uint32_t row_words,
                                                                  uint32_t n_tiles, uint32_t cap, uint32_t sb, uint32_t per,
                                                                  uint32_t lpg, uint64_t n_words,
                                                                  uint32_t* __restrict__ words) {
  extern __shared__ __attribute__((aligned(16))) uint32_t bloom_lds[];  // the range's bits
  // Workgroups are handed to the eight XCDs in turn; neighbouring ranges share
  // the lines where their runs meet, so each XCD takes a contiguous block of
  // ranges and its L2 serves those once.
  const uint32_t each = gridDim.x / kXcds, whole = each * kXcds;
  const uint32_t p = blockIdx.x < whole ? blockIdx.x % kXcds * each + blockIdx.x / kXcds : blockIdx.x;
  const uint32_t n_bits_words = per << (sb - 5);
  for (uint32_t i = threadIdx.x; i < n_bits_words; i += kBloomFillThreads) bloom_lds[i] = 0;
  __syncthreads();
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  const uint32_t gpw = kWave / lpg, in_group = lane % lpg;
  const uint32_t step = gpw * (kBloomFillThreads / kWave);
  const uint32_t s0 = p * per, shift = 16u * (s0 & 1u);
  const uint32_t* const row0 = rows + s0 / 2;
  const uint32_t word_mask = (((1u << (sb - 5)) - 1u) << 2) * 0x10001u;
  constexpr uint32_t kRow = (kBloomMaxPer + 1 + 1) / 2 + 1;  // words that hold the run's starts from either half
  auto load_row = [&](uint32_t t, uint32_t (&r)[kRow]) {
    const MR_GLOBAL uint32_t* q = gp(row0 + (uint64_t)t * row_words);
#pragma unroll
    for (uint32_t i = 0; i < kRow; ++i) r[i] = q[i];
  };
  uint32_t t = wv * gpw + lane / lpg;
  if (lane / lpg >= gpw) t = n_tiles;  // lanes over when lpg does not divide the wave
  uint32_t next[kRow] = {};
  if (t < n_tiles) load_row(t, next);
  for (; t < n_tiles; t += step) {
    uint32_t at[kBloomMaxPer + 1], end = 0;  // starts of the run's sub-ranges, its end among them
#pragma unroll
    for (uint32_t i = 0; i <= kBloomMaxPer; ++i) {
      const uint32_t w = __builtin_amdgcn_alignbit(next[i / 2 + 1], next[i / 2], shift);
      at[i] = i & 1u ? w >> 16 : w & 0xFFFFu;
      if (i <= per) end = at[i];
    }
    if (t + step < n_tiles) load_row(t + step, next);
    const uint16_t* const run = part + (uint64_t)t * cap;
    for (uint32_t a = (at[0] & ~7u) + 8 * in_group; a < end; a += 8 * lpg) {
      const uint4 x = gload16(run + a);
      uint32_t fields = 0;
#pragma unroll
      for (uint32_t i = 1; i < kBloomMaxPer; ++i) {
        if (i < per) {
          int32_t d = (int32_t)at[i] - (int32_t)a;
          d = 2 * (d < 0 ? 0 : d > 8 ? 8 : d);
          fields += 0x11111111u << d << d;
        }
      }
      const uint32_t from = at[0] > a ? at[0] - a : 0u, upto = end - a < 8 ? end - a : 8u;
      const uint32_t in_run = ((1u << upto) - 1u) & ~((1u << from) - 1u);
      const uint32_t v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (uint32_t i = 0; i < 8; ++i) {
        // the byte address of the position's word in its sub-range, for both halves at once
        const uint32_t pair = (v[i / 2] >> 3) & word_mask;
        const uint32_t word = i & 1u ? pair >> 16 : pair & 0xFFFFu;
        const uint32_t bit = i & 1u ? v[i / 2] >> 16 : v[i / 2];
        uint32_t* const at_word =
            reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(bloom_lds) + (((fields >> (4 * i) & 15u) << (sb - 3)) + word));
        atomicOr(at_word, (in_run >> i & 1u) << (bit & 31u));
      }
    }
  }
  __syncthreads();
  const uint64_t w0 = (uint64_t)p * n_bits_words;
  for (uint32_t i = threadIdx.x; i < n_bits_words && w0 + i < n_words; i += kBloomFillThreads) gp(words)[w0 + i] = bloom_lds[i];
}

// Few positions: device atomics on the cleared array. A bit that is there
// already (bits are only ever set, so a stale word costs an atomic at most)
// needs none, which keeps a small filter's few words from queueing.
__global__ __launch_bounds__(kBloomDirectThreads) void k_bloom_direct(const uint8_t* __restrict__ in, uint64_t n_bytes,
                                                                      uint64_t n_kmers, uint32_t k, uint32_t h, uint32_t m,
                                                                      uint32_t* __restrict__ words) {
  const uint64_t e = (uint64_t)blockIdx.x * kBloomDirectThreads + threadIdx.x;
  if (e >= n_kmers) return;
  uint64_t v = 0;
  bool ok = true;
  for (uint32_t q = 0; q < k; ++q) {
    const uint32_t c = gp(in)[e + q];
    ok &= c == 'A' || c == 'C' || c == 'G' || c == 'T';
    v = v << 2 | ((c >> 1 & 3u) ^ (c >> 2 & 1u));
  }
  if (!ok) return;
  const uint64_t x = fmix64(v);
  const uint32_t a = (uint32_t)x, b = (uint32_t)(x >> 32) | 1u;
  for (uint32_t i = 0; i < h; ++i) {
    const uint32_t pos = __umulhi(a + i * b, m), bit = 1u << (pos & 31u);
    if (!(__hip_atomic_load(&words[pos >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit))
      atomicOr(&words[pos >> 5], bit);
  }
}

__global__ void k_bloom_zero_words(uint32_t* __restrict__ words, uint64_t n) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) words[i] = 0u;
}

BloomPlan bloom_plan(uint64_t n_bytes, uint32_t k, uint32_t h, uint64_t m, uint32_t n_cu) {
  BloomPlan b{};
  b.ok = k >= 1 && k <= kBloomMaxK && h >= 1 && h <= kBloomMaxH && m >= 1 && m <= (uint64_t)kBloomMaxSubs << kBloomSubBits;
  if (!b.ok) return b;
  b.n_kmers = n_bytes >= k ? n_bytes - k + 1 : 0;
  b.n_words = (m + 31) / 32;
  b.max_entries = b.n_kmers * h;
  b.ok = b.n_kmers < (1ull << 32) && b.max_entries < (1ull << 32);
  if (!b.ok || b.max_entries < kBloomDirectMax) return b;
  b.sb = kBloomSubBitsMin;
  while (b.sb < kBloomSubBits && ((m - 1) >> b.sb) + 1 > kBloomSubsWanted) ++b.sb;
  b.S = (uint32_t)((m - 1) >> b.sb) + 1;
  // as few sub-ranges per range as fill the chip in whole rounds of workgroups
  const uint32_t slots = kBloomFillPerCu * n_cu;
  const uint32_t rounds = (b.S + slots * kBloomMaxPer - 1) / (slots * kBloomMaxPer);
  b.per = (b.S + slots * rounds - 1) / (slots * rounds);
  b.grid = (b.S + b.per - 1) / b.per;
  const uint32_t tile = bloom_batches(h) * kBloomBatch;
  b.cap = tile * h;
  b.n_tiles = (uint32_t)((b.n_kmers + tile - 1) / tile);
  b.row_words = (b.S + 1 + kBloomRowPad + 1) / 2;
  // lanes per run: the pieces of a run two deviations above the mean, wherever it starts in its first piece
  const double mean = (double)b.cap * b.per / b.S;
  const double pieces = std::ceil((mean + 2.0 * std::sqrt(mean) + 7.0) / 8.0);
  b.lpg = pieces > kWave ? (uint32_t)kWave : (uint32_t)pieces;
  return b;
}

uint64_t bloom_row_bytes(const BloomPlan& b) { return 4ull * b.row_words * b.n_tiles; }
uint64_t bloom_part_bytes(const BloomPlan& b) { return b.n_tiles ? 2 * (b.max_entries + kBloomPartPad) : 0; }

template <uint32_t H>
static hipError_t bloom_tiles(const uint8_t* in, uint64_t n_bytes, uint32_t k, uint32_t m, const BloomPlan& b, uint32_t* rows,
                              uint16_t* part, hipStream_t s) {
  const uint32_t lds = 2 * b.cap + 4 * b.S;
  // (the most any filter takes: calls on other threads set the same)
  constexpr uint32_t kMost = 2 * bloom_batches(H) * kBloomBatch * H + 4 * kBloomMaxSubs;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_bloom_tile<H>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMost);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bloom_tile<H>, dim3(b.n_tiles), dim3(kBloomThreads), lds, s, in, n_bytes, b.n_kmers, k, m, b.sb, b.S,
                     b.row_words, rows, part);
  return hipGetLastError();
}

hipError_t bloom_enqueue(const uint8_t* in, uint64_t n_bytes, uint32_t k, uint32_t h, uint64_t m, const BloomPlan& b,
                         uint32_t* rows, uint16_t* part, uint32_t* words, hipStream_t s) {
  if (b.n_tiles == 0) {
    hipLaunchKernelGGL(k_bloom_zero_words, dim3(256), dim3(256), 0, s, words, b.n_words);
    if (b.n_kmers)
      hipLaunchKernelGGL(k_bloom_direct, dim3((uint32_t)((b.n_kmers + kBloomDirectThreads - 1) / kBloomDirectThreads)),
                         dim3(kBloomDirectThreads), 0, s, in, n_bytes, b.n_kmers, k, h, (uint32_t)m, words);
    return hipGetLastError();
  }
  hipError_t e = hipErrorInvalidValue;
  const uint32_t mb = (uint32_t)m;
  switch (h) {
    case 1: e = bloom_tiles<1>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 2: e = bloom_tiles<2>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 3: e = bloom_tiles<3>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 4: e = bloom_tiles<4>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 5: e = bloom_tiles<5>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 6: e = bloom_tiles<6>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 7: e = bloom_tiles<7>(in, n_bytes, k, mb, b, rows, part, s); break;
    case 8: e = bloom_tiles<8>(in, n_bytes, k, mb, b, rows, part, s); break;
  }
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_bloom_fill), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(kBloomMaxPer << (kBloomSubBits - 3)));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bloom_fill, dim3(b.grid), dim3(kBloomFillThreads), b.per << (b.sb - 3), s, part, rows, b.row_words,
                     b.n_tiles, b.cap, b.sb, b.per, b.lpg, b.n_words, words);
  return hipGetLastError();
}

}  // namespace mr
