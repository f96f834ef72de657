// LSD radix sort by 8-bit digits and the reduce of sorted runs (gfx950): the
// SORT container, the ordering of hash-table outputs and of the Reverse
// Index's pairs.
//
// Elements: a uint32 key, a (uint32 key, uint32 value) pair, or a uint64 key.
// One pass is three kernels: the digit counts of every 8192-element tile, one
// scan over the tiles per digit, and the stable scatter. A tile ranks its
// elements with wave ballots (equal digits of a 64-element row find each
// other in 8 ballots, whatever the distribution), orders itself in LDS and
// writes each digit's run as one contiguous piece (32 elements on average).
//
// The first pass also gathers which key bits differ anywhere in the input. A
// later pass over a digit in which no bit differs would copy its input as it
// stands; its kernels return at once, and every kernel derives from the same
// word where the data is.
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace mr {

constexpr uint32_t kRsThreads = 512;
constexpr uint32_t kRsWaves = kRsThreads / kWave;
constexpr uint32_t kRsDigits = 256;
// Elements per thread (PER below): 16, so that a digit's run of a tile is 32
// elements on average, or 4 for inputs of up to kRsSmall elements, which leave
// CUs idle with tiles of 8192 and wait on one tile's chain of 16 rows (10,000
// pairs: 8.8 us per scatter with 16, 4.2 us with 4).
constexpr uint32_t kRsPerLarge = 16, kRsPerSmall = 4;
constexpr uint64_t kRsSmall = 1ull << 20;

MR_DEV uint64_t rs_key(uint32_t e) { return e; }
MR_DEV uint64_t rs_key(uint2 e) { return e.x; }
MR_DEV uint64_t rs_key(unsigned long long e) { return e; }
MR_DEV uint32_t rs_digit(uint32_t e, uint32_t shift) { return (e >> shift) & 0xFFu; }
MR_DEV uint32_t rs_digit(uint2 e, uint32_t shift) { return (e.x >> shift) & 0xFFu; }
MR_DEV uint32_t rs_digit(unsigned long long e, uint32_t shift) { return (uint32_t)(e >> shift) & 0xFFu; }

MR_DEV bool rs_skip(uint64_t diff, uint32_t shift) { return shift && !((diff >> shift) & 0xFFu); }

// Where the data of a pass is: the input, or one of the two buffers.
template <typename E>
struct RsData {
  // first pass: uint64 elements; or uint32 keys, and for pairs values, `stride` words apart
  const void* in;
  const uint32_t* vals;
  uint32_t stride;
  uint64_t n;
  E *a, *b;
  unsigned long long* diff;  // differing key bits (first pass writes, later ones read)
};

template <typename E>
MR_DEV E rs_in(const RsData<E>& D, uint64_t i) {
  return gp(reinterpret_cast<const E*>(D.in))[i];
}
template <>
MR_DEV uint32_t rs_in<uint32_t>(const RsData<uint32_t>& D, uint64_t i) {
  return gp(reinterpret_cast<const uint32_t*>(D.in))[i * D.stride];
}
template <>
MR_DEV uint2 rs_in<uint2>(const RsData<uint2>& D, uint64_t i) {
  return make_uint2(gp(reinterpret_cast<const uint32_t*>(D.in))[i * D.stride], gp(D.vals)[i * D.stride]);
}

template <typename E>
MR_DEV E rs_load(const E* p, uint64_t i) {
  return gp(p)[i];
}
template <>
MR_DEV uint2 rs_load<uint2>(const uint2* p, uint64_t i) {
  const unsigned long long v = gp(reinterpret_cast<const unsigned long long*>(p))[i];
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}

template <typename E>
MR_DEV void rs_store(E* p, uint64_t i, E x) {
  gp(p)[i] = x;
}
template <>
MR_DEV void rs_store<uint2>(uint2* p, uint64_t i, uint2 x) {
  gp(reinterpret_cast<unsigned long long*>(p))[i] = (unsigned long long)x.y << 32 | x.x;
}

// Digit counts of each tile: hist[digit * n_tiles + tile]. Eight copies of
// the counters, one per lane modulo 8, so that rows of few distinct digits
// (the top digits of small keys, skewed keys) serialise eight lanes, not 64.
// The first pass (FIRST) checks the declared range and gathers the differing
// key bits.
template <typename E, bool FIRST, uint32_t PER>
__global__ __launch_bounds__(kRsThreads) void k_rsort_hist(RsData<E> D, uint32_t shift, uint32_t n_tiles,
                                                           uint32_t* __restrict__ hist, uint64_t R,
                                                           uint32_t* __restrict__ flags) {
  constexpr uint32_t kTile = kRsThreads * PER;
  constexpr uint32_t kCopies = 8, kLd = kRsDigits + 4;  // (copies start 4 banks apart)
  __shared__ uint32_t h[kCopies * kLd];
  __shared__ unsigned long long wdiff[kRsWaves];
  uint64_t diff = 0;
  if (!FIRST) {
    diff = *D.diff;
    if (rs_skip(diff, shift)) return;
  }
  for (uint32_t i = threadIdx.x; i < kCopies * kLd; i += kRsThreads) h[i] = 0;
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  const uint32_t m = D.n - base < kTile ? (uint32_t)(D.n - base) : kTile;
  const E* src = nullptr;
  if (!FIRST) src = rs_moves_before(diff, shift) % 2 ? D.a : D.b;
  E e[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint32_t i = u * kRsThreads + threadIdx.x;
    e[u] = E{};
    if (i < m) e[u] = FIRST ? rs_in<E>(D, base + i) : rs_load<E>(src, base + i);
  }
  __syncthreads();
  uint32_t* const mine = h + (threadIdx.x % kCopies) * kLd;
  uint64_t x = 0;
  bool bad = false;
  const uint64_t k0 = FIRST ? rs_key(rs_in<E>(D, 0)) : 0;
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    if (u * kRsThreads + threadIdx.x >= m) break;
    atomicAdd(&mine[rs_digit(e[u], shift)], 1u);
    if (FIRST) {
      const uint64_t k = rs_key(e[u]);
      x |= k ^ k0;
      bad |= R && k >= R;
    }
  }
  if (FIRST) {
    if (bad) atomicOr(flags, kFlagBadInput);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor((unsigned long long)x, o);
    if (lane_id() == 0) wdiff[threadIdx.x / kWave] = x;
  }
  __syncthreads();
  if (FIRST && threadIdx.x == 0) {
    uint64_t all = 0;
    for (uint32_t w = 0; w < kRsWaves; ++w) all |= wdiff[w];
    // (a stale read only costs an atomic that adds nothing)
    if (all & ~__hip_atomic_load(D.diff, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(D.diff, all);
  }
  if (threadIdx.x < kRsDigits) {
    uint32_t c = 0;
#pragma unroll
    for (uint32_t q = 0; q < kCopies; ++q) c += h[q * kLd + threadIdx.x];
    hist[(uint64_t)threadIdx.x * n_tiles + blockIdx.x] = c;
  }
}

// One workgroup per digit: exclusive scan of its tile counts in place, the
// digit's total to tot[digit]. Each wave takes 64 x kRsScanBatch neighbouring
// counts per step, scanned with DPP lane shifts.
constexpr uint32_t kRsScanThreads = 1024;
constexpr uint32_t kRsScanBatch = 4;

__global__ __launch_bounds__(kRsScanThreads) void k_rsort_scan(uint32_t* __restrict__ hist, uint32_t n_tiles, uint32_t shift,
                                                               const unsigned long long* __restrict__ diff,
                                                               uint32_t* __restrict__ tot) {
  if (rs_skip(*diff, shift)) return;
  __shared__ uint32_t ws[kRsScanThreads / kWave];
  uint32_t* const row = hist + (uint64_t)blockIdx.x * n_tiles;
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  uint32_t carry = 0;
  for (uint32_t b = 0; b < n_tiles; b += kRsScanThreads * kRsScanBatch) {
    uint32_t v[kRsScanBatch], x[kRsScanBatch], sum = 0;
    const uint32_t i0 = b + wv * kWave * kRsScanBatch + lane;
#pragma unroll
    for (uint32_t u = 0; u < kRsScanBatch; ++u) v[u] = i0 + u * kWave < n_tiles ? row[i0 + u * kWave] : 0u;
#pragma unroll
    for (uint32_t u = 0; u < kRsScanBatch; ++u) {
      const uint32_t incl = wave_incl_scan(v[u]);
      x[u] = sum + incl - v[u];
      sum += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    }
    if (lane == 0) ws[wv] = sum;
    __syncthreads();
    uint32_t pre = carry, all = 0;
    for (uint32_t w = 0; w < kRsScanThreads / kWave; ++w) {
      if (w < wv) pre += ws[w];
      all += ws[w];
    }
#pragma unroll
    for (uint32_t u = 0; u < kRsScanBatch; ++u)
      if (i0 + u * kWave < n_tiles) row[i0 + u * kWave] = pre + x[u];
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) tot[blockIdx.x] = carry;
}

// Lanes of the wave whose digit equals this lane's (all 64 lanes take part).
MR_DEV uint64_t rs_match(uint32_t d) {
  uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
  for (uint32_t b = 0; b < 8; ++b) {
    const uint32_t sx = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // all ones where the bit is set
    const uint64_t set = __ballot((int32_t)sx < 0);
    lo &= ~((uint32_t)set ^ sx);
    hi &= ~((uint32_t)(set >> 32) ^ sx);
  }
  return (uint64_t)hi << 32 | lo;
}

// Stable scatter of one tile. Wave w holds the w-th eighth of the tile's
// elements as PER rows of 64; row by row, a lane's rank among the wave's
// elements of its digit is the wave's count so far plus the matching lanes
// below it. The tile's order is (digit, wave, row, lane); it is written to
// LDS and from there to the digits' global places.
template <typename E, bool FIRST, uint32_t PER>
__global__ __launch_bounds__(kRsThreads) void k_rsort_scatter(RsData<E> D, uint32_t shift, uint32_t n_tiles,
                                                              const uint32_t* __restrict__ hist,
                                                              const uint32_t* __restrict__ tot) {
  constexpr uint32_t kTile = kRsThreads * PER;
  __shared__ E st[kTile];
  __shared__ uint32_t wh[kRsWaves][kRsDigits];  // the wave's digit counts, then its first place per digit
  __shared__ uint32_t delta[kRsDigits];         // global place of LDS place i of digit d: delta[d] + i
  __shared__ uint32_t sa[kRsDigits / kWave], sb[kRsDigits / kWave];
  uint64_t diff = 0;
  if (!FIRST) {
    diff = *D.diff;
    if (rs_skip(diff, shift)) return;
  }
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  const uint32_t m = D.n - base < kTile ? (uint32_t)(D.n - base) : kTile;
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  const bool odd = FIRST ? false : rs_moves_before(diff, shift) % 2;
  const E* const src = odd ? D.a : D.b;
  E* const dst = FIRST || !odd ? D.a : D.b;
  E e[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint32_t i = wv * (kWave * PER) + u * kWave + lane;
    e[u] = E{};
    if (i < m) e[u] = FIRST ? rs_in<E>(D, base + i) : rs_load<E>(src, base + i);
  }
  for (uint32_t i = threadIdx.x; i < kRsWaves * kRsDigits; i += kRsThreads) (&wh[0][0])[i] = 0;
  // this tile's global offset of each digit, loaded early
  uint32_t goff = 0, dtot = 0;
  if (threadIdx.x < kRsDigits) {
    goff = hist[(uint64_t)threadIdx.x * n_tiles + blockIdx.x];
    dtot = tot[threadIdx.x];
  }
  __syncthreads();
  uint32_t rank[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    // elements past the end sit behind all others of the tile; they count in
    // the last digit, after every real element, and are not written
    const bool act = wv * (kWave * PER) + u * kWave + lane < m;
    const uint32_t d = act ? rs_digit(e[u], shift) : kRsDigits - 1;
    const uint64_t same = rs_match(d);
    const uint32_t below = mbcnt(same);
    const uint32_t pre = __hip_atomic_load(&wh[wv][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    if (below == 0) __hip_atomic_store(&wh[wv][d], pre + popc64(same), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (LDS operations of a wave run in order)
    rank[u] = pre + below;
  }
  __syncthreads();
  uint32_t cnt = 0;
  uint32_t isum = 0, gsum = 0;
  if (threadIdx.x < kRsDigits) {
#pragma unroll
    for (uint32_t w = 0; w < kRsWaves; ++w) {
      const uint32_t c = wh[w][threadIdx.x];
      wh[w][threadIdx.x] = cnt;
      cnt += c;
    }
    isum = wave_incl_scan(cnt);
    gsum = wave_incl_scan(dtot);
    if (lane == kWave - 1) {
      sa[wv] = isum;
      sb[wv] = gsum;
    }
  }
  __syncthreads();
  if (threadIdx.x < kRsDigits) {
    uint32_t local = isum - cnt, global = gsum - dtot;
    for (uint32_t w = 0; w < wv; ++w) {
      local += sa[w];
      global += sb[w];
    }
#pragma unroll
    for (uint32_t w = 0; w < kRsWaves; ++w) wh[w][threadIdx.x] += local;
    delta[threadIdx.x] = global + goff - local;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const bool act = wv * (kWave * PER) + u * kWave + lane < m;
    const uint32_t d = act ? rs_digit(e[u], shift) : kRsDigits - 1;
    st[wh[wv][d] + rank[u]] = e[u];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint32_t i = u * kRsThreads + threadIdx.x;
    if (i < m) {
      const E x = st[i];
      rs_store<E>(dst, delta[rs_digit(x, shift)] + i, x);
    }
  }
}

// ----------------------------------------------------------------------------
// reduce of sorted runs
// ----------------------------------------------------------------------------
// A wave takes a chunk of PER rows of 64 sorted elements. The first
// kernel counts the chunk's run heads; after the scan, the second writes the
// key of every head and the value of every run that starts in the chunk, as
// far as the chunk sees it, and leaves the value of the elements before the
// first head (a run from an earlier chunk) in lead[chunk]; the third adds
// those to their runs.
// Small inputs take chunks of 4 rows, for the reason given at kRsPerSmall.
constexpr uint32_t kRunThreads = 256;

template <typename E>
MR_DEV const E* rs_sorted(const RsData<E>& D, uint32_t bits) {
  return rs_moves_before(*D.diff, bits) % 2 ? D.a : D.b;
}

template <typename E, uint32_t PER>
__global__ __launch_bounds__(kRunThreads) void k_runs_count(RsData<E> D, uint32_t bits, uint32_t* __restrict__ heads) {
  const E* const s = rs_sorted(D, bits);
  const uint32_t lane = lane_id();
  const uint64_t c = (uint64_t)blockIdx.x * (kRunThreads / kWave) + threadIdx.x / kWave, base = c * (kWave * PER);
  if (base >= D.n) return;
  uint32_t k[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t i = base + u * kWave + lane;
    k[u] = i < D.n ? (uint32_t)rs_key(rs_load<E>(s, i)) : 0u;
  }
  uint32_t last = base ? (uint32_t)rs_key(rs_load<E>(s, base - 1)) : 0u, n = 0;
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t i = base + u * kWave + lane;
    const uint32_t prev = from_prev_lane(k[u], last);
    n += popc64(__ballot(i < D.n && (i == 0 || k[u] != prev)));
    last = (uint32_t)__builtin_amdgcn_readlane((int)k[u], kWave - 1);
  }
  if (lane == 0) heads[c] = n;
}

MR_DEV unsigned long long run_join(int op, unsigned long long a, unsigned long long b) {
  return op <= 1 ? a + b : op == 2 ? (a < b ? a : b) : (a > b ? a : b);
}

MR_DEV unsigned long long readlane64(unsigned long long v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
  return (unsigned long long)hi << 32 | lo;
}

template <int OP>
MR_DEV void run_store(void* out, uint64_t pos, unsigned long long v) {
  if (OP == 1) reinterpret_cast<unsigned long long*>(out)[pos] = v;
  else reinterpret_cast<uint32_t*>(out)[pos] = (uint32_t)v;
}

// The row's value of the run that lane l belongs to, from the run's first
// lane in the row (`start`) up to lane l.
template <int OP>
MR_DEV unsigned long long run_row_value(uint32_t v, uint32_t lane, uint32_t start) {
  if (OP == 0) return lane - start + 1;
  if (OP == 1) {
    // prefix sums of the 16-bit halves (64 of them stay below 2^22); the run's sum is a difference
    const uint32_t lo = wave_incl_scan(v & 0xFFFFu), hi = wave_incl_scan(v >> 16);
    const uint32_t at = start ? start - 1 : 0;
    const uint32_t plo = (uint32_t)__shfl((int)lo, (int)at), phi = (uint32_t)__shfl((int)hi, (int)at);
    return (unsigned long long)(lo - (start ? plo : 0u)) + ((unsigned long long)(hi - (start ? phi : 0u)) << 16);
  }
  uint32_t x = v;
#pragma unroll
  for (uint32_t o = 1; o < kWave; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, o);
    if (lane >= start + o) x = OP == 2 ? (y < x ? y : x) : (y > x ? y : x);
  }
  return x;
}

MR_DEV uint32_t rs_val(uint32_t) { return 1u; }
MR_DEV uint32_t rs_val(uint2 e) { return e.y; }

template <typename E, int OP, uint32_t PER>
__global__ __launch_bounds__(kRunThreads) void k_runs_write(RsData<E> D, uint32_t bits, const uint32_t* __restrict__ heads,
                                                            uint32_t* __restrict__ out_keys, void* __restrict__ out_vals,
                                                            uint64_t cap, unsigned long long* __restrict__ lead) {
  const E* const s = rs_sorted(D, bits);
  const uint32_t lane = lane_id();
  const uint64_t c = (uint64_t)blockIdx.x * (kRunThreads / kWave) + threadIdx.x / kWave, base = c * (kWave * PER);
  if (base >= D.n) return;
  E e[PER];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t i = base + u * kWave + lane;
    e[u] = E{};
    if (i < D.n) e[u] = rs_load<E>(s, i);
  }
  uint32_t last = base ? (uint32_t)rs_key(rs_load<E>(s, base - 1)) : 0u;
  uint64_t pos = heads[c];  // runs before the row
  // the run open at the row's start: its value so far, and whether it started in this chunk
  unsigned long long open = 0;
  bool has_open = false, inside = false, led = false;
  unsigned long long lead_v = 0;
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t r0 = base + u * kWave;
    if (r0 >= D.n) break;
    const uint32_t m = D.n - r0 < kWave ? (uint32_t)(D.n - r0) : kWave;  // elements of the row
    const uint32_t k = (uint32_t)rs_key(e[u]);
    const uint32_t prev = from_prev_lane(k, last);
    const uint64_t H = __ballot(lane < m && (r0 + lane == 0 || k != prev));
    const uint64_t below = H & (lane == 63 ? ~0ull : (2ull << lane) - 1);  // heads up to this lane
    const uint32_t start = below ? 63u - (uint32_t)__builtin_clzll(below) : 0u;
    unsigned long long v = run_row_value<OP>(rs_val(e[u]), lane, start);
    if (has_open && !below) v = run_join(OP, open, v);
    if (H & 1ull) {  // the open run ended with the row before
      if (has_open) {
        if (inside) {
          if (lane == 0 && pos - 1 < cap) run_store<OP>(out_vals, pos - 1, open);
        } else {
          lead_v = open;
          led = true;
        }
      }
    }
    // heads write their key; the last lane of a run that ends in the row writes its value
    const uint64_t o = pos + popc64(below) - 1;  // (of this lane's run; only used where the run started in the chunk)
    if ((H >> lane & 1ull) && o < cap) out_keys[o] = k;
    const bool ends = lane + 1 < m && (H >> (lane + 1) & 1ull);
    const uint64_t first_end = H & ~1ull;  // a run open at the row's start (or the head at lane 0) ends before this bit
    if (ends) {
      if (below || inside) {
        if (o < cap) run_store<OP>(out_vals, o, v);
      }
    }
    if (!(H & 1ull) && first_end && !inside) {  // the run from an earlier chunk ends in this row
      lead_v = readlane64(v, (int)__builtin_ctzll(first_end) - 1);
      led = true;
    }
    open = readlane64(v, (int)m - 1);
    has_open = true;
    inside = inside || H != 0;
    pos += popc64(H);
    last = (uint32_t)__builtin_amdgcn_readlane((int)k, kWave - 1);
  }
  if (inside) {
    if (lane == 0 && pos - 1 < cap) run_store<OP>(out_vals, pos - 1, open);
  } else {
    lead_v = open;
    led = true;
  }
  // (no element before the first head: a value that changes nothing)
  if (lane == 0) lead[c] = led ? lead_v : (OP == 2 ? 0xFFFFFFFFull : 0ull);
}

// Neighbouring chunks inside one long run add to the same place: the lanes of
// a wave join those first (one atomic per run and wave instead of one per
// chunk, which at 16 keys over 16 M elements took 177 us).
template <int OP>
__global__ __launch_bounds__(256) void k_runs_lead(uint64_t n_chunks, const uint32_t* __restrict__ heads,
                                                   const unsigned long long* __restrict__ lead,
                                                   void* __restrict__ out_vals, uint64_t cap) {
  const unsigned long long neutral = OP == 2 ? 0xFFFFFFFFull : 0ull;
  const uint64_t c = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  const uint32_t lane = lane_id();
  // the run that was open where the chunk starts (0: the first chunk, or none)
  const uint32_t h = c < n_chunks ? heads[c] : 0u;
  unsigned long long v = h ? lead[c] : neutral;
#pragma unroll
  for (uint32_t o = 1; o < kWave; o <<= 1) {
    const unsigned long long y = __shfl_up(v, o);
    const uint32_t hy = (uint32_t)__shfl_up((int)h, o);
    if (lane >= o && hy == h) v = run_join(OP, y, v);
  }
  const uint32_t next = (uint32_t)__shfl_down((int)h, 1);
  if (!h || v == neutral || (lane + 1 < kWave && next == h)) return;
  const uint64_t pos = h - 1;
  if (pos >= cap) return;
  if (OP == 1) atomicAdd(&reinterpret_cast<unsigned long long*>(out_vals)[pos], v);
  else if (OP == 0) atomicAdd(&reinterpret_cast<uint32_t*>(out_vals)[pos], (uint32_t)v);
  else if (OP == 2) atomicMin(&reinterpret_cast<uint32_t*>(out_vals)[pos], (uint32_t)v);
  else atomicMax(&reinterpret_cast<uint32_t*>(out_vals)[pos], (uint32_t)v);
}

// ----------------------------------------------------------------------------
// host launchers
// ----------------------------------------------------------------------------

static uint32_t rs_per(uint64_t n) { return n <= kRsSmall ? kRsPerSmall : kRsPerLarge; }

RadixPlan radix_plan(uint64_t n) {
  RadixPlan p{};
  const uint64_t tile = (uint64_t)kRsThreads * rs_per(n), chunk = (uint64_t)kWave * rs_per(n);
  p.n_tiles = (uint32_t)((n + tile - 1) / tile);
  p.n_chunks = (n + chunk - 1) / chunk;
  // (scratch that covers every smaller input too)
  const bool large = n > kRsSmall;
  p.hist_words = (uint64_t)kRsDigits * std::max<uint64_t>(p.n_tiles, large ? kRsSmall / (kRsThreads * kRsPerSmall) : 0);
  p.chunk_cap = std::max<uint64_t>(p.n_chunks, large ? kRsSmall / (kWave * kRsPerSmall) : 0);
  return p;
}

template <typename E, uint32_t PER>
static void rs_sort_per(const RsData<E>& D, uint32_t bits, uint32_t* hist, uint32_t* tot, uint64_t R, uint32_t* flags,
                        hipStream_t s) {
  const uint32_t n_tiles = radix_plan(D.n).n_tiles;
  for (uint32_t sh = 0; sh < bits; sh += 8) {
    if (sh == 0) {
      hipLaunchKernelGGL((k_rsort_hist<E, true, PER>), dim3(n_tiles), dim3(kRsThreads), 0, s, D, sh, n_tiles, hist, R, flags);
    } else {
      hipLaunchKernelGGL((k_rsort_hist<E, false, PER>), dim3(n_tiles), dim3(kRsThreads), 0, s, D, sh, n_tiles, hist, R, flags);
    }
    hipLaunchKernelGGL(k_rsort_scan, dim3(kRsDigits), dim3(kRsScanThreads), 0, s, hist, n_tiles, sh, D.diff, tot);
    if (sh == 0) {
      hipLaunchKernelGGL((k_rsort_scatter<E, true, PER>), dim3(n_tiles), dim3(kRsThreads), 0, s, D, sh, n_tiles, hist, tot);
    } else {
      hipLaunchKernelGGL((k_rsort_scatter<E, false, PER>), dim3(n_tiles), dim3(kRsThreads), 0, s, D, sh, n_tiles, hist, tot);
    }
  }
}

// Sorts by the low `bits` key bits (rounded up to whole digits, at least one).
template <typename E>
static hipError_t rs_sort(const RsData<E>& D, uint32_t bits, uint32_t* hist, uint32_t* tot, uint64_t R, uint32_t* flags,
                          hipStream_t s) {
  if (rs_per(D.n) == kRsPerSmall) rs_sort_per<E, kRsPerSmall>(D, bits, hist, tot, R, flags, s);
  else rs_sort_per<E, kRsPerLarge>(D, bits, hist, tot, R, flags, s);
  return hipGetLastError();
}

template <typename E, int OP, uint32_t PER>
static hipError_t rs_reduce_per(const RsData<E>& D, uint32_t bits, const SortLaunch& L, hipStream_t s) {
  const uint64_t n_chunks = radix_plan(D.n).n_chunks;
  const uint32_t g = (uint32_t)((n_chunks + kRunThreads / kWave - 1) / (kRunThreads / kWave));
  hipLaunchKernelGGL((k_runs_count<E, PER>), dim3(g), dim3(kRunThreads), 0, s, D, bits, L.heads);
  const hipError_t e = scan_exclusive_u32(L.heads, n_chunks, L.scan_sums, L.n_out, s, L.end);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_runs_write<E, OP, PER>), dim3(g), dim3(kRunThreads), 0, s, D, bits, L.heads, L.out_keys, L.out_vals,
                     L.cap, L.lead);
  hipLaunchKernelGGL(k_runs_lead<OP>, dim3((uint32_t)((n_chunks + 255) / 256)), dim3(256), 0, s, n_chunks, L.heads, L.lead,
                     L.out_vals, L.cap);
  return hipGetLastError();
}

template <typename E, int OP>
static hipError_t rs_reduce(const RsData<E>& D, uint32_t bits, const SortLaunch& L, hipStream_t s) {
  return rs_per(D.n) == kRsPerSmall ? rs_reduce_per<E, OP, kRsPerSmall>(D, bits, L, s)
                                    : rs_reduce_per<E, OP, kRsPerLarge>(D, bits, L, s);
}

static uint32_t whole_digits(uint32_t bits) { return bits < 8 ? 8 : (bits + 7) / 8 * 8; }

hipError_t int_enqueue_sort(const SortLaunch& L, hipStream_t s) {
  if (!L.n) return hipSuccess;
  const uint32_t bits = whole_digits(L.bits);
  if (L.op == 0) {  // the keys alone
    const RsData<uint32_t> D{L.in, nullptr, L.stride, L.n, static_cast<uint32_t*>(L.buf0), static_cast<uint32_t*>(L.buf1), L.diff};
    const hipError_t e = rs_sort(D, bits, L.hist, L.tot, L.R, L.flags, s);
    return e != hipSuccess ? e : rs_reduce<uint32_t, 0>(D, bits, L, s);
  }
  const RsData<uint2> D{L.in, L.vals_in, L.stride, L.n, static_cast<uint2*>(L.buf0), static_cast<uint2*>(L.buf1), L.diff};
  const hipError_t e = rs_sort(D, bits, L.hist, L.tot, L.R, L.flags, s);
  if (e != hipSuccess) return e;
  switch (L.op) {
    case 1: return rs_reduce<uint2, 1>(D, bits, L, s);
    case 2: return rs_reduce<uint2, 2>(D, bits, L, s);
    default: return rs_reduce<uint2, 3>(D, bits, L, s);
  }
}

// Hash-table output: pairs (key, index of its value) sorted by key, then keys and values written in order.
__global__ __launch_bounds__(256) void k_pairs_out(RsData<uint2> D, uint32_t bits, const unsigned long long* __restrict__ vals,
                                                   int op, uint32_t* __restrict__ out_keys, void* __restrict__ out_vals,
                                                   uint64_t cap) {
  const uint2* const s = rs_sorted(D, bits);
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < D.n && i < cap; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint2 e = rs_load<uint2>(s, i);
    out_keys[i] = e.x;
    const unsigned long long v = vals[e.y];
    if (op == 1) reinterpret_cast<unsigned long long*>(out_vals)[i] = v;
    else reinterpret_cast<uint32_t*>(out_vals)[i] = (uint32_t)v;
  }
}

hipError_t pairs_enqueue_out(const SortLaunch& L, const unsigned long long* vals, hipStream_t s) {
  if (!L.n) return hipSuccess;
  const RsData<uint2> D{L.in, L.vals_in, L.stride, L.n, static_cast<uint2*>(L.buf0), static_cast<uint2*>(L.buf1), L.diff};
  const hipError_t e = rs_sort(D, 32, L.hist, L.tot, 0, L.flags, s);
  if (e != hipSuccess) return e;
  const uint64_t g = (L.n + 255) / 256;
  hipLaunchKernelGGL(k_pairs_out, dim3((uint32_t)(g < 4096 ? g : 4096)), dim3(256), 0, s, D, 32u, vals, (int)L.op, L.out_keys,
                     L.out_vals, L.cap);
  return hipGetLastError();
}

hipError_t keys64_enqueue_sort(const Keys64Sort& L, hipStream_t s) {
  if (!L.n) return hipSuccess;
  const RsData<unsigned long long> D{L.in, nullptr, 1u, L.n, L.buf0, L.buf1, L.diff};
  return rs_sort(D, whole_digits(L.bits), L.hist, L.tot, 0, nullptr, s);
}

uint32_t keys64_sorted_bits(uint32_t bits) { return whole_digits(bits); }

}  // namespace mr
