// Integer-key MapReduce on gfx950: four reduce containers for uint32 keys.
//
// map: element i emits (key_i, value_i) (value 1 for plain keys);
// reduce: COUNT, SUM (64-bit), MIN or MAX per distinct key; output ascending.
//
// Containers (Section III-A; the choice between the two arrays is the rule of
// Section III-E):
//   LDS_ARRAY    per-workgroup array in LDS for a small declared key range;
//                each workgroup writes its partial array, a second kernel
//                adds the partials key by key (no atomics on shared data).
//   GLOBAL_ARRAY one array over the declared range updated with atomics
//                ("eliminating local arrays"); lanes holding the same hot key
//                merge first so one atomic carries the wave's sum.
//   HASH         a per-workgroup LDS hash cache (the bounded local container of
//                Section III-D) in front of a global open-addressing table;
//                keys fit the CAS word, so claim and compare are one step.
//   SORT         LSD radix sort of the pairs, then a segmented reduce (sort.hip).
// Every container ends in a compaction to distinct keys in ascending order.
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace mr {

// value slot encodings (all start at zero)
//   COUNT: count            SUM: 64-bit sum
//   MIN:   ~min (atomicMax) MAX: max
MR_DEV uint32_t enc_minmax(int op, uint32_t v) { return op == 2 ? ~v : v; }
MR_DEV uint32_t dec_minmax(int op, uint32_t v) { return op == 2 ? ~v : v; }

// ----------------------------------------------------------------------------
// element access
// ----------------------------------------------------------------------------
// Element i: key p[i * stride], value v[i * stride] (v == NULL: every value is
// 1). Interleaved pairs have stride 2 and v = p + 1.
struct IntIn {
  const uint32_t* p;
  const uint32_t* v;
  uint64_t n;
  uint32_t stride;
};

static IntIn int_in(const IntLaunch& L) { return {L.in, L.vals_in, L.n, L.stride}; }

MR_DEV void load_elem(const IntIn& in, uint64_t i, uint32_t& k, uint32_t& v) {
  k = in.p[i * in.stride];
  v = in.v ? in.v[i * in.stride] : 1u;
}

// ----------------------------------------------------------------------------
// state of a job
// ----------------------------------------------------------------------------
// The last small kernel of a job writes the job's state to host memory and
// clears the state block of the next job, so that a job needs neither a fill
// before its kernels nor a copy after them. Called by a whole workgroup;
// thread 0 knows n_out.
MR_DEV void int_publish(const IntEnd& E, unsigned long long n_out, unsigned long long n_claimed) {
  if (!E.host) return;
  for (uint32_t i = threadIdx.x; i < E.clear_words; i += blockDim.x) E.clear[i] = 0u;
  if (threadIdx.x == 0) {
    __hip_atomic_store(&E.host->n_out, n_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&E.host->n_claimed, n_claimed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&E.host->flags, *E.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ----------------------------------------------------------------------------
// LDS array
// ----------------------------------------------------------------------------
constexpr int kIntThreads = 512;
constexpr uint32_t kLdsCopiesBytes = 32 * 1024;  // LDS a workgroup may spend on copies of a small array

// LDS words from one array copy to the next: counts (padded to 8 bytes before
// 64-bit values), then values; with several copies an odd number of values, so
// that a key's copies lie in different banks.
static __host__ __device__ uint32_t lds_copy_words(uint32_t R, uint32_t op, uint32_t copies) {
  if (op == 1) {
    const uint32_t w = ((R + 1) & ~1u) + 2 * R;
    return copies > 1 && w % 4 == 0 ? w + 2 : w;
  }
  const uint32_t w = op == 0 ? R : 2 * R;
  return copies > 1 ? w | 1u : w;
}

// Partials layout: cnt_part[g * R + key], val_part[g * R + key] (val for SUM is 64-bit).
// A small array is kept in `copies` copies (a power of two), lane l adding to
// copy l % copies, so that a frequent key serialises 64 / copies lanes;
// elements are loaded eight at a time. With one copy and a load per step the
// step on 16 M pairs over 300 keys (SUM, skewed) took 250 us without the pairs'
// interleaving, 55 us this way.
template <int OP>
__global__ __launch_bounds__(kIntThreads) void k_lds_array(IntIn in, uint32_t R, uint32_t G, uint32_t copies,
                                                           uint32_t* __restrict__ cnt_part, void* __restrict__ val_part,
                                                           uint32_t* __restrict__ flags) {
  extern __shared__ unsigned long long lds_array[];
  uint32_t* const lds = reinterpret_cast<uint32_t*>(lds_array);
  const uint32_t words = lds_copy_words(R, OP, copies), off = OP == 1 ? (R + 1) & ~1u : R;  // values start `off` words in
  for (uint32_t i = threadIdx.x; i < words * copies; i += kIntThreads) lds[i] = 0;
  __syncthreads();
  uint32_t* const cnt = lds + (threadIdx.x & (copies - 1)) * words;
  unsigned long long* const sum = reinterpret_cast<unsigned long long*>(cnt + off);
  uint32_t* const mm = cnt + off;
  const uint64_t lo = in.n * blockIdx.x / G, hi = in.n * (blockIdx.x + 1) / G;
  const uint32_t stride = in.stride;
  bool bad = false;
  constexpr uint32_t kBatch = 8;
  for (uint64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kBatch * kIntThreads) {
    uint32_t k[kBatch], v[kBatch];
    const MR_GLOBAL uint32_t* kp = gp(in.p) + i0 * stride;
    const MR_GLOBAL uint32_t* vp = gp(in.v) + i0 * stride;
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      k[u] = v[u] = 0;
      if (i0 + u * kIntThreads < hi) {
        k[u] = kp[u * kIntThreads * stride];
        if (OP != 0) v[u] = vp[u * kIntThreads * stride];
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      if (i0 + u * kIntThreads >= hi) break;
      if (k[u] >= R) {
        bad = true;
        continue;
      }
      atomicAdd(&cnt[k[u]], 1u);
      if (OP == 1) atomicAdd(&sum[k[u]], (unsigned long long)v[u]);
      if (OP >= 2) atomicMax(&mm[k[u]], enc_minmax(OP, v[u]));
    }
  }
  if (bad) atomicOr(flags, kFlagBadInput);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < R; i += kIntThreads) {
    uint32_t c = 0, m = 0;
    unsigned long long s = 0;
    for (uint32_t q = 0; q < copies; ++q) {
      const uint32_t* const a = lds + q * words;
      c += a[i];
      if (OP == 1) s += reinterpret_cast<const unsigned long long*>(a + off)[i];
      if (OP >= 2) m = max(m, a[off + i]);
    }
    cnt_part[(uint64_t)blockIdx.x * R + i] = c;
    if (OP == 1) reinterpret_cast<unsigned long long*>(val_part)[(uint64_t)blockIdx.x * R + i] = s;
    if (OP >= 2) reinterpret_cast<uint32_t*>(val_part)[(uint64_t)blockIdx.x * R + i] = m;
  }
}

// G partial rows added into one: 64 keys per workgroup, each wave a
// sixteenth of the rows.
constexpr uint32_t kLdsReduceWaves = 16;

template <int OP>
__global__ __launch_bounds__(kLdsReduceWaves * kWave) void k_lds_array_reduce(uint32_t R, uint32_t G,
                                                                              const uint32_t* __restrict__ cnt_part,
                                                                              const void* __restrict__ val_part,
                                                                              uint32_t* __restrict__ dcnt,
                                                                              void* __restrict__ dval) {
  __shared__ uint32_t wc[kLdsReduceWaves][kWave], wm[kLdsReduceWaves][kWave];
  __shared__ unsigned long long wsum[kLdsReduceWaves][kWave];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave, k = blockIdx.x * kWave + lane;
  uint32_t c = 0, m = 0;
  unsigned long long s = 0;
  if (k < R) {
#pragma unroll 8
    for (uint32_t g = wv; g < G; g += kLdsReduceWaves) {
      c += cnt_part[(uint64_t)g * R + k];
      if (OP == 1) s += reinterpret_cast<const unsigned long long*>(val_part)[(uint64_t)g * R + k];
      if (OP >= 2) m = max(m, reinterpret_cast<const uint32_t*>(val_part)[(uint64_t)g * R + k]);
    }
  }
  wc[wv][lane] = c;
  if (OP == 1) wsum[wv][lane] = s;
  if (OP >= 2) wm[wv][lane] = m;
  __syncthreads();
  if (wv || k >= R) return;
  for (uint32_t w = 1; w < kLdsReduceWaves; ++w) {
    c += wc[w][lane];
    if (OP == 1) s += wsum[w][lane];
    if (OP >= 2) m = max(m, wm[w][lane]);
  }
  dcnt[k] = c;
  if (OP == 1) reinterpret_cast<unsigned long long*>(dval)[k] = s;
  if (OP >= 2) reinterpret_cast<uint32_t*>(dval)[k] = m;
}

// Output of an LDS array by one workgroup: the G partial rows are added (few
// of them; many are added by k_lds_array_reduce first and come as one row),
// the present keys placed by a scan of ballots, and the job's state published.
// One launch instead of the reduce, the block counts, their scan and the
// ordered write.
template <int OP, uint32_t PER>  // keys per thread
__global__ __launch_bounds__(1024) void k_lds_out(uint32_t R, uint32_t G, const uint32_t* __restrict__ cnt_part,
                                                  const void* __restrict__ val_part, uint32_t* __restrict__ out_keys,
                                                  void* __restrict__ out_vals, uint64_t cap,
                                                  unsigned long long* __restrict__ n_out, IntEnd E) {
  constexpr uint32_t kWaves = 1024 / kWave;
  __shared__ uint32_t place[PER * kWaves];  // present keys of (u, wave), then their first place
  __shared__ uint32_t ws[kWaves];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  uint32_t c[PER], m[OP >= 2 ? PER : 1];
  unsigned long long s[OP == 1 ? PER : 1];
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    c[u] = 0;
    if (OP == 1) s[u] = 0;
    if (OP >= 2) m[u] = 0;
  }
  constexpr int kRows = PER <= 4 ? 8 / PER : 1;  // rows in flight
#pragma unroll kRows
  for (uint32_t g = 0; g < G; ++g) {
#pragma unroll
    for (uint32_t u = 0; u < PER; ++u) {
      const uint32_t k = u * 1024 + threadIdx.x;
      if (k < R) {
        c[u] += cnt_part[(uint64_t)g * R + k];
        if (OP == 1) s[u] += reinterpret_cast<const unsigned long long*>(val_part)[(uint64_t)g * R + k];
        if (OP >= 2) m[u] = max(m[u], reinterpret_cast<const uint32_t*>(val_part)[(uint64_t)g * R + k]);
      }
    }
  }
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t b = __ballot(c[u] != 0);
    if (lane == 0) place[u * kWaves + wv] = popc64(b);
  }
  __syncthreads();
  const uint32_t mine = threadIdx.x < PER * kWaves ? place[threadIdx.x] : 0u;
  const uint32_t incl = wave_incl_scan(mine);
  if (lane == kWave - 1) ws[wv] = incl;
  __syncthreads();
  uint32_t pre = incl - mine, all = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    if (w < wv) pre += ws[w];
    all += ws[w];
  }
  if (threadIdx.x < PER * kWaves) place[threadIdx.x] = pre;
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < PER; ++u) {
    const uint64_t b = __ballot(c[u] != 0);
    const uint64_t o = place[u * kWaves + wv] + mbcnt(b);
    if (c[u] && o < cap) {
      out_keys[o] = u * 1024 + threadIdx.x;
      if (OP == 0) reinterpret_cast<uint32_t*>(out_vals)[o] = c[u];
      if (OP == 1) reinterpret_cast<unsigned long long*>(out_vals)[o] = s[u];
      if (OP >= 2) reinterpret_cast<uint32_t*>(out_vals)[o] = dec_minmax(OP, m[u]);
    }
  }
  if (threadIdx.x == 0) *n_out = all;
  int_publish(E, all, 0);
}

// ----------------------------------------------------------------------------
// global array with wave-level aggregation
// ----------------------------------------------------------------------------

// Merge lanes that hold the same key as the current leader, for a few rounds:
// hot keys leave the wave as one atomic; the rest update directly.
constexpr int kAggRounds = 4;

template <int OP>
MR_DEV void wave_combine(uint32_t k, uint32_t v, bool active, uint32_t& cnt_out, unsigned long long& sum_out,
                         uint32_t& mm_out, bool& leader) {
  cnt_out = 0;
  sum_out = 0;
  mm_out = 0;
  leader = false;
  bool pending = active;
#pragma unroll 1
  for (int r = 0; r < kAggRounds; ++r) {
    const uint64_t m = __ballot(pending);
    if (!m) return;
    const int ld = __ffsll((long long)m) - 1;
    const uint32_t lk = __shfl(k, ld);
    const bool same = pending && k == lk;
    const uint64_t grp = __ballot(same);
    // reductions over the group
    unsigned long long s = same ? (unsigned long long)v : 0ull;
    uint32_t mx = same ? enc_minmax(OP, v) : 0u;
    if (OP == 1) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    }
    if (OP >= 2) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
    }
    if ((int)lane_id() == ld) {
      leader = true;
      cnt_out = popc64(grp);
      sum_out = s;
      mm_out = mx;
    }
    if (same) pending = false;
  }
  if (pending) {  // not merged: update alone
    leader = true;
    cnt_out = 1;
    sum_out = v;
    mm_out = enc_minmax(OP, v);
  }
}

template <int OP>
__global__ __launch_bounds__(256) void k_global_array(IntIn in, uint32_t R, uint32_t* __restrict__ dcnt, void* __restrict__ dval,
                                                      uint32_t* __restrict__ flags) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t n_round = (in.n + stride - 1) / stride * stride;  // all lanes iterate together
  bool bad = false;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_round; i += stride) {
    uint32_t k = 0, v = 0;
    bool act = i < in.n;
    if (act) {
      load_elem(in, i, k, v);
      if (k >= R) {
        bad = true;
        act = false;
      }
    }
    uint32_t c, mm;
    unsigned long long s;
    bool lead;
    wave_combine<OP>(k, v, act, c, s, mm, lead);
    if (lead && c) {
      // a leader's own key is k (it leads its own group)
      atomicAdd(&dcnt[k], c);
      if (OP == 1) atomicAdd(&reinterpret_cast<unsigned long long*>(dval)[k], s);
      if (OP >= 2) atomicMax(&reinterpret_cast<uint32_t*>(dval)[k], mm);
    }
  }
  if (bad) atomicOr(flags, kFlagBadInput);
}

// ----------------------------------------------------------------------------
// global array filled by key-range partitions
//
// Device-scope atomics run far below the load rate (and serialise on a
// frequent key), so the array is not updated element by element. Each tile of
// elements is ordered by 2^kb-key range in LDS and written where it stands
// (16-bit offsets, and 32-bit values unless the op counts) with the start of
// each range's run; then workgroups reduce the ranges' runs of every tile in
// LDS arrays. A range is split over as many workgroups as its share of the
// elements asks for, so that neither few ranges nor a frequent key leaves the
// work to a few CUs: a range of one workgroup is stored once, a split range is
// merged into the dense arrays with atomics on neighbouring words.
// ----------------------------------------------------------------------------
constexpr uint32_t kVpPer = 16;                // elements per thread of the tile kernel
constexpr uint32_t kVpMaxParts = 2048;         // ranges
constexpr uint32_t kCompTile = 2048;  // keys per block of the ordered compaction of dense arrays (256 threads x 8)
constexpr uint32_t kUncounted = ~0u;  // a block whose present keys are still to be counted

// Threads of the tile kernel: 16,384-element tiles for counting, 8,192 where
// the staged values take twice the keys' LDS.
constexpr uint32_t vp_threads(uint32_t op) { return op == 0 ? 1024 : 512; }
constexpr uint32_t vp_tile(uint32_t op) { return vp_threads(op) * kVpPer; }
// Threads of the fill: counting takes up to 128 KB of LDS, one workgroup per CU.
constexpr uint32_t vp_fill_threads(uint32_t op) { return op == 0 ? 1024 : 512; }

template <int OP>
__global__ __launch_bounds__(vp_threads(OP), OP == 0 ? 8 : 6) void k_vp_tile(IntIn in, uint64_t R, uint32_t kb, uint32_t P,
                                                            uint32_t* __restrict__ runs, uint16_t* __restrict__ pk,
                                                            uint32_t* __restrict__ pv, uint32_t* __restrict__ flags) {
  constexpr uint32_t kThreads = vp_threads(OP), kTile = vp_tile(OP);
  extern __shared__ uint32_t base[];  // [P + 1] counts, then the start of each range's run in the tile
  __shared__ __attribute__((aligned(16))) uint16_t sk[kTile];
  __shared__ __attribute__((aligned(16))) uint32_t sv[OP == 0 ? 4 : kTile];
  __shared__ uint32_t ws[kThreads / kWave];
  const uint32_t t = blockIdx.x, lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t q = threadIdx.x; q <= P; q += kThreads) base[q] = 0;
  const uint64_t e0 = (uint64_t)t * kTile;
  uint32_t k[kVpPer], v[kVpPer];
  const uint32_t stride = in.stride;
  const MR_GLOBAL uint32_t* kp = gp(in.p) + e0 * stride;
  const MR_GLOBAL uint32_t* vp = gp(in.v) + e0 * stride;
  const uint32_t left = in.n - e0 < kTile ? (uint32_t)(in.n - e0) : kTile;
  uint32_t n_mine = 0;  // this thread's elements: k[0, n_mine)
  if (OP == 0 && stride == 1 && left == kTile && ((uintptr_t)in.p & 15u) == 0) {  // whole 16-byte vectors
    n_mine = kVpPer;
#pragma unroll
    for (uint32_t u = 0; u < kVpPer / 4; ++u) {
      const uint4 x = gload16(in.p + e0 + (u * kThreads + threadIdx.x) * 4);
      k[4 * u] = x.x;
      k[4 * u + 1] = x.y;
      k[4 * u + 2] = x.z;
      k[4 * u + 3] = x.w;
    }
  } else {
#pragma unroll
    for (uint32_t u = 0; u < kVpPer; ++u) {
      const uint32_t i = u * kThreads + threadIdx.x;
      k[u] = ~0u;
      v[u] = 0u;
      if (i < left) {
        ++n_mine;
        k[u] = kp[i * stride];
        if (OP != 0) v[u] = vp[i * stride];
      }
    }
  }
  __syncthreads();
  // Counts of the ranges. With values each element keeps its rank within its
  // range's run; counting takes its place with a second atomic instead, since
  // the ranks would cost the registers of the second workgroup per CU.
  bool bad = false;
  uint32_t rank[OP == 0 ? 1 : kVpPer];
#pragma unroll
  for (uint32_t u = 0; u < kVpPer; ++u) {
    if (k[u] < R) {
      const uint32_t r = atomicAdd(&base[k[u] >> kb], 1u);
      if (OP != 0) rank[u] = r;
    } else {
      bad |= u < n_mine;
    }
  }
  if (bad) atomicOr(flags, kFlagBadInput);
  __syncthreads();
  constexpr uint32_t kPer = kVpMaxParts / kThreads;  // ranges per thread
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t r = threadIdx.x * kPer + q;
    c[q] = r < P ? base[r] : 0u;
    sum += c[q];
  }
  const uint32_t incl = wave_incl_scan(sum);
  if (lane == kWave - 1) ws[wv] = incl;
  __syncthreads();
  uint32_t run = incl - sum, m = 0;
  for (uint32_t w = 0; w < kThreads / kWave; ++w) {
    if (w < wv) run += ws[w];
    m += ws[w];
  }
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t r = threadIdx.x * kPer + q;
    if (r < P) base[r] = run;
    run += c[q];
  }
  if (threadIdx.x == 0) base[P] = m;
  __syncthreads();
  uint32_t* const row = runs + (uint64_t)t * (P + 1);
  for (uint32_t q = threadIdx.x; q <= P; q += kThreads) row[q] = base[q];
  if (OP == 0) __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kVpPer; ++u) {
    if (k[u] >= R) continue;
    const uint32_t at = OP == 0 ? atomicAdd(&base[k[u] >> kb], 1u) : base[k[u] >> kb] + rank[u];
    sk[at] = (uint16_t)(k[u] & ((1u << kb) - 1));
    if (OP != 0) sv[at] = OP == 1 ? v[u] : enc_minmax(OP, v[u]);
  }
  __syncthreads();
  // (rows are whole tiles: the words past the tile's elements are written too and never used)
  for (uint32_t i = threadIdx.x; i * 8 < m; i += kThreads)
    gstore16(pk + e0 + i * 8, *reinterpret_cast<const uint4*>(&sk[i * 8]));
  if (OP != 0)
    for (uint32_t i = threadIdx.x; i * 4 < m; i += kThreads)
      gstore16(pv + e0 + i * 4, *reinterpret_cast<const uint4*>(&sv[i * 4]));
}

// Elements of each range in each of gridDim.y slices of the tiles:
// tot[slice * P + p]. (Adding them up with atomics in k_vp_tile, on the few
// words of 128 ranges, took 60 us of its 85 on 8 M pairs.)
constexpr uint32_t kVpTotThreads = 1024;
constexpr uint32_t kVpMaxSlices = 16;

__global__ __launch_bounds__(kVpTotThreads) void k_vp_totals(const uint32_t* __restrict__ runs, uint32_t P, uint32_t n_tiles,
                                                             uint32_t* __restrict__ tot) {
  __shared__ uint32_t s[kVpTotThreads];
  const uint32_t p = blockIdx.x * kWave + threadIdx.x % kWave;
  const uint32_t t0 = (uint32_t)((uint64_t)n_tiles * blockIdx.y / gridDim.y);
  const uint32_t t1 = (uint32_t)((uint64_t)n_tiles * (blockIdx.y + 1) / gridDim.y);
  uint32_t sum = 0;
  if (p < P) {
#pragma unroll 8
    for (uint32_t t = t0 + threadIdx.x / kWave; t < t1; t += kVpTotThreads / kWave) {
      const uint32_t* row = runs + (uint64_t)t * (P + 1) + p;
      sum += row[1] - row[0];
    }
  }
  s[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x < kWave && p < P) {
    for (uint32_t q = threadIdx.x + kWave; q < kVpTotThreads; q += kWave) sum += s[q];
    tot[blockIdx.y * P + p] = sum;
  }
}

// Workgroups of range p of 2^kb keys: one, up to `split` of its elements or four
// times its keys (a merged range touches all of its keys again), else one per
// `split`; and whether the elements are spread evenly over the slices of the
// tiles (a single slice of fewer than 256 tiles does not tell: finding the
// shares there cost 10 us and gained nothing).
MR_DEV uint32_t vp_parts(const uint32_t* __restrict__ tot, uint32_t slices, uint32_t P, uint32_t p, uint32_t kb,
                         uint32_t split, uint32_t& elems, bool& even) {
  uint32_t c = 0, most = 0;
#pragma unroll 4
  for (uint32_t y = 0; y < slices; ++y) {
    const uint32_t x = tot[y * P + p];
    c += x;
    most = x > most ? x : most;
  }
  elems = c;
  even = (uint64_t)most * slices <= c + (uint64_t)c / 2;
  return c <= split || c <= 4u << kb ? 1u : (c - 1) / split + 1;  // (c may be close to 2^32)
}

// One workgroup per part of a range (found from the parts' scan). LDS: values
// [2^kb] (64-bit for SUM), then one presence byte per key; COUNT: the counts;
// each followed by kVpSinks entries that take the elements of a piece outside
// the run, so that every piece runs the same branch-free code.
// The parts of a range that is spread unevenly over the tiles (sorted input)
// take equal shares of its elements instead of its tiles.
// kList = false: neighbouring lanes take a tile's run together, one
// eight-element piece (a 16-byte load of offsets) each, as many lanes as the
// part's mean run has pieces, pipelined over steps of kBatch tiles per group;
// runs far above the mean are left for whole waves afterwards. (Lanes by the
// mean over all ranges, the rest of a run by them one load after the other,
// and parts by tiles: 8 M sorted pairs over 2^16 keys, SUM, 256 us of a call of
// 356, now 151; 8 M pairs on one of 2^24 keys 1,365 us a call, now 374.)
// kList = true, for counting over many tiles of short runs: a wave takes 64
// tiles at a time, lane l loads tile l's run bounds and lists its run's pieces
// in LDS, and the listed pieces go to the lanes in order, so that every lane
// has a piece whatever the runs' lengths (2^28 elements over 2^24 keys: 228 us;
// groups of eight lanes, of which a run of 32 fills five, 277 us of vector and
// LDS issue). With few tiles per wave the list's chain of loads is not hidden
// (8 M pairs: 78 us against 33).
// A range of one workgroup also counts the present keys of its compaction
// blocks; those of the others are left to k_dense_count.
constexpr uint32_t kVpSinks = 32;
constexpr uint32_t kVpList = 384;  // pieces listed per wave
constexpr uint32_t vp_max_kb(uint32_t op) { return op == 0 ? 15 : 14; }
constexpr uint32_t vp_fill_lds(uint32_t op, uint32_t kb) { return (op == 0 ? 4 : op == 1 ? 9 : 5) * ((1u << kb) + kVpSinks); }

template <int OP, bool kList>
__global__ __launch_bounds__(vp_fill_threads(OP)) void k_vp_fill(uint64_t R, uint32_t kb, uint32_t P, uint32_t n_tiles,
                                                            uint32_t split, const uint32_t* __restrict__ runs,
                                                            const uint16_t* __restrict__ pk, const uint32_t* __restrict__ pv,
                                                            const uint32_t* __restrict__ tot, uint32_t slices,
                                                            uint32_t* __restrict__ dcnt, void* __restrict__ dval,
                                                            uint32_t* __restrict__ blk) {
  constexpr uint32_t kThreads = vp_fill_threads(OP);
  extern __shared__ unsigned long long vp_lds[];
  constexpr uint32_t kWaves = kThreads / kWave;
  // range, part, parts, elements, whether they are spread evenly; bounds of an uneven part; runs left for whole waves
  constexpr uint32_t kFound = 8;
  __shared__ uint32_t ws[kWaves], found[kFound];
  __shared__ uint32_t lists[kList ? kWaves : 1][kList ? kVpList : 1];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave, K = 1u << kb;
  constexpr uint32_t kPer = kVpMaxParts / kThreads;
  const uint32_t per = (P + kThreads - 1) / kThreads;  // ranges per thread
  uint32_t parts[kPer], elems[kPer], sum = 0;
  bool even[kPer];
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t r = threadIdx.x * per + q;
    parts[q] = q < per && r < P ? vp_parts(tot, slices, P, r, kb, split, elems[q], even[q]) : 0u;
    sum += parts[q];
  }
  const uint32_t incl = wave_incl_scan(sum);
  if (lane == kWave - 1) ws[wv] = incl;
  if (threadIdx.x < kFound) found[threadIdx.x] = 0;
  __syncthreads();
  uint32_t first = incl - sum, all = 0;
  for (uint32_t w = 0; w < kThreads / kWave; ++w) {
    if (w < wv) first += ws[w];
    all += ws[w];
  }
  // Workgroups are handed to the eight XCDs in turn; neighbouring ranges share
  // the lines where their runs meet and their run starts, so each XCD takes a
  // contiguous block of parts and its L2 serves those once.
  const uint32_t each = all / kXcds, whole = each * kXcds;
  const uint32_t b = blockIdx.x < whole ? blockIdx.x % kXcds * each + blockIdx.x / kXcds : blockIdx.x;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    if (b >= first && b < first + parts[q]) {
      found[0] = threadIdx.x * per + q;
      found[1] = b - first;
      found[2] = parts[q];
      found[3] = elems[q];
      found[4] = even[q];
    }
    first += parts[q];
  }
  unsigned long long* const sum64 = vp_lds;
  uint32_t* const val32 = reinterpret_cast<uint32_t*>(vp_lds);
  uint8_t* const here = reinterpret_cast<uint8_t*>(vp_lds) + (OP == 1 ? 8u : 4u) * (K + kVpSinks);
  const uint32_t words = vp_fill_lds(OP, kb) / 4;
  const uint32_t sink = K + lane % kVpSinks;
  __syncthreads();
  const uint32_t p = found[0], part = found[1], np = found[2];
  if (np == 0) return;  // more workgroups than parts
  for (uint32_t i = threadIdx.x; i < words; i += kThreads) val32[i] = 0;
  __syncthreads();
  uint32_t t0 = (uint32_t)((uint64_t)n_tiles * part / np), t1 = (uint32_t)((uint64_t)n_tiles * (part + 1) / np);
  if (np > 1 && !found[4]) {
    // equal shares of the elements: a bound is the number of tiles with fewer than so many elements before them
    const uint32_t c0 = (uint32_t)((uint64_t)found[3] * part / np), c1 = (uint32_t)((uint64_t)found[3] * (part + 1) / np);
    const uint32_t each_t = (n_tiles + kThreads - 1) / kThreads, a = threadIdx.x * each_t;
    const uint32_t z = a + each_t < n_tiles ? a + each_t : n_tiles;
    auto run = [&](uint32_t t) {
      const uint32_t* row = runs + (uint64_t)t * (P + 1) + p;
      return *gp(row + 1) - *gp(row);
    };
    uint32_t mine = 0;
    for (uint32_t t = a; t < z; ++t) mine += run(t);
    const uint32_t upto = wave_incl_scan(mine);
    if (lane == kWave - 1) ws[wv] = upto;
    __syncthreads();
    uint32_t before = upto - mine, n0 = 0, n1 = 0;
    for (uint32_t w = 0; w < wv; ++w) before += ws[w];
    for (uint32_t t = a; t < z && before < c1; ++t) {
      n0 += before < c0;
      ++n1;
      before += run(t);
    }
    if (n0) atomicAdd(&found[5], n0);
    if (n1) atomicAdd(&found[6], n1);
    __syncthreads();
    t0 = found[5];
    t1 = found[6];
  }
  constexpr uint32_t kTile = vp_tile(OP);
  struct Piece {
    uint4 k, v0, v1;
  };
  auto load = [&](uint64_t at, Piece& x) {  // eight elements from a multiple of 8
    x.k = gload16(pk + at);
    if (OP != 0) {
      x.v0 = gload16(pv + at);
      x.v1 = gload16(pv + at + 4);
    }
  };
  auto put = [&](uint32_t from, uint32_t upto, const Piece& x) {  // elements [from, upto) of the piece are in the run
    const uint32_t w[4] = {x.k.x, x.k.y, x.k.z, x.k.w};
    const uint32_t v[8] = {x.v0.x, x.v0.y, x.v0.z, x.v0.w, x.v1.x, x.v1.y, x.v1.z, x.v1.w};
    const int32_t in_run = (int32_t)(((1u << upto) - 1u) & ~((1u << from) - 1u));
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
      const uint32_t in = (uint32_t)(in_run << (31 - i) >> 31);  // all ones or zero
      const uint32_t at = (w[i >> 1] >> (16u * (i & 1u))) & 0xFFFFu;
      const uint32_t key = (at & in) | (sink & ~in);
      if (OP == 0) atomicAdd(&val32[key], 1u);
      if (OP == 1) atomicAdd(&sum64[key], (unsigned long long)v[i]);
      if (OP >= 2) atomicMax(&val32[key], v[i]);
      if (OP != 0) here[key] = 1;  // (every writer stores the same byte)
    }
  };
  if constexpr (kList) {
    uint32_t* const list = lists[wv];
    auto load_runs = [&](uint32_t tb, uint32_t& lo, uint32_t& hi) {
      lo = hi = 0;
      if (lane < kWave && tb + lane < t1) {
        const uint32_t* row = runs + (uint64_t)(tb + lane) * (P + 1) + p;
        lo = *gp(row);
        hi = *gp(row + 1);
      }
    };
    constexpr uint32_t kBatch = OP == 0 ? 6 : 3;  // pieces in flight per lane
    uint32_t lo, hi, lo1, hi1;
    load_runs(t0 + wv * kWave, lo, hi);
    for (uint32_t tb = t0 + wv * kWave; tb < t1; tb += kWaves * kWave, lo = lo1, hi = hi1) {
      load_runs(tb + kWaves * kWave, lo1, hi1);
      const uint32_t c = hi > lo ? (hi + 7) / 8 - lo / 8 : 0u;
      const uint32_t incl = wave_incl_scan(c);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
      if (total <= kVpList) {
        // entry: piece (11 bits), from (3), upto (4), tile (6)
        uint32_t at = incl - c;
        for (uint32_t q = lo / 8; 8 * q < hi && c; ++q, ++at) {
          const uint32_t from = lo > 8 * q ? lo - 8 * q : 0u, upto = hi - 8 * q < 8u ? hi - 8 * q : 8u;
          list[at] = q | from << 11 | upto << 14 | lane << 18;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t i0 = 0; i0 < total; i0 += kBatch * kWave) {
          uint32_t ent[kBatch];
          Piece x[kBatch];
#pragma unroll
          for (uint32_t u = 0; u < kBatch; ++u) {
            const uint32_t i = i0 + u * kWave + lane;
            ent[u] = i < total ? list[i] : 0u;  // (a listed piece has upto > 0)
          }
#pragma unroll
          for (uint32_t u = 0; u < kBatch; ++u)
            if (ent[u]) load((uint64_t)(tb + (ent[u] >> 18)) * kTile + 8 * (ent[u] & 0x7FFu), x[u]);
#pragma unroll
          for (uint32_t u = 0; u < kBatch; ++u)
            if (ent[u]) put(ent[u] >> 11 & 7u, ent[u] >> 14 & 15u, x[u]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      } else {
        for (uint32_t u = 0; u < kWave && tb + u < t1; ++u) {
          const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)u);
          const uint32_t h = (uint32_t)__builtin_amdgcn_readlane((int)hi, (int)u);
          for (uint32_t q0 = l / 8 + lane; 8 * (q0 - lane) < h; q0 += kBatch * kWave) {
            Piece x[kBatch];
#pragma unroll
            for (uint32_t g = 0; g < kBatch; ++g)
              if (8 * (q0 + g * kWave) < h) load((uint64_t)(tb + u) * kTile + 8 * (q0 + g * kWave), x[g]);
#pragma unroll
            for (uint32_t g = 0; g < kBatch; ++g) {
              const uint32_t e = 8 * (q0 + g * kWave);
              if (e < h) put(l > e ? l - e : 0u, h - e < 8u ? h - e : 8u, x[g]);
            }
          }
        }
      }
    }
    __syncthreads();
  } else {
    constexpr uint32_t kBatch = OP == 0 ? 4 : 2;
    // lanes per run: the pieces of the part's mean run
    const uint32_t pieces = t1 > t0 ? found[3] / np / (t1 - t0) / 8 + 1 : 1;
    uint32_t lpg_log2 = 0;
    while ((1u << lpg_log2) < kThreads && pieces > 1u << lpg_log2) ++lpg_log2;
    const uint32_t lpg = 1u << lpg_log2, groups = kThreads >> lpg_log2, grp = threadIdx.x >> lpg_log2;
    const uint32_t sub = threadIdx.x & (lpg - 1);
    // runs of more pieces than a few rounds of the group are left for whole waves
    auto left = [&](uint32_t lo, uint32_t hi) { return lpg < kWave && (hi + 7) / 8 - lo / 8 > 4 * lpg; };
    struct Runs {
      uint32_t lo[kBatch], hi[kBatch];
    };
    auto load_runs = [&](uint32_t tb, Runs& r) {
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) {
        const uint32_t t = tb + u * groups + grp;
        r.lo[u] = r.hi[u] = 0;
        if (t < t1) {
          const uint32_t* row = runs + (uint64_t)t * (P + 1) + p;
          r.lo[u] = *gp(row);
          r.hi[u] = *gp(row + 1);
        }
      }
    };
    auto load_pieces = [&](uint32_t tb, const Runs& r, Piece (&x)[kBatch]) {
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) {
        const uint32_t e = (r.lo[u] & ~7u) + 8 * sub;
        if (e < r.hi[u]) load((uint64_t)(tb + u * groups + grp) * kTile + e, x[u]);
      }
    };
    auto put_in = [&](uint32_t e, uint32_t lo, uint32_t hi, const Piece& x) {
      put(lo > e ? lo - e : 0u, hi - e < 8u ? hi - e : 8u, x);
    };
    const uint32_t step = kBatch * groups;
    Runs cur, next;
    Piece x[kBatch], y[kBatch];
    load_runs(t0, cur);
    load_runs(t0 + step, next);
    load_pieces(t0, cur, x);
    for (uint32_t tb = t0; tb < t1; tb += step) {
      Runs after;
      load_pieces(tb + step, next, y);
      load_runs(tb + 2 * step, after);
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) {
        const uint32_t e = (cur.lo[u] & ~7u) + 8 * sub;
        if (e < cur.hi[u]) put_in(e, cur.lo[u], cur.hi[u], x[u]);
      }
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) {  // runs longer than the group's pieces
        if (left(cur.lo[u], cur.hi[u])) {
          found[7] = 1;
          continue;
        }
        const uint64_t e0 = (uint64_t)(tb + u * groups + grp) * kTile;
        for (uint32_t e = (cur.lo[u] & ~7u) + 8 * (sub + lpg); e < cur.hi[u]; e += 8 * lpg) {
          Piece z;
          load(e0 + e, z);
          put_in(e, cur.lo[u], cur.hi[u], z);
        }
      }
      cur = next;
      next = after;
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) x[u] = y[u];
    }
    __syncthreads();
    if (found[7]) {
      // The rest of the long runs. (A wave finds them among 64 tiles at a time.)
      for (uint32_t tb = t0 + wv * kWave; tb < t1; tb += kWaves * kWave) {
        uint32_t lo = 0, hi = 0;
        if (tb + lane < t1) {
          const uint32_t* row = runs + (uint64_t)(tb + lane) * (P + 1) + p;
          lo = *gp(row);
          hi = *gp(row + 1);
        }
        for (uint64_t m = __ballot(left(lo, hi)); m; m &= m - 1) {
          const int u = __builtin_ctzll(m);
          const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)lo, u), h = (uint32_t)__builtin_amdgcn_readlane((int)hi, u);
          const uint64_t e0 = (uint64_t)(tb + u) * kTile;
          for (uint32_t e = (l & ~7u) + 8 * (lpg + lane); e - 8 * lane < h; e += 8 * kWave * kBatch) {
            Piece z[kBatch];
#pragma unroll
            for (uint32_t g = 0; g < kBatch; ++g)
              if (e + 8 * kWave * g < h) load(e0 + e + 8 * kWave * g, z[g]);
#pragma unroll
            for (uint32_t g = 0; g < kBatch; ++g)
              if (e + 8 * kWave * g < h) put_in(e + 8 * kWave * g, l, h, z[g]);
          }
        }
      }
      __syncthreads();
    }
  }
  const uint64_t key0 = (uint64_t)p << kb;
  const uint32_t nk = R - key0 < K ? (uint32_t)(R - key0) : K;
  if (np == 1) {
    for (uint32_t i = threadIdx.x; i < nk; i += kThreads) {
      dcnt[key0 + i] = OP == 0 ? val32[i] : here[i];
      if (OP == 1) reinterpret_cast<unsigned long long*>(dval)[key0 + i] = sum64[i];
      if (OP >= 2) reinterpret_cast<uint32_t*>(dval)[key0 + i] = val32[i];
    }
    for (uint32_t q = wv; q * kCompTile < nk; q += kThreads / kWave) {
      const uint32_t i1 = (q + 1) * kCompTile < nk ? (q + 1) * kCompTile : nk;
      uint32_t present = 0;
      for (uint32_t i = q * kCompTile + lane; i - lane < i1; i += kWave)
        present += popc64(__ballot(i < i1 && (OP == 0 ? val32[i] : here[i]) != 0));
      if (lane == 0) blk[key0 / kCompTile + q] = present;
    }
    return;
  }
  if (part == 0)
    for (uint32_t q = threadIdx.x; q * kCompTile < nk; q += kThreads) blk[key0 / kCompTile + q] = kUncounted;
  for (uint32_t i = threadIdx.x; i < nk; i += kThreads) {  // (the dense arrays are zero before)
    const uint32_t c = OP == 0 ? val32[i] : here[i];
    if (!c) continue;
    if (OP == 0) atomicAdd(&dcnt[key0 + i], c);
    else dcnt[key0 + i] = 1u;  // (present)
    if (OP == 1) atomicAdd(&reinterpret_cast<unsigned long long*>(dval)[key0 + i], sum64[i]);
    if (OP >= 2) atomicMax(&reinterpret_cast<uint32_t*>(dval)[key0 + i], val32[i]);
  }
}

// ----------------------------------------------------------------------------
// ordered compaction of dense arrays: keys with count > 0, ascending
// ----------------------------------------------------------------------------
// (counted: by the partitions' fill, all but the blocks it left at kUncounted)
__global__ __launch_bounds__(256) void k_dense_count(const uint32_t* __restrict__ dcnt, uint32_t R, uint32_t* __restrict__ blk,
                                                     bool counted) {
  if (counted && blk[blockIdx.x] != kUncounted) return;
  __shared__ uint32_t s;
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  const uint64_t base = (uint64_t)blockIdx.x * kCompTile;
  uint32_t c = 0;
  for (uint32_t q = threadIdx.x; q < kCompTile; q += blockDim.x) {
    const uint64_t k = base + q;
    if (k < R && dcnt[k]) ++c;
  }
  atomicAdd(&s, c);
  __syncthreads();
  if (threadIdx.x == 0) blk[blockIdx.x] = s;
}

// Exclusive scan of blk[0, nb) in place by one workgroup; total in *total.
__global__ __launch_bounds__(1024) void k_scan_small(uint32_t* __restrict__ blk, uint32_t nb, unsigned long long* total,
                                                     IntEnd E) {
  __shared__ uint32_t ws[1024 / kWave];
  uint32_t carry = 0;
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t base = 0; base < nb; base += blockDim.x) {
    const uint32_t i = base + threadIdx.x;
    const uint32_t x = i < nb ? blk[i] : 0u;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t t = __shfl_up(inc, o);
      if (lane >= (uint32_t)o) inc += t;
    }
    if (lane == kWave - 1) ws[wv] = inc;
    __syncthreads();
    uint32_t pre = carry, tot = 0;
    for (uint32_t q = 0; q < blockDim.x / kWave; ++q) {
      if (q < wv) pre += ws[q];
      tot += ws[q];
    }
    if (i < nb) blk[i] = pre + inc - x;
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0 && total) *total = carry;
  int_publish(E, carry, 0);
}

// Write the present keys of a dense array in order and clear the arrays.
template <int OP>
__global__ __launch_bounds__(256) void k_dense_write(uint32_t* __restrict__ dcnt, void* __restrict__ dval, uint32_t R,
                                                     const uint32_t* __restrict__ blk, uint32_t* __restrict__ out_keys,
                                                     void* __restrict__ out_vals, uint64_t cap, bool clear) {
  __shared__ uint32_t wsum[256 / kWave];
  const uint64_t base = (uint64_t)blockIdx.x * kCompTile;
  uint32_t carry = blk[blockIdx.x];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t q0 = 0; q0 < kCompTile; q0 += blockDim.x) {
    const uint64_t k = base + q0 + threadIdx.x;
    uint32_t c = 0;
    if (k < R) c = dcnt[k];
    const bool p = c != 0;
    const uint64_t m = __ballot(p);
    if (lane == 0) wsum[wv] = popc64(m);
    __syncthreads();
    uint32_t pre = carry, tot = 0;
    for (uint32_t w = 0; w < blockDim.x / kWave; ++w) {
      if (w < wv) pre += wsum[w];
      tot += wsum[w];
    }
    if (p) {
      const uint64_t o = pre + mbcnt(m);
      if (o < cap) {
        out_keys[o] = (uint32_t)k;
        if (OP == 0) reinterpret_cast<uint32_t*>(out_vals)[o] = c;
        if (OP == 1) reinterpret_cast<unsigned long long*>(out_vals)[o] = reinterpret_cast<unsigned long long*>(dval)[k];
        if (OP >= 2) reinterpret_cast<uint32_t*>(out_vals)[o] = dec_minmax(OP, reinterpret_cast<uint32_t*>(dval)[k]);
      }
      if (clear) {
        dcnt[k] = 0;
        if (OP == 1) reinterpret_cast<unsigned long long*>(dval)[k] = 0;
        if (OP >= 2) reinterpret_cast<uint32_t*>(dval)[k] = 0;
      }
    }
    carry += tot;
    __syncthreads();
  }
}

// ----------------------------------------------------------------------------
// hash: LDS cache + global open-addressing table
// ----------------------------------------------------------------------------
constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;  // key 0xFFFFFFFF itself is kept in a side slot

struct IntTable {
  uint32_t* keys;             // [cap], kEmptyKey when free
  uint32_t* cnt;              // [cap]
  void* val;                  // [cap] (64-bit for SUM)
  uint64_t cap;               // power of two
  uint32_t* claimed;          // slots claimed, in claim order
  unsigned long long* n_claimed;
  uint64_t max_probes;        // slots an insert looks at before the table counts as full
  uint64_t max_claims;        // slots claimed before it does
  uint32_t* side_cnt;         // key 0xFFFFFFFF: count and value
  void* side_val;
  uint32_t* flags;
};

template <int OP>
MR_DEV void apply_global(const IntTable& T, uint64_t i, uint32_t c, unsigned long long s, uint32_t mm) {
  atomicAdd(&T.cnt[i], c);
  if (OP == 1) atomicAdd(&reinterpret_cast<unsigned long long*>(T.val)[i], s);
  if (OP >= 2) atomicMax(&reinterpret_cast<uint32_t*>(T.val)[i], mm);
}

template <int OP>
MR_DEV void g_int_insert(const IntTable& T, uint32_t k, uint32_t c, unsigned long long s, uint32_t mm, uint32_t debug_hash) {
  if (k == kEmptyKey) {
    atomicAdd(T.side_cnt, c);
    if (OP == 1) atomicAdd(reinterpret_cast<unsigned long long*>(T.side_val), s);
    if (OP >= 2) atomicMax(reinterpret_cast<uint32_t*>(T.side_val), mm);
    return;
  }
  const uint64_t mask = T.cap - 1;
  uint64_t i = (debug_hash ? 0ull : hash_u32(k)) & mask;
  for (uint64_t p = 0; p < T.max_probes; ++p) {
    uint32_t cur = __hip_atomic_load(&T.keys[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (cur == kEmptyKey) {
      cur = atomicCAS(&T.keys[i], kEmptyKey, k);
      if (cur == kEmptyKey) {
        const uint64_t at = wave_claim(T.n_claimed);
        T.claimed[at] = (uint32_t)i;
        if (at >= T.max_claims) atomicOr(T.flags, kFlagTableFull);
        apply_global<OP>(T, i, c, s, mm);
        return;
      }
    }
    if (cur == k) {
      apply_global<OP>(T, i, c, s, mm);
      return;
    }
    i = (i + 1) & mask;
    if ((p & 255u) == 255u && (__hip_atomic_load(T.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kFlagTableFull)) return;
  }
  atomicOr(T.flags, kFlagTableFull);
}

template <int OP, int L>
__global__ __launch_bounds__(kIntThreads) void k_int_hash(IntIn in, IntTable T, uint32_t G, uint32_t debug_hash, uint64_t R) {
  constexpr uint32_t S = 1u << L;
  __shared__ uint32_t lk[S];
  __shared__ uint32_t lc[S];
  __shared__ unsigned long long ls[OP == 1 ? S : 1];
  __shared__ uint32_t lm[OP >= 2 ? S : 1];
  for (uint32_t i = threadIdx.x; i < S; i += blockDim.x) {
    lk[i] = kEmptyKey;
    lc[i] = 0;
    if (OP == 1) ls[i] = 0;
    if (OP >= 2) lm[i] = 0;
  }
  __syncthreads();
  const uint64_t lo = in.n * blockIdx.x / G, hi = in.n * (blockIdx.x + 1) / G;
  // A full table ends the pass (it is then cleared, and another way taken):
  // the job's flags are read every kLook elements of a thread and looked at
  // when as many more are done.
  constexpr uint32_t kLook = 32;
  uint32_t fl = 0;
  for (uint64_t i0 = lo + threadIdx.x; i0 < hi && !(fl & kFlagTableFull); i0 += (uint64_t)kLook * blockDim.x) {
    fl = __hip_atomic_load(T.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t i1 = hi - i0 < (uint64_t)kLook * blockDim.x ? hi : i0 + (uint64_t)kLook * blockDim.x;
    for (uint64_t i = i0; i < i1; i += blockDim.x) {
      uint32_t k, v;
      load_elem(in, i, k, v);
      if (R && k >= R) atomicOr(T.flags, kFlagBadInput);
      bool done = false;
      if (k != kEmptyKey) {
        uint32_t s = (uint32_t)(debug_hash ? 0ull : hash_u32(k)) & (S - 1);
#pragma unroll 1
        for (int p = 0; p < 16; ++p) {
          uint32_t cur = lk[s];
          if (cur == kEmptyKey) cur = atomicCAS(&lk[s], kEmptyKey, k);
          if (cur == kEmptyKey || cur == k) {
            atomicAdd(&lc[s], 1u);
            if (OP == 1) atomicAdd(&ls[s], (unsigned long long)v);
            if (OP >= 2) atomicMax(&lm[s], enc_minmax(OP, v));
            done = true;
            break;
          }
          s = (s + 1) & (S - 1);
        }
      }
      if (!done) g_int_insert<OP>(T, k, 1u, v, enc_minmax(OP, v), debug_hash);
    }
  }
  __syncthreads();
  if (fl & kFlagTableFull) return;
  for (uint32_t s = threadIdx.x; s < S; s += blockDim.x) {
    if (lk[s] != kEmptyKey && lc[s])
      g_int_insert<OP>(T, lk[s], lc[s], OP == 1 ? ls[s] : 0ull, OP >= 2 ? lm[s] : 0u, debug_hash);
  }
}

// Distinct keys among kSampleSize elements, one from each of as many equal
// stretches of the input at a place that varies from stretch to stretch (keys
// that recur with the stretches are met like others), counted in an LDS hash
// set by one workgroup; and an estimate of the distinct keys of the whole
// input from the keys met once (f1) and twice (f2), the lower bound of Chao:
// d + f1 (f1 - 1) / (2 (f2 + 1)). They tell inputs of few keys, which the LDS
// caches combine, from the others before any pass over them. Bound by the
// latency of one load per element on one workgroup: 22 us on 16 M elements.
constexpr uint32_t kSampleSize = 8192;

__global__ __launch_bounds__(1024) void k_int_sample(IntIn in, IntPub* host) {
  constexpr uint32_t S = 2 * kSampleSize;
  __shared__ __attribute__((aligned(16))) uint32_t set[S], met[S];
  __shared__ uint32_t n[3];  // keys met, met once, met twice
  for (uint32_t i = threadIdx.x * 4; i < S; i += blockDim.x * 4) {
    *reinterpret_cast<uint4*>(&set[i]) = make_uint4(kEmptyKey, kEmptyKey, kEmptyKey, kEmptyKey);
    *reinterpret_cast<uint4*>(&met[i]) = make_uint4(0, 0, 0, 0);
  }
  if (threadIdx.x < 3) n[threadIdx.x] = 0;
  constexpr uint32_t kPer = kSampleSize / 1024;
  const uint32_t stretch = (uint32_t)(in.n / kSampleSize);  // (at least 1)
  uint32_t k[kPer];
#pragma unroll
  for (uint32_t u = 0; u < kPer; ++u) {
    const uint64_t q = u * 1024 + threadIdx.x;
    k[u] = in.p[(q * in.n / kSampleSize + __umulhi((uint32_t)fmix64(q + 1), stretch)) * in.stride];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kPer; ++u) {
    if (k[u] == kEmptyKey) continue;
    uint32_t s = (uint32_t)hash_u32(k[u]) & (S - 1);
    // (reads first: atomics on a frequent key's slot queue)
    for (;;) {  // (the set has twice the slots: a free one is met)
      uint32_t cur = __hip_atomic_load(&set[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (cur == kEmptyKey) cur = atomicCAS(&set[s], kEmptyKey, k[u]);
      if (cur == kEmptyKey || cur == k[u]) break;
      s = (s + 1) & (S - 1);
    }
    if (__hip_atomic_load(&met[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < 3) atomicAdd(&met[s], 1u);
  }
  __syncthreads();
  // (the counts below 2^16 of a wave's 1024 slots in the halves of one sum)
  uint32_t all = 0, few = 0;
  for (uint32_t i = threadIdx.x * 4; i < S; i += blockDim.x * 4) {
    const uint4 m = *reinterpret_cast<const uint4*>(&met[i]);
    all += (m.x != 0) + (m.y != 0) + (m.z != 0) + (m.w != 0);
    few += (m.x == 1) + (m.y == 1) + (m.z == 1) + (m.w == 1);
    few += (uint32_t)((m.x == 2) + (m.y == 2) + (m.z == 2) + (m.w == 2)) << 16;
  }
  all = wave_incl_scan(all);
  few = wave_incl_scan(few);
  if (lane_id() == kWave - 1) {
    atomicAdd(&n[0], all);
    atomicAdd(&n[1], few & 0xFFFFu);
    atomicAdd(&n[2], few >> 16);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t f1 = n[1];
    __hip_atomic_store(&host->sampled, n[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host->estimate, n[0] + (f1 ? f1 * (f1 - 1) / (2 * (n[2] + 1)) : 0u), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Output of a table of few keys by one workgroup: the claimed slots' keys are
// sorted in LDS (bitonic, with their claim index), the pairs written in order
// and the slots cleared, the side slot appended. Does nothing when there are
// more than kSmallOut keys or the table was full. One launch instead of the
// gather, the radix passes and the split (16 launches, about 80 us).
constexpr uint32_t kSmallOut = 4096;

template <int OP>
__global__ __launch_bounds__(1024) void k_int_small_out(IntTable T, uint32_t* __restrict__ out_keys, void* __restrict__ out_vals,
                                                        uint64_t cap, unsigned long long* __restrict__ n_out, IntEnd E) {
  __shared__ unsigned long long e[kSmallOut];
  const unsigned long long nc = *T.n_claimed;
  if (nc > kSmallOut || (*T.flags & kFlagTableFull)) {
    int_publish(E, 0, nc);
    return;
  }
  const uint32_t n = (uint32_t)nc;
  uint32_t m = 1;
  while (m < n) m *= 2;
  for (uint32_t q = threadIdx.x; q < m; q += blockDim.x)
    e[q] = q < n ? (unsigned long long)T.keys[T.claimed[q]] << 32 | q : ~0ull;  // (claim indices are below 2^32 - 1)
  __syncthreads();
  for (uint32_t size = 2; size <= m; size *= 2) {
    for (uint32_t step = size / 2; step; step /= 2) {
      for (uint32_t q = threadIdx.x; q < m / 2; q += blockDim.x) {
        const uint32_t a = 2 * q - (q & (step - 1)), b = a + step;
        const unsigned long long x = e[a], y = e[b];
        if ((x > y) == ((a & size) == 0)) {
          e[a] = y;
          e[b] = x;
        }
      }
      __syncthreads();
    }
  }
  for (uint32_t r = threadIdx.x; r < n; r += blockDim.x) {
    const uint32_t i = T.claimed[(uint32_t)e[r]];
    if (r < cap) {
      out_keys[r] = (uint32_t)(e[r] >> 32);
      if (OP == 0) reinterpret_cast<uint32_t*>(out_vals)[r] = T.cnt[i];
      else if (OP == 1) reinterpret_cast<unsigned long long*>(out_vals)[r] = reinterpret_cast<unsigned long long*>(T.val)[i];
      else reinterpret_cast<uint32_t*>(out_vals)[r] = dec_minmax(OP, reinterpret_cast<uint32_t*>(T.val)[i]);
    }
    T.keys[i] = kEmptyKey;
    T.cnt[i] = 0;
    if (OP == 1) reinterpret_cast<unsigned long long*>(T.val)[i] = 0;
    if (OP >= 2) reinterpret_cast<uint32_t*>(T.val)[i] = 0;
  }
  if (threadIdx.x == 0) {
    const bool side = *T.side_cnt != 0;  // key 0xFFFFFFFF, after all others
    if (side && n < cap) {
      out_keys[n] = kEmptyKey;
      if (OP == 0) reinterpret_cast<uint32_t*>(out_vals)[n] = *T.side_cnt;
      else if (OP == 1) reinterpret_cast<unsigned long long*>(out_vals)[n] = *reinterpret_cast<unsigned long long*>(T.side_val);
      else reinterpret_cast<uint32_t*>(out_vals)[n] = dec_minmax(OP, *reinterpret_cast<uint32_t*>(T.side_val));
    }
    *n_out = n + (side ? 1u : 0u);
  }
  int_publish(E, n + (*T.side_cnt != 0 ? 1u : 0u), nc);
}

// Claimed slots -> (key, claim index) pairs and values; slots are cleared for reuse.
template <int OP>
__global__ __launch_bounds__(256) void k_int_gather(IntTable T, uint2* __restrict__ rk, unsigned long long* __restrict__ rv) {
  const uint64_t n = *T.n_claimed;
  for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < n; q += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t i = T.claimed[q];
    rk[q] = make_uint2(T.keys[i], (uint32_t)q);
    unsigned long long v;
    if (OP == 0) v = T.cnt[i];
    else if (OP == 1) v = reinterpret_cast<unsigned long long*>(T.val)[i];
    else v = dec_minmax(OP, reinterpret_cast<uint32_t*>(T.val)[i]);
    rv[q] = v;
    T.keys[i] = kEmptyKey;
    T.cnt[i] = 0;
    if (OP == 1) reinterpret_cast<unsigned long long*>(T.val)[i] = 0;
    if (OP >= 2) reinterpret_cast<uint32_t*>(T.val)[i] = 0;
  }
}

// ----------------------------------------------------------------------------
// scans
// ----------------------------------------------------------------------------

// Device-wide exclusive scan of a (in place): per-block sums, scan of sums, add back.
constexpr uint32_t kScanTile = 4096;

// The tile's entries of this thread, 16 in a row, all in flight at once (one
// after the other, with a barrier each: 8.1 and 12.9 us for 308,000 entries,
// now 2.7 and 3.2).
constexpr uint32_t kScanThreads = 256, kScanPer = kScanTile / kScanThreads;
MR_DEV void scan_load(const uint32_t* __restrict__ a, uint64_t n, uint64_t at, uint32_t (&x)[kScanPer]) {
  if (at + kScanPer <= n && ((uintptr_t)a & 15u) == 0) {
#pragma unroll
    for (uint32_t q = 0; q < kScanPer; q += 4) {
      const uint4 v = gload16(a + at + q);
      x[q] = v.x;
      x[q + 1] = v.y;
      x[q + 2] = v.z;
      x[q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (uint32_t q = 0; q < kScanPer; ++q) x[q] = at + q < n ? gp(a)[at + q] : 0u;
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_blocks(const uint32_t* __restrict__ a, uint64_t n,
                                                              uint32_t* __restrict__ sums) {
  __shared__ uint32_t ws[kScanThreads / kWave];
  uint32_t x[kScanPer], c = 0;
  scan_load(a, n, (uint64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer, x);
#pragma unroll
  for (uint32_t q = 0; q < kScanPer; ++q) c += x[q];
  const uint32_t incl = wave_incl_scan(c);
  if (lane_id() == kWave - 1) ws[threadIdx.x / kWave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (uint32_t w = 0; w < kScanThreads / kWave; ++w) s += ws[w];
    sums[blockIdx.x] = s;
  }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(uint32_t* __restrict__ a, uint64_t n, const uint32_t* __restrict__ sums) {
  __shared__ uint32_t ws[kScanThreads / kWave];
  const uint64_t at = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * kScanPer;
  uint32_t run = sums[blockIdx.x], x[kScanPer], c = 0;
  scan_load(a, n, at, x);
#pragma unroll
  for (uint32_t q = 0; q < kScanPer; ++q) c += x[q];
  const uint32_t incl = wave_incl_scan(c), wv = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) ws[wv] = incl;
  __syncthreads();
  for (uint32_t w = 0; w < wv; ++w) run += ws[w];
  run += incl - c;
#pragma unroll
  for (uint32_t q = 0; q < kScanPer; ++q) {
    const uint32_t y = x[q];
    x[q] = run;
    run += y;
  }
  if (at + kScanPer <= n && ((uintptr_t)a & 15u) == 0) {
#pragma unroll
    for (uint32_t q = 0; q < kScanPer; q += 4) gstore16(a + at + q, make_uint4(x[q], x[q + 1], x[q + 2], x[q + 3]));
  } else {
#pragma unroll
    for (uint32_t q = 0; q < kScanPer; ++q)
      if (at + q < n) gp(a)[at + q] = x[q];
  }
}

// Append the side slot (key 0xFFFFFFFF) after the sorted keys when present.
__global__ void k_side_append(const uint32_t* side_cnt, const void* side_val, int op, const unsigned long long* n_claimed,
                              unsigned long long* n_total, uint32_t* out_keys, void* out_vals, uint64_t cap) {
  if (threadIdx.x || blockIdx.x) return;
  uint64_t n = *n_claimed;
  if (*side_cnt) {
    if (n < cap) {
      out_keys[n] = kEmptyKey;
      if (op == 0) reinterpret_cast<uint32_t*>(out_vals)[n] = *side_cnt;
      else if (op == 1) reinterpret_cast<unsigned long long*>(out_vals)[n] = *reinterpret_cast<const unsigned long long*>(side_val);
      else reinterpret_cast<uint32_t*>(out_vals)[n] = dec_minmax(op, *reinterpret_cast<const uint32_t*>(side_val));
    }
    ++n;
  }
  *n_total = n;
}

// ----------------------------------------------------------------------------
// host launchers
// ----------------------------------------------------------------------------

static uint32_t blocks_for(uint64_t n, uint32_t per, uint32_t cap_blocks) {
  const uint64_t b = (n + per - 1) / per;
  return (uint32_t)(b == 0 ? 1 : (b < cap_blocks ? b : cap_blocks));
}

uint32_t int_lds_array_bytes(uint64_t R, uint32_t op) {
  const uint64_t b = 4ull * R + (op == 1 ? 8ull * R + 8 : (op >= 2 ? 4ull * R : 0));
  return (uint32_t)(b < 0xFFFFFFFFull ? b : 0xFFFFFFFFull);
}

// Copies of the LDS array per workgroup: as many as kLdsCopiesBytes hold, at most 32.
static uint32_t lds_copies(uint32_t R, uint32_t op) {
  uint32_t c = 1;
  while (c < 32 && 2 * c * lds_copy_words(R, op, 2 * c) * 4 <= kLdsCopiesBytes) c *= 2;
  return c;
}

// Partial rows the output kernel adds itself: up to 32 rows and kLdsDirect
// values; more are added by the reduce kernel first (its launch costs 5 us, a
// row read by one workgroup about 0.1 us).
constexpr uint64_t kLdsDirect = 64 * 1024;

bool int_lds_direct(uint64_t R, uint32_t G) { return G <= 32 && R * G <= kLdsDirect; }

template <int OP>
static hipError_t lds_enqueue(const IntLaunch& L, hipStream_t s) {
  const uint32_t R = (uint32_t)L.R;
  const uint32_t copies = lds_copies(R, OP);
  hipLaunchKernelGGL(k_lds_array<OP>, dim3(L.G), dim3(kIntThreads), copies * lds_copy_words(R, OP, copies) * 4, s, int_in(L), R, L.G, copies,
                     L.cnt_part, L.val_part, L.flags);
  const uint32_t* cnt = L.cnt_part;
  const void* val = L.val_part;
  uint32_t G = L.G;
  if (!int_lds_direct(L.R, L.G)) {
    hipLaunchKernelGGL(k_lds_array_reduce<OP>, dim3((R + kWave - 1) / kWave), dim3(kLdsReduceWaves * kWave), 0, s, R, L.G,
                       L.cnt_part, L.val_part, L.dcnt, L.dval);
    cnt = L.dcnt;
    val = L.dval;
    G = 1;
  }
  // (an LDS array holds at most 16,384 counts, 8,192 counts with extrema or 5,461 with sums)
  constexpr uint32_t kMost = OP == 0 ? 16 : 8;
  if (R <= 1024) {
    hipLaunchKernelGGL((k_lds_out<OP, 1>), dim3(1), dim3(1024), 0, s, R, G, cnt, val, L.out_keys, L.out_vals, L.cap, L.n_out,
                       L.end);
  } else if (R <= 4096) {
    hipLaunchKernelGGL((k_lds_out<OP, 4>), dim3(1), dim3(1024), 0, s, R, G, cnt, val, L.out_keys, L.out_vals, L.cap, L.n_out,
                       L.end);
  } else {
    hipLaunchKernelGGL((k_lds_out<OP, kMost>), dim3(1), dim3(1024), 0, s, R, G, cnt, val, L.out_keys, L.out_vals, L.cap,
                       L.n_out, L.end);
  }
  return hipGetLastError();
}

// Map, reduce and ordered output.
hipError_t int_enqueue_lds_array(const IntLaunch& L, hipStream_t s) {
  switch (L.op) {
    case 0: return lds_enqueue<0>(L, s);
    case 1: return lds_enqueue<1>(L, s);
    case 2: return lds_enqueue<2>(L, s);
    default: return lds_enqueue<3>(L, s);
  }
}

hipError_t int_enqueue_global_array(const IntLaunch& L, hipStream_t s) {
  const IntIn in = int_in(L);
  const uint32_t g = blocks_for(L.n, 256, 8192);
  switch (L.op) {
    case 0: hipLaunchKernelGGL(k_global_array<0>, dim3(g), dim3(256), 0, s, in, L.R, L.dcnt, L.dval, L.flags); break;
    case 1: hipLaunchKernelGGL(k_global_array<1>, dim3(g), dim3(256), 0, s, in, L.R, L.dcnt, L.dval, L.flags); break;
    case 2: hipLaunchKernelGGL(k_global_array<2>, dim3(g), dim3(256), 0, s, in, L.R, L.dcnt, L.dval, L.flags); break;
    case 3: hipLaunchKernelGGL(k_global_array<3>, dim3(g), dim3(256), 0, s, in, L.R, L.dcnt, L.dval, L.flags); break;
  }
  return hipGetLastError();
}

// Exclusive scan of a[0, n) in place by one workgroup, for n up to
// kScanOneMax: wave w takes a contiguous segment of whole 64-element steps.
// Each wave sums its segment (coalesced loads), the 16 wave totals are
// scanned in LDS, then each wave reads its segment again (from the cache)
// and scans it kScanOneBatch steps at a time with DPP lane shifts (the
// batch's scans are independent, so they overlap), adding a running carry.
// One launch instead of the block sums, their scan and the apply.
constexpr uint32_t kScanOneWaves = 16;
constexpr uint32_t kScanOneSteps = 64;  // 64-element steps per wave at most
constexpr uint32_t kScanOneBatch = 8;   // steps loaded and scanned together
constexpr uint64_t kScanOneMax = (uint64_t)kScanOneWaves * kWave * kScanOneSteps;

__global__ __launch_bounds__(kScanOneWaves * kWave) void k_scan_one(uint32_t* __restrict__ a, uint32_t n,
                                                                   unsigned long long* total, IntEnd E) {
  __shared__ uint32_t ws[kScanOneWaves];
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  const uint32_t steps = (n + kScanOneWaves * kWave - 1) / (kScanOneWaves * kWave);  // <= kScanOneSteps
  const uint32_t b0 = wv * steps * kWave;
  auto at = [&](uint32_t q) { return b0 + q * kWave + lane; };
  uint32_t part = 0;
  for (uint32_t q0 = 0; q0 < steps; q0 += kScanOneBatch) {
    uint32_t v[kScanOneBatch];
#pragma unroll
    for (uint32_t u = 0; u < kScanOneBatch; ++u) v[u] = (q0 + u < steps && at(q0 + u) < n) ? a[at(q0 + u)] : 0u;
#pragma unroll
    for (uint32_t u = 0; u < kScanOneBatch; ++u) part += v[u];
  }
  const uint32_t wsum = wave_incl_scan(part);  // every lane takes part in the lane shifts
  if (lane == kWave - 1) ws[wv] = wsum;
  __syncthreads();
  uint32_t carry = 0, all = 0;
  for (uint32_t w = 0; w < kScanOneWaves; ++w) {
    if (w < wv) carry += ws[w];
    all += ws[w];
  }
  for (uint32_t q0 = 0; q0 < steps; q0 += kScanOneBatch) {
    uint32_t v[kScanOneBatch];
#pragma unroll
    for (uint32_t u = 0; u < kScanOneBatch; ++u) v[u] = (q0 + u < steps && at(q0 + u) < n) ? a[at(q0 + u)] : 0u;
#pragma unroll
    for (uint32_t u = 0; u < kScanOneBatch; ++u) v[u] = wave_incl_scan(v[u]);
#pragma unroll
    for (uint32_t u = 0; u < kScanOneBatch; ++u) {
      const uint32_t ex = from_prev_lane(v[u], 0u);  // exclusive within the step
      if (q0 + u < steps && at(q0 + u) < n) a[at(q0 + u)] = carry + ex;
      carry += (uint32_t)__builtin_amdgcn_readlane((int)v[u], kWave - 1);
    }
  }
  if (threadIdx.x == 0 && total) *total = all;
  int_publish(E, all, 0);
}

// Exclusive scan of a[0, n) in place; the sum of all entries into *total.
hipError_t scan_exclusive_u32(uint32_t* a, uint64_t n, uint32_t* sums, unsigned long long* total, hipStream_t s,
                              const IntEnd& E) {
  if (n <= kScanOneMax) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneWaves * kWave), 0, s, a, (uint32_t)n, total, E);
    return hipGetLastError();
  }
  const uint32_t sb = (uint32_t)((n + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_scan_blocks, dim3(sb ? sb : 1), dim3(kScanThreads), 0, s, a, n, sums);
  hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, s, sums, sb ? sb : 1, total, E);
  hipLaunchKernelGGL(k_scan_apply, dim3(sb ? sb : 1), dim3(kScanThreads), 0, s, a, n, sums);
  return hipGetLastError();
}

uint64_t scan_sums_count(uint64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

// Layout of the partitions: ranges of 2^12 keys up to 512 of them (a SUM
// range's arrays leave room for four workgroups per CU), then the smallest
// that keeps the ranges at 512 (COUNT, up to 2^15 keys in 128 KB of LDS) or
// 2048 (values, up to 2^14 keys), so that a tile's run of a range stays long.
VpPlan vp_plan(uint64_t n, uint64_t R, uint32_t op, uint32_t n_cu) {
  VpPlan p{};
  const uint32_t kb_max = vp_max_kb(op);
  p.kb = 12;
  while (p.kb < kb_max && R > (uint64_t)512 << p.kb && (op == 0 || p.kb == 12 || R > (uint64_t)kVpMaxParts << p.kb)) ++p.kb;
  p.P = (uint32_t)((R + (1ull << p.kb) - 1) >> p.kb);
  const uint64_t tile = vp_tile(op);
  p.n_tiles = (uint32_t)((n + tile - 1) / tile);
  p.elems = (uint64_t)p.n_tiles * tile;
  p.runs = (uint64_t)p.n_tiles * (p.P + 1);
  // two workgroups per CU over all ranges; a merged range touches its 2^kb
  // keys, so twice as many elements at least; and ranges of even shares
  // (within an eighth) are not split where there are enough of them
  uint64_t split = std::max<uint64_t>(n / (2 * n_cu), 2ull << p.kb);
  if (p.P >= 2 * n_cu) split = std::max<uint64_t>(split, n / p.P + n / p.P / 8 + 1024);
  p.split = (uint32_t)std::min<uint64_t>(split, 1u << 30);
  p.grid = (uint32_t)(p.P + n / p.split);
  const uint64_t pieces = n / ((uint64_t)p.P * p.n_tiles + 1) / 8 + 1;  // 16-byte pieces of a run
  p.list = op == 0 && p.n_tiles >= 8192 && pieces <= 5;
  p.slices = std::max(1u, std::min(kVpMaxSlices, p.n_tiles / 128));
  p.usable = p.P <= kVpMaxParts && n >= kVpMin && n < (1ull << 32) && (op == 0 || R < kVpSparse * n);
  return p;
}

template <int OP, bool kList>
static hipError_t vp_enqueue_fill(const IntLaunch& L, const VpPlan& p, const uint32_t* runs, const uint16_t* pk,
                                  const uint32_t* pv, const uint32_t* tot, hipStream_t s) {
  const uint32_t lds = vp_fill_lds(OP, p.kb);
  if (lds > 32 * 1024) {  // (with the static LDS past 64 KB; the most any range takes: calls on other threads set the same)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_vp_fill<OP, kList>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)vp_fill_lds(OP, vp_max_kb(OP)));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_vp_fill<OP, kList>), dim3(p.grid), dim3(vp_fill_threads(OP)), lds, s, L.R, p.kb, p.P, p.n_tiles,
                     p.split, runs, pk, pv, tot, p.slices, L.dcnt, L.dval, L.blk);
  return hipGetLastError();
}

template <int OP>
static hipError_t vp_enqueue(const IntLaunch& L, const VpPlan& p, uint32_t* runs, uint16_t* pk, uint32_t* pv, uint32_t* tot,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_vp_tile<OP>, dim3(p.n_tiles), dim3(vp_threads(OP)), (p.P + 1) * 4, s, int_in(L), L.R, p.kb,
                     p.P, runs, pk, pv, L.flags);
  hipLaunchKernelGGL(k_vp_totals, dim3((p.P + kWave - 1) / kWave, p.slices), dim3(kVpTotThreads), 0, s, runs, p.P, p.n_tiles,
                     tot);
  if constexpr (OP == 0)
    if (p.list) return vp_enqueue_fill<0, true>(L, p, runs, pk, pv, tot, s);
  return vp_enqueue_fill<OP, false>(L, p, runs, pk, pv, tot, s);
}

hipError_t int_enqueue_global_array_vp(const IntLaunch& L, const VpPlan& p, uint32_t* runs, uint16_t* pk, uint32_t* pv,
                                       uint32_t* tot, hipStream_t s) {
  switch (L.op) {
    case 0: return vp_enqueue<0>(L, p, runs, pk, pv, tot, s);
    case 1: return vp_enqueue<1>(L, p, runs, pk, pv, tot, s);
    case 2: return vp_enqueue<2>(L, p, runs, pk, pv, tot, s);
    default: return vp_enqueue<3>(L, p, runs, pk, pv, tot, s);
  }
}

// Compaction of the dense arrays into the outputs; clears them when asked.
// by_parts: partitions filled them.
hipError_t int_enqueue_dense_out(const IntLaunch& L, bool clear, bool by_parts, hipStream_t s) {
  const uint32_t nb = (uint32_t)((L.R + kCompTile - 1) / kCompTile);
  hipLaunchKernelGGL(k_dense_count, dim3(nb ? nb : 1), dim3(256), 0, s, L.dcnt, L.R, L.blk, by_parts);
  if (nb <= kScanOneMax) hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneWaves * kWave), 0, s, L.blk, nb, L.n_out, L.end);
  else hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, s, L.blk, nb, L.n_out, L.end);
  switch (L.op) {
    case 0: hipLaunchKernelGGL(k_dense_write<0>, dim3(nb ? nb : 1), dim3(256), 0, s, L.dcnt, L.dval, L.R, L.blk, L.out_keys, L.out_vals, L.cap, clear); break;
    case 1: hipLaunchKernelGGL(k_dense_write<1>, dim3(nb ? nb : 1), dim3(256), 0, s, L.dcnt, L.dval, L.R, L.blk, L.out_keys, L.out_vals, L.cap, clear); break;
    case 2: hipLaunchKernelGGL(k_dense_write<2>, dim3(nb ? nb : 1), dim3(256), 0, s, L.dcnt, L.dval, L.R, L.blk, L.out_keys, L.out_vals, L.cap, clear); break;
    case 3: hipLaunchKernelGGL(k_dense_write<3>, dim3(nb ? nb : 1), dim3(256), 0, s, L.dcnt, L.dval, L.R, L.blk, L.out_keys, L.out_vals, L.cap, clear); break;
  }
  return hipGetLastError();
}

hipError_t int_enqueue_hash_map(const IntLaunch& L, hipStream_t s) {
  const IntIn in = int_in(L);
  IntTable T{L.t_keys, L.t_cnt, L.t_val, L.t_cap, L.claimed, L.n_claimed, L.max_probes, L.max_claims, L.side_cnt, L.side_val, L.flags};
#define HASH_CASE(OP) \
  case OP: hipLaunchKernelGGL((k_int_hash<OP, 12>), dim3(L.G), dim3(kIntThreads), 0, s, in, T, L.G, L.debug_hash, L.R); break;
  switch (L.op) {
    HASH_CASE(0)
    HASH_CASE(1)
    HASH_CASE(2)
    HASH_CASE(3)
  }
#undef HASH_CASE
  return hipGetLastError();
}

hipError_t int_enqueue_sample(const IntLaunch& L, IntPub* host, hipStream_t s) {
  hipLaunchKernelGGL(k_int_sample, dim3(1), dim3(1024), 0, s, int_in(L), host);
  return hipGetLastError();
}

uint32_t int_small_out_max() { return kSmallOut; }

hipError_t int_enqueue_small_out(const IntLaunch& L, hipStream_t s) {
  IntTable T{L.t_keys, L.t_cnt, L.t_val, L.t_cap, L.claimed, L.n_claimed, L.max_probes, L.max_claims, L.side_cnt, L.side_val, L.flags};
  switch (L.op) {
    case 0: hipLaunchKernelGGL(k_int_small_out<0>, dim3(1), dim3(1024), 0, s, T, L.out_keys, L.out_vals, L.cap, L.n_out, L.end); break;
    case 1: hipLaunchKernelGGL(k_int_small_out<1>, dim3(1), dim3(1024), 0, s, T, L.out_keys, L.out_vals, L.cap, L.n_out, L.end); break;
    case 2: hipLaunchKernelGGL(k_int_small_out<2>, dim3(1), dim3(1024), 0, s, T, L.out_keys, L.out_vals, L.cap, L.n_out, L.end); break;
    case 3: hipLaunchKernelGGL(k_int_small_out<3>, dim3(1), dim3(1024), 0, s, T, L.out_keys, L.out_vals, L.cap, L.n_out, L.end); break;
  }
  return hipGetLastError();
}

hipError_t int_enqueue_hash_out(const IntLaunch& L, uint64_t n_claimed_host, hipStream_t s) {
  IntTable T{L.t_keys, L.t_cnt, L.t_val, L.t_cap, L.claimed, L.n_claimed, L.max_probes, L.max_claims, L.side_cnt, L.side_val, L.flags};
  const uint64_t n = n_claimed_host;
  const uint32_t g = blocks_for(n, 256, 4096);
  switch (L.op) {
    case 0: hipLaunchKernelGGL(k_int_gather<0>, dim3(g), dim3(256), 0, s, T, static_cast<uint2*>(L.pairs), L.vals); break;
    case 1: hipLaunchKernelGGL(k_int_gather<1>, dim3(g), dim3(256), 0, s, T, static_cast<uint2*>(L.pairs), L.vals); break;
    case 2: hipLaunchKernelGGL(k_int_gather<2>, dim3(g), dim3(256), 0, s, T, static_cast<uint2*>(L.pairs), L.vals); break;
    case 3: hipLaunchKernelGGL(k_int_gather<3>, dim3(g), dim3(256), 0, s, T, static_cast<uint2*>(L.pairs), L.vals); break;
  }
  return hipGetLastError();
}

hipError_t int_enqueue_side_append(const IntLaunch& L, hipStream_t s) {
  hipLaunchKernelGGL(k_side_append, dim3(1), dim3(64), 0, s, L.side_cnt, L.side_val, (int)L.op, L.n_claimed, L.n_out,
                     L.out_keys, L.out_vals, L.cap);
  return hipGetLastError();
}

}  // namespace mr
