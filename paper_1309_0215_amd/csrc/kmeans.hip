// One k-means (Lloyd) step on gfx950: map = nearest centroid, reduce = per-
// cluster sum and count (array container over the k clusters).
//
// Assignment (d = 32, k = 64): the scores s_j = |c_j|^2 - 2 <x, c_j> come from
// a contraction on the matrix cores. Points and centroids are split exactly
// into three bfloat16 pieces each (x = xh + xm + xl); the six largest of the
// nine piece products (all but xm.cl, xl.cm, xl.cl, which together stay below
// 2^-20 |x| |c|) are accumulated in float32 by v_mfma_f32_32x32x16_bf16:
// A = 32 centroids x 16 dims, B = 16 dims x 32 points, two steps cover
// d = 32, two centroid blocks cover k = 64. Each lane ends with one point's
// scores for 32 centroids; lanes l and l ^ 32 hold the other 32. The argmin
// takes the lowest index on equal scores. When the float32 gap between the
// best and the second best score is within a rounding bound eps(x) (which
// covers the dropped products), the decision is made again in float64 from
// the direct form sum_t (x_t - c_t)^2.
//
// Update: the per-cluster sums are a second contraction on the matrix cores
// (one-hot assignment x points). Each float32 coordinate is split exactly into
// three bfloat16 pieces (x = hi + mid + lo), so the one-hot products are
// exact and the contraction runs on the bfloat16 unit
// (v_mfma_f32_32x32x16_bf16) with float32 accumulation, as the float32
// contraction did. The float32 sums stay in the accumulators for at most 16
// groups of 32 points per wave and are then added into float64 LDS sums; the
// per-workgroup float64 partials are added in a fixed order at the end.
//
// Any other d and k (and points not 16-byte aligned): float32 matrix-core scores
// with the same float64 re-check (k_km_assign), then the sums in a second kernel
// (k_km_update).
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace mr {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

MR_DEV __bf16 bf16_bits(uint32_t hi16) { return __builtin_bit_cast(__bf16, (unsigned short)hi16); }

// x = hi + mid + lo exactly (finite x above the float32 subnormal range):
// hi keeps the top 8 significant bits, mid the next 8 of the remainder, and
// the last remainder has at most 8 significant bits left.
MR_DEV void split_bf16x3(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
  const uint32_t u0 = __float_as_uint(x);
  const float r1 = x - __uint_as_float(u0 & 0xFFFF0000u);
  const uint32_t u1 = __float_as_uint(r1);
  const float r2 = r1 - __uint_as_float(u1 & 0xFFFF0000u);
  hi = bf16_bits(u0 >> 16);
  mid = bf16_bits(u1 >> 16);
  lo = bf16_bits(__float_as_uint(r2) >> 16);
}

constexpr int kKmThreads = 768;  // 12 waves

// Nonzero float32 magnitudes below 2^-100 (bit patterns 1 .. kTinyBits - 1):
// their bfloat16 pieces can fall below the normal range, where the split
// into pieces is no longer exact, so the matrix-core path is not used.
constexpr uint32_t kTinyBits = 0x0D800000u;  // 2^-100

// Squared norms of the centroids (rounded to float32) and max |c| (float64);
// *tiny is set when a centroid has a nonzero coordinate below 2^-100.
// (d = 32, k = 64: one lane per centroid, all of its coordinates in flight at
// once; a thread's coordinate after the other in four times the threads, and
// a clearing of the two counts before it, took 13 us and 6 us)
__global__ __launch_bounds__(kWave) void k_km_prep(const float* __restrict__ C, float* __restrict__ cn, double* __restrict__ cmax,
                                                   unsigned long long* __restrict__ n_recheck, unsigned long long* __restrict__ tiny) {
  const uint32_t j = threadIdx.x;
  uint4 x[8];
#pragma unroll
  for (uint32_t q = 0; q < 8; ++q) x[q] = gload16(C + j * 32 + 4 * q);
  double s = 0.0;
  bool small = false;
#pragma unroll
  for (uint32_t q = 0; q < 8; ++q) {
    const uint32_t w[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
      const uint32_t b = w[t] & 0x7FFFFFFFu;
      small |= b != 0u && b < kTinyBits;
      const double v = __uint_as_float(w[t]);
      s += v * v;
    }
  }
  cn[j] = (float)s;
  double best = s > 0.0 ? s : 0.0;  // (no NaN)
#pragma unroll
  for (int o = kWave / 2; o; o >>= 1) {
    const double y = __shfl_xor(best, o);
    best = y > best ? y : best;
  }
  const bool any = __ballot(small) != 0ull;
  if (j == 0) {
    *cmax = sqrt(best);
    *n_recheck = 0ull;
    *tiny = any ? 1ull : 0ull;
  }
}

// Assignment + local sums for d = 32, k = 64.
constexpr int kKmFlushIters = 16;  // wave iterations between float32 -> float64 flushes of the sums

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

MR_DEV void load_group(const float* __restrict__ X, uint64_t N, uint64_t g, uint64_t groups, uint32_t col, uint32_t h,
                       float (&xs)[16]) {
  const uint64_t p = g * 32 + col;
  if (g < groups && p < N) {
    // dims 8h..8h+7 (xs[0..7]) and 16+8h..16+8h+7 (xs[8..15])
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4* src = reinterpret_cast<const f32x4*>(X + p * 32 + 16 * (q / 2) + 8 * h + 4 * (q % 2));
      const f32x4 v = __builtin_nontemporal_load(src);
      xs[4 * q + 0] = v.x;
      xs[4 * q + 1] = v.y;
      xs[4 * q + 2] = v.z;
      xs[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int s = 0; s < 16; ++s) xs[s] = 0.f;
  }
}

// Eight consecutive values as their three pieces (split_bf16x3), packed in pairs.
MR_DEV void split8_bf16x3(const float* x, uint4& hi, uint4& mid, uint4& lo) {
  uint32_t* const ph = &hi.x;
  uint32_t* const pm = &mid.x;
  uint32_t* const pl = &lo.x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t u0[2], u1[2], u2[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float v = x[2 * j + e];
      u0[e] = __float_as_uint(v);
      const float r1 = v - __uint_as_float(u0[e] & 0xFFFF0000u);
      u1[e] = __float_as_uint(r1);
      u2[e] = __float_as_uint(r1 - __uint_as_float(u1[e] & 0xFFFF0000u));
    }
    ph[j] = __builtin_amdgcn_perm(u0[1], u0[0], 0x07060302u);  // the upper halves
    pm[j] = __builtin_amdgcn_perm(u1[1], u1[0], 0x07060302u);
    pl[j] = __builtin_amdgcn_perm(u2[1], u2[0], 0x07060302u);
  }
}

MR_DEV bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// The larger of two float32 values (plain fmaxf first quiets each operand that
// it cannot show to be quiet). A quiet NaN gives the other value; a signalling
// one gives a NaN here.
MR_DEV float max_f32(float a, float b) {
  float m;
  asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
  return m;
}

// 0x3F80 (1.0 in bfloat16) in each half of a that equals the half of c, else 0:
// the compiler turns the plain form into a compare and a select per half.
MR_DEV uint32_t one_hot2(uint32_t a, uint32_t c) {
  const uint32_t x = a ^ c, one = 0x00010001u, unit = 0x3F803F80u, less = 0xC080C080u;
  uint32_t m, o;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(x), "v"(one));
  asm("v_pk_mad_u16 %0, %1, %2, %3" : "=v"(o) : "v"(m), "v"(less), "v"(unit));
  return o;
}

// The values that lanes l and l ^ 32 hold, in both lanes alike.
MR_DEV void pair_values(uint32_t v, uint32_t& lower, uint32_t& upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  lower = r[0];
  upper = r[1];
}

// Each wave takes groups of 32 points. Lane (col, h) holds dims 8h..8h+7 and
// 16+8h..16+8h+7 of point col (B operand of the score contraction) and
// centroid rows col and 32 + col come from LDS (A operand); the accumulators
// start at -|c|^2 / 2, so that the largest of them is the nearest centroid.
// After the argmax, the per-cluster sums are a second contraction
// S[c][d] += sum_p [a_p = c] x[p][d]: the one-hot assignment is the A operand
// (clusters x points), and the points' pieces, stored for it as they were split
// for the first and read transposed, are the B operand (points x dims); the
// float32 sums stay in the accumulators until they are flushed into float64
// LDS sums.
// Bound by vector instructions beside the matrix cores. A score keeps its
// accumulator's place within its block of 16 in the four low mantissa bits, so
// that best and second best take an and-or, a maximum and a median a score. One
// workgroup of twelve waves per CU holds the centroids and the float64 sums
// once and leaves room for three waves per SIMD. 16.8 M points: 790 us (the
// matrix cores are busy for 590,000 of 1.38 M clocks, vector instructions take
// 920,000; the clock falls to 1.6..1.8 GHz). With four-wave workgroups, two of
// which were resident, a second split of the transposed float32 values, indices
// carried beside the scores and 715 vector instructions a group of 32 points
// instead of 450: 1,080 us. Collecting the near ties and deciding 64 at a time
// over all centroids: 804 us.
__global__ __launch_bounds__(kKmThreads) void k_km_mfma(const float* __restrict__ X, uint64_t N, const float* __restrict__ C,
                                                        const float* __restrict__ cn_g, const double* __restrict__ cmax_g,
                                                        int32_t* __restrict__ assign, double* __restrict__ part_sum,
                                                        uint32_t* __restrict__ part_cnt, unsigned long long* __restrict__ n_recheck,
                                                        unsigned long long* __restrict__ tiny) {
  constexpr int D = 32, K = 64, W = kKmThreads / kWave;
  __shared__ double s64[K * D];
  __shared__ uint32_t scnt[K];
  __shared__ __attribute__((aligned(16))) float sC[K * D];
  __shared__ __attribute__((aligned(16))) float sCn[K];  // -|c|^2 / 2
  // centroid pieces (hi, mid, lo) as A operands: sCp[piece][row][...] holds
  // the row's four 8-dim chunks, chunk c at position c ^ ((row / 4) % 4), so
  // that the 16 lanes of one 16-byte read (rows r..r+15) meet 16 different
  // bank groups
  __shared__ __attribute__((aligned(16))) __bf16 sCp[3][K][D];
  // per wave: the points' pieces, laid out alike, and the assignments (no
  // cluster for no point)
  __shared__ __attribute__((aligned(16))) uint4 xp[W][3][32][4];
  __shared__ __attribute__((aligned(16))) uint16_t ab[W][32];
  __shared__ uint32_t s_rechecks;
  for (int i = threadIdx.x; i < K * D; i += blockDim.x) {
    s64[i] = 0.0;
    sC[i] = C[i];
    const int r = i / D, e = ((((i % D) / 8) ^ ((r / 4) % 4)) * 8) + i % 8;
    split_bf16x3(C[i], sCp[0][r][e], sCp[1][r][e], sCp[2][r][e]);
  }
  if (threadIdx.x == 0) s_rechecks = 0;
  if (threadIdx.x < K) {
    scnt[threadIdx.x] = 0;
    sCn[threadIdx.x] = -0.5f * cn_g[threadIdx.x];
  }
  __syncthreads();

  const uint32_t lane = lane_id();
  const uint32_t wv = threadIdx.x / kWave;
  const uint32_t h = lane >> 5;     // which half of the dims (0: 0..7 and 16..23, 1: 8..15 and 24..31)
  const uint32_t col = lane & 31u;  // point within the 32-point group / centroid row within a block
  // Where squares, products or sums of them fall below the normal range, each
  // of a score's some 400 operations is off by 2^-126 at most, and the place
  // by 15 x 2^-149: 2^-112 covers both scores. (Without it equal scores of
  // zero differed by their places alone.) The floor stands for norms whose
  // squares vanish: 32 coordinates below 2^-63 have norms below 2^-60.
  constexpr float kAbs = 1.9259299e-34f, kFloor = 3.4694470e-18f, kHuge = 1.3292280e+36f;  // 2^-112, 2^-58, 2^120
  const float cmax = (float)*cmax_g + kFloor;
  const float u = 5.9604645e-08f;                     // 2^-24
  // Error of t = x . c - |c|^2 / 2 as computed. Float32 accumulation of the
  // start value and the piece products: 12 instructions of 16 products each
  // per score, counted as 49 sequential additions (with margin), each relative
  // to |c|^2 / 2 + |x| |c|; the place in the low four mantissa bits, 15 units
  // of the last place at most; the norm's own rounding; the dropped products.
  const float gam = 49.f * u / (1.f - 49.f * u);
  const float place = 1.9073486e-06f;                 // 2^-19
  const float drop = 9.5367432e-07f;                  // 2^-20: the three dropped piece products
  // both scores, x2 margin
  const float e_c = 2.f * (gam + place + u) * cmax * cmax + kAbs;
  const float e_x = 4.f * (gam + place + drop) * cmax;  // times |x|
  // Points from this norm on have squares or products that could pass the
  // float32 range: no score of theirs counts (an infinite one with its place
  // is no number any more), nor of a point that has no norm.
  const float n_max = cmax * cmax < kHuge ? kHuge / cmax : 0.f;

  const uint32_t waves_total = gridDim.x * W;
  const uint32_t wave_g = blockIdx.x * W + wv;
  const uint64_t groups = (N + 31) / 32;
  const uint64_t iters = (groups + waves_total - 1) / waves_total;  // uniform across the grid
  uint32_t rechecks = 0;
  bool any_tiny = false;
  f32x16 sum0 = {}, sum1 = {};  // cluster rows 0..31 and 32..63 x dims (float32, since the last flush)
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  // one group, in xs; the next group's loads go into xn and are in flight meanwhile
  auto group = [&](uint64_t it, float (&xs)[16], float (&xn)[16]) {
    const uint64_t g = it * waves_total + wave_g;
    const uint64_t p = g * 32 + col;
    const bool valid = g < groups && p < N;
    load_group(X, N, g + waves_total, groups, col, h, xn);
    f32x16 acc0, acc1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // register r of lane (col, h) is row 8 (r / 4) + 4 h + r % 4 (+ 32 for acc1)
      const f32x4 c0 = *reinterpret_cast<const f32x4*>(&sCn[8 * q + 4 * h]);
      const f32x4 c1 = *reinterpret_cast<const f32x4*>(&sCn[32 + 8 * q + 4 * h]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc0[4 * q + r] = c0[r];
        acc1[4 * q + r] = c1[r];
      }
    }
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      // B: dims 16 kc + 8h + j of point col (xs[8 kc + j]) as three pieces
      uint4 ph, pm, pl;
      split8_bf16x3(xs + 8 * kc, ph, pm, pl);
      const uint32_t at = (2 * kc + h) ^ ((col / 4) % 4);
      xp[wv][0][col][at] = ph;
      xp[wv][1][col][at] = pm;
      xp[wv][2][col][at] = pl;
      const bf16x8 xh = as_bf16x8(ph), xm = as_bf16x8(pm), xl = as_bf16x8(pl);
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        // A: centroid row blk * 32 + col, the same 8 dims
        const uint32_t row = blk * 32 + col, pc = ((2 * kc + h) ^ ((row / 4) % 4)) * 8;
        const bf16x8 ch = *reinterpret_cast<const bf16x8*>(&sCp[0][row][pc]);
        const bf16x8 cm = *reinterpret_cast<const bf16x8*>(&sCp[1][row][pc]);
        const bf16x8 cl = *reinterpret_cast<const bf16x8*>(&sCp[2][row][pc]);
        f32x16 acc = blk ? acc1 : acc0;
        // smaller products first
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cm, xm, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl, xh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xl, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cm, xh, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xm, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xh, acc, 0, 0, 0);
        if (blk) acc1 = acc; else acc0 = acc;
      }
    }
    // coordinates below 2^-100: zeros are set apart only where there is one
    float amin = fabsf(xs[0]);
#pragma unroll
    for (int t = 1; t < 16; ++t) amin = fminf(amin, fabsf(xs[t]));
    if (__any(amin < __uint_as_float(kTinyBits))) {
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const uint32_t b = __float_as_uint(xs[t]) & 0x7FFFFFFFu;
        any_tiny |= b != 0u && b < kTinyBits;
      }
    }
    // |x| for the bound
    float nx = 0.f;
#pragma unroll
    for (int s = 0; s < 16; ++s) nx = fmaf(xs[s], xs[s], nx);
    uint32_t lo, up;
    pair_values(__float_as_uint(nx), lo, up);
    nx = sqrtf(__uint_as_float(lo) + __uint_as_float(up)) + kFloor;
    // best and second best of this lane's 16 rows of each block
    float b1[2], b2[2];
    uint32_t sc[2][16];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      b1[b] = b2[b] = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t v = (__float_as_uint(b ? acc1[r] : acc0[r]) & ~15u) | (uint32_t)r;
        sc[b][r] = v;
        b2[b] = __builtin_amdgcn_fmed3f(b1[b], b2[b], __uint_as_float(v));
        b1[b] = max_f32(b1[b], __uint_as_float(v));
      }
    }
    const float l1 = fmaxf(b1[0], b1[1]);
    const float l2 = fmaxf(fminf(b1[0], b1[1]), fmaxf(b2[0], b2[1]));
    const uint32_t r = __float_as_uint(l1) & 15u;
    const uint32_t lrow = (b1[1] > b1[0] ? 32u : 0u) + 8 * (r / 4) + 4 * h + r % 4;
    // combine with the partner lane (other 32 rows of the same point)
    uint32_t lo1, up1, lo2, up2, rlo, rup;
    pair_values(__float_as_uint(l1), lo1, up1);
    pair_values(__float_as_uint(l2), lo2, up2);
    pair_values(lrow, rlo, rup);
    const float f1 = __uint_as_float(lo1), g1 = __uint_as_float(up1);
    const float best = fmaxf(f1, g1);
    const float second = fmaxf(fminf(f1, g1), fmaxf(__uint_as_float(lo2), __uint_as_float(up2)));
    int bi = (int)(g1 > f1 ? rup : rlo);
    // Near tie: every score is within eps/2 of its exact value, so the exact
    // nearest is among the rows scoring >= best - eps. Those candidates
    // (usually two) are decided again in float64 from the direct form; both
    // lanes of the pair take part, each for its own rows.
    const float eps = e_c + e_x * nx;
    const bool ranged = nx < n_max;
    const bool need = valid && !(best - second > eps && ranged);
    if (__any(need)) {
      uint32_t cand = 0;
      if (need) {
        const float thr = best - eps;
#pragma unroll
        for (int t = 0; t < 32; ++t) cand |= (__uint_as_float(sc[t / 16][t % 16]) >= thr ? 1u : 0u) << t;
        if (!ranged) cand = ~0u;
      }
      // the partner's half of the point: this lane then holds all 32 dims
      float xo[16];
#pragma unroll
      for (int s = 0; s < 16; ++s) xo[s] = __shfl_xor(xs[s], 32);
      double bd = INFINITY;
      int bj = 0x7fffffff;
#pragma unroll 1
      while (cand) {  // rows in increasing index order: strict < keeps the lowest index
        const int bit = __builtin_ctz(cand);
        cand &= cand - 1u;
        const int rr = bit & 15;
        const int idx = (bit >> 4) * 32 + 8 * (rr / 4) + 4 * (int)h + (rr % 4);
        // own dims first, then the partner's: lane half g holds dims 8g..8g+7
        // and 16+8g..16+8g+7, in xs order
        double dj = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const uint32_t g2 = q < 4 ? h : 1u - h;
          const f32x4 c = *reinterpret_cast<const f32x4*>(sC + idx * D + 16 * ((q % 4) / 2) + 8 * g2 + 4 * (q % 2));
          const float* xv = q < 4 ? xs + 4 * q : xo + 4 * (q - 4);
          float x0 = xv[0], x1 = xv[1], x2 = xv[2], x3 = xv[3];
          // keeps the float64 conversions of x inside this rare loop (hoisted
          // they would hold 64 more registers for the whole kernel)
          asm volatile("" : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3));
          double e;
          e = (double)x0 - (double)c.x; dj = fma(e, e, dj);
          e = (double)x1 - (double)c.y; dj = fma(e, e, dj);
          e = (double)x2 - (double)c.z; dj = fma(e, e, dj);
          e = (double)x3 - (double)c.w; dj = fma(e, e, dj);
        }
        if (dj < bd) {
          bd = dj;
          bj = idx;
        }
      }
      const double obd = __shfl_xor(bd, 32);
      const int obj = __shfl_xor(bj, 32);
      if (obd < bd || (obd == bd && obj < bj)) {
        bd = obd;
        bj = obj;
      }
      if (need) {
        bi = bj;
        if (h == 0) ++rechecks;
      }
      bi = __shfl(bi, (int)col);  // lane col (h = 0) decided for both halves
    }
    if (valid && h == 0) {
      assign[p] = bi;
      if ((uint32_t)bi < (uint32_t)K) atomicAdd(&scnt[bi], 1u);  // (a point with a NaN has no cluster)
    }
    if (h == 0) ab[wv][col] = valid ? (uint16_t)bi : 0xFFFFu;
    wave_sync();
    // Update. 16 points per instruction: lane (col, h) supplies A[col][8h + j]
    // = [a_p = blk * 32 + col] and B[8h + j][col] = x[p][col] (as three pieces)
    // for the points p = 16 kc + 8h + j, j = 0..7. A transposing read takes
    // four rows (points) of 16 columns (dims) per 16 lanes: lane l names the
    // eight bytes of row l / 4, columns 4 (l % 4) .., and receives column l of
    // the four rows.
    const uint32_t c0 = col * 0x10001u, c1 = c0 + 0x200020u;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const uint4 aw = *reinterpret_cast<const uint4*>(&ab[wv][16 * kc + 8 * h]);
      const uint32_t a4[4] = {aw.x, aw.y, aw.z, aw.w};
      uint32_t o0[4], o1[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        o0[j] = one_hot2(a4[j], c0);
        o1[j] = one_hot2(a4[j], c1);
      }
      const bf16x8 v0 = as_bf16x8(make_uint4(o0[0], o0[1], o0[2], o0[3]));
      const bf16x8 v1 = as_bf16x8(make_uint4(o1[0], o1[1], o1[2], o1[3]));
#pragma unroll
      for (int piece = 0; piece < 3; ++piece) {
        s16x4 half[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t p0 = 16 * kc + 8 * h + 4 * q, l = lane & 15u;
          const uint32_t chunk = (2 * (col / 16) + (l % 4) / 2) ^ ((p0 / 4) % 4);
          half[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4*)(reinterpret_cast<short*>(&xp[wv][piece][p0 + l / 4][chunk]) + 4 * (l % 2)));
        }
        const uint2 x0 = __builtin_bit_cast(uint2, half[0]), x1 = __builtin_bit_cast(uint2, half[1]);
        const bf16x8 xv = as_bf16x8(make_uint4(x0.x, x0.y, x1.x, x1.y));
        sum0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v0, xv, sum0, 0, 0, 0);
        sum1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v1, xv, sum1, 0, 0, 0);
      }
    }
    wave_sync();
    if ((it + 1) % kKmFlushIters == 0 || it + 1 == iters) {
      // D layout: register r of lane (col, h) is cluster 8 (r / 4) + 4 h + r % 4 (+ 32 for sum1), dim col
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int c = 8 * (q / 4) + 4 * (int)h + (q % 4);
        atomicAdd(&s64[c * D + col], (double)sum0[q]);
        atomicAdd(&s64[(32 + c) * D + col], (double)sum1[q]);
      }
      sum0 = f32x16{};
      sum1 = f32x16{};
    }
  };
  float xa[16], xb[16];
  load_group(X, N, wave_g, groups, col, h, xa);
  for (uint64_t it = 0; it < iters; it += 2) {
    group(it, xa, xb);
    if (it + 1 < iters) group(it + 1, xb, xa);
  }
  if (rechecks) atomicAdd(&s_rechecks, rechecks);
  __syncthreads();
  if (threadIdx.x == 0 && s_rechecks) atomicAdd(n_recheck, (unsigned long long)s_rechecks);
  if (any_tiny) atomicOr(tiny, 1ull);
  for (int i = threadIdx.x; i < K * D; i += blockDim.x) part_sum[(uint64_t)blockIdx.x * K * D + i] = s64[i];
  if (threadIdx.x < K) part_cnt[(uint64_t)blockIdx.x * K + threadIdx.x] = scnt[threadIdx.x];
}

// ----------------------------------------------------------------------------
// any d, k: assignment on the float32 matrix cores, update in LDS
// ----------------------------------------------------------------------------
// Quotient of a small index by a fixed divisor: exact for i * y < 2^32.
struct SmallDiv {
  uint32_t y, m;
  MR_DEV explicit SmallDiv(uint32_t y_) : y(y_), m(0xFFFFFFFFu / y_ + 1u) {}
  MR_DEV uint32_t div(uint32_t i) const { return y == 1 ? i : __umulhi(i, m); }
};

// Centroids in the order the score contraction reads them: block kb holds
// centroids 32 kb .. 32 kb + 31, and its 8-dim chunk q is one 1 KiB row, lane
// (col, h) holding dims 8q + 4h .. 8q + 4h + 3 of centroid 32 kb + col (zero
// past d or k). cn: squared norms (+inf past k, so a padded row never wins);
// cmax[kb]: the block's largest |c| (float64). One workgroup of 256 per block.
__global__ __launch_bounds__(256) void k_km_pack(const float* __restrict__ C, uint32_t k, uint32_t d, uint32_t dq,
                                                 float* __restrict__ Cp, float* __restrict__ cn, double* __restrict__ cmax) {
  __shared__ double m[32];
  const uint32_t kb = blockIdx.x, lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t i = threadIdx.x; i < dq * kWave * 4; i += blockDim.x) {
    const uint32_t q = i / (kWave * 4), l = i / 4 % kWave, e = i % 4;
    const uint32_t j = kb * 32 + l % 32, t = 8 * q + 4 * (l / 32) + e;
    Cp[(uint64_t)kb * dq * kWave * 4 + i] = j < k && t < d ? C[(uint64_t)j * d + t] : 0.f;
  }
  for (uint32_t r = wv; r < 32; r += 256 / kWave) {
    const uint32_t j = kb * 32 + r;
    double s = 0.0;
    if (j < k)
      for (uint32_t t = lane; t < d; t += kWave) {
        const double v = C[(uint64_t)j * d + t];
        s += v * v;
      }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) {
      cn[j] = j < k ? (float)s : INFINITY;
      m[r] = s;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double b = 0.0;
    for (int r = 0; r < 32; ++r) b = m[r] > b ? m[r] : b;
    cmax[kb] = sqrt(b);
  }
}

// float64 direct-form squared distance (the definition of the step), summed in
// index order, of the row x (zero past d) to packed centroid j.
MR_DEV double dist64(const float* x, const float* __restrict__ Cp, uint32_t dq, uint32_t j) {
  double s = 0.0;
  const float* c = Cp + ((uint64_t)(j / 32) * dq * kWave + j % 32) * 4;
#pragma unroll 2
  for (uint32_t q = 0; q < 2 * dq; ++q, c += kWave / 2 * 4) {
    const f32x4 cv = *gp(reinterpret_cast<const f32x4*>(c));
    const f32x4 xv = *reinterpret_cast<const f32x4*>(x + 4 * q);
    double e;
    e = (double)xv.x - (double)cv.x; s = fma(e, e, s);
    e = (double)xv.y - (double)cv.y; s = fma(e, e, s);
    e = (double)xv.z - (double)cv.z; s = fma(e, e, s);
    e = (double)xv.w - (double)cv.w; s = fma(e, e, s);
  }
  return s;
}

// Nearest centroid of every point for any d <= 256 and k <= 1024. A wave
// takes 32 points: it stages their rows in its own LDS slab (whole rows, read
// coalesced; the row stride is an odd number of 16-byte units, so the 16-byte
// operand reads of 32 rows spread over the banks) and takes their scores
// |c|^2 - 2 <x, c> against KB blocks of 32 centroids at a time with
// v_mfma_f32_32x32x2_f32, the packed centroids coming 1 KiB per load from the
// cache. Each lane keeps the best and second best score of its rows; a point
// whose gap is within the rounding bound is decided again by the whole wave
// from the float64 direct form over all k, so the decisions are those of
// dist64 for every point. Its floor is the matrix cores' float32 rate (32 x 32 x 2
// multiply-adds per 64 cycles and SIMD: 52 us at 500,003 x 64, k = 100, padded
// to 128); it takes 136 us there, two waves per SIMD hiding the row loads and
// the comparisons (five vector instructions per score). One thread per point
// with float64 distances and global atomics for the sums took 48.8 ms.
constexpr uint32_t kKmSlabMax = 16 * 1024;  // LDS bytes of a wave's slab with which four waves share a workgroup

MR_DEV uint32_t km_slab_stride(uint32_t dq) { return 8 * dq + 4; }

template <int KB>
__global__ __launch_bounds__(256) void k_km_assign(const float* __restrict__ X, uint64_t N,
                                                   const float* __restrict__ Cp, const float* __restrict__ cn,
                                                   const double* __restrict__ cmax_g, uint32_t k, uint32_t d, uint32_t dq,
                                                   uint32_t nkb, int32_t* __restrict__ assign) {
  extern __shared__ float slabs[];
  const uint32_t lane = lane_id(), h = lane >> 5, col = lane & 31u;
  const uint32_t wv = threadIdx.x / kWave, ld = km_slab_stride(dq), D8 = 8 * dq;
  float* const xs = slabs + wv * 32 * ld;
  double cmax64 = 0.0;
  for (uint32_t b = 0; b < nkb; ++b) cmax64 = cmax_g[b] > cmax64 ? cmax_g[b] : cmax64;
  const uint64_t step = (uint64_t)gridDim.x * (blockDim.x / kWave) * 32;
  // (waves are independent: no workgroup barriers below)
  for (uint64_t p0 = ((uint64_t)blockIdx.x * (blockDim.x / kWave) + wv) * 32; p0 < N; p0 += step) {
    const uint32_t np = N - p0 < 32 ? (uint32_t)(N - p0) : 32u;
    const float* const Xp = X + p0 * d;
    constexpr int kBatch = 8;  // loads in flight per lane
    if (d % 4 == 0 && ((uintptr_t)X & 15u) == 0) {
      const SmallDiv by(D8 / 4);
      const uint32_t total = 32 * D8 / 4;
      for (uint32_t i0 = 0; i0 < total; i0 += kBatch * kWave) {
        f32x4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t i = i0 + u * kWave + lane, r = by.div(i), c = 4 * (i - r * by.y);
          v[u] = f32x4{};
          if (r < np && c < d) v[u] = *gp(reinterpret_cast<const f32x4*>(Xp + r * d + c));
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t i = i0 + u * kWave + lane, r = by.div(i), c = 4 * (i - r * by.y);
          if (i < total) *reinterpret_cast<f32x4*>(xs + r * ld + c) = v[u];
        }
      }
    } else {
      const SmallDiv by(D8);
      const uint32_t total = 32 * D8;
      for (uint32_t i0 = 0; i0 < total; i0 += kBatch * kWave) {
        float v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t i = i0 + u * kWave + lane, r = by.div(i), c = i - r * by.y;
          v[u] = r < np && c < d ? *gp(Xp + r * d + c) : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t i = i0 + u * kWave + lane, r = by.div(i), c = i - r * by.y;
          if (i < total) xs[r * ld + c] = v[u];
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    float b1 = INFINITY, b2 = INFINITY, nx = 0.f;
    uint32_t i1 = 0;
    const float* const xrow = xs + col * ld + 4 * h;
    for (uint32_t g0 = 0; g0 < nkb; g0 += KB) {
      f32x16 acc[KB];
#pragma unroll
      for (int b = 0; b < KB; ++b) acc[b] = f32x16{};
      const float* const cp = Cp + (uint64_t)g0 * dq * (kWave * 4) + lane * 4;
      auto load_c = [&](uint32_t q, f32x4 (&c)[KB]) {
#pragma unroll
        for (int b = 0; b < KB; ++b)  // (blocks past the last read the first of the group; their scores are not looked at)
          c[b] = *gp(reinterpret_cast<const f32x4*>(cp + ((uint64_t)(g0 + b < nkb ? b : 0) * dq + q) * (kWave * 4)));
      };
      f32x4 cnext[KB];
      load_c(0, cnext);
      for (uint32_t q = 0; q < dq; ++q) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(xrow + 8 * q);
        f32x4 c[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) c[b] = cnext[b];
        load_c(q + 1 < dq ? q + 1 : q, cnext);  // the next chunk's centroids are in flight during this one
        if (g0 == 0) nx = fmaf(x.w, x.w, fmaf(x.z, x.z, fmaf(x.y, x.y, fmaf(x.x, x.x, nx))));
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(c[b].x, x.x, acc[b], 0, 0, 0);
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(c[b].y, x.y, acc[b], 0, 0, 0);
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(c[b].z, x.z, acc[b], 0, 0, 0);
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(c[b].w, x.w, acc[b], 0, 0, 0);
        }
      }
#pragma unroll
      for (int b = 0; b < KB; ++b) {
        if (g0 + b >= nkb) break;
#pragma unroll
        for (int r = 0; r < 16; ++r) {  // rows in increasing index order: strict < keeps the lowest index
          const uint32_t idx = (g0 + b) * 32 + 8 * (r / 4) + 4 * h + (r % 4);
          const float v = *gp(cn + idx) - 2.f * acc[b][r];
          const bool better = v < b1;
          b2 = better ? b1 : (v < b2 ? v : b2);
          i1 = better ? idx : i1;
          b1 = better ? v : b1;
        }
      }
    }
    // combine with the partner lane (the other half of every block's rows)
    const float o1 = __shfl_xor(b1, 32), o2 = __shfl_xor(b2, 32);
    const uint32_t oi = (uint32_t)__shfl_xor((int)i1, 32);
    const bool other = o1 < b1 || (o1 == b1 && oi < i1);
    const float best = other ? o1 : b1;
    const float second = other ? (b1 < o2 ? b1 : o2) : (b2 < o1 ? b2 : o1);
    uint32_t bi = other ? oi : i1;
    // Rounding bound of a gap between two scores, four times (|c|^2 and the
    // product's factor 2, two scores) the bounds of the norm, the accumulation
    // of 8 dq products and the subtraction, and a quarter more for the
    // roundings of the bound itself. The floors keep the bound valid where squares or products fall below the
    // normal range; where they could pass the float32 range, every decision is
    // made again.
    constexpr float u = 5.9604645e-08f;  // 2^-24
    constexpr float kFloor = 3.4694470e-18f, kAbs = 7.8886091e-31f, kHuge = 1.3292280e+36f;  // 2^-58, 2^-100, 2^120
    nx += __shfl_xor(nx, 32);
    nx = sqrtf(nx) + kFloor;
    const float cmax = (float)cmax64 + kFloor;
    const float ops = (float)(2 * D8 + 8) * u, gam = ops / (1.f - ops);
    const float eps = 5.f * u * cmax * cmax + 5.f * (gam + u) * cmax * nx + kAbs;
    const bool sure = second - best > eps && nx * cmax < kHuge && cmax * cmax < kHuge;
    uint64_t again = __ballot(!sure && col < np) & 0xFFFFFFFFull;
    while (again) {
      const int r = __builtin_ctzll(again);
      again &= again - 1;
      double bd = INFINITY;
      uint32_t bj = ~0u;
      for (uint32_t j = lane; j < k; j += kWave) {
        const double dj = dist64(xs + r * ld, Cp, dq, j);
        if (dj < bd) {
          bd = dj;
          bj = j;
        }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double od = __shfl_xor(bd, o);
        const uint32_t oj = (uint32_t)__shfl_xor((int)bj, o);
        if (od < bd || (od == bd && oj < bj)) {
          bd = od;
          bj = oj;
        }
      }
      if (col == (uint32_t)r) bi = bj == ~0u ? 0u : bj;  // no distance below infinity: index 0
    }
    if (h == 0 && col < np) assign[p0 + col] = (int32_t)bi;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Per-cluster float64 sums and counts of the assigned points. A workgroup
// takes a range of points and a slice of `ds` dims (all of them where k x d
// float64 sums fit its LDS). It orders a tile of points by cluster (counting
// sort in LDS); a wave - or each of its groups of lanes, where a row takes at
// most half a wave - takes an equal part of that order and adds its rows, one
// dim per lane, in a float64 register that goes to the LDS sums when the
// cluster changes, so a run of one cluster costs one LDS atomic per dim
// instead of one per point (float64 LDS atomics take about a cycle per lane: 61 us with one per point and
// dim, 27 us this way, at 500,003 x 64, k = 100). The workgroup's sums are one partial of k_km_final.
constexpr uint32_t kKmUpdThreads = 1024;
constexpr uint32_t kKmUpdTile = 4096;        // points per tile
constexpr uint32_t kKmUpdLds = 124 * 1024;   // LDS bytes of the sums and counts

__global__ __launch_bounds__(kKmUpdThreads) void k_km_update(const float* __restrict__ X, uint64_t N, uint32_t k, uint32_t d,
                                                             uint32_t ds, uint32_t G, const int32_t* __restrict__ assign,
                                                             double* __restrict__ part_sum, uint32_t* __restrict__ part_cnt) {
  extern __shared__ double s64[];
  __shared__ uint32_t order[kKmUpdTile];  // (cluster << 16) | point of the tile
  __shared__ uint32_t next[kKmUpdThreads];
  __shared__ uint32_t wsum[kKmUpdThreads / kWave];
  const uint32_t g = blockIdx.x % G, t0 = blockIdx.x / G * ds;
  const uint32_t w = d - t0 < ds ? d - t0 : ds;  // dims of this slice
  uint32_t* const cnt = reinterpret_cast<uint32_t*>(s64 + (uint64_t)k * w);
  const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
  for (uint32_t i = threadIdx.x; i < k * w; i += blockDim.x) s64[i] = 0.0;
  for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) cnt[i] = 0;
  // lanes of one point: the power of two that covers the slice, at most a wave
  uint32_t lpp = 1;
  while (lpp < w && lpp < kWave) lpp *= 2;
  const uint32_t side = kWave / lpp, sub = lane / lpp, t = lane % lpp;
  const uint64_t lo = N * g / G, hi = N * (g + 1) / G;
  for (uint64_t base = lo; base < hi; base += kKmUpdTile) {
    const uint32_t m = hi - base < kKmUpdTile ? (uint32_t)(hi - base) : kKmUpdTile;
    // 1. the tile's points ordered by cluster
    constexpr uint32_t kPer = kKmUpdTile / kKmUpdThreads;
    uint32_t a[kPer];
    next[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t i = u * kKmUpdThreads + threadIdx.x;
      a[u] = i < m ? (uint32_t)assign[base + i] : ~0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u)
      if (a[u] != ~0u) atomicAdd(&next[a[u]], 1u);
    __syncthreads();
    const uint32_t c = next[threadIdx.x];  // (at most 1024 clusters: one per thread)
    const uint32_t incl = wave_incl_scan(c);
    if (lane == kWave - 1) wsum[wv] = incl;
    __syncthreads();
    uint32_t run = incl - c;
    for (uint32_t q = 0; q < wv; ++q) run += wsum[q];
    next[threadIdx.x] = run;
    if (threadIdx.x < k) cnt[threadIdx.x] += c;
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u)
      if (a[u] != ~0u) order[atomicAdd(&next[a[u]], 1u)] = a[u] << 16 | (u * kKmUpdThreads + threadIdx.x);
    __syncthreads();
    // 2. each group of lpp lanes takes an equal part of the order
    const uint32_t grp = wv * side + sub, groups = (kKmUpdThreads / kWave) * side;
    const uint32_t b0 = m * grp / groups, b1 = m * (grp + 1) / groups;
    const float* const Xb = X + base * d + t0;
    constexpr uint32_t kBatch = 16;  // rows in flight per lane
    for (uint32_t tc = t; tc < w; tc += kWave) {
      double s = 0.0;
      uint32_t cur = ~0u;
      for (uint32_t i0 = b0; i0 < b1; i0 += kBatch) {
        uint32_t e[kBatch];
        float v[kBatch];
#pragma unroll
        for (uint32_t u = 0; u < kBatch; ++u) e[u] = order[i0 + u < b1 ? i0 + u : b1 - 1];
#pragma unroll
        for (uint32_t u = 0; u < kBatch; ++u) v[u] = *gp(Xb + (e[u] & 0xFFFFu) * d + tc);
#pragma unroll
        for (uint32_t u = 0; u < kBatch; ++u) {
          const uint32_t j = e[u] >> 16;
          if (i0 + u >= b1) v[u] = 0.f;  // (repeats the last point's cluster)
          if (j != cur) {
            if (cur != ~0u) atomicAdd(&s64[cur * w + tc], s);
            cur = j;
            s = 0.0;
          }
          s += (double)v[u];
        }
      }
      if (cur != ~0u) atomicAdd(&s64[cur * w + tc], s);
    }
    __syncthreads();
  }
  for (uint32_t i = threadIdx.x; i < k * w; i += blockDim.x)
    part_sum[((uint64_t)g * k + i / w) * d + t0 + i % w] = s64[i];
  if (t0 == 0)
    for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) part_cnt[(uint64_t)g * k + i] = cnt[i];
}

// Dims per slice and partials of the update: slices as wide as the LDS sums
// allow; enough partials for one workgroup per CU, each with at least 256
// points and, over all, at most 2^21 float64 sums to write and add.
KmUpdPlan km_upd_plan(uint64_t N, uint32_t k, uint32_t d, uint32_t n_cu) {
  KmUpdPlan u{};
  u.ds = std::min<uint32_t>(d, (kKmUpdLds - 4 * k) / (8 * k));
  u.slices = (d + u.ds - 1) / u.ds;
  uint64_t g = std::max<uint32_t>(1, n_cu / u.slices);
  g = std::min<uint64_t>(g, (N + 255) / 256);
  g = std::min<uint64_t>(g, (1ull << 21) / ((uint64_t)k * d));
  u.G = (uint32_t)std::max<uint64_t>(1, g);
  return u;
}

// Sum the G partials in a fixed order (deterministic), write float32 sums,
// counts and new centroids (old centroid for an empty cluster). Workgroup =
// 64 consecutive (cluster, dim) entries x 16 waves; wave w adds partials
// g = w, w + 16, ... (loads unrolled, in flight together), then the 16 wave
// sums are added in wave order. The same split for every launch keeps the
// result bit-identical from run to run.
constexpr int kFinalWaves = 16;

__global__ __launch_bounds__(kFinalWaves * kWave) void k_km_final(const double* __restrict__ part_sum,
                                                                  const uint32_t* __restrict__ part_cnt, uint32_t G,
                                                                  uint32_t k, uint32_t d, const float* __restrict__ C,
                                                                  float* __restrict__ sums, uint32_t* __restrict__ counts,
                                                                  float* __restrict__ cent) {
  __shared__ double ws[kFinalWaves][kWave];
  __shared__ unsigned long long wn[kFinalWaves][kWave];
  const uint64_t kd = (uint64_t)k * d;
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  const uint64_t i = (uint64_t)blockIdx.x * kWave + lane;
  double s = 0.0;
  unsigned long long n = 0;
  if (i < kd) {
    const uint32_t j = (uint32_t)(i / d);
    uint32_t g = w;
    for (; g + 3 * kFinalWaves < G; g += 4 * kFinalWaves) {
      const double a0 = part_sum[(uint64_t)g * kd + i], a1 = part_sum[(uint64_t)(g + kFinalWaves) * kd + i];
      const double a2 = part_sum[(uint64_t)(g + 2 * kFinalWaves) * kd + i];
      const double a3 = part_sum[(uint64_t)(g + 3 * kFinalWaves) * kd + i];
      const uint32_t c0 = part_cnt[(uint64_t)g * k + j], c1 = part_cnt[(uint64_t)(g + kFinalWaves) * k + j];
      const uint32_t c2 = part_cnt[(uint64_t)(g + 2 * kFinalWaves) * k + j];
      const uint32_t c3 = part_cnt[(uint64_t)(g + 3 * kFinalWaves) * k + j];
      s += a0;
      s += a1;
      s += a2;
      s += a3;
      n += (unsigned long long)c0 + c1 + c2 + c3;
    }
    for (; g < G; g += kFinalWaves) {
      s += part_sum[(uint64_t)g * kd + i];
      n += part_cnt[(uint64_t)g * k + j];
    }
  }
  ws[w][lane] = s;
  wn[w][lane] = n;
  __syncthreads();
  if (w == 0 && i < kd) {
    double t = 0.0;
    unsigned long long c = 0;
    for (int q = 0; q < kFinalWaves; ++q) {
      t += ws[q][lane];
      c += wn[q][lane];
    }
    const uint32_t j = (uint32_t)(i / d);
    if (sums) sums[i] = (float)t;
    if (cent) cent[i] = c ? (float)(t / (double)c) : C[i];
    if (counts && i % d == 0) counts[j] = (uint32_t)c;
  }
}

// Any d, k in a caller workspace that the packed centroids do not fit (few
// dimensions or clusters, whose single partial is smaller than they are): a
// thread per point, float64 direct distances, sums by atomics on one partial.
// (500,000 points, d = 64, k = 100: 48.7 ms, the packed path 0.19 ms.)
__global__ void k_km_clear(double* __restrict__ sum, uint64_t n_sum, uint32_t* __restrict__ cnt, uint32_t k) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_sum; i += (uint64_t)gridDim.x * blockDim.x) {
    sum[i] = 0.0;
    if (i < k) cnt[i] = 0u;
  }
}

__global__ __launch_bounds__(256) void k_km_direct(const float* __restrict__ X, uint64_t N, const float* __restrict__ C,
                                                   uint32_t k, uint32_t d, int32_t* __restrict__ assign,
                                                   double* __restrict__ sum, uint32_t* __restrict__ cnt) {
  for (uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; p < N; p += (uint64_t)gridDim.x * blockDim.x) {
    const float* const x = X + p * d;
    double bd = INFINITY;
    uint32_t bj = 0;
    for (uint32_t j = 0; j < k; ++j) {
      double s = 0.0;
#pragma unroll 1
      for (uint32_t t = 0; t < d; ++t) {
        const double e = (double)x[t] - (double)C[(uint64_t)j * d + t];
        s += e * e;
      }
      if (s < bd) {
        bd = s;
        bj = j;
      }
    }
    assign[p] = (int32_t)bj;
    atomicAdd(&cnt[bj], 1u);
    for (uint32_t t = 0; t < d; ++t) atomicAdd(&sum[(uint64_t)bj * d + t], (double)x[t]);
  }
}

static hipError_t km_enqueue_generic(const KmLaunch& L, hipStream_t s) {
  const uint32_t dq = (L.d + 7) / 8, nkb = (L.k + 31) / 32;
  if (L.N) {
    const uint32_t slab = 32 * (8 * dq + 4) * sizeof(float);
    const uint32_t waves = slab <= kKmSlabMax ? 4 : 1;
    const uint64_t grid = std::min<uint64_t>((L.N + 32 * waves - 1) / (32 * waves), 1u << 16);
#define MR_KM_ASSIGN(KB)                                                                                          \
  hipLaunchKernelGGL(k_km_assign<KB>, dim3((uint32_t)grid), dim3(waves * kWave), waves * slab, s, L.X, L.N,      \
                     L.cp, L.cn, L.cmax, L.k, L.d, dq, nkb, L.assign)
    if (nkb == 1) MR_KM_ASSIGN(1);
    else if (nkb == 2) MR_KM_ASSIGN(2);
    else MR_KM_ASSIGN(4);
#undef MR_KM_ASSIGN
  }
  const KmUpdPlan u = L.upd;
  const uint32_t lds = 8u * L.k * u.ds + 4u * L.k;
  if (lds > 32 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_km_update),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kKmUpdLds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_km_update, dim3(u.G * u.slices), dim3(kKmUpdThreads), lds, s, L.X, L.N, L.k, L.d, u.ds, u.G,
                     L.assign, L.part_sum, L.part_cnt);
  return hipGetLastError();
}

hipError_t km_enqueue(const KmLaunch& L, hipStream_t s, hipEvent_t map0, hipEvent_t map1) {
  if (L.direct)
    hipLaunchKernelGGL(k_km_clear, dim3(256), dim3(256), 0, s, L.part_sum, (uint64_t)L.k * L.d, L.part_cnt, L.k);
  else if (L.mfma) hipLaunchKernelGGL(k_km_prep, dim3(1), dim3(kWave), 0, s, L.C, L.cn, L.cmax, L.n_recheck, L.tiny);
  else
    hipLaunchKernelGGL(k_km_pack, dim3((L.k + 31) / 32), dim3(256), 0, s, L.C, L.k, L.d, (L.d + 7) / 8, L.cp, L.cn, L.cmax);
  if (map0) (void)hipEventRecord(map0, s);
  if (L.direct) {
    const uint64_t b = std::max<uint64_t>(1, std::min<uint64_t>((L.N + 255) / 256, 4096));
    hipLaunchKernelGGL(k_km_direct, dim3((uint32_t)b), dim3(256), 0, s, L.X, L.N, L.C, L.k, L.d, L.assign, L.part_sum, L.part_cnt);
  } else if (L.mfma) {
    hipLaunchKernelGGL(k_km_mfma, dim3(L.G), dim3(kKmThreads), 0, s, L.X, L.N, L.C, L.cn, L.cmax, L.assign, L.part_sum,
                       L.part_cnt, L.n_recheck, L.tiny);
  } else {
    const hipError_t e = km_enqueue_generic(L, s);
    if (e != hipSuccess) return e;
  }
  if (map1) (void)hipEventRecord(map1, s);
  const uint64_t kd = (uint64_t)L.k * L.d;
  hipLaunchKernelGGL(k_km_final, dim3((uint32_t)((kd + kWave - 1) / kWave)), dim3(kFinalWaves * kWave), 0, s, L.part_sum, L.part_cnt,
                     L.direct ? 1u : L.mfma ? L.G : L.upd.G, L.k, L.d, L.C, L.sums, L.counts, L.cent);
  return hipGetLastError();
}

}  // namespace mr
