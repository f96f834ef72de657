// Internal launch interfaces between the host planner (api.cpp) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "jobs.h"

namespace mr {

// Small results to pinned host memory at the end of a job's kernels: ranges of
// 32-bit words (unused: 0 words), copied by a kernel, so that a job needs no
// copy after its last one.
struct PubRange {
  const void* from;
  void* to;
  uint32_t words;
};
struct Publish {
  PubRange r[3];
};
hipError_t publish_enqueue(const Publish& P, hipStream_t s);

struct WordsLaunch {
  const WordJob* jobs;        // device array [n_jobs]
  const uint64_t* tile_base;  // device array [n_jobs + 1]
  uint32_t n_jobs;
  WordJob one;                // the descriptor of a single job, which the preparation kernel stores
  uint64_t total_tiles;
  uint64_t total_slots;       // sum of table capacities
  uint32_t map_grid;
  uint32_t sort_grid;
  int lds_log2;
  uint32_t debug_hash;
  bool any_records;
  bool wave_combine;          // merge equal words of a wave before the LDS cache (the wave-level combiner)
  uint32_t* totals;           // device [2]: buckets, record tiles
  uint32_t* bucket_cnt;       // device [n_jobs * kMaxBuckets]
  unsigned long long* bucket_bytes;
  uint32_t* bucket_start;
  unsigned long long* bucket_bstart;
  uint32_t* bucket_fill;
  JobState* states;           // device [n_jobs]
  Publish pub;                // states (and markers found) to host memory
  uint32_t n_parts;            // partitions of the two-phase reduce through partition queues (0: none)
  // Reverse Index map instead of the word map (one job)
  bool links;
  uint32_t link_grid;
  uint32_t* link_marks;       // device [link_cap] marker offsets
  unsigned long long* link_n; // device: markers found
  uint64_t link_cap;
  uint32_t* link_pair_slot;          // device [link_cap] table slot of the link's URL (all ones: no link)
  uint32_t* link_pair_file;          // device [link_cap] record of the link
};

hipError_t words_enqueue_zero_states(const WordsLaunch& L, hipStream_t s);
hipError_t words_enqueue_prep(const WordsLaunch& L, hipStream_t s);
hipError_t words_enqueue_map(const WordsLaunch& L, hipStream_t s);
hipError_t words_enqueue_reduce(const WordsLaunch& L, hipStream_t s);

// Reverse Index file lists from the pairs and the sorted URLs (links.hip)
struct LinksPost {
  const uint32_t* pair_slot;    // table slot of each link's URL (all ones: no link)
  const uint32_t* pair_file;
  uint64_t n;                   // pairs (markers)
  const uint32_t* slot_rank;    // output rank of the URL in each table slot
  uint64_t n_keys;              // distinct URLs
  uint64_t file_mod;            // sort key = rank * file_mod + record (file_mod: the record count, at least 1)
  int sort_bits;                // key bits, a multiple of 8, with 2^sort_bits > n_keys * file_mod
  unsigned long long *k0, *k1, *k2;  // [n] each: sort keys and the sort's two buffers
  unsigned long long* diff;     // device: differing key bits
  uint32_t* hist;               // radix histogram
  uint32_t* tot;                // [256]
  uint32_t* scan_sums;
  uint32_t* head;               // [n]
  unsigned long long* total;    // device: distinct (URL, file) pairs
  unsigned long long* n_valid;  // device: links
  uint32_t* flags;              // device: internal errors
  uint32_t* first;              // [n_keys + 1] first sorted pair of each rank
};
hipError_t links_enqueue_rank_sort(const LinksPost& P, hipStream_t s);
hipError_t links_enqueue_write(const LinksPost& P, uint32_t* ids, uint64_t cap_ids, uint64_t* list_off,
                               uint32_t* counts, hipStream_t s);

// Allocation-free histogram: partial rows in a static device array of
// kRgbStaticRows rows (3 MiB per GPU). rgb_static_init looks up its address
// on a device (once); rgb_static_rows is the row count for an input (at most
// kRgbStaticRows); rgb_static_enqueue launches the two kernels on it.
constexpr uint32_t kRgbStaticRows = 1024;
hipError_t rgb_static_init(int device);
uint32_t rgb_static_rows(uint64_t n, int n_cu);
hipError_t rgb_static_enqueue(int device, const uint8_t* in, uint64_t n, uint32_t G, unsigned long long* out,
                              hipStream_t s);
uint32_t rgb_grid(uint64_t n, int n_cu);
// map0 / map1 (optional) are recorded around k_rgb_partial.
hipError_t rgb_enqueue(const uint8_t* in, uint64_t n, uint32_t* partials, uint32_t G, unsigned long long* out,
                       hipStream_t s, hipEvent_t map0, hipEvent_t map1);
// Adds the same sequence to an empty graph g, with event-record nodes for the
// non-null events: all0, map0, k_rgb_partial, map1, k_rgb_reduce, all1.
hipError_t rgb_graph_build(hipGraph_t g, const uint8_t* in, uint64_t n, uint32_t* partials, uint32_t G,
                           unsigned long long* out, hipEvent_t all0, hipEvent_t map0, hipEvent_t map1,
                           hipEvent_t all1);

// End of an integer-key job: its state goes to host memory, and the other
// state block is cleared for the next job. host == NULL: not done.
struct IntPub {  // pinned host memory
  uint32_t flags, sampled, estimate, pad;
  unsigned long long n_out, n_claimed;
};
struct IntEnd {
  const uint32_t* flags;
  IntPub* host;
  uint32_t* clear;
  uint32_t clear_words;
};

// Integer-key jobs: one launch description shared by the four containers.
struct IntLaunch {
  const uint32_t* in;   // keys
  const uint32_t* vals_in;  // values (NULL: keys alone, every value 1)
  uint32_t stride;      // words from one key, and one value, to the next
  uint64_t n;           // elements
  uint32_t op;          // 0 COUNT, 1 SUM, 2 MIN, 3 MAX
  uint64_t R;           // declared key range (0 = none)
  uint32_t G;           // workgroups of the map kernels
  uint32_t debug_hash;
  uint32_t* flags;      // device job flags
  // array containers
  uint32_t* cnt_part;
  void* val_part;
  uint32_t* dcnt;       // dense counts [R]
  void* dval;           // dense values [R] (64-bit for SUM)
  uint32_t* blk;        // compaction block counts
  // hash container
  uint32_t* t_keys;
  uint32_t* t_cnt;
  void* t_val;
  uint64_t t_cap;
  uint32_t* claimed;
  unsigned long long* n_claimed;
  uint64_t max_probes;  // slots an insert looks at before the table counts as full
  uint64_t max_claims;  // slots claimed before it does
  uint32_t* side_cnt;
  void* side_val;
  // hash output: (key, index) pairs and values of the claimed slots
  void* pairs;
  unsigned long long* vals;
  // outputs
  uint32_t* out_keys;
  void* out_vals;
  uint64_t cap;
  unsigned long long* n_out;  // device: number of distinct keys
  IntEnd end;
};

// Radix sort of all elements and the reduce of the runs (sort.hip).
struct RadixPlan {
  uint32_t n_tiles;
  uint64_t n_chunks;    // chunks of the reduce
  // scratch sizes, not below those of any smaller n
  uint64_t hist_words;  // digit counts of all tiles
  uint64_t chunk_cap;   // entries per chunk array
};
RadixPlan radix_plan(uint64_t n);
struct SortLaunch {
  const uint32_t* in;
  uint64_t n;              // elements, below 2^32
  const uint32_t* vals_in;   // as in IntLaunch
  uint32_t stride, op;
  uint64_t R;              // declared key range (0 = none)
  uint32_t bits;           // key bits that can differ
  uint32_t* flags;
  unsigned long long* diff;  // zero at the start: gathers the differing key bits
  void *buf0, *buf1;       // [n] each: uint32 keys for COUNT, (key, value) pairs otherwise
  uint32_t* hist;          // [hist_words]
  uint32_t* tot;           // [256]
  uint32_t* heads;         // [chunk_cap] run heads per chunk
  uint32_t* scan_sums;     // scan_sums_count(chunk_cap)
  unsigned long long* lead;  // [chunk_cap]
  uint32_t* out_keys;
  void* out_vals;
  uint64_t cap;
  unsigned long long* n_out;
  IntEnd end;
};
hipError_t int_enqueue_sort(const SortLaunch& L, hipStream_t s);
// in: n pairs (key, index into vals); writes keys ascending and their values
// (uses in, n, op, flags, diff, buf0, buf1, hist, tot and the outputs).
hipError_t pairs_enqueue_out(const SortLaunch& L, const unsigned long long* vals, hipStream_t s);
// Sort of uint64 keys by their low `bits` bits. The result is in buf0 when
// rs_moves_before(*diff, keys64_sorted_bits(bits)) is odd, else in buf1.
struct Keys64Sort {
  const unsigned long long* in;
  uint64_t n;
  uint32_t bits;
  unsigned long long* diff;  // device, zero at the start
  unsigned long long *buf0, *buf1;
  uint32_t* hist;            // [radix_plan(n).hist_words]
  uint32_t* tot;             // [256]
};
hipError_t keys64_enqueue_sort(const Keys64Sort& L, hipStream_t s);
uint32_t keys64_sorted_bits(uint32_t bits);

hipError_t int_enqueue_lds_array(const IntLaunch& L, hipStream_t s);
bool int_lds_direct(uint64_t R, uint32_t G);  // whether its output needs no reduced arrays (dcnt, dval)
// device-wide exclusive scan of uint32 counts (sums: scan_sums_count(n) entries)
hipError_t scan_exclusive_u32(uint32_t* a, uint64_t n, uint32_t* sums, unsigned long long* total, hipStream_t s,
                              const IntEnd& E = IntEnd{});
uint64_t scan_sums_count(uint64_t n);

// Bloom filter build: plan and enqueue (see bloom.hip)
struct BloomPlan {
  uint64_t n_kmers;      // k-mers of the input
  uint64_t n_words;      // uint32 words of the m-bit filter
  uint64_t max_entries;  // positions emitted at most (n_kmers * h)
  // 0 tiles: few positions, set by device atomics
  uint32_t n_tiles, cap;  // tiles, positions a tile holds at most
  uint32_t sb, S;         // bits of a sub-range's size, sub-ranges
  uint32_t per, grid;     // sub-ranges per range, ranges
  uint32_t row_words;     // words of a tile's row of sub-range starts (16-bit)
  uint32_t lpg;           // lanes that take a tile's run of a range together
  bool ok;                // parameters and sizes within the kernels' limits
};
BloomPlan bloom_plan(uint64_t n_bytes, uint32_t k, uint32_t h, uint64_t m, uint32_t n_cu);
uint64_t bloom_row_bytes(const BloomPlan& b);
uint64_t bloom_part_bytes(const BloomPlan& b);
hipError_t bloom_enqueue(const uint8_t* in, uint64_t n_bytes, uint32_t k, uint32_t h, uint64_t m, const BloomPlan& b,
                         uint32_t* rows, uint16_t* part, uint32_t* words, hipStream_t s);
hipError_t int_enqueue_global_array(const IntLaunch& L, hipStream_t s);
// global array filled by key-range partitions, for a range and element count the plan finds usable
// Fewer elements take atomics on the array: 131,072 uniform pairs over 20,000
// keys 104 us, 113 us partitioned (three more launches); 262,144 pairs 70 to
// 110 us partitioned whatever the keys, atomics 65 to 340 us on skewed ones.
constexpr uint64_t kVpMin = 1ull << 18;
// So do elements with values on so many times as many keys, since the ranges'
// counts and values are all written whatever they hold: 2^18 pairs over 2^25
// keys, SUM, 178 us by atomics and 280 us partitioned, 2^19 pairs 209 and
// 304 us, 2^21 pairs 405 and 360 us. (Counts alone are level there: 2^18 over
// 2^26 keys 255 and 258 us.)
constexpr uint64_t kVpSparse = 64;
struct VpPlan {
  uint32_t kb, P;       // ranges of 2^kb keys
  uint32_t n_tiles;
  uint64_t elems, runs; // partitioned elements; (P + 1) run starts per tile
  uint32_t split, grid; // elements per workgroup of the fill; its workgroups at most
  uint32_t slices;      // slices of the tiles whose elements are counted per range
  bool list;            // counting: runs' pieces listed per wave instead
  bool usable;
};
VpPlan vp_plan(uint64_t n, uint64_t R, uint32_t op, uint32_t n_cu);
hipError_t int_enqueue_global_array_vp(const IntLaunch& L, const VpPlan& p, uint32_t* runs, uint16_t* pk, uint32_t* pv,
                                       uint32_t* tot, hipStream_t s);
hipError_t int_enqueue_dense_out(const IntLaunch& L, bool clear, bool by_parts, hipStream_t s);
hipError_t int_enqueue_hash_map(const IntLaunch& L, hipStream_t s);
hipError_t int_enqueue_sample(const IntLaunch& L, IntPub* host, hipStream_t s);  // -> host->sampled, estimate (n at least 8192)
uint32_t int_small_out_max();  // keys int_enqueue_small_out handles
hipError_t int_enqueue_small_out(const IntLaunch& L, hipStream_t s);
hipError_t int_enqueue_hash_out(const IntLaunch& L, uint64_t n_claimed_host, hipStream_t s);
hipError_t int_enqueue_side_append(const IntLaunch& L, hipStream_t s);
uint32_t int_lds_array_bytes(uint64_t R, uint32_t op);

// One k-means step.
// Update of the generic path: dims per LDS slice, slices, and partials (ranges of points).
struct KmUpdPlan {
  uint32_t ds, slices, G;
};
KmUpdPlan km_upd_plan(uint64_t N, uint32_t k, uint32_t d, uint32_t n_cu);

struct KmLaunch {
  const float* X;       // points [N][d]
  uint64_t N;
  const float* C;       // centroids [k][d]
  uint32_t k, d;
  float* cn;            // scratch [k rounded up to 32]
  double* cmax;         // scratch [k / 32, rounded up]
  float* cp;            // generic path: centroids packed for the score contraction (shares the partials' memory)
  KmUpdPlan upd;        // generic path
  uint32_t G;           // workgroups of the assignment kernel (matrix-core path at d = 32, k = 64)
  bool mfma;            // d == 32, k == 64 and X 16-byte aligned
  bool direct;          // a caller workspace too small for the packed centroids
  int32_t* assign;      // [N]
  double* part_sum;     // [G][k][d] (generic path: upd.G partials)
  uint32_t* part_cnt;   // [G][k]
  unsigned long long* n_recheck;
  unsigned long long* tiny;  // set when a coordinate is nonzero and below 2^-100 (the step is then redone generically)
  float* sums;          // [k][d]
  uint32_t* counts;     // [k]
  float* cent;          // [k][d]
};

hipError_t km_enqueue(const KmLaunch& L, hipStream_t s, hipEvent_t map0, hipEvent_t map1);

// Selector: features of a job and the network kernels.
// Selector features: one sampling workgroup per window writes its window's
// results into the state, and a finishing workgroup merges them.
uint64_t feature_state_bytes();
hipError_t features_enqueue(const uint8_t* in, uint64_t bytes, int kind, int op, uint64_t key_range, uint32_t lds_budget,
                            float* feats, void* state, hipStream_t s);
hipError_t mlp_forward_enqueue(const float* P, const float* X, uint32_t B, float* H1, float* H2, float* Y, hipStream_t s);
hipError_t select_enqueue(const float* feats, const float* norm, const float* P, uint32_t feas, int32_t* choice,
                          hipStream_t s);
hipError_t mlp_backward_enqueue(const float* P, const float* X, const float* H1, const float* H2, const float* Y,
                                const float* T, const float* M, uint32_t B, float* dY, float* dZ1, float* dZ2, float* loss,
                                float* G, hipStream_t s);
hipError_t adam_enqueue(float* P, const float* G, float* m, float* v, uint32_t step, float lr, float b1, float b2, float eps,
                        hipStream_t s);

// Word hashing one character per lane per step (strhash.hip): word starts per
// 16-byte chunk and their exclusive scan (counts[n_chunks] in place, total
// = number of words); the word list (offsets, lengths, uint32); FNV-1a 64 of
// every word with the padding or the stream schedule, `units` lanes per
// wavefront, one wavefront per `block` words; sched optional ([word][3]).
hipError_t hw_enqueue_list(const uint8_t* in, uint64_t n, uint32_t* counts, uint64_t n_chunks, uint32_t* scan_sums,
                           unsigned long long* total, hipStream_t s);
hipError_t hw_enqueue_words(const uint8_t* in, uint64_t n, const uint32_t* first, uint64_t n_chunks, uint32_t* off,
                            uint32_t* len, hipStream_t s);
hipError_t hw_enqueue_hash(const uint8_t* in, const uint32_t* off, const uint32_t* len, uint64_t n_words, bool stream,
                           uint32_t units, uint64_t block, unsigned long long* hashes, uint32_t* sched, hipStream_t s);

}  // namespace mr
