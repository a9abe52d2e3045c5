// gfx950 kernels for KVpop's running top-k ranking (App. B.3, App. C.2, Sec. 3.1
// eqs. eligible_set and teacher_label).
//
// Per (batch row, KV head) sequence of scores r_t:
//   * static priority (eq. static_priority_app, decay step 1), in float32:
//       prio_t = fl(r_t - fl(t * log_gamma));
//   * rank_t = position of t in descending priority order, ties to the earlier t;
//   * running cutoff: at query q the eligible set is E(q) = {t : s <= t <= q - w};
//     cutoff_q = the k-th smallest rank in E(q) once |E(q)| >= k, else T (all kept);
//   * teacher label of t_new = q - w (+1 kept, -1 dropped, 0 if E(q) is empty) and
//     the boundary token (the kept eligible token with the largest rank).
//
// The paper scans q with a Fenwick tree, one dependent tree walk per query. Here
// every step is spread over the chip:
//   1. topk_chunk_sort_kernel: chunks of 4096 positions, each sorted by one workgroup
//      (a stable LSD radix sort of 32-bit priority keys in LDS, 8 bits per pass).
//   2. topk_merge_kernel: runs of up to 32 sorted chunks, each workgroup merging the
//      stretch of every chunk that lies between two sampled keys, about 4096 keys in all.
//      With one run (T <= 131072) a key's place is its rank.
//   3. topk_merge_runs_kernel (T > 131072): adds, for each key of a sorted run, the
//      number of every other run's keys ordered before it.
//   4. topk_census_kernel: how many eligible tokens of each bucket of consecutive ranks
//      lie before each block of positions.
//   5. topk_query_kernel: one workgroup per 1024 consecutive queries. k is fixed and
//      the eligible set only grows, so while the block's new tokens arrive the cutoff
//      only walks down from where it stood before the block, past at most one kept
//      token per arrival. The census gives the bucket that holds the k-th rank before
//      the block; one scan of it finds that rank; a scan downwards from there to the
//      block's last cutoff lists its candidates (2048 at most) in rank order; and each
//      wave then answers its 64 queries from that list.
//   6. topk_evict_kernel: each token's first query with a cutoff below its rank.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "kvpop.h"
#include "kvpop_internal.h"

namespace kvpop {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kSortJ = 4;                      // elements per thread
constexpr int kRankChunk = kSortJ * kThreads;  // positions per sorted chunk
constexpr int kRunChunks = 32;                 // most sorted chunks per run
constexpr int kRun = kRunChunks * kRankChunk;  // positions per run: 131072
constexpr int kBlock = 1024;                   // queries per workgroup, ranks per scan step
constexpr int kMaxBuckets = 1024;              // most rank buckets (and position blocks) of the census

// Monotone map from float to uint32 such that larger floats give larger keys;
// inverted so that an ascending sort puts the highest priority first. -0.0 and
// +0.0 compare equal as numbers, so both map to the key of +0.0.
__device__ __forceinline__ uint32_t desc_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  const uint32_t asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ~asc;
}

// fl(r - fl(t * lg)): two roundings, never fused into one fma, so that the ranking
// decided by these values is reproducible from their float32 definition.
__device__ __forceinline__ float static_priority(float r, float t, float lg) {
#pragma clang fp contract(off)
  const float d = t * lg;
  return r - d;
}

// Workgroup barrier after this wave's LDS operations have completed (lgkmcnt(0)),
// without waiting for its outstanding global accesses as __syncthreads() does: for
// barriers that only exchange LDS data.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt at their maxima
  asm volatile("s_barrier" ::: "memory");
}

// Between a wave's LDS writes and its other lanes' reads of them: a wave's LDS
// operations complete in order, so only the compiler has to keep them so.
__device__ __forceinline__ void wave_sync() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ int lanes_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive scan over the 64 lanes by DPP: four shifts within rows of 16 lanes, then
// the last lanes of earlier rows broadcast. `id` is the identity of the operation.
template <bool MAX>
__device__ __forceinline__ int wave_scan(int x) {
  constexpr int id = MAX ? INT32_MIN : 0;
  auto op = [](int a, int b) { return MAX ? max(a, b) : a + b; };
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x111, 0xF, 0xF, false));  // row_shr:1
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x112, 0xF, 0xF, false));  // row_shr:2
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x114, 0xF, 0xF, false));  // row_shr:4
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x118, 0xF, 0xF, false));  // row_shr:8
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x142, 0xA, 0xF, false));  // row_bcast:15 into rows 1, 3
  x = op(x, __builtin_amdgcn_update_dpp(id, x, 0x143, 0xC, 0xF, false));  // row_bcast:31 into rows 2, 3
  return x;
}

// Reduction over each row of 16 lanes, the result in all of them.
template <bool MAX>
__device__ __forceinline__ int row_reduce(int x) {
  auto op = [](int a, int b) { return MAX ? max(a, b) : a + b; };
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, false));  // row_ror:8
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, false));
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xF, 0xF, false));
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xF, 0xF, false));
  return x;
}

// Scratch of the block-wide exchanges below: two sets of per-wave values, used in
// turn, so that one barrier per exchange suffices (a wave that writes a set has passed
// the barrier after the last reads of it).
struct Exchange {
  int v[2][kWaves];
};

// Combines one value per wave over the block: `before` gets the reduction over the
// earlier waves, `total` over all of them. Every thread calls it.
template <bool MAX>
__device__ __forceinline__ void wave_totals(int mine, Exchange& ex, int& turn, int& before, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int* s = ex.v[turn & 1];
  ++turn;
  if (lane == 0) s[wave] = mine;
  lds_barrier();
  const int x = s[lane & (kWaves - 1)];
  total = __builtin_amdgcn_readfirstlane(row_reduce<MAX>(x));
  before = __builtin_amdgcn_readfirstlane(row_reduce<MAX>((lane & (kWaves - 1)) < wave ? x : (MAX ? INT32_MIN : 0)));
}

// Threads before this one (in thread order) with the flag set, and the block's total.
__device__ __forceinline__ int block_count(bool flag, Exchange& ex, int& turn, int& total) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(flag);
  int before;
  wave_totals<false>(__builtin_popcountll(m), ex, turn, before, total);
  return before + lanes_below(m);
}

// ---------------------------------------------------------------------------
// Workspace of one sequence
// ---------------------------------------------------------------------------
struct SegWork {
  uint32_t* ka;      // keys and positions of the sorted chunks
  uint32_t* va;
  uint32_t* kb;      // and of the sorted runs (T > kRun)
  uint32_t* vb;
  int32_t* ps;       // positions in rank order
  uint32_t* census;  // [blocks][buckets], see topk_census_kernel
};

__device__ __forceinline__ SegWork seg_work(void* ws, size_t per_seg_words, int seg, int T) {
  SegWork s;
  s.ka = reinterpret_cast<uint32_t*>(ws) + (size_t)seg * per_seg_words;
  s.kb = s.ka + T;
  s.va = s.kb + T;
  s.vb = s.va + T;
  s.ps = reinterpret_cast<int32_t*>(s.vb + T);
  s.census = reinterpret_cast<uint32_t*>(s.ps + T);
  return s;
}

// log2 of the ranks per census bucket, and of the positions per block: 10, or more
// where that would make over kMaxBuckets of them (T > 2^20).
__host__ __device__ inline int census_shift(int T) {
  int sh = 10;
  while (((T - 1) >> sh) >= kMaxBuckets) ++sh;
  return sh;
}
__host__ __device__ inline int census_buckets(int T) { return ((T - 1) >> census_shift(T)) + 1; }

// ---------------------------------------------------------------------------
// 1. Chunk sort
// ---------------------------------------------------------------------------
// LDS of the chunk sort, 76 KB with J = 4 elements per thread: two workgroups share a CU. Digit d's counters of a
// (slot, wave) row sit at slot(d) = 64 (d % 4) + d / 4, 16 waves side by side, so that
// the thread that sums digit 4 lane + e reads and writes whole 16-byte rows next to its
// neighbour lanes'.
template <int J>
struct SortSmem {
  alignas(16) uint8_t cnt[J][256][kWaves];         // elements of a digit per (slot, wave): at most 64
  alignas(16) uint16_t dst[J][256][kWaves];        // where the first of them goes
  alignas(16) int part[J][256];                    // per digit and slot
  alignas(16) uint32_t key[J * kThreads];
  alignas(16) uint16_t idx[J * kThreads];          // position within the chunk
  int census[J][J];
};

// One stable counting-sort pass on the 8-bit digit at `shift`. Thread tid holds the
// elements 1024 j + tid, j < J, before and after. An element goes to (elements with
// smaller digits) + (elements of its digit in earlier (j, wave) rows) + (earlier lanes
// of its wave with its digit, found with eight ballots). Bound by vector instructions,
// about 290 per wave: 7000 cycles per pass, 16.8 us for the whole sort of up to 256 chunks
// (28-31 us with a histogram by LDS atomics and one thread per digit's 64 counters).
template <int J>
__device__ __forceinline__ void sort_pass(uint32_t (&k)[J], uint32_t (&v)[J], int shift, SortSmem<J>& sm) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int row[J], rk[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint32_t d = (k[j] >> shift) & 255u;
    uint32_t lo = ~0u, hi = ~0u;  // lanes with the same digit
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      uint32_t own = (uint32_t)__builtin_amdgcn_sbfe((int)k[j], shift + b, 1);  // all ones if the bit is set
      asm("" : "+v"(own));
      const uint64_t bb = __builtin_amdgcn_ballot_w64((int)own < 0);
      // lo & ~(bb ^ own), one instruction per half
      lo = __builtin_amdgcn_bitop3_b32(lo, own, (uint32_t)bb, 0x90);
      hi = __builtin_amdgcn_bitop3_b32(hi, own, (uint32_t)(bb >> 32), 0x90);
    }
    rk[j] = (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    row[j] = (int)(64u * (d & 3u) + (d >> 2));
    if (rk[j] == 0) sm.cnt[j][row[j]][wave] = (uint8_t)(__popc(lo) + __popc(hi));
  }
  lds_barrier();
  // Thread (e, g, lane) owns digit 4 lane + e of slot g: e = wave % 4, g = wave / 4
  // (with J < 4 slots the last waves own none).
  const int e = wave & 3, g = wave >> 2, r = 64 * e + lane;
  uint32_t c[4] = {0u, 0u, 0u, 0u};
  if (g < J) {
    const uint4 c4 = *reinterpret_cast<const uint4*>(&sm.cnt[g][r][0]);
    *reinterpret_cast<uint4*>(&sm.cnt[g][r][0]) = uint4{0u, 0u, 0u, 0u};  // for the next pass
    c[0] = c4.x, c[1] = c4.y, c[2] = c4.z, c[3] = c4.w;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_sad_u8(c[i], 0u, sum);
    sm.part[g][4 * lane + e] = (int)sum;
  }
  lds_barrier();
  if (g < J) {
    int p[J][4], tot = 0;
#pragma unroll
    for (int i = 0; i < J; ++i) {
      const int4 x = *reinterpret_cast<const int4*>(&sm.part[i][4 * lane]);
      p[i][0] = x.x, p[i][1] = x.y, p[i][2] = x.z, p[i][3] = x.w;
      tot += x.x + x.y + x.z + x.w;
    }
    int at = wave_scan<false>(tot) - tot;  // elements with digits below 4 lane
#pragma unroll
    for (int i = 0; i < J; ++i)
#pragma unroll
      for (int f = 0; f < 4; ++f)
        if (f < e || (f == e && i < g)) at += p[i][f];
    uint32_t out[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t a = (uint32_t)at;
      at += (int)((c[i >> 1] >> (16 * (i & 1))) & 255u);
      out[i] = a | ((uint32_t)at << 16);
      at += (int)((c[i >> 1] >> (16 * (i & 1) + 8)) & 255u);
    }
    *reinterpret_cast<uint4*>(&sm.dst[g][r][0]) = uint4{out[0], out[1], out[2], out[3]};
    *reinterpret_cast<uint4*>(&sm.dst[g][r][8]) = uint4{out[4], out[5], out[6], out[7]};
  }
  lds_barrier();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int d = (int)sm.dst[j][row[j]][wave] + rk[j];
    sm.key[d] = k[j];
    sm.idx[d] = (uint16_t)v[j];
  }
  lds_barrier();
#pragma unroll
  for (int j = 0; j < J; ++j) {
    k[j] = sm.key[j * kThreads + tid];
    v[j] = sm.idx[j * kThreads + tid];
  }
}

// One workgroup per (sequence, chunk of 1024 J positions): J = 4, or fewer for a sequence
// that fits one chunk of them (J = 1: 6.1-6.8 us, J = 2: 9.6, J = 4: 15.6-17.5). Positions past T sort
// last: they have the largest key and enter last. With a single chunk the sorted order
// is the ranking: the kernel then writes the ranks, the positions in rank order and the
// census itself.
template <int J>
__global__ __launch_bounds__(kThreads) void topk_chunk_sort_kernel(const float* __restrict__ scores,
                                                                   const float* __restrict__ log_gamma, int nseg, int H,
                                                                   int T, int s, void* ws, size_t per_seg_words,
                                                                   int32_t* __restrict__ rank) {
  __shared__ SortSmem<J> sm;
  const int tid = threadIdx.x, lane = tid & 63;
  constexpr int kChunk = J * kThreads;
  const int nch = (T + kChunk - 1) / kChunk;
  const int c = (int)blockIdx.x / nseg, seg = (int)blockIdx.x - c * nseg;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const float lg = log_gamma ? log_gamma[seg % H] : 0.f;
  const float* r = scores + (size_t)seg * T;
  const int t0 = c * kChunk, n = min(kChunk, T - t0);

  uint32_t k[J], v[J];
  float x[J];
#pragma unroll
  for (int j = 0; j < J; ++j) x[j] = r[min(t0 + j * kThreads + tid, T - 1)];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = j * kThreads + tid;
    asm volatile("" : "+v"(x[j]));  // the loads stay together, not each in a branch of its own
    k[j] = i < n ? desc_key(static_priority(x[j], (float)(t0 + i), lg)) : ~0u;
    v[j] = (uint32_t)i;
  }
  if (tid < J * 256) reinterpret_cast<uint4*>(sm.cnt)[tid] = uint4{0u, 0u, 0u, 0u};
  if (tid < J * J) (&sm.census[0][0])[tid] = 0;
  lds_barrier();
  sort_pass<J>(k, v, 0, sm);
  sort_pass<J>(k, v, 8, sm);
  sort_pass<J>(k, v, 16, sm);
  sort_pass<J>(k, v, 24, sm);
  if (nch > 1) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int i = j * kThreads + tid;
      if (i < n) {
        w.ka[t0 + i] = k[j];
        w.va[t0 + i] = (uint32_t)t0 + v[j];
      }
    }
    return;
  }
  // census[block][bucket], see topk_census_kernel: slot j holds bucket j's ranks.
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = j * kThreads + tid, t = (int)v[j];
    if (i < n) {
      rank[(size_t)seg * T + t] = i;
      w.ps[i] = t;
    }
#pragma unroll
    for (int b = 1; b < J; ++b) {
      const int cb = __builtin_popcountll(__builtin_amdgcn_ballot_w64(i < n && t >= s && t < b * kBlock));
      if (lane == 0 && cb) atomicAdd(&sm.census[b][j], cb);
    }
  }
  lds_barrier();
  const int nb = census_buckets(T);
  if (tid < J * J) {
    const int blk = tid / J, b = tid - blk * J;
    if (blk < nb && b < nb) w.census[blk * nb + b] = (uint32_t)sm.census[blk][b];
  }
}

// ---------------------------------------------------------------------------
// 2, 3. Merges
// ---------------------------------------------------------------------------
// For four ascending keys, the number of entries of the sorted array B[0, len) in LDS
// ordered before each: those below it, and with LE (entries of earlier positions) those
// equal to it too. The first key is searched over the whole array; the others only up
// to the next thread's first key, a few entries away. near: LDS for the first keys'
// results. Every thread of the block calls it.
template <bool LE>
__device__ __forceinline__ void count_before(const uint32_t* __restrict__ B, int len,
                                             const uint32_t (&key)[kSortJ], int (&at)[kSortJ], int* near) {
  const int tid = threadIdx.x;
  auto before = [&](uint32_t x, uint32_t y) { return LE ? x <= y : x < y; };
  int lo = 0;
  for (int step = len > 0 ? 1 << (31 - __builtin_clz(len)) : 0; step > 0; step >>= 1) {
    const int np = lo + step;
    lo = np <= len && before(B[min(np, len) - 1], key[0]) ? np : lo;
  }
  near[tid] = lo;
  lds_barrier();
  const int hi = tid + 1 < kThreads ? near[tid + 1] : len;
  at[0] = lo;
  int l[kSortJ], m[kSortJ];
#pragma unroll
  for (int j = 1; j < kSortJ; ++j) {
    l[j] = lo;
    m[j] = hi - lo;
  }
  while (__builtin_amdgcn_ballot_w64((m[1] | m[2] | m[3]) > 0) != 0) {
#pragma unroll
    for (int j = 1; j < kSortJ; ++j) {
      const int half = m[j] >> 1;
      const bool some = m[j] > 0;
      const bool b = some && before(B[some ? l[j] + half : 0], key[j]);
      l[j] = b ? l[j] + half + 1 : l[j];
      m[j] = b ? m[j] - half - 1 : half;
    }
  }
#pragma unroll
  for (int j = 1; j < kSortJ; ++j) at[j] = l[j];
  lds_barrier();  // near is free again
}

constexpr int kGap = 128;                      // a sample of a sorted chunk is every 128th key
constexpr int kSamples = kRankChunk / kGap;    // per chunk
constexpr int kMergeCap = kRankChunk + kRunChunks * kGap;  // keys between two splitters: fewer, see topk_merge_kernel

// Merges neighbouring lists pairwise, in LDS: with n lists at off[i << shift] .. off[(i +
// 1) << shift], lists 2 i and 2 i + 1 become one, equal keys of list 2 i first. Each
// thread writes `per` consecutive outputs: it finds where they start in the two lists by
// a binary search along the merge path, then takes the smaller head each time.
__device__ __forceinline__ void merge_level(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                            uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, const int* off,
                                            int shift, int npairs, int total, int per) {
  int e = (int)threadIdx.x * per;
  const int end = min(e + per, total);
  if (e >= end) return;
  int i = 0;  // the pair that output e belongs to
  for (int step = npairs >> 1; step > 0; step >>= 1)
    if (off[(i + step) << (shift + 1)] <= e) i += step;
  const int a0 = off[i << (shift + 1)];
  int a1 = off[(2 * i + 1) << shift], b1 = off[(i + 1) << (shift + 1)];
  const int d = e - a0;
  int lo = max(0, d - (b1 - a1)), hi = min(d, a1 - a0);
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    const bool first = kin[a0 + mid] <= kin[a1 + d - 1 - mid];
    lo = first ? mid + 1 : lo;
    hi = first ? hi : mid;
  }
  int a = a0 + lo, b = a1 + d - lo;
  // Heads of both lists and the keys behind them, so that no step waits for the read it
  // issues.
  auto at = [&](int i) __attribute__((always_inline)) { return kin[min(i, total - 1)]; };
  uint32_t ka = at(a), ka1 = at(a + 1), kb = at(b), kb1 = at(b + 1);
  for (; e < end; ++e) {
    while (a == a1 && b == b1) {  // on to the next pair that is not empty
      ++i;
      a = b1;
      a1 = b = off[(2 * i + 1) << shift];
      b1 = off[(i + 1) << (shift + 1)];
      ka = at(a), ka1 = at(a + 1), kb = at(b), kb1 = at(b + 1);
    }
    const bool first = a < a1 && (b >= b1 || ka <= kb);
    kout[e] = first ? ka : kb;
    vout[e] = vin[first ? a : b];
    a += first ? 1 : 0;
    b += first ? 0 : 1;
    const uint32_t next = at((first ? a : b) + 1);
    ka = first ? ka1 : ka;
    kb = first ? kb : kb1;
    ka1 = first ? next : ka1;
    kb1 = first ? kb1 : next;
  }
}

// One workgroup per (sequence, chunk): as many workgroups as chunks share a run's keys
// evenly. The run's samples (every kGap-th key of each chunk) are merged, in key order with
// ties to the earlier chunk, and workgroup b of nc takes the keys from the sample b / nc of
// the way up to the one (b + 1) / nc of the way. That is at most kSamples samples, so at
// most kRankChunk keys and kGap - 1 more per chunk: under kMergeCap. Where a splitter falls
// in a chunk is known to within the keys between two samples, which one wave reads. The
// stretches are gathered in LDS in chunk order and merged pairwise; equal keys keep the
// chunks' order, so ties go to the earlier position. FINAL (the only run): places are
// ranks, written with the positions in rank order. Otherwise the run's keys and positions
// go to its sorted arrays.
// Bound by the LDS latency of the merge levels (a search and about five outputs per
// thread and level), then by the scattered writes of the ranks: 20.2 us for 4 x 8 x 32768,
// 29.0 us for 1 x 8 x 131072 (27 and about 120 us when every key was searched in every
// other chunk).
template <bool FINAL>
__global__ __launch_bounds__(kThreads) void topk_merge_kernel(int nseg, int T, void* ws, size_t per_seg_words,
                                                                   int32_t* __restrict__ rank) {
  __shared__ uint32_t key[2][kMergeCap], pos[2][kMergeCap];
  __shared__ int off[kRunChunks + 1];
  __shared__ int wlo[2 * kRunChunks], wlen[2 * kRunChunks];  // window of a boundary; its first entry and length
  __shared__ uint32_t wkey[2 * kRunChunks];
  __shared__ int bound[2 * kRunChunks];                      // boundaries of chunk c's stretch: 2 c, 2 c + 1
  __shared__ int totals[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nch = (T + kRankChunk - 1) / kRankChunk;
  const int c0 = (int)blockIdx.x / nseg, seg = (int)blockIdx.x - c0 * nseg;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const int run = c0 / kRunChunks, b = c0 - run * kRunChunks;
  const int r0 = run * kRun, n = min(kRun, T - r0);
  const int nc = (n + kRankChunk - 1) / kRankChunk;
  int lg = 0;  // lists: a power of two, the last ones empty
  while ((1 << lg) < nc) ++lg;
  const int P = 1 << lg;
  const uint32_t* ka = w.ka + r0;
  const uint32_t* va = w.va + r0;

  // Samples: [0] keeps them chunk by chunk, the merges alternate between 1 and 2.
  constexpr int kMost = kRunChunks * kSamples;
  static_assert(kMost <= kThreads, "one sample per thread");
  uint32_t(*sk)[kMost] = reinterpret_cast<uint32_t(*)[kMost]>(&key[0][0]);
  uint32_t(*sv)[kMost] = reinterpret_cast<uint32_t(*)[kMost]>(&pos[0][0]);
  const int ns = P * kSamples;
  if (tid < ns) {
    const int i = tid * kGap;
    const uint32_t x = ka[min(i, n - 1)];
    sk[0][tid] = i < n ? x : ~0u;
    sv[0][tid] = (uint32_t)tid;
  }
  if (tid <= P) off[tid] = tid * kSamples;
  lds_barrier();
  int cur = 0;
  for (int l = 0; l < lg; ++l) {
    const int nxt = cur == 1 ? 2 : 1;
    merge_level(sk[cur], sv[cur], sk[nxt], sv[nxt], off, l, P >> (l + 1), ns, 1);
    cur = nxt;
    lds_barrier();
  }
  // Where the two splitters fall in each chunk: thread 2 c + e, e = 0 the lower one.
  const int nsamp = (n + kGap - 1) / kGap;
  if (tid < 2 * P) {
    const int c = tid >> 1, e = tid & 1;
    const int m = min(kRankChunk, max(0, n - c * kRankChunk));  // keys of the chunk
    int lo, len = 0;
    uint32_t kk = 0;
    if (e == 0 && b == 0) {
      lo = 0;
    } else if (e == 1 && b == nc - 1) {
      lo = m;
    } else {
      const int id = (int)sv[cur][(int)((long long)(b + e) * nsamp / nc)];
      const int g = id / kSamples;
      kk = sk[0][id];
      if (c == g) {
        lo = (id - g * kSamples) * kGap;
      } else {
        int x = 0;  // the chunk's samples before the splitter
        for (int step = kSamples; step > 0; step >>= 1) {
          const int np = x + step;
          const uint32_t y = sk[0][c * kSamples + min(np, kSamples) - 1];
          x = np <= kSamples && (c < g ? y <= kk : y < kk) ? np : x;
        }
        // (the padding of a partial or missing chunk is never before: such a chunk is a
        // later one than g, and no key is above it)
        lo = x > 0 ? (x - 1) * kGap + 1 : 0;
        len = x > 0 ? min(x * kGap, m) - lo : 0;
        len |= c < g ? 1 << 30 : 0;  // equal keys are before the splitter too
      }
    }
    wlo[tid] = lo;
    wlen[tid] = len;
    wkey[tid] = kk;
  }
  lds_barrier();
  {
    // A window has at most kGap - 1 entries: two per lane, all windows' reads in flight.
    static_assert(kGap <= 128, "two entries per lane");
    constexpr int U = 2 * kRunChunks / kWaves;
    uint32_t x[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = wave + u * kWaves;
      if (i < 2 * nc) {
        const int lo = wlo[i], len = wlen[i] & 0xFFFF;
        const uint32_t* p = ka + (i >> 1) * kRankChunk + lo;
        x[u][0] = lane < len ? p[lane] : 0u;
        x[u][1] = lane + 64 < len ? p[lane + 64] : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = wave + u * kWaves;
      if (i < 2 * nc) {
        const int len = wlen[i] & 0xFFFF;
        const bool le = wlen[i] >> 30;
        const uint32_t kk = wkey[i];
        const bool b0 = lane < len && (le ? x[u][0] <= kk : x[u][0] < kk);
        const bool b1 = lane + 64 < len && (le ? x[u][1] <= kk : x[u][1] < kk);
        const int cnt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(b0)) +
                        __builtin_popcountll(__builtin_amdgcn_ballot_w64(b1));
        if (lane == 0) bound[i] = wlo[i] + cnt;
      }
    }
  }
  lds_barrier();
  if (wave == 0) {
    const bool some = lane < nc;
    const int lo = some ? bound[2 * min(lane, nc - 1)] : 0, hi = some ? bound[2 * min(lane, nc - 1) + 1] : 0;
    const int incl = wave_scan<false>(hi - lo), before = wave_scan<false>(lo);
    if (lane < P) off[lane + 1] = incl;
    if (lane == 0) off[0] = 0;
    if (lane == 63) {
      totals[0] = incl;
      totals[1] = before;
    }
  }
  lds_barrier();
  const int total = totals[0], base = totals[1];
  for (int e = tid; e < total; e += kThreads) {
    int c = 0;
    for (int step = P >> 1; step > 0; step >>= 1)
      if (off[c + step] <= e) c += step;
    const int i = c * kRankChunk + bound[2 * c] + e - off[c];
    key[0][e] = ka[i];
    pos[0][e] = va[i];
  }
  lds_barrier();
  const int per = (total + kThreads - 1) / kThreads | 1;  // odd: the threads' outputs spread over the banks
  cur = 0;
  for (int l = 0; l < lg; ++l) {
    merge_level(key[cur], pos[cur], key[cur ^ 1], pos[cur ^ 1], off, l, P >> (l + 1), total, per);
    cur ^= 1;
    lds_barrier();
  }
  for (int e = tid; e < total; e += kThreads) {
    const int t = (int)pos[cur][e];
    if (FINAL) {
      rank[(size_t)seg * T + t] = base + e;
      w.ps[base + e] = t;
    } else {
      w.kb[r0 + base + e] = key[cur][e];
      w.vb[r0 + base + e] = (uint32_t)t;
    }
  }
}

// First entry of the sorted array B[0, n) in global memory that is not ordered before
// `key`, by one wave: 64 samples at a time, so three dependent reads for a run.
template <bool LE>
__device__ __forceinline__ int wave_lower(const uint32_t* __restrict__ B, int n, uint32_t key) {
  const int lane = threadIdx.x & 63;
  int lo = 0;
  while (n > 0) {  // the answer is in [lo, lo + n]
    const int step = (n + 63) >> 6;
    const int i = lane * step;  // entries lo, lo + step, ...
    const uint32_t x = B[lo + min(i, n - 1)];
    const bool before = i < n && (LE ? x <= key : x < key);
    const int m = __builtin_popcountll(__builtin_amdgcn_ballot_w64(before));  // samples before the key
    if (m == 0) return lo;
    lo += (m - 1) * step + 1;  // past the last of them
    n = min(step - 1, n - ((m - 1) * step + 1));
  }
  return lo;
}

// One workgroup per (sequence, run, kRankChunk consecutive keys of the sorted run): adds,
// for every other run, the number of its keys ordered before each (equal ones too if the
// run is an earlier one), which gives the ranks. The workgroup's first and last key bound
// the stretch of the other run to search: about kRankChunk keys where the runs are alike,
// none or all of them where one lies wholly past the other.
__global__ __launch_bounds__(kThreads) void topk_merge_runs_kernel(int nseg, int T, void* ws, size_t per_seg_words,
                                                                   int32_t* __restrict__ rank) {
  constexpr int kMaxRuns = (1 << 24) / kRun;
  constexpr int kPiece = 32768;  // keys of another run in LDS at a time
  __shared__ uint32_t stretch[kPiece];
  __shared__ int near[kThreads];
  __shared__ int from[kMaxRuns], to[kMaxRuns];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nch = (T + kRankChunk - 1) / kRankChunk, nr = (T + kRun - 1) / kRun;
  const int c = (int)blockIdx.x / nseg, seg = (int)blockIdx.x - c * nseg;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const int own = c / kRunChunks;
  const int i0 = c * kRankChunk, n = min(kRankChunk, T - i0);  // entries of the sorted runs
  uint32_t key[kSortJ];
  int rk[kSortJ];
#pragma unroll
  for (int j = 0; j < kSortJ; ++j) {
    const int i = kSortJ * tid + j;
    key[j] = w.kb[i0 + min(i, n - 1)];
    rk[j] = i0 - own * kRun + i;
  }
  const uint32_t first = w.kb[i0], last = w.kb[i0 + n - 1];
  for (int g = wave; g < nr; g += kWaves) {
    if (g == own) continue;
    const uint32_t* B = w.kb + (size_t)g * kRun;
    const int m = min(kRun, T - g * kRun);
    const int a = g < own ? wave_lower<true>(B, m, first) : wave_lower<false>(B, m, first);
    const int b = g < own ? wave_lower<true>(B, m, last) : wave_lower<false>(B, m, last);
    if ((tid & 63) == 0) {
      from[g] = a;
      to[g] = b;
    }
  }
  lds_barrier();
  for (int g = 0; g < nr; ++g) {
    if (g == own) continue;
    const int a = __builtin_amdgcn_readfirstlane(from[g]), z = __builtin_amdgcn_readfirstlane(to[g]);
#pragma unroll
    for (int j = 0; j < kSortJ; ++j) rk[j] += a;
    for (int p = a; p < z; p += kPiece) {
      const uint32_t* B = w.kb + (size_t)g * kRun + p;
      const int len = min(kPiece, z - p);
      for (int i = tid; i < len; i += 8 * kThreads) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = B[min(i + u * kThreads, len - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (i + u * kThreads < len) stretch[i + u * kThreads] = x[u];
      }
      lds_barrier();
      int at[kSortJ];
      if (g < own) count_before<true>(stretch, len, key, at, near);
      else count_before<false>(stretch, len, key, at, near);  // ends with a barrier: stretch is free
#pragma unroll
      for (int j = 0; j < kSortJ; ++j) rk[j] += at[j];
    }
  }
#pragma unroll
  for (int j = 0; j < kSortJ; ++j) {
    const int i = kSortJ * tid + j;
    if (i < n) {
      const int t = (int)w.vb[i0 + i];
      rank[(size_t)seg * T + t] = rk[j];
      w.ps[rk[j]] = t;
    }
  }
}

// ---------------------------------------------------------------------------
// 4. Census
// ---------------------------------------------------------------------------
// census[block][bucket] = eligible tokens (t >= s) whose rank lies in the bucket (2^shift
// consecutive ranks) and whose position lies before the block (2^shift positions).
// A workgroup counts max(4096, 2^shift) consecutive ranks: each token adds one to its
// (bucket, block) counter in LDS, and one wave per bucket sums the counters.
__global__ __launch_bounds__(kThreads) void topk_census_kernel(int nseg, int T, int s, void* ws, size_t per_seg_words) {
  __shared__ int cnt[kSortJ * kMaxBuckets];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sh = census_shift(T), nb = census_buckets(T);
  const int per = max(kRankChunk, 1 << sh);  // ranks per workgroup
  const int g = (int)blockIdx.x / nseg, seg = (int)blockIdx.x - g * nseg;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const int r0 = g * per, r1 = min(T, r0 + per);
  const int b0 = r0 >> sh, rows = ((r1 - 1) >> sh) - b0 + 1;  // at most kSortJ buckets
  for (int i = tid; i < rows * nb; i += kThreads) cnt[i] = 0;
  lds_barrier();
  for (int i = r0 + tid; i < r1; i += kRankChunk) {
    int t[kSortJ];
#pragma unroll
    for (int j = 0; j < kSortJ; ++j) t[j] = w.ps[min(i + j * kThreads, T - 1)];
#pragma unroll
    for (int j = 0; j < kSortJ; ++j) {
      const int r = i + j * kThreads;
      if (r < r1 && t[j] >= s) atomicAdd(&cnt[((r >> sh) - b0) * nb + (t[j] >> sh)], 1);
    }
  }
  lds_barrier();
  if (wave < rows) {
    int run = 0;
    for (int p = 0; p < nb; p += 64) {
      const int i = p + lane;
      const int x = i < nb ? cnt[wave * nb + i] : 0;
      const int incl = wave_scan<false>(x);
      if (i < nb) w.census[(size_t)i * nb + b0 + wave] = (uint32_t)(run + incl - x);
      run += __builtin_amdgcn_readlane(incl, 63);
    }
  }
}

// ---------------------------------------------------------------------------
// 5. Queries
// ---------------------------------------------------------------------------
// A block of queries adds at most kBlock tokens, so its last cutoff is within the kBlock + 1
// largest ranks below the cutoff before it, and the earlier ones are not below it; the scan
// that lists these ranks stops at a multiple of kBlock ranks, with at most kBlock entries
// more than the kBlock it may hold before its last step.
constexpr int kMaxCand = 2 * kBlock;
constexpr int kMaxLocal = 192;  // a wave's own candidates: 64 + 64 kept, 64 new

struct QuerySmem {
  Exchange ex;
  int cnt[kMaxBuckets];         // census remainder (T > 2^20)
  int found[3];
  uint32_t cand[kMaxCand];      // candidate ranks, descending
  uint16_t tag[kMaxCand];       // 0: kept before the block, else 1 + its place in the block
  uint32_t local[kWaves][kMaxLocal];  // (rank << 7) | (0: kept before the wave's queries, else 1 + lane)
  uint8_t place[kWaves][64];          // a lane's token's place in the wave's list, or 255
};

// The cutoffs of a wave's 64 queries from its list of n <= 32 W candidates: lane j's is
// the want-th of those present at its query, which are the candidates kept before and
// the tokens of lanes 0 .. j. Each lane builds the bitmap of the candidates present (an or
// over the earlier lanes' tokens) and selects the want-th set bit.
template <int W>
__device__ __forceinline__ int local_cutoff(const uint32_t* local, uint8_t* place, int n, int want) {
  const int lane = threadIdx.x & 63;
  place[lane] = 255;
  wave_sync();
  uint32_t here[W];
#pragma unroll
  for (int u = 0; u < W / 2; ++u) {
    const int i = 64 * u + lane;
    const int tg = i < n ? (int)(local[i] & 127u) : 127;
    const uint64_t mb = __builtin_amdgcn_ballot_w64(tg == 0);
    here[2 * u] = (uint32_t)mb;
    here[2 * u + 1] = (uint32_t)(mb >> 32);
    if (tg >= 1 && tg <= 64) place[tg - 1] = (uint8_t)i;
  }
  wave_sync();
  const int mine = (int)place[lane];
#pragma unroll
  for (int u = 0; u < W; ++u) {
    int x = (mine >> 5) == u ? 1 << (mine & 31) : 0;
    x |= __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);
    x |= __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x |= __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x |= __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x |= __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x |= __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    here[u] |= (uint32_t)x;
  }
  uint32_t sel = here[0];
  int at = 0;
#pragma unroll
  for (int u = 0; u + 1 < W; ++u) {
    const int c = __popc(here[u]);
    const bool next = at == 32 * u && want > c;
    want -= next ? c : 0;
    sel = next ? here[u + 1] : sel;
    at += next ? 32 : 0;
  }
#pragma unroll
  for (int half = 16; half > 0; half >>= 1) {
    const int c = __popc(sel & ((1u << half) - 1u));
    const bool next = want > c;
    want -= next ? c : 0;
    sel = next ? sel >> half : sel;
    at += next ? half : 0;
  }
  return (int)(local[at] >> 7);
}

// One workgroup per (sequence, kBlock consecutive new tokens t0 ..): the queries t + w.
// The first one also writes the queries before w, which have no eligible token.
// With p tokens eligible before the block, "old" are the eligible tokens before t0 and
// "new" those of the block; U is one above the k-th smallest old rank (T if p < k). Ranks
// from U on never matter again. Let D be the new tokens below U so far, less k - p
// if p < k: the cutoff is then the (D + 1)-th largest rank below U present.
// Bound by instruction issue once the chip is full (about 700 vector instructions per wave)
// and by the reads' latency below that: 20.5 us for 4 x 8 x 32768 (1024 workgroups), 7.4 us
// for 1 x 8 x 4096, against 224 and 42 us to build and walk a wavelet matrix. A block
// whose cutoff falls far reads those ranks one step of 1024 after the other: 53 us for 1 x 8 x
// 131072 live targets, where one block's cutoff falls by 115 steps, 21 for normal scores (38).
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(8, 8))) void
topk_query_kernel(int T, int s, int w_win, int k, void* ws, size_t per_seg_words,
                  const int32_t* __restrict__ ranks, int32_t* __restrict__ cutoff, int32_t* __restrict__ label,
                  int32_t* __restrict__ boundary) {
  __shared__ QuerySmem sm;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = (int)blockIdx.x, blk = (int)blockIdx.y;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const int32_t* rank = ranks + (size_t)seg * T;
  int32_t* cut_o = cutoff + (size_t)seg * T;
  int32_t* lab_o = label ? label + (size_t)seg * T : nullptr;
  int32_t* bnd_o = boundary ? boundary + (size_t)seg * T : nullptr;
  int turn = 0;

  if (blk == 0) {
    for (int q = tid; q < min(w_win, T); q += kThreads) {
      cut_o[q] = T;
      if (lab_o) lab_o[q] = 0;
      if (bnd_o) bnd_o[q] = -1;
    }
    if (w_win >= T) return;
  }
  const int t0 = blk * kBlock;
  const int tl = min(t0 + kBlock, T - w_win) - 1;  // last new token with a query
  const int t = t0 + tid;
  const bool active = t <= tl;
  const bool elig = active && t >= s;
  const int r = rank[min(t, tl)];
  const int q = t + w_win;
  const int p0 = max(t0 - s, 0);            // eligible before the block
  const int p = t - s + 1;                  // eligible at this thread's query (<= 0: none)
  const int p_last = tl - s + 1;
  int cut = T, bnd = -1;

  // The k-th smallest old rank, or the largest one if fewer than k are old. Before
  // saturation it is wanted for the boundary tokens only; up to kScanOld old tokens are then
  // scanned (a few reads in flight together, where the census takes four barriers), so that
  // a block's work does not grow with T for any k (8 x 4194304, k = T: 6.4 ms a call, 39
  // when every block scanned all its old tokens).
  constexpr int kScanOld = 4 * kBlock;
  const bool unsaturated = bnd_o && p_last >= 1 && p0 + 1 < k;  // at the block's first query
  int old_k = INT32_MIN;
  if (p0 >= k || (unsaturated && p0 > kScanOld)) {
    const int kth = min(k, p0);
    const int sh = census_shift(T), nb = census_buckets(T);
    int cb = tid < nb ? (int)w.census[(size_t)(t0 >> sh) * nb + tid] : 0;
    const int rest = (t0 >> sh) << sh;  // first position that the census does not count
    if (rest < t0) {                    // only where blocks are wider than kBlock
      sm.cnt[tid] = 0;
      lds_barrier();
      for (int i = max(rest, s) + tid; i < t0; i += kThreads) atomicAdd(&sm.cnt[rank[i] >> sh], 1);
      lds_barrier();
      cb += sm.cnt[tid];
    }
    // The bucket with the kth old rank: inclusive counts over the buckets.
    const int incl = wave_scan<false>(cb);
    int before, total;
    wave_totals<false>(__builtin_amdgcn_readlane(incl, 63), sm.ex, turn, before, total);
    const int upto = before + incl;
    if (upto >= kth && upto - cb < kth) {
      sm.found[0] = tid;
      sm.found[1] = kth - (upto - cb);  // its place among the bucket's old ranks, from 1
    }
    lds_barrier();
    int v0 = __builtin_amdgcn_readfirstlane(sm.found[0]) << sh;
    int kk = __builtin_amdgcn_readfirstlane(sm.found[1]);
    for (;;) {  // one round unless buckets are wider than kBlock
      const int v = v0 + tid;
      const int pos = v < T ? w.ps[v] : INT32_MAX;
      const bool old = pos >= s && pos < t0;
      int tot;
      const int at = block_count(old, sm.ex, turn, tot);
      if (old && at == kk - 1) sm.found[2] = v;
      if (kk <= tot || v0 + kThreads >= T) break;
      kk -= tot;
      v0 += kThreads;
    }
    lds_barrier();
    old_k = __builtin_amdgcn_readfirstlane(sm.found[2]);
  }

  // Before saturation every eligible token is kept: the boundary token is the one with
  // the largest rank.
  if (unsaturated) {
    int before, total;
    if (p0 <= kScanOld) {
      int old = INT32_MIN;
      for (int i = s + tid; i < t0; i += kThreads) old = max(old, rank[i]);
      wave_totals<true>(__builtin_amdgcn_readlane(wave_scan<true>(old), 63), sm.ex, turn, before, old_k);
    }
    const int incl = wave_scan<true>(elig ? r : INT32_MIN);
    wave_totals<true>(__builtin_amdgcn_readlane(incl, 63), sm.ex, turn, before, total);
    const int mx = max(old_k, max(before, incl));
    if (elig && p < k) bnd = w.ps[mx];
  }

  if (p_last >= k) {
    // U, and D before the block.
    const int U = p0 >= k ? old_k + 1 : T, D0 = p0 >= k ? 0 : p0 - k;
    // New tokens below U.
    const bool in = elig && r < U;
    const uint64_t inm = __builtin_amdgcn_ballot_w64(in);
    int before, m;
    wave_totals<false>(__builtin_popcountll(inm), sm.ex, turn, before, m);
    if (m == 0) {  // p0 >= k here: the cutoff stays
      cut = U - 1;
    } else {
      // Candidates: old and new ranks below U, descending, until D0 + m + 1 are listed. At
      // the block's last query all of them are present, so the last one is its cutoff, and
      // no cutoff of the block is below it (at least that many exist: k + m old and new ones
      // once p0 >= k, p0 + m before). The blocks' scans do not overlap, so a sequence costs
      // at most T / 1024 steps and one more per block, for any k.
      const int need = D0 + m + 1;
      int nc = 0;
      int v = U - 1 - tid;
      int pos = v >= 0 ? w.ps[v] : -1;
      for (int top = U; top > 0 && nc < need; top -= kThreads) {
        const int pv = v, pp = pos;
        v -= kThreads;
        pos = v >= 0 ? w.ps[v] : -1;  // the next step's, in flight during this one
        const bool old = pp >= s && pp < t0;
        const bool keep = old || (pp >= max(s, t0) && pp <= tl);
        int tot;
        const int at = block_count(keep, sm.ex, turn, tot);
        if (keep) {
          const int i = nc + at;
          sm.cand[i] = (uint32_t)pv;
          sm.tag[i] = (uint16_t)(old ? 0 : pp - t0 + 1);
        }
        nc += tot;
      }
      lds_barrier();
      // This wave's queries: D before them, and the place i0 of the cutoff there (the
      // list's start before saturation).
      const int D = D0 + before;
      const int lo_tag = 64 * wave;  // tags up to this are present before the wave's queries
      int i0 = 0, want;              // want: place of this lane's cutoff among those present from i0 on, from 1
      if (D >= 0) {
        int seen = 0;
        bool hit = false;
        for (int i = 0; i < nc && !hit; i += 256) {
          uint64_t mb[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = i + 64 * u + lane;
            mb[u] = __builtin_amdgcn_ballot_w64(e < nc && (int)sm.tag[min(e, nc - 1)] <= lo_tag);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int c = __builtin_popcountll(mb[u]);
            if (!hit && seen + c > D) {
              hit = true;
              const uint64_t at =
                  __builtin_amdgcn_ballot_w64(((mb[u] >> lane) & 1) && lanes_below(mb[u]) == D - seen);
              i0 = i + 64 * u + __builtin_ctzll(at);
            }
            seen += c;
          }
        }
      }
      const int c0 = (int)sm.cand[i0];
      // The wave's own tokens that lower the cutoff: those below it.
      const uint64_t f = __builtin_amdgcn_ballot_w64(in && (D < 0 || r < c0));
      const int own = lanes_below(f) + (int)((f >> lane) & 1);  // up to and with this lane's
      want = D < 0 ? D + own + 1 : own + 1;
      const int most = D < 0 ? D + __builtin_popcountll(f) + 1 : __builtin_popcountll(f) + 1;
      cut = D < 0 ? T : c0;
      if (most > (D < 0 ? 0 : 1)) {
        int n = 0, kept = 0;
        for (int i = i0 & ~63; i < nc && kept < most; i += 64) {
          const int e = min(i + lane, nc - 1);
          const int tg = (int)sm.tag[e];
          const bool ok = i + lane >= i0 && i + lane < nc;
          const bool base = ok && tg <= lo_tag;
          const bool mine = ok && tg > lo_tag && tg <= lo_tag + 64;
          const uint64_t mm = __builtin_amdgcn_ballot_w64(base || mine);
          if (base || mine)
            sm.local[wave][n + lanes_below(mm)] = sm.cand[e] << 7 | (uint32_t)(base ? 0 : tg - lo_tag);
          n += __builtin_popcountll(mm);
          kept += __builtin_popcountll(__builtin_amdgcn_ballot_w64(base));
        }
        wave_sync();
        const uint32_t* local = sm.local[wave];
        uint8_t* place = sm.place[wave];
        cut = n <= 64 ? local_cutoff<2>(local, place, n, want) : n <= 128 ? local_cutoff<4>(local, place, n, want)
                                                                          : local_cutoff<6>(local, place, n, want);
      }
    }
    if (p < k) cut = T;
    else if (bnd_o && active) bnd = w.ps[cut];
  }
  if (active) {
    cut_o[q] = cut;
    if (lab_o) lab_o[q] = p < 1 ? 0 : (r <= cut ? 1 : -1);
    if (bnd_o) bnd_o[q] = bnd;
  }
}

// ---------------------------------------------------------------------------
// 6. Evictions
// ---------------------------------------------------------------------------
// One workgroup per (sequence, kRankChunk consecutive ranks): the query at which each of
// their tokens leaves the mask. The cutoff never increases with q, so the queries whose
// cutoff lies among the workgroup's ranks are consecutive: two rounds of 1024 samples find
// them. Each notes the first query of its cutoff in LDS, and a rank's first query with a
// smaller cutoff is the least one noted below it (a minimum scan in rank order), or the
// first query past the range. Bound by the latency of the samples' reads and of the
// scattered writes: 9.7 us for 4 x 8 x 32768 (15 us with a binary search over the cutoffs
// per token).
__global__ __launch_bounds__(kThreads) void topk_evict_kernel(int nseg, int T, int s, int w_win, void* ws,
                                                              size_t per_seg_words, const int32_t* __restrict__ cutoff,
                                                              int32_t* __restrict__ evict) {
  __shared__ alignas(16) int first[kRankChunk];
  __shared__ Exchange ex;
  int turn = 0;
  const int tid = threadIdx.x;
  const int g = (int)blockIdx.x / nseg, seg = (int)blockIdx.x - g * nseg;
  SegWork w = seg_work(ws, per_seg_words, seg, T);
  const int32_t* cut = cutoff + (size_t)seg * T;
  const int r0 = g * kRankChunk, r1 = min(T, r0 + kRankChunk);
  int t[kSortJ];
#pragma unroll
  for (int j = 0; j < kSortJ; ++j) t[j] = w.ps[min(r0 + j * kThreads + tid, T - 1)];
  // qa, qb: first queries with a cutoff below r1 and below r0 (T if there is none).
  int qa = 0, qb = 0;
  {
    const int step = (T + kThreads - 1) / kThreads;  // 16384 at most
    const int x = cut[min(tid * step, T - 1)];
    const bool in = tid * step < T;
    int before, total;
    wave_totals<false>(__builtin_popcountll(__builtin_amdgcn_ballot_w64(in && x >= r1)) << 16 |
                           __builtin_popcountll(__builtin_amdgcn_ballot_w64(in && x >= r0)),
                       ex, turn, before, total);
    const int na = total >> 16, nb = total & 0xFFFF;  // samples not below
    // The answers lie past the last such sample, within `step` queries.
    const int ba = na ? (na - 1) * step + 1 : 0, la = na ? min(step - 1, T - ba) : 0;
    const int bb = nb ? (nb - 1) * step + 1 : 0, lb = nb ? min(step - 1, T - bb) : 0;
    int ca = 0, cb = 0;
    for (int i = tid; i < step; i += kThreads) {
      ca += i < la && cut[min(ba + i, T - 1)] >= r1;
      cb += i < lb && cut[min(bb + i, T - 1)] >= r0;
    }
    wave_totals<false>(__builtin_amdgcn_readlane(wave_scan<false>(ca), 63), ex, turn, before, total);
    qa = ba + total;
    wave_totals<false>(__builtin_amdgcn_readlane(wave_scan<false>(cb), 63), ex, turn, before, total);
    qb = bb + total;
  }
  reinterpret_cast<int4*>(first)[tid] = int4{INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
  lds_barrier();
  for (int q0 = qa; q0 < qb; q0 += kRankChunk) {
    int c[kSortJ], p[kSortJ];
#pragma unroll
    for (int j = 0; j < kSortJ; ++j) {
      const int q = min(q0 + j * kThreads + tid, qb - 1);
      c[j] = cut[q];
      p[j] = cut[max(q - 1, 0)];
    }
#pragma unroll
    for (int j = 0; j < kSortJ; ++j) {
      const int q = q0 + j * kThreads + tid;
      if (q < qb && (q == qa || c[j] != p[j])) first[c[j] - r0] = q;
    }
  }
  lds_barrier();
  // Exclusive minimum over the ranks before each of this thread's four, as a maximum of
  // the negated values.
  {
    const int4 f = reinterpret_cast<const int4*>(first)[tid];
    const int m0 = -f.x, m1 = max(m0, -f.y), m2 = max(m1, -f.z), m3 = max(m2, -f.w);
    const int incl = wave_scan<true>(m3);
    int before, total;
    wave_totals<true>(__builtin_amdgcn_readlane(incl, 63), ex, turn, before, total);
    const int prev = __builtin_amdgcn_update_dpp(INT32_MIN, incl, 0x138, 0xF, 0xF, false);  // wave_shr:1
    const int e = max(max(before, prev), -qb);
    reinterpret_cast<int4*>(first)[tid] = int4{-e, -max(e, m0), -max(e, m1), -max(e, m2)};
  }
  lds_barrier();
#pragma unroll
  for (int j = 0; j < kSortJ; ++j) {
    const int i = j * kThreads + tid;
    if (r0 + i < T) {
      const long long leave = (long long)t[j] + w_win;
      evict[(size_t)seg * T + t[j]] = t[j] < s ? T : (int)min((long long)T, max((long long)first[i], leave));
    }
  }
}

}  // namespace

static int topk_levels(int T) {
  int L = 1;
  while ((1 << L) < T) ++L;
  return L;
}

// A caller's workspace: the arrays of SegWork fit in it with room to spare for every T
// (5 T words and the census, at most 2^20 words and less than T where T < 2^20).
size_t topk_workspace_words_per_seq(int T) {
  const int L = topk_levels(T);
  const size_t W1 = (size_t)(T + 31) / 32 + 1;
  return 6 * (size_t)T + 2 * (size_t)L * W1 + (size_t)L + 4;
}

// Scratch of kvpop_running_topk_noalloc: the workspace of the ranking kernels in a
// file-scope device array instead of caller memory. Every GPU the library runs on
// holds its own copy until the process ends; all calls on one GPU share it.
static __device__ __align__(256) uint32_t scratch[KVPOP_NOALLOC_SCRATCH_BYTES / 4];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the device of `stream` (the current device for
// the null stream), resolved once per device with that device current. In host
// code the array's name is only a handle for the runtime, never an address.
int noalloc_scratch(void* stream, void** ptr) {
  int dev = 0;
  hipError_t e = stream ? hipStreamGetDevice((hipStream_t)stream, &dev) : hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = 0;
    e = hipGetDevice(&cur);
    if (e != hipSuccess) return (int)e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return (int)e;
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) {
      const hipError_t e2 = hipSetDevice(cur);
      if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return 0;
}

int launch_running_topk(const TopkLaunch& L) {
  const int nseg = L.B * L.H, T = L.T;
  const size_t per = topk_workspace_words_per_seq(T);
  hipStream_t st = (hipStream_t)L.stream;
  const unsigned chunks = (unsigned)((long long)nseg * ((T + kRankChunk - 1) / kRankChunk));
  const dim3 wg(kThreads);
  const auto sort = T <= kThreads       ? topk_chunk_sort_kernel<1>
                    : T <= 2 * kThreads ? topk_chunk_sort_kernel<2>
                                        : topk_chunk_sort_kernel<kSortJ>;
  hipLaunchKernelGGL(sort, dim3(chunks), wg, 0, st, L.scores, L.log_gamma, nseg, L.H, T, L.sinks, L.workspace, per,
                     L.rank);
  int e = (int)hipGetLastError();
  if (e) return e;
  if (T > kRankChunk) {
    if (T <= kRun) {
      hipLaunchKernelGGL(topk_merge_kernel<true>, dim3(chunks), wg, 0, st, nseg, T, L.workspace, per, L.rank);
    } else {
      hipLaunchKernelGGL(topk_merge_kernel<false>, dim3(chunks), wg, 0, st, nseg, T, L.workspace, per, L.rank);
      if ((e = (int)hipGetLastError())) return e;
      hipLaunchKernelGGL(topk_merge_runs_kernel, dim3(chunks), wg, 0, st, nseg, T, L.workspace, per, L.rank);
    }
    if ((e = (int)hipGetLastError())) return e;
    const int ranks = 1 << census_shift(T) > kRankChunk ? 1 << census_shift(T) : kRankChunk;
    hipLaunchKernelGGL(topk_census_kernel, dim3((unsigned)((long long)nseg * ((T + ranks - 1) / ranks))), wg, 0, st,
                       nseg, T, L.sinks, L.workspace, per);
    if ((e = (int)hipGetLastError())) return e;
  }
  // Query blocks along y (16384 at most): a dimension holds under 2^32 work-items, and a
  // longer one wraps without an error, which one of all blocks would from 2^21 sequences of
  // 1025 positions on.
  const int nqb = L.window >= T ? 1 : (T - L.window + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(topk_query_kernel, dim3((unsigned)nseg, (unsigned)nqb), wg, 0, st, T, L.sinks, L.window, L.topk,
                     L.workspace, per, L.rank, L.cutoff, L.label, L.boundary);
  if ((e = (int)hipGetLastError()) || !L.evict) return e;
  hipLaunchKernelGGL(topk_evict_kernel, dim3(chunks), wg, 0, st, nseg, T, L.sinks, L.window, L.workspace, per,
                     L.cutoff, L.evict);
  return (int)hipGetLastError();
}

}  // namespace kvpop
