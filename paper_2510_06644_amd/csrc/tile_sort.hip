// Step 2 of the forward pass (Sec. 2.1): each tile's list gathered from the
// binning chunks' runs and sorted by (depth, Gaussian index).
//
// A key is 64 bits, depth bits over index, and is compared as a double: depths
// are positive and at most infinity (float32), so the exponent field is below
// 0x7ff and the order of the doubles is the order of the keys; minimum and
// maximum are then one instruction each.  +infinity pads.
//
// A sort in LDS is bound by dependent round trips and barriers, so as much of
// it as possible runs in registers: a wave sorts 64 K keys (K per lane) by a
// bitonic network whose exchanges between lanes are lane swaps and DPP moves,
// without LDS; then log2(waves) merge levels join the waves' runs in one LDS
// buffer (each thread finds its K outputs on the merge path, keeps them in
// registers, and writes them back after a barrier).
//
// Measured, sorting only (both kernels), before (merge sort in LDS from runs of
// four keys, lists over 1024 keys in a second kernel of 1024 threads):
//   1200x680 / 300k (825 keys a tile)          50 -> 41 us
//   1200x680 / 500k (1370 keys a tile)        190 -> 59 us
//   1200x680 / 500k at 1 in 4 (about 4000)     98 -> 64 us
//   640x480 / 100k (550 keys a tile)           25 -> 19 us
// What is left is VALU issue (16.0M wave instructions at 1200x680 / 300k, 27 of
// 37 us in the first kernel) and, beside it, the gather's waits on the L2 for a line
// of run offsets and of keys per chunk and tile (47% of the wave cycles are waits).
#include "rtgs_internal.h"

namespace rtgs {
namespace {

__device__ __forceinline__ double key_pad() { return __longlong_as_double(0x7ff0000000000000ll); }

__device__ __forceinline__ void cas(double& a, double& b) {
  const double lo = __builtin_fmin(a, b), hi = __builtin_fmax(a, b);
  a = lo;
  b = hi;
}

// Sorting networks: 5 comparators for 4 keys, Batcher's 19 for 8.
__device__ __forceinline__ void sort_network(double (&k)[4]) {
  cas(k[0], k[1]); cas(k[2], k[3]);
  cas(k[0], k[2]); cas(k[1], k[3]);
  cas(k[1], k[2]);
}
__device__ __forceinline__ void sort_network(double (&k)[8]) {
  cas(k[0], k[1]); cas(k[2], k[3]); cas(k[4], k[5]); cas(k[6], k[7]);
  cas(k[0], k[2]); cas(k[1], k[3]); cas(k[4], k[6]); cas(k[5], k[7]);
  cas(k[1], k[2]); cas(k[5], k[6]);
  cas(k[0], k[4]); cas(k[1], k[5]); cas(k[2], k[6]); cas(k[3], k[7]);
  cas(k[2], k[4]); cas(k[3], k[5]);
  cas(k[1], k[2]); cas(k[3], k[4]); cas(k[5], k[6]);
}

// Position of a lane in the wave's sorted order, bit i of it flipped by the
// i-th of the lane exchanges 32, 16, 1, 2, 7, 8 (xor of the lane number, cheap
// ones first: bit i takes part in 6 - i levels).
__device__ __forceinline__ int lane_order(int lane) {
  const int b2 = (lane >> 2) & 1;
  return ((lane >> 5) & 1) | (((lane >> 4) & 1) << 1) | (((lane & 1) ^ b2) << 2) |
         ((((lane >> 1) & 1) ^ b2) << 3) | (b2 << 4) | (((lane >> 3) & 1) << 5);
}

__device__ __forceinline__ double as_double(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ unsigned lo_of(double v) {
  return (unsigned)(unsigned long long)__double_as_longlong(v);
}
__device__ __forceinline__ unsigned hi_of(double v) {
  return (unsigned)((unsigned long long)__double_as_longlong(v) >> 32);
}

// Swaps odd halves (32) or rows (16) of a with even ones of b: an involution.
template <int LANES>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
  unsigned l0, l1, h0, h1;
  if (LANES == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(lo_of(a), lo_of(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi_of(a), hi_of(b), false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(lo_of(a), lo_of(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi_of(a), hi_of(b), false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  }
  a = as_double(l0, h0);
  b = as_double(l1, h1);
}

// One compare-exchange of every key with the same key of the lane whose
// position differs in bit BIT (the lower position keeps the smaller).
template <int BIT, int K>
__device__ __forceinline__ void exchange(double (&k)[K], int order) {
  if (BIT <= 1) {
    // after the swap a lane holds both keys of a pair of lanes
#pragma unroll
    for (int s = 0; s < K; s += 2) {
      lane_swap<BIT == 0 ? 32 : 16>(k[s], k[s + 1]);
      cas(k[s], k[s + 1]);
      lane_swap<BIT == 0 ? 32 : 16>(k[s], k[s + 1]);
    }
  } else {
    // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_ror:8
    constexpr int kCtrl = BIT == 2 ? 0xB1 : BIT == 3 ? 0x4E : BIT == 4 ? 0x141 : 0x128;
    const bool upper = (order >> BIT) & 1;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const double o = as_double(
          (unsigned)__builtin_amdgcn_update_dpp(0, (int)lo_of(k[s]), kCtrl, 0xf, 0xf, true),
          (unsigned)__builtin_amdgcn_update_dpp(0, (int)hi_of(k[s]), kCtrl, 0xf, 0xf, true));
      k[s] = (k[s] < o) != upper ? k[s] : o;
    }
  }
}

// Sign bit flipped where `down`: the order reversed.
template <int K>
__device__ __forceinline__ void reverse_if(double (&k)[K], bool down) {
  const unsigned m = down ? 0x80000000u : 0u;
#pragma unroll
  for (int s = 0; s < K; ++s) k[s] = as_double(lo_of(k[s]), hi_of(k[s]) ^ m);
}

template <int K>
__device__ __forceinline__ void merge_in_lane(double (&k)[K]) {
#pragma unroll
  for (int m = K / 2; m >= 1; m >>= 1)
#pragma unroll
    for (int s = 0; s < K; ++s)
      if (!(s & m)) cas(k[s], k[s + m]);
}

// One bitonic level: exchanges of bits BIT .. 0, then within the lanes.
template <int BIT, int K>
__device__ __forceinline__ void merge_level(double (&k)[K], int order) {
  exchange<BIT, K>(k, order);
  if constexpr (BIT > 0)
    merge_level<BIT - 1, K>(k, order);
  else
    merge_in_lane(k);
}

// The wave's 64 K keys sorted: key s of the lane at position p of lane_order
// becomes element K p + s.  Blocks alternate in direction from level to level;
// a descending block holds its keys negated and is sorted as the others.
template <int K>
__device__ __forceinline__ void wave_sort(double (&k)[K], int order) {
  reverse_if(k, order & 1);
  sort_network(k);
  reverse_if(k, (order ^ (order >> 1)) & 1);
  merge_level<0, K>(k, order);
  reverse_if(k, ((order >> 1) ^ (order >> 2)) & 1);
  merge_level<1, K>(k, order);
  reverse_if(k, ((order >> 2) ^ (order >> 3)) & 1);
  merge_level<2, K>(k, order);
  reverse_if(k, ((order >> 3) ^ (order >> 4)) & 1);
  merge_level<3, K>(k, order);
  reverse_if(k, ((order >> 4) ^ (order >> 5)) & 1);
  merge_level<4, K>(k, order);
  reverse_if(k, (order >> 5) & 1);
  merge_level<5, K>(k, order);
}

// LDS position of key e of a sort buffer: one spare key after every eight, so
// that the threads' runs of K keys fall on different banks.
__device__ __forceinline__ int sp(int e) { return e + (e >> 3); }

// Keys a sort buffer of n keys holds with the spare ones.
constexpr int sort_buf_keys(int n) { return n + n / 8; }

// The workgroup's keys sorted: NT threads with K keys each in registers (list
// positions n and above are padding, and so is every key of a wave past the
// list), the ids written to ids[0..n).  buf: NT K keys of LDS.  All threads
// call it.
template <int NT, int K>
__device__ __forceinline__ void block_sort(double (&k)[K], int n, double* buf, uint32_t* ids) {
  constexpr int kRun = 64 * K;
  const int wave = threadIdx.x >> 6, order = lane_order(threadIdx.x & 63);
  const int pos = (wave * 64 + order) * K;          // first of this thread's K outputs
  const int runs = (n + kRun - 1) / kRun;           // waves with keys
  if (wave < runs) wave_sort(k, order);
  for (int L = kRun; L < runs * kRun; L <<= 1) {
    if (wave < runs) {
#pragma unroll
      for (int s = 0; s < K; ++s) buf[sp(pos + s)] = k[s];
    }
    __syncthreads();
    if (pos < n) {
      const int have = runs * kRun;                 // keys past these read as padding
      auto at = [&](int e) { return e < have ? buf[sp(e)] : key_pad(); };
      const int base = pos & ~(2 * L - 1), r = pos - base;
      const int a0 = base, b0 = base + L;           // the two runs being merged
      // number of A keys among the first r outputs (ties are padding)
      int lo = r > L ? r - L : 0, hi = r < L ? r : L;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (at(a0 + mid) <= at(b0 + r - 1 - mid)) lo = mid + 1;
        else hi = mid;
      }
      int i = lo, j = r - lo;
      double x = i < L ? at(a0 + i) : key_pad(), y = j < L ? at(b0 + j) : key_pad();
#pragma unroll
      for (int s = 0; s < K; ++s) {
        const bool take_a = x <= y;
        k[s] = take_a ? x : y;
        if (take_a) {
          ++i;
          x = i < L ? at(a0 + i) : key_pad();
        } else {
          ++j;
          y = j < L ? at(b0 + j) : key_pad();
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < K; ++s)
    if (pos + s < n) ids[pos + s] = lo_of(k[s]);
}

// The tile's list is the concatenation of its run in every chunk of its
// session (chunk-major keys, run offsets in the chunks' histogram rows).
// First each run's source and place in the list (a thread per chunk, a block
// scan of the run lengths, both kept in LDS for up to kGatherChunks chunks);
// then each thread finds the run of its first position by binary search and
// loads its positions together.  Sessions with more chunks copy run by run to
// the tile-major buffer (keys_tm).
constexpr int kGatherChunks = 1020;
constexpr int kSortThreads = 256;

struct RunTable {
  uint32_t at[kGatherChunks + 1];    // place of each run in the list; then n
  uint32_t src[kGatherChunks];       // its first key
};

// Fills T (spread sessions) or copies the list to dst; ends with a barrier.
__device__ __forceinline__ void list_runs(const WsPtrs& W, const SessionDev& S, int lt, int n,
                                          bool spread, RunTable& T, uint32_t* s_part,
                                          unsigned long long* dst) {
  const int ts = S.tiles_x * S.tiles_y;
  const int nc = (S.n + kChunk - 1) / kChunk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int c0 = 0; c0 < nc; c0 += kSortThreads) {
    const int c = c0 + (int)threadIdx.x;
    uint32_t cnt = 0, src = 0;
    if (c < nc) {
      const uint32_t* row = W.hist + S.hist_base + (int64_t)c * ts;
      const uint32_t off = row[lt];
      const uint32_t nxt = lt + 1 < ts ? row[lt + 1] : W.chunk_total[S.chunk_base + c];
      cnt = nxt - off;
      src = W.chunk_off[S.chunk_base + c] + off;
    }
    const uint32_t x = wave_scan(cnt);
    if (lane == 63) s_part[wave] = x;
    __syncthreads();
    uint32_t at = carry + x - cnt, tot = 0;
    for (int q = 0; q < kSortThreads / 64; ++q) {
      at += q < wave ? s_part[q] : 0u;
      tot += s_part[q];
    }
    if (spread) {
      if (c < nc) {
        T.at[c] = at;
        T.src[c] = src;
      }
    } else {
      for (uint32_t j = 0; j < cnt; ++j) dst[at + j] = W.keys[src + j];
    }
    carry += tot;
    __syncthreads();                        // s_part is reused
  }
  if (spread && threadIdx.x == 0) T.at[nc] = (uint32_t)n;
  __threadfence_block();                    // dst is read by other threads
  __syncthreads();
}

// List positions p0 to p0 + K - 1 (below n; the rest padding).
template <int K>
__device__ __forceinline__ void load_keys(const WsPtrs& W, const RunTable& T, int nc, bool spread,
                                          const unsigned long long* tm, int n, int p0,
                                          double (&k)[K]) {
#pragma unroll
  for (int j = 0; j < K; ++j) k[j] = key_pad();
  if (p0 >= n) return;
  if (!spread) {
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (p0 + j < n) k[j] = __longlong_as_double((long long)tm[p0 + j]);
    return;
  }
  int c = 0, hi = nc - 1;                   // last run with at <= p0
  while (c < hi) {
    const int mid = (c + hi + 1) >> 1;
    if (T.at[mid] <= (uint32_t)p0) c = mid; else hi = mid - 1;
  }
#pragma unroll
  for (int j = 0; j < K; ++j)
    if (p0 + j < n) {
      const uint32_t p = (uint32_t)(p0 + j);
      while (p >= T.at[c + 1]) ++c;         // runs are contiguous in the list
      k[j] = __longlong_as_double((long long)W.keys[T.src[c] + (p - T.at[c])]);
    }
}

// One workgroup per tile (neighbouring tiles on one XCD, whose L2 then holds
// the chunk rows and runs they share): lists of up to 1024 keys with four keys
// a thread, of up to 2048 with eight; longer ones are gathered to the
// tile-major buffer and queued for k_sort_big_tiles.
constexpr int kSmallKeys = 8 * kSortThreads;

template <bool ONE>
__global__ __launch_bounds__(kSortThreads) void k_sort_tiles(Batch B, WsPtrs W) {
  // the run table is read before the buffer is written (barriers between)
  __shared__ union {
    RunTable runs;
    double buf[sort_buf_keys(kSmallKeys)];
  } sh;
  __shared__ uint32_t s_part[kSortThreads / 64];
  const int per = (B.t_total + 7) >> 3;
  const int t = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (t >= B.t_total) return;
  const uint32_t st = W.tile_start[t];
  const int n = (int)(W.tile_start[t + 1] - st);   // all empty after an overflow
  if (n <= 0) return;
  // no pair of this call's lists has sums yet (a share of the flags as large as the
  // list; by the emit, whose workgroups may hold very unequal numbers of pairs,
  // 500 Gaussians of 12000 tiles each took 1200 us there, 1070 without)
  for (int k = threadIdx.x; k < n; k += kSortThreads) reinterpret_cast<uint32_t*>(W.live)[st + k] = 0u;
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, t,
                                         [](const SessionDev& x) { return x.tile_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int nc = (S.n + kChunk - 1) / kChunk;
  const bool spread = nc <= kGatherChunks;
  unsigned long long* const tm = W.keys_tm + st;
  list_runs(W, S, t - S.tile_base, n, spread, sh.runs, s_part, tm);
  const int pos = (((int)threadIdx.x & ~63) + lane_order(threadIdx.x & 63));
  if (n <= 4 * kSortThreads) {
    double k[4];
    load_keys<4>(W, sh.runs, nc, spread, tm, n, 4 * pos, k);
    __syncthreads();
    block_sort<kSortThreads, 4>(k, n, sh.buf, W.ids + st);
  } else if (n <= kSmallKeys) {
    double k[8];
    load_keys<8>(W, sh.runs, nc, spread, tm, n, 8 * pos, k);
    __syncthreads();
    block_sort<kSortThreads, 8>(k, n, sh.buf, W.ids + st);
  } else {
    if (spread) {
      for (int p0 = 4 * (int)threadIdx.x; p0 < n; p0 += 4 * kSortThreads) {
        double k[4];
        load_keys<4>(W, sh.runs, nc, true, tm, n, p0, k);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (p0 + j < n) tm[p0 + j] = (unsigned long long)__double_as_longlong(k[j]);
      }
    }
    if (threadIdx.x == 0) {
      const unsigned long long q = atomicAdd((unsigned long long*)&W.counters[2], 1ull);
      W.big_tiles[q] = (uint32_t)t;
    }
  }
}

// Bitonic sorting network on a[0..n) (ascending), all merges in the "flip"
// form so that virtual +inf padding up to the next power of two never moves:
// each compare-exchange puts the minimum at the lower index, hence a pair
// whose upper index is >= n is left alone.
__device__ void bitonic_sort(unsigned long long* a, int n) {
  int npow = 1;
  while (npow < n) npow <<= 1;
  const int half = npow >> 1;
  for (int k = 2; k <= npow; k <<= 1) {
    const int hk = k >> 1;
    for (int p = threadIdx.x; p < half; p += blockDim.x) {
      const int r = p & (hk - 1);
      const int i = (p / hk) * k + r;
      const int j = i + k - 1 - 2 * r;
      if (j < n) {
        const unsigned long long x = a[i], y = a[j];
        if (y < x) { a[i] = y; a[j] = x; }
      }
    }
    __threadfence_block();
    __syncthreads();
    for (int m = k >> 2; m >= 1; m >>= 1) {
      for (int p = threadIdx.x; p < half; p += blockDim.x) {
        const int i = (p / m) * 2 * m + (p & (m - 1));
        const int j = i + m;
        if (j < n) {
          const unsigned long long x = a[i], y = a[j];
          if (y < x) { a[i] = y; a[j] = x; }
        }
      }
      __threadfence_block();
      __syncthreads();
    }
  }
}

// Queued long lists (gathered to the tile-major buffer): up to 4096 keys with
// four keys a thread, up to 8192 with eight; longer ones by the bitonic
// network in place in global memory.  One launch whatever the lengths.
constexpr int kBigThreads = 1024;

__global__ __launch_bounds__(kBigThreads) void k_sort_big_tiles(WsPtrs W) {
  __shared__ double buf[sort_buf_keys(8 * kBigThreads)];
  const long long count = W.counters[2];
  for (long long q = blockIdx.x; q < count; q += gridDim.x) {
    const int t = (int)W.big_tiles[q];
    const int64_t st = W.tile_start[t];
    const int n = (int)(W.tile_start[t + 1] - st);
    unsigned long long* g = W.keys_tm + st;
    const int pos = ((int)threadIdx.x & ~63) + lane_order(threadIdx.x & 63);
    if (n <= 4 * kBigThreads) {
      double k[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        k[j] = 4 * pos + j < n ? __longlong_as_double((long long)g[4 * pos + j]) : key_pad();
      block_sort<kBigThreads, 4>(k, n, buf, W.ids + st);
    } else if (n <= 8 * kBigThreads) {
      double k[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        k[j] = 8 * pos + j < n ? __longlong_as_double((long long)g[8 * pos + j]) : key_pad();
      block_sort<kBigThreads, 8>(k, n, buf, W.ids + st);
    } else {
      bitonic_sort(g, n);
      for (int i = threadIdx.x; i < n; i += blockDim.x) W.ids[st + i] = (uint32_t)g[i];
    }
    __syncthreads();
  }
}

}  // namespace

void launch_tile_sort(const Batch& b, const WsPtrs& w, hipStream_t st) {
  const int grid = 8 * ((b.t_total + 7) / 8);
  if (b.n_sessions == 1)
    k_sort_tiles<true><<<grid, kSortThreads, 0, st>>>(b, w);
  else
    k_sort_tiles<false><<<grid, kSortThreads, 0, st>>>(b, w);
  if (b.n_total > kSmallKeys)            // no list is longer than that
    k_sort_big_tiles<<<b.t_total < 512 ? b.t_total : 512, kBigThreads, 0, st>>>(w);
}

}  // namespace rtgs
