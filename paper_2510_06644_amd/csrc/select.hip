// The two redundancy reductions of Sec. 4 as device-side selections.
//
// prune_by_grad (Sec. 4.1, Eq. 7): importance = ||dL/dmu|| + lambda ||dL/dSigma||_F
// per Gaussian (float64, rounded to float32), then the floor(ratio V) lowest
// (score, index) among visible, unmasked Gaussians join the mask.  The k-th
// smallest score is found by a radix select over the float bits (scores are
// >= 0, so bit order is value order) in three passes of 11, 11 and 10 bits,
// ties at the threshold go to the lowest indices through per-block counts.
// Everything stays on the device; a 64 KB scratch owned by the handle holds
// histograms and block counts.
//
// Five streaming passes over 36 bytes per Gaussian, each a launch of its own
// (every pass needs the totals of the one before); what a pass derives from
// those totals (digit, rank, offsets) each of its blocks works out for itself,
// so no single-block launches stand between them.  Most scores of a tracking
// iteration are exactly zero: a wave adds the count of its first lane's bin
// at once instead of lane by lane; 256 histogram blocks rather than 1024, whose
// additions to the same bins queue up (23 us a pass instead of 8.8).  500k
// Gaussians: four 8-bit passes with a single-block pick after each and a serial
// scan of the block counts, 14 launches, 150 us -> 6 launches, 50 us.
//
// downsample_mask (Sec. 4.2): one thread per block of 2^ceil(j/2) x
// 2^floor(j/2) pixels keeps the pixel with the lowest previous final T.
#include "rtgs_internal.h"

namespace rtgs {
namespace {

constexpr int kBins = 2048;            // bins of a pass
constexpr int kHist = 0;               // three histograms
constexpr int kBlockCnt = 3 * kBins;   // per-block counts of threshold keys
constexpr int kSelBlocks = 2048;       // max blocks of the final passes
constexpr int kSelThreads = 1024;
constexpr int kHistThreads = 1024;
static_assert(kBlockCnt + kSelBlocks <= kPruneScratchWords, "scratch holds the counts");

// Digit of pass p (0: the top 11 bits, 1: the next 11, 2: the last 10).
constexpr int pass_shift(int p) { return p == 0 ? 21 : p == 1 ? 10 : 0; }
constexpr uint32_t pass_mask(int p) { return p == 2 ? 1023u : 2047u; }

__device__ __forceinline__ bool candidate(const uint8_t* vis, const uint8_t* mask, int i) {
  return (vis == nullptr || vis[i] != 0) && (mask == nullptr || mask[i] == 0);
}

__device__ __forceinline__ uint32_t score_bits(const float* gm, const float* gc, float lam, int i) {
  const double a = gm[3 * i], b = gm[3 * i + 1], c = gm[3 * i + 2];
  const double xx = gc[6 * i], xy = gc[6 * i + 1], xz = gc[6 * i + 2];
  const double yy = gc[6 * i + 3], yz = gc[6 * i + 4], zz = gc[6 * i + 5];
  const double fro = sqrt(xx * xx + yy * yy + zz * zz + 2.0 * (xy * xy + xz * xz + yz * yz));
  const float s = (float)(sqrt(a * a + b * b + c * c) + (double)lam * fro);
  return __float_as_uint(s);
}

__global__ __launch_bounds__(kHistThreads) void k_prune_init(uint32_t* scr, int* n_masked) {
  const int i = blockIdx.x * kHistThreads + threadIdx.x;
  if (i < 3 * kBins) scr[kHist + i] = 0;
  if (i == 0 && n_masked) *n_masked = 0;
}

// The digit of a pass's histogram that holds rank `rank` (1-based, at most the
// total), and the rank inside it, by the block's NT threads.  s: NT / 64 + 2
// words of LDS.  Returns the total in `total`.
template <int NT>
__device__ __forceinline__ void pick_digit(const uint32_t* hist, uint32_t rank, uint32_t* s,
                                           uint32_t& digit, uint32_t& inside, uint32_t& total) {
  constexpr int kPer = kBins / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t h[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    h[i] = hist[tid * kPer + i];
    sum += h[i];
  }
  const uint32_t x = wave_scan(sum);
  if (lane == 63) s[wave] = x;
  __syncthreads();
  uint32_t before = x - sum;
  total = 0;
  for (int q = 0; q < NT / 64; ++q) {
    before += q < wave ? s[q] : 0u;
    total += s[q];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (before < rank && rank <= before + h[i]) {
      s[NT / 64] = (uint32_t)(tid * kPer + i);
      s[NT / 64 + 1] = rank - before;
    }
    before += h[i];
  }
  __syncthreads();
  digit = s[NT / 64];
  inside = s[NT / 64 + 1];
  __syncthreads();
}

// What `passes` passes have settled: k = floor(ratio V) of the V candidates,
// the threshold's leading digits, and the rank among the keys that share them.
struct Select {
  uint32_t k, prefix, rank;
};

template <int NT>
__device__ __forceinline__ Select selected(const uint32_t* scr, float ratio, int passes,
                                           uint32_t* s) {
  Select r{0, 0, 0};
  uint32_t total = 0, d = 0, in = 0;
  pick_digit<NT>(scr + kHist, 0, s, d, in, total);            // V
  r.k = (uint32_t)floor((double)ratio * (double)total);
  r.rank = r.k;
  if (r.k == 0) return r;
  for (int p = 0; p < passes; ++p) {
    pick_digit<NT>(scr + kHist + p * kBins, r.rank, s, d, in, total);
    r.prefix = (r.prefix << (p == 2 ? 10 : 11)) | d;
    r.rank = in;
  }
  return r;
}

// Histogram of pass PASS's digit among candidates whose higher digits are the
// threshold's.
template <int PASS>
__global__ __launch_bounds__(kHistThreads) void k_prune_hist(const float* gm, const float* gc,
                                                             float lam, const uint8_t* vis,
                                                             const uint8_t* mask, int n,
                                                             float ratio, uint32_t* scr) {
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t s[kHistThreads / 64 + 2];
  for (int i = threadIdx.x; i < kBins; i += kHistThreads) h[i] = 0;
  Select sel{0, 0, 0};
  if (PASS > 0) {
    sel = selected<kHistThreads>(scr, ratio, PASS, s);
    if (sel.k == 0) return;
  }
  __syncthreads();
  const int stride = gridDim.x * kHistThreads;
  for (int i0 = blockIdx.x * kHistThreads; i0 < n; i0 += stride) {
    const int i = i0 + threadIdx.x;
    bool in = i < n && candidate(vis, mask, i);
    uint32_t key = 0;
    if (in) {
      key = score_bits(gm, gc, lam, i);
      in = PASS == 0 || (key >> pass_shift(PASS > 0 ? PASS - 1 : 0)) == sel.prefix;
    }
    const uint32_t d = (key >> pass_shift(PASS)) & pass_mask(PASS);
    // the bin of the first lane in one addition, the others one by one
    const unsigned long long m = __ballot(in);
    if (m == 0) continue;
    const int first = __builtin_ctzll(m);
    const uint32_t d0 = (uint32_t)__shfl((int)d, first);
    const unsigned long long same = __ballot(in && d == d0);
    if ((int)(threadIdx.x & 63) == first)
      atomicAdd(&h[d0], (uint32_t)__popcll(same));
    else if (in && d != d0)
      atomicAdd(&h[d], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kBins; i += kHistThreads)
    if (h[i]) atomicAdd(&scr[kHist + PASS * kBins + i], h[i]);
}

__device__ __forceinline__ int sel_chunk(int n, int nb) {
  const int per = (n + nb - 1) / nb;
  return ((per + kSelThreads - 1) / kSelThreads) * kSelThreads;
}

// Per-block count of candidates whose key equals the threshold.
__global__ __launch_bounds__(kSelThreads) void k_prune_eqcount(const float* gm, const float* gc,
                                                              float lam, const uint8_t* vis,
                                                              const uint8_t* mask, int n, int nb,
                                                              float ratio, uint32_t* scr) {
  __shared__ uint32_t s[kSelThreads / 64 + 2];
  const Select sel = selected<kSelThreads>(scr, ratio, 3, s);
  const int chunk = sel_chunk(n, nb);
  const int beg = blockIdx.x * chunk, end = min(n, beg + chunk);
  uint32_t mine = 0;                       // of the wave, in every lane
  if (sel.k > 0)
    for (int i0 = beg; i0 < end; i0 += kSelThreads) {
      const int i = i0 + threadIdx.x;
      const bool eq = i < end && candidate(vis, mask, i) &&
                      score_bits(gm, gc, lam, i) == sel.prefix;
      mine += (uint32_t)__popcll(__ballot(eq));
    }
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int q = 0; q < kSelThreads / 64; ++q) t += s[q];
    scr[kBlockCnt + blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kSelThreads) void k_prune_final(const float* gm, const float* gc,
                                                            float lam, const uint8_t* vis,
                                                            const uint8_t* mask_in, int n, int nb,
                                                            float ratio, const uint32_t* scr,
                                                            uint8_t* mask_out, int* n_masked,
                                                            float* score_out) {
  __shared__ uint32_t s[kSelThreads / 64 + 2];
  __shared__ uint32_t wsum[kSelThreads / 64];
  const Select sel = selected<kSelThreads>(scr, ratio, 3, s);
  const uint32_t tau = sel.prefix, take = sel.rank;
  const bool any = sel.k > 0;
  if (blockIdx.x == 0 && threadIdx.x == 0 && n_masked) *n_masked = (int)sel.k;
  const int chunk = sel_chunk(n, nb);
  const int beg = blockIdx.x * chunk, end = min(n, beg + chunk);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // threshold keys in the blocks before this one
  uint32_t run = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += kSelThreads) run += scr[kBlockCnt + b];
  for (int off = 32; off >= 1; off >>= 1) run += __shfl_xor(run, off);
  if (lane == 0) wsum[wave] = run;
  __syncthreads();
  run = 0;
  for (int q = 0; q < kSelThreads / 64; ++q) run += wsum[q];
  __syncthreads();
  for (int base = beg; base < end; base += kSelThreads) {
    const int i = base + threadIdx.x;
    bool cand = false, eq = false, lt = false;
    uint32_t key = 0;
    if (i < end) {
      cand = candidate(vis, mask_in, i);
      key = score_bits(gm, gc, lam, i);
      if (score_out) score_out[i] = __uint_as_float(key);
      eq = cand && key == tau;
      lt = cand && key < tau;
    }
    const unsigned long long bal = __ballot(eq);
    const uint32_t before_in_wave = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = (uint32_t)__popcll(bal);
    __syncthreads();
    uint32_t before = run + before_in_wave;
    for (int q = 0; q < wave; ++q) before += wsum[q];
    uint32_t tot = 0;
    for (int q = 0; q < kSelThreads / 64; ++q) tot += wsum[q];
    __syncthreads();
    if (i < end) {
      const bool sel_i = any && (lt || (eq && before < take));
      const bool was = mask_in != nullptr && mask_in[i] != 0;
      mask_out[i] = (was || sel_i) ? 1 : 0;
    }
    run += tot;
  }
}

// (every block keeps one pixel, so the count is the number of blocks)
__global__ void k_downsample(const float* T, int w, int h, int bw, int bh, uint8_t* mask,
                             int* n_active) {
  const int nbx = (w + bw - 1) / bw, nby = (h + bh - 1) / bh;
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b == 0 && n_active) *n_active = nbx * nby;
  if (b >= nbx * nby) return;
  const int x0 = (b % nbx) * bw, y0 = (b / nbx) * bh;
  const int x1 = min(w, x0 + bw), y1 = min(h, y0 + bh);
  int best = y0 * w + x0;
  float bt = T[best];
  for (int y = y0; y < y1; ++y)
    for (int x = x0; x < x1; ++x) {
      const int p = y * w + x;
      const float t = T[p];
      if (t < bt) { bt = t; best = p; }       // row-major visit: first minimum wins
    }
  for (int y = y0; y < y1; ++y)
    for (int x = x0; x < x1; ++x) mask[y * w + x] = (y * w + x == best) ? 1 : 0;
}

}  // namespace

hipError_t launch_prune(const float* g_means, const float* g_cov3d, const uint8_t* visible,
                        const uint8_t* mask_in, int n, float lambda, float ratio,
                        uint8_t* mask_out, int* n_masked, float* score_out, uint32_t* scr,
                        hipStream_t st) {
  k_prune_init<<<3 * kBins / kHistThreads, kHistThreads, 0, st>>>(scr, n_masked);
  if (n <= 0) return hipGetLastError();
  const int grid = min(256, (n + kHistThreads - 1) / kHistThreads);
  k_prune_hist<0><<<grid, kHistThreads, 0, st>>>(g_means, g_cov3d, lambda, visible, mask_in, n,
                                                 ratio, scr);
  k_prune_hist<1><<<grid, kHistThreads, 0, st>>>(g_means, g_cov3d, lambda, visible, mask_in, n,
                                                 ratio, scr);
  k_prune_hist<2><<<grid, kHistThreads, 0, st>>>(g_means, g_cov3d, lambda, visible, mask_in, n,
                                                 ratio, scr);
  const int nb = min(kSelBlocks, (n + kSelThreads - 1) / kSelThreads);
  k_prune_eqcount<<<nb, kSelThreads, 0, st>>>(g_means, g_cov3d, lambda, visible, mask_in, n, nb,
                                               ratio, scr);
  k_prune_final<<<nb, kSelThreads, 0, st>>>(g_means, g_cov3d, lambda, visible, mask_in, n, nb,
                                             ratio, scr, mask_out, n_masked, score_out);
  return hipGetLastError();
}

hipError_t launch_downsample(const float* final_T, int w, int h, int j, uint8_t* mask_out,
                             int* n_active, hipStream_t st) {
  const int bw = 1 << ((j + 1) / 2), bh = 1 << (j / 2);
  const int nb = ((w + bw - 1) / bw) * ((h + bh - 1) / bh);
  k_downsample<<<(nb + 255) / 256, 256, 0, st>>>(final_T, w, h, bw, bh, mask_out,
                                                            n_active);
  return hipGetLastError();
}

}  // namespace rtgs
