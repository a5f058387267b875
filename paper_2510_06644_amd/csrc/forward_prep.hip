// Steps 1 and 2 of the forward pass (Sec. 2.1): projection of every Gaussian
// (Step 1-1), tile intersection (Step 1-2) and per-tile depth sorting
// (Step 2), for a batch of sessions sharing one tile space.
//
// Design for gfx950:
//  * projection runs one thread per Gaussian in float64: it is HBM bound
//    (56 B in, 64 B out per Gaussian), and float64 lets the raster kernels see
//    pixel-space centres split as hi + lo float32 parts, so their float32
//    compositing matches the float64 definition far below 1e-4;
//  * binning is a counting sort by tile without global atomics (device-scope
//    atomics cross the XCDs and serialise).  Each workgroup takes a chunk of
//    1024 Gaussians and counts its (tile, Gaussian) pairs per tile in an LDS
//    histogram.  Column sums over the chunks give each tile's list length and
//    start.  A second pass over the chunk orders its pairs by tile in LDS
//    and writes them as one contiguous block (chunk-major: every store is
//    coalesced, where scattering 8-byte keys into the tile ranges made the
//    memory system merge millions of partial lines).  One workgroup per tile
//    then gathers the tile's run from every chunk and sorts it (tile_sort.hip).
//    The same pass writes each Gaussian's first slot in Gaussian-major pair
//    order, which the backward uses to merge gradients without atomics.  No
//    host sync: the pair total stays on the device, and a capacity overflow
//    publishes empty tile lists (every list entry is always a real pair).
#include "rtgs_internal.h"

namespace rtgs {
namespace {

constexpr int kScanThreads = 1024;

__global__ void k_init(WsPtrs W) {
  if (threadIdx.x < 8) W.counters[threadIdx.x] = 0;
  W.order_n[threadIdx.x] = 0u;
}

// Two counts to host memory, and zero in their place.
__global__ void k_take_counts(unsigned long long* d, unsigned long long* host) {
  if (threadIdx.x < 2) {
    host[threadIdx.x] = d[threadIdx.x];
    d[threadIdx.x] = 0;
  }
}

struct Proj {
  double u, v, z, sxx, sxy, syy;
  bool ok;
};

// Step 1-1 for one Gaussian in float64 (EWA, first order).
__device__ __forceinline__ void project_one(const SessionDev& S, const float* vm, int li,
                                            double& o, Proj& P) {
  const double mx = S.means[3 * li + 0], my = S.means[3 * li + 1], mz = S.means[3 * li + 2];
  const double qw = S.quats[4 * li + 0], qx = S.quats[4 * li + 1];
  const double qy = S.quats[4 * li + 2], qz = S.quats[4 * li + 3];
  double ss[3];
  activate(S, li, ss, o);
  P.ok = false;
  // camera-space centre p = R_c mu + t_c
  const double x = vm[0] * mx + vm[1] * my + vm[2] * mz + vm[3];
  const double y = vm[4] * mx + vm[5] * my + vm[6] * mz + vm[7];
  const double z = vm[8] * mx + vm[9] * my + vm[10] * mz + vm[11];
  P.z = z;
  if (!(z > kNearZ) || !(255.0 * o >= 1.0)) return;
  if (S.gmask && S.gmask[li]) return;
  // rotation of the normalised quaternion (w, x, y, z)
  const double qn = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
  const double w = qw * qn, a = qx * qn, b = qy * qn, c = qz * qn;
  double R[9] = {1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                 2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                 2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)};
  // M = R diag(s); Sigma = M M^T
  double M[9];
  for (int r = 0; r < 3; ++r)
    for (int k = 0; k < 3; ++k) M[3 * r + k] = R[3 * r + k] * ss[k];
  // EWA Jacobian with the field-of-view clamp
  const double limx = kFovClamp * 0.5 * S.width / S.fx;
  const double limy = kFovClamp * 0.5 * S.height / S.fy;
  const double iz = 1.0 / z;      // once: a float64 division is a long instruction sequence
  const double rx = x * iz, ry = y * iz;
  const double tx = fmin(limx, fmax(-limx, rx));
  const double ty = fmin(limy, fmax(-limy, ry));
  const double j00 = S.fx * iz, j02 = -S.fx * tx * iz;
  const double j11 = S.fy * iz, j12 = -S.fy * ty * iz;
  // T = J W (2x3), W = R_c
  double T0[3], T1[3];
  for (int k = 0; k < 3; ++k) {
    T0[k] = j00 * vm[0 + k] + j02 * vm[8 + k];
    T1[k] = j11 * vm[4 + k] + j12 * vm[8 + k];
  }
  // A = T M (2x3); Sigma' = A A^T + dilation
  double A0[3], A1[3];
  for (int k = 0; k < 3; ++k) {
    A0[k] = T0[0] * M[0 + k] + T0[1] * M[3 + k] + T0[2] * M[6 + k];
    A1[k] = T1[0] * M[0 + k] + T1[1] * M[3 + k] + T1[2] * M[6 + k];
  }
  P.sxx = A0[0] * A0[0] + A0[1] * A0[1] + A0[2] * A0[2] + kDilation;
  P.sxy = A0[0] * A1[0] + A0[1] * A1[1] + A0[2] * A1[2];
  P.syy = A1[0] * A1[0] + A1[1] * A1[1] + A1[2] * A1[2] + kDilation;
  P.u = S.fx * rx + S.cx;
  P.v = S.fy * ry + S.cy;
  const double det = P.sxx * P.syy - P.sxy * P.sxy;
  P.ok = det > 0.0;
}

__device__ __forceinline__ void split(double x, float& hi, float& lo) {
  hi = (float)x;
  lo = (float)(x - (double)hi);
}

// Step 1-1 + the tile rectangle of Step 1-2 + per-tile pair counts.
// REUSE: the tile lists (and with them each Gaussian's tile rectangle, pair
// count and slots) stay those of the workspace's last full forward; only the
// raster records are recomputed for the current pose.
template <bool REUSE, bool ONE>
__global__ __launch_bounds__(kGaussPerBlock) void k_preprocess(Batch B, WsPtrs W) {
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, (int)blockIdx.x,
                                         [](const SessionDev& x) { return x.block_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int li = ((int)blockIdx.x - S.block_base) * kGaussPerBlock + (int)threadIdx.x;
  // the call's counters start at zero (the binning passes run after this kernel)
  if (!REUSE && blockIdx.x == 0 && threadIdx.x < 8) W.counters[threadIdx.x] = 0;
  static_assert(8 * kOrderClasses == kGaussPerBlock, "a thread per class");
  if (blockIdx.x == 0) W.order_n[threadIdx.x] = 0u;
  if (li >= S.n) return;
  const int gid = S.gauss_base + li;
  float vm[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) vm[k] = S.viewmat[k];
  double o;
  Proj P;
  project_one(S, vm, li, o, P);
  int4 rect = make_int4(0, 0, -1, -1);
  GaussRec r;
  if (P.ok) {
    const double det = P.sxx * P.syy - P.sxy * P.sxy;
    const double inv = 1.0 / det;
    float uh, ul, vh, vl;
    split(P.u, uh, ul);
    split(P.v, vh, vl);
    const float zf = (float)P.z;
    // bounding box of the alpha = 1/255 ellipse: d^T M d <= 2 ln(255 o)
    const double t = 2.0 * (double)logf((float)(255.0 * o));
    const float ex = (float)sqrt(t * P.sxx);
    const float ey = (float)sqrt(t * P.syy);
    r.pos = make_float4(uh, vh, ul, vl);
    r.conic = make_float4((float)(P.syy * inv), (float)(-P.sxy * inv), (float)(P.sxx * inv),
                          (float)o);
    r.col = make_float4(S.colors[3 * li + 0], S.colors[3 * li + 1], S.colors[3 * li + 2], zf);
    r.ext.y = ex;
    r.ext.z = (float)t;
    r.ext.w = ey;
    // padded pixel range in float32, fixed operation order (see the replay)
    const float lox = floorf((uh - ex) - 1.5f), hix = ceilf((uh + ex) + 0.5f);
    const float loy = floorf((vh - ey) - 1.5f), hiy = ceilf((vh + ey) + 0.5f);
    if (!(hix < 0.f || lox > (float)(S.width - 1) || hiy < 0.f || loy > (float)(S.height - 1))) {
      const int i0 = (int)fmaxf(lox, 0.f), i1 = (int)fminf(hix, (float)(S.width - 1));
      const int j0 = (int)fmaxf(loy, 0.f), j1 = (int)fminf(hiy, (float)(S.height - 1));
      const int shx = 4 + S.sub_sx, shy = 4 + S.sub_sy;   // tile = (16 bw) x (16 bh)
      rect = make_int4(i0 >> shx, j0 >> shy, i1 >> shx, j1 >> shy);
    }
  } else {
    r.pos = make_float4(0.f, 0.f, 0.f, 0.f);
    r.conic = make_float4(0.f, 0.f, 0.f, 0.f);
    r.col = make_float4(0.f, 0.f, 0.f, (float)P.z);
    // a negative alpha-ellipse bound fails every quadrant test: a culled or
    // masked Gaussian left in a reused list costs the rasterizer nothing
    r.ext.z = -1.f;
    r.ext.y = r.ext.w = 0.f;
  }
  if (REUSE) rect = W.rect[gid];
  // the lists' rectangle, from which the raster backward takes the pair's slot
  const int rw = rect.z - rect.x + 1;
  static_assert(kMaxTilesPerSession <= 1 << 15, "tile and width in half a word each");
  r.ext.x = __int_as_float(((rect.y * rw + rect.x) << 16) | rw);
  W.rec[gid] = r;
  if (REUSE) {
    if (S.visible) S.visible[li] = rect.z >= rect.x ? 1 : 0;
    return;
  }
  W.rect[gid] = rect;
  // the depth bits of the Gaussian's sort key, read by the emit from this
  // dense array rather than from the 64-byte records
  W.zkey[gid] = __float_as_uint((float)P.z);
  const bool vis = rect.z >= rect.x;
  if (S.visible) S.visible[li] = vis ? 1 : 0;
  W.cnt[gid] = vis ? (uint32_t)((rect.z - rect.x + 1) * (rect.w - rect.y + 1)) : 0u;
}

// Threads per workgroup of the binning passes over a chunk: one Gaussian per
// thread, so the few hundred chunks of a frame still fill the chip.
constexpr int kBinThreads = 1024;
static_assert(kChunk % kBinThreads == 0, "whole rounds per chunk");

// The tile rectangles and pair counts of this thread's Gaussians of chunk c
// (local index i = j * kBinThreads + thread for round j), loaded together at
// the start of a binning pass so that their latencies overlap.
constexpr int kChunkRounds = kChunk / kBinThreads;
struct ChunkIn {
  int4 rect[kChunkRounds];
  uint32_t cnt[kChunkRounds];
};

__device__ __forceinline__ ChunkIn load_chunk(const SessionDev& S, const WsPtrs& W, int c) {
  ChunkIn in;
#pragma unroll
  for (int j = 0; j < kChunkRounds; ++j) {
    const int li = c * kChunk + j * kBinThreads + (int)threadIdx.x;
    in.rect[j] = li < S.n ? W.rect[S.gauss_base + li] : make_int4(0, 0, -1, -1);
    in.cnt[j] = li < S.n ? W.cnt[S.gauss_base + li] : 0u;
  }
  return in;
}

// The chunk's tile rectangles in LDS, so the pair walk below never waits on
// a dependent global load.  Visible after the barrier in chunk_offsets.
__device__ __forceinline__ void stage_rects(const ChunkIn& in, int4* s_rect) {
#pragma unroll
  for (int j = 0; j < kChunkRounds; ++j) s_rect[j * kBinThreads + threadIdx.x] = in.rect[j];
}

// In-chunk exclusive offsets of the Gaussians' tile counts, in local index
// order, into s_off[0..kChunk]; s_off[kChunk] = the chunk's pair total, which
// is returned.
__device__ uint32_t chunk_offsets(const ChunkIn& in, uint32_t* s_off, uint32_t* s_wave) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int j = 0; j < kChunkRounds; ++j) {
    const int i = j * kBinThreads + (int)threadIdx.x;
    const uint32_t n = in.cnt[j];
    const uint32_t x = wave_scan(n);
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int q = 0; q < kBinThreads / 64; ++q) {
      before += q < wave ? s_wave[q] : 0u;
      tot += s_wave[q];
    }
    s_off[i] = carry + before + x - n;
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) s_off[kChunk] = carry;
  __syncthreads();
  return carry;
}

// Walk this thread's share of the chunk's pairs: pairs [m0, m1) in
// Gaussian-major order, m0 = thread * ceil(total / kBinThreads), with the
// chunk's tile rectangles staged in LDS (s_rect[i] for local index i).  One binary search
// finds the first Gaussian; after that the walk steps through tiles of the
// Gaussian's rectangle row by row and on to the next Gaussian, so pairs are
// spread evenly however many tiles a Gaussian touches.  f(local index, tile)
// is called for every pair.
template <typename F>
__device__ __forceinline__ void chunk_pairs(const SessionDev& S, const int4* s_rect, int c,
                                            const uint32_t* s_off, uint32_t total, F f) {
  const uint32_t per = (total + kBinThreads - 1) / kBinThreads;
  const uint32_t m0 = threadIdx.x * per;
  const uint32_t m1 = min(total, m0 + per);
  if (m0 >= m1) return;
  int lo = 0, hi = kChunk - 1;          // last i with s_off[i] <= m0
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_off[mid] <= m0) lo = mid; else hi = mid - 1;
  }
  int i = lo;
  int4 r = s_rect[i];
  int w = r.z - r.x + 1;
  const int k0 = (int)(m0 - s_off[i]);
  int tx = r.x + k0 % w, ty = r.y + k0 / w;
  for (uint32_t m = m0; m < m1; ++m) {
    while (m >= s_off[i + 1]) {           // next Gaussian with pairs
      ++i;
      if (m < s_off[i + 1]) {
        r = s_rect[i];
        w = r.z - r.x + 1;
        tx = r.x;
        ty = r.y;
      }
    }
    f(i, ty * S.tiles_x + tx);
    if (++tx > r.z) {
      tx = r.x;
      ++ty;
    }
  }
}

// Per chunk of kChunk Gaussians: pair counts per tile of the session (LDS
// histogram), and the chunk's pair total.
template <bool ONE>
__global__ __launch_bounds__(kBinThreads) void k_chunk_hist(Batch B, WsPtrs W) {
  extern __shared__ uint32_t s_hist[];
  __shared__ uint32_t s_off[kChunk + 1];
  __shared__ int4 s_rect[kChunk];
  __shared__ uint32_t s_wave[kBinThreads / 64];
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, (int)blockIdx.x,
                                         [](const SessionDev& x) { return x.chunk_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int c = (int)blockIdx.x - S.chunk_base;
  const int ts = S.tiles_x * S.tiles_y;
  const ChunkIn in = load_chunk(S, W, c);
  for (int t = threadIdx.x; t < ts; t += kBinThreads) s_hist[t] = 0u;
  stage_rects(in, s_rect);
  const uint32_t total = chunk_offsets(in, s_off, s_wave);
  // pairs are dealt evenly over the threads, whatever the Gaussians' sizes
  chunk_pairs(S, s_rect, c, s_off, total, [&](int, int tile) { atomicAdd(&s_hist[tile], 1u); });
  __syncthreads();
  uint32_t* h = W.hist + S.hist_base + (int64_t)c * ts;
  for (int t = threadIdx.x; t < ts; t += kBinThreads) h[t] = s_hist[t];
  if (threadIdx.x == 0) W.chunk_total[blockIdx.x] = total;
}

// Column sums of the per-(chunk, tile) counts, one thread per (tile, group
// of chunks); k_scan_tiles adds the groups.
constexpr int kScanGroups = 16;

__device__ __forceinline__ void tile_groups(const SessionDev& S, int g, int& c0, int& c1) {
  const int nc = (S.n + kChunk - 1) / kChunk;
  const int per = (nc + kScanGroups - 1) / kScanGroups;
  c0 = min(nc, g * per);
  c1 = min(nc, c0 + per);
}

template <bool ONE>
__global__ __launch_bounds__(kBlock) void k_tile_group_sums(Batch B, WsPtrs W) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  const int g = blockIdx.y;
  if (t >= B.t_total) return;
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, t,
                                         [](const SessionDev& x) { return x.tile_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int ts = S.tiles_x * S.tiles_y;
  int c0, c1;
  tile_groups(S, g, c0, c1);
  const uint32_t* h = W.hist + S.hist_base + (t - S.tile_base);
  uint32_t sum = 0;
#pragma unroll 8
  for (int c = c0; c < c1; ++c) sum += h[(int64_t)c * ts];
  W.gsum[(int64_t)g * B.t_total + t] = sum;
}

// Exclusive scan of n values in[0..n) into out[0..n]; out[n] = total.  Each
// thread sums a contiguous run; the run sums are scanned inside each wave by
// lane shifts, then across the waves through LDS (part[kScanThreads / 64]),
// so two barriers in all.
__device__ uint32_t block_scan_1024(const uint32_t* in, uint32_t* out, int n, uint32_t* part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + kScanThreads - 1) / kScanThreads;
  const int beg = min(tid * per, n), end = min(beg + per, n);
  uint32_t sum = 0;
  for (int i = beg; i < end; ++i) sum += in[i];
  const uint32_t x = wave_scan(sum);
  if (lane == 63) part[wave] = x;
  __syncthreads();
  uint32_t before = 0, total = 0;
  for (int q = 0; q < kScanThreads / 64; ++q) {
    const uint32_t v = part[q];
    before += q < wave ? v : 0u;
    total += v;
  }
  uint32_t run = before + x - sum;
  for (int i = beg; i < end; ++i) {
    const uint32_t v = in[i];
    out[i] = run;
    run += v;
  }
  if (tid == 0) out[n] = total;
  __syncthreads();                        // part is reused by the next call
  return total;
}

// Exclusive scan across the block of the values v[0..P) that each thread
// holds for positions P tid .. P tid + P - 1; v becomes the exclusive
// prefixes, and the block total is returned.  Same two-barrier structure as
// block_scan_1024.
template <int P>
__device__ uint32_t block_scan_regs(uint32_t (&v)[P], uint32_t* part) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) sum += v[i];
  const uint32_t x = wave_scan(sum);
  if (lane == 63) part[wave] = x;
  __syncthreads();
  uint32_t before = 0, total = 0;
  for (int q = 0; q < kScanThreads / 64; ++q) {
    const uint32_t w = part[q];
    before += q < wave ? w : 0u;
    total += w;
  }
  uint32_t run = before + x - sum;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const uint32_t w = v[i];
    v[i] = run;
    run += w;
  }
  __syncthreads();                        // part is reused by the next call
  return total;
}

// Tile ranges (scan of the per-tile counts, each the sum of `groups` rows of
// src, one per group of chunks or per chunk), chunk offsets (scan of the
// per-chunk totals), and the pair total.
// Up to PER tiles and kScanPer chunks per thread the counts are loaded together
// with coalesced loads into LDS, scanned in registers (each thread a
// contiguous run) and stored coalesced from LDS: one round trip to memory.
// (Six served frames, 10.5k tiles: through global memory 15 us, so 12.)
// Larger batches scan through global memory.  When the pairs exceed the
// capacity every tile list is published empty (the call's output is invalid
// and reported, and no list holds a pair that was not stored).
constexpr int kScanPer = 4, kScanPerMany = 12;

__device__ __forceinline__ uint32_t column_sum(const uint32_t* src, int groups, int64_t stride,
                                               int t) {
  uint32_t sum = 0;
#pragma unroll 16
  for (int g = 0; g < groups; ++g) sum += src[g * stride + t];
  return sum;
}

template <int PER>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(WsPtrs W, const uint32_t* src,
                                                             int groups, int t_total, int c_total,
                                                             unsigned long long* max_pairs) {
  __shared__ uint32_t part[kScanThreads / 64];
  __shared__ uint32_t s_t[PER * kScanThreads], s_c[kScanPer * kScanThreads];
  __shared__ uint32_t s_wn[kScanPer * kScanThreads];
  const int tid = threadIdx.x;
  uint32_t total;
  if (t_total <= PER * kScanThreads && c_total <= kScanPer * kScanThreads) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int t = k * kScanThreads + tid;
      s_t[t] = t < t_total ? column_sum(src, groups, t_total, t) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      const int c = k * kScanThreads + tid;
      s_c[c] = c < c_total ? W.chunk_total[c] : 0u;
    }
    __syncthreads();
    uint32_t tv[PER], cv[kScanPer], wv[kScanPer];
#pragma unroll
    for (int i = 0; i < PER; ++i) tv[i] = s_t[tid * PER + i];
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
      cv[i] = s_c[tid * kScanPer + i];
      wv[i] = (cv[i] + kWindow - 1) / kWindow;
    }
    total = block_scan_regs<PER>(tv, part);             // its barriers order the LDS reuse
    const uint32_t ctot = block_scan_regs<kScanPer>(cv, part);
    const uint32_t wtot = block_scan_regs<kScanPer>(wv, part);
#pragma unroll
    for (int i = 0; i < PER; ++i) s_t[tid * PER + i] = tv[i];
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
      s_c[tid * kScanPer + i] = cv[i];
      s_wn[tid * kScanPer + i] = wv[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int t = k * kScanThreads + tid;
      if (t < t_total) W.tile_start[t] = s_t[t];
    }
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      const int c = k * kScanThreads + tid;
      if (c < c_total) {
        W.chunk_off[c] = s_c[c];
        W.win_off[c] = s_wn[c];
      }
    }
    if (tid == 0) {
      W.tile_start[t_total] = total;
      W.chunk_off[c_total] = ctot;
      W.win_off[c_total] = wtot;
    }
    __syncthreads();                      // tile_start complete before an overflow clears it
  } else {
    for (int t = tid; t < t_total; t += kScanThreads)
      W.tile_count[t] = column_sum(src, groups, t_total, t);
    __syncthreads();
    total = block_scan_1024(W.tile_count, W.tile_start, t_total, part);
    block_scan_1024(W.chunk_total, W.chunk_off, c_total, part);
    // the chunks' windows, counted in place of their offsets first
    for (int c = tid; c < c_total; c += kScanThreads)
      W.win_off[c] = (W.chunk_total[c] + kWindow - 1) / kWindow;
    __syncthreads();
    block_scan_1024(W.win_off, W.win_off, c_total, part);
  }
  if ((int64_t)total > W.cap)
    for (int t = threadIdx.x; t <= t_total; t += kScanThreads) W.tile_start[t] = 0u;
  if (threadIdx.x == 0) {
    W.counters[0] = (long long)total;
    // [0]: largest pair count of any call; [1]: largest count of a call whose
    // capacity it exceeded (0 if none)
    atomicMax(&max_pairs[0], (unsigned long long)total);
    if ((int64_t)total > W.cap) atomicMax(&max_pairs[1], (unsigned long long)total);
  }
}

// For the backward's merge: the chunk's Gaussians that have pairs, in order
// (vlist, closed by the chunk's end), and the chunk's windows of kWindow pairs
// with the vlist entries they meet.  s_off: the Gaussians' pair offsets in the
// chunk; s_wave: LDS of a word per wave.
__device__ void list_windows(const WsPtrs& W, int chunk, int gauss0, uint32_t base, uint32_t total,
                             const uint32_t* s_off, uint32_t* s_wave) {
  static_assert(kChunkRounds == 1, "one Gaussian per thread");
  const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
  const uint32_t o = s_off[i], e = s_off[i + 1];
  const bool has = e > o;
  const unsigned long long m = __ballot(has);
  if (lane == 0) s_wave[wave] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t rank = (uint32_t)__popcll(m & ((1ull << lane) - 1ull)), count = 0;
  for (int q = 0; q < kBinThreads / 64; ++q) {
    rank += q < wave ? s_wave[q] : 0u;
    count += s_wave[q];
  }
  const uint32_t v0 = (uint32_t)chunk * (kChunk + 1);
  if (has) {
    W.vlist[v0 + rank] = make_uint2((uint32_t)(gauss0 + i), base + o);
    uint32_t* win = reinterpret_cast<uint32_t*>(W.window + W.win_off[chunk]);
    // windows that begin in this Gaussian's pairs, and those that end in them
    for (uint32_t k = (o + kWindow - 1) / kWindow; k * kWindow < e; ++k) {
      win[4 * k] = base + k * kWindow;
      win[4 * k + 1] = base + min(total, (k + 1) * kWindow);
      win[4 * k + 2] = v0 + rank;
    }
    for (uint32_t k = o / kWindow; k * kWindow < e; ++k) {
      const uint32_t end = min(total, (k + 1) * kWindow);
      if (end > o && end <= e) win[4 * k + 3] = v0 + rank;
    }
  }
  if (i == 0) W.vlist[v0 + count] = make_uint2(0u, base + total);
}

// Per chunk: each Gaussian's first Gaussian-major slot; the chunk's pairs
// ordered by tile, written as one block at chunk_off (chunk-major layout;
// inside it, tile t's run starts at the exclusive scan of the chunk's tile
// counts, which replaces the counts in this chunk's histogram row for the
// sort's gather).  The pairs are staged in LDS as 16-bit local indices and
// written with coalesced stores; a chunk with more than kStagePairs pairs
// writes them directly inside its block.
constexpr int kStagePairs = 12288;

template <bool ONE>
__global__ __launch_bounds__(kBinThreads) void k_emit(Batch B, WsPtrs W) {
  extern __shared__ uint32_t s_dyn[];       // [ts] tile cursors, then [kStagePairs] uint16
  __shared__ uint32_t s_off[kChunk + 1];
  __shared__ int4 s_rect[kChunk];
  __shared__ uint32_t s_zb[kChunk];
  __shared__ uint32_t s_wave[kBinThreads / 64];
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, (int)blockIdx.x,
                                         [](const SessionDev& x) { return x.chunk_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int c = (int)blockIdx.x - S.chunk_base;
  const int ts = S.tiles_x * S.tiles_y;
  uint32_t* s_cur = s_dyn;
  uint16_t* s_loc = reinterpret_cast<uint16_t*>(s_dyn + ts);
  uint32_t* h = W.hist + S.hist_base + (int64_t)c * ts;
  // every global load of the prologue issued together: the Gaussians' inputs,
  // their key depths and this thread's run of the chunk's tile counts
  const ChunkIn in = load_chunk(S, W, c);
  uint32_t zb[kChunkRounds];
#pragma unroll
  for (int j = 0; j < kChunkRounds; ++j) {
    const int li = c * kChunk + j * kBinThreads + (int)threadIdx.x;
    zb[j] = li < S.n ? W.zkey[S.gauss_base + li] : 0u;
  }
  constexpr int kRunMax = (kMaxTilesPerSession + kBinThreads - 1) / kBinThreads;
  const int per = (ts + kBinThreads - 1) / kBinThreads;
  const int beg = min((int)threadIdx.x * per, ts), end = min(beg + per, ts);
  uint32_t hv[kRunMax];
#pragma unroll
  for (int k = 0; k < kRunMax; ++k) hv[k] = beg + k < end ? h[beg + k] : 0u;
  // exclusive scan of the chunk's tile counts: each thread a contiguous run of
  // tiles, the run sums scanned across the waves
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kRunMax; ++k) sum += hv[k];
    const uint32_t x = wave_scan(sum);
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    uint32_t run = x - sum;
    for (int q = 0; q < wave; ++q) run += s_wave[q];
#pragma unroll
    for (int k = 0; k < kRunMax; ++k) {
      if (beg + k < end) {
        s_cur[beg + k] = run;
        h[beg + k] = run;
      }
      run += hv[k];
    }
    __syncthreads();                        // s_wave is reused below
  }
  stage_rects(in, s_rect);
#pragma unroll
  for (int j = 0; j < kChunkRounds; ++j) s_zb[j * kBinThreads + threadIdx.x] = zb[j];
  const uint32_t total = chunk_offsets(in, s_off, s_wave);
  const uint32_t base = W.chunk_off[blockIdx.x];
  for (int j = 0; j < kChunk / kBinThreads; ++j) {
    const int i = j * kBinThreads + (int)threadIdx.x;
    const int li = c * kChunk + i;
    if (li < S.n) W.goff[S.gauss_base + li] = base + s_off[i];
  }
  if (W.chunk_off[B.c_total] <= (uint64_t)W.cap)
    list_windows(W, blockIdx.x, S.gauss_base + c * kChunk, base, total, s_off, s_wave);
  const uint32_t g0 = S.gauss_base + c * kChunk;
  const bool staged = total <= kStagePairs;
  chunk_pairs(S, s_rect, c, s_off, total, [&](int i, int tile) {
    const uint32_t pos = atomicAdd(&s_cur[tile], 1u);
    if (staged)
      s_loc[pos] = (uint16_t)i;
    else if ((int64_t)base + pos < W.cap)
      W.keys[base + pos] = ((unsigned long long)s_zb[i] << 32) | (g0 + i);
  });
  if (staged) {
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < total; k += kBinThreads) {
      const uint32_t i = s_loc[k];
      if ((int64_t)base + k < W.cap)
        W.keys[base + k] = ((unsigned long long)s_zb[i] << 32) | (g0 + i);
    }
  }
}

__global__ void k_debug_stage(Batch B, WsPtrs W, float* stage, int* rect, int* ranges, int* ids,
                              int64_t ids_cap) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < B.n_total) {
    if (stage) {
      const GaussRec R = W.rec[i];
      const float4 r0 = R.pos, r1 = R.conic, r2 = R.col;
      const float4 e = R.ext;
      float* o = stage + 12 * (int64_t)i;
      o[0] = r0.x; o[1] = r0.y; o[2] = r1.x; o[3] = r1.y; o[4] = r1.z; o[5] = r1.w;
      o[6] = r2.w; o[7] = e.y; o[8] = e.w; o[9] = r2.x; o[10] = r2.y; o[11] = r2.z;
    }
    if (rect) {
      const int4 r = W.rect[i];
      rect[4 * i + 0] = r.x; rect[4 * i + 1] = r.y; rect[4 * i + 2] = r.z; rect[4 * i + 3] = r.w;
    }
  }
  if (i < B.t_total && ranges) {
    ranges[2 * i] = (int)W.tile_start[i];
    ranges[2 * i + 1] = (int)W.tile_start[i + 1];
  }
  if (ids) {
    const int64_t total = min((int64_t)W.tile_start[B.t_total], min(W.cap, ids_cap));
    for (int64_t k = i; k < total; k += (int64_t)gridDim.x * blockDim.x) ids[k] = (int)W.ids[k];
  }
}

// The reduce-scatter of the raster backward on values 0 to 5 and 4 to 9, each
// total stored by the lane that stores it there (of the eight l, added up here).
__global__ void k_wave_sum_test(const float* in, float* out, int n_waves) {
  constexpr int NV = kWaveSumValues;
  const int w = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  if (w >= n_waves) return;     // whole waves exit together
  const int lane = threadIdx.x & 63, value = rows8_value(lane);
  for (int first = 0; first <= NV - 6; first += NV - 6) {
    float v[6], x[2];
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = in[((int64_t)w * NV + first + i) * 64 + lane];
    rows8_reduce_scatter(v, x);
    float t = lane & 8 ? x[1] : x[0];
    for (int off = 4; off >= 1; off >>= 1) t += __shfl_xor(t, off);
    if ((lane & 7) == 0 && value >= 0) out[(int64_t)w * NV + first + value] = t;
  }
}

}  // namespace

hipError_t launch_take_counts(unsigned long long* d, unsigned long long* host, hipStream_t st) {
  k_take_counts<<<1, 64, 0, st>>>(d, host);
  return hipGetLastError();
}

// One session with few chunks and tiles: the scan adds the chunks' counts
// itself, a launch less, while one workgroup reads them faster than that launch
// takes.  Scan and sums, so and with the launch: 20 chunks of 300 tiles 6.2 and
// 8.2 us, 61 of 1196 13.8 and 10.4, 98 of 1200 12.2 and 9.9.
constexpr int64_t kDirectCounts = 16384;

hipError_t launch_forward_prep(const Batch& b, const WsPtrs& w, unsigned long long* max_pairs,
                               bool reuse_lists, hipStream_t st, StageTimer* tm) {
  const bool one = b.n_sessions == 1;
  if (reuse_lists) {
    if (b.b_total > 0) {
      Scope sc(tm, kStPreprocess, st);
      if (one)
        k_preprocess<true, true><<<b.b_total, kGaussPerBlock, 0, st>>>(b, w);
      else
        k_preprocess<true, false><<<b.b_total, kGaussPerBlock, 0, st>>>(b, w);
    }
    return hipGetLastError();
  }
  const size_t lds = sizeof(uint32_t) * (size_t)(b.t_max > 0 ? b.t_max : 1);
  if (b.b_total <= 0) {
    // no Gaussians: k_preprocess (which zeroes the counters) does not run
    Scope sc(tm, kStInit, st);
    k_init<<<1, 8 * kOrderClasses, 0, st>>>(w);
  }
  if (b.b_total > 0) {
    Scope sc(tm, kStPreprocess, st);
    if (one)
      k_preprocess<false, true><<<b.b_total, kGaussPerBlock, 0, st>>>(b, w);
    else
      k_preprocess<false, false><<<b.b_total, kGaussPerBlock, 0, st>>>(b, w);
  }
  if (b.c_total > 0) {
    Scope sc(tm, kStBinCount, st);
    if (one)
      k_chunk_hist<true><<<b.c_total, kBinThreads, lds, st>>>(b, w);
    else
      k_chunk_hist<false><<<b.c_total, kBinThreads, lds, st>>>(b, w);
  }
  {
    Scope sc(tm, kStScan, st);
    const dim3 grid((b.t_total + kBlock - 1) / kBlock, kScanGroups);
    const uint32_t* src = w.gsum;
    int groups = kScanGroups;
    if (one && (int64_t)b.c_total * b.t_total <= kDirectCounts) {
      src = w.hist;
      groups = b.c_total;
    } else if (one) {
      k_tile_group_sums<true><<<grid, kBlock, 0, st>>>(b, w);
    } else {
      k_tile_group_sums<false><<<grid, kBlock, 0, st>>>(b, w);
    }
    if (b.t_total <= kScanPer * kScanThreads)
      k_scan_tiles<kScanPer><<<1, kScanThreads, 0, st>>>(w, src, groups, b.t_total, b.c_total,
                                                         max_pairs);
    else
      k_scan_tiles<kScanPerMany><<<1, kScanThreads, 0, st>>>(w, src, groups, b.t_total, b.c_total,
                                                             max_pairs);
  }
  if (b.c_total > 0) {
    Scope sc(tm, kStEmit, st);
    const size_t lds_emit = lds + sizeof(uint16_t) * kStagePairs;
    if (one)
      k_emit<true><<<b.c_total, kBinThreads, lds_emit, st>>>(b, w);
    else
      k_emit<false><<<b.c_total, kBinThreads, lds_emit, st>>>(b, w);
  }
  if (b.t_total > 0) {
    Scope sc(tm, kStSort, st);
    launch_tile_sort(b, w, st);
  }
  return hipGetLastError();
}

hipError_t launch_debug_stage(const Batch& b, const WsPtrs& w, float* stage, int* rect,
                              int* ranges, int* ids, int64_t ids_cap, hipStream_t st) {
  const int n = b.n_total > b.t_total ? b.n_total : b.t_total;
  const int grid = (n + 255) / 256 > 0 ? (n + 255) / 256 : 1;
  k_debug_stage<<<grid, 256, 0, st>>>(b, w, stage, rect, ranges, ids, ids_cap);
  return hipGetLastError();
}

hipError_t launch_wave_sum_test(const float* in, float* out, int n_waves, hipStream_t st) {
  if (n_waves <= 0) return hipSuccess;
  k_wave_sum_test<<<(n_waves + 3) / 4, 256, 0, st>>>(in, out, n_waves);
  return hipGetLastError();
}

}  // namespace rtgs
