// Step 5, preprocessing backpropagation (Sec. 2.2): the per-Gaussian 2D
// gradients merged by the raster backward are pushed through the EWA
// projection to the map parameters, and in tracking summed over Gaussians to
// the camera-pose gradient dL/dP (the paper's Preprocessing Engine and
// Merging Tree, Secs. 5.1 and 5.4).  In mapping the Adam update of the map
// (Sec. 3.1) can follow in the same pass.
//
// Two kernels.  The tile -> Gaussian merge (the role of the paper's Stage
// Buffer): each Gaussian's 2D gradient is the fixed-order sum of its
// (tile, Gaussian, quadrant) slots, 40 B each.  Then one thread per Gaussian in float64 through the
// projection (56 B of parameters and 40 B of merged gradient in), writing
// the gradients (56 B) or, fused, applying Adam to the Gaussian's 14
// parameters right away (parameters and both moments read and written,
// 280 B), so the gradients never go through memory.  That kernel needs many
// float64 registers, hence few waves: the merge stays apart, where
// occupancy hides its loads.  The pose partials are summed per workgroup in
// LDS, then per session in a fixed order by a third kernel, so the pose
// reduction adds no float atomics of its own.
//
// Chain (all derivatives exact for the forward of forward_prep.hip):
//   conic (a, b, c) -> Sigma' :  dL/dSigma' = -M G_M M,  G_M = [[ga, gb/2],
//                                [gb/2, gc]]
//   Sigma' = A A^T + 0.3 I, A = T M, T = J W, M = R diag(s):
//     dL/dA = 2 G' A,  dL/dM = T^T dL/dA,  dL/dT = dL/dA M^T
//   T = J W:  dL/dJ = dL/dT W^T,  dL/dW|cov = J^T dL/dT
//   J(p), u(p), v(p), z: dL/dp;  dL/dmu = W^T dL/dp
//   view matrix [W | t]: dL/dW = dL/dW|cov + dL/dp mu^T, dL/dt = dL/dp,
//     summed over Gaussians; the pose (left perturbation at xi = 0) is then
//     dL/drho = dL/dt and dL/dphi = the axial vector of the antisymmetric
//     part of A = dL/dW W^T + dL/dt t^T: (A21 - A12, A02 - A20, A10 - A01)
//   M -> scales (dL/dl = s dL/ds) and R(q/|q|) -> quaternion.
#include "rtgs_internal.h"

namespace rtgs {
namespace {

// Sums over runs of LANES (8 or 16) lanes of each DPP row; the run's last
// lane holds its total.
template <int LANES, int NV>
__device__ __forceinline__ void row_sums(float (&acc)[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    float v = acc[i];
    v += dpp_f<kDppRowShr1, 0xf, true>(v);
    v += dpp_f<kDppRowShr2, 0xf, true>(v);
    v += dpp_f<kDppRowShr4, 0xf, true>(v);
    if (LANES == 16) v += dpp_f<kDppRowShr8, 0xf, true>(v);
    acc[i] = v;
  }
}

// Tile -> Gaussian merge: the quadrant sums of each Gaussian's pairs added up.
// A pair's four flag bytes say which of its sums the raster backward wrote (at
// 1200x680 / 300k three pairs in ten have any); only those are read, and the
// flags are zeroed for the next backward.
//
// Bound by memory latency (the sums' loads depend on the flags') and by the
// spread of the work: a Gaussian touches from one pair to over a thousand, and
// following each Gaussian's flags with lanes of its own makes the largest
// Gaussians' chains of dependent loads the kernel's time.  So the work is cut
// by pairs: a window is kWindow consecutive pairs of one binning chunk (the
// emit lists the windows, and each chunk's Gaussians that have pairs).  A
// workgroup reads a window's flags together and lists the items (pair,
// quadrant) found in LDS; then 8 lanes per Gaussian, or a wave for one with
// more than kItemsWave items, add its items.  A Gaussian that crosses a
// window's end leaves a partial sum per window in `edge`, added up in window
// order by the preprocessing backward.  Every sum is in a fixed order:
// deterministic.  1200x680 / 300k: 38 us (42 with a store a value and the scan by
// shuffles, and, of that form: 8 lanes per Gaussian following its own
// flags 72, all items staged in LDS first 47 to 57, kItemsWave 64 no change, 128
// three more, the next window's flags prefetched no change; the wave's sums in
// float four less, with a larger error than a slot by slot sum).
constexpr int kItemsWave = 32;

// A pair's flag bytes (0 or 1) as four bits.
__device__ __forceinline__ uint32_t live_bits(uint32_t f) {
  return (f & 1u) | ((f >> 7) & 2u) | ((f >> 14) & 4u) | ((f >> 21) & 8u);
}

// acc += the sums of items lo + lane, lo + lane + LANES, ... below hi of the
// list, two in flight; src: the window's first slot.
template <int NV, int LANES, typename Acc>
__device__ __forceinline__ void add_items(const float2* src, const uint16_t* list, int lo, int hi,
                                          int lane, Acc (&acc)[NV]) {
  for (int i0 = lo + lane; i0 < hi; i0 += 2 * LANES) {
    const bool two = i0 + LANES < hi;
    const int a = (int)list[i0], b = two ? (int)list[i0 + LANES] : a;
    float2 v[NV / 2], w[NV / 2];
    // NV floats at an 8-byte aligned offset: NV / 2 8-byte loads
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
      v[i] = src[a * (NV / 2) + i];
      w[i] = src[b * (NV / 2) + i];
    }
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
      acc[2 * i] += v[i].x;
      acc[2 * i + 1] += v[i].y;
    }
    if (two) {
#pragma unroll
      for (int i = 0; i < NV / 2; ++i) {
        acc[2 * i] += w[i].x;
        acc[2 * i + 1] += w[i].y;
      }
    }
  }
}

// a + b of a pair of doubles after swapping halves (32) or rows (16) of lanes,
// as swap32_add and swap16_add do for floats.
template <int LANES>
__device__ __forceinline__ double swap_add(double a, double b) {
  const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const unsigned xl = (unsigned)x, xh = (unsigned)(x >> 32);
  const unsigned yl = (unsigned)y, yh = (unsigned)(y >> 32);
  unsigned l0, l1, h0, h1;
  if (LANES == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    l0 = l[0]; l1 = l[1]; h0 = h[0]; h1 = h[1];
  }
  return __longlong_as_double(((unsigned long long)h0 << 32) | l0) +
         __longlong_as_double(((unsigned long long)h1 << 32) | l1);
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const unsigned long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Wavefront reduce-scatter of NV doubles (NV / 2 odd): halves, then rows, then
// along the rows.  Lane 16 (2 h + p) + 15 ends with the totals of values
// h NV / 2 + p + 2 j in x[j] for j < NV / 4, of h NV / 2 + NV / 2 - 1 in x[NV / 4].
template <int NV>
__device__ __forceinline__ void wave_sums(const double (&v)[NV], double (&x)[(NV / 2 + 1) / 2]) {
  constexpr int H = NV / 2;
  double w[H];
#pragma unroll
  for (int i = 0; i < H; ++i) w[i] = swap_add<32>(v[i], v[i + H]);
#pragma unroll
  for (int j = 0; j < (H + 1) / 2; ++j) {
    double s = swap_add<16>(w[2 * j], w[2 * j + 1 < H ? 2 * j + 1 : 2 * j]);
    s += dpp_d<kDppRowShr1>(s);
    s += dpp_d<kDppRowShr2>(s);
    s += dpp_d<kDppRowShr4>(s);
    s += dpp_d<kDppRowShr8>(s);
    x[j] = s;
  }
}

// Stores sum i over window w (pairs [p0, p1)) of the Gaussian with pairs
// [first, last): to grad2d, or to the window's edge it crosses (see
// merged_sums; in double, as what many windows' sums add up to may cancel).
template <typename Acc>
__device__ __forceinline__ void merge_store(const WsPtrs& W, int w, uint32_t p0, uint32_t p1,
                                            uint32_t gid, uint32_t first, uint32_t last, int i,
                                            Acc v) {
  if (first >= p0 && last <= p1)
    W.grad2d[(int64_t)gid * 10 + i] = (float)v;
  else
    W.edge[((int64_t)w * 2 + (first < p0 ? 0 : 1)) * 10 + i] = (double)v;
}

template <int NV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7)))
void k_merge(Batch B, WsPtrs W) {
  static_assert(kWindow == 512, "two pairs a thread");
  __shared__ uint16_t s_item[4 * kWindow];            // 4 pair + quadrant, in order
  __shared__ uint16_t s_cum[kWindow + 1];             // items before each pair
  __shared__ uint32_t s_w[4];
  __shared__ int s_big[4 * kWindow / kItemsWave], s_nbig;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = tid & 7;
  uint32_t* const live = reinterpret_cast<uint32_t*>(W.live);
  if (W.counters[0] > W.cap) return;                  // no lists
  const int n_win = (int)W.win_off[B.c_total];
  for (int w = blockIdx.x; w < n_win; w += gridDim.x) {
    const uint4 d = W.window[w];                      // pairs [x, y), list entries [z, w]
    const uint32_t p0 = d.x, p1 = d.y;
    if (p0 < W.sum_lo) {                              // of the pass before; its last pairs
      for (uint32_t p = W.sum_lo + tid; p < p1; p += 256) live[p] = 0u;   // are set again in this one
      continue;
    }
    if (p0 - W.sum_lo >= W.sum_span) continue;        // of a later pass
    const uint32_t a = p0 + tid, b = a + 256;
    const uint32_t fa = a < p1 ? live[a] : 0u, fb = b < p1 ? live[b] : 0u;
    if (tid == 0) s_nbig = 0;
    // items before each pair: one scan for the two halves of the pairs
    const uint32_t have = (uint32_t)__popc(fa) | ((uint32_t)__popc(fb) << 16);
    const uint32_t x = wave_scan(have);
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      before += q < wave ? s_w[q] : 0u;
      all += s_w[q];
    }
    const uint32_t ex = before + x - have;
    const int na = (int)(all & 0xffffu);
    int at = (int)(ex & 0xffffu);
    s_cum[tid] = (uint16_t)at;
    for (uint32_t m = live_bits(fa); m; m &= m - 1)
      s_item[at++] = (uint16_t)(4 * tid + __builtin_ctz(m));
    at = na + (int)(ex >> 16);
    s_cum[256 + tid] = (uint16_t)at;
    for (uint32_t m = live_bits(fb); m; m &= m - 1)
      s_item[at++] = (uint16_t)(4 * (256 + tid) + __builtin_ctz(m));
    if (tid == 0) s_cum[kWindow] = (uint16_t)(na + (int)(all >> 16));
    __syncthreads();
    if (fa) live[a] = 0u;
    if (fb) live[b] = 0u;
    const float2* const src = reinterpret_cast<const float2*>(W.partial + (int64_t)(p0 - W.sum_lo) * 4 * NV);
    for (uint32_t e0 = d.z; e0 <= d.w; e0 += 256 / 8) {
      const uint32_t e = e0 + tid / 8;
      uint2 g = make_uint2(0, 0);
      uint32_t last = 0;
      int lo = 0, hi = 0;
      bool mine = e <= d.w;
      if (mine) {
        g = W.vlist[e];                               // Gaussian, its first pair
        last = W.vlist[e + 1].y;                      // the next one's, or the chunk's end
        lo = s_cum[g.y > p0 ? g.y - p0 : 0u];
        hi = s_cum[min(last - p0, (uint32_t)kWindow)];
        if (hi - lo > kItemsWave) {
          if (sub == 0) s_big[atomicAdd(&s_nbig, 1)] = (int)e;
          mine = false;
          hi = lo;
        }
      }
      float acc[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i) acc[i] = 0.f;
      add_items<NV, 8>(src, s_item, lo, hi, sub, acc);
      row_sums<8, NV>(acc);
      if (mine && sub == 7) {
        if (g.y >= p0 && last <= p1) {
          float2* dst = reinterpret_cast<float2*>(W.grad2d + (int64_t)g.x * 10);
#pragma unroll
          for (int i = 0; i < NV / 2; ++i) dst[i] = make_float2(acc[2 * i], acc[2 * i + 1]);
        } else {
          double2* dst = reinterpret_cast<double2*>(W.edge + ((int64_t)w * 2 + (g.y < p0 ? 0 : 1)) * 10);
#pragma unroll
          for (int i = 0; i < NV / 2; ++i)
            dst[i] = make_double2((double)acc[2 * i], (double)acc[2 * i + 1]);
        }
      }
    }
    __syncthreads();
    // the list's order depends on timing; each Gaussian's sum does not
    const int nbig = s_nbig;
    for (int q = wave; q < nbig; q += 4) {
      const uint32_t e = (uint32_t)s_big[q];
      const uint2 g = W.vlist[e];
      const uint32_t last = W.vlist[e + 1].y;
      const int lo = s_cum[g.y > p0 ? g.y - p0 : 0u], hi = s_cum[min(last - p0, (uint32_t)kWindow)];
      // (in double: a float's error would grow with the number of items)
      double acc[NV], x[(NV / 2 + 1) / 2];
#pragma unroll
      for (int i = 0; i < NV; ++i) acc[i] = 0.0;
      add_items<NV, 64>(src, s_item, lo, hi, lane, acc);
      wave_sums<NV>(acc, x);
      if ((lane & 15) == 15) {
        const int odd = (lane >> 4) & 1, v0 = (lane >> 5) * (NV / 2);
#pragma unroll
        for (int j = 0; j < NV / 4; ++j)
          merge_store(W, w, p0, p1, g.x, g.y, last, v0 + odd + 2 * j, x[j]);
        if (!odd) merge_store(W, w, p0, p1, g.x, g.y, last, v0 + NV / 2 - 1, x[NV / 4]);
      }
    }
    __syncthreads();                                  // the LDS lists are reused
  }
}

// The merged sums of a Gaussian: of its one window, or its partial sums over
// the windows it crosses, in order (the end of the first, the beginning of
// each following one).  c: its chunk; [first, last): its pairs.
template <int NV>
__device__ __forceinline__ void merged_sums(const WsPtrs& W, int c, int64_t gid, uint32_t first,
                                            uint32_t n, double (&m)[NV]) {
  const uint32_t c0 = W.chunk_off[c];
  const int w0 = (int)(W.win_off[c] + (first - c0) / kWindow);
  const int w1 = (int)(W.win_off[c] + (first + n - 1 - c0) / kWindow);
  if (w0 == w1) {
    const float* p = W.grad2d + gid * 10;
#pragma unroll
    for (int i = 0; i < NV; ++i) m[i] = p[i];
    return;
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) m[i] = W.edge[((int64_t)w0 * 2 + 1) * 10 + i];
  for (int w = w0 + 1; w <= w1; ++w)
#pragma unroll
    for (int i = 0; i < NV; ++i) m[i] += W.edge[(int64_t)w * 2 * 10 + i];
}

// Bound by memory latency behind few waves (float64 registers), so what a call
// does not write is not compiled into its kernel (pose only 162 -> 114
// registers), and the pose's partials are summed by lane swaps instead of
// shuffles through LDS: pose only 1200x680 / 500k 25 -> 16 us, six served frames
// 74 -> 34 us; all gradients and the pose 34 -> 32 us (kept to three waves a
// SIMD, which spills, 36); Adam fused, 300k: 32 us, the rate of a copy.
template <int NV, bool ADAM, bool ONE, bool SCORE, bool POSE>
__global__ __launch_bounds__(kGaussPerBlock) __attribute__((amdgpu_waves_per_eu(NV == 6 ? 4 : POSE ? 2 : 3)))
void k_gauss_bwd(Batch B, WsPtrs W, int flags) {
  __shared__ double s_red[kGaussPerBlock / 64][12];
  const int s = ONE ? 0 : find_session(session_table(B), B.n_sessions, (int)blockIdx.x,
                                       [](const SessionDev& x) { return x.block_base; });
  const SessionDev& S = batch_session<ONE>(B, s);
  const int li0 = ((int)blockIdx.x - S.block_base) * kGaussPerBlock;
  // ---- projection backward, one thread per Gaussian
  const int li = li0 + (int)threadIdx.x;
  constexpr bool want_map = NV == 10;
  const bool want_cov = (flags & RTGS_GRAD_COV3D) != 0 && S.g_cov3d != nullptr;
  // score inputs only (dL/dmu, dL/dSigma) on the pose-only raster path
  const bool want_score = SCORE && S.g_means != nullptr && S.g_cov3d != nullptr;
  double pose[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};   // dL/dW (9), dL/dt (3)
  if (li < S.n) {
    const int gid = S.gauss_base + li;
    const int4 rect = W.rect[gid];
    double gm[3] = {0, 0, 0}, gl[3] = {0, 0, 0}, gq[4] = {0, 0, 0, 0}, go_eta = 0;
    double gcol[3] = {0, 0, 0}, gsig[6] = {0, 0, 0, 0, 0, 0};
    if (rect.z >= rect.x) {
      // the Gaussian's sums of the raster backward; pose only: without those
      // of the opacity and the colours
      double g2[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      if (W.counters[0] <= W.cap) {       // no pairs have sums after an overflow
        double m[NV];
        merged_sums<NV>(W, S.chunk_base + li0 / kChunk, gid, W.goff[gid],
                        (uint32_t)((rect.z - rect.x + 1) * (rect.w - rect.y + 1)), m);
        if (NV == 10) {
#pragma unroll
          for (int i = 0; i < 10; ++i) g2[i] = m[i];
        } else {
#pragma unroll
          for (int i = 0; i < 5; ++i) g2[i] = m[i];
          g2[9] = m[5];
        }
      }
      gcol[0] = g2[6]; gcol[1] = g2[7]; gcol[2] = g2[8];
      const double gdep = g2[9];
      double vm[12];
      for (int k = 0; k < 12; ++k) vm[k] = S.viewmat[k];
      const double mx = S.means[3 * li], my = S.means[3 * li + 1], mz = S.means[3 * li + 2];
      const double qw = S.quats[4 * li], qx = S.quats[4 * li + 1];
      const double qy = S.quats[4 * li + 2], qz = S.quats[4 * li + 3];
      double sc[3], o;
      activate(S, li, sc, o);
      const double x = vm[0] * mx + vm[1] * my + vm[2] * mz + vm[3];
      const double y = vm[4] * mx + vm[5] * my + vm[6] * mz + vm[7];
      const double z = vm[8] * mx + vm[9] * my + vm[10] * mz + vm[11];
      // reciprocals taken once (a float64 division is a long instruction sequence)
      const double qn = sqrt(qw * qw + qx * qx + qy * qy + qz * qz), iqn = 1.0 / qn;
      const double w = qw * iqn, a = qx * iqn, b = qy * iqn, c = qz * iqn;
      const double R[9] = {1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                           2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                           2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)};
      double M[9];
      for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) M[3 * r + k] = R[3 * r + k] * sc[k];
      const double limx = kFovClamp * 0.5 * S.width / S.fx;
      const double limy = kFovClamp * 0.5 * S.height / S.fy;
      const double iz = 1.0 / z, iz2 = iz * iz, iz3 = iz2 * iz;
      const double rx = x * iz, ry = y * iz;
      const bool inx = rx > -limx && rx < limx, iny = ry > -limy && ry < limy;
      const double tx = fmin(limx, fmax(-limx, rx)), ty = fmin(limy, fmax(-limy, ry));
      const double j00 = S.fx * iz, j02 = -S.fx * tx * iz, j11 = S.fy * iz, j12 = -S.fy * ty * iz;
      double T0[3], T1[3], A0[3], A1[3];
      for (int k = 0; k < 3; ++k) {
        T0[k] = j00 * vm[k] + j02 * vm[8 + k];
        T1[k] = j11 * vm[4 + k] + j12 * vm[8 + k];
      }
      for (int k = 0; k < 3; ++k) {
        A0[k] = T0[0] * M[k] + T0[1] * M[3 + k] + T0[2] * M[6 + k];
        A1[k] = T1[0] * M[k] + T1[1] * M[3 + k] + T1[2] * M[6 + k];
      }
      const double sxx = A0[0] * A0[0] + A0[1] * A0[1] + A0[2] * A0[2] + kDilation;
      const double sxy = A0[0] * A1[0] + A0[1] * A1[1] + A0[2] * A1[2];
      const double syy = A1[0] * A1[0] + A1[1] * A1[1] + A1[2] * A1[2] + kDilation;
      const double inv = 1.0 / (sxx * syy - sxy * sxy);
      const double ca = syy * inv, cb = -sxy * inv, cc = sxx * inv;
      // the conic and the opacity applied to the sums over pixels
      const double gu = ca * g2[0] + cb * g2[1], gv = cb * g2[0] + cc * g2[1];
      const double ga = 0.5 * g2[2], gb = g2[3], gc = 0.5 * g2[4];
      // dL/dSigma' (symmetric matrix entries)
      const double Gxx = -(ga * ca * ca + gb * ca * cb + gc * cb * cb);
      const double Gyy = -(ga * cb * cb + gb * cb * cc + gc * cc * cc);
      const double Gxy = -(ga * ca * cb + 0.5 * gb * (ca * cc + cb * cb) + gc * cb * cc);
      double dA0[3], dA1[3], dM[9], dT0[3], dT1[3];
      for (int k = 0; k < 3; ++k) {
        dA0[k] = 2.0 * (Gxx * A0[k] + Gxy * A1[k]);
        dA1[k] = 2.0 * (Gxy * A0[k] + Gyy * A1[k]);
      }
      for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) dM[3 * r + k] = T0[r] * dA0[k] + T1[r] * dA1[k];
      for (int r = 0; r < 3; ++r) {
        dT0[r] = dA0[0] * M[3 * r] + dA0[1] * M[3 * r + 1] + dA0[2] * M[3 * r + 2];
        dT1[r] = dA1[0] * M[3 * r] + dA1[1] * M[3 * r + 1] + dA1[2] * M[3 * r + 2];
      }
      // T0 = j00 W0 + j02 W2, T1 = j11 W1 + j12 W2 (W rows)
      const double dj00 = dT0[0] * vm[0] + dT0[1] * vm[1] + dT0[2] * vm[2];
      const double dj02 = dT0[0] * vm[8] + dT0[1] * vm[9] + dT0[2] * vm[10];
      const double dj11 = dT1[0] * vm[4] + dT1[1] * vm[5] + dT1[2] * vm[6];
      const double dj12 = dT1[0] * vm[8] + dT1[1] * vm[9] + dT1[2] * vm[10];
      double dW[9];
      for (int k = 0; k < 3; ++k) {
        dW[k] = j00 * dT0[k];
        dW[3 + k] = j11 * dT1[k];
        dW[6 + k] = j02 * dT0[k] + j12 * dT1[k];
      }
      // dL/dp from u, v, J and the depth output
      double gx = gu * S.fx * iz + (inx ? dj02 * (-S.fx * iz2) : 0.0);
      double gy = gv * S.fy * iz + (iny ? dj12 * (-S.fy * iz2) : 0.0);
      const double dj02dz = S.fx * tx * iz2 + (inx ? S.fx * x * iz3 : 0.0);
      const double dj12dz = S.fy * ty * iz2 + (iny ? S.fy * y * iz3 : 0.0);
      double gz = gdep - gu * S.fx * x * iz2 - gv * S.fy * y * iz2 - dj00 * S.fx * iz2 -
                  dj11 * S.fy * iz2 + dj02 * dj02dz + dj12 * dj12dz;
      // view matrix: dL/dW = dL/dW|cov + dL/dp mu^T, dL/dt = dL/dp
      const double gp3[3] = {gx, gy, gz}, mu[3] = {mx, my, mz};
      for (int i = 0; i < 3; ++i) {
        for (int j = 0; j < 3; ++j) pose[3 * i + j] = dW[3 * i + j] + gp3[i] * mu[j];
        pose[9 + i] = gp3[i];
      }
      if (want_score) {
        for (int k = 0; k < 3; ++k) gm[k] = vm[k] * gx + vm[4 + k] * gy + vm[8 + k] * gz;
        double GT0[3], GT1[3];
        for (int k = 0; k < 3; ++k) {
          GT0[k] = Gxx * T0[k] + Gxy * T1[k];
          GT1[k] = Gxy * T0[k] + Gyy * T1[k];
        }
        const int ii[6] = {0, 0, 0, 1, 1, 2}, jj[6] = {0, 1, 2, 1, 2, 2};
        for (int k = 0; k < 6; ++k) gsig[k] = T0[ii[k]] * GT0[jj[k]] + T1[ii[k]] * GT1[jj[k]];
      }
      if (want_map) {
        // dL/dmu = W^T dL/dp
        for (int k = 0; k < 3; ++k) gm[k] = vm[k] * gx + vm[4 + k] * gy + vm[8 + k] * gz;
        // M = R diag(s): dR[r][k] = dM[r][k] s_k, ds_k = sum_r R[r][k] dM[r][k]
        double dR[9];
        for (int r = 0; r < 3; ++r)
          for (int k = 0; k < 3; ++k) dR[3 * r + k] = dM[3 * r + k] * sc[k];
        for (int k = 0; k < 3; ++k)
          gl[k] = sc[k] * (R[k] * dM[k] + R[3 + k] * dM[3 + k] + R[6 + k] * dM[6 + k]);
        // R(w, a, b, c) -> unit-quaternion gradient
        const double gw =
            2 * (-c * dR[1] + b * dR[2] + c * dR[3] - a * dR[5] - b * dR[6] + a * dR[7]);
        const double gx4 = 2 * (b * dR[1] + c * dR[2] + b * dR[3] - 2 * a * dR[4] - w * dR[5] +
                                c * dR[6] + w * dR[7] - 2 * a * dR[8]);
        const double gy4 = 2 * (-2 * b * dR[0] + a * dR[1] + w * dR[2] + a * dR[3] + c * dR[5] -
                                w * dR[6] + c * dR[7] - 2 * b * dR[8]);
        const double gz4 = 2 * (-2 * c * dR[0] - w * dR[1] + a * dR[2] + w * dR[3] - 2 * c * dR[4] +
                                b * dR[5] + a * dR[6] + b * dR[7]);
        const double dot = w * gw + a * gx4 + b * gy4 + c * gz4;
        gq[0] = (gw - w * dot) * iqn;
        gq[1] = (gx4 - a * dot) * iqn;
        gq[2] = (gy4 - b * dot) * iqn;
        gq[3] = (gz4 - c * dot) * iqn;
        go_eta = -g2[5] * (1.0 - o);       // dL/do = -(sum of n) / o
        if (want_cov) {
          // dL/dSigma = T^T G' T
          double GT0[3], GT1[3];
          for (int k = 0; k < 3; ++k) {
            GT0[k] = Gxx * T0[k] + Gxy * T1[k];
            GT1[k] = Gxy * T0[k] + Gyy * T1[k];
          }
          const int ii[6] = {0, 0, 0, 1, 1, 2}, jj[6] = {0, 1, 2, 1, 2, 2};
          for (int k = 0; k < 6; ++k) gsig[k] = T0[ii[k]] * GT0[jj[k]] + T1[ii[k]] * GT1[jj[k]];
        }
      }
    }
    if (want_map) {
      if (S.g_means) for (int k = 0; k < 3; ++k) S.g_means[3 * li + k] = (float)gm[k];
      if (S.g_log_scales) for (int k = 0; k < 3; ++k) S.g_log_scales[3 * li + k] = (float)gl[k];
      if (S.g_quats) for (int k = 0; k < 4; ++k) S.g_quats[4 * li + k] = (float)gq[k];
      if (S.g_opac) S.g_opac[li] = (float)go_eta;
      if (S.g_colors) for (int k = 0; k < 3; ++k) S.g_colors[3 * li + k] = (float)gcol[k];
      if (want_cov) for (int k = 0; k < 6; ++k) S.g_cov3d[6 * li + k] = (float)gsig[k];
    }
    if (want_score) {
      for (int k = 0; k < 3; ++k) S.g_means[3 * li + k] = (float)gm[k];
      for (int k = 0; k < 6; ++k) S.g_cov3d[6 * li + k] = (float)gsig[k];
    }
    // ---- Adam on the Gaussian's parameters (the update of adam_step, on
    // the same float32 gradients).  The constants, then every parameter and
    // moment, are read before the first store: the stores may alias them, so
    // read element by element each would wait for the previous one's store.
    if (ADAM && S.adam.on) {
      const MapAdamDev& A = S.adam;
      const float beta1 = A.beta1, beta2 = A.beta2, omb1 = A.omb1, omb2 = A.omb2, eps = A.eps;
      const float isb2 = A.inv_sqrt_bc2;
      float step[5];
      float* par[5] = {const_cast<float*>(S.means), const_cast<float*>(S.log_scales),
                       const_cast<float*>(S.quats), const_cast<float*>(S.opac),
                       const_cast<float*>(S.colors)};
      float *pm[5], *pv2[5];
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        step[t] = A.step_size[t];
        pm[t] = A.m[t];
        pv2[t] = A.v[t];
      }
      const float g14[14] = {(float)gm[0], (float)gm[1], (float)gm[2], (float)gl[0],
                             (float)gl[1], (float)gl[2], (float)gq[0], (float)gq[1],
                             (float)gq[2], (float)gq[3], (float)go_eta, (float)gcol[0],
                             (float)gcol[1], (float)gcol[2]};
      constexpr int kDim[5] = {3, 3, 4, 1, 3};
      float P[14], Mo[14], Vo[14];
      {
        int at = 0;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
#pragma unroll
          for (int k = 0; k < kDim[t]; ++k) {
            const int64_t e = (int64_t)kDim[t] * li + k;
            P[at + k] = par[t][e];
            Mo[at + k] = pm[t][e];
            Vo[at + k] = pv2[t][e];
          }
          at += kDim[t];
        }
      }
      {
        int at = 0;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
#pragma unroll
          for (int k = 0; k < kDim[t]; ++k)
            adam_update(P[at + k], g14[at + k], Mo[at + k], Vo[at + k], beta1, beta2, omb1, omb2,
                        eps, step[t], isb2);
          at += kDim[t];
        }
      }
      {
        int at = 0;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
#pragma unroll
          for (int k = 0; k < kDim[t]; ++k) {
            const int64_t e = (int64_t)kDim[t] * li + k;
            par[t][e] = P[at + k];
            pm[t][e] = Mo[at + k];
            pv2[t][e] = Vo[at + k];
          }
          at += kDim[t];
        }
      }
    }
  }
  // block partial of the pose gradient: wave shuffles, then the 4 waves in LDS
  if (!POSE) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 12; k += 6) {
    const double v[6] = {pose[k],     pose[k + 1], pose[k + 2],
                         pose[k + 3], pose[k + 4], pose[k + 5]};
    double x[2];
    wave_sums<6>(v, x);
    if ((lane & 15) == 15) {
      const int h = lane >> 5, p = (lane >> 4) & 1;
      s_red[wave][k + 3 * h + p] = x[0];
      if (p == 0) s_red[wave][k + 3 * h + 2] = x[1];
    }
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    double t = 0;
    for (int q = 0; q < kGaussPerBlock / 64; ++q) t += s_red[q][threadIdx.x];
    W.pose_part[(int64_t)blockIdx.x * 16 + threadIdx.x] = t;
  }
}

// One workgroup per session: fixed-order sum of its block partials into the
// view-matrix gradient, and the pose (left-perturbation) gradient from it.
// One workgroup a session: 1024 threads so that the blocks' partials are in
// flight together, then lane swaps and one pass through LDS (500k Gaussians:
// 256 threads and a tree in LDS 10.5 -> 9 us; 100k 5.8 -> 4.7).
constexpr int kReduceThreads = 1024;

__global__ __launch_bounds__(kReduceThreads) void k_pose_reduce(Batch B, WsPtrs W) {
  __shared__ double s_acc[kReduceThreads / 64][12];
  const SessionDev& S = session_of(B, blockIdx.x);
  const int b0 = S.block_base;
  const int b1 = (blockIdx.x + 1 < (unsigned)B.n_sessions)
                     ? session_of(B, blockIdx.x + 1).block_base
                     : B.b_total;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double acc[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = b0 + (int)threadIdx.x; b < b1; b += kReduceThreads) {
    const double2* p = reinterpret_cast<const double2*>(W.pose_part + (int64_t)b * 16);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const double2 v = p[k];
      acc[2 * k] += v.x;
      acc[2 * k + 1] += v.y;
    }
  }
#pragma unroll
  for (int k = 0; k < 12; k += 6) {
    const double v[6] = {acc[k], acc[k + 1], acc[k + 2], acc[k + 3], acc[k + 4], acc[k + 5]};
    double x[2];
    wave_sums<6>(v, x);
    if ((lane & 15) == 15) {
      const int h = lane >> 5, p = (lane >> 4) & 1;
      s_acc[wave][k + 3 * h + p] = x[0];
      if (p == 0) s_acc[wave][k + 3 * h + 2] = x[1];
    }
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    double t = 0;
    for (int q = 0; q < kReduceThreads / 64; ++q) t += s_acc[q][threadIdx.x];
    s_acc[0][threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double* g = s_acc[0];        // dL/dW row-major (9), dL/dt (3)
    if (S.g_viewmat)
      for (int i = 0; i < 3; ++i) {
        for (int j = 0; j < 3; ++j) S.g_viewmat[4 * i + j] = (float)g[3 * i + j];
        S.g_viewmat[4 * i + 3] = (float)g[9 + i];
      }
    if (S.g_pose6) {
      double vm[12];
      for (int k = 0; k < 12; ++k) vm[k] = S.viewmat[k];
      double A[9];                     // A = dL/dW W^T + dL/dt t^T
      for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
          A[3 * i + j] = g[3 * i] * vm[4 * j] + g[3 * i + 1] * vm[4 * j + 1] +
                         g[3 * i + 2] * vm[4 * j + 2] + g[9 + i] * vm[4 * j + 3];
      S.g_pose6[0] = (float)g[9];
      S.g_pose6[1] = (float)g[10];
      S.g_pose6[2] = (float)g[11];
      S.g_pose6[3] = (float)(A[7] - A[5]);
      S.g_pose6[4] = (float)(A[2] - A[6]);
      S.g_pose6[5] = (float)(A[3] - A[1]);
    }
  }
}

}  // namespace

template <int NV, bool ADAM, bool SCORE, bool POSE>
static void gauss_bwd(const Batch& b, const WsPtrs& w, int grad_flags, hipStream_t st) {
  if (b.n_sessions == 1)
    k_gauss_bwd<NV, ADAM, true, SCORE, POSE>
        <<<b.b_total, kGaussPerBlock, 0, st>>>(b, w, grad_flags);
  else
    k_gauss_bwd<NV, ADAM, false, SCORE, POSE>
        <<<b.b_total, kGaussPerBlock, 0, st>>>(b, w, grad_flags);
}

template <int NV, bool ADAM, bool SCORE>
static void gauss_bwd(const Batch& b, const WsPtrs& w, int grad_flags, hipStream_t st) {
  if (grad_flags & RTGS_GRAD_POSE)
    gauss_bwd<NV, ADAM, SCORE, true>(b, w, grad_flags, st);
  else
    gauss_bwd<NV, ADAM, SCORE, false>(b, w, grad_flags, st);
}

hipError_t launch_merge(const Batch& b, const WsPtrs& w, bool map, hipStream_t st, StageTimer* tm) {
  if (b.n_total > 0) {
    Scope sc(tm, kStMerge, st);
    // windows: at most one per kWindow pairs of capacity and one per chunk; a
    // workgroup takes several where the capacity leaves far more than the chip
    // holds at once
    const int64_t most = w.cap / kWindow + b.c_total;
    const int grid = (int)(most < 16384 ? most : 16384);
    if (map)
      k_merge<10><<<grid, 256, 0, st>>>(b, w);
    else
      k_merge<6><<<grid, 256, 0, st>>>(b, w);
  }
  return hipGetLastError();
}

hipError_t launch_preprocess_bwd(const Batch& b, const WsPtrs& w, int grad_flags, hipStream_t st,
                                 StageTimer* tm) {
  if (b.b_total > 0) {
    Scope sc(tm, kStPreprocessBwd, st);
    if (grad_flags & RTGS_GRAD_ADAM)
      gauss_bwd<10, true, false>(b, w, grad_flags, st);
    else if (grad_flags & RTGS_GRAD_MAP)
      gauss_bwd<10, false, false>(b, w, grad_flags, st);
    else if (grad_flags & RTGS_GRAD_SCORE)
      gauss_bwd<6, false, true>(b, w, grad_flags, st);
    else                                // the pose alone
      gauss_bwd<6, false, false, true>(b, w, grad_flags, st);
  }
  if ((grad_flags & RTGS_GRAD_POSE) && b.n_sessions > 0) {
    Scope sc(tm, kStPoseReduce, st);
    k_pose_reduce<<<b.n_sessions, kReduceThreads, 0, st>>>(b, w);
  }
  return hipGetLastError();
}

}  // namespace rtgs
