// Step 3 (rendering: alpha computing, Eq. 2, and alpha blending, Eq. 3) and
// Step 4 (rendering backpropagation, the exact derivative of Eq. 3 that
// Eqs. 4-5 sketch) for a batch of sessions sharing one tile space.
//
// Lists are per 16x16 tile; a workgroup is one wave64 with an 8x8 quadrant of a
// tile of its own, so a Gaussian whose ellipse misses a quadrant is skipped by
// that whole wave (the GPU counterpart of the paper's 4x4 subtiles) and no wave
// waits for another.
//
// Forward: per lane, alpha = min(0.99, o exp(power)); skip alpha < 1/255;
// stop before T would fall below 1e-4; saves final T and the position of the
// last blended pair (the per-pixel state the backward reuses instead of
// re-running the forward, the role of the paper's R&B buffer, Sec. 5.2).
// With a session's loss targets it also writes the gradient of the L1 loss
// (Eq. 6) of every pixel it writes, so no loss pass reads the image back.
//
// Backward: one wave per quadrant walks its part of the list from its last
// blended position down, recovering T before each blended fragment as
// T / (1 - alpha) (Eq. 5 read as the reverse recurrence) and the normalised
// suffix colour/depth.  The pixels' gradients of a list entry are summed per
// quadrant (k_raster_bwd) and stored in a slot of the (tile, Gaussian,
// quadrant): the pixel -> tile merge of the paper's Gradient Merging Unit
// (Sec. 5.3).  The tile -> Gaussian merge (its Stage Buffer) adds a Gaussian's
// slots in the preprocessing backward; no float atomics anywhere, so gradients
// are bitwise reproducible.
#include <type_traits>

#include "rtgs_internal.h"

namespace rtgs {
namespace {

// The tile and quadrant of a one-wave workgroup of the forward.  Workgroups
// are dealt round-robin to the 8 XCDs; each XCD gets a contiguous band of
// tiles, the four quadrants of a tile in a row, so neighbours share its L2
// (runs of 4 or 16 tiles dealt in turn: 3 of 87 us slower).
__device__ __forceinline__ bool wave_of_block(int t_total, int& tile, int& wave) {
  const int per = (t_total + 7) >> 3;
  tile = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 5);
  wave = ((int)blockIdx.x >> 3) & 3;
  return (int)(blockIdx.x >> 5) < per && tile < t_total;
}

// The backward takes a band's quadrants by falling work: at 12.9k waves on
// 6144 places (six a SIMD) the last waves to start decide when the kernel ends (taken in
// tile order it drained for 62 of 166 us at 1200x680 / 300k).  The forward
// files each quadrant under the entries it walked up to its last blended one,
// kOrderStep to a class.  Quadrants without work are not filed, nor those with
// little: they are marked and taken in tile order after the others, since filing
// thousands of them in one class makes their additions to its counter queue up
// (1920x1600 with 10k Gaussians: forward 107 us filed, 52 marked, 1200x680 with 2k 25
// and 14.5; marked below 16 entries only 60 and 14.6, below 48 as below 32; the
// backward 84 and 91 us, 15 and 17).
constexpr int kOrderStep = 16, kSmallWork = 32;
static_assert(kOrderClasses == 32, "a class per lane of half a wave");

__device__ __forceinline__ void file_work(const WsPtrs& W, int t_total, int tile, int wave,
                                          int entries) {
  const bool small = entries < kSmallWork;
  W.small[4 * (int64_t)tile + wave] = small && entries > 0;
  if (small) return;
  const int per = (t_total + 7) >> 3, band = (int)blockIdx.x & 7;
  const int cls = band * kOrderClasses +
                  min((entries - kSmallWork) / kOrderStep, kOrderClasses - 1);
  const uint32_t at = atomicAdd(&W.order_n[cls], 1u);
  W.order[(int64_t)cls * 4 * per + at] = (uint32_t)(4 * tile + wave);
}

// The tile and quadrant of a workgroup of the backward: the band's next one,
// classes from the largest; tile order without an order (see raster_order).
__device__ __forceinline__ bool wave_by_work(const WsPtrs& W, int t_total, int& tile, int& wave) {
  const int per = (t_total + 7) >> 3, band = (int)blockIdx.x & 7, lane = threadIdx.x;
  if (!W.order) return wave_of_block(t_total, tile, wave);
  uint32_t i = blockIdx.x >> 3;
  if (i >= (uint32_t)(4 * per)) {          // a quadrant with little work, in tile order
    i -= (uint32_t)(4 * per);
    tile = band * per + (int)(i >> 2);
    wave = (int)(i & 3u);
    return tile < t_total && W.small[4 * (int64_t)tile + wave] != 0;
  }
  const int cls = band * kOrderClasses + kOrderClasses - 1 - (lane & (kOrderClasses - 1));
  const uint32_t n = W.order_n[cls];
  uint32_t x = n;                          // inclusive scan from the largest class
#pragma unroll
  for (int off = 1; off < kOrderClasses; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, kOrderClasses);
    if ((lane & (kOrderClasses - 1)) >= off) x += y;
  }
  const unsigned long long past = __builtin_amdgcn_ballot_w64(x > i);
  if (past == 0) return false;
  const int c = __builtin_ctzll(past);     // lane of the class
  const uint32_t before = (uint32_t)__shfl(x - n, c);
  const int64_t list = (int64_t)(band * kOrderClasses + kOrderClasses - 1 - c) * 4 * per;
  const uint32_t q = __builtin_amdgcn_readfirstlane(W.order[list + (i - before)]);
  tile = (int)(q >> 2);
  wave = (int)(q & 3u);
  return tile < t_total;
}

// A tile holds 16x16 samples: one per pixel normally, or one per block of
// 2^sub_sx x 2^sub_sy pixels for a downsampled frame (the pixel the mask keeps
// in that block).  Wave w owns the 8x8 samples of quadrant w.
struct TileCtx {
  int s;
  int lt;                       // tile index within the session
  int tile_x0, tile_y0;         // first pixel of the tile
  int bx0, by0;                 // first pixel of this lane's sample block
  int px, py;                   // the lane's sample pixel
  bool inside;                  // the block lies (partly) in the image
  bool has;                     // a sample pixel exists (mask) in the block
  int pix;
};

// The sample a lane takes by default: wave w the 8x8 quadrant w.
__device__ __forceinline__ int quadrant_sample(int wave, int lane) {
  return ((wave >> 1) * 8 + (lane >> 3)) * 16 + (wave & 1) * 8 + (lane & 7);
}

// sidx: the thread's sample of the tile, row-major 0..255.
template <bool ONE>
__device__ __forceinline__ TileCtx tile_ctx(const Batch& B, int tile, int sidx) {
  TileCtx c;
  c.s = ONE ? 0
            : find_session(session_table(B), B.n_sessions, tile,
                           [](const SessionDev& x) { return x.tile_base; });
  const SessionDev& S = batch_session<ONE>(B, c.s);
  c.lt = tile - S.tile_base;
  c.tile_x0 = (c.lt % S.tiles_x) << (4 + S.sub_sx);
  c.tile_y0 = (c.lt / S.tiles_x) << (4 + S.sub_sy);
  const int sx = sidx & 15, sy = sidx >> 4;
  c.bx0 = c.tile_x0 + (sx << S.sub_sx);
  c.by0 = c.tile_y0 + (sy << S.sub_sy);
  c.inside = c.bx0 < S.width && c.by0 < S.height;
  c.px = c.bx0;
  c.py = c.by0;
  c.has = c.inside;
  if (c.inside && (S.sub_sx | S.sub_sy)) {
    // the block's sample: its first masked-in pixel in raster order
    c.has = false;
    const int x1 = min(S.width, c.bx0 + (1 << S.sub_sx));
    const int y1 = min(S.height, c.by0 + (1 << S.sub_sy));
    for (int y = c.by0; y < y1 && !c.has; ++y)
      for (int x = c.bx0; x < x1; ++x)
        if (S.pmask[y * S.width + x]) {
          c.px = x;
          c.py = y;
          c.has = true;
          break;
        }
  }
  c.pix = c.py * S.width + c.px;
  return c;
}

// Smallest value of the quadratic form q(d) = a dx^2 + 2 b dx dy + c dy^2
// over the box [x0, x1] x [y0, y1] of offsets d.  q decreases towards the
// centre (d = 0), so the least value lies where the box faces it: on the line
// dx = X, X the box's dx nearest 0, or dy = Y, each a 1D quadratic minimised
// in closed form and clamped to the box (both at d = 0 if the box holds it).
// ia, ic: 1/a and 1/c (0 where a or c is not positive).
__device__ __forceinline__ float box_min_quad(float a, float b, float c, float ia, float ic,
                                              float x0, float x1, float y0, float y1) {
  const float X = fminf(x1, fmaxf(x0, 0.f)), Y = fminf(y1, fmaxf(y0, 0.f));
  const float dy = fminf(y1, fmaxf(y0, -b * X * ic));
  const float dx = fminf(x1, fmaxf(x0, -b * Y * ia));
  const float b2 = 2.f * b;
  const float qx = __builtin_fmaf(a * X, X, dy * __builtin_fmaf(c, dy, b2 * X));
  const float qy = __builtin_fmaf(c * Y, Y, dx * __builtin_fmaf(a, dx, b2 * Y));
  return fminf(qx, qy);
}

// Whether the alpha >= 1/255 ellipse (q <= t) of the Gaussian can reach a
// pixel centre of the box of samples (x0, y0) to (x1, y1) of a tile at pixel
// (tx0, ty0), sample blocks of 2^sx x 2^sy pixels.  The margin keeps the test
// conservative against the float32 evaluation of alpha and of the test.
__device__ __forceinline__ bool box_hit(float4 r0, float4 r1, float level, int tx0, int ty0, int sx,
                                        int sy, int x0, int y0, int x1, int y1) {
  const float u = r0.x + r0.z, v = r0.y + r0.w;
  const float t = __builtin_fmaf(level, 1.f + 1e-3f, 1e-3f);
  const float ia = r1.x > 0.f ? __builtin_amdgcn_rcpf(r1.x) : 0.f;
  const float ic = r1.z > 0.f ? __builtin_amdgcn_rcpf(r1.z) : 0.f;
  const float qx0 = (float)(tx0 + (x0 << sx)) + 0.5f - u;
  const float qy0 = (float)(ty0 + (y0 << sy)) + 0.5f - v;
  const float qx1 = (float)(tx0 + ((x1 + 1) << sx) - 1) + 0.5f - u;
  const float qy1 = (float)(ty0 + ((y1 + 1) << sy) - 1) + 0.5f - v;
  return box_min_quad(r1.x, r1.y, r1.z, ia, ic, qx0, qx1, qy0, qy1) <= t;
}

// Index of the mask of list entries b0 to b0 + 63 (b0 = start + 64 j) that
// quadrant `wave` of a tile can reach: a tile's masks begin at
// start / 64 + tile, which leaves every tile room for its last, partial mask.
__device__ __forceinline__ int64_t hits_at(int start, int tile, int b0, int wave) {
  return ((int64_t)(start >> 6) + tile + ((b0 - start) >> 6)) * 4 + wave;
}

// Saved fragments (the per-fragment state of the paper's R&B buffer): for
// every list entry a wave evaluates, the 64-bit mask of its lanes that
// blended it, and for those lanes, in entry order and compacted by lane rank,
// (alpha, 1 - alpha) with alpha negated where it was clamped to 0.99.  The
// stream of wave w of a tile with list [start, end) begins at float2 index
// 64 (4 start + w (end - start)): room for every lane blending every entry.
__device__ __forceinline__ int64_t frag_base(int start, int end, int wave) {
  return 64 * (4 * (int64_t)start + (int64_t)wave * (end - start));
}

__device__ __forceinline__ uint32_t lane_rank(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A wave's 256 keys, four a lane, sorted by a bitonic network: compare-exchanges
// of every key with that of the lane whose position differs in bit BIT, positions
// being dealt so that the first bits are flipped by lane swaps, the others by DPP.
__device__ __forceinline__ int sort_position(int lane) {
  const int b2 = (lane >> 2) & 1;
  return ((lane >> 5) & 1) | (((lane >> 4) & 1) << 1) | (((lane & 1) ^ b2) << 2) |
         ((((lane >> 1) & 1) ^ b2) << 3) | (b2 << 4) | (((lane >> 3) & 1) << 5);
}

__device__ __forceinline__ void cas(uint32_t& a, uint32_t& b) {
  const uint32_t lo = min(a, b), hi = max(a, b);
  a = lo;
  b = hi;
}

template <int BIT>
__device__ __forceinline__ void merge_level(uint32_t (&k)[4], int pos) {
  if constexpr (BIT <= 1) {
#pragma unroll
    for (int s = 0; s < 4; s += 2) {
      // after the swap a lane holds both keys of a pair of lanes
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if constexpr (BIT == 0) {
          const auto x = __builtin_amdgcn_permlane32_swap(k[s], k[s + 1], false, false);
          const uint32_t a = x[0], b = x[1];
          k[s] = a; k[s + 1] = b;
        } else {
          const auto x = __builtin_amdgcn_permlane16_swap(k[s], k[s + 1], false, false);
          const uint32_t a = x[0], b = x[1];
          k[s] = a; k[s + 1] = b;
        }
        if (r == 0) cas(k[s], k[s + 1]);
      }
    }
  } else {
    // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_ror:8
    constexpr int kCtrl = BIT == 2 ? 0xB1 : BIT == 3 ? 0x4E : BIT == 4 ? 0x141 : kDppRowRor8;
    const bool upper = (pos >> BIT) & 1;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint32_t o =
          (uint32_t)__builtin_amdgcn_update_dpp(0, (int)k[s], kCtrl, 0xf, 0xf, true);
      k[s] = (k[s] < o) != upper ? k[s] : o;
    }
  }
  if constexpr (BIT > 0) {
    merge_level<BIT - 1>(k, pos);
  } else {
    cas(k[0], k[2]); cas(k[1], k[3]);
    cas(k[0], k[1]); cas(k[2], k[3]);
  }
}

// Keys of descending blocks are held inverted and sorted as the others.
__device__ __forceinline__ void invert_if(uint32_t (&k)[4], int bit) {
#pragma unroll
  for (int s = 0; s < 4; ++s) k[s] ^= bit & 1 ? ~0u : 0u;
}

// Lanes assigned by previous work (the GPU form of the paper's workload
// scheduling unit, Sec. 5.2): the tile's 256 samples sorted by the list
// entries each walked in a previous forward (S.lane_work; ties and missing
// values by sample index), wave w taking ranks 64 w to 64 w + 63, so each
// wave's lanes finish together.  Writes the permutation for both rasterizers.
// A wave a tile.  Bound by VALU issue: sorted in registers 1200x680 takes 5.9 us,
// where counting each key's rank over the other 255 in LDS took 15.
__global__ __launch_bounds__(64) void k_lane_schedule(Batch B, WsPtrs W) {
  const int tile = blockIdx.x, lane = threadIdx.x;
  const int s = find_session(session_table(B), B.n_sessions, tile,
                             [](const SessionDev& x) { return x.tile_base; });
  const SessionDev& S = batch_session<false>(B, s);
  const int lt = tile - S.tile_base;
  // samples 4 lane to 4 lane + 3, a quarter of a row
  const int by = ((lt / S.tiles_x) * 16 + (lane >> 2)) << S.sub_sy;
  uint32_t k[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int bx = ((lt % S.tiles_x) * 16 + (lane & 3) * 4 + i) << S.sub_sx;
    uint32_t work = 0;
    if (S.lane_work && bx < S.width && by < S.height) work = S.lane_work[by * S.width + bx];
    k[i] = (work << 8) | (uint32_t)(4 * lane + i);
  }
  const int pos = sort_position(lane);
  invert_if(k, pos);
  cas(k[0], k[1]); cas(k[2], k[3]);
  cas(k[0], k[2]); cas(k[1], k[3]);
  cas(k[1], k[2]);
  invert_if(k, pos ^ (pos >> 1));
  merge_level<0>(k, pos);
  invert_if(k, (pos >> 1) ^ (pos >> 2));
  merge_level<1>(k, pos);
  invert_if(k, (pos >> 2) ^ (pos >> 3));
  merge_level<2>(k, pos);
  invert_if(k, (pos >> 3) ^ (pos >> 4));
  merge_level<3>(k, pos);
  invert_if(k, (pos >> 4) ^ (pos >> 5));
  merge_level<4>(k, pos);
  invert_if(k, pos >> 5);
  merge_level<5>(k, pos);
  reinterpret_cast<uint32_t*>(W.lane_perm + (int64_t)tile * kBlock)[pos] =
      (k[0] & 0xffu) | ((k[1] & 0xffu) << 8) | ((k[2] & 0xffu) << 16) | ((k[3] & 0xffu) << 24);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// LDS traffic between the lanes of one wave: a wave's LDS operations execute
// in order, so only the compiler has to be held.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kFwdStage = 16;             // entries walked at a time (16, 32, 8: 87, 90, 100 us)
constexpr int kFwdQueue = kFwdStage + 64; // < kFwdStage left over + 64 new ones
// Words of an entry's table for COLS columns and rows of samples: dx of the
// columns, the two terms of the rows, (A, opacity).  Even; spreads the banks.
constexpr int tab_words(int cols) { return 3 * cols + 2; }

// One wave per workgroup, for one 8x8 quadrant of a tile (as the backward).
// It tests 64 list entries at a time, one a lane, against its quadrant (the
// mask is saved for the backward), queues the ones that reach it in LDS, and
// lets its pixels walk the queue kFwdStage entries at a time.
//
// Bound by VALU issue: instructions per walked entry are what counts.
//  * The offsets of the 8 columns and, of the 8 rows, the two terms of the
//    exponent that depend on the row alone are formed once per entry, by four
//    lanes an entry, so that a pixel's exponent is two FMAs on three LDS
//    values instead of nine operations; the values are frag_alpha's, bit for
//    bit.  One sample a block of 2x2 pixels takes 16 columns and rows; other
//    samples off the pixel grid (larger blocks, BAL) use frag_alpha itself.
//  * C += w (r, g, b, z) is one 4x4x1 MFMA: block i of four lanes multiplies
//    the entry's four values (row j: value j) with its lanes' four weights,
//    an exact FMA per element; the A operand of four entries is one LDS read,
//    lane l holding value l & 3 of entry (l >> 2) & 3, broadcast by blocks.
//  * A stopped pixel's T is negative, so `T' < 1e-4` also keeps it stopped.
// Measured (kernel trace) at 1200x680 / 300k: 92 -> 84 us (51.8M -> 35.0M wave
// VALU instructions; 70 us of issue, exp at quarter rate included, the rest the
// last waves draining); 640x480 / 100k 55 -> 47 us, 320x240 / 20k 21.6 -> 17 us;
// 1200x680 at 1 in 4 / 500k 109 -> 71 us by the tables of 16 columns.
// Before, four waves of a tile shared batches of 256 entries, 29 VALU
// instructions a walked entry.
//
// STATS: also count, per pixel, the fragments blended and the list entries
// visited (the work counts of a frame); off in ordinary renders.
// FRAG: also save the fragments' alpha (see frag_base).
// BAL: lanes assigned by previous work (k_lane_schedule); also writes each
// sample's walked entries to S.lane_work_out for the next forward.
template <bool STATS, bool FRAG, bool BAL, bool ONE, bool IRR>
__global__ __launch_bounds__(64) void k_raster_fwd(Batch B, WsPtrs W) {
  constexpr int kMaxCols = IRR && !BAL ? 16 : 8;
  __shared__ __align__(16) float s_tab[kFwdStage * tab_words(kMaxCols)];
  __shared__ float4 s_r0[kFwdQueue], s_k4[kFwdQueue], s_col[kFwdQueue];
  __shared__ int s_pos[kFwdQueue];
  int tile, wave;
  if (!wave_of_block(B.t_total, tile, wave)) return;
  const int lane = threadIdx.x;
  const int sidx = BAL ? (int)W.lane_perm[(int64_t)tile * kBlock + wave * 64 + lane]
                       : quadrant_sample(wave, lane);
  const TileCtx c = tile_ctx<ONE>(B, tile, sidx);
  const SessionDev& S = batch_session<ONE>(B, c.s);
  const bool active = c.has && (S.pmask == nullptr || S.pmask[c.pix] != 0);
  const float pxf = (float)c.px + 0.5f, pyf = (float)c.py + 0.5f;
  // the box of samples the wave culls against
  int x0 = (wave & 1) * 8, y0 = (wave >> 1) * 8, x1 = x0 + 7, y1 = y0 + 7;
  if (BAL) {
    x0 = x1 = sidx & 15;
    y0 = y1 = sidx >> 4;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      x0 = min(x0, __shfl_xor(x0, off));
      x1 = max(x1, __shfl_xor(x1, off));
      y0 = min(y0, __shfl_xor(y0, off));
      y1 = max(y1, __shfl_xor(y1, off));
    }
  }
  // the quadrant's first pixel, and the lane's sample from there
  const int ox = c.tile_x0 + (x0 << S.sub_sx), oy = c.tile_y0 + (y0 << S.sub_sy);
  const float qx = (float)ox + 0.5f, qy = (float)oy + 0.5f;
  // list positions fit in int32: the pair capacity is below 2^31
  const int start = (int)min((int64_t)W.tile_start[tile], W.cap);
  const int end = (int)min((int64_t)W.tile_start[tile + 1], W.cap);
  // T carries the pixel's stop in its sign: T > 0 while the pixel walks
  // (T >= 1e-4 > 0 until the stop), -T once it has stopped (or never walks)
  float T = active ? 1.f : -1.f;
  f32x4 C = {0.f, 0.f, 0.f, 0.f};           // colour, depth
  int last = -1;
  int stop = end;               // list position where the pixel stopped
  int nblend = 0;
  uint32_t fcur = 0;            // saved fragments of this wave so far
  float2* fout = FRAG ? W.fdata + frag_base(start, end, wave) : nullptr;
  unsigned long long fmask = 0; // lanes 0 to 3: who blended that entry of a group of four
  const float* const col_words = reinterpret_cast<const float*>(s_col) + (lane & 15);
  int walked = 0, done = 0;     // entries walked up to the lane's last blended one; in all
  // COLS: the columns and rows that the samples lie in (0: any number)
  auto walk = [&](auto cols) {
    constexpr int COLS = decltype(cols)::value, kTab = tab_words(COLS);
    const float* const t_x = s_tab + (COLS == 8 ? lane & 7 : c.px - ox);
    const float2* const t_y =
        reinterpret_cast<const float2*>(s_tab + COLS) + (COLS == 8 ? lane >> 3 : c.py - oy);
    int head = 0, queued = 0;     // head: a multiple of kFwdStage, so no batch wraps around
    // the record this lane tests next, and the Gaussian after it: a list's test
    // steps would otherwise wait for a dependent load each
    uint32_t nid = start + lane < end ? W.ids[start + lane] : 0u;
    GaussRec next;
    if (start + lane < end) next = W.rec[nid];
    nid = start + 64 + lane < end ? W.ids[start + 64 + lane] : 0u;
    for (int b0 = start; b0 < end; b0 += 64) {
      const GaussRec r = next;
      bool hit = b0 + lane < end;
      if (b0 + 64 + lane < end) next = W.rec[nid];
      if (b0 + 128 + lane < end) nid = W.ids[b0 + 128 + lane];
      if (hit) {
        hit = box_hit(r.pos, r.conic, r.ext.z, c.tile_x0, c.tile_y0, S.sub_sx, S.sub_sy, x0, y0, x1,
                      y1);
      }
      const unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
      if (lane == 0) W.hits[hits_at(start, tile, b0, wave)] = m;
      if (hit) {
        int at = head + queued + (int)lane_rank(m);
        at -= at >= kFwdQueue ? kFwdQueue : 0;
        s_r0[at] = r.pos;
        s_k4[at] = conic_log2(r.conic);
        s_col[at] = r.col;
        s_pos[at] = b0 + lane;
      }
      queued += __popcll(m);
      while (queued >= kFwdStage || (b0 + 64 >= end && queued > 0)) {
        const int n = min(kFwdStage, queued);
        // entries of opacity 0 fill the last group of four up
        if (lane < (-n & 3)) {
          const int at = head + n + lane;
          s_r0[at] = s_k4[at] = s_col[at] = make_float4(0.f, 0.f, 0.f, 0.f);
          s_pos[at] = 0;
        }
        wave_lds_order();
        if (COLS > 0) {
          // kParts lanes an entry, each its share of the columns and rows
          constexpr int kParts = 64 / kFwdStage, kShare = COLS / kParts;
          const int e = lane % kFwdStage, h = (lane / kFwdStage) * kShare;
          const float4 r0 = s_r0[head + e], k4 = s_k4[head + e];
          float* t = s_tab + e * kTab;
          if (e < ((n + 3) & ~3)) {
#pragma unroll
            for (int i = 0; i < kShare; i += 2) {
              const float d0 = (r0.x - (qx + (float)(h + i))) + r0.z;
              const float d1 = (r0.x - (qx + (float)(h + i + 1))) + r0.z;
              *reinterpret_cast<float2*>(t + h + i) = make_float2(d0, d1);
            }
#pragma unroll
            for (int i = 0; i < kShare; ++i) {
              const float dy = (r0.y - (qy + (float)(h + i))) + r0.w;
              *reinterpret_cast<float2*>(t + COLS + 2 * (h + i)) =
                  make_float2(k4.y * dy, (k4.z * dy) * dy);
            }
            if (h == 0) *reinterpret_cast<float2*>(t + 3 * COLS) = make_float2(k4.x, k4.w);
          }
          wave_lds_order();
        }
        int lastk = -1;               // the lane's last blended entry of these
        int stopk = -1;               // and the one it stopped at
        // every lane evaluates each entry; the decisions are selects, not
        // branches: skip (alpha < 1/255), stop (T would fall below 1e-4; the
        // fragment is excluded) or blend
        auto weight = [&](int k) -> float {
          Frag f;
          float raw;
          if (COLS > 0) {
            const float dx = t_x[k * kTab];
            const float2 y = t_y[k * (kTab / 2)];
            const float2 ao = *reinterpret_cast<const float2*>(s_tab + k * kTab + 3 * COLS);
            const float p2 = __builtin_fmaf(dx, __builtin_fmaf(ao.x, dx, y.x), y.y);
            f.e = __builtin_amdgcn_exp2f(p2);
            raw = ao.y * f.e;
            f.alpha = fminf(kAlphaMax, raw);
            f.om = fmaxf(1.f - kAlphaMax, __builtin_fmaf(-ao.y, f.e, 1.f));
          } else {
            const float4 kk = s_k4[head + k];
            f = frag_alpha(s_r0[head + k], kk, pxf, pyf);
            raw = kk.w * f.e;
          }
          const float tn = T * f.om;
          const bool seen = !(f.alpha < kAlphaMin);
          const bool blend = seen && !(tn < kTMin);
          if (STATS || BAL) stopk = T > 0.f && seen && !blend ? k : stopk;
          const float w = blend ? f.alpha * T : 0.f;       // adds exactly 0 otherwise
          T = blend ? tn : (seen ? -fabsf(T) : T);
          lastk = blend ? k : lastk;
          if (STATS) nblend += blend ? 1 : 0;
          if (FRAG) {                   // (entries past the last: no lane)
            const unsigned long long bm = __builtin_amdgcn_ballot_w64(blend);
            if (lane == (k & 3)) fmask = bm;
            if (blend)
              fout[lane_rank(bm)] = make_float2(raw > kAlphaMax ? -f.alpha : f.alpha, f.om);
            fout += __popcll(bm);
            fcur += (uint32_t)__popcll(bm);
          }
          return w;
        };
        // all unrolled, so that every position is an immediate and the LDS reads of the
        // next entries go ahead (by a factor of four: 88 us instead of 83)
#pragma unroll
        for (int k = 0; k < kFwdStage; k += 4) {
          if (k >= n || __builtin_amdgcn_ballot_w64(T > 0.f) == 0) break;     // or the whole wave has stopped
          const float a = col_words[4 * (head + k)];
          C = __builtin_amdgcn_mfma_f32_4x4x1f32(a, weight(k), C, 2, 0, 0);
          C = __builtin_amdgcn_mfma_f32_4x4x1f32(a, weight(k + 1), C, 2, 1, 0);
          C = __builtin_amdgcn_mfma_f32_4x4x1f32(a, weight(k + 2), C, 2, 2, 0);
          C = __builtin_amdgcn_mfma_f32_4x4x1f32(a, weight(k + 3), C, 2, 3, 0);
          // the group's masks, a lane an entry
          if (FRAG && lane < 4 && k + lane < n)
            W.fmask[(int64_t)s_pos[head + k + lane] * 4 + wave] = fmask;
        }
        if (lastk >= 0) {
          last = s_pos[head + lastk];
          walked = done + lastk + 1;
        }
        if ((STATS || BAL) && stopk >= 0) stop = s_pos[head + stopk];
        done += n;
        wave_lds_order();
        queued -= n;
        head = head == kFwdQueue - kFwdStage ? 0 : head + kFwdStage;
      }
      if (__builtin_amdgcn_ballot_w64(T > 0.f) == 0) break;
    }
  };
  if (!IRR || (!BAL && (S.sub_sx | S.sub_sy) == 0))
    walk(std::integral_constant<int, 8>{});
  else if (!BAL && S.sub_sx <= 1 && S.sub_sy <= 1)
    walk(std::integral_constant<int, 16>{});
  else
    walk(std::integral_constant<int, 0>{});
  if (FRAG && lane == 0) W.fcount[(int64_t)tile * 4 + wave] = fcur;
  if (W.order) {                // (not when the backward recomputes the state)
    int w = walked;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) w = max(w, __shfl_xor(w, off));
    if (lane == 0) file_work(W, B.t_total, tile, wave, w);
  }
  T = fabsf(T);
  if (!c.inside) return;
  if (BAL && S.lane_work_out) {
    const int visited = active ? min(stop + 1, end) - start : 0;
    S.lane_work_out[c.by0 * S.width + c.bx0] = (uint16_t)min(visited, 65535);
  }
  const int64_t hw = (int64_t)S.width * S.height;
  // loss gradient (Eq. 6, L1 colour and depth, means over the active pixels):
  // the arithmetic of the separate loss pass on the values written here
  float l1_sc = 0.f, l1_sd = 0.f;
  if (S.l1_dcolor) {
    const float n = S.l1_n_active ? fmaxf((float)*S.l1_n_active, 1.f) : (float)hw;
    l1_sc = S.l1_w_color / (3.f * n);
    l1_sd = S.l1_w_depth / n;
  }
  // every pixel of the lane's block: the sample gets its result, the others
  // (masked out) render as background
  const int ex = min(S.width, c.bx0 + (1 << S.sub_sx));
  const int ey = min(S.height, c.by0 + (1 << S.sub_sy));
  for (int y = c.by0; y < ey; ++y)
    for (int x = c.bx0; x < ex; ++x) {
      const int p = y * S.width + x;
      const bool me = p == c.pix;
      if (S.color) {
        S.color[p] = me ? C[0] : 0.f;
        S.color[hw + p] = me ? C[1] : 0.f;
        S.color[2 * hw + p] = me ? C[2] : 0.f;
      }
      if (S.l1_dcolor) {
        const float m = S.pmask ? (S.pmask[p] ? 1.f : 0.f) : 1.f;
        const float v[4] = {me ? C[0] : 0.f, me ? C[1] : 0.f, me ? C[2] : 0.f, me ? C[3] : 0.f};
#pragma unroll
        for (int k = 0; k < 3; ++k)
          S.l1_dcolor[k * hw + p] = m * l1_sc * sign_of(v[k] - S.l1_tcolor[k * hw + p]);
        S.l1_ddepth[p] = m * l1_sd * sign_of(v[3] - S.l1_tdepth[p]);
      }
      if (S.depth) S.depth[p] = me ? C[3] : 0.f;
      if (S.alpha) S.alpha[p] = me ? 1.f - T : 0.f;
      if (S.final_T) S.final_T[p] = me ? T : 1.f;
      if (S.last_idx) S.last_idx[p] = me ? last : -1;
      if (STATS && S.stats) {
        // work counts: fragments blended, list entries up to the stop (or
        // the end of the list), list entries up to the last blended one
        S.stats[p] = me ? nblend : 0;
        S.stats[hw + p] = me && active ? min(stop + 1, end) - start : 0;
        S.stats[2 * hw + p] = me && last >= 0 ? last - start + 1 : 0;
      }
    }
}

// Entries per group of the backward's two passes, and the LDS layout of a
// group: -dL/dpower of entry k at the wave's 64 pixels in row k, the blend
// weights in row kGrp + k.  Rows are 17 units of 16 bytes long, and pass 2's
// lanes are dealt to (entry, row of pixels) and (entry, 4 pixels) so that a
// quarter wave's reads touch every bank once (see prow and pblock there).
constexpr int kGrp = 8;
constexpr int kRowWords = 68;
constexpr int kBwdQueue = 2 * kGrp + 64; // < 2 kGrp left over + 64 new ones
// Words of an entry's table: as the forward's, then list position and pair.
constexpr int bwd_tab_words(int cols) { return 3 * cols + 4; }

// NV = 10 (all parameters) or 6 (pose only) sums per list entry.  GA: some
// session has an alpha-image gradient (without one, its term of dL/dalpha is
// left out rather than added as zero).
//
// One wave per workgroup, for one 8x8 quadrant of a tile: nothing is shared
// between the quadrants, so no wave waits at a barrier for a busier one and a
// finished wave's place is refilled at once.  Each (tile, Gaussian, quadrant)
// that some pixel blended gets the sums of its pixels in a slot of its own and
// a flag byte; everything else is neither written nor read.
//
// Bound by VALU issue, so the design minimises instructions per (list entry,
// wave).  The entries that reach the quadrant go through a queue, in falling
// list order, and are worked on in groups of kGrp without branches, so that the
// latencies of one entry hide behind the others; half a wave fetches the next
// group's records meanwhile (64 bytes, a lane a quarter).  Two passes a group:
//  1. lane = pixel: alpha again (with the forward's tables of offsets and row
//     terms), T and the suffix recovered, giving two values per (entry, pixel),
//     n = -dL/dpower and the blend weight w, stored to LDS.  The products of an
//     entry's (r, g, b, z) with the pixels' upstream gradients are 4x4x1 MFMAs,
//     four entries at a time;
//  2. lane = (entry, row of 8 pixels): the sums of n over the row's pixels, the
//     offsets to the Gaussian's centre from the tables; one reduce-scatter over
//     the 8 rows for all 8 entries.  The sums of w times the upstream gradients
//     are 4x4x1 MFMAs again (entry by value, over the pixels) and a sum over the
//     16 groups of pixels; pose only, the one value goes with the sums of n.
// The sums, d = centre - pixel: n dx, n dy, n dx^2, n dx dy, n dy^2, n (NV = 10
// only), w g_r, w g_g, w g_b (NV = 10 only), w g_z; the conic and the opacity
// are applied once per Gaussian by the preprocessing backward:
//   d power / d(u, v) = -(a dx + b dy, b dx + c dy), d power / d(a, b, c) =
//   -(dx^2 / 2, dx dy, dy^2 / 2), dL/do = sum alpha dL/dalpha / o.
// All sums are formed in a fixed order: bitwise reproducible, no float atomics.
// (Moments of n about the quadrant's middle, one 16x16x4 MFMA chain a group and
// shifted to the centre in double, cost digits: narrow Gaussians cancel.)
//
// Measured (kernel trace) at 1200x680 / 300k, NV = 10: 241 -> 133 us (109M -> 63M
// wave VALU instructions, 123 us of issue; the rest the last waves draining); pose
// only at 640x480 / 100k 109 -> 59 to 63 us, 1200x680 at 1 in 4 / 500k 135 -> 123 us.
// Before, four waves of a tile met at two barriers per 64 entries, summed ten
// values over the wave per entry (lane swaps and DPP, 29 instructions), and
// every pair without a gradient was written as zeros.  One wave a quadrant with
// pass 2 on the VALU and entries one by one: 147, 72 and 138 us; the same with
// the MFMAs but a branch an entry: 179 us.
//
// FRAG: the forward saved its fragments (frag_base): each entry's blending
// lanes and their (alpha, 1 - alpha) are read instead of re-evaluating alpha,
// and entries no lane of the wave blended are skipped without arithmetic; the
// values are those the forward computed, so the gradients are bitwise those
// of the re-evaluating form.
// BAL: the forward assigned lanes by previous work (k_lane_schedule); the same
// samples go to the same lanes here (the saved quadrant bits are per wave).
// IRR: some tile's samples may not form the 8x8 pixel grid of its quadrants
// (downsampled frames, BAL).  A uniform branch outside the loops takes the grid's
// code, that of tables of 16 columns and rows (blocks of up to 2x2 pixels) or
// frag_alpha; off the grid pass 2 takes each sample's own centre.
// EU: waves a SIMD the registers are kept to (raster_bwd_variant).
template <int NV, bool GA, bool FRAG, bool BAL, bool ONE, bool IRR, int EU>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(EU)))
void k_raster_bwd(Batch B, WsPtrs W) {
  __shared__ uint2 s_queue[kBwdQueue];                      // (Gaussian, list position)
  __shared__ float4 s_rec[4 * kGrp];                        // the group's records
  __shared__ unsigned long long s_fm[FRAG ? kBwdQueue : 1];
  __shared__ __align__(16) float s_rows[2 * kGrp * kRowWords];   // see kGrp
  constexpr int kMaxCols = IRR && !BAL ? 16 : 8;
  __shared__ __align__(16) float s_tab[kGrp * bwd_tab_words(kMaxCols)];
  __shared__ float2 s_xy[IRR ? 64 : 1];                     // sample centres
  int tile, wave;
  if (W.sum_lo > 0 && (int64_t)W.sum_lo >= W.counters[0]) return;   // a pass past the last pair
  if (!wave_by_work(W, B.t_total, tile, wave)) return;
  const int lane = threadIdx.x;
  const int sidx = BAL ? (int)W.lane_perm[(int64_t)tile * kBlock + wave * 64 + lane]
                       : quadrant_sample(wave, lane);
  const TileCtx c = tile_ctx<ONE>(B, tile, sidx);
  const SessionDev& S = batch_session<ONE>(B, c.s);
  const int ltx = c.lt % S.tiles_x, lty = c.lt / S.tiles_x;
  const bool active = c.has && (S.pmask == nullptr || S.pmask[c.pix] != 0);
  const int64_t hw = (int64_t)S.width * S.height;
  const int start = (int)min((int64_t)W.tile_start[tile], W.cap);
  const int end = (int)min((int64_t)W.tile_start[tile + 1], W.cap);
  int last = -1;
  float Tc = 1.f, g0 = 0.f, g1 = 0.f, g2 = 0.f, gD = 0.f, gA = 0.f;
  if (active) {
    last = S.last_idx[c.pix];
    Tc = S.final_T[c.pix];
    g0 = S.dl_color[c.pix];
    g1 = S.dl_color[hw + c.pix];
    g2 = S.dl_color[2 * hw + c.pix];
    gD = S.dl_depth[c.pix];
    if (GA && S.dl_alpha) gA = S.dl_alpha[c.pix];
  }
  const float gAT = gA * Tc;        // dA/dalpha_j = T_final / (1 - alpha_j)
  // the wave's last blended position; one outside this tile's list (state of
  // another forward) is never followed past the list
  int hi = last;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) hi = max(hi, __shfl_xor(hi, off));
  hi = __builtin_amdgcn_readfirstlane(min(hi, end - 1));
  if (hi < start) return;
  const float pxf = (float)c.px + 0.5f, pyf = (float)c.py + 0.5f;
  // saved fragments: the wave's stream and cursor
  uint32_t fcur = 0;
  int64_t fbase = 0;
  if (FRAG) {
    fcur = W.fcount[(int64_t)tile * 4 + wave];
    fbase = frag_base(start, end, wave);
  }
  // pass 2: this lane's entry of a group and its row of samples; the upstream
  // gradients it takes: of z along the row (pose only), or r, g, b, z (lane & 3)
  // at four pixels
  const int ge = lane & 7, prow = (lane >> 4) | ((lane >> 1) & 4);
  const int pblock = 4 * (((lane >> 2) & 3) * 4 + (lane >> 4));
  float G[NV == 10 ? 4 : 8];
  {
    s_rows[lane] = NV == 10 ? g0 : gD;
    if (NV == 10) {
      s_rows[64 + lane] = g1;
      s_rows[128 + lane] = g2;
      s_rows[192 + lane] = gD;
    }
    if (IRR) s_xy[lane] = make_float2(pxf, pyf);
    wave_lds_order();
#pragma unroll
    for (int u = 0; u < (NV == 10 ? 1 : 2); ++u) {
      const float4 q = *reinterpret_cast<const float4*>(
          s_rows + (NV == 10 ? 64 * (lane & 3) + pblock : 8 * prow + 4 * u));
      G[4 * u] = q.x; G[4 * u + 1] = q.y; G[4 * u + 2] = q.z; G[4 * u + 3] = q.w;
    }
    wave_lds_order();
  }
  // the quadrant's first pixel
  const int ox = c.tile_x0 + (((wave & 1) * 8) << S.sub_sx);
  const int oy = c.tile_y0 + (((wave >> 1) * 8) << S.sub_sy);
  const float qx = (float)ox + 0.5f, qy = (float)oy + 0.5f;
  // what the lane stores of a group's sums, and where in a pair's slots: lane
  // (h, p, bit 3, entry) sum 3 h + p, with bit 3 sum 3 h + 2 (p = 0) or the flag
  // (p = 1); lane (h, p, bit 3, bit 2, value) the w sum of entry 4 h + 2 bit 3 + p
  const uint32_t room = W.sum_n;                 // pairs whose sums are kept, below 2^31
  uint8_t* const live = W.live + (int64_t)W.sum_lo * 4 + wave;
  const int lh = lane >> 5, lp = (lane >> 4) & 1, sum = rows8_value(lane);
  const int we = 4 * lh + (lane & 8 ? 2 : 0) + lp;
  const bool sum_lane = sum >= 0;
  const bool flag_lane = (lane & 8) && lp && lh == 0;
  const bool w_lane = NV == 10 && !(lane & 4);
  float* const sum_dst = W.partial + wave * NV + sum;
  float* const w_dst = W.partial + wave * NV + 6 + (lane & 3);
  float* const wr = s_rows + lane;
  const float* const rn = s_rows + ge * kRowWords + 8 * prow;
  const float* const rw = NV == 10 ? s_rows + (kGrp + (lane & 3)) * kRowWords + pblock
                                   : rn + kGrp * kRowWords;
  // S_j . g: the colour and depth of the fragments behind j, normalised by
  // the transmittance T_{j+1} they start from, dotted with the upstream gradient
  float SG = 0.f;
  // COLS: the columns and rows that the samples lie in (0: any number); 8: they
  // are the 8x8 pixel grid
  auto walk = [&](auto cols) {
    constexpr int COLS = decltype(cols)::value, kTab = bwd_tab_words(COLS);
    constexpr bool G8 = COLS == 8;
    const float* const t_x = s_tab + (G8 ? lane & 7 : c.px - ox);
    const float2* const t_y =
        reinterpret_cast<const float2*>(s_tab + COLS) + (G8 ? lane >> 3 : c.py - oy);
    int head = 0, queued = 0;     // head: a multiple of kGrp, so no group wraps around
    // the entries the quadrant can reach, of the 64 queued next (saved by the
    // forward up to the wave's last blended one at least), and this lane's
    int b0 = start + ((hi - start) & ~63);
    unsigned long long nh = W.hits[hits_at(start, tile, b0, wave)];
    uint32_t nid = b0 + lane <= hi ? W.ids[b0 + lane] : 0u;
    // lane (entry l >> 2, quarter l & 3) of half a wave fetches the next group's
    // records while the group before is worked on; quarter 3 becomes the pair's slot
    float4 rec = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t goff = 0;
    int pos_next = 0;
    auto fetch = [&](int at, int n) {
      at = at >= kBwdQueue ? at - kBwdQueue : at;
      if (lane < 4 * kGrp) {
        if (n < kGrp) {           // entries past the last: opacity 0
          rec = make_float4(0.f, 0.f, 0.f, 0.f);
          pos_next = 0;
        }
        if ((lane >> 2) < n) {
          const uint2 q = s_queue[at + (lane >> 2)];
          rec = reinterpret_cast<const float4*>(W.rec + q.x)[lane & 3];
          if ((lane & 3) == 3) goff = W.goff[q.x];
          pos_next = (int)q.y;
        }
      }
    };
    bool first = true;
    for (;;) {
      // two groups ahead, so that the next one's records can be fetched
      while (queued < 2 * kGrp && b0 >= start) {
        bool hit = b0 + lane <= hi && ((nh >> lane) & 1ull) != 0;
        unsigned long long fm = 0;
        if (FRAG && hit) {
          fm = W.fmask[(int64_t)(b0 + lane) * 4 + wave];
          hit = fm != 0;              // no lane of the wave blended it
        }
        const unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
        const int found = __popcll(m);
        if (hit) {                    // in falling list order
          int at = head + queued + found - 1 - (int)lane_rank(m);
          at -= at >= kBwdQueue ? kBwdQueue : 0;
          s_queue[at] = make_uint2(nid, (uint32_t)(b0 + lane));
          if (FRAG) s_fm[at] = fm;
        }
        queued += found;
        b0 -= 64;
        if (b0 >= start) {
          nh = W.hits[hits_at(start, tile, b0, wave)];
          nid = W.ids[b0 + lane];
        }
      }
      if (queued == 0) break;
      const int n = min(kGrp, queued);
      wave_lds_order();
      if (first) fetch(head, n);
      first = false;
      if (lane < 4 * kGrp) {
        const int part = lane & 3;
        s_rec[lane] = COLS == 0 && part == 1 ? conic_log2(rec) : rec;
        // the pair's slot: Gaussian-major, then row-major in its tile rectangle,
        // from the first pair whose sums are kept (those before it come out above 2^31)
        if (part == 3)
          *reinterpret_cast<int2*>(s_tab + (lane >> 2) * kTab + 3 * COLS + 2) =
              make_int2(pos_next, (int)(goff - W.sum_lo - (__float_as_uint(rec.x) >> 16)) +
                                      lty * (int)(__float_as_uint(rec.x) & 0xffffu) + ltx);
      }
      if (queued > n) fetch(head + kGrp, min(kGrp, queued - n));
      wave_lds_order();
      const float4 re = s_rec[4 * ge];         // this lane's entry in the table and in pass 2
      if (COLS > 0) {
        // an entry's columns and rows prow, prow + 8 (see k_raster_fwd)
        float* t = s_tab + ge * kTab;
        const float4 k4 = conic_log2(s_rec[4 * ge + 1]);
#pragma unroll
        for (int i = 0; i < COLS; i += 8) {
          t[prow + i] = (re.x - (qx + (float)(prow + i))) + re.z;
          const float dy = (re.y - (qy + (float)(prow + i))) + re.w;
          *reinterpret_cast<float2*>(t + COLS + 2 * (prow + i)) =
              make_float2(k4.y * dy, (k4.z * dy) * dy);
        }
        if (prow == 0) *reinterpret_cast<float2*>(t + 3 * COLS) = make_float2(k4.x, k4.w);
        wave_lds_order();
      }
      // ---- pass 1
      unsigned some = 0;            // the entries some pixel blended
#pragma unroll
      for (int j = 0; j < kGrp; j += 4) {
        // (colour, depth) of four entries dotted with the upstream gradient
        f32x4 cg4 = {0.f, 0.f, 0.f, 0.f};
        const float4 col = s_rec[4 * (j + (lane & 3)) + 2];
        cg4 = __builtin_amdgcn_mfma_f32_4x4x1f32(col.x, g0, cg4, 0, 0, 0);
        cg4 = __builtin_amdgcn_mfma_f32_4x4x1f32(col.y, g1, cg4, 0, 0, 0);
        cg4 = __builtin_amdgcn_mfma_f32_4x4x1f32(col.z, g2, cg4, 0, 0, 0);
        cg4 = __builtin_amdgcn_mfma_f32_4x4x1f32(col.w, gD, cg4, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = j + i;
          Frag f;
          bool contrib, clamped;
          if (FRAG) {
            const unsigned long long bm = k < n ? s_fm[head + k] : 0ull;
            fcur -= (uint32_t)__popcll(bm);
            contrib = ((bm >> lane) & 1ull) != 0;
            float2 rec = make_float2(0.f, 1.f);
            if (contrib) rec = W.fdata[fbase + fcur + lane_rank(bm)];
            f.alpha = fabsf(rec.x);
            f.om = rec.y;
            clamped = rec.x < 0.f;
          } else {
            float raw;
            int pos;
            if (COLS > 0) {
              const float dx = t_x[k * kTab];
              const float2 y = t_y[k * (kTab / 2)];
              const float4 ao = *reinterpret_cast<const float4*>(s_tab + k * kTab + 3 * COLS);
              const float p2 = __builtin_fmaf(dx, __builtin_fmaf(ao.x, dx, y.x), y.y);
              f.e = __builtin_amdgcn_exp2f(p2);
              raw = ao.y * f.e;
              pos = __float_as_int(ao.z);
              f.alpha = fminf(kAlphaMax, raw);
              f.om = fmaxf(1.f - kAlphaMax, __builtin_fmaf(-ao.y, f.e, 1.f));
            } else {
              const float4 k4 = s_rec[4 * k + 1];
              f = frag_alpha(s_rec[4 * k], k4, pxf, pyf);
              raw = k4.w * f.e;
              pos = __float_as_int(s_tab[k * kTab + 3 * COLS + 2]);
            }
            // entries at or before `last` lie before the pixel's stop
            contrib = pos <= last && !(f.alpha < kAlphaMin);
            clamped = raw > kAlphaMax;
          }
          some |= __builtin_amdgcn_ballot_w64(contrib) != 0 ? 1u << k : 0u;
          // lanes that did not blend it take alpha = 0 and 1 - alpha = 1, so
          // every update below leaves their state unchanged and their
          // gradients exactly zero (selects, not branches)
          const float al = contrib ? f.alpha : 0.f;
          const float om = contrib ? f.om : 1.f;
          const float rom = __builtin_amdgcn_rcpf(om);
          const float Tj = Tc * rom;                     // T before this fragment (rcp(1) = 1)
          const float w = al * Tj;
          // (0 where the lane did not blend it: a colour or depth that is not finite
          // reaches the pixels that blended it alone; saved fragments queue no
          // entry that no lane blended)
          const float cg = FRAG || contrib ? cg4[i] : 0.f;
          // dL/dalpha_j = T_j (c_j - S_j) . g + T_final gA / (1 - alpha_j)
          const float dla = GA ? __builtin_fmaf(Tj, cg - SG, gAT * rom) : Tj * (cg - SG);
          SG = __builtin_fmaf(al, cg, om * SG);
          Tc = Tj;
          // the clamp alpha = 0.99 has no gradient to o or to the power
          const bool live = contrib && !clamped;
          const float nk = live ? -(f.alpha * dla) : 0.f;   // -dL/dpower
          wr[k * kRowWords] = nk;
          wr[(kGrp + k) * kRowWords] = w;
        }
      }
      wave_lds_order();
      if (some) {
        // ---- pass 2
        // w g over four pixels, of entries 0 to 3 and 4 to 7: lane = (pixels, value);
        // pose only: over the row instead, in place of the sum of n
        f32x4 wa = {0.f, 0.f, 0.f, 0.f}, wb = {0.f, 0.f, 0.f, 0.f};
        if (NV == 10) {
          const float4 p = *reinterpret_cast<const float4*>(rw);
          const float4 q = *reinterpret_cast<const float4*>(rw + 4 * kRowWords);
          wa = __builtin_amdgcn_mfma_f32_4x4x1f32(p.x, G[0], wa, 0, 0, 0);
          wb = __builtin_amdgcn_mfma_f32_4x4x1f32(q.x, G[0], wb, 0, 0, 0);
          wa = __builtin_amdgcn_mfma_f32_4x4x1f32(p.y, G[1], wa, 0, 0, 0);
          wb = __builtin_amdgcn_mfma_f32_4x4x1f32(q.y, G[1], wb, 0, 0, 0);
          wa = __builtin_amdgcn_mfma_f32_4x4x1f32(p.z, G[2], wa, 0, 0, 0);
          wb = __builtin_amdgcn_mfma_f32_4x4x1f32(q.z, G[2], wb, 0, 0, 0);
          wa = __builtin_amdgcn_mfma_f32_4x4x1f32(p.w, G[3], wa, 0, 0, 0);
          wb = __builtin_amdgcn_mfma_f32_4x4x1f32(q.w, G[3], wb, 0, 0, 0);
        }
        // n times the offsets from the Gaussian's centre: lane = (entry, row)
        float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float nn[8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float4 q = *reinterpret_cast<const float4*>(rn + 4 * u);
          nn[4 * u] = q.x; nn[4 * u + 1] = q.y; nn[4 * u + 2] = q.z; nn[4 * u + 3] = q.w;
        }
        float a0 = 0.f, a1 = 0.f, a2 = 0.f;      // sums of n, n dx, n dx^2 along the row
        if (G8) {
          float dxs[8];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const float4 q = *reinterpret_cast<const float4*>(s_tab + ge * kTab + 4 * u);
            dxs[4 * u] = q.x; dxs[4 * u + 1] = q.y; dxs[4 * u + 2] = q.z; dxs[4 * u + 3] = q.w;
          }
          a0 = nn[0];
          a1 = nn[0] * dxs[0];
          a2 = a1 * dxs[0];
#pragma unroll
          for (int i = 1; i < 8; ++i) {
            const float nd = nn[i] * dxs[i];
            a0 += nn[i];
            a1 += nd;
            a2 = __builtin_fmaf(nd, dxs[i], a2);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float2 xy = s_xy[(8 * prow + i) % (IRR ? 64 : 1)];
            const float dx = (re.x - xy.x) + re.z, dy = (re.y - xy.y) + re.w;
            const float nx = nn[i] * dx, ny = nn[i] * dy;
            v[0] += nx;
            v[1] += ny;
            v[2] = __builtin_fmaf(nx, dx, v[2]);
            v[3] = __builtin_fmaf(nx, dy, v[3]);
            v[4] = __builtin_fmaf(ny, dy, v[4]);
            v[5] += nn[i];
          }
        }
        if (G8) {
          const float dy = (re.y - (qy + (float)prow)) + re.w;
          v[0] = a1;
          v[1] = dy * a0;
          v[2] = a2;
          v[3] = dy * a1;
          v[4] = dy * v[1];
          v[5] = a0;
        }
        if (NV == 6) {
          const float4 p = *reinterpret_cast<const float4*>(rw);
          const float4 q = *reinterpret_cast<const float4*>(rw + 4);
          const float ww[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
          v[5] = ww[0] * G[0];
#pragma unroll
          for (int i = 1; i < 8; ++i) v[5] = __builtin_fmaf(ww[i], G[i % (NV == 10 ? 4 : 8)], v[5]);
        }
        float x[2];
        rows8_reduce_scatter(v, x);
        // the w sums over the 16 groups of pixels (NV = 10): lane bits 5 to 2
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = swap32_add(wa[i], wb[i]);
        float y0 = swap16_add(r[0], r[1]), y1 = swap16_add(r[2], r[3]);
        y0 += dpp_f<kDppRowRor8, 0xf, true>(y0);
        y1 += dpp_f<kDppRowRor8, 0xf, true>(y1);
        y0 += dpp_f<kDppRowRor4, 0xf, true>(y0);
        y1 += dpp_f<kDppRowRor4, 0xf, true>(y1);
        const float y = lane & 8 ? y1 : y0;
        {
          // lane (h, p, bit 3, entry ge): sum 3 h + p; with bit 3: 3 h + 2, and the flag
          const uint32_t pair = __float_as_uint(s_tab[ge * kTab + 3 * COLS + 3]);
          const bool has = ((some >> ge) & 1u) && pair < room;
          const float z = lane & 8 ? x[1] : x[0];
          if (has && sum_lane) sum_dst[(int64_t)pair * (4 * NV)] = z;
          if (has && flag_lane) live[(int64_t)pair * 4] = 1;
        }
        if (NV == 10) {
          // lane (h, p, bit 3, bit 2, value) of the w sums
          const uint32_t pair = __float_as_uint(s_tab[we * kTab + 3 * COLS + 3]);
          if (((some >> we) & 1u) && pair < room && w_lane) w_dst[(int64_t)pair * (4 * NV)] = y;
        }
        wave_lds_order();
      }
      queued -= n;
      head = head == kBwdQueue - kGrp ? 0 : head + kGrp;
    }
  };
  if (!IRR || (!BAL && (S.sub_sx | S.sub_sy) == 0))
    walk(std::integral_constant<int, 8>{});
  else if (!BAL && S.sub_sx <= 1 && S.sub_sy <= 1)
    walk(std::integral_constant<int, 16>{});
  else
    walk(std::integral_constant<int, 0>{});
}

}  // namespace

template <bool STATS>
static void raster_fwd_variant(const Batch& b, const WsPtrs& w, bool frags, bool bal, int grid,
                               hipStream_t st) {
  const bool one = b.n_sessions == 1, irr = b.any_sub != 0;
  if (frags) {
    if (bal)
      k_raster_fwd<STATS, true, true, false, true><<<grid, 64, 0, st>>>(b, w);
    else if (irr)
      k_raster_fwd<STATS, true, false, false, true><<<grid, 64, 0, st>>>(b, w);
    else
      k_raster_fwd<STATS, true, false, false, false><<<grid, 64, 0, st>>>(b, w);
  } else if (bal) {
    k_raster_fwd<STATS, false, true, false, true><<<grid, 64, 0, st>>>(b, w);
  } else if (irr) {
    if (one)
      k_raster_fwd<STATS, false, false, true, true><<<grid, 64, 0, st>>>(b, w);
    else
      k_raster_fwd<STATS, false, false, false, true><<<grid, 64, 0, st>>>(b, w);
  } else {
    if (one)
      k_raster_fwd<STATS, false, false, true, false><<<grid, 64, 0, st>>>(b, w);
    else
      k_raster_fwd<STATS, false, false, false, false><<<grid, 64, 0, st>>>(b, w);
  }
}

// Waves of both rasterizers: four per tile, in bands of tiles per XCD.
static int raster_grid(const Batch& b) { return 32 * ((b.t_total + 7) / 8); }

// The backward's order by work is for grids whose waves are not all on the chip
// at once: up to four a SIMD (1024 tiles) they are, and neighbours then share
// the L2 better in tile order.  Measured, backward in tile order and by work:
// 836 tiles (1200x680 at 1 in 4, 500k) 136 and 141 us; 1200 tiles (640x480 /
// 100k) 84 and 71 us; 3225 tiles (1200x680 / 300k) 165 and 146 us.
constexpr int kFewTiles = 1024;

static WsPtrs raster_order(const Batch& b, const WsPtrs& w) {
  WsPtrs r = w;
  if (b.t_total <= kFewTiles) r.order = nullptr;
  return r;
}

hipError_t launch_raster_fwd(const Batch& b, const WsPtrs& w0, bool stats, bool frags, bool bal,
                             hipStream_t st, StageTimer* tm) {
  if (b.t_total <= 0) return hipSuccess;
  const int grid = raster_grid(b);
  const WsPtrs w = raster_order(b, w0);
  Scope sc(tm, kStRasterFwd, st);
  if (bal) k_lane_schedule<<<b.t_total, 64, 0, st>>>(b, w);
  if (stats)
    raster_fwd_variant<true>(b, w, frags, bal, grid, st);
  else
    raster_fwd_variant<false>(b, w, frags, bal, grid, st);
  return hipGetLastError();
}

// Waves a SIMD that the backward's registers are kept to: four where all waves
// are on the chip at once then (up to 1024 tiles; a fifth would not be used),
// otherwise five, or six for all gradients, at the price of a few spilled
// registers.  Measured with four and five: 836 tiles (1200x680 at 1 in 4, 500k)
// 120 and 128 us, 900 tiles of three frames (640x480 at 1 in 4, 100k) 125 and 128; six
// frames with downsampled ones among them (10.5k tiles) 297 and 284 us.  All
// gradients with four, five and six: 1200x680 / 300k 145, 138 and 133 us, / 500k 128
// and 123, three mapped frames 213 and 202 (the latter two five and six).  All
// gradients of downsampled frames need 124 registers and stay at four; the pose's on
// the pixel grid need 90 at most, five waves under any rule.
template <int NV, bool GA, bool IRR, int EU>
static void raster_bwd_waves(const Batch& b, const WsPtrs& w, int grid, hipStream_t st) {
  if (b.n_sessions == 1)
    k_raster_bwd<NV, GA, false, false, true, IRR, EU><<<grid, 64, 0, st>>>(b, w);
  else
    k_raster_bwd<NV, GA, false, false, false, IRR, EU><<<grid, 64, 0, st>>>(b, w);
}

template <int NV, bool GA>
static void raster_bwd_variant(const Batch& b, const WsPtrs& w, bool frags, bool bal, int grid,
                               hipStream_t st) {
  const bool irr = b.any_sub != 0, few = b.t_total <= kFewTiles;
  constexpr bool kMap = NV == 10;
  if (frags) {
    if (bal)
      k_raster_bwd<NV, GA, true, true, false, true, 4><<<grid, 64, 0, st>>>(b, w);
    else
      k_raster_bwd<NV, GA, true, false, false, true, 4><<<grid, 64, 0, st>>>(b, w);
  } else if (bal) {
    k_raster_bwd<NV, GA, false, true, false, true, 4><<<grid, 64, 0, st>>>(b, w);
  } else if (irr) {
    if (few)
      raster_bwd_waves<NV, GA, true, 4>(b, w, grid, st);
    else
      raster_bwd_waves<NV, GA, true, kMap ? 4 : 5>(b, w, grid, st);
  } else {
    if (few)
      raster_bwd_waves<NV, GA, false, kMap ? 4 : 5>(b, w, grid, st);
    else
      raster_bwd_waves<NV, GA, false, kMap ? 6 : 5>(b, w, grid, st);
  }
}

hipError_t launch_raster_bwd(const Batch& b, const WsPtrs& w0, int pose_only, bool alpha_grad,
                             bool frags, bool bal, hipStream_t st, StageTimer* tm) {
  if (b.t_total <= 0) return hipGetLastError();
  const WsPtrs w = raster_order(b, w0);
  // those in order of work, then those with little
  const int grid = raster_grid(b) * (w.order ? 2 : 1);
  Scope sc(tm, kStRasterBwd, st);
  if (pose_only) {
    if (alpha_grad)
      raster_bwd_variant<6, true>(b, w, frags, bal, grid, st);
    else
      raster_bwd_variant<6, false>(b, w, frags, bal, grid, st);
  } else {
    if (alpha_grad)
      raster_bwd_variant<10, true>(b, w, frags, bal, grid, st);
    else
      raster_bwd_variant<10, false>(b, w, frags, bal, grid, st);
  }
  return hipGetLastError();
}

}  // namespace rtgs
