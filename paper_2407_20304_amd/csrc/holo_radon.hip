// Joseph ray sums R_k (Eq. 14) and their transpose for gfx950 (MI355X).
//
//   block_volume  z-blocked copies of the volume (and of its x/y transpose)
//                 with zero-padded rows, read by the forward
//   radon_fwd     Joseph ray sums, angle groups sharing row windows staged in
//                 LDS by LDS-direct loads (16 lanes cover the 64 slices of
//                 one bin group, each thread owns 4 slices x 4 bins), fused
//                 exp(i kappa p) epilogue
//   split_sino    the sinogram as pairs of half-precision terms, in place
//   radon_adj     transpose as products on the matrix cores (a workgroup per
//                 16 x 16 voxel tile and 64 slices, all angles), sinogram
//                 segments staged in LDS per angle group by LDS-direct loads
//   radon_adj_few the same over up to four angles, without the split pass
// None is bound by HBM: every voxel is revisited once per angle.
#include <algorithm>
#include <type_traits>

#include "holo_internal.hpp"

namespace holo {

// Z-blocked copies of the volume for the ray sums: ub[z / ZT][y][P + x][z % ZT]
// (walks along y) and uTb[z / ZT][x][P + y][z % ZT] (walks along x, i.e. the
// x/y-transposed volume), rows padded by P = kFwdPad zero columns on each
// side.  A workgroup moves a 16 x 16 x ZT brick; the workgroups at the
// first and last brick column also clear the padding of their 16 rows.
__global__ __launch_bounds__(kThreads) void k_block_volume(const float2* __restrict__ u,
                                                           float2* __restrict__ ub,
                                                           float2* __restrict__ uTb,
                                                           unsigned* __restrict__ smax, int W) {
  constexpr int ZT = kVolZB, P = kFwdPad;
  // one 16 x 17 plane per slice, planes 274 elements apart: the write phase
  // reads down the slices (the 16 lanes of consecutive z at one position,
  // the next 16 at the neighbouring one), which a plane stride of 272 put
  // on two bank pairs; 274 = 18 (mod 32) spreads the 16 slices over the
  // even bank pairs and their neighbours over the odd ones
  constexpr int PL = 16 * 17 + 2;
  __shared__ float2 brick[ZT * PL];
  const int nt = W / 16, Wf = vol_row(W);
  const int x0 = (blockIdx.x % nt) * 16, y0 = (blockIdx.x / nt) * 16;
  const int zb = blockIdx.y;
  // the sinogram's slice maxima, which pass D raises, start at zero
  if (blockIdx.x == 0 && threadIdx.x < ZT) smax[zb * ZT + threadIdx.x] = 0u;
  const size_t WW = (size_t)W * W, WWf = (size_t)W * Wf;
  // read along x (contiguous)
  for (int i = threadIdx.x; i < ZT * 256; i += kThreads) {
    const int xx = i & 15, yy = (i >> 4) & 15, zz = i >> 8;
    brick[zz * PL + yy * 17 + xx] = u[(size_t)(zb * ZT + zz) * WW + (size_t)(y0 + yy) * W + x0 + xx];
  }
  __syncthreads();
  float2* bb = ub + (size_t)zb * WWf * ZT;
  float2* tb = uTb ? uTb + (size_t)zb * WWf * ZT : nullptr;
  // write with z fastest (contiguous 128-byte runs)
  for (int i = threadIdx.x; i < ZT * 256; i += kThreads) {
    const int zz = i % ZT, p = i / ZT;
    const int a = p & 15, b = p >> 4;
    bb[((size_t)(y0 + b) * Wf + P + x0 + a) * ZT + zz] = brick[zz * PL + b * 17 + a];
    if (tb) tb[((size_t)(x0 + b) * Wf + P + y0 + a) * ZT + zz] = brick[zz * PL + a * 17 + b];
  }
  // padding: rows y0..y0+15 of ub (brick column 0 / last) and rows
  // x0..x0+15 of uTb (brick row 0 / last)
  const float2 zero = make_float2(0.f, 0.f);
  const bool lo = x0 == 0, hi = x0 == W - 16;
  if (lo || hi) {
    for (int i = threadIdx.x; i < 16 * P * ZT; i += kThreads) {
      const int zz = i % ZT, c = (i / ZT) % P, r = i / (ZT * P);
      const int col = lo ? c : P + W + c;
      bb[((size_t)(y0 + r) * Wf + col) * ZT + zz] = zero;
    }
  }
  const bool tlo = y0 == 0, thi = y0 == W - 16;
  if (tb && (tlo || thi)) {
    for (int i = threadIdx.x; i < 16 * P * ZT; i += kThreads) {
      const int zz = i % ZT, c = (i / ZT) % P, r = i / (ZT * P);
      const int col = tlo ? c : P + W + c;
      tb[((size_t)(x0 + r) * Wf + col) * ZT + zz] = zero;
    }
  }
}

// ---------------------------------------------------------------------------
// Joseph ray sums and their transpose
// ---------------------------------------------------------------------------

// Forward.  A workgroup owns up to kFwdNA consecutive angles of one walk
// direction (one wave per angle), NB (16 by default, or 8: a tuning choice)
// consecutive bins and kFwdZT slices.
// Within a wave, 16 consecutive lanes cover the 64 slices of one group of NB/4
// consecutive bins: lane l takes the slice pairs (2 (l % 16), + 1) and
// (32 + 2 (l % 16), + 1), so one tap position and weight serve 4 slices and
// each tap of a pair is one 16-byte LDS read.  The workgroup walks the rows
// of the volume one at a time: each row's column window that all its rays
// cross (shared by the angles of the group) is copied straight from memory
// into LDS, [column][slice], by LDS-direct loads two rows ahead of use
// (three row buffers), so staging costs no registers and no LDS writes by
// the waves.  The 16 lanes of one LDS pass read the 256 contiguous bytes of
// one column: free of bank conflicts.  Angles that walk along x read the
// x/y-transposed volume, so both walk directions use the same code.  The
// host groups angles so that every window fits.
// HALF (NB = 8): half of a 16-bin block, with windows of its own.  Tap positions are taken from the lowest column of the whole
// block's window and its thread's first bin, so every tap and weight, and
// with them the fields, are the bits that a 16-bin workgroup gives.  The taps
// of a half span 8 columns less than a group may (its angles' bins all run the
// same way, at least a column each): kFwdSeg - 12, so 26 columns hold them and
// their margins.
constexpr int kHalfSeg = 26;
static_assert(kHalfSeg == kFwdSeg - 6 && kHalfSeg % 2 == 0, "window of a half");
template <int NB, bool HALF>
__global__ __launch_bounds__(kThreads, 2) void k_radon_fwd(const float2* __restrict__ u,
                                                         const float2* __restrict__ uT,  // z-blocked
                                                         float2* __restrict__ psi, DevGeom g,
                                                         const double* __restrict__ ang,
                                                         const int2* __restrict__ groups,
                                                         int g0, int ngroups, int c0, int c1) {
  constexpr int ZT = kFwdZT, SEG = HALF ? kHalfSeg : kFwdSeg, ZB = kVolZB;
  constexpr int BPT = NB / 4;                       // bins per thread
  constexpr int NBUF = 3;                           // row buffers (loads run 2 rows ahead)
  constexpr int ROWF2 = SEG * ZT;                   // float2 per staged row
  constexpr int C4 = ZT / 2;                        // float4 per staged column
  static_assert(ZT == 64 && (NB == 16 || NB == 8) && SEG <= 32 && kThreads == 256, "tiling");
  static_assert(!HALF || NB == 8, "half of a 16-bin block");
  __shared__ float4 tile4[NBUF * ROWF2 / 2];
  // rows' windows: 16 (xl + 64) + pairs of columns - 1.  HALF: xl of the whole
  // block, from bit 16 the half's first column from there (at most 12), or
  // kMoved and its own xl where it was moved
  constexpr int kMoved = 1 << 20;
  __shared__ typename std::conditional<HALF, unsigned, unsigned short>::type s_win[kMaxW];
  __shared__ int s_first, s_last;                   // rows whose window meets the volume
  const int W = g.W, H = g.H;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int pz = lane & 15, bg = lane >> 4;
  // logical order: angle group fastest, then bin block, then slice block,
  // so the groups reading the same windows run together on one XCD
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const int gi = L % ngroups, rest = L / ngroups;
  const int nbb = W / NB;
  const int sb = (rest % nbb) * NB;
  const int s0 = sb + bg * BPT;                     // first bin of this thread
  const int z0 = (rest / nbb) * ZT;
  const int2 grp = groups[g0 + gi];
  const int gf = max(grp.x, c0), gl = min(grp.x + grp.y, c1);
  const int na = gl - gf;
  const bool active = wave < na;
  const int k = active ? gf + wave : gf;
  const double* aw = ang + (size_t)k * kAngleStride;
  const float2* vol = (aw[kBranch] != 0.0) ? uT : u;
  const double B = aw[kB], D = aw[kD];
  // base bin of the thread's tap positions, and its own first bin from there
  const int sB = HALF ? s0 & ~3 : s0;
  const float bo = HALF ? (float)(s0 & 3) : 0.f;
  const double fA = aw[kA] + (double)sB * B;
  const float Bf = (float)B;
  // Range of the per-row base that keeps every tap of the thread's bins and
  // its right neighbour inside the staged window.  Inside the volume the
  // host's grouping keeps every tap at least one column inside the window,
  // so the clamp changes nothing there; a window moved into the zero
  // padding reads zeros wherever the taps land.
  const float span = (float)((HALF ? 4 : BPT) - 1) * Bf;
  const float rel_lo = fmaxf(0.0f, -span), rel_hi = (float)(SEG - 1) - fmaxf(0.0f, span) - 0.01f;

  // Window of every row, over the group's angles and the block's end bins:
  // from the lowest tap minus one column to the highest tap's right
  // neighbour plus one, columns of margin for rounding (the grouping on the
  // host keeps that within SEG).  Only the rows whose window meets the
  // volume are walked: the others add zeros.  A window wholly outside the
  // volume between two such rows is moved into the zero padding, all SEG
  // columns of it, since the taps are clamped to them.
  if (threadIdx.x == 0) { s_first = W; s_last = -1; }
  __syncthreads();
  int first = W, last = -1;                         // of the wave
  for (int r0 = 0; r0 < W; r0 += kThreads) {
    const int r = r0 + (int)threadIdx.x;            // W is a multiple of 64
    if (r - lane >= W) break;
    double mn = 1e300, mx = -1e300, mn16 = 1e300;
#pragma unroll
    for (int a = 0; a < kFwdNA; ++a) {              // (unrolled: the loads go together)
      const double* ap = ang + (size_t)(gf + min(a, na - 1)) * kAngleStride;
      const double fr = ap[kA] + (double)r * ap[kD];
      const double f0 = fr + (double)sb * ap[kB], f1 = fr + (double)(sb + NB - 1) * ap[kB];
      mn = fmin(mn, fmin(f0, f1));
      mx = fmax(mx, fmax(f0, f1));
      // (the whole block's other end bin)
      if constexpr (HALF) mn16 = fmin(mn16, fr + (double)((sb & 8) != 0 ? sb - 8 : sb + 15) * ap[kB]);
    }
    const int lo = (int)floor(mn) - 1, hi = (int)floor(mx) + 2;   // columns lo .. hi
    const int xl = min(max(lo, -kFwdPad), W + kFwdPad - SEG);
    const int pairs = xl == lo ? min((hi - lo + 2) / 2, SEG / 2) : SEG / 2;
    if constexpr (HALF) {
      const int lo16 = xl == lo ? (int)floor(fmin(mn, mn16)) - 1 : xl;
      s_win[r] = (unsigned)(16 * (lo16 + 64) + pairs - 1 + (xl == lo ? (lo - lo16) << 16 : kMoved));
    } else {
      s_win[r] = (unsigned short)(16 * (xl + 64) + pairs - 1);
    }
    const unsigned long long in = __ballot(hi >= 0 && lo < W);
    if (in) {
      first = min(first, r - lane + __builtin_ctzll(in));
      last = r - lane + 63 - __builtin_clzll(in);
    }
  }
  if (lane == 0 && last >= 0) { atomicMin(&s_first, first); atomicMax(&s_last, last); }
  __syncthreads();
  const int y_end = __builtin_amdgcn_readfirstlane(s_last + 1);
  const int y_beg = min(__builtin_amdgcn_readfirstlane(s_first), y_end);

  // The volume copies are slice-blocked and padded, vol[z / ZB][row][P + col][z % ZB].
  // A load moves one pair of columns (1 KB), pairs w, w + 4, ... of a row by
  // wave w: lane l brings slices 2 (l % 8) and 2 (l % 8) + 1 of slice block
  // (l / 8) % 4 of column 2 pair + l / 32, which is where the [column][slice]
  // row layout wants them (lane l lands at byte 16 l of the load's 1 KB).
  // With 16 pairs in every row these loads set the time (512^3 x 900 angles:
  // 27.2 ms, 19.4 without them, 26.6 without the tap reads), so a row brings
  // no more pairs than its taps read: 23.3 ms, and 21.6 with the rows' windows
  // read from LDS a row before use.
  const int Wf = vol_row(W);
  const size_t plane = (size_t)W * Wf * ZB;
  const float2* vl = vol + (size_t)(z0 / ZB + ((lane >> 3) & 3)) * plane +
                     (size_t)(kFwdPad + 2 * wave + (lane >> 5)) * ZB + 2 * (lane & 7);
  // The loads are issued as inline assembly: the compiler does not track
  // them, so it adds no waits of its own; the loop below waits for them
  // explicitly (vector-memory counter) before the barrier that publishes a
  // row.  M0 holds the wave's LDS destination of each load.
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float4*)tile4;
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  // loads of row y (its s_win entry: win) into buffer buf; returns how many
  // this wave issued
  auto base_of = [](int win) { return (HALF ? win >> 4 & 0xfff : win >> 4) - 64; };   // of the taps
  auto dx_of = [](int win) { return HALF ? win >> 16 & 15 : 0; };
  auto issue = [&](int y, int win, int buf) {
    const int xl = base_of(win) + dx_of(win), n = ((win & 15) + 4 - wv) >> 2;
    const float2* row = vl + ((ptrdiff_t)y * Wf + xl) * ZB;
    const unsigned dst = lds0 + (unsigned)((buf * (ROWF2 / 2) + wv * 64) * 16);
    auto load = [&](int i) {
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %1, off"
          :
          : "s"(dst + 4096u * i), "v"(row + 8 * i * ZB)
          : "memory", "m0");
    };
    if (n >= 3) {                                   // the common counts, 3 and 4
      load(0);
      load(1);
      load(2);
      if (n > 3) load(3);
    } else {
      if (n > 0) load(0);
      if (n > 1) load(1);
    }
    return n;
  };
  // all but the newest n loads of this wave are complete, its LDS reads too
  auto wait_but = [&](int n) {
    if (n >= 3) {
      if (n > 3) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)" ::: "memory");
    } else {
      if (n == 2) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" ::: "memory");
      else if (n == 1) asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    }
  };

  // accumulators: [bin][slice e] with slice 32 (e / 2) + 2 pz + e % 2
  float ax[BPT][4], ay[BPT][4];
  double ox[BPT][4], oy[BPT][4];
#pragma unroll
  for (int b = 0; b < BPT; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) { ax[b][e] = ay[b][e] = 0.f; ox[b][e] = oy[b][e] = 0.0; }

  auto win_of = [&](int y) {
    return __builtin_amdgcn_readfirstlane((int)s_win[min(y, W - 1)]);
  };
  // windows of rows y, y + 1 and y + 2 (read from LDS a row before use)
  int win0 = win_of(y_beg), win1 = win_of(y_beg + 1), win2 = win_of(y_beg + 2);
  int cur = 0, fly = 0;                             // buffer of row y; loads of row y + 1
  if (y_beg < y_end) issue(y_beg, win0, 0);
  if (y_beg + 1 < y_end) fly = issue(y_beg + 1, win1, 1);
  for (int y = y_beg; y < y_end; ++y) {
    // this wave's loads of row y are complete (those of row y + 1 may be in
    // flight) and its LDS reads of row y - 1 have returned; the barrier then
    // publishes row y of every wave and retires row y - 1, whose buffer the
    // loads of row y + 2 reuse
    wait_but(fly);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fly = y + 2 < y_end ? issue(y + 2, win2, cur == 0 ? 2 : cur - 1) : 0;
    const int win3 = (int)s_win[min(y + 3, W - 1)];
    if (active) {
      // tap position of the thread's first bin relative to the window, in
      // double precision; the other bins add b B (< 4 sqrt(2))
      float rel = (float)(fA + (double)y * D - (double)base_of(win0));
      // (HALF: only moved windows, whose clamp fits the narrower window)
      if (!HALF || (win0 & kMoved) != 0) rel = fminf(fmaxf(rel, rel_lo), rel_hi);
      int tb = cur * (ROWF2 / 2) - dx_of(win0) * C4 + pz;
      asm volatile("" : "+v"(tb));                     // one base register per row
      const float4* tr = tile4 + tb;
      // software pipeline: the taps of bin b + 1 are requested before bin b
      // is accumulated
      float4 v[BPT][2][2];                             // [bin][pair][tap]
      auto fetch_bin = [&](int b) {
        const float q = fmaf(bo + (float)b, Bf, rel);     // >= dx, < dx + SEG - 1
        const float4* tp = tr + (int)q * C4;             // truncation = floor here
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          v[b][p][0] = tp[16 * p];
          v[b][p][1] = tp[C4 + 16 * p];
        }
      };
      fetch_bin(0);
#pragma unroll
      for (int b = 0; b < BPT; ++b) {
        if (b + 1 < BPT) fetch_bin(b + 1);
        const float w1 = __builtin_amdgcn_fractf(fmaf(bo + (float)b, Bf, rel)), w0 = 1.0f - w1;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const float4 t0 = v[b][p][0], t1 = v[b][p][1];
          ax[b][2 * p] = fmaf(w1, t1.x, fmaf(w0, t0.x, ax[b][2 * p]));
          ay[b][2 * p] = fmaf(w1, t1.y, fmaf(w0, t0.y, ay[b][2 * p]));
          ax[b][2 * p + 1] = fmaf(w1, t1.z, fmaf(w0, t0.z, ax[b][2 * p + 1]));
          ay[b][2 * p + 1] = fmaf(w1, t1.w, fmaf(w0, t0.w, ay[b][2 * p + 1]));
        }
      }
      if ((y & 31) == 31) {
#pragma unroll
        for (int b = 0; b < BPT; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ox[b][e] += (double)ax[b][e];
            oy[b][e] += (double)ay[b][e];
            ax[b][e] = ay[b][e] = 0.f;
          }
      }
    }
    cur = cur == NBUF - 1 ? 0 : cur + 1;
    win0 = win1;
    win1 = win2;
    win2 = __builtin_amdgcn_readfirstlane(win3);
  }
  if (!active) return;
  const double scale = aw[kScale];
  const double kap = (double)g.kappa;
  const double twopi = 6.283185307179586476925;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float2 o[BPT];
#pragma unroll
    for (int b = 0; b < BPT; ++b) {
      const double px = (ox[b][e] + (double)ax[b][e]) * scale;
      const double py = (oy[b][e] + (double)ay[b][e]) * scale;
      double ph = kap * px;
      ph -= twopi * rint(ph / twopi);
      float sn, cs;
      sincosf((float)ph, &sn, &cs);
      const float mag = expf((float)(-kap * py));
      o[b] = make_float2(mag * cs, mag * sn);
    }
    // the thread's BPT bins of one slice are 8 BPT contiguous bytes
    const int z = z0 + 32 * (e >> 1) + 2 * pz + (e & 1);
    float4* dst = reinterpret_cast<float4*>(psi + ((size_t)(k - c0) * H + z) * W + s0);
#pragma unroll
    for (int b = 0; b < BPT; b += 2) dst[b / 2] = make_float4(o[b].x, o[b].y, o[b + 1].x, o[b + 1].y);
  }
}

// ---------------------------------------------------------------------------
// Transpose on the matrix cores
// ---------------------------------------------------------------------------

// The transpose is a contraction: a 4 x 4 block of voxels projects at one
// angle onto at most 7 consecutive bins (its positions span at most
// 3 sqrt(2), and each footprint max(0, 1 - |i - q| / h) / h is at most two
// bins wide), the same ones for every slice, so
//   g[16 voxels][slices x (re, im)] += w[16 voxels][4 angles x 8 bins]
//                                      h[4 angles x 8 bins][slices x (re, im)]
// is one 16 x 16 x 32 product per 8 slices.  Operands are single-precision
// numbers split into two half-precision terms each, x = x1 + x2 (the second
// term the rounded remainder: x to one unit in its last place, 2^-23),
// multiplied as w1 h1 + w1 h2 + w2 h1 with single-precision sums; the dropped
// w2 h2 is at most 2^-22 of its product, a quarter of what single precision
// leaves of a weight of 1 (positions of up to 21 bins, held to 2^-20).  On
// the vector units the same sums took 8.6 instructions and 8 bytes of LDS
// reads per voxel, slice and angle against 4 bytes and 24 products of
// 16 x 16 x 32 per 16 x 64 x 4 of them here: 345 -> 190 ms at 1024^3 x 1800
// angles, conversion included.  Every slice of h is scaled by a power of two
// (its largest finite value to 2^14 .. 2^15) and the weights by
// 2^kAdjWScale; h2 is stored times 2^kAdjTail and multiplied by w1
// 2^-kAdjTail, so the two terms have about the same size and hold a sample to
// one part in 2^21 down to 2^-30 of its slice's largest, and never worse
// than 2^-51 of that (unscaled, second terms were lost from 2^-17 on).
// The result is scaled back exactly.

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

// Power of two of the second terms of h against their weights (a remainder
// is at most 2^-11 of its sample: 2^12 keeps it below the largest half).
constexpr int kAdjTail = 12;

// Power of two that brings a largest finite magnitude (its bits) to
// 2^14 .. 2^15, within what a float holds together with its inverse; 1 for
// zero.
__device__ __forceinline__ int split_exponent(unsigned bits) {
  if (bits == 0u) return 0;
  return min(14 - ((int)(bits >> 23) - 127), 120);
}

__device__ __forceinline__ unsigned pack_half2(_Float16 a, _Float16 b) {
  half2v v = {a, b};
  return __builtin_bit_cast(unsigned, v);
}

// Four slices of one bin (real parts x, imaginary parts y, bits of the slices'
// largest magnitudes m) as first and second terms.
struct SplitTerms {
  uint4 first, second;
};
__device__ __forceinline__ SplitTerms split_samples(float4 re, float4 im, const unsigned* m) {
  const float x[4] = {re.x, re.y, re.z, re.w}, y[4] = {im.x, im.y, im.z, im.w};
  unsigned a[4], b[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float sc = ldexpf(1.0f, split_exponent(m[c]));
    const float u = x[c] * sc, v = y[c] * sc;
    const _Float16 u1 = (_Float16)u, v1 = (_Float16)v;
    a[c] = pack_half2(u1, v1);
    constexpr float tail = (float)(1 << kAdjTail);
    b[c] = pack_half2((_Float16)((u - (float)u1) * tail), (_Float16)((v - (float)v1) * tail));
  }
  return SplitTerms{make_uint4(a[0], a[1], a[2], a[3]), make_uint4(b[0], b[1], b[2], b[3])};
}

// The sinogram as pass D leaves it to the split form that k_radon_adj stages,
// in the same memory.  Both are [k][z / 64][2][(z / 8) % 8][bin][z % 8]
// words of 32 bits: pass D puts the real part in half 0 and the imaginary
// part in half 1, the split form the first terms of both (two half-precision
// numbers) in half 0 and the second terms (times 2^kAdjTail) in half 1.  An
// infinity or NaN stays one and leaves its slice's scale alone.  The two words
// of a sample are read and written by one thread.  Bound by HBM: 8 bytes read and
// written per bin and slice.
__global__ __launch_bounds__(kThreads) void k_split_sino(unsigned* __restrict__ S,
                                                         const unsigned* __restrict__ smax,
                                                         size_t n, int Wp, int nzb) {
  // item: 4 consecutive slices of one bin
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads) {
    const size_t half = (size_t)8 * Wp * 2;            // items per half block
    const size_t blk = i / half, o = i % half;         // (k, z / 64), offset in it
    const int z = (int)(blk % nzb) * kAdjZT + (int)(o / (2 * Wp)) * 8 + (int)(o & 1) * 4;
    float4* lo = reinterpret_cast<float4*>(S) + blk * 2 * half + o;
    float4* hi = lo + half;
    const SplitTerms t = split_samples(*lo, *hi, smax + z);
    *reinterpret_cast<uint4*>(lo) = t.first;
    *reinterpret_cast<uint4*>(hi) = t.second;
  }
}

// Per-angle constants of a tile: fractional bin of its corner voxel relative
// to the first staged bin, the steps per voxel in x and y, the lowest corner
// of a 4 x 4 block relative to its first voxel, footprint 1/h and 1/h^2
// (times 2^kAdjWScale), the first staged bin and the sinogram row.
struct AdjAngle {
  float f0, c, s, mn;
  float ih, ih2;
  int bin0, row;
};

// The first staged bin is the tile's lowest projection, moved into
// [-kAdjPad, W + kAdjPad - kAdjBins] (a segment outside that range lies wholly
// off the detector, and the padding it is moved to holds zeros); so are those
// of angles that are not `live`, with weight 0.  Double precision; (X0, Y0):
// the tile's corner from the grid's centre.
__device__ __forceinline__ AdjAngle adj_angle(const double* ap, bool live, double cW, double X0,
                                              double Y0, int W, int row) {
  const double C = ap[kCos], Sn = ap[kSin], ih = live ? ap[kInvH] : 0.0;
  const double q0 = cW + X0 * C + Y0 * Sn;
  int sl = (int)floor(q0 + 15.0 * fmin(C, 0.0) + 15.0 * fmin(Sn, 0.0));
  sl = live ? min(max(sl, -kAdjPad), W + kAdjPad - kAdjBins) : -kAdjPad;
  AdjAngle a;
  a.f0 = (float)(q0 - (double)sl);
  a.c = (float)C;
  a.s = (float)Sn;
  a.mn = (float)(3.0 * fmin(C, 0.0) + 3.0 * fmin(Sn, 0.0));
  const double ws = (double)(1 << kAdjWScale);
  a.ih = (float)(ih * ws);
  a.ih2 = (float)(ih * ih * ws);
  a.bin0 = sl + kAdjPad;
  a.row = row;
  return a;
}

// Tile of workgroup L (see k_radon_adj): corner and slice block.
struct AdjTile {
  int x0, y0, zb;
};
__device__ __forceinline__ AdjTile adj_tile(int L, int W) {
  const int nt = W / 16;
  const int GS = (nt % 8 == 0) ? 8 : (nt % 4 == 0) ? 4 : (nt % 2 == 0) ? 2 : 1;
  const int tl = L % (nt * nt), grp = tl / (GS * GS), in_grp = tl % (GS * GS);
  return AdjTile{((grp % (nt / GS)) * GS + in_grp % GS) * 16,
                 ((grp / (nt / GS)) * GS + in_grp / GS) * 16, L / (nt * nt)};
}

// A lane's operands of one 4 x 4 block at one angle: its 8 weights as first
// terms, second terms and first terms times 2^-kAdjTail, and the block's first
// bin.  (fbx, fby): the block's first voxel, (vx, vy): the lane's.
struct AdjWeights {
  half8 w1, w2, wt;
  int bin;
};
__device__ __forceinline__ AdjWeights adj_weights(AdjAngle A, float fbx, float fby, float vx,
                                                  float vy, float minus1) {
  AdjWeights o;
  // the block's lowest bin, and the voxel's position above it
  const float low = fmaf(fby, A.s, fmaf(fbx, A.c, A.f0) + A.mn);
  const float jf = fminf(fmaxf(floorf(low), 0.f), (float)(kAdjBins - 8));
  const float d = fmaf(vy, A.s, fmaf(vx, A.c, A.f0)) - jf;
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const float u = fmaxf(0.0f, fmaf(-fabsf(d - (float)i), A.ih2, A.ih));
    const float v = fmaxf(0.0f, fmaf(-fabsf(d - (float)(i + 1)), A.ih2, A.ih));
    // one packed conversion, whose halves the remainders are then taken from
    unsigned pu = pack_half2((_Float16)u, (_Float16)v);
    asm volatile("" : "+v"(pu));
    const half2v p = __builtin_bit_cast(half2v, pu);
    const half2v r = {(_Float16)fmaf((float)p[0], minus1, u), (_Float16)fmaf((float)p[1], minus1, v)};
    const half2v t = p * (half2v)((_Float16)(1.0f / (1 << kAdjTail)));
    o.w1[i] = p[0];
    o.w1[i + 1] = p[1];
    o.w2[i] = r[0];
    o.w2[i + 1] = r[1];
    o.wt[i] = t[0];
    o.wt[i + 1] = t[1];
  }
  o.bin = (int)jf;
  return o;
}

// Store of one 16-column tile of a block's result: the lane holds column m
// (slice z, re or im) of rows 4 ga .. 4 ga + 3, which are the four voxels from
// `row` on.  Lanes m and m ^ 1 exchange halves, so each stores two complex
// voxels.
__device__ __forceinline__ void adj_store(float4v r, const unsigned* smax, int z, bool im, float2* row) {
  const float sc = ldexpf(1.0f, -split_exponent(smax[z]) - kAdjWScale);
  const float4v v = r * sc;
  const float s0 = im ? v[0] : v[2], s1 = im ? v[1] : v[3];
  const float r0 = __shfl_xor(s0, 1, 64), r1 = __shfl_xor(s1, 1, 64);
  const float4 o = im ? make_float4(r0, v[2], r1, v[3]) : make_float4(v[0], r0, v[1], r1);
  *reinterpret_cast<float4*>(row + (im ? 2 : 0)) = o;
}

// 8 bins of one column from two transposing LDS reads (o: in 8 bytes from wp).
typedef __attribute__((address_space(3))) short4v* LdsHalf4;
__device__ __forceinline__ half8 adj_read8(LdsHalf4 wp, int o) {
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(wp + o);
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(wp + o + 32);
  return __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// A workgroup of 8 waves owns 16 x 16 voxels and 64 slices; wave w the two
// 4 x 4 blocks at x = 4 (w % 4), y = 8 (w / 4) and y + 4.  It walks the
// angles in groups of 4 (one per 16 lanes of a wave): the bins of each angle
// that the tile projects onto (its corners span at most 15 sqrt(2) bins) are
// copied from the split sinogram into LDS by LDS-direct loads two
// groups ahead (three buffers of 52 KB).  Per block a lane forms the 8 footprint
// weights of its voxel and angle (single precision, positions as small
// offsets from double-precision bases) and splits them; the sinogram's
// operand comes from transposing LDS reads: 16 lanes read 4 bins x 16 columns
// stored with the columns fastest, and each lane receives the 4 bins of one
// column (two-address reads of single words took 4.4 clocks of LDS per 512
// bytes, these 2.1 in the counters, and any first bin is aligned).  In LDS the
// 32 bytes (16 columns) of one bin alternate between two angles: the 4 bins of
// two angles that one pass of a read serves lie on different banks wherever
// their windows start.  Partial sums of 32 angles
// are added into outer sums.
__global__ __launch_bounds__(kAdjThreads, 2) void k_radon_adj(const unsigned* __restrict__ S,
                                                              float2* __restrict__ gu, DevGeom g,
                                                              const double* __restrict__ ang,
                                                              int k0, int K,
                                                              const unsigned* __restrict__ smax) {
  constexpr int NA = 4, NB = kAdjBins, TW = kAdjWin;
  constexpr int NT = kAdjZT / 8;                    // 16-column tiles of the result
  // LDS of a group: [angle / 2][tile][half][bin][angle % 2][16 half-precision]
  constexpr int ROWS = 2 * NT * 2 * NB;             // of 64 bytes
  constexpr int LOADS = ROWS / 16;                  // LDS-direct loads (1 KB) per group
  constexpr int LPW = (LOADS + 7) / 8;              // per wave
  static_assert(ROWS % 32 == 0 && LOADS > 8 * (LPW - 1) && NB % 2 == 0 && NB <= kAdjPad, "staging");
  __shared__ uint4 tile4[3 * ROWS * 4];
  __shared__ AdjAngle s_ang[2][TW];
  const int W = g.W, H = g.H, Wp = sino_row(W);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // logical order: slice blocks slowest; within one, the tiles in square
  // groups of GS x GS (x fastest within a group, groups in rows), so the
  // workgroups resident on one XCD cover a compact patch of the slice block
  // whose sinogram segments, per angle, are few and stay in that XCD's L2
  const int L = xcd_logical(blockIdx.x, gridDim.x);
  const AdjTile tile = adj_tile(L, W);
  const int x0 = tile.x0, y0 = tile.y0, zb = tile.zb, nzb = H / kAdjZT;
  const size_t angw = (size_t)nzb * Wp * 128;       // words per angle
  // this workgroup's share of the angle groups (of gridDim.y), whose sums go
  // to a volume of their own
  {
    const int groups = (K + NA - 1) / NA, y = blockIdx.y, ny = gridDim.y;
    const int a0 = NA * (int)((long long)groups * y / ny);
    const int a1 = min(NA * (int)((long long)groups * (y + 1) / ny), K);
    k0 += a0;
    K = a1 - a0;
    S += (size_t)a0 * angw;
    gu += (size_t)y * H * W * W;
  }
  const double X0 = (double)x0 - g.cW, Y0 = (double)y0 - g.cW;
  const int ng = (K + NA - 1) / NA;

  // Constants of angles [w TW, (w + 1) TW) by threads t < TW; those past the
  // last are not live.
  auto setup_window = [&](int w) {
    const int t = threadIdx.x;
    if (t < TW) {
      const int ka = min(w * TW + t, K - 1);
      s_ang[w & 1][t] = adj_angle(ang + (size_t)(k0 + ka) * kAngleStride, w * TW + t < K, g.cW, X0, Y0, W, ka);
    }
  };

  // Loads of a group: load i of wave w brings rows 16 (8 i + w) .. + 15 of
  // LDS; lane l the half l % 2 (8 columns) of the 32 bytes of angle parity
  // (l / 2) % 2 of row l / 4.  The global word of each load relative to the
  // angle's first bin is formed once.  The loads of the next group are
  // spread over the products of the current one: a wave waits at a load
  // until the memory pipeline takes it, and issued together at the start of
  // a group the 52 loads of 1 KB held every wave up (512^3 x 900 angles: 14.9
  // ms with one group ahead, 13.6 spread out, 12.7 spread out and two groups
  // ahead, 10.6 without any; 6.6 is the products alone).  Issued as inline
  // assembly (M0 = LDS destination) so the compiler adds no waits of its
  // own; the loop waits for them explicitly.
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint4*)tile4;
  unsigned goff[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int row = min(16 * (8 * i + wave) + (lane >> 2), ROWS - 1) % (ROWS / 2);
    const int bin = row % NB, th = row / NB;        // th = tile * 2 + half
    goff[i] = (unsigned)(((th & 1) * 8 + (th >> 1)) * Wp + bin) * 8u + 4u * (lane & 1);
  }
  const unsigned* Sz = S + (size_t)zb * (Wp * 128);
  const unsigned* src0 = S;                         // first bins of the lane's two angles
  const unsigned* src1 = S;
  unsigned dst = 0;
  auto issue_begin = [&](int gi, unsigned buf) {
    const AdjAngle* a = &s_ang[((gi * NA) / TW) & 1][(gi * NA) % TW + ((lane >> 1) & 1)];
    src0 = Sz + (size_t)a[0].row * angw + 8u * (unsigned)a[0].bin0;
    src1 = Sz + (size_t)a[2].row * angw + 8u * (unsigned)a[2].bin0;
    dst = __builtin_amdgcn_readfirstlane(lds0 + buf + (unsigned)(wave * 1024));
  };
  auto issue = [&](int i) {
    constexpr int HALF = LOADS / 2;                 // loads of angles 0 and 1
    if (8 * i + 8 <= LOADS || 8 * i + wave < LOADS) {
      const unsigned* src = (8 * i + 8 <= HALF ? src0 : 8 * i >= HALF ? src1
                             : 8 * i + wave < HALF ? src0 : src1) + goff[i];
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "s_nop 0\n\t"
          "global_load_lds_dwordx4 %1, off"
          :
          : "s"(dst + 8192u * i), "v"(src)
          : "memory", "m0");
    }
  };

  // lane: voxel m of a block (A rows) or column m of a tile (B columns), angle
  // ga of the group
  const int m = lane & 15, ga = lane >> 4;
  const int bx = 4 * (wave & 3), by = 8 * (wave >> 2);
  const float vx = (float)(bx + (m & 3)), vy = (float)(by + (m >> 2));
  const float fbx = (float)bx, fby = (float)by;
  float4v acc[2][NT], out[2][NT];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int t = 0; t < NT; ++t) { acc[b][t] = (float4v)(0.f); out[b][t] = (float4v)(0.f); }

  // Operands of block b of group gi, and the LDS address of the lane's words
  // of the block's first pair.
  AdjWeights aw;
  unsigned bp;
  const unsigned lp = lds0 + (unsigned)((ga >> 1) * (ROWS * 32) + (m >> 2) * 64 + (ga & 1) * 32 + (m & 3) * 8);
  float minus1 = -1.0f;
  asm volatile("" : "+s"(minus1));                  // (keeps the mixed-precision FMA of the remainders)
  auto weights = [&](int gi, int b, unsigned buf) {
    const int p0 = gi * NA;
    aw = adj_weights(s_ang[(p0 / TW) & 1][p0 % TW + ga], fbx, fby + 4.f * b, vx, vy + 4.f * b, minus1);
    bp = lp + buf + 64u * (unsigned)aw.bin;
  };

  constexpr int GPW = TW / NA;                      // groups per set-up window
  setup_window(0);
  __syncthreads();
  // LDS offsets of the buffers of groups gi, gi + 1 and gi + 2
  constexpr unsigned BUF = ROWS * 64;
  unsigned buf0 = 0, buf1 = BUF, buf2 = 2 * BUF;
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    issue_begin(min(n, ng - 1), n * BUF);
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue(i);
  }
  weights(0, 0, 0);
  for (int gi = 0; gi < ng; ++gi) {
    // this wave's loads of group gi are complete (those of group gi + 1, at
    // least LPW - 1, may be in flight) and its LDS reads of group gi - 1 have
    // returned; the barrier publishes group gi of every wave, retires group
    // gi - 1 (whose buffer the loads of gi + 2 reuse) and the set-up window
    // written below
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPW - 1) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // (past the last group: its loads again, into an idle buffer)
    issue_begin(min(gi + 2, ng - 1), buf2);
    // the next window's set-up, written three groups before its first group
    // is used, into the slot of the window before the current one
    if ((gi + 3) % GPW == 0 && gi + 3 < ng) setup_window((gi + 3) / GPW);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      // The operands of tile t + LA are requested before tile t is
      // multiplied, and the next block's weights are formed between the
      // products.
      constexpr int LA = 2;
      const half8 w1 = aw.w1, w2 = aw.w2, wt = aw.wt;
      const LdsHalf4 wp = (LdsHalf4)(uintptr_t)bp;
      half8 h1[NT], h2[NT];
      auto fetch = [&](int t) {
        h1[t] = adj_read8(wp, (2 * t) * NB * 8);
        h2[t] = adj_read8(wp, (2 * t + 1) * NB * 8);
      };
#pragma unroll
      for (int t = 0; t < LA; ++t) fetch(t);
      // (the last group's next weights are formed from the window's last
      // entries again and not used)
      weights(b == 0 ? gi : min(gi + 1, ng - 1), 1 - b, b == 0 ? buf0 : buf1);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t + LA < NT) fetch(t + LA);
        if ((8 * b + t) % 2 == 1 && (8 * b + t) / 2 < LPW) issue((8 * b + t) / 2);
        const half8 x1 = h1[t], x2 = h2[t];
        acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w2, x1, acc[b][t], 0, 0, 0);
        acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wt, x2, acc[b][t], 0, 0, 0);
        acc[b][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w1, x1, acc[b][t], 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 3 * NT; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // VALU
      }
    }
    // (formed above, not sunk below the branch)
    asm volatile("" : "+v"(aw.w1), "+v"(aw.w2), "+v"(aw.wt), "+v"(bp));
    const unsigned next = buf0;
    buf0 = buf1;
    buf1 = buf2;
    buf2 = next;
    // two-level single-precision sums: partials of up to 32 angles
    if ((gi & 7) == 7 || gi + 1 == ng) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int t = 0; t < NT; ++t) { out[b][t] += acc[b][t]; acc[b][t] = (float4v)(0.f); }
    }
  }
  // no load may arrive in LDS after the workgroup has ended
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // tile t of block b: column m is slice 8 t + m / 2, row ga of the block
  const size_t WW = (size_t)W * W;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int z = zb * kAdjZT + 8 * t + (m >> 1);
      adj_store(out[b][t], smax, z, (m & 1) != 0,
                gu + (size_t)z * WW + (size_t)(y0 + by + 4 * b + ga) * W + x0 + bx);
    }
}

// The same for a single group (up to 4 angles), from the sinogram as pass D
// leaves it: nothing to pipeline, so the samples are split on their way into
// one LDS buffer, and two workgroups per CU hide each other's reads and the
// stores, which bound it.  One angle, against the general kernel and its split
// pass: 64^3 14.6 -> 9.8 us, 256^3 51.5 -> 34.8, 1024^3 2.40 -> 1.80 ms (8.6
// GB written).
__global__ __launch_bounds__(kAdjThreads, 4) void k_radon_adj_few(const float* __restrict__ S,
                                                                  float2* __restrict__ gu, DevGeom g,
                                                                  const double* __restrict__ ang,
                                                                  int k0, int K,
                                                                  const unsigned* __restrict__ smax) {
  constexpr int NA = 4, NB = kAdjBins, NT = kAdjZT / 8, ROWS = 2 * NT * 2 * NB;
  __shared__ uint4 tile4[ROWS * 4];                 // the layout of k_radon_adj's buffers
  __shared__ AdjAngle s_ang[NA];
  const int W = g.W, Wp = sino_row(W), nzb = g.H / kAdjZT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const AdjTile tile = adj_tile(xcd_logical(blockIdx.x, gridDim.x), W);
  const size_t angw = (size_t)nzb * Wp * 128;       // words per angle
  if (threadIdx.x < NA) {
    const int ka = min((int)threadIdx.x, K - 1);
    s_ang[threadIdx.x] = adj_angle(ang + (size_t)(k0 + ka) * kAngleStride, (int)threadIdx.x < K, g.cW,
                                   (double)tile.x0 - g.cW, (double)tile.y0 - g.cW, W, ka);
  }
  __syncthreads();
  // item: 4 slices (l) of one bin, slice octet and angle
  const float* Sz = S + (size_t)tile.zb * (Wp * 128);
  for (int i = threadIdx.x; i < NA * NT * NB * 2; i += kAdjThreads) {
    const int l = i & 1, bin = (i >> 1) % NB, o = (i >> 1) / NB, t = o % NT, a = o / NT;
    const AdjAngle A = s_ang[a];
    const float* src = Sz + (size_t)A.row * angw + (size_t)(t * Wp + A.bin0 + bin) * 8 + 4 * l;
    const SplitTerms s = split_samples(*reinterpret_cast<const float4*>(src),
                                       *reinterpret_cast<const float4*>(src + (size_t)Wp * 64),
                                       smax + tile.zb * kAdjZT + 8 * t + 4 * l);
    uint4* dst = tile4 + ((a >> 1) * (ROWS / 2) + 2 * t * NB + bin) * 4 + (a & 1) * 2 + l;
    dst[0] = s.first;
    dst[NB * 4] = s.second;
  }
  __syncthreads();
  const int m = lane & 15, ga = lane >> 4;
  const int bx = 4 * (wave & 3), by = 8 * (wave >> 2);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) uint4*)tile4;
  const unsigned lp = lds0 + (unsigned)((ga >> 1) * (ROWS * 32) + (m >> 2) * 64 + (ga & 1) * 32 + (m & 3) * 8);
  float minus1 = -1.0f;
  asm volatile("" : "+s"(minus1));
  const size_t WW = (size_t)W * W;
#pragma unroll 1
  for (int b = 0; b < 2; ++b) {
    const int yb = by + 4 * b;
    const AdjWeights w = adj_weights(s_ang[ga], (float)bx, (float)yb, (float)(bx + (m & 3)),
                                     (float)(yb + (m >> 2)), minus1);
    const LdsHalf4 wp = (LdsHalf4)(uintptr_t)(lp + 64u * (unsigned)w.bin);
#pragma unroll 2
    for (int t = 0; t < NT; ++t) {
      const half8 h1 = adj_read8(wp, (2 * t) * NB * 8), h2 = adj_read8(wp, (2 * t + 1) * NB * 8);
      float4v r = (float4v)(0.f);
      r = __builtin_amdgcn_mfma_f32_16x16x32_f16(w.w2, h1, r, 0, 0, 0);
      r = __builtin_amdgcn_mfma_f32_16x16x32_f16(w.wt, h2, r, 0, 0, 0);
      r = __builtin_amdgcn_mfma_f32_16x16x32_f16(w.w1, h1, r, 0, 0, 0);
      const int z = tile.zb * kAdjZT + 8 * t + (m >> 1);
      adj_store(r, smax, z, (m & 1) != 0,
                gu + (size_t)z * WW + (size_t)(tile.y0 + yb + ga) * W + tile.x0 + bx);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_radon_fwd(const DevGeom& g, const float2* ub, const float2* uTb, float2* psi,
                            const double* ang, const int2* groups, int g0, int ngroups, int c0,
                            int c1, int nb, bool by_size, hipStream_t st) {
  const unsigned n16 = (unsigned)(g.W / kFwdNB) * (unsigned)(g.H / kFwdZT) * (unsigned)ngroups;
  const unsigned n8 = n16 * (kFwdNB / 8);
  // Grids of fewer than two 16-bin workgroups per CU take halves of them: twice
  // as many, each with half the work between a row's barriers.  96 workgroups
  // of 16 bins (64 px, 90 angles) 41.3 -> 35.4 us, 240 (128 px) 74.8 -> 68.6
  // us, but 704 (256 px) 256 -> 325.
  if (nb == 8)
    k_radon_fwd<8, false><<<n8, kThreads, 0, st>>>(ub, uTb, psi, g, ang, groups, g0, ngroups, c0, c1);
  else if (nb == kFwdNB && by_size && n16 < 512)
    k_radon_fwd<8, true><<<n8, kThreads, 0, st>>>(ub, uTb, psi, g, ang, groups, g0, ngroups, c0, c1);
  else if (nb == kFwdNB)
    k_radon_fwd<kFwdNB, false><<<n16, kThreads, 0, st>>>(ub, uTb, psi, g, ang, groups, g0, ngroups,
                                                         c0, c1);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// out = sum over s < ns of P[s n + i], in order.
__global__ __launch_bounds__(kThreads) void k_sum_volumes(const float2* __restrict__ P, int ns, size_t n,
                                                          float2* __restrict__ out) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  float2 a = P[i];
#pragma unroll 8
  for (int s = 1; s < ns; ++s) {
    const float2 v = P[(size_t)s * n + i];
    a = make_float2(a.x + v.x, a.y + v.y);
  }
  out[i] = a;
}

hipError_t launch_radon_adj(const DevGeom& g, float2* S, float2* gu, const double* ang, int k0,
                            int K, const unsigned* smax, float2* tmp, size_t tmp_volumes,
                            hipStream_t st) {
  if (K < 1 || g.H % kAdjZT != 0 || g.W % 16 != 0) return hipErrorInvalidValue;
  unsigned* Sw = reinterpret_cast<unsigned*>(S);
  const int Wp = sino_row(g.W), nzb = g.H / kAdjZT;
  const unsigned n = (unsigned)(g.W / 16) * (unsigned)(g.W / 16) * (unsigned)nzb;
  if (K <= 4) {
    k_radon_adj_few<<<n, kAdjThreads, 0, st>>>(reinterpret_cast<const float*>(S), gu, g, ang, k0, K, smax);
    return hipGetLastError();
  }
  const size_t ns = (size_t)K * nzb * Wp * 16;
  k_split_sino<<<split_sino_blocks(ns), kThreads, 0, st>>>(Sw, smax, ns, Wp, nzb);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // A volume of fewer tiles than CUs (one workgroup each) shares its angles
  // out too, at least 4 groups of them to a share, into volumes in `tmp`.
  // 64^3, 90 angles (16 tiles): 45 -> 27 us in 5 shares; 128^3, 180 angles
  // (128 tiles): 86 -> 69 us in 2.
  const size_t groups = (size_t)(K + 3) / 4;
  const size_t parts = std::min({(size_t)256 / n, groups / 4, tmp_volumes});
  if (parts > 1) {
    k_radon_adj<<<dim3(n, (unsigned)parts), kAdjThreads, 0, st>>>(Sw, tmp, g, ang, k0, K, smax);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const size_t nv = (size_t)g.H * g.W * g.W;
    k_sum_volumes<<<(unsigned)((nv + kThreads - 1) / kThreads), kThreads, 0, st>>>(tmp, (int)parts, nv, gu);
    return hipGetLastError();
  }
  k_radon_adj<<<n, kAdjThreads, 0, st>>>(Sw, gu, g, ang, k0, K, smax);
  return hipGetLastError();
}

hipError_t launch_block_volume(const DevGeom& g, const float2* u, float2* ub, float2* uTb,
                               unsigned* smax, hipStream_t st) {
  const dim3 grid((g.W / 16) * (g.W / 16), g.H / kVolZB);
  k_block_volume<<<grid, kThreads, 0, st>>>(u, ub, uTb, smax, g.W);
  return hipGetLastError();
}

}  // namespace holo
