// Fourier-slice ray sums and their transpose for gfx950 (the alternative
// discretisation of R_k; see holo.h, HOLO_PROJECTOR_FOURIER).
//
// The projection of a slice at angle theta is the inverse W-point DFT of the
// slice's discrete-time Fourier transform F(xi) = sum u[y][x]
// e^{-2 pi i xi.(x', y') / W} sampled at xi = m (cos, sin), m = -W/2 .. W/2
// (the two Nyquist samples averaged).  F is evaluated by gridding: the slice,
// divided by the Fourier transform of the spreading kernel, is embedded in an
// M x M grid (M = 2W, twice oversampled) and transformed by 2-D FFT; F(xi)
// is then the kernel-weighted sum of the KW x KW grid values around grid
// position 2 xi.  The kernel is exp(beta (sqrt(1 - (2x/KW)^2) - 1)) on
// |x| < KW/2 (the "exponential of semicircle" shape); with KW = 8 and
// beta = 2.3 KW the gridding error is a few 1e-8 relative.  The transpose
// runs the same steps backwards: per angle a DFT of the bin line, the polar
// samples spread onto the grid (written as a gather: every grid point sums
// the samples within its kernel reach, found from its polar angle through a
// table of the angles sorted modulo pi, so no atomics and a fixed order),
// inverse 2-D FFT, the centre W x W, divided by the kernel's transform.
//
// Slices are processed in slabs of kFsSlab = 8 (every supported height is a
// multiple of 64); the 8 slices of a slab lie next to each other in its grid, G[y][x][slice], and in the
// transpose's polar samples, A[angle][m][slice] (one 64-byte line per grid
// point or sample), so positions and kernel weights are formed once for all
// of them and every gather reads whole lines.  Frequency zero is at (M/2,
// M/2): the slices are multiplied by (-1)^(x' + y') before the forward
// transforms (and after the inverse ones), so that the taps of a sample are
// contiguous except at the grid's edges.  Small slices are processed several
// slabs per launch.  The forward writes psi = exp(i kappa p) of every angle
// into the sinogram buffer (the frame passes copy one chunk at a time from
// there; pass D then overwrites them with h, which the transpose reads).
#include <cmath>

#include "holo_internal.hpp"
#include "fft_lds.hpp"

namespace holo {

namespace {

constexpr int KW = kFsWidth;       // kernel taps per axis
constexpr int SL = kFsSlab;        // slices of a grid point
static_assert(SL == 8, "one 64-byte line per grid point");
typedef float float4v __attribute__((ext_vector_type(4)));

// Threads per line: at most one wavefront, so no transform needs a workgroup
// barrier; 8 lines (the slices of one row, column or angle) per workgroup.
__host__ __device__ constexpr int fs_tl(int N) { return fft_row_threads(N) < 64 ? fft_row_threads(N) : 64; }
__host__ __device__ constexpr int fs_nt(int N) { return SL * fs_tl(N); }
// Pitch of a line in LDS: the padded line plus 4, so that the accesses across
// the lines (slices fastest) spread over the banks.
__host__ __device__ constexpr int fs_pitch(int N) { return fft_line_len(N) + 4; }

// Kernel value at distance x (grid units) from a sample.
__device__ __forceinline__ float es_kernel(float x, float beta) {
  const float z = x * (2.0f / (float)KW);
  const float r = 1.0f - z * z;
  return r > 0.0f ? expf(beta * (sqrtf(r) - 1.0f)) : 0.0f;
}

__device__ __forceinline__ int wrap(int i, int M) { return i < 0 ? i + M : (i >= M ? i - M : i); }

// lines[z][fpi(n)] <-> 64-byte records rec(n) of 8 slices: 4 threads per
// record, 16 bytes each.
template <int N, class F>
__device__ __forceinline__ void fs_records_in(float2* lines, F&& rec) {
  for (int i = threadIdx.x; i < N * 4; i += fs_nt(N)) {
    const int n = i >> 2, q = i & 3;
    const float4 v = rec(n, q);
    lines[(2 * q) * fs_pitch(N) + fpi(n)] = make_float2(v.x, v.y);
    lines[(2 * q + 1) * fs_pitch(N) + fpi(n)] = make_float2(v.z, v.w);
  }
}
template <int N, class F>
__device__ __forceinline__ void fs_records_out(const float2* lines, F&& rec) {
  for (int i = threadIdx.x; i < N * 4; i += fs_nt(N)) {
    const int n = i >> 2, q = i & 3;
    const float2 a = lines[(2 * q) * fs_pitch(N) + fpi(n)];
    const float2 b = lines[(2 * q + 1) * fs_pitch(N) + fpi(n)];
    rec(n, q, make_float4(a.x, a.y, b.x, b.y));
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward: rows (deapodise, embed, FFT), columns (FFT), gridding + inverse
// DFT of the lines of one angle + exp(i kappa p).
// ---------------------------------------------------------------------------

// Row y of the slab's slices: u[z][y][.] / (phihat(x') phihat(y')) (-1)^(x' + y')
// placed at x' mod M (x' = x - W/2), transformed, stored as grid row y' mod M.
template <int W>
__global__ __launch_bounds__(fs_nt(2 * W)) void k_fs_rows(const float2* __restrict__ u,
                                                          float2* __restrict__ G, FsArgs f,
                                                          const float2* __restrict__ tw) {
  constexpr int M = 2 * W, TL = fs_tl(M), E = M / TL, NT = fs_nt(M);
  __shared__ float2 s_tw[fft_line_len(M)];
  __shared__ float2 s_line[SL * fs_pitch(M)];
  const int z = threadIdx.x / TL, lt = threadIdx.x % TL;
  const int y = blockIdx.x, slab = blockIdx.y;
  for (int i = threadIdx.x; i < M; i += NT) s_tw[fpi(i)] = tw[i];
  const float2* row = u + ((size_t)(slab * SL + z) * W + y) * W;
  const float dy = (y & 1) != 0 ? -f.dinv[y] : f.dinv[y];   // W/2 is even
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = lt + e * TL;
    const int xp = n < W / 2 ? n : n - M;             // x' of grid column n
    v[e] = make_float2(0.f, 0.f);
    if (xp >= -W / 2 && xp < W / 2) {
      const int x = xp + W / 2;
      const float s = (x & 1) != 0 ? -dy * f.dinv[x] : dy * f.dinv[x];
      const float2 a = row[x];
      v[e] = make_float2(s * a.x, s * a.y);
    }
  }
  __syncthreads();                                    // s_tw
  float2* Ln = s_line + z * fs_pitch(M);
  fft_e<M, TL, false, true, true>(v, Ln, s_tw, lt);
  fft_sync<true>();
#pragma unroll
  for (int e = 0; e < E; ++e) Ln[fpi(lt + e * TL)] = v[e];
  __syncthreads();
  const int yp = y - W / 2;
  float4* out = reinterpret_cast<float4*>(
      G + (((size_t)slab * M + (yp < 0 ? yp + M : yp)) * M) * SL);
  fs_records_out<M>(s_line, [&](int n, int q, float4 r) { out[n * 4 + q] = r; });
}

// Column transforms of the slab's grids, one grid column (8 slices) per
// workgroup.  Forward: only the W rows y' mod M hold data (the others are
// zero), all M rows are written.  Inverse (the transpose): all M rows are
// read, only those W rows are written.
template <int W, bool INV>
__global__ __launch_bounds__(fs_nt(2 * W)) void k_fs_cols(float2* __restrict__ G,
                                                          const float2* __restrict__ tw) {
  constexpr int M = 2 * W, TL = fs_tl(M), E = M / TL, NT = fs_nt(M);
  __shared__ float2 s_tw[fft_line_len(M)];
  __shared__ float2 s_line[SL * fs_pitch(M)];
  const int z = threadIdx.x / TL, lt = threadIdx.x % TL;
  const int x = xcd_logical(blockIdx.x, gridDim.x), slab = blockIdx.y;
  float4* g = reinterpret_cast<float4*>(G + ((size_t)slab * M * M + x) * SL);
  for (int i = threadIdx.x; i < M; i += NT) s_tw[fpi(i)] = tw[i];
  auto data = [](int r) { return r < W / 2 || r >= M - W / 2; };
  fs_records_in<M>(s_line, [&](int r, int q) {
    return INV || data(r) ? g[(size_t)r * M * 4 + q] : make_float4(0.f, 0.f, 0.f, 0.f);
  });
  __syncthreads();
  float2* Ln = s_line + z * fs_pitch(M);
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = Ln[fpi(lt + e * TL)];
  fft_e<M, TL, INV, true, true>(v, Ln, s_tw, lt);
  fft_sync<true>();
#pragma unroll
  for (int e = 0; e < E; ++e) Ln[fpi(lt + e * TL)] = v[e];
  __syncthreads();
  fs_records_out<M>(s_line, [&](int r, int q, float4 v4) {
    if (!INV || data(r)) g[(size_t)r * M * 4 + q] = v4;
  });
}

// The lines of one angle, 8 slices: F(m (cos, sin)) by gridding for m = -W/2
// .. W/2, the line Q[m mod W] = (-1)^m F (Nyquist samples averaged), p =
// IDFT(Q) / W, psi = exp(i kappa p) written to the sinogram rows
// S[k][z0 + z][kAdjPad + s].  Four threads share a sample, two slices each:
// they form its 16 kernel values (four each, exchanged within the quad) and
// read every tap's 64-byte line together.  Bound by those reads (64 lines a
// sample): with one thread per slice and sample, scattered 8-byte reads and
// every thread forming all weights, a slab of 512^2 slices and 450 angles
// took 218 us, now 64 (94 without consecutive angles on one XCD).
template <int W>
__global__ __launch_bounds__(fs_nt(W), 4) void k_fs_project(const float2* __restrict__ G,
                                                         float2* __restrict__ S, FsArgs f,
                                                         const float2* __restrict__ twW, int H,
                                                         int z0, float kappa) {
  constexpr int M = 2 * W, TL = fs_tl(W), E = W / TL, NT = fs_nt(W);
  __shared__ float2 s_tw[fft_line_len(W)];
  __shared__ float2 s_line[SL * fs_pitch(W)];
  // consecutive angles on one XCD: their samples share its L2's part of the grid
  const int k = xcd_logical(blockIdx.x, gridDim.x), slab = blockIdx.y;
  for (int i = threadIdx.x; i < W; i += NT) s_tw[fpi(i)] = twW[i];
  const double* ap = f.ang + (size_t)(f.k0 + k) * kAngleStride;
  const double C = 2.0 * ap[kCos], Sn = 2.0 * ap[kSin];    // grid units per m
  const float beta = f.beta;
  const int q = threadIdx.x & 3;
  const char* g = reinterpret_cast<const char*>(G + (size_t)slab * M * M * SL);   // < 2^32 bytes
  // F at m, the thread's two slices
  auto grid_at = [&](int m) {
    const FsTap tx = fs_tap(m, C, M), ty = fs_tap(m, Sn, M);
    float wx[KW], wy[KW / 4];                         // wy: rows 4 b + q
#pragma unroll
    for (int b = 0; b < KW / 4; ++b) {
      const float x = es_kernel(fs_dist(tx.r, 4 * b + q), beta);
      wy[b] = es_kernel(fs_dist(ty.r, 4 * b + q), beta);
#pragma unroll
      for (int c = 0; c < 4; ++c) wx[4 * b + c] = __shfl(x, c, 4);
    }
    unsigned cx[KW];                                  // bytes; periodic at the edges
#pragma unroll
    for (int b = 0; b < KW; ++b) cx[b] = (unsigned)wrap(tx.i0 + b, M) * 64u + 16u * (unsigned)q;
    float4v acc = (float4v)(0.f);
#pragma unroll
    for (int h = 0; h < KW / 4; ++h) {
      // (rolled: unrolled, the loads of all 64 taps are hoisted and spill)
#pragma unroll 1
      for (int c = 0; c < 4; ++c) {
        const float w = __shfl(wy[h], c, 4);
        const unsigned row = (unsigned)wrap(ty.i0 + 4 * h + c, M) * (unsigned)(M * 64);
        float4v v[KW];
#pragma unroll
        for (int b = 0; b < KW; ++b) v[b] = *reinterpret_cast<const float4v*>(g + (row + cx[b]));
        float4v r = v[0] * wx[0];
#pragma unroll
        for (int b = 1; b < KW; ++b) r = __builtin_elementwise_fma((float4v)(wx[b]), v[b], r);
        acc = __builtin_elementwise_fma((float4v)(w), r, acc);
      }
    }
    return acc;
  };
  for (int mp = threadIdx.x >> 2; mp < W; mp += NT / 4) {
    const int m = mp - W / 2;
    float4v v = grid_at(m);
    if (mp == 0) v = 0.5f * (v + grid_at(W / 2));   // Nyquist: average of -W/2 and +W/2
    const float sg = (m & 1) ? -1.0f : 1.0f;        // (-1)^m: bins start at s = -W/2
    const int n = fpi(m < 0 ? m + W : m);
    s_line[(2 * q) * fs_pitch(W) + n] = make_float2(sg * v.x, sg * v.y);
    s_line[(2 * q + 1) * fs_pitch(W) + n] = make_float2(sg * v.z, sg * v.w);
  }
  __syncthreads();
  const int z = threadIdx.x / TL, lt = threadIdx.x % TL;
  float2* Ln = s_line + z * fs_pitch(W);
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = Ln[fpi(lt + e * TL)];
  fft_e<W, TL, true, true, true>(v, Ln, s_tw, lt);
  const double twopi = 6.283185307179586476925;
  const int Wp = W + 2 * kAdjPad;
  float2* out = S + ((size_t)k * H + z0 + slab * SL + z) * Wp + kAdjPad;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const float2 p = v[e];
    double ph = (double)kappa * ((double)p.x / (double)W);
    ph -= twopi * rint(ph / twopi);
    float sn, cs;
    sincosf((float)ph, &sn, &cs);
    const float mag = expf(-kappa * (p.y / (float)W));
    out[lt + e * TL] = make_float2(mag * cs, mag * sn);
  }
}

// ---------------------------------------------------------------------------
// Transpose: DFT of the lines of one angle, gather-spread, inverse columns,
// inverse rows + deapodisation.
// ---------------------------------------------------------------------------

// A[k][m + W/2][z] = (-1)^m DFT(h)[m mod W] / W for m = -W/2 .. W/2, the two
// Nyquist entries halved (the transpose of the forward's line step).
template <int W>
__global__ __launch_bounds__(fs_nt(W)) void k_fs_line_T(const float2* __restrict__ S,
                                                        float2* __restrict__ A, FsArgs f,
                                                        const float2* __restrict__ twW, int H,
                                                        int z0) {
  constexpr int TL = fs_tl(W), E = W / TL, NT = fs_nt(W);
  __shared__ float2 s_tw[fft_line_len(W)];
  __shared__ float2 s_line[SL * fs_pitch(W)];
  const int z = threadIdx.x / TL, lt = threadIdx.x % TL;
  const int k = blockIdx.x, slab = blockIdx.y;
  for (int i = threadIdx.x; i < W; i += NT) s_tw[fpi(i)] = twW[i];
  const int Wp = W + 2 * kAdjPad;
  const float2* in = S + ((size_t)k * H + z0 + slab * SL + z) * Wp + kAdjPad;
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = in[lt + e * TL];
  __syncthreads();
  float2* Ln = s_line + z * fs_pitch(W);
  fft_e<W, TL, false, true, true>(v, Ln, s_tw, lt);
  fft_sync<true>();
#pragma unroll
  for (int e = 0; e < E; ++e) Ln[fpi(lt + e * TL)] = v[e];
  __syncthreads();
  float4* out = reinterpret_cast<float4*>(A + ((size_t)slab * f.n_angles + k) * (W + 1) * SL);
  const float sc = 1.0f / (float)W;
  fs_records_out<W>(s_line, [&](int n, int q, float4 r) {
    const int m = n < W / 2 ? n : n - W;
    float s = (m & 1) ? -sc : sc;
    if (m == -W / 2) s *= 0.5f;
    r = make_float4(s * r.x, s * r.y, s * r.z, s * r.w);
    out[(m + W / 2) * 4 + q] = r;
    if (m == -W / 2) out[W * 4 + q] = r;            // m = +W/2 shares the halved value
  });
}

// Every grid point of the slab sums the kernel-weighted polar samples within
// its reach (the transpose of the gridding), for all slices of the slab at
// once: no atomics and a fixed order.  A workgroup owns a 16 x 16 tile of
// grid points, a wave 8 x 8 of them.  The lines that can reach any point of
// the tile are those within d = 8 sqrt(2) + KW sqrt(2)/2 of the tile centre:
// an angle window around the centre's polar angle (found through the table
// of angles sorted modulo pi).  Lines are taken in batches of kSpLines: each
// wave lists the samples of its lines whose taps meet the tile, forms their
// 16 kernel values (the forward's own) and copies their 8 slices into LDS;
// then every wave walks all samples that meet its 8 x 8 points, each sample
// one step of 16 FMAs for all 64 lanes.  Tiles near the grid's edge also
// visit the periodic images that polar samples (radius <= M/2) can reach.
// Near the centre every line of the plan meets the tile, and one workgroup
// would work on it long after the others: such tiles are shared between
// `parts` workgroups (an even share of the window's lines each, sums in
// partial grids that k_fs_join adds in order).  Bound by VALU and LDS; with
// every point testing every line in double precision and the centre tiles
// whole, a slab of 512^2 slices and 450 angles took 1281 us, now 153 + 5.
constexpr int kSpTile = 16, kSpLines = 16, kSpPer = 18;   // samples a line can have in 24 x 24
constexpr int kSpWave = kSpLines / 4 * kSpPer;            // list of one wave

template <int W>
__global__ __launch_bounds__(256) void k_fs_spread(const float2* __restrict__ A,
                                                   float2* __restrict__ G,
                                                   float2* __restrict__ Part, FsArgs f) {
  constexpr int M = 2 * W, NTI = M / kSpTile;
  __shared__ float4 s_a[4 * kSpWave * 4];
  __shared__ float s_wx[4 * kSpWave * KW], s_wy[4 * kSpWave * KW];
  __shared__ int s_ij[4 * kSpWave];                 // first taps relative to the tile
  __shared__ int s_src[4 * kSpWave];
  __shared__ double2 s_r[4 * kSpWave];               // distances from the first taps
  __shared__ int s_cnt[4];
  const FsItem it = f.items[blockIdx.x];
  const int slab = blockIdx.y;
  const int tx = (it.tile % NTI) * kSpTile, ty = (it.tile / NTI) * kSpTile;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // the lane's point, relative to the tile
  const int px = 8 * (wave & 1) + (lane & 7), py = 8 * (wave >> 1) + (lane >> 3);
  const float4* A4 = reinterpret_cast<const float4*>(A + (size_t)slab * f.n_angles * (W + 1) * SL);
  const float beta = f.beta;
  const float d = 8.0f * 1.41421357f + 0.5f * KW * 1.41421357f + 0.05f;
  const float pi = 3.14159265f, bsc = (float)kFsBins / pi;
  float2 acc[SL];
#pragma unroll
  for (int z = 0; z < SL; ++z) acc[z] = make_float2(0.f, 0.f);

  for (int im = 0; im < 9; ++im) {
    // tile origin of this image, frequency zero at 0
    const int ox = tx - M / 2 + (im % 3 - 1) * M, oy = ty - M / 2 + (im / 3 - 1) * M;
    const float icx = (float)ox + 7.5f, icy = (float)oy + 7.5f;
    const float rc = sqrtf(icx * icx + icy * icy);
    if (rc > 0.5f * M + d) continue;                // uniform over the workgroup
    // the tile's angle window: sorted positions, one or two segments (bins
    // are wide against the single-precision angles; one spare on each side)
    int seg[2][2] = {{0, f.n_angles}, {0, 0}};
    if (rc > d) {
      const float dl = asinf(fminf(1.0f, d / rc));
      float phi = atan2f(icy, icx);
      if (phi < 0.0f) phi += pi;
      if (phi >= pi) phi -= pi;
      const int b0 = (int)floorf((phi - dl) * bsc) - 1, b1 = (int)floorf((phi + dl) * bsc) + 1;
      if (b1 - b0 + 1 < kFsBins) {
        if (b0 < 0) {
          seg[0][0] = f.bin_first[b0 + kFsBins];
          seg[1][1] = f.bin_first[b1 + 1];
        } else if (b1 >= kFsBins) {
          seg[0][0] = f.bin_first[b0];
          seg[1][1] = f.bin_first[b1 - kFsBins + 1];
        } else {
          seg[0][0] = f.bin_first[b0];
          seg[0][1] = f.bin_first[b1 + 1];
        }
      }
    }
    // this workgroup's share of the window's lines
    const int n0 = seg[0][1] - seg[0][0], n = n0 + seg[1][1] - seg[1][0];
    const int lo = n * it.part / it.parts, hi = n * (it.part + 1) / it.parts;
    for (int l0 = lo; l0 < hi; l0 += kSpLines) {
      __syncthreads();                              // the previous batch is read
      // list the samples: wave w takes lines l0 + 4 w .. + 3, 20 candidate
      // samples each
      int cnt = 0;
      for (int c0 = 0; c0 < 80; c0 += 64) {
        const int c = c0 + lane, li = l0 + 4 * wave + c / 20, j = c % 20;
        bool ok = c < 80 && li < hi;
        int kk = 0, m = 0;
        FsTap ax{0, 0.0}, ay{0, 0.0};
        if (ok) {
          kk = f.sorted_k[li < n0 ? seg[0][0] + li : seg[1][0] + li - n0] - f.k0;
          ok = kk >= 0 && kk < f.K;
        }
        if (ok) {
          const double* ap = f.ang + (size_t)(f.k0 + kk) * kAngleStride;
          const double C = 2.0 * ap[kCos], Sn = 2.0 * ap[kSin];
          // samples of the line within d of the tile's centre: |2 m - c.e| <= d
          const float ce = 0.5f * (icx * (float)C + icy * (float)Sn);
          m = (int)ceilf(0.5f * (ce - d)) - 1 + j;
          ax = fs_tap(m, C, 0);
          ay = fs_tap(m, Sn, 0);
          ax.i0 -= ox;
          ay.i0 -= oy;
          ok = m >= -W / 2 && m <= W / 2 && ax.i0 > -KW && ax.i0 < kSpTile && ay.i0 > -KW && ay.i0 < kSpTile;
        }
        const unsigned long long mask = __ballot(ok);
        if (ok) {
          const int e = wave * kSpWave + cnt + __popcll(mask & ((1ull << lane) - 1));
          s_ij[e] = (ax.i0 & 0xffff) | (ay.i0 << 16);
          s_src[e] = kk * (W + 1) + m + W / 2;
          s_r[e] = make_double2(ax.r, ay.r);
        }
        cnt += __popcll(mask);
      }
      if (lane == 0) s_cnt[wave] = cnt;
      fft_sync<true>();
      // kernel values (8 lanes per sample, one x and one y tap each) and the
      // slices (4 lanes per sample)
      for (int i = lane; i < cnt * 8; i += 64) {
        const int e = wave * kSpWave + (i >> 3), b = i & 7;
        const double2 r = s_r[e];
        s_wx[e * KW + b] = es_kernel(fs_dist(r.x, b), beta);
        s_wy[e * KW + b] = es_kernel(fs_dist(r.y, b), beta);
      }
      for (int i = lane; i < cnt * 4; i += 64) {
        const int e = wave * kSpWave + (i >> 2);
        s_a[e * 4 + (i & 3)] = A4[(size_t)s_src[e] * 4 + (i & 3)];
      }
      __syncthreads();
      // every sample whose taps meet the wave's 8 x 8 points
      for (int w = 0; w < 4; ++w) {
        const int cw = s_cnt[w];
        for (int c0 = 0; c0 < cw; c0 += 64) {
          const int ij = c0 + lane < cw ? s_ij[w * kSpWave + c0 + lane] : 0x7fff7fff;
          const int bi = (int)(short)(ij & 0xffff) - 8 * (wave & 1), bj = (ij >> 16) - 8 * (wave >> 1);
          unsigned long long mask = __ballot(bi > -KW && bi < 8 && bj > -KW && bj < 8);
          while (mask) {
            const int l = __builtin_ctzll(mask);
            mask &= mask - 1;
            const int e = w * kSpWave + c0 + l;      // uniform
            const int dx = (lane & 7) - __builtin_amdgcn_readlane(bi, l);
            const int dy = (lane >> 3) - __builtin_amdgcn_readlane(bj, l);
            const bool in = (unsigned)dx < (unsigned)KW && (unsigned)dy < (unsigned)KW;
            const float wxy = s_wx[e * KW + (dx & (KW - 1))] * s_wy[e * KW + (dy & (KW - 1))];
            const float wt = in ? wxy : 0.0f;
#pragma unroll
            for (int z = 0; z < SL / 2; ++z) {
              const float4 a = s_a[e * 4 + z];
              acc[2 * z].x = fmaf(wt, a.x, acc[2 * z].x);
              acc[2 * z].y = fmaf(wt, a.y, acc[2 * z].y);
              acc[2 * z + 1].x = fmaf(wt, a.z, acc[2 * z + 1].x);
              acc[2 * z + 1].y = fmaf(wt, a.w, acc[2 * z + 1].y);
            }
          }
        }
      }
    }
  }
  float4* out = it.parts > 1
      ? reinterpret_cast<float4*>(Part + ((size_t)slab * f.n_parts + it.slot) * (256 * SL)) +
            (py * kSpTile + px) * 4
      : reinterpret_cast<float4*>(G + ((size_t)slab * M + ty + py) * M * SL) + (tx + px) * 4;
#pragma unroll
  for (int z = 0; z < SL / 2; ++z)
    out[z] = make_float4(acc[2 * z].x, acc[2 * z].y, acc[2 * z + 1].x, acc[2 * z + 1].y);
}

// The shared tiles: the sum of their parts, in order.  The items of a shared
// tile follow each other, and the shared tiles come first.
template <int W>
__global__ __launch_bounds__(256) void k_fs_join(const float2* __restrict__ Part,
                                                 float2* __restrict__ G, FsArgs f) {
  constexpr int M = 2 * W, NTI = M / kSpTile;
  const FsItem it = f.items[blockIdx.x];
  if (it.part != 0) return;                          // one workgroup per tile
  const int slab = blockIdx.y;
  const float4* p = reinterpret_cast<const float4*>(
      Part + ((size_t)slab * f.n_parts + it.slot) * (256 * SL));
  for (int i = threadIdx.x; i < 256 * 4; i += 256) {
    float4 s = p[i];
    for (int n = 1; n < it.parts; ++n) {
      const float4 v = p[(size_t)n * 256 * 4 + i];
      s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
    }
    const int pt = i >> 2, px = pt % kSpTile, py = pt / kSpTile;
    const int tx = (it.tile % NTI) * kSpTile, ty = (it.tile / NTI) * kSpTile;
    reinterpret_cast<float4*>(G + ((size_t)slab * M + ty + py) * M * SL)[(tx + px) * 4 + (i & 3)] = s;
  }
}

// Row y' mod M of the slab's grid: inverse transform, the W entries x' mod M,
// divided by phihat(x') phihat(y') and times (-1)^(x' + y') -> g_u[z][y][x].
template <int W>
__global__ __launch_bounds__(fs_nt(2 * W)) void k_fs_rows_T(const float2* __restrict__ G,
                                                            float2* __restrict__ gu, FsArgs f,
                                                            const float2* __restrict__ tw) {
  constexpr int M = 2 * W, TL = fs_tl(M), E = M / TL, NT = fs_nt(M);
  __shared__ float2 s_tw[fft_line_len(M)];
  __shared__ float2 s_line[SL * fs_pitch(M)];
  const int z = threadIdx.x / TL, lt = threadIdx.x % TL;
  const int y = blockIdx.x, slab = blockIdx.y;
  for (int i = threadIdx.x; i < M; i += NT) s_tw[fpi(i)] = tw[i];
  const int yp = y - W / 2;
  const float4* in = reinterpret_cast<const float4*>(
      G + (((size_t)slab * M + (yp < 0 ? yp + M : yp)) * M) * SL);
  fs_records_in<M>(s_line, [&](int n, int q) { return in[n * 4 + q]; });
  __syncthreads();
  float2* Ln = s_line + z * fs_pitch(M);
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = Ln[fpi(lt + e * TL)];
  fft_e<M, TL, true, true, true>(v, Ln, s_tw, lt);
  const float dy = (y & 1) != 0 ? -f.dinv[y] : f.dinv[y];
  float2* out = gu + ((size_t)(slab * SL + z) * W + y) * W;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = lt + e * TL;
    const int xp = n < W / 2 ? n : n - M;
    if (xp >= -W / 2 && xp < W / 2) {
      const int x = xp + W / 2;
      const float s = (x & 1) != 0 ? -dy * f.dinv[x] : dy * f.dinv[x];
      out[x] = make_float2(s * v[e].x, s * v[e].y);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// Work items of the spread: the tiles whose angle windows hold more than
// kSpShare of the plan's lines, in shares of at most that many, then the
// others.  Lines are counted as the kernel finds them, images and spare bins
// included, so that scans over part of the half-turn are shared as evenly as
// full ones; 128 lines keep a workgroup about as long as the outer tiles of
// its launch take together.
constexpr int kSpShare = 128;

void fs_build_items(int W, int n_angles, const std::vector<int>& bin_first, std::vector<FsItem>& items,
                    int& n_parts) {
  const int M = 2 * W, nti = M / kSpTile;
  const double d = 8.0 * 1.4142135623730951 + 0.5 * KW * 1.4142135623730951 + 0.05;
  items.clear();
  n_parts = 0;
  std::vector<FsItem> whole;
  // lines of an image whose centre is (cx, cy) from frequency zero
  auto image_lines = [&](double cx, double cy) {
    const double rc = std::sqrt(cx * cx + cy * cy);
    if (rc > 0.5 * M + d) return 0;
    if (rc <= d) return n_angles;
    const double dl = std::asin(d / rc), bsc = kFsBins / M_PI;
    double phi = std::atan2(cy, cx);
    if (phi < 0.0) phi += M_PI;
    if (phi >= M_PI) phi -= M_PI;
    const int b0 = (int)std::floor((phi - dl) * bsc) - 1, b1 = (int)std::floor((phi + dl) * bsc) + 1;
    if (b1 - b0 + 1 >= kFsBins) return n_angles;
    if (b0 < 0) return n_angles - bin_first[b0 + kFsBins] + bin_first[b1 + 1];
    if (b1 >= kFsBins) return n_angles - bin_first[b0] + bin_first[b1 - kFsBins + 1];
    return bin_first[b1 + 1] - bin_first[b0];
  };
  for (int t = 0; t < nti * nti; ++t) {
    const double cx = (t % nti) * kSpTile - M / 2 + 7.5, cy = (t / nti) * kSpTile - M / 2 + 7.5;
    int lines = 0;
    for (int im = 0; im < 9; ++im)
      lines = std::max(lines, image_lines(cx + (im % 3 - 1) * M, cy + (im / 3 - 1) * M));
    const int parts = (lines + kSpShare - 1) / kSpShare;
    if (parts <= 1) {
      whole.push_back(FsItem{t, 0, 1, 0});
      continue;
    }
    for (int p = 0; p < parts; ++p) items.push_back(FsItem{t, p, parts, n_parts + p});
    n_parts += parts;
  }
  items.insert(items.end(), whole.begin(), whole.end());
}

bool fs_size_supported(int W) {
  switch (W) {
    case 64: case 128: case 192: case 256: case 384: case 512: case 1024:
      return true;
    default:
      return false;
  }
}

#define HOLO_FS_SIZES(X) X(64) X(128) X(192) X(256) X(384) X(512) X(1024)

hipError_t launch_fs_forward(const DevGeom& g, const FsArgs& f, const float2* u, float2* G,
                             float2* S, int z0, int nslab, hipStream_t st) {
  if (!g.tw2W || nslab < 1 || z0 + nslab * SL > g.H) return hipErrorInvalidValue;
  const unsigned ns = (unsigned)nslab;
  switch (g.W) {
#define CASE(N)                                                                                 \
  case N: {                                                                                     \
    constexpr int M = 2 * N;                                                                    \
    k_fs_rows<N><<<dim3(N, ns), fs_nt(M), 0, st>>>(u, G, f, g.tw2W);                            \
    k_fs_cols<N, false><<<dim3(M, ns), fs_nt(M), 0, st>>>(G, g.tw2W);                           \
    k_fs_project<N><<<dim3(f.K, ns), fs_nt(N), 0, st>>>(G, S, f, g.twW, g.H, z0, g.kappa);      \
    break;                                                                                      \
  }
    HOLO_FS_SIZES(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fs_adjoint(const DevGeom& g, const FsArgs& f, const float2* S, float2* A,
                             float2* G, float2* Part, float2* gu, int z0, int nslab,
                             hipStream_t st) {
  if (!g.tw2W || nslab < 1 || z0 + nslab * SL > g.H) return hipErrorInvalidValue;
  const unsigned ns = (unsigned)nslab;
  switch (g.W) {
#define CASE(N)                                                                                 \
  case N: {                                                                                     \
    constexpr int M = 2 * N;                                                                    \
    k_fs_line_T<N><<<dim3(f.K, ns), fs_nt(N), 0, st>>>(S, A, f, g.twW, g.H, z0);                \
    k_fs_spread<N><<<dim3(f.n_items, ns), 256, 0, st>>>(A, G, Part, f);                         \
    if (f.n_parts) k_fs_join<N><<<dim3(f.n_parts, ns), 256, 0, st>>>(Part, G, f);               \
    k_fs_cols<N, true><<<dim3(M, ns), fs_nt(M), 0, st>>>(G, g.tw2W);                            \
    k_fs_rows_T<N><<<dim3(N, ns), fs_nt(M), 0, st>>>(G, gu, f, g.tw2W);                         \
    break;                                                                                      \
  }
    HOLO_FS_SIZES(CASE)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace holo
