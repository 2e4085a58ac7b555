// Image-plane kernels (gfx950): periodic PSF convolution (LDS-tiled direct sum), sky / noise /
// flux -> magnitude.  Sec. 2.1 of the paper: each band's image is convolved with its PSF, sky and
// shot noise are added and pixel counts become magnitudes.
#include <math.h>

#include <algorithm>

#include "pcmd_device.h"
#include "pcmd_internal.h"

namespace pcmd {

__global__ void __launch_bounds__(256) k_copy_f32(const float *__restrict__ src, float *__restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t launch_copy_f32(const float *src, float *dst, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_copy_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Noise and magnitude of one pixel of band b with flux G (FP64 arithmetic).  Bound by the vector
// instructions of a Philox block, Box-Muller and a logarithm (4096 x 4096 x 3 as a pass of its own:
// 566 -> 317 us; with the library's functions, among them a power per pixel, 443 instructions each).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ float noise_mag(const NoiseArgs &a, int b, int p, float Gf) {
  constexpr double MAG = -1.0857362047581296;  // -2.5 / ln 10
  const double G = (double)Gf;
  double m;
  if (a.noise_model == PCMD_NOISE_NONE) {
    m = G > 0.0 ? MAG * ln_pos(G) : INFINITY;
  } else {
    const u4 w = philox10((uint32_t)p, (uint32_t)b, TAG_NOISE, 0u, a.k0, a.k1);
    const double z = box_muller(w.x, w.y);
    if (a.noise_model == PCMD_NOISE_GAUSS_MAG) {
      m = G > 0.0 ? MAG * ln_pos(G) + a.sigma[b] * z : INFINITY;
    } else {
      // in this order, and divided: neither t 10^(0.4 zp) nor 1 / t need be finite
      const double t = a.exptime[b], c = G * t * a.zp_flux[b] + a.sky[b];
      const double c2 = c + sqrt(c > 0.0 ? c : 0.0) * z - a.sky[b];
      m = c2 > 0.0 ? MAG * ln_pos(c2 / t) + a.zp[b] : INFINITY;
    }
  }
  return (float)m;
}

// ---------------------------------------------------------------------------------------
// Direct periodic convolution.  G[y][x] = sum_{u,v} P[u][v] F[(y-u+h) mod N][(x-v+h) mod N].
// Each thread owns NX neighbouring outputs of one row of a 64-column tile.  The input tile with its
// K-1 halo (wrapped periodically) and the flipped PSF (rows zero-padded to a multiple of 4) are staged
// in LDS as FP32 and read 16 bytes at a time: tile values into a sliding register window, PSF values
// as broadcasts.  For every PSF row the thread forms the NX K-term dot products in FP32 (all terms
// positive, ascending column; the zero padding adds exact zeros) and adds them to FP64 accumulators
// in ascending row order.
// Bound by FP32 multiply-adds: eight outputs take 32 of them (128 cycles of a SIMD) per two 16-byte
// reads, where four outputs' 64 cycles had the four SIMDs wait for the one LDS.  4096 x 4096 x 3,
// 31 x 31 PSF: 3.07 -> 1.32 ms (2.3 times the FP32 rate, 0.9 of the peak without packed
// instructions).
//
// RS > 1 splits the PSF rows: RS groups of threads share one tile, group g taking rows [g K / RS,
// (g + 1) K / RS); the groups leave their FP64 sums in LDS, where they are added in group order.  Used
// when the image is too small for one-group blocks to fill the chip (256 x 256 x 3, 31 x 31: 24.6 -> 16
// us).
//
// The tile's results go through LDS (the input tile's) to threads of neighbouring pixels, which add the
// noise and store the magnitudes: a launch and a trip of the image through memory less (64 x 64 x 2:
// 9.0 -> 7.7 us, 256 x 256 x 3: 20.7 -> 18.2, 4096 x 4096 x 3: 1615 -> 1611, bound by the arithmetic of both).
// ---------------------------------------------------------------------------------------
constexpr int CT_X = 64, NX = 8;
constexpr int CT_Y1 = 32, CT_YS = 16;  // tile rows: one group of 256 threads, or RS groups of 128
constexpr int CONV_RS = 8;
constexpr int conv_group(int rows) { return rows * (CT_X / NX); }  // threads of a group

__host__ __device__ inline int conv_kp(int K) { return (K + 3) & ~3; }
// the last thread's window ends at column (CT_X - NX) + Kp + NX - 1 and is read in fours
__host__ __device__ inline int conv_tile_w(int K) { return CT_X + conv_kp(K) + 4; }

// Stride of a group's sums [NX][TG]: the 64 pixels of a tile row, (NX indices) x 8 threads, then lie in
// different banks.
constexpr int conv_part_ld(int rows) { return conv_group(rows) + 8; }

static size_t conv_tile_bytes(int K, int rows) {
  return ((size_t)(rows + K - 1) * conv_tile_w(K) + (size_t)K * conv_kp(K)) * sizeof(float);
}
// the tile and the PSF, and afterwards in their place the groups' sums or the results
static size_t conv_lds_bytes(int K, int RS, int rows) {
  const size_t out = RS > 1 ? (size_t)RS * NX * conv_part_ld(rows) * sizeof(double) : (size_t)rows * CT_X * sizeof(float);
  return std::max(conv_tile_bytes(K, rows), out);
}
// The largest PSF that the direct path takes is set by the smaller tile's LDS.
size_t conv_direct_lds_bytes(int K) { return conv_tile_bytes(K, CT_YS); }

// One PSF (band, and region of the sub-pixel grid) checked by one wave, beside the convolution's first tile
// of it: finite, non-negative and summing to one within 1e-3 (a failure sets a status bit reported by
// pcmd_sync).  Per-lane FP64 sums, then a shuffle reduction.
__device__ __forceinline__ void psf_check_wave(const ConvArgs &a, int b) {
  const int KK = a.K * a.K, lane = (int)(threadIdx.x & 63u);
  double s = 0.0;
  bool bad = false;
  for (int i = lane; i < KK; i += 64) {
    const float v = a.psf[(size_t)b * KK + i];
    if (!(v >= 0.0f) || !isfinite(v)) bad = true;
    s += (double)v;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if (lane == 0 && (__ballot(bad) != 0ull || !(fabs(s - 1.0) <= 1e-3))) atomicOr(a.status, STATUS_BAD_PSF);
}

template <int RS, int CT_Y>
__device__ __forceinline__ void conv_direct_body(const ConvArgs &ca, const NoiseArgs &na) {
  extern __shared__ float4 lds4[];
  constexpr int TG = conv_group(CT_Y), THREADS = TG * RS;
  float *tile = reinterpret_cast<float *>(lds4);
  const float *__restrict__ F = ca.F;
  const int N = ca.N, K = ca.K, Kp = conv_kp(K);
  // blockIdx.z = band * grid^2 + region; region (ry, rx) holds the pixels with
  // floor(grid y / N) = ry and floor(grid x / N) = rx, i.e. y in [ceil(ry N / grid), ceil((ry+1) N / grid))
  const int R = ca.grid * ca.grid;
  const int b = blockIdx.z / R, r = blockIdx.z - b * R;
  const int ry = r / ca.grid, rx = r - ry * ca.grid;
  const int y0r = (ry * N + ca.grid - 1) / ca.grid, y1r = ((ry + 1) * N + ca.grid - 1) / ca.grid;
  const int x0r = (rx * N + ca.grid - 1) / ca.grid, x1r = ((rx + 1) * N + ca.grid - 1) / ca.grid;
  const int ox = x0r + blockIdx.x * CT_X, oy = y0r + blockIdx.y * CT_Y;
  if (ox >= x1r || oy >= y1r) return;  // the grid is sized for the largest region
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 64) psf_check_wave(ca, (int)blockIdx.z);
  const int h = (K - 1) >> 1;
  const int TW = conv_tile_w(K), TH = CT_Y + K - 1;
  float *Pf = tile + TW * TH;  // Pf[a][c] = P[K-1-a][K-1-c], 0 for c >= K
  const float *Fb = F + (size_t)b * N * N;
  const float *psf = ca.psf + (size_t)blockIdx.z * K * K;
  // tile[ty][tx] = F[(oy - h + ty) mod N][(ox - h + tx) mod N]; columns past the halo are padding.  A
  // wave stages whole rows (no division per element); an index is at most a few sides out of range
  auto wrap = [N](int i) {
    if (i < 0) i += N;  // i >= -h > -N
    while (i >= N) i -= N;
    return i;
  };
  for (int ty = threadIdx.x >> 6; ty < TH; ty += THREADS / 64) {
    const float *row = Fb + (size_t)wrap(oy - h + ty) * N;
    for (int tx = threadIdx.x & 63; tx < TW; tx += 64) tile[ty * TW + tx] = row[wrap(ox - h + tx)];
  }
  for (int a = threadIdx.x >> 6; a < K; a += THREADS / 64)
    for (int c = threadIdx.x & 63; c < Kp; c += 64) Pf[a * Kp + c] = c < K ? psf[(size_t)(K - 1 - a) * K + (K - 1 - c)] : 0.0f;
  __syncthreads();
  const int grp = RS > 1 ? threadIdx.x / TG : 0, lt = threadIdx.x % TG;
  const int tx = (lt % (CT_X / NX)) * NX, ty = lt / (CT_X / NX);
  // output (oy + ty, ox + tx + i) = sum_{a,c} Pf[a][c] tile[ty + a][tx + i + c]
  double acc[NX];
#pragma unroll
  for (int i = 0; i < NX; ++i) acc[i] = 0.0;
  const int a0 = grp * K / RS, a1 = (grp + 1) * K / RS;
  for (int a = a0; a < a1; ++a) {
    const float *row = tile + (ty + a) * TW + tx;
    const float *prow = Pf + a * Kp;
    float d[NX], w[NX + 4];
#pragma unroll
    for (int i = 0; i < NX; ++i) d[i] = 0.0f;
#pragma unroll
    for (int q = 0; q < NX; q += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(row + q);
      w[q] = v.x;
      w[q + 1] = v.y;
      w[q + 2] = v.z;
      w[q + 3] = v.w;
    }
    for (int c = 0; c < Kp; c += 4) {
      const float4 hi = *reinterpret_cast<const float4 *>(row + c + NX);
      const float4 p4 = *reinterpret_cast<const float4 *>(prow + c);
      w[NX] = hi.x;
      w[NX + 1] = hi.y;
      w[NX + 2] = hi.z;
      w[NX + 3] = hi.w;
      const float pk[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < NX; ++i) d[i] = fmaf(pk[k], w[i + k], d[i]);
#pragma unroll
      for (int i = 0; i < NX; ++i) w[i] = w[i + 4];
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) acc[i] += (double)d[i];
  }
  __syncthreads();
  constexpr int PLD = conv_part_ld(CT_Y);
  double *part = reinterpret_cast<double *>(lds4);  // [RS][NX][PLD]
  if (RS > 1) {
#pragma unroll
    for (int i = 0; i < NX; ++i) part[(grp * NX + i) * PLD + lt] = acc[i];
  } else {
#pragma unroll
    for (int i = 0; i < NX; ++i) tile[ty * CT_X + tx + i] = (float)acc[i];
  }
  __syncthreads();
#pragma unroll 1
  for (int o = threadIdx.x; o < CT_X * CT_Y; o += THREADS) {
    const int x = ox + (o & (CT_X - 1)), y = oy + o / CT_X;
    if (x >= x1r || y >= y1r) continue;
    float g;
    if (RS > 1) {
      const double *q = part + (o & (NX - 1)) * PLD + o / NX;  // thread o / NX of a group, its output o % NX
      double v = q[0];
#pragma unroll
      for (int k = 1; k < RS; ++k) v += q[k * NX * PLD];
      g = (float)v;
    } else {
      g = tile[o];
    }
    const int p = y * N + x;
    if (ca.G) ca.G[(size_t)b * N * N + p] = g;
    na.mags[(size_t)b * N * N + p] = noise_mag(na, b, p, g);
  }
}

template <int RS, int CT_Y>
__global__ void __launch_bounds__(conv_group(CT_Y) * RS) k_conv_direct(ConvArgs a, NoiseArgs na) { conv_direct_body<RS, CT_Y>(a, na); }
template <int RS, int CT_Y>
__global__ void __launch_bounds__(conv_group(CT_Y) * RS) k_conv_direct_job(const ConvArgs *__restrict__ t,
                                                                                const NoiseArgs *__restrict__ tn, int j) {
  const ConvArgs a = t[j];
  conv_direct_body<RS, CT_Y>(a, tn[j]);
}

// Blocks per region side: the largest region of a grid x grid split is ceil(N / grid) wide.
static dim3 conv_grid(int B, int N, int grid, int rows) {
  const int side = (N + grid - 1) / grid;
  return dim3((side + CT_X - 1) / CT_X, (side + rows - 1) / rows, B * grid * grid);
}

template <int RS_, int ROWS_>
struct ConvShape {
  static constexpr int RS = RS_, ROWS = ROWS_;
};
// Calls launch(shape, grid, LDS bytes): row splits when one-group blocks would leave SIMDs with a
// single wave (fewer than 1,024 blocks) and the split's sums fit, else the taller tile, or for the
// widest PSFs the shorter one.
template <typename F>
static hipError_t conv_launch(int B, int N, int K, int grid, F &&launch) {
  constexpr size_t most = 160 * 1024;
  const dim3 g1 = conv_grid(B, N, grid, CT_Y1), gs = conv_grid(B, N, grid, CT_YS);
  const size_t split = conv_lds_bytes(K, CONV_RS, CT_YS), tall = conv_lds_bytes(K, 1, CT_Y1), low = conv_direct_lds_bytes(K);
  if ((int64_t)g1.x * g1.y * g1.z < 1024 && split <= most)
    launch(ConvShape<CONV_RS, CT_YS>{}, gs, split);
  else if (tall <= most)
    launch(ConvShape<1, CT_Y1>{}, g1, tall);
  else if (low <= most)
    launch(ConvShape<1, CT_YS>{}, gs, low);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_conv_direct(const ConvArgs &a, const NoiseArgs &na, hipStream_t s) {
  return conv_launch(a.B, a.N, a.K, a.grid, [&](auto shape, dim3 g, size_t lds) {
    using S = decltype(shape);
    hipLaunchKernelGGL((k_conv_direct<S::RS, S::ROWS>), g, dim3(conv_group(S::ROWS) * S::RS), lds, s, a, na);
  });
}
hipError_t launch_conv_direct_job(const ConvArgs *table, const NoiseArgs *noise, int j, int B, int N, int K, int grid, hipStream_t s) {
  return conv_launch(B, N, K, grid, [&](auto shape, dim3 g, size_t lds) {
    using S = decltype(shape);
    hipLaunchKernelGGL((k_conv_direct_job<S::RS, S::ROWS>), g, dim3(conv_group(S::ROWS) * S::RS), lds, s, table, noise, j);
  });
}

// Noise and magnitudes of an image that no convolution has produced here (no PSF, or the Fourier path): one
// thread per pixel and band.
__device__ __forceinline__ void noise_mag_body(const NoiseArgs &a, int p) {
  const int b = blockIdx.y;
  if (p >= a.npx) return;
  const size_t o = (size_t)b * a.npx + p;
  a.mags[o] = noise_mag(a, b, p, a.G[o]);
}

__global__ void __launch_bounds__(256) k_noise_mag(NoiseArgs a) { noise_mag_body(a, blockIdx.x * blockDim.x + threadIdx.x); }
// (the record stays in memory, as in k_reduce_job)
__global__ void __launch_bounds__(256) k_noise_mag_job(const NoiseArgs *__restrict__ t, int j) {
  noise_mag_body(t[j], blockIdx.x * blockDim.x + threadIdx.x);
}

hipError_t launch_noise_mag_job(const NoiseArgs *table, int j, int npx, int B, hipStream_t s) {
  hipLaunchKernelGGL(k_noise_mag_job, dim3((npx + 255) / 256, B), dim3(256), 0, s, table, j);
  return hipGetLastError();
}

hipError_t launch_noise_mag(const NoiseArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_noise_mag, dim3((a.npx + 255) / 256, a.B), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace pcmd
