// FFT path of the periodic PSF convolution (gfx950), for power-of-two image sides.
//
// G_b = IFFT2( FFT2(F_b) * FFT2(P~_b) ) / N^2, where P~_b is the K x K PSF wrapped onto the N x N
// torus with its centre at the origin; this is the same periodic convolution as the direct sum
// (Sec. 2.1 of the paper convolves each band with its PSF).  FP64 arithmetic (full rate on MI355X),
// so the result agrees with the direct sum to ~1e-15 relative to the image's RMS.
//
// Images are real, so half of the spectrum is kept: two rows are one complex transform (row y +
// i row y + 1), taken apart into the columns kx = 0 .. N / 2 - 1 of both; the real columns 0 and N / 2
// share column 0 (real and imaginary part).  The half spectrum is stored transposed, X[kx][y], so
// that the three passes of an image -- rows forward, columns forward x spectrum x inverse in place,
// rows inverse -- all read and write contiguous memory without passes for transposing.  Bound by
// memory for large images, by launches for small ones; 2048 x 2048 x 3: rows 45, columns 62 (4.8 TB/s),
// rows 43 us (full complex transforms, radix-2 stages in LDS and two transposes took 720 us);
// 4096 x 4096 x 3: 200, 280 and 232 us (3.0 ms).
//
// The PSF spectra and twiddles are kept between calls: a workgroup compares the
// caller's PSF with the copy the spectra were built from (and takes the new one), and the
// spectrum kernels return at once unless something changed, so repeated evaluations with one
// PSF transform only the image.  With the 4 x 4 sub-pixel grid (Sec. 2.2) each of the 16 regions
// has its own spectrum: the image is transformed forward once, and per region the product is
// transformed back (all columns, then the rows of the region's band of rows) and only the
// region's pixels are kept.
#include <math.h>

#include <algorithm>

#include "pcmd_device.h"
#include "pcmd_internal.h"

namespace pcmd {

struct alignas(16) cplx {
  double x, y;
};

__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return cplx{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return cplx{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return cplx{a.x - b.x, a.y - b.y}; }

int fft_supported(int N) { return N >= 8 && N <= 4096 && (N & (N - 1)) == 0; }

static int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Row pitch of a half spectrum: 128 bytes past N, so that the same rows of different columns do not
// all fall on one memory channel.
static size_t fft_pitch(int N) { return (size_t)N + 8; }
static size_t fft_band(int N) { return (size_t)(N / 2) * fft_pitch(N); }

// Scratch layout (complex doubles unless noted): [twiddles N/2][image half spectrum B bands]
// [per-region inverse B bands, sub-pixel grid only][PSF spectra R B bands][PSF copy R B K K floats]
// [change flag u32]
static size_t fft_psf_copy_offset(int B, int N, int R) {
  return sizeof(cplx) * ((size_t)N / 2 + (size_t)((R > 1 ? 2 : 1) + R) * B * fft_band(N));
}
size_t fft_scratch_bytes(int B, int N, int K, int R) {
  return fft_psf_copy_offset(B, N, R) + sizeof(float) * (size_t)R * B * K * K + 256;
}

// Block 0: flag = force or (any element of psf differs from copy); copy = psf (each thread compares its
// elements with their old copies before overwriting them).  The other blocks check one PSF each: finite,
// non-negative and summing to one within 1e-3 (a failure sets a status bit reported by pcmd_sync).
// Latency of a few dependent loads: eight at a time.
__global__ void __launch_bounds__(1024) k_psf_update(const float *__restrict__ psf, float *copy, int64_t n, int KK, int force,
                                                      uint32_t *__restrict__ flag, uint32_t *status) {
  __shared__ int any;
  __shared__ double red[16];
  if (blockIdx.x > 0) {
    const float *P = psf + (size_t)(blockIdx.x - 1) * KK;
    double s = 0.0;
    bool bad = false;
#pragma unroll 8
    for (int i = threadIdx.x; i < KK; i += 1024) {
      const float v = P[i];
      bad = bad || !(v >= 0.0f) || !isfinite(v);
      s += (double)v;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (__any(bad)) s = NAN;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 16; ++w) s += red[w];
      if (!(fabs(s - 1.0) <= 1e-3)) atomicOr(status, STATUS_BAD_PSF);
    }
    return;
  }
  if (threadIdx.x == 0) any = force;
  __syncthreads();
  int d = 0;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += 8192) {
    float v[8], c[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = i0 + 1024 * k;
      v[k] = i < n ? psf[i] : 0.0f;
      c[k] = i < n ? copy[i] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = i0 + 1024 * k;
      if (__float_as_uint(v[k]) != __float_as_uint(c[k])) {
        d = 1;
        copy[i] = v[k];
      }
    }
  }
  if (d) any = 1;
  __syncthreads();
  if (threadIdx.x == 0) *flag = (uint32_t)any;
}

__global__ void k_twiddles(cplx *tw, int N) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < N / 2) {
    double s, c;
    sincospi(-2.0 * (double)m / (double)N, &s, &c);  // exp(-2 pi i m / N)
    tw[m] = cplx{c, s};
  }
}

// ---------------------------------------------------------------------------------------
// A transform of N points by T = N / E threads with E = min(16, N) points each in registers
// (Stockham's order): thread t holds the points t + T m.  Passes of radix 16 (the last one of what is
// left), with an exchange through LDS between two passes: two exchanges at 512 .. 4096 points, where
// two radix-2 stages per exchange took five or six and a pass for the bit reversal.  Results are in
// natural order: thread t ends with the frequencies t + T m, and the inverse transform (real and
// imaginary part swapped before and after) starts from where the forward one ends.
// ---------------------------------------------------------------------------------------
template <int LOGN>
struct FftDim {
  static constexpr int N = 1 << LOGN, E = N < 16 ? N : 16, LOGT = LOGN < 4 ? 0 : LOGN - 4, T = 1 << LOGT;
};

__device__ __forceinline__ void dft4(cplx &a, cplx &b, cplx &c, cplx &d) {
  const cplx t0 = cadd(a, c), t1 = csub(a, c), t2 = cadd(b, d), t3 = csub(b, d);
  a = cadd(t0, t2);
  c = csub(t0, t2);
  b = cplx{t1.x + t3.y, t1.y - t3.x};
  d = cplx{t1.x - t3.y, t1.y + t3.x};
}

// In-register transform of u[0 .. R), natural order in and out.
template <int R>
__device__ __forceinline__ void dft(cplx *u) {
  constexpr double H = 0.7071067811865476, C1 = 0.9238795325112867, S1 = 0.3826834323650898;  // cos pi/4, cos, sin pi/8
  if (R == 2) {
    const cplx a = u[0], b = u[1];
    u[0] = cadd(a, b);
    u[1] = csub(a, b);
  } else if (R == 4) {
    dft4(u[0], u[1], u[2], u[3]);
  } else if (R == 8) {
    dft4(u[0], u[2], u[4], u[6]);
    dft4(u[1], u[3], u[5], u[7]);
    const cplx e[4] = {u[0], u[2], u[4], u[6]};
    const cplx o[4] = {u[1], cplx{H * (u[3].x + u[3].y), H * (u[3].y - u[3].x)}, cplx{u[5].y, -u[5].x},
                       cplx{H * (u[7].y - u[7].x), -H * (u[7].x + u[7].y)}};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      u[k] = cadd(e[k], o[k]);
      u[k + 4] = csub(e[k], o[k]);
    }
  } else if (R == 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) dft4(u[i], u[i + 4], u[i + 8], u[i + 12]);
    // u[n + 4 k] times W16^(n k)
    u[5] = cmul(u[5], cplx{C1, -S1});
    u[9] = cplx{H * (u[9].x + u[9].y), H * (u[9].y - u[9].x)};
    u[13] = cmul(u[13], cplx{S1, -C1});
    u[6] = cplx{H * (u[6].x + u[6].y), H * (u[6].y - u[6].x)};
    u[10] = cplx{u[10].y, -u[10].x};
    u[14] = cplx{H * (u[14].y - u[14].x), -H * (u[14].x + u[14].y)};
    u[7] = cmul(u[7], cplx{S1, -C1});
    u[11] = cplx{H * (u[11].y - u[11].x), -H * (u[11].x + u[11].y)};
    u[15] = cmul(u[15], cplx{-C1, S1});
#pragma unroll
    for (int i = 0; i < 16; i += 4) dft4(u[i], u[i + 1], u[i + 2], u[i + 3]);
    // frequency k + 4 j is in u[4 k + j]
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = k + 1; j < 4; ++j) {
        const cplx v = u[4 * k + j];
        u[4 * k + j] = u[4 * j + k];
        u[4 * j + k] = v;
      }
  }
}

// Element i of the block's transform f: 16-byte slots permuted so that the strided writes of the first
// pass and the reads of different transforms at one frequency spread over the banks.
template <int LOGN>
__device__ __forceinline__ int fft_slot(int f, int i) {
  constexpr int M = FftDim<LOGN>::E - 1;
  return (f << LOGN) + (i ^ (((i >> 4) ^ (f << 2)) & M));
}

template <int LOGN, int LOGNS>
__device__ __forceinline__ void fft_passes(cplx *a, cplx *lds, int f, int t, const cplx *__restrict__ tw) {
  using D = FftDim<LOGN>;
  if constexpr (LOGNS < LOGN) {
    constexpr int LOGR = LOGN - LOGNS < 4 ? LOGN - LOGNS : 4, R = 1 << LOGR, S = D::E / R;
    constexpr int NS = 1 << LOGNS, STEP = 1 << (LOGN - LOGNS - LOGR);  // exp(-2 pi i k / (NS R)) = tw[k STEP]
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int j = t + i * D::T;
      cplx u[R];
#pragma unroll
      for (int r = 0; r < R; ++r) u[r] = a[i + r * S];
      if (LOGNS > 0) {
        const int k = (j & (NS - 1)) * STEP;
        cplx w[R];  // w^r from w, w^2, w^4, w^8: at most three roundings more than a table of all
        w[0] = cplx{1.0, 0.0};
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const int hi = r >= 8 ? 8 : r >= 4 ? 4 : r >= 2 ? 2 : 1;
          w[r] = r == hi ? tw[k * hi] : cmul(w[hi], w[r - hi]);
          u[r] = cmul(u[r], w[r]);
        }
      }
      dft<R>(u);
#pragma unroll
      for (int r = 0; r < R; ++r) a[i + r * S] = u[r];
    }
    if constexpr (LOGNS + LOGR < LOGN) {
#pragma unroll
      for (int i = 0; i < S; ++i) {
        const int j = t + i * D::T, o = ((j >> LOGNS) << (LOGNS + LOGR)) + (j & (NS - 1));
#pragma unroll
        for (int r = 0; r < R; ++r) lds[fft_slot<LOGN>(f, o + r * NS)] = a[i + r * S];
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < D::E; ++m) a[m] = lds[fft_slot<LOGN>(f, t + m * D::T)];
      __syncthreads();
      fft_passes<LOGN, LOGNS + LOGR>(a, lds, f, t, tw);
    }
  }
}

// Rows forward: block x transforms the rows y0 = 2 nf x .. of band blockIdx.y (nf = blockDim / T pairs)
// into the columns of X.  Of F, or (psf given) of band b's PSF at psf + b pstride, wrapped:
// P~[(u - h) mod N][(v - h) mod N] = P[u][v], zero elsewhere.  With `skip` given, the kernel does
// nothing unless *skip is non-zero (PSF spectra that are current).
template <int LOGN>
__global__ void __launch_bounds__(512) k_fft_rows_fwd(const float *__restrict__ F, const float *__restrict__ psf, int K,
                                                       int64_t pstride, cplx *__restrict__ X, int pitch, int lognf,
                                                       const cplx *__restrict__ tw, const uint32_t *__restrict__ skip) {
  using D = FftDim<LOGN>;
  extern __shared__ cplx lds[];
  if (skip && *skip == 0u) return;
  const int f = threadIdx.x >> D::LOGT, t = threadIdx.x & (D::T - 1), b = blockIdx.y;
  const int y0 = blockIdx.x << (lognf + 1), y = y0 + 2 * f;
  cplx a[D::E];
  if (psf) {
    const int h = (K - 1) / 2, u0 = (y + h) & (D::N - 1), u1 = (y + 1 + h) & (D::N - 1);
    const float *P = psf + b * pstride;
#pragma unroll
    for (int m = 0; m < D::E; ++m) {
      const int v = (t + m * D::T + h) & (D::N - 1);
      a[m].x = u0 < K && v < K ? (double)P[u0 * K + v] : 0.0;
      a[m].y = u1 < K && v < K ? (double)P[u1 * K + v] : 0.0;
    }
  } else {
    const float *r = F + ((size_t)b * D::N + y) * D::N + t;
    float x0[D::E], x1[D::E];
#pragma unroll
    for (int m = 0; m < D::E; ++m) {
      x0[m] = r[m * D::T];
      x1[m] = r[D::N + m * D::T];
    }
#pragma unroll
    for (int m = 0; m < D::E; ++m) a[m] = cplx{(double)x0[m], (double)x1[m]};
  }
  fft_passes<LOGN, 0>(a, lds, f, t, tw);
#pragma unroll
  for (int m = 0; m < D::E; ++m) lds[fft_slot<LOGN>(f, t + m * D::T)] = a[m];
  __syncthreads();
  // row y0 + g (g = 2 f' or 2 f' + 1) at kx: (Z[kx] + conj Z[-kx]) / 2 or (Z[kx] - conj Z[-kx]) / 2i
  const int logg = lognf + 1, g = threadIdx.x & ((1 << logg) - 1);
  cplx *out = X + (size_t)b * (D::N / 2) * pitch + y0;
#pragma unroll
  for (int m = 0; m < D::E; ++m) {
    const int i = threadIdx.x + m * blockDim.x;
    const int gi = blockDim.x >= (1u << logg) ? g : i & ((1 << logg) - 1), kx = i >> logg;
    const cplx z = lds[fft_slot<LOGN>(gi >> 1, kx)];
    const cplx w = lds[fft_slot<LOGN>(gi >> 1, kx == 0 ? D::N / 2 : D::N - kx)];
    cplx v = gi & 1 ? cplx{0.5 * (z.y + w.y), 0.5 * (w.x - z.x)} : cplx{0.5 * (z.x + w.x), 0.5 * (z.y - w.y)};
    if (kx == 0) v = gi & 1 ? cplx{z.y, w.y} : cplx{z.x, w.x};
    out[(size_t)kx * pitch + gi] = v;
  }
}

// Z[k], Z[-k] of the shared column 0 times S likewise: the real columns' products, packed again.
__device__ __forceinline__ cplx mul_packed(cplx z, cplx zc, cplx s, cplx sc) {
  const cplx c0{0.5 * (z.x + zc.x), 0.5 * (z.y - zc.y)}, cn{0.5 * (z.y + zc.y), 0.5 * (zc.x - z.x)};
  const cplx s0{0.5 * (s.x + sc.x), 0.5 * (s.y - sc.y)}, sn{0.5 * (s.y + sc.y), 0.5 * (sc.x - s.x)};
  const cplx p = cmul(c0, s0), q = cmul(cn, sn);
  return cplx{p.x - q.y, p.y + q.x};
}

// Columns: block x takes blockDim / T columns of band blockIdx.y.  mode 0: forward, in place.  mode 1:
// forward, times the spectrum S, inverse, in place (Y = X).  mode 2: X (forward already) times S,
// inverse, into Y.
template <int LOGN>
__global__ void __launch_bounds__(256) k_fft_cols(const cplx *X, const cplx *__restrict__ S, cplx *Y, int pitch, int mode,
                                                   const cplx *__restrict__ tw, const uint32_t *__restrict__ skip) {
  using D = FftDim<LOGN>;
  extern __shared__ cplx lds[];
  if (skip && *skip == 0u) return;
  const int f = threadIdx.x >> D::LOGT, t = threadIdx.x & (D::T - 1);
  const int kx = blockIdx.x * (blockDim.x >> D::LOGT) + f;
  const size_t base = ((size_t)blockIdx.y * (D::N / 2) + kx) * pitch;
  cplx a[D::E];
#pragma unroll
  for (int m = 0; m < D::E; ++m) a[m] = X[base + t + m * D::T];
  if (mode != 2) fft_passes<LOGN, 0>(a, lds, f, t, tw);
  if (mode != 0) {
    if (blockIdx.x == 0) {
#pragma unroll
      for (int m = 0; m < D::E; ++m) lds[fft_slot<LOGN>(f, t + m * D::T)] = a[m];
      __syncthreads();
    }
    if (kx == 0) {
#pragma unroll
      for (int m = 0; m < D::E; ++m) {
        const int k = t + m * D::T, c = (D::N - k) & (D::N - 1);
        a[m] = mul_packed(a[m], lds[fft_slot<LOGN>(f, c)], S[base + k], S[base + c]);
      }
    } else {
#pragma unroll
      for (int m = 0; m < D::E; ++m) a[m] = cmul(a[m], S[base + t + m * D::T]);
    }
    if (blockIdx.x == 0) __syncthreads();
#pragma unroll
    for (int m = 0; m < D::E; ++m) a[m] = cplx{a[m].y, a[m].x};
    fft_passes<LOGN, 0>(a, lds, f, t, tw);
#pragma unroll
    for (int m = 0; m < D::E; ++m) a[m] = cplx{a[m].y, a[m].x};
  }
#pragma unroll
  for (int m = 0; m < D::E; ++m) Y[base + t + m * D::T] = a[m];
}

// Rows inverse: block x makes the rows ya + 2 nf x .. of band blockIdx.y, the columns [xa, xb) of them.
template <int LOGN>
__global__ void __launch_bounds__(512) k_fft_rows_inv(const cplx *__restrict__ X, float *__restrict__ G, int pitch, int lognf,
                                                       const cplx *__restrict__ tw, int ya, int xa, int xb) {
  using D = FftDim<LOGN>;
  extern __shared__ cplx lds[];
  const int f = threadIdx.x >> D::LOGT, t = threadIdx.x & (D::T - 1), b = blockIdx.y;
  const int y0 = ya + (blockIdx.x << (lognf + 1)), logg = lognf + 1;
  const cplx *in = X + (size_t)b * (D::N / 2) * pitch + y0;
  cplx a[D::E];
  // A = the even row's, B = the odd row's spectrum at kx: Z = A + i B there, conj A + i conj B at -kx;
  // of a pair of neighbouring lanes one makes each.  Stored with the parts swapped (inverse).
#pragma unroll
  for (int m = 0; m < D::E; ++m) {
    const int i = threadIdx.x + m * blockDim.x, g = i & ((1 << logg) - 1), kx = i >> logg;
    const cplx *q = in + (size_t)kx * pitch + (g & ~1);
    const cplx A = q[0], B = q[1];
    a[m] = g & 1 ? cplx{B.x - A.y, A.x + B.y} : cplx{A.y + B.x, A.x - B.y};
    if (kx == 0) a[m] = g & 1 ? cplx{B.y, A.y} : cplx{B.x, A.x};
  }
#pragma unroll
  for (int m = 0; m < D::E; ++m) {
    const int i = threadIdx.x + m * blockDim.x, g = i & ((1 << logg) - 1), kx = i >> logg;
    lds[fft_slot<LOGN>(g >> 1, g & 1 ? (kx == 0 ? D::N / 2 : D::N - kx) : kx)] = a[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < D::E; ++m) a[m] = lds[fft_slot<LOGN>(f, t + m * D::T)];
  __syncthreads();
  fft_passes<LOGN, 0>(a, lds, f, t, tw);
  constexpr double scale = 1.0 / ((double)D::N * (double)D::N);
  float *r = G + ((size_t)b * D::N + y0 + 2 * f) * D::N;
#pragma unroll
  for (int m = 0; m < D::E; ++m) {
    const int x = t + m * D::T;
    if (x >= xa && x < xb) {
      r[x] = (float)(a[m].y * scale);
      r[D::N + x] = (float)(a[m].x * scale);
    }
  }
}

// Row pairs per block: eight rows fill the 128-byte lines of X (four at 4096, where a pair takes 64 KB
// of LDS); short rows take enough pairs for a wave.
template <int LOGN>
static int row_pairs_log(int rows) {
  int l = LOGN >= 12 ? 1 : 2;
  while ((FftDim<LOGN>::T << l) < 64) ++l;
  while ((2 << l) > rows) --l;
  return l;
}

template <int LOGN>
static hipError_t conv_fft(const float *F, const float *psf, int B, int K, int grid, float *G, void *scratch, bool fresh,
                           uint32_t *status, hipStream_t s) {
  using D = FftDim<LOGN>;
  constexpr int N = D::N;
  const int R = grid * grid, pitch = (int)fft_pitch(N);
  const size_t band = fft_band(N);
  cplx *tw = (cplx *)scratch;
  cplx *X = tw + N / 2;
  cplx *Y = X + (size_t)B * band;                    // sub-pixel grid only
  cplx *Sp = R > 1 ? Y + (size_t)B * band : Y;       // [R][B][N / 2][pitch]
  float *copy = (float *)((char *)scratch + fft_psf_copy_offset(B, N, R));
  uint32_t *flag = (uint32_t *)(copy + (size_t)R * B * K * K);
  const int lf = row_pairs_log<LOGN>(N), nf = 1 << lf;
  const dim3 rgrid(N / 2 / nf, B), rblk(nf * D::T);
  const size_t rlds = sizeof(cplx) * nf * N;
  const int nc = std::min(std::max(128 / D::T, 1), N / 2);  // columns per block: two waves or more
  const dim3 cgrid(N / 2 / nc, B), cblk(nc * D::T);
  const size_t clds = sizeof(cplx) * nc * N;
  if (fresh) hipLaunchKernelGGL(k_twiddles, dim3((N / 2 + 255) / 256), dim3(256), 0, s, tw, N);
  // PSF spectra, rebuilt only when the PSF (or the layout: fresh) changed.  psf is
  // [B][K][K] (grid 1) or [B][16][K][K]: region r of band b at psf + (b R + r) K K.
  hipLaunchKernelGGL(k_psf_update, dim3(1 + R * B), dim3(1024), 0, s, psf, copy, (int64_t)R * B * K * K, K * K, fresh ? 1 : 0,
                     flag, status);
  for (int r = 0; r < R; ++r) {
    cplx *Sr = Sp + (size_t)r * B * band;
    hipLaunchKernelGGL(k_fft_rows_fwd<LOGN>, rgrid, rblk, rlds, s, nullptr, psf + (size_t)r * K * K, K, (int64_t)R * K * K,
                       Sr, pitch, lf, tw, flag);
    hipLaunchKernelGGL(k_fft_cols<LOGN>, cgrid, cblk, clds, s, Sr, nullptr, Sr, pitch, 0, tw, flag);
  }
  hipLaunchKernelGGL(k_fft_rows_fwd<LOGN>, rgrid, rblk, rlds, s, F, nullptr, 0, 0, X, pitch, lf, tw, nullptr);
  if (R == 1) {
    hipLaunchKernelGGL(k_fft_cols<LOGN>, cgrid, cblk, clds, s, X, Sp, X, pitch, 1, tw, nullptr);
    hipLaunchKernelGGL(k_fft_rows_inv<LOGN>, rgrid, rblk, rlds, s, X, G, pitch, lf, tw, 0, 0, N);
    return hipGetLastError();
  }
  // sub-pixel grid: columns forward once; per region the product transformed back, the rows of
  // the region's band of rows, only its columns written
  hipLaunchKernelGGL(k_fft_cols<LOGN>, cgrid, cblk, clds, s, X, nullptr, X, pitch, 0, tw, nullptr);
  const int side = N / grid, ls = row_pairs_log<LOGN>(side), ns = 1 << ls;
  for (int r = 0; r < R; ++r) {
    const int ry = r / grid, rx = r - ry * grid;
    hipLaunchKernelGGL(k_fft_cols<LOGN>, cgrid, cblk, clds, s, X, Sp + (size_t)r * B * band, Y, pitch, 2, tw, nullptr);
    hipLaunchKernelGGL(k_fft_rows_inv<LOGN>, dim3(side / 2 / ns, B), dim3(ns * D::T), sizeof(cplx) * ns * N, s, Y, G, pitch,
                       ls, tw, ry * side, rx * side, (rx + 1) * side);
  }
  return hipGetLastError();
}

hipError_t launch_conv_fft(const float *F, const float *psf, int B, int N, int K, int grid, float *G, void *scratch,
                           bool fresh, uint32_t *status, hipStream_t s) {
  if (!fft_supported(N) || (grid != 1 && grid != 4)) return hipErrorInvalidValue;
  switch (ilog2(N)) {
#define PCMD_FFT(L) \
  case L: return conv_fft<L>(F, psf, B, K, grid, G, scratch, fresh, status, s);
    PCMD_FFT(3) PCMD_FFT(4) PCMD_FFT(5) PCMD_FFT(6) PCMD_FFT(7) PCMD_FFT(8) PCMD_FFT(9) PCMD_FFT(10) PCMD_FFT(11) PCMD_FFT(12)
#undef PCMD_FFT
  }
  return hipErrorInvalidValue;
}

}  // namespace pcmd
