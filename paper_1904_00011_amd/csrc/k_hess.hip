// Hess diagram (LDS-privatised histogram) and binned log-likelihood reduction (gfx950).
// Sec. 2.5 of the paper: pixels are binned in colour and magnitude (0.05 mag bins) and the
// model and data Hess diagrams are compared bin by bin, with a term for the difference of the
// mean colour and magnitude.
#include <math.h>

#include "pcmd_device.h"
#include "pcmd_internal.h"

namespace pcmd {

__global__ void __launch_bounds__(256) k_fill_u32(uint32_t *__restrict__ p, uint32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

constexpr int HESS_THREADS = 1024;
// Two blocks per CU, each with a private histogram (40 KB for 100 x 100 bins): fewer blocks mean
// fewer merges into the result by device-wide atomics, and HESS_UNROLL pixels in flight per lane
// cover the memory latency.  Bound by the reads of its bands: 4096 x 4096 pixels, two bands, 67 ->
// 42 us (3.2 TB/s; 1,024 blocks of 512 threads with a fence per block before).
constexpr int HESS_MAX_BLOCKS = 512;
constexpr int HESS_LDS_MAX_BINS = 40000;  // 160,000 bytes of LDS (of 163,840 per workgroup)
constexpr int HESS_UNROLL = 4;            // pixels per lane whose loads are issued together
// Up to this many pixels one block bins the whole image, and then stores its histogram and sums
// instead of merging them: no launch to clear the result, no atomics (64 x 64 pixels: 12.6 + 2.2 ->
// 7.1 us; from 8,193 pixels two blocks and the clearing 10.6).
// A diagram beyond LDS has nothing to clear or to merge in a block, and its small images are spread over blocks of
// a pixel per lane, up to HESS_SPREAD (256 x 256 bins, 8,192 pixels: 16.9 us in one block, 8.7 in eight).
constexpr int64_t HESS_ONE_BLOCK = 8192;
constexpr int HESS_SPREAD = HESS_ONE_BLOCK / HESS_THREADS;
int hess_max_blocks() { return HESS_MAX_BLOCKS; }

__device__ __forceinline__ int bin_of(double t, int n) {
  // clamp(floor(t), 0, n-1), NaN -> 0
  if (!(t >= 0.0)) return 0;
  if (t >= (double)n) return n - 1;
  return (int)t;
}

// bin_of(d / dx) without the division where it cannot matter: t = d * (1 / dx) is within 2^-51 |t|
// of the correctly rounded quotient (two roundings of the product, one of the quotient), so for
// |t| < 2^20 and a fraction of t more than 2^-30 from 0 and 1 the quotient has the same floor.
// Everything else (near a bin edge, far outside, infinite, NaN) takes the FP64 division.
__device__ __forceinline__ int bin_fast(double d, double inv_dx, double dx, int n) {
  const double t = d * inv_dx;
  const double f = __builtin_amdgcn_fract(t);
  if (f > 0x1p-30 && f < 1.0 - 0x1p-30 && fabs(t) < 0x1p20) return min(max((int)t, 0), n - 1);
  return bin_of(d / dx, n);
}

// The three sums over the block in v, in a fixed order: shuffles within each wave, then the waves in
// order (one barrier on each side for all three).
__device__ __forceinline__ void block_sum3(double (&v)[3], double (*red)[3]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] += __shfl_down(v[c], off, 64);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int c = 0; c < 3; ++c) red[threadIdx.x >> 6][c] = v[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) v[c] = 0.0;
  if (threadIdx.x == 0)  // the only thread that uses the sums
    for (int w = 0; w < HESS_THREADS / 64; ++w)
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] += red[w][c];
}

// Does not fall as npx grows: a launch over several jobs has the blocks of the largest.
__host__ __device__ static inline int hess_blocks_of(int64_t npx, int nbins) {
  const bool lds = nbins <= HESS_LDS_MAX_BINS;
  if (lds && npx <= HESS_ONE_BLOCK) return 1;
  // enough pixels per block to amortise clearing and merging the private histogram
  int64_t blocks = (npx + 4095) / 4096;
  if (!lds && blocks < HESS_SPREAD) {
    blocks = (npx + HESS_THREADS - 1) / HESS_THREADS;
    if (blocks > HESS_SPREAD) blocks = HESS_SPREAD;
  }
  if (blocks > HESS_MAX_BLOCKS) blocks = HESS_MAX_BLOCKS;
  return (int)blocks;
}
int hess_blocks(int64_t npx, int nbins) { return hess_blocks_of(npx, nbins); }
bool hess_use_lds(int nbins) { return nbins <= HESS_LDS_MAX_BINS; }
// one block with a private histogram: the result needs no clearing
static bool hess_stores(int64_t npx, int nbins) { return hess_use_lds(nbins) && hess_blocks(npx, nbins) == 1; }

// by nblk blocks
__device__ __forceinline__ void hess_body(const HessArgs &a, unsigned nblk) {
  extern __shared__ uint32_t lh[];
  __shared__ double red[HESS_THREADS / 64][3];
  __shared__ bool last;
  const int nb = a.nx * a.ny;
  if (a.use_lds) {
    for (int j = threadIdx.x; j < nb; j += HESS_THREADS) lh[j] = 0u;
    __syncthreads();
  }
  double sum[3] = {0.0, 0.0, 0.0};  // x, y, pixels
  const double inv_dx = 1.0 / a.dx, inv_dy = 1.0 / a.dy;
  const float *mb = a.mags + (size_t)a.bb * a.npx;
  const float *mr = a.mags + (size_t)a.br * a.npx;
  const float *mm = a.mags + (size_t)a.bm * a.npx;
  const uint32_t npx = (uint32_t)a.npx, stride = nblk * HESS_THREADS;  // at most 2^31 pixels
  for (uint32_t p0 = blockIdx.x * HESS_THREADS + threadIdx.x; p0 < npx; p0 += HESS_UNROLL * stride) {
    float fb[HESS_UNROLL], fr[HESS_UNROLL], fm[HESS_UNROLL];
#pragma unroll
    for (int k = 0; k < HESS_UNROLL; ++k) {
      const uint32_t p = min(p0 + k * stride, npx - 1u);  // past the end: the last pixel again, not counted
      fb[k] = mb[p];
      fr[k] = mr[p];
      fm[k] = a.bm == a.br ? fr[k] : a.bm == a.bb ? fb[k] : mm[p];
    }
#pragma unroll
    for (int k = 0; k < HESS_UNROLL; ++k) {
      if (p0 + k * stride >= npx) break;
      const double x = (double)fb[k] - (double)fr[k], y = (double)fm[k];
      const int ix = bin_fast(x - a.x0, inv_dx, a.dx, a.nx);
      const int iy = bin_fast(y - a.y0, inv_dy, a.dy, a.ny);
      const int j = iy * a.nx + ix;
      if (a.use_lds)
        atomicAdd(&lh[j], 1u);
      else
        atomicAdd(&a.hess[j], 1u);
      // the difference of two FP32 values is finite in FP64 exactly when both are
      if (isfinite(x) && isfinite(y)) {
        sum[0] += x;
        sum[1] += y;
        sum[2] += 1.0;
      }
    }
  }
  const bool one = nblk == 1;
  if (a.use_lds) {
    __syncthreads();
    for (int j = threadIdx.x; j < nb; j += HESS_THREADS) {
      const uint32_t v = lh[j];
      if (one)
        a.hess[j] = v;
      else if (v)
        atomicAdd(&a.hess[j], v);
    }
  }
  block_sum3(sum, red);
  if (one) {
    if (threadIdx.x == 0)
#pragma unroll
      for (int c = 0; c < 3; ++c) a.moments[c] = sum[c];
    return;
  }
  if (threadIdx.x == 0) {
    // The partial goes out by device-scope stores, which reach memory that every XCD reads, and is
    // complete before the block counts itself.  A __threadfence or a releasing count would write back the whole
    // L2 of the XCD, once per block (4096 x 4096 pixels: 116 us, 101 so).
#pragma unroll
    for (int c = 0; c < 3; ++c)
      __hip_atomic_store(a.mom_part + blockIdx.x * 3 + c, sum[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint32_t prev = atomicAdd(a.counter, 1u);
    last = (prev == nblk - 1);
  }
  __syncthreads();
  if (last) {
    // every block's partial is in memory: thread t adds blocks t, t + HESS_THREADS, ... in order
    // (device-scope loads), then the fixed-order block sum (the combination does not depend on
    // which block is last)
#pragma unroll
    for (int c = 0; c < 3; ++c) sum[c] = 0.0;
    for (unsigned k = threadIdx.x; k < nblk; k += HESS_THREADS)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        sum[c] += __hip_atomic_load(a.mom_part + k * 3 + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    block_sum3(sum, red);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) a.moments[c] = sum[c];
      *a.counter = 0u;  // ready for the next call (also under graph replay)
    }
  }
}

__global__ void __launch_bounds__(HESS_THREADS, 8) k_hess(HessArgs a) { hess_body(a, gridDim.x); }
__global__ void __launch_bounds__(HESS_THREADS, 8) k_hess_jobs(const HessArgs *__restrict__ t) {
  const HessArgs a = t[blockIdx.y];
  const unsigned nblk = (unsigned)hess_blocks_of(a.npx, a.nx * a.ny);  // those of the same single call
  if (blockIdx.x < nblk) hess_body(a, nblk);
}

hipError_t launch_hess(const HessArgs &a, hipStream_t s) {
  const int nb = a.nx * a.ny;
  if (!hess_stores(a.npx, nb)) {
    const hipError_t e = launch_fill_u32(a.hess, 0u, nb, s);
    if (e != hipSuccess) return e;
  }
  const size_t lds = a.use_lds ? (size_t)nb * sizeof(uint32_t) : 0;
  hipLaunchKernelGGL(k_hess, dim3((unsigned)hess_blocks(a.npx, nb)), dim3(HESS_THREADS), lds, s, a);
  return hipGetLastError();
}

__global__ void __launch_bounds__(256) k_hess_clear_jobs(const HessArgs *__restrict__ t, int nbins) {
  uint32_t *h = t[blockIdx.y].hess;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nbins) h[i] = 0u;
}

// The diagrams of n jobs cleared, for the blocks that add to them (a small image's one block stores).
hipError_t launch_hess_clear_jobs(const HessArgs *table, int n, int nbins, hipStream_t s) {
  hipLaunchKernelGGL(k_hess_clear_jobs, dim3((nbins + 255) / 256, n), dim3(256), 0, s, table, nbins);
  return hipGetLastError();
}

// The diagrams of n jobs, cleared before, of at most npx_max pixels.  (24 uneven jobs 24 x 11 us one by one,
// 26 together.)
hipError_t launch_hess_jobs(const HessArgs *table, int n, int64_t npx_max, int nbins, hipStream_t s) {
  const size_t lds = hess_use_lds(nbins) ? (size_t)nbins * sizeof(uint32_t) : 0;
  hipLaunchKernelGGL(k_hess_jobs, dim3((unsigned)hess_blocks(npx_max, nbins), n), dim3(HESS_THREADS), lds, s, table);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Log-likelihood.  A diagram of up to LL_ONE_BINS bins is scored by one block of LL_ONE_THREADS
// threads, which loads all its bins before it uses the first, so that the totals N_m, N_d, the bins'
// terms and the mean-colour / mean-magnitude term take one launch and no scratch: bound by a launch (1,000
// bins: 9.5 us in two launches, 4.7 us in one), and from some thousand bins by one CU's FP64 rate, which the
// logarithms of the bins with data take (4,096 bins 5.9 us, 10,000 bins 9.5 us, 7.8 us where most waves' bins
// hold none, 14.1 us if every bin's count is beyond the table of factorials).  Larger diagrams take
// ceil(nbins / LL_THREADS) blocks, each of which recomputes the totals (integer sums are exact, so they agree) and
// writes its sum to part[block]; a second one-block kernel adds the sums in block order (10,000 bins 9.5 us, 16,384
// bins 10.8 us, where one block takes 15; 40,000 bins: 21.5 + 4.6 us, and one block has four
// times the work of 10,000 bins and 1/256 of the chip).
// The order of every sum depends on nbins alone.
// ---------------------------------------------------------------------------------------

// One bin's term, from its counts and the totals.  Poisson bins without data need no logarithm
// (0 ln lam = 0; with no data at all lam = 0 and the term is 0 ln 0, not a number).
struct BinTerm {
  int mode;
  double eps, Nm, Nd, den, inv;  // den: N_m + eps n_bins or N_m
  bool near;                     // inv = 1 / den is a normal number (eps near either end of the range: it may not be)
  const double *lnfact64;
  __device__ __forceinline__ BinTerm(const LoglikeArgs &a, double nm, double nd)
      : mode(a.mode), eps(a.eps), Nm(nm), Nd(nd), lnfact64(a.lnfact64) {
    den = mode == PCMD_LL_POISSON ? nm + a.eps * (double)a.nbins : nm;
    inv = 1.0 / den;
    near = inv >= 0x1p-1022 && inv < INFINITY;
  }
  // x / den: with the rounded reciprocal, and the quotient corrected by its exact remainder, the rounded
  // quotient (Markstein) in three operations
  __device__ __forceinline__ double over_den(double x) const {
    if (!near) return x / den;
    const double q = x * inv;
    return fma(fma(-den, q, x), inv, q);
  }
  __device__ __forceinline__ double operator()(uint32_t hm, uint32_t hd) const {
    const double m = (double)hm, d = (double)hd;
    if (mode == PCMD_LL_POISSON) {
      const double lam = over_den(Nd * (m + eps));
      if (hd == 0u && Nd != 0.0) return -lam;
      const double lf = hd < (uint32_t)LNFACT64_N ? lnfact64[hd] : ln_factorial_large(hd);
      // d ln lam with ln lam = hi + lo: two roundings less than product and sums one by one, and half the
      // instructions of the library's logarithm (10,000 bins 12.0 -> 9.8 us, of large counts 21.9 -> 14.1)
      double lo;
      double hi = ln_split(lam, lo);
      if (!(lam > 0.0 && lam < INFINITY)) {
        hi = lam == 0.0 ? -INFINITY : lam;
        lo = 0.0;
      }
      return fma(d, hi, fma(d, lo, -lam - lf));
    }
    // Gaussian: sigma^2 = max(variance, 2^2)
    double df, var;
    if (mode == PCMD_LL_GAUSS_PAPER) {
      const double mh = over_den(m * Nd);
      df = d - mh;
      var = d + mh;
    } else {
      df = d / Nd - m / Nm;
      var = d * d + m * m;
    }
    return -df * df / (2.0 * fmax(var, 4.0));
  }
};

// The mean-colour / mean-magnitude term.
__device__ __forceinline__ double mean_term(const LoglikeArgs &a) {
  if (a.mode == PCMD_LL_POISSON) return 0.0;
  const double Cm = a.mom_m[0] / a.mom_m[2], Mm = a.mom_m[1] / a.mom_m[2];
  const double Cd = a.mom_d[0] / a.mom_d[2], Md = a.mom_d[1] / a.mom_d[2];
  return -(Cd - Cm) * (Cd - Cm) / (2.0 * 0.05 * 0.05) - (Md - Mm) * (Md - Mm) / (2.0 * 0.05 * 0.05);
}

constexpr int LL_ONE_THREADS = 1024;
constexpr int LL_ONE_BINS = 10 * LL_ONE_THREADS;

// Sum over the block's waves in order, of values already summed within each wave.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// R: bins per thread, nbins <= R LL_ONE_THREADS.
template <int R>
__device__ __forceinline__ void loglike_one_body(const LoglikeArgs &a) {
  constexpr int W = LL_ONE_THREADS / 64;
  __shared__ unsigned long long tot[W][2];
  __shared__ double sums[W];
  const int t = threadIdx.x, wave = t >> 6;
  uint32_t vm[R], vd[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int j = min(t + k * LL_ONE_THREADS, a.nbins - 1);
    vm[k] = a.hm[j];
    vd[k] = a.hd[j];
  }
  unsigned long long sm = 0, sd = 0;
#pragma unroll
  for (int k = 0; k < R; ++k)
    if (t + k * LL_ONE_THREADS < a.nbins) {
      sm += vm[k];
      sd += vd[k];
    }
  sm = wave_sum(sm);
  sd = wave_sum(sd);
  if ((t & 63) == 0) {
    tot[wave][0] = sm;
    tot[wave][1] = sd;
  }
  __syncthreads();
  sm = sd = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    sm += tot[w][0];
    sd += tot[w][1];
  }
  const BinTerm term(a, (double)sm, (double)sd);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < R; ++k)
    if (t + k * LL_ONE_THREADS < a.nbins) acc += term(vm[k], vd[k]);
  acc = wave_sum(acc);
  if ((t & 63) == 0) sums[wave] = acc;
  __syncthreads();
  if (t != 0) return;
  double r = 0.0;
#pragma unroll
  for (int w = 0; w < W; ++w) r += sums[w];
  r += mean_term(a);
  a.out[0] = a.accumulate ? a.out[0] + r : r;
}

// Fixed-order sum over the block (tree in LDS).
template <typename T>
__device__ __forceinline__ T block_sum_ordered(T v, T *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = LL_THREADS / 2; s > 0; s >>= 1) {
    if (t < s) sh[t] = sh[t] + sh[t + s];
    __syncthreads();
  }
  const T r = sh[0];
  __syncthreads();
  return r;
}

__device__ __forceinline__ void loglike_bins_body(const LoglikeArgs &a, int blk) {
  const uint32_t *__restrict__ hm = a.hm;
  const uint32_t *__restrict__ hd = a.hd;
  const int nbins = a.nbins;
  __shared__ unsigned long long shu[LL_THREADS];
  __shared__ double shd[LL_THREADS];
  const int t = threadIdx.x;
  unsigned long long sm = 0, sd = 0;
  // batches of 8 bins per thread loaded into separate registers before they are added, so the
  // 16 loads are in flight together (one register reused for every load serialised them)
  for (int j0 = t; j0 < nbins; j0 += 8 * LL_THREADS) {
    uint32_t vm[8], vd[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u * LL_THREADS;
      vm[u] = j < nbins ? hm[j] : 0u;
      vd[u] = j < nbins ? hd[j] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      sm += vm[u];
      sd += vd[u];
    }
  }
  const double Nm = (double)block_sum_ordered(sm, shu);
  const double Nd = (double)block_sum_ordered(sd, shu);
  const int j = blk * LL_THREADS + t;
  const BinTerm term(a, Nm, Nd);
  const double bsum = block_sum_ordered(j < nbins ? term(hm[j], hd[j]) : 0.0, shd);
  if (t == 0) a.part[blk] = bsum;
}

__device__ __forceinline__ void loglike_final_body(const LoglikeArgs &a) {
  // the 64 lanes fetch the block sums together; lane 0 adds them in block order
  __shared__ double ps[256];
  const int nb = loglike_blocks(a.nbins);
  double r = 0.0;
  for (int b0 = 0; b0 < nb; b0 += 256) {
    const int n = min(256, nb - b0);
    for (int k = threadIdx.x; k < n; k += 64) ps[k] = a.part[b0 + k];
    __syncthreads();
    if (threadIdx.x == 0)
      for (int k = 0; k < n; ++k) r += ps[k];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  r += mean_term(a);
  a.out[0] = a.accumulate ? a.out[0] + r : r;
}

template <int R>
__global__ void __launch_bounds__(LL_ONE_THREADS) k_loglike_one(LoglikeArgs a) { loglike_one_body<R>(a); }
__global__ void __launch_bounds__(LL_THREADS) k_loglike_bins(LoglikeArgs a) { loglike_bins_body(a, blockIdx.x); }
__global__ void __launch_bounds__(64) k_loglike_final(LoglikeArgs a) { loglike_final_body(a); }
// batched: grid.y (bins) / grid.x (final) runs over the jobs of a descriptor table
template <int R>
__global__ void __launch_bounds__(LL_ONE_THREADS) k_loglike_one_jobs(const LoglikeArgs *__restrict__ t) {
  const LoglikeArgs a = t[blockIdx.x];
  loglike_one_body<R>(a);
}
__global__ void __launch_bounds__(LL_THREADS) k_loglike_bins_jobs(const LoglikeArgs *__restrict__ t) {
  const LoglikeArgs a = t[blockIdx.y];
  loglike_bins_body(a, blockIdx.x);
}
__global__ void __launch_bounds__(64) k_loglike_final_jobs(const LoglikeArgs *__restrict__ t) {
  const LoglikeArgs a = t[blockIdx.x];
  loglike_final_body(a);
}

hipError_t launch_loglike(const LoglikeArgs &a, hipStream_t s) {
  const dim3 one(LL_ONE_THREADS);
  if (a.nbins <= 4 * LL_ONE_THREADS) {
    hipLaunchKernelGGL(k_loglike_one<4>, dim3(1), one, 0, s, a);
  } else if (a.nbins <= LL_ONE_BINS) {
    hipLaunchKernelGGL(k_loglike_one<10>, dim3(1), one, 0, s, a);
  } else {
    hipLaunchKernelGGL(k_loglike_bins, dim3((unsigned)loglike_blocks(a.nbins)), dim3(LL_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_loglike_final, dim3(1), dim3(64), 0, s, a);
  }
  return hipGetLastError();
}
hipError_t launch_loglike_jobs(const LoglikeArgs *table, int n_jobs, int nbins, hipStream_t s) {
  const dim3 one(LL_ONE_THREADS), jobs((unsigned)n_jobs);
  if (nbins <= 4 * LL_ONE_THREADS) {
    hipLaunchKernelGGL(k_loglike_one_jobs<4>, jobs, one, 0, s, table);
  } else if (nbins <= LL_ONE_BINS) {
    hipLaunchKernelGGL(k_loglike_one_jobs<10>, jobs, one, 0, s, table);
  } else {
    hipLaunchKernelGGL(k_loglike_bins_jobs, dim3((unsigned)loglike_blocks(nbins), (unsigned)n_jobs), dim3(LL_THREADS), 0,
                       s, table);
    hipLaunchKernelGGL(k_loglike_final_jobs, jobs, dim3(64), 0, s, table);
  }
  return hipGetLastError();
}

}  // namespace pcmd
