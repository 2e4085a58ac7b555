// Surrogate network kernels (gfx950): BF16 MFMA matrix products with FP32 accumulation and fused
// epilogues (bias, GELU, GELU derivative), MSE gradient, bias gradients, Adam with BF16 shadow
// weights, and the surrogate Poisson log-likelihood.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "pcmd_device.h"
#include "pcmd_internal.h"
#include "pcmd_mlp.h"

namespace pcmd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.3989422804014327f;
}

// ---------------------------------------------------------------------------------------
// C[M][N] = sum_k A[m][k] B[n][k] on v_mfma_f32_32x32x16_bf16 (both operands K-contiguous).
// (64 WM) x 128 block tile, 2 WM waves of 64 x 64 (2 x 2 MFMA tiles of 32 x 32): WM = 2 for most
// products, WM = 4 for large ones, whose blocks then read a quarter less from L2 per multiply-add.  Four
// waves per SIMD either way: the K loop is bound by the latency of its loads (4096 x 10000 x 512: 92 us
// with 256 x 128 tiles by four waves of 128 x 64, two per SIMD, 80 with eight waves; 32 of them are the
// output's stores).  K step 32 staged in
// LDS as [row][k] (row stride 40 halves = 80 bytes, so every 8-element run is 16-byte aligned).
// Two LDS buffers: the next K step's global loads are issued into registers before the MFMAs of
// the current one and written to the other buffer after them, one barrier per K step.  An
// operand stored K-major (A(m, k) = A[k][m]) is first transposed into the workspace by
// k_transpose_bf16, so that every product runs this one layout with 16-byte loads and stores.
// ---------------------------------------------------------------------------------------
constexpr int GBM = 128, GBN = 128, GBK = 32, GLDS = GBK + 8;

// Eight elements from any address: a 16-byte load needs no alignment here.  (Operands whose rows are no multiple
// of 16 bytes were staged an element at a time: the backward pass of 12-500-500-2500 with 1,024 samples 432 ->
// 138 us, of 12-512-512-2512 108.)
__device__ __forceinline__ bf16x8 load8(const __bf16 *p) {
  typedef bf16x8 any_address __attribute__((aligned(2)));
  return *reinterpret_cast<const any_address *>(p);
}
// The first n of them (all from 8 on, none up to 0), zeros after.
__device__ __forceinline__ bf16x8 load8_part(const __bf16 *p, int n) {
  if (n >= 8) return load8(p);
  bf16x8 v;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = i < n ? p[i] : (__bf16)0.0f;
  return v;
}

// One thread's share of a (rows) x GBK operand tile: RUNS = rows GBK / (256 8) runs of 8 elements.
template <int RUNS>
struct TileRegs {
  bf16x8 v[RUNS];
};

// rows x K row-major: run idx takes row idx / (GBK / 8), k run idx mod (GBK / 8).  Whole steps of a
// 16-byte aligned operand load without a branch (rows past the end read the last row: what they
// produce is not stored); a branch per run had made each load wait for the one before it.
template <int THREADS, int RUNS>
__device__ __forceinline__ void load_regs(TileRegs<RUNS> &t, const __bf16 *__restrict__ src, int ld, int rows, int K,
                                          int r0, int k0, bool vec_ok) {
  if (vec_ok && k0 + GBK <= K) {
#pragma unroll
    for (int it = 0; it < RUNS; ++it) {
      const int idx = threadIdx.x + THREADS * it;
      const int gr = min(r0 + idx / (GBK / 8), rows - 1), gk = k0 + (idx % (GBK / 8)) * 8;
      t.v[it] = *reinterpret_cast<const bf16x8 *>(src + (size_t)gr * ld + gk);
    }
    return;
  }
#pragma unroll
  for (int it = 0; it < RUNS; ++it) {
    const int idx = threadIdx.x + THREADS * it;
    const int gr = min(r0 + idx / (GBK / 8), rows - 1), gk = k0 + (idx % (GBK / 8)) * 8;
    t.v[it] = load8_part(src + (size_t)gr * ld + gk, K - gk);
  }
}

// A whole step, or (PART) the last, from any address.
template <int THREADS, bool PART, int RUNS>
__device__ __forceinline__ void load_step(TileRegs<RUNS> &t, const __bf16 *__restrict__ src, int ld, int rows, int K,
                                          int r0, int k0) {
#pragma unroll
  for (int it = 0; it < RUNS; ++it) {
    const int idx = threadIdx.x + THREADS * it;
    const int gr = min(r0 + idx / (GBK / 8), rows - 1), gk = k0 + (idx % (GBK / 8)) * 8;
    const __bf16 *p = src + (size_t)gr * ld + gk;
    t.v[it] = PART ? load8_part(p, K - gk) : load8(p);
  }
}

template <int THREADS, int RUNS>
__device__ __forceinline__ void store_lds(__bf16 *lds, const TileRegs<RUNS> &t) {
#pragma unroll
  for (int it = 0; it < RUNS; ++it) {
    const int idx = threadIdx.x + THREADS * it;
    *reinterpret_cast<bf16x8 *>(lds + (idx / (GBK / 8)) * GLDS + (idx % (GBK / 8)) * 8) = t.v[it];
  }
}

// dst[c][r] = src[r][c] for r < rows, c < cols (64 x 64 tiles through LDS, padded rows so that
// the column reads hit distinct banks).
__global__ void __launch_bounds__(256) k_transpose_bf16(const __bf16 *__restrict__ src, int lds_, int rows, int cols,
                                                        __bf16 *__restrict__ dst, int ldd) {
  __shared__ uint16_t tile[64][66];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const uint16_t *s16 = reinterpret_cast<const uint16_t *>(src);
  uint16_t *d16 = reinterpret_cast<uint16_t *>(dst);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = r0 + ty + 4 * i, c = c0 + tx;
    tile[ty + 4 * i][tx] = (r < rows && c < cols) ? s16[(size_t)r * lds_ + c] : (uint16_t)0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = c0 + ty + 4 * i, r = r0 + tx;
    if (c < cols && r < rows) d16[(size_t)c * ldd + r] = tile[tx][ty + 4 * i];
  }
}

// Row index of batch sample k: rows[k] when a row vector is given (one outside [0, n_total) is
// taken as row 0 and flagged in *status), else k.
__device__ __forceinline__ int64_t batch_row(const int32_t *__restrict__ rows, int64_t k, int64_t n_total,
                                             uint32_t *status) {
  if (!rows) return k;
  const int32_t r = rows[k];
  if (r < 0 || (int64_t)r >= n_total) {
    atomicOr(status, STATUS_BAD_ROW);
    return 0;
  }
  return r;
}

template <int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &g, int row, int col, float v) {
  if (EPI == EPI_STORE) {
    g.C[(size_t)row * g.ldc + col] = v;
  } else if (EPI == EPI_BIAS) {
    g.C[(size_t)row * g.ldc + col] = v + g.bias[col];
  } else if (EPI == EPI_BIAS_GELU) {
    v += g.bias[col];
    if (g.C) g.C[(size_t)row * g.ldc + col] = v;
    g.Cb[(size_t)row * g.ldcb + col] = (__bf16)gelu_f(v);
  } else {  // EPI_GELU_GRAD: dz_prev = bf16(dx * GELU'(z_prev))
    g.Cb[(size_t)row * g.ldcb + col] = (__bf16)(v * gelu_grad_f(g.Z[(size_t)row * g.ldz + col]));
  }
}

// Tile (x, y, z) of a product's nx x ny tiles and nz K ranges for block `id`.  Blocks go to the eight
// XCDs in turn, each with an L2 of its own, so the id's low three bits pick what one XCD keeps to
// itself: every eighth K range when there are at least eight (an XCD then reads its ranges' operands once),
// else every eighth tile row or column, whichever there are more of (an XCD reads its rows of that
// operand once and shares the other).  The grid is padded to whole turns; a tile outside is left out.
// The ranges past the last eight are shared out by tiles, from three blocks per CU on: of nine ranges one
// XCD had twice the others' work (64 x 8000 x 2304 20.9 -> 17.2 us, x 10000 51 -> 39), while fewer blocks all
// run at once either way (512 x 512 x 2304 14.1 us, shared out 14.9).
struct TileId {
  int x, y, z;
  bool inside;
};
__host__ __device__ inline bool xcd_share_rest(int tiles) { return tiles >= 768; }
__host__ __device__ inline unsigned xcd_blocks(int nx, int ny, int nz) {
  if (nz >= 8) return (unsigned)(xcd_share_rest(nx * ny * nz) ? nz / 8 * 8 * nx * ny + (nz % 8 * nx * ny + 7) / 8 * 8 : (nz + 7) / 8 * 8 * nx * ny);
  return (unsigned)((nx > ny ? (nx + 7) / 8 * 8 * ny : (ny + 7) / 8 * 8 * nx) * nz);
}
__device__ __forceinline__ TileId xcd_tile(unsigned id, int nx, int ny, int nz) {
  const int xcd = (int)(id & 7u);
  int j = (int)(id >> 3);
  TileId t;
  if (nz >= 8) {
    const int n = nx * ny, whole = nz / 8 * n, rest = nz % 8 * n;
    int i = j;
    t.z = j / n * 8 + xcd;
    if (j >= whole && xcd_share_rest(n * nz)) {
      i = rest / 8 * xcd + min(xcd, rest % 8) + j - whole;
      t.z = j - whole < rest / 8 + (xcd < rest % 8 ? 1 : 0) ? nz / 8 * 8 + i / n : nz;
    }
    t.x = i % n % nx;
    t.y = i % n / nx;
  } else {
    const int per = xcd_blocks(nx, ny, 1) / 8;
    t.z = j / per;
    j -= t.z * per;
    if (nx > ny) {
      const int nxl = (nx + 7) / 8;
      t.x = j % nxl * 8 + xcd;
      t.y = j / nxl;
    } else {
      t.x = j % nx;
      t.y = j / nx * 8 + xcd;
    }
  }
  t.inside = t.x < nx && t.y < ny && t.z < nz;
  return t;
}

// The same for four consecutive columns (col a multiple of 4, 16-byte aligned rows).
template <int EPI>
__device__ __forceinline__ void gemm_epilogue4(const GemmArgs &g, int row, int col, float4 v) {
  float *c = g.C + (size_t)row * g.ldc + col;
  if (EPI == EPI_STORE) {
    *reinterpret_cast<float4 *>(c) = v;
  } else {
    const float4 b = *reinterpret_cast<const float4 *>(g.bias + col);
    v.x += b.x;
    v.y += b.y;
    v.z += b.z;
    v.w += b.w;
    if (EPI != EPI_BIAS_GELU || g.C) *reinterpret_cast<float4 *>(c) = v;
    if (EPI == EPI_BIAS_GELU) {
      bf16x4 o;
      o[0] = (__bf16)gelu_f(v.x);
      o[1] = (__bf16)gelu_f(v.y);
      o[2] = (__bf16)gelu_f(v.z);
      o[3] = (__bf16)gelu_f(v.w);
      *reinterpret_cast<bf16x4 *>(g.Cb + (size_t)row * g.ldcb + col) = o;
    }
  }
}

// EPI_BIAS_MSE: the prediction y = v + bias is compared with the targets at once and never stored: dy
// = 2 (y - t) scale in BF16 (unless Cb is NULL); returns (y - t)^2 in FP64.
__device__ __forceinline__ double mse_epilogue(const GemmArgs &g, int row, int col, float v) {
  const float d = (v + g.bias[col]) - g.T[(size_t)batch_row(g.rows, row, g.n_total, g.status) * g.N + col];
  if (g.Cb) g.Cb[(size_t)row * g.ldcb + col] = (__bf16)(g.gscale * d);
  return (double)d * (double)d;
}
__device__ __forceinline__ double mse_epilogue4(const GemmArgs &g, int row, int col, float4 v) {
  const float4 b = *reinterpret_cast<const float4 *>(g.bias + col);
  const float4 t = *reinterpret_cast<const float4 *>(g.T + (size_t)batch_row(g.rows, row, g.n_total, g.status) * g.N + col);
  const float d0 = (v.x + b.x) - t.x, d1 = (v.y + b.y) - t.y, d2 = (v.z + b.z) - t.z, d3 = (v.w + b.w) - t.w;
  if (g.Cb) {
    bf16x4 o;
    o[0] = (__bf16)(g.gscale * d0);
    o[1] = (__bf16)(g.gscale * d1);
    o[2] = (__bf16)(g.gscale * d2);
    o[3] = (__bf16)(g.gscale * d3);
    *reinterpret_cast<bf16x4 *>(g.Cb + (size_t)row * g.ldcb + col) = o;
  }
  return ((double)d0 * (double)d0 + (double)d1 * (double)d1) + ((double)d2 * (double)d2 + (double)d3 * (double)d3);
}
// A wave's sum of squared errors to its slot of lpart (tile-major, `slots` waves per tile).
constexpr int LOSS_WAVES = 4;
__device__ __forceinline__ void store_loss_part(const GemmArgs &g, double s, int tile, int slots, int wave) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  if ((threadIdx.x & 63u) == 0u) g.lpart[(size_t)tile * slots + wave] = s;
}

constexpr int GEPI_LD = 72;  // epilogue slab row stride (floats): 32 x 72 x 4 B per wave

// WM x 2 waves of 64 x 64 (64 VGPRs of accumulators, four waves per SIMD).
//
// STEPS: the K loop has whole steps alone, and the last one's partial loads follow it.  As a branch in the
// loop they make the compiler wait for A's loads before it issues B's (1024 x 8192 x 4096: 114 us, 94
// without).
template <int EPI, int WM, bool STEPS>
__global__ void __launch_bounds__(128 * WM) __attribute__((amdgpu_waves_per_eu(4, 8))) k_gemm(GemmArgs g) {
  constexpr int MI = 2, BM = 64 * WM, TH = 128 * WM;  // block tile rows, threads
  constexpr int RA = BM * GBK / (TH * 8), RB = GBN * GBK / (TH * 8);
  // the two A and two B tiles, and after the loop the epilogue slabs
  constexpr int TILES = 2 * (BM + GBN) * GLDS, SLABS = 2 * WM * 32 * GEPI_LD * 2;
  __shared__ __attribute__((aligned(16))) __bf16 smem[TILES > SLABS ? TILES : SLABS];
  __bf16 (*As)[BM * GLDS] = reinterpret_cast<__bf16 (*)[BM * GLDS]>(smem);
  __bf16 (*Bs)[GBN * GLDS] = reinterpret_cast<__bf16 (*)[GBN * GLDS]>(smem + 2 * BM * GLDS);
  const int nx = (g.N + GBN - 1) / GBN, ny = (g.M + BM - 1) / BM;
  TileId tl;
  if (g.nz > 1) {  // K ranges over blocks, each into its part of the workspace (EPI_STORE)
    const int xy = (int)blockIdx.x % (nx * ny), z = (int)blockIdx.x / (nx * ny), kb = z * g.kchunk;
    tl = TileId{xy % nx, xy / nx, z, true};
    g.A += kb;
    g.B += kb;
    g.K = min(g.K - kb, g.kchunk);
    g.C = g.part + (size_t)z * g.M * g.N;
    g.ldc = g.N;
  } else {
    tl = xcd_tile(blockIdx.x, nx, ny, 1);
  }
  if (!tl.inside) return;
  const int bm = tl.y * BM, bn = tl.x * GBN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = (wave >> 1) * 32 * MI, wn = (wave & 1) * 64;
  const bool va = (g.lda % 8 == 0) && (((uintptr_t)g.A & 15) == 0);
  const bool vb = (g.ldb % 8 == 0) && (((uintptr_t)g.B & 15) == 0);
  f32x16 acc[MI][2];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;
  const int r = lane & 31, kh = (lane >> 5) * 8;
  TileRegs<RA> ra;
  TileRegs<RB> rb;
  auto load = [&](int k0) {
    load_regs<TH>(ra, g.A, g.lda, g.M, g.K, bm, k0, va);
    load_regs<TH>(rb, g.B, g.ldb, g.N, g.K, bn, k0, vb);
  };
  auto load_one = [&](int k0, auto part) {
    load_step<TH, decltype(part)::value>(ra, g.A, g.lda, g.M, g.K, bm, k0);
    load_step<TH, decltype(part)::value>(rb, g.B, g.ldb, g.N, g.K, bn, k0);
  };
  auto store = [&](int buf) {
    store_lds<TH>(As[buf], ra);
    store_lds<TH>(Bs[buf], rb);
  };
  auto multiply = [&](int buf) {
    const __bf16 *as = As[buf];
    const __bf16 *bs = Bs[buf];
#pragma unroll
    for (int ks = 0; ks < GBK; ks += 16) {
      bf16x8 a[MI], b[2];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) a[mi] = *reinterpret_cast<const bf16x8 *>(&as[(wm + mi * 32 + r) * GLDS + ks + kh]);
#pragma unroll
      for (int ni = 0; ni < 2; ++ni) b[ni] = *reinterpret_cast<const bf16x8 *>(&bs[(wn + ni * 32 + r) * GLDS + ks + kh]);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b[ni], acc[mi][ni], 0, 0, 0);
    }
  };
  if constexpr (STEPS) {
    constexpr std::integral_constant<bool, false> whole{};
    constexpr std::integral_constant<bool, true> part{};
    const int steps = g.K / GBK;
    if (steps > 0)
      load_one(0, whole);
    else
      load_one(0, part);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int kt = 1; kt < steps; ++kt, cur ^= 1) {
      load_one(kt * GBK, whole);
      __builtin_amdgcn_sched_barrier(0);  // issued before the products, not among them
      multiply(cur);
      store(cur ^ 1);
      __syncthreads();
    }
    if (steps > 0 && g.K % GBK != 0) {
      load_one(steps * GBK, part);
      multiply(cur);
      cur ^= 1;
      store(cur);
      __syncthreads();
    }
    multiply(cur);
    __syncthreads();
  } else {
    const int nk = (g.K + GBK - 1) / GBK;
    load(0);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      const bool more = kt + 1 < nk;
      if (more) load((kt + 1) * GBK);
      multiply(kt & 1);
      if (more) store((kt & 1) ^ 1);
      __syncthreads();
    }
  }
  // Epilogue through LDS (the A/B buffers are free after the last barrier): accumulator element e
  // of a 32 x 32 tile sits at row 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32, so a lane
  // holds no two neighbours of a row.  Each wave writes its 64 x 64 sub-tile in two parts of 32
  // rows into its own LDS slab (row stride GEPI_LD floats: the two half-waves of one store land
  // in different banks), then reads them back four consecutive columns per lane and writes 16
  // bytes per lane (C) or 8 bytes (BF16 outputs).
  float *slab = reinterpret_cast<float *>(smem) + wave * (32 * GEPI_LD);
  const bool v4 = EPI == EPI_BIAS_MSE
                      ? g.N % 4 == 0 && g.ldcb % 4 == 0 && ((((uintptr_t)g.bias) | ((uintptr_t)g.T)) & 15) == 0 &&
                            ((uintptr_t)g.Cb & 7) == 0
                      : EPI != EPI_GELU_GRAD && g.ldc % 4 == 0 && ((uintptr_t)g.C & 15) == 0 &&
                            (EPI == EPI_STORE || ((uintptr_t)g.bias & 15) == 0) &&
                            (EPI != EPI_BIAS_GELU || (g.ldcb % 4 == 0 && ((uintptr_t)g.Cb & 7) == 0));
  double loss = 0.0;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        slab[(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * GEPI_LD + ni * 32 + (lane & 31)] = acc[mi][ni][e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // 32 rows x 16 runs of 4 columns = 512 runs, 8 per lane; 16 lanes cover one row
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      const int idx = it * 64 + lane;
      const int rr = idx >> 4, c4 = (idx & 15) * 4;
      const int row = bm + wm + mi * 32 + rr, col = bn + wn + c4;
      if (row >= g.M) continue;
      const float4 v = *reinterpret_cast<const float4 *>(&slab[rr * GEPI_LD + c4]);
      if (v4 && col + 4 <= g.N) {
        if constexpr (EPI == EPI_BIAS_MSE)
          loss += mse_epilogue4(g, row, col, v);
        else
          gemm_epilogue4<EPI>(g, row, col, v);
      } else {
        const float vv[4] = {v.x, v.y, v.z, v.w};
        for (int q = 0; q < 4; ++q) {
          if (col + q >= g.N) break;
          if constexpr (EPI == EPI_BIAS_MSE)
            loss += mse_epilogue(g, row, col + q, vv[q]);
          else
            gemm_epilogue<EPI>(g, row, col + q, vv[q]);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if constexpr (EPI == EPI_BIAS_MSE) store_loss_part(g, loss, tl.y * nx + tl.x, 2 * WM, wave);
}

// Sum of the split-K partial products in split order, then the epilogue.
template <int EPI>
__global__ void __launch_bounds__(256) k_gemm_splitk_reduce(GemmArgs g, int splits) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t mn = (int64_t)g.M * g.N;
  if (idx >= mn) return;
  float v = 0.0f;
  for (int z = 0; z < splits; ++z) v += g.part[(size_t)z * mn + idx];
  gemm_epilogue<EPI>(g, (int)(idx / g.N), (int)(idx % g.N), v);
}

// ---------------------------------------------------------------------------------------
// The same product in 64 x 64 tiles, for products whose 128 x 128 tiles would leave most of the chip
// idle (every hidden layer's).  Such a product is bound by latency: a block of G groups of 256 threads
// (4 waves of one 32 x 32 MFMA tile each) reads 128 K elements per operand row and stage, the next
// stage's loads in flight during the products.  Group g takes the K range [g kchunk, (g + 1) kchunk)
// of a split product and group 0 adds the groups' sums in order, the sums and order of
// k_gemm + k_gemm_splitk_reduce without their launch and trip through memory.  More ranges than 4 go
// to further blocks and the workspace.  TA / TB: that operand is stored K-major (A(m, k) =
// A[k][m]) and transposed on its way into LDS: a thread reads an 8 x 8 block in eight 16-byte rows and
// permutes it in registers, where a transpose launch had copied the operand first.  AF32: A is the
// FP32 input batch (rows of it by the row vector), rounded on the way.
// Measured, products and what went with them (split sums, transposes, rounding of the input): one
// sample through 12-512-512-512-512-10000 65 -> 30 us, 4,096 samples' hidden layers 90 -> 50 us; all
// results the same bit for bit.
// ---------------------------------------------------------------------------------------
constexpr int HB = 64, HK = 128, HLD = HK + 8;  // tile, K stage, LDS row stride (rows 4 banks apart)
// Element (row, 8 unit) of a staged tile.  The units of a row are permuted by its number over 8, so that
// a transposed 8 x 8 block's stores (eight lanes, rows 8 apart: 32 banks or none) fall in different
// banks, as the row-wise stores and the fragment reads do.
__device__ __forceinline__ int lds64(int row, int unit) { return row * HLD + (unit ^ ((row >> 3) & 7)) * 8; }

union Run8 {
  bf16x8 v;
  uint32_t w[4];
};

// A whole stage of an operand goes through registers.  Rows past the end keep what the
// registers hold (what they produce is not stored): a value given to them made every load wait for
// the one before it, and reading the last row instead (64 times, for one sample, by every block)
// crowded one L2 channel.
// So does a last stage of whole steps of 16 (a layer of 64 or 96: one element at a time its staging took
// 2 us a product): in place of a run from ke on the last one is loaded, and nothing reads it in LDS.
__device__ __forceinline__ bool whole_steps64(int k0, int ke) { return k0 < ke && (k0 + HK <= ke || (ke - k0) % 16 == 0); }
// Row-major: 4 runs of 8 k; thread t's run i is row (t + 256 i) / 16.
__device__ __forceinline__ void load_rows64(Run8 (&x)[4], const __bf16 *__restrict__ src, int ld, int rows, int r0, int k0,
                                            int ke, int t) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = t + 256 * i;
    const int r = r0 + (idx >> 4), k = min(k0 + (t & 15) * 8, ke - 8);
    if (r < rows) x[i].v = load8(src + (size_t)r * ld + k);
  }
}
__device__ __forceinline__ void store_rows64(__bf16 *lds, const Run8 (&x)[4], int t) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int idx = t + 256 * i;
    *reinterpret_cast<bf16x8 *>(lds + lds64(idx >> 4, idx & 15)) = x[i].v;
  }
}
// Any other last stage, zeros from ke on.
__device__ __forceinline__ void stage_rows64(__bf16 *lds, const __bf16 *__restrict__ src, int ld, int rows, int r0, int k0,
                                             int ke, int t) {
#pragma unroll 1
  for (int idx = t; idx < 64 * 16; idx += 256) {
    const int r = r0 + (idx >> 4), k = k0 + (idx & 15) * 8;
    if (r >= rows || k >= ke + 8) continue;
    *reinterpret_cast<bf16x8 *>(lds + lds64(idx >> 4, idx & 15)) = load8_part(src + (size_t)r * ld + k, ke - k);
  }
}
// K-major: block b holds k 8 (b / 8) .. + 7 and rows 8 (b % 8) .. + 7 of the tile's, the last rows again where
// there are not as many (cols64_row: the first of them; a tile has eight or more).
__device__ __forceinline__ int cols64_row(int rows, int r0, int b) { return min((b & 7) * 8, rows - r0 - 8); }
__device__ __forceinline__ void load_cols64(Run8 (&x)[8], const __bf16 *__restrict__ src, int ld, int rows, int r0, int k0,
                                            int ke, int b) {
  const int k = min(k0 + (b >> 3) * 8, ke - 8);
  const __bf16 *p = src + (size_t)k * ld + r0 + cols64_row(rows, r0, b);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i].v = load8(p + (size_t)i * ld);
}
__device__ __forceinline__ void store_cols64(__bf16 *lds, const Run8 (&x)[8], int row, int unit) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    Run8 o;  // row m of the block: its k pairs from the k-th and (k + 1)-th words
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o.w[j] = __builtin_amdgcn_perm(x[2 * j + 1].w[m >> 1], x[2 * j].w[m >> 1], (m & 1) ? 0x07060302u : 0x05040100u);
    *reinterpret_cast<bf16x8 *>(lds + lds64(row + m, unit)) = o.v;
  }
}
// Any other stage: the last, or of a tile of fewer than eight rows; zeros from ke on.
__device__ __forceinline__ void stage_cols64(__bf16 *lds, Run8 (&x)[8], const __bf16 *__restrict__ src, int ld, int rows,
                                             int r0, int k0, int ke, int b) {
  const int k = k0 + (b >> 3) * 8;
  if (k >= ke + 8) return;
  const int row = max(cols64_row(rows, r0, b), 0);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i].v = load8_part(src + (size_t)min(k + i, ke - 1) * ld + r0 + row, k + i < ke ? rows - r0 - row : 0);
  store_cols64(lds, x, row, b >> 3);
}
// The FP32 input batch, rounded, one element at a time straight into LDS: k0 .. ke - 1 (at most HK), zeros up to
// the next multiple of 16.
__device__ __forceinline__ void stage_f32_64(__bf16 *lds, const GemmArgs &g, int ke, int r0, int k0, int t, bool first_column) {
  const int steps = (max(0, min(HK, ke - k0)) + 15) / 16;
  const int n = max(1, min(HB, g.M - r0));
  const int lg = n > 1 ? 32 - __builtin_clz((unsigned)(n - 1)) : 0;  // 2^lg >= n rows
  for (int idx = t; idx < steps << (4 + lg); idx += 256) {
    // neighbouring threads read neighbouring elements
    const int rr = (idx >> 4) & ((1 << lg) - 1), kk = (idx & 15) + (idx >> (4 + lg)) * 16;
    const int r = r0 + rr, k = k0 + kk;
    __bf16 v = (__bf16)0.0f;
    if (r < g.M && k < ke) {
      v = (__bf16)g.A32[batch_row(g.rows, r, g.n_total, g.status) * g.lda + k];
      if (g.Aout && first_column) g.Aout[(size_t)r * g.lda + k] = v;
    }
    lds[lds64(rr, kk >> 3) + (kk & 7)] = v;
  }
}

template <int EPI, int G, bool TA, bool TB, bool AF32>
__device__ __forceinline__ void gemm64_block(const GemmArgs &g, unsigned block, char *smem64) {
  const int grp = threadIdx.x >> 8, t = threadIdx.x & 255;
  __bf16 *As = reinterpret_cast<__bf16 *>(smem64) + (size_t)grp * 2 * HB * HLD, *Bs = As + HB * HLD;
  const int nx = (g.N + HB - 1) / HB;
  const TileId tl = xcd_tile(block, nx, (g.M + HB - 1) / HB, g.nz);
  if (!tl.inside) return;
  const int bm = tl.y * HB, bn = tl.x * HB;
  const int wave = t >> 6, lane = t & 63;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  // operands whose whole stages go through registers
  const bool va = !AF32 && (!TA || g.M - bm >= 8), vb = !TB || g.N - bn >= 8;
  const int chunk = G > 1 ? grp : tl.z;
  const int kb = chunk * g.kchunk, ke = min(g.K, kb + g.kchunk);
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
  const int r = lane & 31, kh = (lane >> 5) * 8;
  // every group runs the stages of the longest range (group 0's): the barriers are the block's
  const int stages = (min(g.K, g.kchunk) + HK - 1) / HK;
  // K-major operands: the first 128 threads hold A's blocks, the others B's, where both are; else
  // the first 128 threads
  constexpr bool BOTH = TA && TB;
  const int cb = BOTH ? t & 127 : t;
  const bool has_a = TA && (BOTH ? t < 128 : t < 128), has_b = TB && (BOTH ? t >= 128 : t < 128);
  Run8 ra[4] = {}, rb[4] = {}, rc[8] = {};
  auto load = [&](int k0) {
    if (!whole_steps64(k0, ke)) return;
    if (va) {
      if constexpr (!TA) load_rows64(ra, g.A, g.lda, g.M, bm, k0, ke, t);
      if constexpr (TA)
        if (has_a) load_cols64(rc, g.A, g.lda, g.M, bm, k0, ke, cb);
    }
    if (vb) {
      if constexpr (!TB) load_rows64(rb, g.B, g.ldb, g.N, bn, k0, ke, t);
      if constexpr (TB)
        if (has_b) load_cols64(rc, g.B, g.ldb, g.N, bn, k0, ke, cb);
    }
  };
  load(kb);
  for (int st = 0; st < stages; ++st) {
    const int k0 = kb + st * HK;
    const bool whole = whole_steps64(k0, ke);
    if (st > 0) __syncthreads();  // the previous stage's reads are over
    if constexpr (AF32) {
      stage_f32_64(As, g, ke, bm, k0, t, tl.x == 0);
    } else if constexpr (TA) {
      if (has_a && whole && va)
        store_cols64(As, rc, cols64_row(g.M, bm, cb), cb >> 3);
      else if (has_a)
        stage_cols64(As, rc, g.A, g.lda, g.M, bm, k0, ke, cb);
    } else {
      if (whole)
        store_rows64(As, ra, t);
      else
        stage_rows64(As, g.A, g.lda, g.M, bm, k0, ke, t);
    }
    if constexpr (TB) {
      if (has_b && whole && vb)
        store_cols64(Bs, rc, cols64_row(g.N, bn, cb), cb >> 3);
      else if (has_b)
        stage_cols64(Bs, rc, g.B, g.ldb, g.N, bn, k0, ke, cb);
    } else {
      if (whole)
        store_rows64(Bs, rb, t);
      else
        stage_rows64(Bs, g.B, g.ldb, g.N, bn, k0, ke, t);
    }
    __syncthreads();
    if (st + 1 < stages) load(k0 + HK);
    // whole steps of 16 up to the range's end (what lies past it in the stage is zero)
#pragma unroll
    for (int ks = 0; ks < HK; ks += 16) {
      if (k0 + ks >= ke) break;
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&As[lds64(wm + r, (ks + kh) / 8)]);
      const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&Bs[lds64(wn + r, (ks + kh) / 8)]);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
  }
  // With groups, every group leaves its sums in LDS and finishes a G-th of the tile's elements: adds
  // the groups' sums in group order and runs the epilogue (GELU and its derivative are ~100
  // instructions an element, which one group's four waves alone took 5 us for).
  constexpr int EN = 16 / G;
  float *sums = reinterpret_cast<float *>(smem64);  // [G][16][256]
  if (G > 1) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) sums[(grp * 16 + e) * 256 + t] = acc[e];
    __syncthreads();
  }
  // accumulator element e: row 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32
  float *part = g.part ? g.part + (size_t)tl.z * g.M * g.N : nullptr;
  const int col = bn + wn + (lane & 31);
  double loss = 0.0;
#pragma unroll
  for (int i = 0; i < EN; ++i) {
    const int e = G > 1 ? grp * EN + i : i;
    float v;
    if constexpr (G > 1) {
      v = sums[e * 256 + t];
#pragma unroll
      for (int q = 1; q < G; ++q) v += sums[(q * 16 + e) * 256 + t];
    } else {
      v = acc[i];
    }
    const int row = bm + wm + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    if (row >= g.M || col >= g.N) continue;
    if constexpr (EPI == EPI_BIAS_MSE) {
      loss += mse_epilogue(g, row, col, v);
    } else {
      if (part)
        part[(size_t)row * g.N + col] = v;
      else
        gemm_epilogue<EPI>(g, row, col, v);
    }
  }
  if constexpr (EPI == EPI_BIAS_MSE) store_loss_part(g, loss, tl.y * nx + tl.x, G * LOSS_WAVES, grp * LOSS_WAVES + wave);
}

template <int EPI, int G, bool TA, bool TB, bool AF32>
__global__ void __launch_bounds__(256 * G) k_gemm64(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) char smem64[];
  gemm64_block<EPI, G, TA, TB, AF32>(g, blockIdx.x, smem64);
}

// db[m] = sum_n dz[n][m] in FP32.  A block takes 64 columns (one per lane, so every row read is
// 128 contiguous bytes) and COLSUM_WAVES waves split the rows: wave w sums rows w, w + COLSUM_WAVES, ...
// in order, and the partial sums are added in wave order.  The order is fixed by n alone, so results do
// not depend on the launch: W waves take COLSUM_WAVES / W of those sums each.
constexpr int COLSUM_WAVES = 16;
template <int W>
__device__ __forceinline__ void colsum_block(const ColsumArgs &a, unsigned block, char *smem) {
  float(*part)[64] = reinterpret_cast<float(*)[64]>(smem);
  constexpr int PER = COLSUM_WAVES / W;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = block * 64 + lane;
  float s[PER] = {};
  if (c < a.m) {
    int r = w;
#pragma unroll 8
    for (; r + (PER - 1) * W < a.n; r += COLSUM_WAVES)
#pragma unroll
      for (int k = 0; k < PER; ++k) s[k] += (float)a.dz[(size_t)(r + k * W) * a.m + c];
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (r + k * W < a.n) s[k] += (float)a.dz[(size_t)(r + k * W) * a.m + c];
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) part[w + k * W][lane] = s[k];
  __syncthreads();
  if (w == 0 && c < a.m) {
    float t = part[0][lane];
#pragma unroll
    for (int k = 1; k < COLSUM_WAVES; ++k) t += part[k][lane];
    a.db[c] = t;
  }
}

__global__ void __launch_bounds__(64 * COLSUM_WAVES) k_colsum(ColsumArgs a) {
  __shared__ float part[COLSUM_WAVES][64];
  colsum_block<COLSUM_WAVES>(a, blockIdx.x, reinterpret_cast<char *>(part));
}

// A layer's backward products in one launch: the bias gradients (blocks [0, nbc)), dx = dz W (the next nbx)
// and dW = dz^T x.  They read the same dz and nothing of each other, and each alone leaves most of
// the chip idle (512 wide, 1,024 samples: 128 blocks, 64 and 8: 26 -> 12 us; the
// 10,000-bin output layer 65 -> 61 us).
template <int GW, int GX>
__global__ void __launch_bounds__(256 * (GW > GX ? GW : GX))
k_gemm64_back(GemmArgs w, GemmArgs x, ColsumArgs c, unsigned nbc, unsigned nbx) {
  extern __shared__ __attribute__((aligned(16))) char smem64[];
  const unsigned id = blockIdx.x;
  // whole waves leave a product with fewer groups (a barrier waits for the waves that are left)
  const unsigned thread0 = (unsigned)__builtin_amdgcn_readfirstlane((int)threadIdx.x);
  if (id < nbc) {
    if (id * 64u < (unsigned)c.m) colsum_block<4 * (GW > GX ? GW : GX)>(c, id, smem64);
  } else if (id < nbc + nbx) {
    if (thread0 < 256 * GX) gemm64_block<EPI_GELU_GRAD, GX, false, false, false>(x, id - nbc, smem64);
  } else {
    if (thread0 < 256 * GW) gemm64_block<EPI_STORE, GW, true, true, false>(w, id - nbc - nbx, smem64);
  }
}

// Split over K when the output tile grid cannot fill the chip and K is long enough: about two
// blocks per CU, at least 256 K elements per split.
static int gemm_splits(int M, int N, int K, int &kchunk) {
  const int blocks = ((M + GBM - 1) / GBM) * ((N + GBN - 1) / GBN);
  kchunk = K;
  if (blocks >= 128 || K < 512) return 1;
  int splits = min((512 + blocks - 1) / blocks, K / 256);
  if (splits < 2) return 1;
  kchunk = ((K + splits - 1) / splits + GBK - 1) / GBK * GBK;
  return (K + kchunk - 1) / kchunk;
}

// 256-row block tiles where the product is large enough to keep every CU busy with them.
static bool gemm_tall(int M, int N) { return M >= 4096 && N >= 2048; }
// Whether a product takes 64 x 64 tiles: its 128 x 128 tiles would not give every CU two blocks.
static bool gemm_use64(int M, int N) { return (int64_t)((M + GBM - 1) / GBM) * ((N + GBN - 1) / GBN) < 512; }

// Workspace layout: [A transposed: M x ldk bf16][B transposed: N x ldk bf16][split-K partials:
// splits x M x N FP32], each part 256-byte aligned and present only when needed (the 64 x 64 tiles
// read K-major operands as they are and add up to four splits inside a block).
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static int transposed_ld(int K) { return (K + 7) & ~7; }  // keeps the 16-byte loads of k_gemm
constexpr int G64_SPLITS = 4;

size_t gemm_workspace_bytes(int M, int N, int K, bool at, bool bt) {
  int kchunk;
  const int splits = gemm_splits(M, N, K, kchunk);
  const bool t64 = gemm_use64(M, N);
  const size_t lk = (size_t)transposed_ld(K);
  size_t b = 0;
  if (at && !t64) b += align256((size_t)M * lk * 2);
  if (bt && !t64) b += align256((size_t)N * lk * 2);
  if (splits > (t64 ? G64_SPLITS : 1)) b += (size_t)splits * M * N * 4;
  return b;
}

static hipError_t launch_transpose(const __bf16 *src, int ld, int rows, int cols, __bf16 *dst, int ldd, hipStream_t s) {
  dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64));
  hipLaunchKernelGGL(k_transpose_bf16, grid, dim3(256), 0, s, src, ld, rows, cols, dst, ldd);
  return hipGetLastError();
}

template <int EPI, bool TA, bool TB, bool AF32>
static hipError_t launch_gemm64_t(GemmArgs g, int splits, void *ws, hipStream_t s) {
  const bool inside = splits <= G64_SPLITS;
  g.part = inside ? nullptr : (float *)ws;
  g.nz = inside ? 1 : splits;
  const dim3 grid(xcd_blocks((g.N + HB - 1) / HB, (g.M + HB - 1) / HB, g.nz));
  constexpr size_t lds = 2 * HB * HLD * sizeof(__bf16);  // one group's tiles
  if (inside && splits > 2)  // a third or fourth range may be empty
    hipLaunchKernelGGL((k_gemm64<EPI, 4, TA, TB, AF32>), grid, dim3(1024), 4 * lds, s, g);
  else if (inside && splits == 2)
    hipLaunchKernelGGL((k_gemm64<EPI, 2, TA, TB, AF32>), grid, dim3(512), 2 * lds, s, g);
  else
    hipLaunchKernelGGL((k_gemm64<EPI, 1, TA, TB, AF32>), grid, dim3(256), lds, s, g);
  if constexpr (EPI == EPI_BIAS_MSE) {
    if (!inside) return hipErrorInvalidValue;  // gemm_loss_parts() == 0
  } else if (!inside) {
    const unsigned rblocks = (unsigned)(((int64_t)g.M * g.N + 255) / 256);
    hipLaunchKernelGGL((k_gemm_splitk_reduce<EPI>), dim3(rblocks), dim3(256), 0, s, g, splits);
  }
  return hipGetLastError();
}

static hipError_t launch_gemm64(const GemmArgs &g, int splits, bool at, bool bt, int epi, void *ws, hipStream_t s) {
  if (g.A32) {
    if (at || bt) return hipErrorInvalidValue;
    if (epi == EPI_BIAS) return launch_gemm64_t<EPI_BIAS, false, false, true>(g, splits, ws, s);
    if (epi == EPI_BIAS_GELU) return launch_gemm64_t<EPI_BIAS_GELU, false, false, true>(g, splits, ws, s);
    return hipErrorInvalidValue;
  }
  if (epi == EPI_STORE) {
    if (at && bt) return launch_gemm64_t<EPI_STORE, true, true, false>(g, splits, ws, s);
    if (at) return launch_gemm64_t<EPI_STORE, true, false, false>(g, splits, ws, s);
    if (bt) return launch_gemm64_t<EPI_STORE, false, true, false>(g, splits, ws, s);
    return launch_gemm64_t<EPI_STORE, false, false, false>(g, splits, ws, s);
  }
  if (at || bt) return hipErrorInvalidValue;  // the network's other products are row-major
  if (epi == EPI_BIAS) return launch_gemm64_t<EPI_BIAS, false, false, false>(g, splits, ws, s);
  if (epi == EPI_BIAS_GELU) return launch_gemm64_t<EPI_BIAS_GELU, false, false, false>(g, splits, ws, s);
  if (epi == EPI_GELU_GRAD) return launch_gemm64_t<EPI_GELU_GRAD, false, false, false>(g, splits, ws, s);
  if (epi == EPI_BIAS_MSE) return launch_gemm64_t<EPI_BIAS_MSE, false, false, false>(g, splits, ws, s);
  return hipErrorInvalidValue;
}

int64_t gemm_loss_parts(int M, int N, int K) {
  int kchunk;
  if (gemm_use64(M, N)) {
    const int splits = gemm_splits(M, N, K, kchunk), groups = splits > 2 ? 4 : splits;
    return splits > G64_SPLITS ? 0 : (int64_t)((M + HB - 1) / HB) * ((N + HB - 1) / HB) * groups * LOSS_WAVES;
  }
  const int wm = gemm_tall(M, N) ? 4 : 2;  // wave rows of k_gemm
  return (int64_t)((M + 64 * wm - 1) / (64 * wm)) * ((N + GBN - 1) / GBN) * 2 * wm;
}

// Every 64-column tile rounds the FP32 rows again, an element at a time, where a pass of its own costs a launch: 64
// rows or more (of each tile) cross between 32 and 48 inputs, 16 rows between 128 and 192, a single
// row not up to 8,192.  Into 512-512: 1,024 rows of 12 inputs 16.6 us against 18.4 rounded first, of 64 18.7
// against 17.0, of 2,048 52 against 36; 16 rows of 128 13.8 against 13.9; one of 2,048 13.9 against 15.2.
bool gemm_reads_f32(int M, int N, int K) {
  return gemm_use64(M, N) && (M == 1 || (int64_t)std::min(M, HB) * K <= 2048);
}

// Row starts that fall on 64 bytes: a step's loads of a row (32 elements) then take one cache line.
static bool gemm_aligned64(const GemmArgs &g) {
  return g.lda % 32 == 0 && g.ldb % 32 == 0 && (((uintptr_t)g.A | (uintptr_t)g.B) & 63) == 0;
}
// Whether an unsplit product takes the loop of whole steps: with two blocks per CU (1024 x 8192 x 4096: 114 -> 94 us);
// of many more, those that run ahead find less in L2 (4096 x 10000 x 512: 72 -> 96 us).
static bool gemm_steps(int M, int N) {
  return !gemm_tall(M, N) && (int64_t)((M + GBM - 1) / GBM) * ((N + GBN - 1) / GBN) <= 512;
}
// Whether a product over K ranges of row-major operands takes 128 x 128 tiles after all: its 64 x 64 tiles
// would not all run at once (four blocks per CU), the larger tiles waste no more of their rows and columns, and
// the ranges are short, so that the larger tiles' fewer operand reads show (1024 x 512 x 2048: 22.5 -> 20 us, x
// 3000 26 -> 21; 512 x 512 x 2048, 512 blocks, 13 and 15; 900 x 1100 x 4096 33 and 36), or long ones and the
// blocks whole turns over the CUs (1024 x 1024 x 16384: 77 -> 63 us, 640 x 640 x 10000, 525 blocks, 32 and 38).
static bool gemm_split128(const GemmArgs &g, int splits, bool at, bool bt) {
  if (splits <= G64_SPLITS || at || bt || g.A32) return false;
  const int64_t b128 = (int64_t)((g.M + GBM - 1) / GBM) * ((g.N + GBN - 1) / GBN) * splits;
  const int64_t b64 = (int64_t)((g.M + HB - 1) / HB) * ((g.N + HB - 1) / HB) * splits;
  const bool turns = (b128 + 255) / 256 * 256 * 100 <= b128 * 106;
  return b64 >= 1024 && 4 * b128 * 100 <= b64 * 106 && (g.K <= 4096 || (turns && gemm_aligned64(g)));
}

static hipError_t launch_split128(GemmArgs g, int splits, int epi, void *ws, hipStream_t s) {
  g.part = (float *)ws;
  g.nz = splits;
  const unsigned blocks = (unsigned)((g.M + GBM - 1) / GBM * ((g.N + GBN - 1) / GBN) * splits);
  const unsigned rblocks = (unsigned)(((int64_t)g.M * g.N + 255) / 256);
  // the loop of whole steps where rows fall on cache lines (1024 x 512 x 3000, which do not: 25.5 us, 21.5 without)
  if (gemm_aligned64(g))
    hipLaunchKernelGGL((k_gemm<EPI_STORE, 2, true>), dim3(blocks), dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((k_gemm<EPI_STORE, 2, false>), dim3(blocks), dim3(256), 0, s, g);
#define PCMD_REDUCE_CASE(E_) \
  if (epi == E_) hipLaunchKernelGGL((k_gemm_splitk_reduce<E_>), dim3(rblocks), dim3(256), 0, s, g, splits);
  PCMD_REDUCE_CASE(EPI_STORE)
  PCMD_REDUCE_CASE(EPI_BIAS)
  PCMD_REDUCE_CASE(EPI_BIAS_GELU)
  PCMD_REDUCE_CASE(EPI_GELU_GRAD)
#undef PCMD_REDUCE_CASE
  return epi == EPI_BIAS_MSE ? hipErrorInvalidValue : hipGetLastError();  // gemm_loss_parts() == 0
}

hipError_t launch_gemm(const GemmArgs &g0, bool at, bool bt, int epi, void *ws, size_t ws_bytes, hipStream_t s) {
  GemmArgs g = g0;
  if (ws_bytes < gemm_workspace_bytes(g.M, g.N, g.K, at, bt)) return hipErrorInvalidValue;
  int kchunk;
  const int splits = gemm_splits(g.M, g.N, g.K, kchunk);
  const bool split = splits > 1;
  g.kchunk = split ? kchunk : g.K;
  if (gemm_split128(g, splits, at, bt)) return launch_split128(g, splits, epi, ws, s);
  if (gemm_use64(g.M, g.N)) return launch_gemm64(g, splits, at, bt, epi, ws, s);
  if (g.A32) return hipErrorInvalidValue;
  char *w = (char *)ws;
  const int lk = transposed_ld(g.K);
  if (at) {  // A(m, k) = A[k][m]: K rows of M
    __bf16 *t = (__bf16 *)w;
    const hipError_t e = launch_transpose(g.A, g.lda, g.K, g.M, t, lk, s);
    if (e != hipSuccess) return e;
    g.A = t;
    g.lda = lk;
    w += align256((size_t)g.M * lk * 2);
  }
  if (bt) {
    __bf16 *t = (__bf16 *)w;
    const hipError_t e = launch_transpose(g.B, g.ldb, g.K, g.N, t, lk, s);
    if (e != hipSuccess) return e;
    g.B = t;
    g.ldb = lk;
    w += align256((size_t)g.N * lk * 2);
  }
  // 512 blocks or more are never split (gemm_splits splits below 128)
  g.part = nullptr;
  g.nz = 1;
  const bool tall = gemm_tall(g.M, g.N), steps = gemm_steps(g.M, g.N);
  const dim3 grid(xcd_blocks((g.N + GBN - 1) / GBN, (g.M + (tall ? 2 * GBM : GBM) - 1) / (tall ? 2 * GBM : GBM), 1));
#define PCMD_GEMM_CASE(E_)                                                                             \
  if (epi == E_) {                                                                                     \
    if (tall)                                                                                          \
      hipLaunchKernelGGL((k_gemm<E_, 4, false>), grid, dim3(512), 0, s, g);                            \
    else if (steps)                                                                                    \
      hipLaunchKernelGGL((k_gemm<E_, 2, true>), grid, dim3(256), 0, s, g);                             \
    else                                                                                               \
      hipLaunchKernelGGL((k_gemm<E_, 2, false>), grid, dim3(256), 0, s, g);                            \
    return hipGetLastError();                                                                          \
  }
  PCMD_GEMM_CASE(EPI_STORE)
  PCMD_GEMM_CASE(EPI_BIAS)
  PCMD_GEMM_CASE(EPI_BIAS_GELU)
  PCMD_GEMM_CASE(EPI_GELU_GRAD)
  PCMD_GEMM_CASE(EPI_BIAS_MSE)
#undef PCMD_GEMM_CASE
  return hipErrorInvalidValue;
}

static hipError_t launch_colsum(const ColsumArgs &c, hipStream_t s) {
  hipLaunchKernelGGL(k_colsum, dim3((c.m + 63) / 64), dim3(64 * COLSUM_WAVES), 0, s, c);
  return hipGetLastError();
}

template <int GW, int GX>
static void launch_back_t(const GemmArgs &w, const GemmArgs &x, const ColsumArgs &c, unsigned nbw, unsigned nbx, hipStream_t s) {
  constexpr int G = GW > GX ? GW : GX;
  constexpr size_t lds = 2 * HB * HLD * sizeof(__bf16);  // one group's tiles
  const unsigned nbc = (unsigned)((c.m + 63) / 64 + 7) / 8 * 8;  // whole turns over the XCDs
  hipLaunchKernelGGL((k_gemm64_back<GW, GX>), dim3(nbc + nbx + nbw), dim3(256 * G), G * lds, s, w, x, c, nbc, nbx);
}

hipError_t launch_backward(const GemmArgs &w0, const GemmArgs *x0, const ColsumArgs &c, void *ws, size_t ws_bytes,
                           hipStream_t s) {
  GemmArgs w = w0, x = x0 ? *x0 : GemmArgs{};
  int kw = w.K, kx = x.K;
  const int sw = gemm_splits(w.M, w.N, w.K, kw), sx = x0 ? gemm_splits(x.M, x.N, x.K, kx) : 1;
  const bool iw = sw <= G64_SPLITS, ix = sx <= G64_SPLITS;
  const int gw = !iw ? 1 : sw > 2 ? 4 : sw, gx = !ix ? 1 : sx > 2 ? 4 : sx;
  w.nz = iw ? 1 : sw;
  x.nz = ix ? 1 : sx;
  const unsigned nbw = xcd_blocks((w.N + HB - 1) / HB, (w.M + HB - 1) / HB, w.nz);
  const unsigned nbx = x0 ? xcd_blocks((x.N + HB - 1) / HB, (x.M + HB - 1) / HB, x.nz) : 0;
  // One launch where both take 64 x 64 tiles and have the workspace to themselves, and blocks with
  // different numbers of groups only where they all run at once (the smaller ones hold the larger ones' LDS)
  const bool one = gemm_use64(w.M, w.N) && (!x0 || gemm_use64(x.M, x.N)) && (iw || ix) &&
                   (!x0 || gw == gx || nbw + nbx + (c.m + 63) / 64 <= 256);
  if (!one) {
    hipError_t e = launch_gemm(w0, true, true, EPI_STORE, ws, ws_bytes, s);
    if (e == hipSuccess) e = launch_colsum(c, s);
    if (e == hipSuccess && x0) e = launch_gemm(*x0, false, false, EPI_GELU_GRAD, ws, ws_bytes, s);
    return e;
  }
  if (ws_bytes < gemm_workspace_bytes(w.M, w.N, w.K, true, true) ||
      (x0 && ws_bytes < gemm_workspace_bytes(x.M, x.N, x.K, false, false)))
    return hipErrorInvalidValue;
  w.kchunk = sw > 1 ? kw : w.K;
  x.kchunk = sx > 1 ? kx : x.K;
  w.part = iw ? nullptr : (float *)ws;
  x.part = ix ? nullptr : (float *)ws;
#define PCMD_BACK(W_, X_) \
  if (gw == W_ && gx == X_) launch_back_t<W_, X_>(w, x, c, nbw, nbx, s);
  if (!x0) {  // the first layer: no dx
    PCMD_BACK(1, 1) PCMD_BACK(2, 1) PCMD_BACK(4, 1)
  } else {
    PCMD_BACK(1, 1) PCMD_BACK(1, 2) PCMD_BACK(1, 4) PCMD_BACK(2, 1) PCMD_BACK(2, 2) PCMD_BACK(2, 4) PCMD_BACK(4, 1)
    PCMD_BACK(4, 2) PCMD_BACK(4, 4)
  }
#undef PCMD_BACK
  if (!iw)
    hipLaunchKernelGGL((k_gemm_splitk_reduce<EPI_STORE>), dim3((unsigned)(((int64_t)w.M * w.N + 255) / 256)), dim3(256), 0, s, w, sw);
  if (!ix)
    hipLaunchKernelGGL((k_gemm_splitk_reduce<EPI_GELU_GRAD>), dim3((unsigned)(((int64_t)x.M * x.N + 255) / 256)), dim3(256), 0, s, x, sx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Elementwise and reduction kernels.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_f32_to_bf16(const float *__restrict__ x, __bf16 *__restrict__ y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (__bf16)x[i];
}

hipError_t launch_f32_to_bf16(const float *x, void *y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_f32_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, (__bf16 *)y, n);
  return hipGetLastError();
}

// y[k][j] = bf16(x[row k][j]) for a batch of n samples of d inputs.
__global__ void __launch_bounds__(256) k_gather_f32_to_bf16(const float *__restrict__ x, const int32_t *__restrict__ rows,
                                                            int64_t n_total, int d, int64_t n, __bf16 *__restrict__ y,
                                                            uint32_t *status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * d) return;
  const int64_t k = i / d, j = i - k * d;
  y[i] = (__bf16)x[batch_row(rows, k, n_total, status) * d + j];
}

hipError_t launch_gather_f32_to_bf16(const float *x, const int32_t *rows, int64_t n_total, int d, int64_t n, void *y,
                                     uint32_t *status, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_f32_to_bf16, dim3((unsigned)((n * d + 255) / 256)), dim3(256), 0, s, x, rows, n_total, d,
                     n, (__bf16 *)y, status);
  return hipGetLastError();
}

// Training targets of the surrogate: out[r][j] = ln((H[r][j] + 1/2) / (N_r + n_bins / 2)) with
// N_r the row's total, in FP64 (one block per row; the total is exact in FP64 below 2^53).
__global__ void __launch_bounds__(256) k_log_hess_target(const uint32_t *__restrict__ h, int nbins,
                                                         float *__restrict__ out) {
  __shared__ uint64_t red[256];
  const uint32_t *hr = h + (size_t)blockIdx.x * nbins;
  float *o = out + (size_t)blockIdx.x * nbins;
  const int t = threadIdx.x;
  uint64_t n = 0;
  for (int j = t; j < nbins; j += 256) n += hr[j];
  red[t] = n;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (t < k) red[t] += red[t + k];
    __syncthreads();
  }
  const double den = (double)red[0] + 0.5 * (double)nbins;
  for (int j = t; j < nbins; j += 256) o[j] = (float)log(((double)hr[j] + 0.5) / den);
}

hipError_t launch_log_hess_target(const uint32_t *h, int n, int nbins, float *out, hipStream_t s) {
  hipLaunchKernelGGL(k_log_hess_target, dim3(n), dim3(256), 0, s, h, nbins, out);
  return hipGetLastError();
}

// dy = 2 (y - t) / (n M) stored in BF16 (skipped when dy is NULL); per-block partial sums of
// (y - t)^2 in FP64.  y is [n / M][M]; the target row of sample k is batch_row(rows, k).  Threads
// take runs of four elements (16-byte loads, 8-byte stores) when the pointers and the row length
// allow it.
__global__ void __launch_bounds__(256) k_mse_grad(const float *__restrict__ y, const float *__restrict__ t, int64_t n,
                                                  int M, const int32_t *__restrict__ rows, int64_t n_total,
                                                  double scale, __bf16 *__restrict__ dy, double *__restrict__ part,
                                                  uint32_t *status) {
  __shared__ double red[256];
  double s = 0.0;
  const float g = (float)(2.0 * scale);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool vec = ((((uintptr_t)y) | ((uintptr_t)t)) & 15) == 0 && (((uintptr_t)dy) & 7) == 0 && (M & 3) == 0;
  const int64_t n4 = vec ? n / 4 : 0;
  for (int64_t i = first; i < n4; i += stride) {
    const int64_t k = (4 * i) / M, j = 4 * i - k * M;
    const float4 a = reinterpret_cast<const float4 *>(y)[i];
    const float4 b = *reinterpret_cast<const float4 *>(t + batch_row(rows, k, n_total, status) * M + j);
    const float d0 = a.x - b.x, d1 = a.y - b.y, d2 = a.z - b.z, d3 = a.w - b.w;
    if (dy) {
      bf16x4 o;
      o[0] = (__bf16)(g * d0);
      o[1] = (__bf16)(g * d1);
      o[2] = (__bf16)(g * d2);
      o[3] = (__bf16)(g * d3);
      reinterpret_cast<bf16x4 *>(dy)[i] = o;
    }
    s += (double)d0 * (double)d0;
    s += (double)d1 * (double)d1;
    s += (double)d2 * (double)d2;
    s += (double)d3 * (double)d3;
  }
  for (int64_t i = 4 * n4 + first; i < n; i += stride) {
    const int64_t k = i / M, j = i - k * M;
    const float d = y[i] - t[batch_row(rows, k, n_total, status) * M + j];
    if (dy) dy[i] = (__bf16)(g * d);
    s += (double)d * (double)d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

hipError_t launch_mse_grad(const float *y, const float *t, int64_t n, int M, const int32_t *rows, int64_t n_total,
                           double scale, void *dy, double *part, uint32_t *status, hipStream_t s) {
  hipLaunchKernelGGL(k_mse_grad, dim3(MSE_BLOCKS), dim3(256), 0, s, y, t, n, M, rows, n_total, scale, (__bf16 *)dy,
                     part, status);
  return hipGetLastError();
}

// out = scale x the sum of nb partials: thread t sums partials t, t + 256, ... in order, then a
// fixed tree over the block (the order depends on nb alone).
template <typename T>
__global__ void __launch_bounds__(256) k_sum_partials(const double *__restrict__ part, int64_t nb, double scale,
                                                      T *__restrict__ out) {
  __shared__ double red[256];
  double s = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < nb; i += 256) s += part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (T)(red[0] * scale);
}

hipError_t launch_sum_partials(const double *part, int64_t nb, double scale, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_partials<double>, dim3(1), dim3(256), 0, s, part, nb, scale, out);
  return hipGetLastError();
}
hipError_t launch_sum_partials(const double *part, int64_t nb, double scale, float *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_partials<float>, dim3(1), dim3(256), 0, s, part, nb, scale, out);
  return hipGetLastError();
}

// Adam on the FP32 master weights [out][in] and biases of every layer in one launch, refreshing the
// BF16 copies W [out][in] and W^T [in][out].  Without an update only the copies are refreshed.  A
// block takes a tile of ROWS rows and 64 columns of one layer's weights (tiles of layer l are blocks first[l] ..
// first[l + 1] - 1; the tile's rows' biases go with the first tile of a row), a row of a wave at a time, and writes
// W^T's rows from an LDS copy of the tile: a column-strided 2-byte store per weight had cost the
// update half its time.  Bound by the 32 bytes per weight (moments, master, gradient, copies).
// 5.4 million weights: 67 us in five launches -> 37 us in one, 33 us (5.2 TB/s) with the short tiles below.
// Networks of up to 1,535 64-row tiles are bound by the latency of a wave's rows one after another, and take 16 rows
// (four to a wave): 512 x 512 11.0 -> 5.0 us, 3 -> 580 13.8 -> 5.9 us, 2048 x 1024 (512 tiles) 18.8 -> 11.4 us; at
// 1,504 tiles 39 us with either, at 4,096 tiles 110 with 16 rows and 96 with 64 (W^T in pieces of 128 bytes, not 32).
constexpr int AT = 64, ADAM_SHORT = 16;
constexpr int64_t ADAM_SHORT_BLOCKS = 1536;

template <int ROWS>
__global__ void __launch_bounds__(256) k_adam(AdamArgs a) {
  __shared__ __bf16 tile[ROWS][AT + 2];
  int l = 0;
  while (l + 1 < a.n_layers && (int)blockIdx.x >= a.first[l + 1]) ++l;
  const int n_in = a.dims[l], n_out = a.dims[l + 1];
  const int tiles_in = (n_in + AT - 1) / AT;
  const int q = (int)blockIdx.x - a.first[l];
  const int o0 = (q / tiles_in) * ROWS, i0 = (q % tiles_in) * AT;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = a.off[l];
  auto step = [&](int64_t i) {
    float x = a.master[i];
    if (a.update) {
      const float g = a.grad[i];
      const float m = a.beta1 * a.m[i] + (1.0f - a.beta1) * g;
      const float v = a.beta2 * a.v[i] + (1.0f - a.beta2) * g * g;
      a.m[i] = m;
      a.v[i] = v;
      const float mh = m / a.bc1, vh = v / a.bc2;
      x = x - a.lr * mh / (sqrtf(vh) + a.eps);
      a.master[i] = x;
    }
    return (__bf16)x;
  };
#pragma unroll 4
  for (int r = w; r < ROWS; r += 4) {
    const int o = o0 + r, i = i0 + lane;
    if (o >= n_out || i >= n_in) continue;
    const __bf16 wb = step(base + (int64_t)o * n_in + i);
    ((__bf16 *)a.w_bf16)[a.woff[l] + (int64_t)o * n_in + i] = wb;
    tile[r][lane] = wb;
  }
  if (i0 == 0 && threadIdx.x < ROWS && o0 + (int)threadIdx.x < n_out)
    (void)step(base + (int64_t)n_out * n_in + o0 + threadIdx.x);
  __syncthreads();
  for (int t = threadIdx.x; t < AT * ROWS; t += 256) {
    const int i = i0 + t / ROWS, o = o0 + t % ROWS;
    if (i < n_in && o < n_out) ((__bf16 *)a.wt_bf16)[a.woff[l] + (int64_t)i * n_out + o] = tile[t % ROWS][t / ROWS];
  }
}

hipError_t launch_adam(AdamArgs a, hipStream_t s) {
  if (a.n_layers < 1 || a.n_layers > PCMD_MLP_MAX_LAYERS) return hipErrorInvalidValue;
  auto lay_out = [&](int rows) {
    int64_t blocks = 0;
    for (int l = 0; l < a.n_layers && blocks <= 0x7FFFFFFF; ++l) {
      a.first[l] = (int)blocks;
      blocks += (int64_t)((a.dims[l] + AT - 1) / AT) * ((a.dims[l + 1] + rows - 1) / rows);
    }
    a.first[a.n_layers] = (int)blocks;
    return blocks;
  };
  int64_t blocks = lay_out(AT);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (blocks < ADAM_SHORT_BLOCKS) {
    blocks = lay_out(ADAM_SHORT);
    hipLaunchKernelGGL(k_adam<ADAM_SHORT>, dim3((unsigned)blocks), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_adam<AT>, dim3((unsigned)blocks), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// Surrogate log-likelihood.  With x_j = y_j - max y and se = sum exp(x_j), bin j expects lam_j = N_d
// exp(x_j) / se, so ln lam_j = x_j + ln(N_d / se) and sum lam_j = N_d:
//   logL = sum_j d_j x_j + N_d ln(N_d / se) - N_d - sum_j ln d_j!
// needs one exponential per bin, where the term-by-term form took two and a logarithm (FP64, so
// bound by their vector instructions).  A block walks samples, its share of the data
// (N_d, the factorials' sum, each thread's counts of the first SLL_REG rounds) kept from one to the
// next; a thread also keeps its bins of y between the maximum and the exponentials.  The order of a
// sample's sums depends on the number of bins alone.
// 10,000 bins: one sample 42 -> 9.4 us, 4,096 samples 431 -> 78 us (156 with the library's exponential,
// a block per sample and the data's sums formed for each); no spills, which had cost half of that.
// SLL_THREADS threads to a block, or SLL_FEW where their registers hold every bin: the passes over a sample's barriers
// are then of four waves, and eight samples run on a CU at a time where two do (100 bins: 512 samples 5.5 us, 11.9 in
// blocks of 1,024 threads, 4,096 samples 14.5 and 45; 2,500 bins 7.1 and 12.5, 21 and 50; 4,096 bins, beyond the
// registers, 10.3 and 13.1, but one sample 9.0 and 7.8, and 10,000 bins 26 and 16).
constexpr int SLL_THREADS = 1024, SLL_FEW = 256, SLL_REG = 10;
constexpr int SLL_BLOCKS = 512;  // of SLL_THREADS threads: what the chip holds
constexpr int SLL_SAMPLES = 64;  // samples per block, at most

// The sums of u and v over the block in a fixed order (trees of shuffles in each wave, then over the
// waves).
template <int THREADS>
__device__ __forceinline__ void sll_sum2(double &u, double &v, double (*red)[2]) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    u += __shfl_xor(u, d, 64);
    v += __shfl_xor(v, d, 64);
  }
  if ((threadIdx.x & 63u) == 0u) {
    red[threadIdx.x >> 6][0] = u;
    red[threadIdx.x >> 6][1] = v;
  }
  __syncthreads();
  constexpr unsigned W = THREADS / 64;  // a power of two
  u = red[threadIdx.x & (W - 1)][0];
  v = red[threadIdx.x & (W - 1)][1];
#pragma unroll
  for (int d = W / 2; d > 0; d >>= 1) {
    u += __shfl_xor(u, d, 64);
    v += __shfl_xor(v, d, 64);
  }
}

template <int THREADS>
__global__ void __launch_bounds__(THREADS, 8) k_surrogate_loglike(const float *__restrict__ y, int n, int nbins,
                                                                  const uint32_t *__restrict__ d,
                                                                  double *__restrict__ out,
                                                                  const double *__restrict__ lnfact64, int nlf) {
  __shared__ double red[2][THREADS / 64][2];
  __shared__ float redf[THREADS / 64];
  __shared__ double fin[SLL_SAMPLES][2];  // se and sum d x of the block's samples
  const int t = threadIdx.x;
  uint32_t dv[SLL_REG];
#pragma unroll
  for (int k = 0; k < SLL_REG; ++k) {
    dv[k] = 0u;
    if ((uint32_t)t + k * THREADS < (uint32_t)nbins) dv[k] = (d + k * THREADS)[(uint32_t)t];
  }
  double nd = 0.0, lf = 0.0;
  bool large = false;
#pragma unroll
  for (int k = 0; k < SLL_REG; ++k) {  // ln 0! = ln 1! = 0
    nd += (double)dv[k];
    if (dv[k] > 1u) lf += lnfact64[dv[k] < (uint32_t)nlf ? dv[k] : 0u];
    large = large || dv[k] >= (uint32_t)nlf;
  }
  // counts beyond the table and bins beyond the registers
#pragma unroll 1
  for (int j = large ? t : t + SLL_REG * THREADS; j < nbins; j += THREADS) {
    const uint32_t dj = d[j];
    const bool kept = j < SLL_REG * THREADS;
    if (!kept) nd += (double)dj;
    if (dj >= (uint32_t)nlf)
      lf += ln_factorial_large(dj);
    else if (!kept && dj > 1u)
      lf += lnfact64[dj];
  }
  sll_sum2<THREADS>(nd, lf, red[0]);
  int q0 = 0;
  for (int s = blockIdx.x; s < n; s += gridDim.x, ++q0) {
    const float *ys = y + (size_t)s * nbins;
    float v[SLL_REG];
#pragma unroll
    for (int k = 0; k < SLL_REG; ++k) {
      v[k] = -INFINITY;
      if ((uint32_t)t + k * THREADS < (uint32_t)nbins) v[k] = (ys + k * THREADS)[(uint32_t)t];
    }
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < SLL_REG; ++k) m = fmaxf(m, v[k]);
    for (int j = t + SLL_REG * THREADS; j < nbins; j += THREADS) m = fmaxf(m, ys[j]);
#pragma unroll
    for (int q = 32; q > 0; q >>= 1) m = fmaxf(m, __shfl_xor(m, q, 64));
    if ((t & 63) == 0) redf[t >> 6] = m;
    __syncthreads();
    m = redf[t & (THREADS / 64 - 1)];
#pragma unroll
    for (int q = THREADS / 128; q > 0; q >>= 1) m = fmaxf(m, __shfl_xor(m, q, 64));
    const double mx = (double)m;
    double se = 0.0, dx = 0.0;
    auto bin = [&](float yj, uint32_t dj) {
      const double x = (double)yj - mx;
      const double e = exp_nonpos(x);
      se += e;
      // a bin whose expectation underflows to zero counts as ln 0, also where it holds no data
      dx += (double)dj * (e == 0.0 ? -INFINITY : x);
    };
#pragma unroll
    for (int k = 0; k < SLL_REG; ++k) {
      // converted here for each sample: kept in FP64, the counts would spill
      asm volatile("" : "+v"(dv[k]));
      if (t + k * THREADS < nbins) bin(v[k], dv[k]);
    }
    for (int j = t + SLL_REG * THREADS; j < nbins; j += THREADS) bin(ys[j], d[j]);
    sll_sum2<THREADS>(se, dx, red[1]);  // its barrier also parts this sample's redf from the next one's
    if (t == 0) {
      fin[q0][0] = se;
      fin[q0][1] = dx;
    }
  }
  __syncthreads();
  if (t < q0) out[blockIdx.x + t * gridDim.x] = fin[t][1] + nd * ln_pos(nd / fin[t][0]) - nd - lf;
}

hipError_t launch_surrogate_loglike(const float *y, int n, int nbins, const uint32_t *d, double *out,
                                   const double *lnfact64, int nlf, hipStream_t s) {
  if (!lnfact64 || nlf < 1000) return hipErrorInvalidValue;
  auto launch = [&](auto threads) {
    constexpr int T = decltype(threads)::value;
    const int blocks = std::max(std::min(n, SLL_BLOCKS * (SLL_THREADS / T)), (n + SLL_SAMPLES - 1) / SLL_SAMPLES);
    hipLaunchKernelGGL(k_surrogate_loglike<T>, dim3((unsigned)blocks), dim3(T), 0, s, y, n, nbins, d, out, lnfact64, nlf);
  };
  if (nbins <= SLL_FEW * SLL_REG)
    launch(std::integral_constant<int, SLL_FEW>{});
  else
    launch(std::integral_constant<int, SLL_THREADS>{});
  return hipGetLastError();
}

}  // namespace pcmd
