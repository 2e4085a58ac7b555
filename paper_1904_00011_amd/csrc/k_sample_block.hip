// Block-skip sampler: the per-pixel star counts by Poisson superposition (Sec. 2.1 footnote).
//
// A sum of independent Poisson counts is Poisson with the summed mean, and given that sum the
// individual counts are multinomial.  Per pixel and per block b of SBLK = 64 consecutive entries:
//   * the block total N ~ Poisson(Lambda_b), Lambda_b = sum of the block's lambda_i (FP64, left
//     to right): below 10 by inversion of word 0 of Philox(p, b, TAG_BLOCK, 0), from 10 on by
//     transformed rejection on Philox(p, b, TAG_BLOCK_PTRS, j) (the per-entry routines);
//   * star s of the block takes word s mod 4 of Philox(p, b, TAG_STAR, s / 4) and lands on the
//     first entry i whose cumulative threshold C_i = floor(2^32 cum_i / Lambda_b) exceeds it
//     (entry i with probability lambda_i / Lambda_b to 2^-32);
//   * star s is behind the dust screen iff word s mod 4 of Philox(p, b, TAG_STAR_SPLIT, s / 4)
//     is below floor(F 2^32) (F = 1: every star; no dust: none).
// The law of the counts is that of the per-entry rule; the random stream is a different one.
// At low stellar density most blocks draw nothing in every pixel of a wave and cost one Philox
// block and one compare, instead of the per-entry rule's sixteen Philox blocks.
//
// Layout: a wave takes 64 or 128 pixels; its 64 lanes also hold one block's 64 cumulative thresholds and
// entry fluxes in registers, so each star's binary search and flux gather are cross-lane reads
// (ds_bpermute).  Slices interleave blocks like k_sample's interleaved 16-entry blocks and write the
// same partial-sum layout, which k_reduce then sums in the same order.
#include <algorithm>

#include "pcmd_device.h"
#include "pcmd_internal.h"

namespace pcmd {

// One wave per block: lane l takes entry SBLK b + l.
__device__ __forceinline__ void prep_block_body(const BlockPrepArgs &a) {
  __shared__ double lam_s[4][SBLK];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int b = blockIdx.x * 4 + w;
  if (b >= a.nb) return;  // whole waves only: nothing below synchronises across waves
  const int i = b * SBLK + lane;
  double l = 0.0;
  if (i < a.E) {
    double fv[4];  // every load before the first store
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // band min(k, B - 1) is always in range: no branch around the load
      const float v = a.flux[(size_t)min(k, a.B - 1) * a.E + i];
      fv[k] = k < a.B ? (double)v : 0.0;
    }
    l = a.lam[i];
    for (int k = 0; k < a.BP; ++k) a.fl64[(size_t)i * a.BP + k] = fv[k];
    if (!(l >= 0.0 && l < 4194304.0)) {  // NaN, negative or too large: drawn as zero, reported
      atomicOr(a.status, STATUS_BAD_LAMBDA);
      l = 0.0;
    }
  }
  lam_s[w][lane] = l;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  // cum_l: every lane sums the entries 0..l of its block left to right, the order of Lambda_b (a fixed
  // count, so that the reads run ahead of the additions; entries past l add exact zeros)
  double cum = 0.0;
#pragma unroll 16
  for (int k = 0; k < SBLK; ++k) {
    const double v = lam_s[w][k];
    cum += k <= lane ? v : 0.0;
  }
  const double L = __shfl(cum, SBLK - 1, 64);  // Lambda_b = cum_63
  BlockRec r{{0u, 0u, 0u}, KIND_ZERO, (uint32_t)SBLK - 1u, {0u, 0u, 0u}};
  if (a.hybrid && L >= 10.0) {  // hybrid: this block's entries go to the per-point rule
    r.pad[0] = 1u;
  } else if (!(L < 4194304.0)) {  // the block total must stay in the per-entry rule's range
    if (lane == 0) atomicOr(a.status, STATUS_BAD_LAMBDA);
  } else if (L > 0.0) {
    // C_l = floor(2^32 cum_l / Lambda_b); the last entry with stars reaches cum = Lambda_b
    // exactly (same additions), so C = 2^32 from there on
    const double C = floor(cum / L * 4294967296.0);
    const uint64_t full = __ballot(C >= 4294967296.0);  // lane 63 always
    const uint32_t istar = (uint32_t)__builtin_ctzll(full);
    a.cth[(size_t)b * SBLK + lane] = (uint32_t)lane < istar ? (uint32_t)C : 0xFFFFFFFFu;
    r.istar = istar;
    if (lane == 0) {
      if (L >= 10.0) {
        ((PtrsConst *)a.pc)[b] = ptrs_constants(L);
        r.kk = KIND_PTRS;
      } else {
        uint32_t first[3] = {0u, 0u, 0u};
        const uint32_t K = inversion_table(L, a.thr + (size_t)b * THR_STRIDE, 1, first);
        if (K > 0) {
#pragma unroll
          for (uint32_t k = 0; k < 3; ++k) r.T[k] = k < K ? first[k] : r.T[k];
          r.kk = (K << 8) | KIND_INV;
        }
      }
    }
  }
  if (lane == 0) a.brec[b] = r;
}

__global__ void __launch_bounds__(256) k_prep_block(BlockPrepArgs a) { prep_block_body(a); }
// batched: the arguments of job j of a descriptor table
__global__ void __launch_bounds__(256) k_prep_block_job(const BlockPrepArgs *__restrict__ t, int j) {
  const BlockPrepArgs a = t[j];
  prep_block_body(a);
}

hipError_t launch_prep_block(const BlockPrepArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_prep_block, dim3((unsigned)((a.nb + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_prep_block_job(const BlockPrepArgs *table, int j, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_prep_block_job, dim3((unsigned)((nb + 3) / 4)), dim3(256), 0, s, table, j);
  return hipGetLastError();
}

// Groups of four stars per pixel queued at a time (two leave LDS for six waves per SIMD).
constexpr int BQG = 2;

// Pixels per lane: two pack the queue better (4096 x 4096 above: 2.07 ms with one, 1.75 with two; four leave
// LDS for three waves per SIMD: 2.72), one gives twice the waves where an image has few.  The line lies
// at three two-pixel workgroups per CU: 128 x 128 with 26 slices (832 workgroups) 27 us with one and 24
// with two, 180 x 180 with 11 (704) 145 and 191, 67 x 67 with 11 blocks of 380 stars each (99) 543 and 1071.
static int block_ppl(int npx, int nchunks, int nb) {
  return (int64_t)((npx + 511) / 512) * std::min(nchunks, nb) < 768 ? 1 : 2;
}

// The stars of one block over a wave's 64 PPL pixels are queued as tasks (pixel, group of four stars of
// it, how many), which the lanes then take 64 at a time: a lane per pixel would draw words and search for
// as many stars as the fullest of 64 pixels has, 18% to 36% of them there.  A task's stars go to
// any pixel, so the sums are in LDS (FP64 adds; one wave's, in its own order).  Vector issue and LDS are
// both busy three quarters of the time.  4096 x 4096 x 3 at 10^3 stars per pixel, 12 blocks: 2103 ->
// 1561 us; 250 x 250, 726 blocks: 260 -> 193 us.
template <int B, int S, bool DBG, int PPL>
__device__ __forceinline__ void sample_block_body(const BlockSampleArgs &a) {
  constexpr int BP = B <= 2 ? 2 : 4, PX = 64 * PPL;
  __shared__ double acc_s[4][S * B][PX];
  __shared__ uint16_t task_s[4][PX * BQG];
  const int nblk_px = (a.npx + 4 * PX - 1) / (4 * PX);
  const int chunk = blockIdx.x / nblk_px;
  const int wv = threadIdx.x >> 6;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t p0 = (uint32_t)((blockIdx.x - chunk * nblk_px) * 4 + wv) * PX;  // the wave's first pixel
  if (p0 >= (uint32_t)a.npx) return;  // whole waves: no barrier below
  const PCMD_CONST BlockRec *brec = (const PCMD_CONST BlockRec *)a.brec;
  const PCMD_CONST uint32_t *thr = (const PCMD_CONST uint32_t *)a.thr;
  const PCMD_CONST PtrsConst *pc = (const PCMD_CONST PtrsConst *)a.pc;
  const bool draw_split = S == 2 && (a.split_mode == SPLIT_HALF || a.split_mode == SPLIT_GENERAL);
  double(*acc)[PX] = acc_s[wv];
  uint16_t *task = task_s[wv];
#pragma unroll
  for (int k = 0; k < S * B; ++k)
#pragma unroll
    for (int q = 0; q < PPL; ++q) acc[k][q * 64 + lane] = 0.0;

  uint32_t ptrs_failed = 0u;
  // every lane runs every step below, so the cross-lane reads always find their source lane active;
  // branches on the counts go through wave-wide votes
  for (int b = chunk; b < a.nb; b += a.nchunks) {
    const BlockRec r = ld_const(brec + b);
    const uint32_t kind = r.kk & KIND_MASK;
    if (kind == KIND_ZERO) continue;
    uint32_t n[PPL];
    bool some = false;
    if (kind == KIND_INV) {
      // N = #{k < K : T_k <= u}, walking up while any lane of the wave is still above
      uint32_t u[PPL];
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        u[q] = philox10(p0 + 64u * q + lane, (uint32_t)b, TAG_BLOCK, 0u, a.k0, a.k1).x;
        n[q] = u[q] >= r.T[0] ? 1u : 0u;
        some = some || n[q] != 0u;
      }
      if (!wave_any(some)) continue;
      const uint32_t K = r.kk >> 8;
      for (uint32_t k = 1; k < K; ++k) {
        const uint32_t t = k < 3 ? r.T[k] : thr[(size_t)b * THR_STRIDE + k];
        bool more = false;
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
          const bool c = u[q] >= t;
          n[q] += c ? 1u : 0u;
          more = more || c;
        }
        if (!wave_any(more)) break;
      }
    } else {
      const PtrsConst cst = ld_const(pc + b);
#pragma unroll
      for (int q = 0; q < PPL; ++q) {
        n[q] = ptrs_draw(cst, p0 + 64u * q + lane, (uint32_t)b, TAG_BLOCK_PTRS, a.k0, a.k1, a.lnfact, ptrs_failed);
        some = some || n[q] != 0u;
      }
      if (!wave_any(some)) continue;
    }
    // the block's thresholds and fluxes (FP32 values), one entry per lane
    const int e = b * SBLK + (int)lane;
    const int cl = (int)a.cth[(size_t)b * SBLK + lane];
    int fl[B];
#pragma unroll
    for (int k = 0; k < B; ++k) fl[k] = e < a.E ? __float_as_int((float)a.fl64[(size_t)e * BP + k]) : 0;
    const uint32_t istar = r.istar;
    const uint32_t c16 = (uint32_t)__builtin_amdgcn_readlane(cl, 15), c32 = (uint32_t)__builtin_amdgcn_readlane(cl, 31),
                   c48 = (uint32_t)__builtin_amdgcn_readlane(cl, 47);
#pragma unroll
    for (int q = 0; q < PPL; ++q)
      if (p0 + 64u * q + lane >= (uint32_t)a.npx) n[q] = 0u;
    for (uint32_t g0 = 0;; g0 += BQG) {
      // task: pixel | (group - g0) << 8 | (stars - 1) << 9
      uint32_t tasks = 0u;
      for (uint32_t gg = 0; gg < BQG; ++gg) {
        const uint32_t before = tasks, first = 4u * (g0 + gg);
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
          const uint64_t m = __ballot(n[q] > first);
          if (m == 0ull) continue;
          const uint32_t at = tasks + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          if (n[q] > first) task[at] = (uint16_t)(lane + 64u * q + (gg << 8) + ((min(n[q] - first, 4u) - 1u) << 9));
          tasks += (uint32_t)__popcll(m);
        }
        if (tasks == before) break;
      }
      if (tasks == 0u) break;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (uint32_t t0 = 0; t0 < tasks; t0 += 64u) {
        const bool mine = t0 + lane < tasks;
        const uint32_t t = task[mine ? t0 + lane : 0u];
        const uint32_t c = mine ? (t >> 9) + 1u : 0u, px = t & 255u, g = g0 + ((t >> 8) & 1u);
        const u4 ws = philox10(p0 + px, (uint32_t)b, TAG_STAR, g, a.k0, a.k1);
        u4 wr{0u, 0u, 0u, 0u};
        if (draw_split) wr = philox10(p0 + px, (uint32_t)b, TAG_STAR_SPLIT, g, a.k0, a.k1);
#pragma unroll
        for (uint32_t s = 0; s < 4u; s += 2u) {  // two stars at a time: their searches overlap
          if (s > 0u && !wave_any(s < c)) break;
          // number of thresholds <= u among the 64 (sorted; the count stops at 63), then capped at
          // istar: the first entry whose threshold exceeds u.  Byte offsets of lanes.
          uint32_t pos[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {  // the first two halvings without cross-lane reads
            const uint32_t u = word_of(ws, (int)s + j);
            const bool hi = u >= c32;
            pos[j] = (hi ? 4u * 32u : 0u) + (u >= (hi ? c48 : c16) ? 4u * 16u : 0u);
          }
#pragma unroll
          for (uint32_t st = 8u; st != 0u; st >>= 1)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const uint32_t v = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(pos[j] + 4u * (st - 1u)), cl);
              pos[j] += v <= word_of(ws, (int)s + j) ? 4u * st : 0u;
            }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const uint32_t cat = min(pos[j], 4u * istar);
            float f[B];
#pragma unroll
            for (int k = 0; k < B; ++k) f[k] = __int_as_float(__builtin_amdgcn_ds_bpermute((int)cat, fl[k]));
            const bool red = S == 2 && (a.split_mode == SPLIT_ALL || (draw_split && word_of(wr, (int)s + j) < a.split_q));
            if (s + (uint32_t)j < c) {
              double *o = &acc[red ? B : 0][px];
#pragma unroll
              for (int k = 0; k < B; ++k)
                __hip_atomic_fetch_add(o + k * PX, (double)f[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
              const int i = b * SBLK + (int)(cat >> 2);
              if (DBG && (int64_t)(p0 + px) >= a.px0 && (int64_t)(p0 + px) < a.px1 && i < a.E) {  // always: cat <= istar, an entry with stars
                const size_t d = (size_t)((int64_t)(p0 + px) - a.px0) * (size_t)a.E + (size_t)i;
                atomicAdd(a.dbg_counts + d, 1u);
                if (red && a.dbg_red) atomicAdd(a.dbg_red + d, 1u);
              }
            }
          }
        }
      }
    }
  }
  if (wave_any(ptrs_failed != 0u) && lane == 0u) atomicOr(a.status, STATUS_PTRS_RETRY);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const size_t plane = (size_t)a.npx;
#pragma unroll
  for (int k = 0; k < S * B; ++k)
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
      const uint32_t p = p0 + 64u * q + lane;
      if (p >= (uint32_t)a.npx) continue;
      float *o = a.part + ((size_t)chunk * S * B + k) * plane + p;
      const double v = acc[k][q * 64 + lane];
      *o = (float)(a.accumulate ? (double)*o + v : v);
    }
}

static dim3 sample_block_grid(int npx, int nchunks, int ppl) {
  return dim3((unsigned)((npx + 256 * ppl - 1) / (256 * ppl) * nchunks));
}

template <int B, int S, bool DBG, int PPL>
__global__ void __launch_bounds__(256) k_sample_block(BlockSampleArgs a) {
  sample_block_body<B, S, DBG, PPL>(a);
}
// batched: job j of a descriptor table, both partial streams (as every batch job)
template <int B, int PPL>
__global__ void __launch_bounds__(256) k_sample_block_job(const BlockSampleArgs *__restrict__ t, int j) {
  const BlockSampleArgs a = t[j];
  sample_block_body<B, 2, false, PPL>(a);
}

template <int B, int PPL>
static hipError_t launch_sample_block_b(const BlockSampleArgs &a, hipStream_t s) {
  const dim3 grid = sample_block_grid(a.npx, a.nchunks, PPL);
  const bool dbg = a.dbg_counts != nullptr;
  if (a.S == 2 && dbg)
    hipLaunchKernelGGL((k_sample_block<B, 2, true, PPL>), grid, dim3(256), 0, s, a);
  else if (a.S == 2)
    hipLaunchKernelGGL((k_sample_block<B, 2, false, PPL>), grid, dim3(256), 0, s, a);
  else if (dbg)
    hipLaunchKernelGGL((k_sample_block<B, 1, true, PPL>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_sample_block<B, 1, false, PPL>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_sample_block(const BlockSampleArgs &a, hipStream_t s) {
  const bool two = block_ppl(a.npx, a.nchunks, a.nb) == 2;
  switch (a.B) {
    case 1: return two ? launch_sample_block_b<1, 2>(a, s) : launch_sample_block_b<1, 1>(a, s);
    case 2: return two ? launch_sample_block_b<2, 2>(a, s) : launch_sample_block_b<2, 1>(a, s);
    case 3: return two ? launch_sample_block_b<3, 2>(a, s) : launch_sample_block_b<3, 1>(a, s);
    case 4: return two ? launch_sample_block_b<4, 2>(a, s) : launch_sample_block_b<4, 1>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int PPL>
static hipError_t launch_sample_block_job_p(const BlockSampleArgs *table, int j, int B, int npx, int nchunks, hipStream_t s) {
  const dim3 grid = sample_block_grid(npx, nchunks, PPL);
  switch (B) {
    case 1: hipLaunchKernelGGL((k_sample_block_job<1, PPL>), grid, dim3(256), 0, s, table, j); break;
    case 2: hipLaunchKernelGGL((k_sample_block_job<2, PPL>), grid, dim3(256), 0, s, table, j); break;
    case 3: hipLaunchKernelGGL((k_sample_block_job<3, PPL>), grid, dim3(256), 0, s, table, j); break;
    case 4: hipLaunchKernelGGL((k_sample_block_job<4, PPL>), grid, dim3(256), 0, s, table, j); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sample_block_job(const BlockSampleArgs *table, int j, int B, int npx, int nchunks, int nb, hipStream_t s) {
  return block_ppl(npx, nchunks, nb) == 2 ? launch_sample_block_job_p<2>(table, j, B, npx, nchunks, s)
                                          : launch_sample_block_job_p<1>(table, j, B, npx, nchunks, s);
}

}  // namespace pcmd
