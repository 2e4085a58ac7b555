// Weighted entries, per-entry sampler tables, the pixel x entry Poisson sampler with fused
// flux accumulation, and the chunk reduction with the dust / distance epilogue (gfx950).
//
// Sec. 2.1 of the paper: every pixel draws an independent Poisson count for every weighted
// isochrone point, the stars' fluxes are reddened by dust, dimmed by the distance modulus and
// summed into the pixel.  One lane owns one pixel; the entry table is wave-uniform, so it is
// read through the scalar cache.  A wave handles 64 pixels x one chunk of CHUNK entries and
// keeps the per-band sums in FP64 registers; chunk partials are written once, rounded to FP32
// (a relative error of at most 2^-24 per partial, and the partials are non-negative, so the
// pixel sum keeps that bound), and combined in FP64 in ascending chunk order by the reduction
// kernel, which fixes the summation order independently of the launch shape.
#include <math.h>

#include <algorithm>

#include "pcmd_device.h"
#include "pcmd_internal.h"

namespace pcmd {

// ---------------------------------------------------------------------------------------
// a0: lambda_i = scale[iso(i)] * imf_w_i   (scale_k = Npix w_k / sum_k w_k S_k)
// ---------------------------------------------------------------------------------------
struct IsoScale {
  double v[PCMD_MAX_ISO];
};

__global__ void __launch_bounds__(256) k_entries(int E, int n_iso, const int32_t *__restrict__ iso,
                                                 const double *__restrict__ imf_w, IsoScale scale,
                                                 double *__restrict__ lam, uint32_t *__restrict__ status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= E) return;
  const int k = iso[i];
  if (k < 0 || k >= n_iso) {  // malformed grid: no stars, reported by pcmd_sync
    atomicOr(status, STATUS_BAD_LAMBDA);
    lam[i] = 0.0;
    return;
  }
  lam[i] = scale.v[k] * imf_w[i];
}

hipError_t launch_entries(const pcmd_grid *g, const double *scale, double *lam, uint32_t *status, hipStream_t s) {
  IsoScale sc;
  for (int k = 0; k < PCMD_MAX_ISO; ++k) sc.v[k] = k < g->n_iso ? scale[k] : 0.0;
  const int E = g->n_entries;
  hipLaunchKernelGGL(k_entries, dim3((E + 255) / 256), dim3(256), 0, s, E, g->n_iso, g->iso_of_entry, g->imf_w, sc,
                     lam, status);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Per-entry tables: inversion thresholds (lambda < ALIAS_MIN), an alias marker (the columns come
// from k_prep_alias) or rejection constants (lambda >= ALIAS_MAX)
// and the FP64 star fluxes, in each entry's record.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void prep_body(const PrepArgs &a, int i) {
  // every lane of the block takes part in the group summary below (no early return)
  const int E = a.E, B = a.B;
  EntryRec r{{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, KIND_ZERO, {0.0, 0.0, 0.0, 0.0}};
  bool red_alias = false;  // the entry is thinned and its reddened part is on the alias rule
  bool dense = false;      // an entry drawn by inversion of which a wave usually has a lane with three stars
  if (i < E) {
    // every load before the first store (the output could alias the inputs for the compiler,
    // which otherwise waits for each load in turn)
    double fv[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {  // band min(b, B - 1) is always in range: no branch around the load
      const float v = a.flux[(size_t)min(b, B - 1) * E + i];
      fv[b] = b < B ? (double)v : 0.0;
    }
    double l = a.lam[i];
    const bool block_rule = a.brec && a.brec[i / SBLK].pad[0] == 0u;  // hybrid: the block rule draws it
#pragma unroll
    for (int b = 0; b < 4; ++b) r.fl[b] = fv[b];
    if (!(l >= 0.0 && l < 4194304.0)) {  // NaN, negative or too large: drawn as zero, reported
      atomicOr(a.status, STATUS_BAD_LAMBDA);
      l = 0.0;
    }
    if (block_rule) l = 0.0;
    // thinned: the unreddened and reddened counts are two independent parts
    const bool thin = l >= ALIAS_MIN && (a.thin == THIN_TABLE || (a.thin == THIN_HALF_HIGH && l >= LAM_THIN_HALF));
    if (a.thin != THIN_NONE) a.rdesc[i] = KIND_ZERO;  // overwritten below for a thinned entry
    if (l >= ALIAS_MIN) {
      // table entry: the count (or, thinned, the unreddened part) in slot 0, the reddened part in
      // slot 1; alias parts are built by k_prep_alias, which completes their descriptors
      const double l0 = thin ? l * (1.0 - a.frac) : l;
      if (l0 >= ALIAS_MAX) {
        ((PtrsConst *)a.pc)[2 * (size_t)i] = ptrs_constants(l0);
        r.kk = KIND_PTRS;
      } else {
        r.kk = KIND_ALIAS;
      }
      if (thin) {
        r.kk |= FLAG_THIN;
        if (a.thin_seen) *a.thin_seen = a.gen;  // every writer stores the same value
        const double l1 = l * a.frac;
        if (l1 >= ALIAS_MAX) {
          ((PtrsConst *)a.pc)[2 * (size_t)i + 1] = ptrs_constants(l1);
          a.rdesc[i] = KIND_PTRS;
        } else {
          a.rdesc[i] = KIND_ALIAS;
          // F = 1/2: both halves have the same lambda and so the same table, the unreddened half's
          red_alias = a.thin != THIN_HALF_HIGH;
        }
      }
    } else if (l > 0.0) {
      // k-major: threshold k of entry i at thr[k EP + i], so that a wave's stores coalesce
      uint32_t first[3] = {0u, 0u, 0u};
      const uint32_t K = inversion_table(l, a.thr + i, (size_t)entries_padded(E), first);
      if (K > 0) {
        // T_0 >= 1 below ALIAS_MIN, so u >= T_k is exactly u > T_k - 1; an absent threshold's
        // 0xFFFFFFFF is never exceeded
#pragma unroll
        for (uint32_t k = 0; k < 3; ++k) r.T[k] = k < K ? first[k] - 1u : r.T[k];
        r.kk = (K << 8) | KIND_INV;
        dense = l >= LAM_DENSE;
      }
    }
  }
  const int EP = entries_padded(E);
  if (i < EP) a.rec[i] = r;
  if (a.alias_list) {
    // the alias parts (i << 1 | part) to the call's list, one reservation per wave; a count word
    // not prepared for this generation (the previous call stopped early) is left alone, and
    // k_prep_alias then walks every entry
    const bool al0 = i < E && (r.kk & KIND_MASK) == KIND_ALIAS, al1 = i < E && red_alias;
    const uint64_t b0 = __ballot(al0), b1 = __ballot(al1);
    const uint32_t cnt = (uint32_t)(__popcll(b0) + __popcll(b1));
    if (cnt != 0u) {
      unsigned long long old = 0ull;
      if ((threadIdx.x & 63u) == 0u) old = atomicAdd(a.alias_n + (a.gen & 1u), (unsigned long long)cnt);
      const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(old >> 32), 0, 64);
      const uint32_t base = (uint32_t)__shfl((int)(uint32_t)old, 0, 64);
      if (hi == a.gen && (uint64_t)base + cnt <= 2ull * (uint64_t)E) {
        const uint64_t below = (1ull << (threadIdx.x & 63u)) - 1ull;
        if (al0) a.alias_list[base + (uint32_t)__popcll(b0 & below)] = (uint32_t)i << 1;
        if (al1) a.alias_list[base + (uint32_t)__popcll(b0) + (uint32_t)__popcll(b1 & below)] = ((uint32_t)i << 1) | 1u;
      }
    }
  }

  // group of entries GRP g .. GRP g + GRP - 1 = neighbouring lanes of one wave (256-thread blocks)
  const uint32_t kind = r.kk & KIND_MASK;
  const uint32_t fl = (r.kk & FLAG_THIN) ? GRP_THIN | (GRP_THIN_ENTRY << (i & (GRP - 1)))
                      : kind == KIND_INV ? GRP_INV | (dense ? GRP_DENSE_ENTRY << (i & (GRP - 1)) : 0u)
                      : kind == KIND_PTRS || kind == KIND_ALIAS ? GRP_TABLE | (GRP_TABLE_ENTRY << (i & (GRP - 1))) : 0u;
  const int first = (int)(threadIdx.x & 63u) & ~(GRP - 1);
  GroupRec gr;
  gr.flags = 0u;
#pragma unroll
  for (int q = 0; q < GRP; ++q) {
    gr.t0m1[q] = (uint32_t)__shfl((int)(dense ? 0xFFFFFFFFu : r.T[0]), first + q, 64);
    gr.flags |= (uint32_t)__shfl((int)fl, first + q, 64);
  }
#pragma unroll
  for (int q = 0; q < 7; ++q) gr.pad[q] = 0u;
  if ((i & (GRP - 1)) == 0 && i < EP) a.grp[i / GRP] = gr;
}

__global__ void __launch_bounds__(256) k_prep(PrepArgs a) { prep_body(a, blockIdx.x * blockDim.x + threadIdx.x); }
// batched: the jobs j + blockIdx.z of a descriptor table, the grid sized for the first of them, the largest (the
// table is sorted, and the host ends the run where most of such a grid would be empty; a launch
// per job left most of the chip idle in each: 24 uneven jobs' tables 24 x 18 us, sums 24 x 25)
__global__ void __launch_bounds__(256) k_prep_job(const PrepArgs *__restrict__ t, int j) {
  const PrepArgs a = t[j + blockIdx.z];
  if (blockIdx.x * blockDim.x >= (unsigned)entries_padded(a.E)) return;
  prep_body(a, blockIdx.x * blockDim.x + threadIdx.x);
}

// Alias columns of the entries with ALIAS_MIN <= lambda < ALIAS_MAX (rule C1b), one wave per
// entry at a time.  The wave runs the inversion rule's FP64 recurrence without its cap until T_k
// reaches 2^32 - 1 (that threshold then counts as 2^32: the FP64 sum can stall just below 1); with
// k_lo = #{k : T_k = 0}, outcome k_lo + j has mass m_j = T_{k_lo+j} - T_{k_lo+j-1}
// (T_{k_lo-1} = 0).  M = the smallest power of two >= the number of outcomes, at least 16.
// Vose's construction then splits the masses over M columns of 2^32 / M words: "small"
// (m < 2^32 / M) and "large" column stacks, both filled in ascending order; pop s from small and
// l from large, column s keeps height m_s and alias l, m_l -= 2^32 / M - m_s, and l goes back on
// the stack its mass now selects; columns left on the large stack are full (the wave computes the
// same table from prefix sums, below).  All integer: the table selects every outcome on exactly
// m_j of the 2^32 words.  A part so small (below about
// 2^-32) that T_0 already reaches 2^32 - 1 has the single outcome 0: every column then holds
// height 0 and alias 0.  The record keeps k_lo << 12 | log2 M << 8 | KIND_ALIAS.
// Each wave walks entries w, w + W, w + 2W, ... (W = waves in the grid), reusing its LDS: a grid
// of one launch per entry held most of its blocks' LDS for waves without an alias part and
// dispatched tens of thousands of blocks that had nothing to do.
constexpr int ALIAS_WAVES = 4;      // waves per 256-thread block
constexpr int ALIAS_BLOCKS = 1024;  // blocks over both parts: 4 per CU (bound by LDS) on 256 CUs

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sums, in pop order (list position n - 1 - k for pop index k), of the deficits
// cap - m (small) or excesses m - cap (large) of the n listed columns: dst[k] for k < n (every
// partial sum is below 2^32).  Each
// lane sums a run of consecutive pop indices, then a wave scan of the run totals offsets them.
__device__ __forceinline__ void scan_pop_order(const uint16_t *list, int n, const uint32_t *m, uint32_t cap,
                                               bool small, uint32_t *dst, int lane) {
  const int per = (n + 63) >> 6;
  const int k0 = min(n, lane * per), k1 = min(n, k0 + per);
  uint32_t tot = 0u;
  for (int k = k0; k < k1; ++k) {
    const uint32_t c = m[list[n - 1 - k]];
    tot += small ? cap - c : c - cap;
  }
  uint32_t x = tot;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, (unsigned)d, 64);
    if (lane >= d) x += y;
  }
  uint32_t run = x - tot;
  for (int k = k0; k < k1; ++k) {
    const uint32_t c = m[list[n - 1 - k]];
    run += small ? cap - c : c - cap;
    dst[k] = run;
  }
}

__device__ __forceinline__ void prep_alias_body(const PrepArgs &a, int i, int part) {
  __shared__ uint32_t m_s[ALIAS_WAVES][ALIAS_COLS];
  __shared__ uint16_t small_s[ALIAS_WAVES][ALIAS_COLS], large_s[ALIAS_WAVES][ALIAS_COLS];
  __shared__ uint32_t D_s[ALIAS_WAVES][ALIAS_COLS + 1], E_s[ALIAS_WAVES][ALIAS_COLS];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (i >= a.E) return;  // whole waves: i is wave-uniform
  // part 0: the entry's count (or its unreddened part); part 1: the reddened part (thinned)
  // (rdesc holds KIND_ZERO for every entry that is not thinned whenever thinning is on)
  // (at F = 1/2 the reddened half reads the unreddened half's table)
  if (part == 0 ? (a.rec[i].kk & KIND_MASK) != KIND_ALIAS
                : a.thin != THIN_TABLE || (a.rdesc[i] & KIND_MASK) != KIND_ALIAS)
    return;
  uint32_t *m = m_s[wv];
  uint16_t *sm = small_s[wv], *lg = large_s[wv];
  for (int j = lane; j < ALIAS_COLS; j += 64) m[j] = 0u;
  wave_lds_sync();
  const double lam = a.lam[i];
  // part 1 exists only for a thinned entry; part 0 of one is its unreddened share (at F = 1/2 the
  // reddened half has the same lambda and reads the same table)
  const bool thin = part == 1 || (a.rec[i].kk & FLAG_THIN) != 0u;
  const double l = !thin ? lam : part == 0 ? lam * (1.0 - a.frac) : lam * a.frac;
  // Every lane runs the recurrence on the same values (a wave issues the same instructions for one
  // lane as for 64), 64 outcomes at a time, and lane j keeps the sum of outcome k0 + j; thresholds and
  // masses are then taken by all lanes at once.  (A decision per outcome kept the chain waiting for
  // scalar reads and branches: 512 x 512 at 10^6 stars per pixel, 10,000 tables up to lambda = 512,
  // 152 -> 68 us; k_prep with the same division, 52,500 entries, 16.3 -> 5.4 us.)
  double pk = exp(-l), F = pk;
  int klo = -1, J = 0;
  bool single = false;
  uint32_t prev = 0u;
  for (int k0 = 0; k0 < KRCP; k0 += 64) {
    double Fl = F;
#pragma unroll 16
    for (int j = 0; j < 64; ++j) {
      if (k0 + j > 0) {
        pk = div_count(pk * l, k0 + j, k_rcp.v[k0 + j]);
        F = F + pk;
      }
      Fl = lane == j ? F : Fl;
    }
    const double t = floor(Fl * 4294967296.0);
    // the first outcome at the last word or more takes the rest of the mass
    const uint64_t last = __ballot(t >= 4294967295.0);
    const int e = last ? (int)__builtin_ctzll(last) : 64;
    const uint32_t T = lane < e ? (uint32_t)t : 0u;
    const uint64_t pos = __ballot(T > 0u);
    if (klo < 0 && pos) klo = k0 + (int)__builtin_ctzll(pos);
    if (klo >= 0) {
      const int j = k0 + lane - klo;
      uint32_t before = (uint32_t)__shfl_up((int)T, 1u, 64);
      if (lane == 0) before = prev;
      if (j >= 0 && j < ALIAS_COLS && lane < e) m[j] = T - before;
      J = k0 + e - klo;
      if (J >= ALIAS_COLS) {  // wider than the table (not reached below ALIAS_MAX)
        if (lane == 0) atomicOr(a.status, STATUS_BAD_LAMBDA);
        J = ALIAS_COLS;
        break;
      }
      const uint32_t ahead = (uint32_t)__shfl((int)T, e > 0 ? e - 1 : 0, 64);
      prev = e > 0 ? ahead : prev;
    }
    if (last) {
      if (klo < 0) {  // all of it (a part below about 2^-32): every word draws the outcome
        klo = k0 + e;
        single = true;
      } else {
        if (lane == 0) m[J] = 0u - prev;  // 2^32 - T_{k-1}; prev >= 1 here (T_{klo} > 0)
        ++J;
      }
      break;
    }
  }
  int bits = 4;
  while ((1 << bits) < J) ++bits;
  if (lane == 0) {
    const uint32_t desc = ((uint32_t)klo << 12) | ((uint32_t)bits << 8) | KIND_ALIAS;
    if (part == 0)
      a.rec[i].kk = desc | (a.rec[i].kk & FLAG_THIN);
    if (part == 1) a.rdesc[i] = desc;
  }
  wave_lds_sync();
  const int M = 1 << bits;
  const uint32_t cap = 1u << (32 - bits);
  uint32_t *out = a.alias + ((size_t)i * 2 + part) * ALIAS_COLS;
  if (single) {  // one outcome: height 0 and alias 0 in every column, n = k_lo always
    for (int j = lane; j < M; j += 64) out[j] = 0u;
    return;
  }
  // stacks in ascending column order: each lane takes one column of every 64, ballots give the
  // positions
  int ns = 0, nl = 0;
  const uint64_t below = (1ull << lane) - 1ull;
  for (int c0 = 0; c0 < M; c0 += 64) {
    const int j = c0 + lane;
    const bool in = j < M;
    const bool is_small = in && m[j] < cap;
    const bool is_large = in && !(m[j] < cap);
    const uint64_t bs = __ballot(is_small), bl = __ballot(is_large);
    if (is_small) sm[ns + __popcll(bs & below)] = (uint16_t)j;
    if (is_large) lg[nl + __popcll(bl & below)] = (uint16_t)j;
    ns += __popcll(bs);
    nl += __popcll(bl);
  }
  wave_lds_sync();
  // Vose's loop pops both lists from the top (highest column first): a large column takes the
  // small columns in pop order until its excess m - cap is used up, then is itself the next small
  // column, taken by the next large one.  With D(i) the deficits cap - m of the first i smalls
  // popped and E(j) the excesses of the first j larges, the i-th small gets the first large j with
  // E(j) >= D(i - 1); the j-th large turns small after the first small a with D(a) > E(j), keeping
  // height cap + E(j) - D(a) and the alias large j + 1; larges that never turn small are full.
  // The sums are exact integers below 2^32 (the total deficit equals the total excess, and that
  // is below M cap = 2^32), so prefix sums and searches give the loop's table exactly, every lane
  // working instead of one walking the loop through LDS.
  uint32_t *Dp = D_s[wv], *Ep = E_s[wv];
  if (lane == 0) Dp[0] = 0u;
  scan_pop_order(sm, ns, m, cap, true, Dp + 1, lane);  // Dp[k] = D(k)
  scan_pop_order(lg, nl, m, cap, false, Ep, lane);     // Ep[j] = E(j + 1)
  wave_lds_sync();
  for (int i = lane; i < ns; i += 64) {  // pop index i: small number i + 1
    const int col = sm[ns - 1 - i];
    const uint32_t need = Dp[i];
    int lo = 0, hi = nl - 1;  // first j with Ep[j] >= need
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (Ep[mid] >= need)
        hi = mid;
      else
        lo = mid + 1;
    }
    const uint32_t al = nl > 0 ? (uint32_t)lg[nl - 1 - lo] : (uint32_t)col;  // nl = 0 only for malformed masses
    out[col] = (m[col] << bits) | al;
  }
  for (int j = lane; j < nl; j += 64) {  // pop index j: large number j + 1
    const int col = lg[nl - 1 - j];
    const uint32_t ex = Ep[j];
    int lo = 1, hi = ns + 1;  // first k in [1, ns] with Dp[k] > ex (ns + 1: none)
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (Dp[mid] > ex)
        hi = mid;
      else
        lo = mid + 1;
    }
    // a column whose alias is itself is full (2^32 / M words, stored as 2^32 / M - 1: the last
    // word then falls to the alias, the column itself)
    uint32_t word = ((cap - 1u) << bits) | (uint32_t)col;
    if (lo <= ns && j + 1 < nl) word = ((cap - (Dp[lo] - ex)) << bits) | (uint32_t)lg[nl - 2 - j];  // Dp[lo] - ex <= cap
    out[col] = word;
  }
}

__device__ __forceinline__ void prep_alias_walk(const PrepArgs &a) {
  const int w = (int)blockIdx.x * ALIAS_WAVES + (int)(threadIdx.x >> 6), stride = (int)gridDim.x * ALIAS_WAVES;
  if (a.alias_list) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)  // the next call's count word
      a.alias_n[(a.gen + 1u) & 1u] = (unsigned long long)(a.gen + 1u) << 32;
    const unsigned long long v = a.alias_n[a.gen & 1u];
    const uint32_t n = (uint32_t)v;
    // the list, when k_prep filled it in this call and it has at most one part per wave of the
    // first grid row (a longer one, spread by arrival order, balanced worse than the entry walk)
    if ((uint32_t)(v >> 32) == a.gen && n <= (uint32_t)stride && n <= 2u * (uint32_t)a.E) {
      if (blockIdx.y == 0 && w < (int)n) {
        const uint32_t it = a.alias_list[w];
        prep_alias_body(a, (int)(it >> 1), (int)(it & 1u));
      }
      return;
    }
  }
  for (int i = w; i < a.E; i += stride) prep_alias_body(a, i, (int)blockIdx.y);  // grid.y: the part
}
__global__ void __launch_bounds__(64 * ALIAS_WAVES) k_prep_alias(PrepArgs a) { prep_alias_walk(a); }
__global__ void __launch_bounds__(64 * ALIAS_WAVES) k_prep_alias_job(const PrepArgs *__restrict__ t, int j) {
  const PrepArgs a = t[j + blockIdx.z];
  prep_alias_walk(a);
}

static dim3 prep_alias_grid(int E, int parts) {
  const int per_part = ALIAS_BLOCKS / parts;
  return dim3((unsigned)std::min((E + ALIAS_WAVES - 1) / ALIAS_WAVES, per_part), (unsigned)parts);
}
hipError_t launch_prep_alias(const PrepArgs &a, hipStream_t s) {
  // grid.y: part 1 (the reddened part of a thinned entry) has a table of its own only when
  // 0 < F < 1 and F != 1/2
  hipLaunchKernelGGL(k_prep_alias, prep_alias_grid(a.E, a.thin == THIN_TABLE ? 2 : 1), dim3(64 * ALIAS_WAVES), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_prep_alias_job(const PrepArgs *table, int j, int n, int E, int parts, hipStream_t s) {
  if (parts != 1 && parts != 2) return hipErrorInvalidValue;
  dim3 grid = prep_alias_grid(E, parts);
  grid.z = (unsigned)n;
  hipLaunchKernelGGL(k_prep_alias_job, grid, dim3(64 * ALIAS_WAVES), 0, s, table, j);
  return hipGetLastError();
}

hipError_t launch_prep(const PrepArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_prep, dim3((a.E + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_prep_job(const PrepArgs *table, int j, int n, int E, hipStream_t s) {
  hipLaunchKernelGGL(k_prep_job, dim3((E + 255) / 256, 1, n), dim3(256), 0, s, table, j);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Sampler.
// ---------------------------------------------------------------------------------------

__device__ __forceinline__ uint32_t low_mask(uint32_t cnt) { return cnt >= 32u ? 0xFFFFFFFFu : ((1u << cnt) - 1u); }

// Reddened stars among n (dust split).  F = 1/2: one bit per star, the first 8 from the
// entry's byte of its 16-entry split block, the rest from (p, i, TAG_SPLIT_X, j) blocks.
// Other fractions: star s compares word s mod 4 of (p, i, TAG_SPLIT_X, s / 4) with fq.
constexpr uint32_t SPLIT_FIRST_BITS = 8;

__device__ __forceinline__ uint32_t split_count(uint32_t n, uint32_t word, uint32_t shift, int mode, uint32_t fq,
                                                uint32_t p, uint32_t i, uint32_t k0, uint32_t k1) {
  if (mode == SPLIT_ALL) return n;
  if (mode == SPLIT_NONE) return 0u;
  uint32_t red = 0;
  if (mode == SPLIT_HALF) {
    // no lane with more than one star (most entries of a sparse field): the byte's first bit
    if (!wave_any(n > 1u)) return n & __builtin_amdgcn_ubfe(word, shift, 1u);
    // no lane with more stars than the byte has bits
    if (!wave_any(n > SPLIT_FIRST_BITS)) return __popc(__builtin_amdgcn_ubfe(word, shift, n));
    // the entry's byte sits at bit `shift` of `word`; its low min(n, 8) bits decide the first stars
    red = __popc(__builtin_amdgcn_ubfe(word, shift, min(n, SPLIT_FIRST_BITS)));
    const uint32_t extra = n > SPLIT_FIRST_BITS ? n - SPLIT_FIRST_BITS : 0u;
    for (uint32_t j = 0; wave_any(extra > 128u * j); ++j) {
      const u4 x = philox10(p, i, TAG_SPLIT_X, j, k0, k1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t base = 128u * j + 32u * (uint32_t)q;
        const uint32_t cnt = extra > base ? min(extra - base, 32u) : 0u;
        red += __popc(word_of(x, q) & low_mask(cnt));
      }
    }
    return red;
  }
  for (uint32_t j = 0; wave_any(n > 4u * j); ++j) {
    const u4 x = philox10(p, i, TAG_SPLIT_X, j, k0, k1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t st = 4u * j + (uint32_t)q;
      red += (n > st && word_of(x, q) < fq) ? 1u : 0u;
    }
  }
  return red;
}

// Poisson count of one table part: desc = k_lo << 12 | log2 M << 8 | KIND_ALIAS (one column of
// the alias table: n = k_lo + (c if r < height_c else alias_c), u = c << (32 - b) | r) or
// KIND_PTRS (transformed rejection on (p, i, tag, j) with the part's constants).
__device__ __forceinline__ uint32_t alias_column_of(uint32_t desc, uint32_t u) { return u >> (32u - ((desc >> 8) & 0xFu)); }
// the count from column word x of the column that u selects
__device__ __forceinline__ uint32_t alias_count(uint32_t desc, uint32_t u, uint32_t x) {
  const uint32_t b = (desc >> 8) & 0xFu;
  const uint32_t c = u >> (32u - b);
  // r < height, both shifted to the top and r's low b bits set: r 2^b + 2^b - 1 < height 2^b + alias (b >= 1)
  return (desc >> 12) + (__builtin_amdgcn_alignbit(u, 0xFFFFFFFFu, 32u - b) < x ? c : (x & ((1u << b) - 1u)));
}

__device__ __forceinline__ uint32_t table_draw(uint32_t desc, uint32_t u, const uint32_t *__restrict__ tab,
                                               const PCMD_CONST PtrsConst *pcp, uint32_t p, uint32_t i, uint32_t tag,
                                               uint32_t k0, uint32_t k1, const float *__restrict__ lnfact,
                                               uint32_t &failed) {
  if ((desc & KIND_MASK) == KIND_ALIAS) return alias_count(desc, u, tab[alias_column_of(desc, u)]);
  const PtrsConst cst = ld_const(pcp);
  return ptrs_draw(cst, p, i, tag, k0, k1, lnfact, failed);
}

// Adds f to acc in the lanes of `mask` only.  Called with all 64 lanes of the wave active (a tile's
// control flow is wave-uniform), which the last instruction restores.  Written out because the
// compiler turns a short divergent branch into selects, and a branch it does keep into additions
// to copies of the sums with moves back.
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

template <int B>
__device__ __forceinline__ void masked_add(double (&acc)[B], const double (&f)[B], uint64_t mask) {
  static_assert(B >= 1 && B <= 4, "bands");
  if constexpr (B == 1)
    asm volatile("s_mov_b64 exec, %1\n\tv_add_f64 %0, %0, %2\n\ts_mov_b64 exec, -1" : "+v"(acc[0]) : "s"(mask), "s"(f[0]));
  else if constexpr (B == 2)
    asm volatile("s_mov_b64 exec, %2\n\tv_add_f64 %0, %0, %3\n\tv_add_f64 %1, %1, %4\n\ts_mov_b64 exec, -1"
                 : "+v"(acc[0]), "+v"(acc[1])
                 : "s"(mask), "s"(f[0]), "s"(f[1]));
  else if constexpr (B == 3)
    asm volatile("s_mov_b64 exec, %3\n\tv_add_f64 %0, %0, %4\n\tv_add_f64 %1, %1, %5\n\tv_add_f64 %2, %2, %6\n\t"
                 "s_mov_b64 exec, -1"
                 : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2])
                 : "s"(mask), "s"(f[0]), "s"(f[1]), "s"(f[2]));
  else
    asm volatile("s_mov_b64 exec, %4\n\tv_add_f64 %0, %0, %5\n\tv_add_f64 %1, %1, %6\n\tv_add_f64 %2, %2, %7\n\t"
                 "v_add_f64 %3, %3, %8\n\ts_mov_b64 exec, -1"
                 : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
                 : "s"(mask), "s"(f[0]), "s"(f[1]), "s"(f[2]), "s"(f[3]));
}

// acc += n f (f wave-uniform), the sum staying in its register: where paths join, the compiler's own
// form left six register moves per path.
__device__ __forceinline__ void fma_in_place(double &acc, double n, double f) {
  asm volatile("v_fma_f64 %0, %1, %2, %0" : "+v"(acc) : "v"(n), "s"(f));
}

// The arguments again, for fields read once per group of entries or less: loaded there through the
// scalar cache.  The compiler cannot see that the pointer is the same, so it does not load them
// ahead of the loop, where they would push the loop's own values out of the scalar registers into
// vector lanes (a vector instruction for each word read back).
template <typename T>
__device__ __forceinline__ const PCMD_CONST T *rare(const PCMD_CONST T *p) {
  asm volatile("" : "+s"(p));
  return p;
}

// Values held in scalar registers from here on: the compiler otherwise loads them again, each time
// behind a wait, where they are used.
template <typename T>
__device__ __forceinline__ void keep_scalar(const PCMD_CONST T *&p) {
  asm volatile("" : "+s"(p));
}

__device__ __forceinline__ void keep_scalar(uint32_t &a, uint32_t &b) { asm volatile("" : "+s"(a), "+s"(b)); }
template <int B>
__device__ __forceinline__ void keep_scalar(double (&f)[B]) {
#pragma unroll
  for (int b = 0; b < B; ++b) asm volatile("" : "+s"(f[b]));
}

// Slice `chunk` of nchunks takes the 16-entry blocks chunk, chunk + nchunks, chunk + 2 nchunks,
// ...: every slice then spans all isochrones and masses, so slices cost about the same (runs of
// consecutive entries differ in cost several-fold: high-lambda low-mass stars cluster at the start
// of each isochrone).  The j-th group of GRP entries of the slice is group slice_group(j) of the
// table.  Calls body(group, flags) for the slice's groups with a flag of `want`.
//
// Lane l reads the flags of the slice's group jb + l: one vector load finds the groups with
// entries to draw among the next 64, where one dependent scalar load per group kept a wave waiting
// through runs of groups with nothing to draw (pruned isochrones; the hybrid sampler's block-rule
// entries).
template <typename F>
__device__ __forceinline__ void for_groups(const GroupRec *grp, int E, int nchunks, int chunk, uint32_t want, F &&body) {
  static_assert(GRP == 8, "two groups per 16-entry block");
  const int ngrp = entries_padded(E) / GRP;
  const int stride = nchunks * (16 / GRP);
  auto slice_group = [&](int j) { return chunk * (16 / GRP) + (j >> 1) * stride + (j & 1); };
  const int lane = (int)(threadIdx.x & 63u);
  for (int jb = 0; slice_group(jb) < ngrp; jb += 64) {
    const int gl = slice_group(jb + lane);
    const uint32_t fl = gl < ngrp ? grp[gl].flags : 0u;
    for (uint64_t pend = __ballot((fl & want) != 0u); pend != 0ull; pend &= pend - 1ull) {
      const int lsel = (int)__builtin_ctzll(pend);  // wave-uniform
      // slice_group(jb + lsel), read from lane lsel: one vector instruction instead of seven scalar
      body(__builtin_amdgcn_readlane(gl, lsel), (uint32_t)__builtin_amdgcn_readlane((int)fl, lsel));
    }
  }
}

// Adds the counts n, of them red reddened, of an entry with fluxes f.
template <int B, int S>
__device__ __forceinline__ void add_counts(double (&acc_c)[B], double (&acc_r)[B], const double (&f)[B], uint32_t n,
                                           uint32_t red) {
  // the unreddened stream has a star whenever the entry has one, nearly always: added without a
  // test (zero counts add exact zeros); the reddened stream is skipped when no lane has a
  // reddened star
  const double dc = (double)(n - red);
#pragma unroll
  for (int b = 0; b < B; ++b) fma_in_place(acc_c[b], dc, f[b]);
  if (S == 2 && wave_any(red != 0u)) {
    const double dr = (double)red;
#pragma unroll
    for (int b = 0; b < B; ++b) fma_in_place(acc_r[b], dr, f[b]);
  }
}

// PASS (SamplePass): PASS_ALL draws every entry, the thinned ones (FLAG_THIN: two independent
// parts, k_prep's choice under a split 0 < F < 1) inline; PASS_MAIN leaves the thinned ones to
// sample_thin_tile.
//
// Bound by vector-instruction issue (90% of cycles), of which two Philox blocks per eight draws (8
// instructions a draw) are the part that no layout can drop.  What the loop does beyond them is
// kept small: one compare per entry, whose lane masks also drive the additions; nothing that the
// loop uses spilled to vector lanes.  256 x 256 pixels, 52,500 entries, 3 bands, 10^3.4 stars per
// pixel: 675 -> 587 million wave instructions, 1481 -> 1223 us; 512 x 512 at 10^6: 7.18 -> 6.0 ms.
template <int B, int S, bool DBG, int PASS>
__device__ __forceinline__ void sample_tile(const PCMD_CONST SampleArgs *ap, uint32_t p, int chunk) {
  const GroupRec *grp = ap->grp;
  const int E = ap->E, nchunks = ap->nchunks;
  const uint32_t k0 = ap->k0, k1 = ap->k1;
  bool live, dbg = false;
  {
    const PCMD_CONST SampleArgs *ca = rare(ap);
    live = p < (uint32_t)ca->npx;
    if (DBG) dbg = live && (int64_t)p >= ca->px0 && (int64_t)p < ca->px1;
  }
  auto write_dbg = [&](uint32_t i, uint32_t n, uint32_t red) {
    if (DBG && dbg) {
      const PCMD_CONST SampleArgs *ca = rare(ap);
      const size_t o = (size_t)((int64_t)p - ca->px0) * (size_t)ca->E + i;
      ca->dbg_counts[o] = n;
      if (ca->dbg_red) ca->dbg_red[o] = red;
    }
  };

  double acc_c[B], acc_r[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    acc_c[b] = 0.0;
    acc_r[b] = 0.0;
  }
  uint32_t ptrs_failed = 0u;  // per lane, kept in a vector register

  {
    const int split_mode = S == 2 ? ap->split_mode : SPLIT_NONE;
    // the split bits of 16-entry block split_blk; where F is not 1/2 (split_blk = NO_SPLIT) all ones
    // for F = 1, else zero
    constexpr int NO_SPLIT = -2;
    int split_blk = split_mode == SPLIT_HALF ? -1 : NO_SPLIT;
    const uint32_t fixed = split_mode == SPLIT_ALL ? 0xFFFFFFFFu : 0u;
    u4 sw{fixed, fixed, fixed, fixed};
    auto split_word = [&](int gi, int h) {  // the word of quad h of group gi
      const uint32_t lo = h ? sw.y : sw.x, hi = h ? sw.w : sw.z;
      return gi & 1 ? hi : lo;
    };
    // The entries drawn by inversion.
    for_groups(grp, E, nchunks, chunk, GRP_INV, [&](int gi, uint32_t flags) {
      const u4 wa = philox10(p, (uint32_t)(2 * gi), TAG_MAIN, 0u, k0, k1);
      const u4 wb = philox10(p, (uint32_t)(2 * gi + 1), TAG_MAIN, 0u, k0, k1);
      // the first thresholds are loaded only now: held across the Philox rounds they pushed the
      // scalar register file into spilling inside this loop
      __builtin_amdgcn_sched_barrier(0);
      // the lanes with a star, per entry (the threshold of a dense entry, which is always counted, or
      // of one not drawn by inversion is never exceeded): at small lambda most groups end after two Philox blocks and eight compares,
      // without touching the entry records
      const PCMD_CONST GroupRec *gr = (const PCMD_CONST GroupRec *)rare(ap)->grp + gi;
      const u32x8 w = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
      uint64_t hit[GRP], any = 0ull;
#pragma unroll
      for (int q = 0; q < GRP; ++q) any |= hit[q] = __ballot(w[q] > gr->t0m1[q]);
      uint32_t counted = flags / GRP_DENSE_ENTRY;
      if (any == 0ull && counted == 0u) return;
      // the split bits of the group's 16-entry block: a group with a star almost always has one to
      // split, and the two groups of a block share them
      if (S == 2 && split_blk != NO_SPLIT && split_blk != (gi >> 1)) {
        sw = philox10(p, (uint32_t)(gi >> 1), TAG_SPLIT, 0u, k0, k1);
        split_blk = gi >> 1;
      }
      const uint32_t sq0 = split_word(gi, 0), sq1 = split_word(gi, 1);
      const PCMD_CONST EntryRec *rg = (const PCMD_CONST EntryRec *)rare(ap)->rec + gi * GRP;
      keep_scalar(rg);
      // Entries of which no lane has three stars first, then the counted ones: as the two branches
      // of one loop, the compiler moved all sums at the end of either.
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        if (hit[q] == 0ull) continue;
        const uint32_t u = w[q];
        // thresholds and fluxes behind one wait
        uint32_t t1m1 = rg[q].T[1], t2m1 = rg[q].T[2];
        double fv[B];
#pragma unroll
        for (int b = 0; b < B; ++b) fv[b] = rg[q].fl[b];
        keep_scalar(t1m1, t2m1);
        keep_scalar(fv);
        const uint32_t word = q < 4 ? sq0 : sq1;
        const uint64_t two = __ballot(u > t1m1);
        if (PASS == PASS_ALL || (two != 0ull && wave_any(u > t2m1))) {
          counted |= 1u << q;
          continue;
        }
        // No lane has three stars of the entry, which holds for most entries below lambda ~ 0.3.
        // The lanes with a first and a second star add the flux to one of their two streams under
        // the execution mask: six additions each, where counts cost two conversions, six
        // multiply-adds and the integer steps between.  PASS_ALL (one word per star) takes counts.
        const uint64_t red = S == 2 ? __ballot((word & (1u << (8 * (q & 3)))) != 0u) & hit[q] : 0ull;
        masked_add<B>(acc_c, fv, hit[q] & ~red);
        if (S == 2) masked_add<B>(acc_r, fv, red);
        uint64_t red2 = 0ull;
        if (two != 0ull) {
          red2 = S == 2 ? __ballot((word & (2u << (8 * (q & 3)))) != 0u) & two : 0ull;
          masked_add<B>(acc_c, fv, two & ~red2);
          if (S == 2) masked_add<B>(acc_r, fv, red2);
        }
        if (DBG)
          write_dbg((uint32_t)(gi * GRP + q),
                    (__builtin_amdgcn_inverse_ballot_w64(hit[q]) ? 1u : 0u) + (__builtin_amdgcn_inverse_ballot_w64(two) ? 1u : 0u),
                    (__builtin_amdgcn_inverse_ballot_w64(red) ? 1u : 0u) + (__builtin_amdgcn_inverse_ballot_w64(red2) ? 1u : 0u));
      }
      if (counted == 0u) return;
#pragma unroll
      for (int q = 0; q < GRP; ++q) {
        if (!(counted & (1u << q))) continue;
        const uint32_t i = (uint32_t)(gi * GRP + q);
        const uint32_t u = w[q];
        EntryHead rq = ld_const((const PCMD_CONST EntryHead *)(rg + q));
        double fv[B];
#pragma unroll
        for (int b = 0; b < B; ++b) fv[b] = rg[q].fl[b];
        keep_scalar(fv);
        const uint32_t word = q < 4 ? sq0 : sq1;
        // n = #{k < K : T_k <= u}, walking up while any lane of the wave is still above
        uint32_t n = (u > rq.T[0] ? 1u : 0u) + (u > rq.T[1] ? 1u : 0u);
        uint32_t c = u > rq.T[2] ? 1u : 0u;
        if (wave_any(c != 0u)) {
          n += c;
          const uint32_t K = rq.kk >> 8;
          const size_t ep = (size_t)entries_padded(E);
          const PCMD_CONST uint32_t *t = (const PCMD_CONST uint32_t *)rare(ap)->thr + i + 3 * ep;  // threshold k at [k EP]
          for (uint32_t k = 3; k < K; ++k, t += ep) {
            c = u >= *t ? 1u : 0u;
            if (!wave_any(c != 0u)) break;
            n += c;
          }
        }
        uint32_t red = 0u;
        if (S == 2) {
          const uint32_t q_split = PASS == PASS_ALL ? rare(ap)->split_q : 0u;
          red = split_count(n, word, 8u * (uint32_t)(q & 3), split_mode, q_split, p, i, k0, k1);
        }
        add_counts<B, S>(acc_c, acc_r, fv, n, red);
        write_dbg(i, n, red);
      }
    });
    // The table entries (in a loop of their own, so that their code and operands stay out of the
    // one above): slot 0 holds the count (or, thinned, the unreddened part), slot 1 the reddened
    // part, each an alias column read or a rejection draw.
    constexpr uint32_t want = PASS == PASS_ALL ? GRP_TABLE | GRP_THIN : GRP_TABLE;
    for_groups(grp, E, nchunks, chunk, want, [&](int gi, uint32_t flags) {
      const uint32_t tab = flags / GRP_TABLE_ENTRY | (PASS == PASS_ALL ? flags / GRP_THIN_ENTRY : 0u);
      const PCMD_CONST SampleArgs *ca = rare(ap);
      const PCMD_CONST EntryRec *rec = (const PCMD_CONST EntryRec *)ca->rec;
      const PCMD_CONST PtrsConst *pc = (const PCMD_CONST PtrsConst *)ca->pc;
      const uint32_t *alias = ca->alias;
      const float *lnfact = ca->lnfact;
      if (S == 2 && split_blk != NO_SPLIT && split_blk != (gi >> 1)) {
        sw = philox10(p, (uint32_t)(gi >> 1), TAG_SPLIT, 0u, k0, k1);
        split_blk = gi >> 1;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (((tab >> (4 * h)) & 0xFu) == 0u) continue;
        const u4 w = philox10(p, (uint32_t)(2 * gi + h), TAG_MAIN, 0u, k0, k1);
        const uint32_t sq = split_word(gi, h);
        u4 wr{0u, 0u, 0u, 0u};  // thinned entries: the quad's reddened-part words
        if (S == 2 && PASS == PASS_ALL && ((flags / GRP_THIN_ENTRY >> (4 * h)) & 0xFu) != 0u)
          wr = philox10(p, (uint32_t)(2 * gi + h), TAG_RED, 0u, k0, k1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (((tab >> (4 * h + q)) & 1u) == 0u) continue;
          const uint32_t i = (uint32_t)(gi * GRP + 4 * h + q);
          const uint32_t kk = rec[i].kk;
          uint32_t n = table_draw(kk, word_of(w, q), alias + (size_t)i * 2 * ALIAS_COLS, pc + 2 * (size_t)i, p, i, TAG_PTRS, k0,
                                  k1, lnfact, ptrs_failed);
          uint32_t red = 0u;
          if (S == 2 && PASS == PASS_ALL && (kk & FLAG_THIN)) {
            const uint32_t d = ((const PCMD_CONST uint32_t *)ca->rdesc)[i];
            red = table_draw(d, word_of(wr, q), alias + ((size_t)i * 2 + 1) * ALIAS_COLS, pc + 2 * (size_t)i + 1, p, i,
                             TAG_PTRS_RED, k0, k1, lnfact, ptrs_failed);
            n += red;
          } else if (S == 2 && wave_any(n != 0u)) {
            red = split_count(n, sq, 8u * (uint32_t)q, ca->split_mode, ca->split_q, p, i, k0, k1);
          }
          if (!wave_any(n != 0u)) continue;
          const PCMD_CONST double *f = rec[i].fl;
          double fv[B];
#pragma unroll
          for (int b = 0; b < B; ++b) fv[b] = f[b];
          add_counts<B, S>(acc_c, acc_r, fv, n, red);
          write_dbg(i, n, red);
        }
      }
    });
  }
  const PCMD_CONST SampleArgs *ca = rare(ap);
  if (wave_any(ptrs_failed != 0u) && (threadIdx.x & 63) == 0) atomicOr(ca->status, STATUS_PTRS_RETRY);
  if (!live) return;
  const size_t plane = (size_t)ca->npx;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    float *pc = ca->part + ((size_t)(chunk * S + 0) * B + b) * plane + p;
    float *pr = ca->part + ((size_t)(chunk * S + 1) * B + b) * plane + p;
    *pc = (float)acc_c[b];
    if (S == 2) *pr = (float)acc_r[b];
  }
}

// The thinned entries of a tile (PASS_THIN: F = 1/2), added to the partial sums that PASS_MAIN stored:
// a pass of its own, so that the thinning code (live state that slows the common path) is not in the
// main pass.  The two halves of an entry have one lambda, so one rule and one table serve both.
//
// Bound by vector-instruction issue: per entry two words of Philox (17 instructions), two column reads
// and counts (8 each) and the additions.  The column reads of a quad are issued before the first is used;
// rejection draws (halves from ALIAS_MAX on) are in one place, where sixteen inlined copies made the code
// larger than the instruction cache.  4096 x 4096
// pixels, 55 thinned entries: 1969 -> 1390 us; 512 x 512, about 10,000 of them: 4.50 -> 2.99 ms.
template <int B, bool DBG>
__device__ __forceinline__ void sample_thin_tile(const PCMD_CONST SampleArgs *ap, uint32_t p, int chunk) {
  const int E = ap->E, nchunks = ap->nchunks;
  const uint32_t k0 = ap->k0, k1 = ap->k1;
  const bool live = p < (uint32_t)ap->npx;
  double acc_c[B], acc_r[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    acc_c[b] = 0.0;
    acc_r[b] = 0.0;
  }
  uint32_t ptrs_failed = 0u;  // per lane, kept in a vector register
  auto add = [&](const PCMD_CONST EntryRec *r, uint32_t i, uint32_t nc, uint32_t red) {
    double fv[B];
#pragma unroll
    for (int b = 0; b < B; ++b) fv[b] = r->fl[b];
    const double dc = (double)nc, dr = (double)red;  // a lane without stars adds exact zeros
#pragma unroll
    for (int b = 0; b < B; ++b) fma_in_place(acc_c[b], dc, fv[b]);
#pragma unroll
    for (int b = 0; b < B; ++b) fma_in_place(acc_r[b], dr, fv[b]);
    if (DBG) {
      const PCMD_CONST SampleArgs *ca = rare(ap);
      if (live && (int64_t)p >= ca->px0 && (int64_t)p < ca->px1) {
        const size_t o = (size_t)((int64_t)p - ca->px0) * (size_t)ca->E + i;
        ca->dbg_counts[o] = nc + red;
        if (ca->dbg_red) ca->dbg_red[o] = red;
      }
    }
  };
  for_groups(ap->grp, E, nchunks, chunk, GRP_THIN, [&](int gi, uint32_t flags) {
    const PCMD_CONST EntryRec *rec = (const PCMD_CONST EntryRec *)rare(ap)->rec + gi * GRP;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t thin = (flags / GRP_THIN_ENTRY >> (4 * h)) & 0xFu;
      if (thin == 0u) continue;
      uint32_t kk[4], tab = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) kk[q] = rec[4 * h + q].kk;
#pragma unroll
      for (int q = 0; q < 4; ++q) tab |= (kk[q] & KIND_MASK) == KIND_ALIAS ? 1u << q : 0u;
      tab &= thin;
      if (tab != 0u) {
        const uint32_t *alias = rare(ap)->alias + (size_t)(gi * GRP + 4 * h) * (2 * ALIAS_COLS);
        const u4 w = philox10(p, (uint32_t)(2 * gi + h), TAG_MAIN, 0u, k0, k1);
        const u4 wr = philox10(p, (uint32_t)(2 * gi + h), TAG_RED, 0u, k0, k1);
        uint32_t x0[4], x1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          x0[q] = 0u;
          x1[q] = 0u;
          if (tab >> q & 1u) {
            // byte offsets in 32 bits from a scalar base
            const char *col = (const char *)(alias + q * (2 * ALIAS_COLS));
            x0[q] = *(const uint32_t *)(col + (alias_column_of(kk[q], word_of(w, q)) << 2));
            x1[q] = *(const uint32_t *)(col + (alias_column_of(kk[q], word_of(wr, q)) << 2));
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (tab >> q & 1u)
            add(rec + 4 * h + q, (uint32_t)(gi * GRP + 4 * h + q), alias_count(kk[q], word_of(w, q), x0[q]),
                alias_count(kk[q], word_of(wr, q), x1[q]));
      }
#pragma unroll 1
      for (uint32_t rej = thin & ~tab; rej != 0u; rej &= rej - 1u) {
        const int q = 4 * h + (int)__builtin_ctz(rej);
        const uint32_t i = (uint32_t)(gi * GRP + q);
        const PCMD_CONST SampleArgs *ca = rare(ap);
        const PtrsConst c = ld_const((const PCMD_CONST PtrsConst *)ca->pc + 2 * (size_t)i);
        uint32_t n[2] = {0u, 0u};
#pragma unroll 1
        for (int part = 0; part < 2; ++part) {
          n[1] = n[0];
          n[0] = ptrs_draw(c, p, i, part ? TAG_PTRS : TAG_PTRS_RED, k0, k1, ca->lnfact, ptrs_failed);
        }
        add(rec + q, i, n[0], n[1]);
      }
    }
  });
  const PCMD_CONST SampleArgs *ca = rare(ap);
  if (wave_any(ptrs_failed != 0u) && (threadIdx.x & 63) == 0) atomicOr(ca->status, STATUS_PTRS_RETRY);
  if (!live) return;
  const size_t plane = (size_t)ca->npx;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    float *pc = ca->part + ((size_t)(chunk * 2 + 0) * B + b) * plane + p;
    float *pr = ca->part + ((size_t)(chunk * 2 + 1) * B + b) * plane + p;
    // exact zeros change nothing: a slice without thinned stars skips
    if (acc_c[b] != 0.0) *pc = (float)((double)*pc + acc_c[b]);
    if (acc_r[b] != 0.0) *pr = (float)((double)*pr + acc_r[b]);
  }
}

// The scalar unit issues about as many instructions as the vector unit here, so scalar-load
// latency is hidden by other waves: the sampler kernels are held to the 80 scalar registers that
// allow 8 waves per SIMD (the compiler moves the rest into vector-register lanes), which measured
// faster than 7 waves without those moves.
template <int B, int S, bool DBG, int PASS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_sample(SampleArgs a) {
  if (PASS == PASS_THIN && a.thin_seen && *(const PCMD_CONST uint32_t *)a.thin_seen != a.gen) return;  // nothing thinned
  const int nblk_px = (a.npx + 255) >> 8;
  const int chunk = blockIdx.x / nblk_px;
  const uint32_t p = (uint32_t)((blockIdx.x - chunk * nblk_px) * 256 + threadIdx.x);
  // the arguments where the launch put them (the kernel's only parameter)
  const PCMD_CONST SampleArgs *ap = (const PCMD_CONST SampleArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if constexpr (PASS == PASS_THIN)
    sample_thin_tile<B, DBG>(ap, p, chunk);
  else
    sample_tile<B, S, DBG, PASS>(ap, p, chunk);
}

template <int B, int PASS>
static void launch_sample_pass(const SampleArgs &a, dim3 grid, hipStream_t s) {
  const bool dbg = a.dbg_counts != nullptr;
  if (a.S == 2 && dbg)
    hipLaunchKernelGGL((k_sample<B, 2, true, PASS>), grid, dim3(256), 0, s, a);
  else if (a.S == 2)
    hipLaunchKernelGGL((k_sample<B, 2, false, PASS>), grid, dim3(256), 0, s, a);
  else if (dbg)
    hipLaunchKernelGGL((k_sample<B, 1, true, PASS_MAIN>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_sample<B, 1, false, PASS_MAIN>), grid, dim3(256), 0, s, a);
}

// Thinning of every table entry (0 < F < 1, F != 1/2): one pass with the thinned entries inline.
// F = 1/2 (only entries at lambda >= LAM_THIN_HALF thinned): the main pass, then the thinned
// entries' pass.  Otherwise nothing is thinned: the main pass alone.
template <int B>
static hipError_t launch_sample_b(const SampleArgs &a, hipStream_t s) {
  const int nblk_px = (a.npx + 255) / 256;
  dim3 grid((unsigned)(nblk_px * a.nchunks));
  const int tm = a.S == 2 ? thin_mode_of_split(a.split_mode) : THIN_NONE;
  if (tm == THIN_TABLE) {
    launch_sample_pass<B, PASS_ALL>(a, grid, s);
  } else {
    launch_sample_pass<B, PASS_MAIN>(a, grid, s);
    if (tm == THIN_HALF_HIGH) {
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      launch_sample_pass<B, PASS_THIN>(a, grid, s);
    }
  }
  return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs &a, hipStream_t s) {
  switch (a.B) {
    case 1: return launch_sample_b<1>(a, s);
    case 2: return launch_sample_b<2>(a, s);
    case 3: return launch_sample_b<3>(a, s);
    case 4: return launch_sample_b<4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------------------
// Persistent batched sampler.  Workgroups take tiles (job, pixel block, chunk) from one atomic
// counter until none is left; jobs appear in the table in execution order (the host puts the
// most expensive first) and each job's tiles are contiguous items, pixel block fastest.  Every
// tile is computed exactly as by k_sample, so the schedule never changes a result.
// ---------------------------------------------------------------------------------------
__global__ void k_reset_counter(uint32_t *c) { *c = 0u; }

hipError_t launch_reset_counter(uint32_t *counter, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, s, counter);
  return hipGetLastError();
}

// The job owning an item: the last one with item0 <= item (binary search over the table).
__device__ __forceinline__ int job_of_item(const PCMD_CONST BatchSampleJob *cj, int n_jobs, int item) {
  int lo = 0, hi = n_jobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cj[mid].item0 <= item)
      lo = mid;
    else
      hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Persistent batched sampler: every wave takes (job, 64-pixel block, slice) items from one
// atomic counter until none is left, so no wave waits for another (items of one job are
// consecutive; jobs come in the host's order).
template <int B>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) k_sample_persistent(const BatchSampleJob *__restrict__ jobs, int n_jobs,
                                                           int total_items, uint32_t *__restrict__ counter) {
  const PCMD_CONST BatchSampleJob *cj = (const PCMD_CONST BatchSampleJob *)jobs;
  const uint32_t lane = threadIdx.x & 63u;
  for (;;) {
    uint32_t got = 0u;
    if (lane == 0) got = atomicAdd(counter, 1u);
    const int item = (int)__builtin_amdgcn_readfirstlane(got);
    if (item >= total_items) break;
    const int j = job_of_item(cj, n_jobs, item);
    const int local = item - cj[j].item0;
    const int pblocks = cj[j].pblocks;  // 64-pixel blocks of the job
    const int chunk = local / pblocks;
    const int pblk = local - chunk * pblocks;
    const PCMD_CONST SampleArgs *ap = &cj[j].a;
    // batch jobs always carry two streams; F = 1/2 jobs draw their thinned entries afterwards in
    // a launch of their own (k_sample_thin_jobs), as pcmd_simulate does
    if (thin_mode_of_split(ap->split_mode) == THIN_TABLE)
      sample_tile<B, 2, false, PASS_ALL>(ap, (uint32_t)(pblk * 64) + lane, chunk);
    else
      sample_tile<B, 2, false, PASS_MAIN>(ap, (uint32_t)(pblk * 64) + lane, chunk);
  }
}

// The thinned entries' pass of a batch: a wave takes one (job, 64-pixel block, slice) item of the persistent
// sampler's table; items of jobs that are not at F = 1/2, or whose k_prep thinned nothing, return on a few
// scalar loads.  (A launch per job left the chip idle at each one's end: 24 uneven jobs 2.85 -> 2.61 ms.)
// Held to 8 waves per SIMD like the other sampler kernels.
template <int B>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_sample_thin_jobs(const BatchSampleJob *__restrict__ jobs, int n_jobs, int first_item, int total_items) {
  const PCMD_CONST BatchSampleJob *cj = (const PCMD_CONST BatchSampleJob *)jobs;
  const int item = first_item + __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (item >= total_items) return;
  const int j = job_of_item(cj, n_jobs, item);
  const PCMD_CONST SampleArgs *ap = &cj[j].a;
  if (thin_mode_of_split(ap->split_mode) != THIN_HALF_HIGH) return;
  if (ap->thin_seen && *(const PCMD_CONST uint32_t *)ap->thin_seen != ap->gen) return;  // nothing thinned
  const int local = item - cj[j].item0, pblocks = cj[j].pblocks, chunk = local / pblocks;
  sample_thin_tile<B, false>(ap, (uint32_t)((local - chunk * pblocks) * 64) + (threadIdx.x & 63u), chunk);
}

// A grid dimension holds fewer than 2^32 threads, 64 to an item: five 4096 x 4096 jobs of 52,500 entries
// have more items than that.
constexpr int THIN_LAUNCH_ITEMS = 1 << 25;

template <int B>
static hipError_t launch_sample_thin_jobs_b(const BatchSampleJob *jobs, int n_jobs, int total_items, hipStream_t s) {
  for (int64_t first = 0; first < total_items; first += THIN_LAUNCH_ITEMS) {
    const int64_t n = std::min<int64_t>(total_items - first, THIN_LAUNCH_ITEMS);
    hipLaunchKernelGGL(k_sample_thin_jobs<B>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, jobs, n_jobs, (int)first,
                       (int)(first + n));
  }
  return hipGetLastError();
}
hipError_t launch_sample_thin_jobs(const BatchSampleJob *jobs, int n_jobs, int total_items, int B, hipStream_t s) {
  switch (B) {
    case 1: return launch_sample_thin_jobs_b<1>(jobs, n_jobs, total_items, s);
    case 2: return launch_sample_thin_jobs_b<2>(jobs, n_jobs, total_items, s);
    case 3: return launch_sample_thin_jobs_b<3>(jobs, n_jobs, total_items, s);
    case 4: return launch_sample_thin_jobs_b<4>(jobs, n_jobs, total_items, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_sample_persistent(const BatchSampleJob *jobs, int n_jobs, int total_items, int B, uint32_t *counter,
                                    int n_workgroups, hipStream_t s) {
  dim3 grid((unsigned)n_workgroups);
  switch (B) {
    case 1: hipLaunchKernelGGL(k_sample_persistent<1>, grid, dim3(256), 0, s, jobs, n_jobs, total_items, counter); break;
    case 2: hipLaunchKernelGGL(k_sample_persistent<2>, grid, dim3(256), 0, s, jobs, n_jobs, total_items, counter); break;
    case 3: hipLaunchKernelGGL(k_sample_persistent<3>, grid, dim3(256), 0, s, jobs, n_jobs, total_items, counter); break;
    case 4: hipLaunchKernelGGL(k_sample_persistent<4>, grid, dim3(256), 0, s, jobs, n_jobs, total_items, counter); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Slice reduction + epilogue: F_b = 10^(-0.4 mu_d) (F_clr_b + F_red_b 10^(-0.4 R_b E_p)).
// The partials of all slices are loaded in batches of eight before they are added, in ascending
// slice order (the order fixes the rounding).  Small images take a thread per (band, pixel), to
// have enough waves for the memory's latency; from REDUCE_WIDE pixels on (1,024 blocks, four on
// every CU) a thread takes all the bands of its pixel, so that the pixel's dust screen (a Philox
// block, Box-Muller and a power) is drawn once.  4096 x 4096 x 3 with a drawn screen, two
// slices: 510 -> 344 us, 3.0 TB/s; 256 x 256 x 3, 11 slices, a batch job: 35 -> 25 us.
// ---------------------------------------------------------------------------------------
constexpr int RED_BATCH = 8;
constexpr int REDUCE_WIDE = 262144;

__device__ __forceinline__ void reduce_body(const ReduceArgs &a, int p) {
  const bool wide = a.npx >= REDUCE_WIDE;
  const int b0 = wide ? 0 : blockIdx.y, b1 = wide ? a.B : b0 + 1;
  if (p >= a.npx) return;
  const size_t plane = (size_t)a.npx;
  const size_t step = (size_t)a.S * a.B * plane;  // from one slice to the next
  double ebv = 0.0;
  if (a.dust_model == PCMD_DUST_SCREEN) {
    ebv = exp10_any(a.dust_mu);
  } else if (a.dust_model != PCMD_DUST_NONE) {
    const u4 w = philox10((uint32_t)p, 0u, TAG_DUST, 0u, a.k0, a.k1);
    ebv = exp10_any(a.dust_mu + a.dust_sigma * box_muller(w.x, w.y));
  }
  for (int b = b0; b < b1; ++b) {
    const float *pc = a.part + (size_t)b * plane + p;
    const float *pr = pc + (size_t)a.B * plane;  // reddened stream (S == 2)
    double c = 0.0, r = 0.0;
    int ch = 0;
    for (; ch + RED_BATCH <= a.nchunks; ch += RED_BATCH) {
      float xc[RED_BATCH], xr[RED_BATCH];
#pragma unroll
      for (int k = 0; k < RED_BATCH; ++k) {
        xc[k] = pc[(size_t)(ch + k) * step];
        xr[k] = a.S == 2 ? pr[(size_t)(ch + k) * step] : 0.f;
      }
#pragma unroll
      for (int k = 0; k < RED_BATCH; ++k) {
        c += (double)xc[k];
        r += (double)xr[k];
      }
    }
    for (; ch < a.nchunks; ++ch) {
      c += (double)pc[(size_t)ch * step];
      if (a.S == 2) r += (double)pr[(size_t)ch * step];
    }
    const double F = a.dist * (a.dust_model == PCMD_DUST_NONE ? c + r : c + r * exp10_any(-0.4 * a.dust_R[b] * ebv));
    a.F[(size_t)b * plane + p] = (float)F;
  }
}

__global__ void __launch_bounds__(256) k_reduce(ReduceArgs a) { reduce_body(a, blockIdx.x * blockDim.x + threadIdx.x); }
// The jobs j + blockIdx.z, as in k_prep_job.  The record stays in memory: its uniform words are scalar loads,
// and a copy indexed by the band would lie in scratch.
__global__ void __launch_bounds__(256) k_reduce_job(const ReduceArgs *__restrict__ t, int j) {
  reduce_body(t[j + blockIdx.z], blockIdx.x * blockDim.x + threadIdx.x);
}

bool reduce_wide(int npx) { return npx >= REDUCE_WIDE; }

hipError_t launch_reduce(const ReduceArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3((a.npx + 255) / 256, reduce_wide(a.npx) ? 1 : a.B), dim3(256), 0, s, a);
  return hipGetLastError();
}
// n jobs on one side of REDUCE_WIDE, the largest of npx_max pixels
hipError_t launch_reduce_job(const ReduceArgs *table, int j, int n, int npx_max, int B, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_job, dim3((npx_max + 255) / 256, reduce_wide(npx_max) ? 1 : B, n), dim3(256), 0, s, table, j);
  return hipGetLastError();
}

}  // namespace pcmd
