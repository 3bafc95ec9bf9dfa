// Ranking inside one workgroup (gfx950), shared by the kernels that rank a sequence's slots: keys in registers, Eq. 4 as a threshold
// found by narrowing histograms, places of the kept slots.  Not part of the public ABI.
#pragma once

#include "adsa_device.h"
#include "adsa_internal.h"
#include "adsa_partition.h"

namespace adsa {
namespace {

constexpr int kBins = 512, kBinBits = 9;

// LDS of one ranking workgroup (9 KB).
struct RankShared {
  uint32_t hist[4][kBins];           // one histogram per narrowing step: 32-bit keys, 9 bits a step
  uint32_t list[kWave];              // the keys of the bin the threshold lies in, once they fit a wave
  uint32_t list_n;
  uint32_t red[2][3][16];            // per wave: candidates (bit 31: malformed entry), largest key, largest ~key
  uint32_t newest[16];               // per wave: 1 + newest position among the candidates with the smallest key
  uint32_t tot[128];                 // per (u, wave): kept | equal << 16
  uint32_t first;                    // first slot that is not kept
};

// Larger key == kept first.  -0 is folded into +0 so that they tie (IEEE equality).
__device__ __forceinline__ uint32_t order_key(float x, bool keep_largest) {
  if (x == 0.0f) x = 0.0f;
  uint32_t u = __float_as_uint(x);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return keep_largest ? u : ~u;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {       // lanes without a source (or masked out) get 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
// row_shr:1, 2, 4, 8 inside the 16-lane rows, then lane 15 -> next row, lane 31 -> upper half
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp_u<0x111, 0xF>(v); v += dpp_u<0x112, 0xF>(v); v += dpp_u<0x114, 0xF>(v); v += dpp_u<0x118, 0xF>(v);
  v += dpp_u<0x142, 0xA>(v); v += dpp_u<0x143, 0xC>(v);
  return v;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {     // of unsigned values; uniform result
  v = max(v, dpp_u<0x111, 0xF>(v)); v = max(v, dpp_u<0x112, 0xF>(v)); v = max(v, dpp_u<0x114, 0xF>(v)); v = max(v, dpp_u<0x118, 0xF>(v));
  v = max(v, dpp_u<0x142, 0xA>(v)); v = max(v, dpp_u<0x143, 0xC>(v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}
__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); }

// zeroes what the ranking adds to; the barrier inside block_stats orders it before the first addition
template <int NT>
__device__ __forceinline__ void rank_clear(RankShared& sh) {
  uint4* const h = reinterpret_cast<uint4*>(&sh.hist[0][0]);
  for (int i = threadIdx.x; i < 4 * kBins / 4; i += NT) h[i] = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x == 0) { sh.list_n = 0u; sh.first = 0xFFFFFFFFu; }
}

struct Stats { uint32_t n_cand, kmin, kmax; bool bad; };

// candidates of the workgroup, their key range and whether any entry is malformed; one barrier (AT: the words it uses)
template <int NT, int S, int AT = 0>
__device__ __forceinline__ Stats block_stats(RankShared& sh, const uint32_t (&key)[S], uint32_t candm, bool bad) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = wave_id();
  uint32_t n = 0, hi = 0, nlo = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const bool c = (candm >> u) & 1u;
    n += (uint32_t)__popcll(__ballot(c));
    hi = max(hi, c ? key[u] : 0u);
    nlo = max(nlo, c ? ~key[u] : 0u);
  }
  hi = wave_max(hi);
  nlo = wave_max(nlo);
  if (__ballot(bad) != 0) n |= 0x80000000u;
  if (lane == 0) { sh.red[AT][0][wave] = n; sh.red[AT][1][wave] = hi; sh.red[AT][2][wave] = nlo; }
  __syncthreads();
  Stats st = {0u, 0u, 0u, false};
  uint32_t a = 0, flags = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t x = sh.red[AT][0][w];
    flags |= x;
    a += x & 0x7FFFFFFFu;
    st.kmax = max(st.kmax, sh.red[AT][1][w]);
    st.kmin = max(st.kmin, sh.red[AT][2][w]);
  }
  st.n_cand = a;
  st.kmin = ~st.kmin;
  st.bad = (flags >> 31) != 0;
  return st;
}

// Eq. 4 as a threshold: returns T and need_eq such that {key > T} plus the first need_eq slots with key == T (ascending
// slot) are exactly the `want` best candidates.  Each step spreads the remaining key range [lo, hi] over 512 bins and
// keeps the bin the threshold lies in, until that bin is taken whole, holds one value, or fits one wave, which then ranks its
// keys against each other.  Keys of one magnitude need one step and the ranking: 2 barriers (a radix select over all 32 key
// bits took 16); the bins follow the float's exponent, so outliers and infinities cost at most the 4 steps of the key
// width.  Every wave works the scan out for itself instead of waiting for one to broadcast it.
template <int NT, int S>
__device__ __forceinline__ void top_threshold(RankShared& sh, const uint32_t (&key)[S], uint32_t in, const Stats& st, uint32_t want,
                                              uint32_t* T, uint32_t* need_eq) {
  *T = 0xFFFFFFFFu; *need_eq = 0u;
  if (want == 0) return;
  *T = 0u; *need_eq = 0xFFFFFFFFu;
  if (want >= st.n_cand) return;
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t lo = st.kmin, hi = st.kmax, r = want;             // the r best of the candidates inside [lo, hi] are wanted
  for (int it = 0; lo != hi; ++it) {
    const int shift = max(0, (32 - __builtin_clz(hi - lo)) - kBinBits);
    uint32_t* const hist = sh.hist[it];
#pragma unroll
    for (int u = 0; u < S; ++u)
      if ((in >> u) & 1u) atomicAdd(&hist[(key[u] - lo) >> shift], 1u);
    __syncthreads();
    // lane l owns bins 511-8l .. 504-8l; scan from the largest down
    const uint4 c1 = reinterpret_cast<const uint4*>(hist)[2 * (kWave - 1 - lane)], c0 = reinterpret_cast<const uint4*>(hist)[2 * (kWave - 1 - lane) + 1];
    const uint32_t c[8] = {c0.w, c0.z, c0.y, c0.x, c1.w, c1.z, c1.y, c1.x};
    const uint32_t local = ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
    const uint32_t incl = wave_incl_scan(local);
    const int first = __ffsll((long long)__ballot(incl >= r)) - 1;     // exists: r <= candidates in the range
    uint32_t run = incl - local, digit = 0, above = 0, n_bin = 0;
    bool found = false;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool here = !found && run + c[k] >= r;
      if (here) { digit = (uint32_t)(kBins - 1 - 8 * lane - k); above = run; n_bin = c[k]; found = true; }
      run += c[k];
    }
    digit = lane_of(digit, first);
    r -= lane_of(above, first);
    n_bin = lane_of(n_bin, first);
    const uint32_t span = (1u << shift) - 1u;
    lo += digit << shift;
    hi = lo + min(hi - lo, span);
    if (r == n_bin) {                                        // the bin is taken whole
      if (lo == 0u) { *T = 0u; *need_eq = 0xFFFFFFFFu; }
      else { *T = lo - 1u; *need_eq = 0u; }
      return;
    }
#pragma unroll
    for (int u = 0; u < S; ++u)
      if (key[u] < lo || key[u] > hi) in &= ~(1u << u);
    if (n_bin <= kWave) {
#pragma unroll
      for (int u = 0; u < S; ++u)
        if ((in >> u) & 1u) sh.list[atomicAdd(&sh.list_n, 1u)] = key[u];
      __syncthreads();
      const uint32_t k = lane < (int)n_bin ? sh.list[lane] : 0u;
      uint32_t gt = 0, ge = 0;
      for (int j = 0; j < (int)n_bin; ++j) {
        const uint32_t kj = lane_of(k, j);
        gt += kj > k;
        ge += kj >= k;
      }
      const int at = __ffsll((long long)__ballot(lane < (int)n_bin && gt < r && r <= ge)) - 1;
      *T = lane_of(k, at);
      *need_eq = r - lane_of(gt, at);
      return;
    }
  }
  *T = lo;
  *need_eq = r;
}

// Places of the kept slots in ascending slot order: kept are those of `sure` and the first need_eq of `eq`.  dest[u] and bit u
// of the result for this thread's slots; *count gets the number kept.  One barrier.
template <int NT, int S>
__device__ __forceinline__ uint32_t place_kept(RankShared& sh, uint32_t sure, uint32_t eq, uint32_t need_eq, uint32_t (&dest)[S], uint32_t* count) {
  constexpr int NW = NT / kWave, E = S * NW;
  static_assert(E <= 2 * kWave, "one or two entries per lane");
  const int lane = threadIdx.x & (kWave - 1), wave = wave_id();
  unsigned long long am[S], em[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    am[u] = __ballot((sure >> u) & 1u);
    em[u] = __ballot((eq >> u) & 1u);
    if (lane == 0) sh.tot[u * NW + wave] = (uint32_t)__popcll(am[u]) | ((uint32_t)__popcll(em[u]) << 16);
  }
  __syncthreads();
  const uint32_t x0 = lane < E ? sh.tot[lane] : 0u;
  const uint32_t i0 = wave_incl_scan(x0);
  uint32_t total = lane_of(i0, kWave - 1), x1 = 0, i1 = 0;
  if constexpr (E > kWave) {
    x1 = kWave + lane < E ? sh.tot[kWave + lane] : 0u;
    i1 = wave_incl_scan(x1) + total;
    total = lane_of(i1, kWave - 1);
  }
  uint32_t take = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int at = u * NW + wave;
    const uint32_t base = (E > kWave && at >= kWave) ? lane_of(i1 - x1, at - kWave) : lane_of(i0 - x0, min(at, kWave - 1));
    const uint32_t e = (base >> 16) + lanes_below(em[u]);
    dest[u] = (base & 0xFFFFu) + lanes_below(am[u]) + min(e, need_eq);
    if (((sure >> u) & 1u) || (((eq >> u) & 1u) && e < need_eq)) take |= 1u << u;
  }
  *count = (total & 0xFFFFu) + min(total >> 16, need_eq);
  return take;
}

// The small arguments of the ranking kernels as preloaded dwords (see k_attend on what a load of the argument block costs):
// flags: score rows | score mode << 10 | eviction policy << 13 | two switches << 15, 16
struct RankFlags {
  int rows, mode, policy;
  bool a, b;
  __device__ __forceinline__ explicit RankFlags(uint32_t f) : rows(f & 0x3FF), mode((f >> 10) & 7), policy((f >> 13) & 3), a((f >> 15) & 1), b((f >> 16) & 1) {}
};
static inline uint32_t rank_flags(const adsa_params& p, bool a, bool b) {
  return score_rows(p) | p.score_mode << 10 | p.evict_policy << 13 | (a ? 1u << 15 : 0u) | (b ? 1u << 16 : 0u);
}
static inline float inv_width(const adsa_params& p) { return 1.0f / (float)p.grid_w; }

// element i of an array at a uniform address, without 64-bit arithmetic per lane
template <typename T>
__device__ __forceinline__ ADSA_GLOBAL T& elem(ADSA_GLOBAL T* base, uint32_t i) { return *(ADSA_GLOBAL T*)((gchar*)base + i * (uint32_t)sizeof(T)); }
template <typename T>
__device__ __forceinline__ T elem(const ADSA_GLOBAL T* base, uint32_t i) { return *(const ADSA_GLOBAL T*)((const gchar*)base + i * (uint32_t)sizeof(T)); }

// v[u] = sum over the score rows of slot idx[u], ascending row order, plain fp32 adds.  The loads of all slots and of two
// batches of rows are in flight together: one memory round trip for up to 2 * RB + 1 rows.
// SHARED: by loads that see what other workgroups of the same launch have stored with scope agent, whichever XCD they ran on.  All reads
// of score[] in such a launch have to be these: a plain one may find an older line in its own L2.
template <bool SHARED>
__device__ __forceinline__ float score_at(const gfloat* row, uint32_t i) {
  if constexpr (SHARED) return __hip_atomic_load((const gfloat*)((const gchar*)row + i * 4u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return elem(row, i);
}
constexpr int rank_batch(int S) { return S == 1 ? 24 : S == 2 ? 12 : S <= 4 ? 8 : 4; }
template <int S, int RB, bool SHARED = false>
__device__ __forceinline__ void rank_values(const gfloat* score, int rows, int cap, const int (&idx)[S], float (&v)[S]) {
  float cur[S][RB], nxt[S][RB];
  auto load_rows = [&](int r0, float (&t)[S][RB]) {
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
      for (int u = 0; u < S; ++u) t[u][k] = score_at<SHARED>(score + (size_t)min(r0 + k, rows - 1) * cap, idx[u]);    // (rows past the last: not added)
  };
#pragma unroll
  for (int u = 0; u < S; ++u) v[u] = score_at<SHARED>(score, idx[u]);
  if (rows == 1) return;
  load_rows(1, cur);
  for (int r = 1; r < rows; r += RB) {
    if (r + RB < rows) load_rows(r + RB, nxt);
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
      for (int u = 0; u < S; ++u) v[u] = r + k < rows ? v[u] + cur[u][k] : v[u];
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
      for (int k = 0; k < RB; ++k) cur[u][k] = nxt[u][k];
  }
}

// The fused V-cosine form's rows: rows 2h and 2h+1 hold head h's share of |v|^2 and of v.u.  Both sums over the heads,
// ascending, with two batches of loads in flight like rank_values.
template <int S>
__device__ __forceinline__ void rank_pairs(const gfloat* score, int heads, int cap, const int (&idx)[S], float (&ss)[S], float (&dot)[S]) {
  constexpr int RB = S == 1 ? 8 : S <= 3 ? 4 : S == 4 ? 2 : 1;
  float a[2][S][RB], b[2][S][RB];
  auto load_rows = [&](int h0, float (&x)[S][RB], float (&y)[S][RB]) {
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const gfloat* const at = score + (size_t)(2 * min(h0 + k, heads - 1)) * cap;
        x[u][k] = elem(at, idx[u]);
        y[u][k] = elem(at + cap, idx[u]);
      }
  };
#pragma unroll
  for (int u = 0; u < S; ++u) ss[u] = dot[u] = 0.0f;
  load_rows(0, a[0], b[0]);
  for (int h = 0; h < heads; h += RB) {
    if (h + RB < heads) load_rows(h + RB, a[1], b[1]);
#pragma unroll
    for (int k = 0; k < RB; ++k)
#pragma unroll
      for (int u = 0; u < S; ++u) {
        ss[u] = h + k < heads ? ss[u] + a[0][u][k] : ss[u];
        dot[u] = h + k < heads ? dot[u] + b[0][u][k] : dot[u];
      }
#pragma unroll
    for (int u = 0; u < S; ++u)
#pragma unroll
      for (int k = 0; k < RB; ++k) { a[0][u][k] = a[1][u][k]; b[0][u][k] = b[1][u][k]; }
  }
}

__device__ __forceinline__ bool keep_largest_of(int mode) {
  return mode == ADSA_SCORE_ATTN_MASS || mode == ADSA_SCORE_EXT_LARGEST;
}

}  // namespace
}  // namespace adsa
