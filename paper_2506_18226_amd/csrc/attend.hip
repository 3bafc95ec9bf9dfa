// Gather flash-decode of the ADSA decode path (gfx950): Eq. 5's gather fused with softmax
// attention over the selected slots, plus the cache append (Section 4.2) and the per-head
// attention-mass update, in ONE launch.
//
//  k_attend<EB, D, HT, U, NW, VF, DIRECT> : grid (token chunk, HT heads, sequence), NW waves.
//    HT = 1: a 16-byte-per-lane streaming load of one wave covers RPW = 64 / (D*EB/16) consecutive tokens of ONE head.
//    That holds for [slot][head][D] caches too: a row is 128 bytes or more, whole cache lines, so a workgroup that
//    walks one head's rows at a stride fetches nothing it does not use.  But it visits every page of the sequence for its
//    128 or 256 bytes a token, and so do the workgroups of the other heads: large launches over such caches take
//    512 bytes of a token (HT heads) per workgroup; the rule and its figures stand in make_attend_plan.
//    q.k is reduced over the lanes of a row with DPP; every lane keeps an online-softmax state (m, l, acc) in
//    registers, fp32, log2 domain.  The lane groups of a wave merge in registers (DPP and 16-/32-lane
//    swaps), the waves through one small LDS record each.
//    With one chunk per (sequence, head) the workgroup writes out / lse itself and adds the probabilities it produced
//    to its OWN head's row of score[]: no workgroup ever talks to another one.
//    With several chunks, each writes a partial and the scaled logits to the workspace and a second kernel,
//    k_attend_finish, merges them and updates the scores.
//    VF (ADSA_SCORE_VCOS_FUSED): every V row that streams through also yields its head's share of |v|^2
//    and of v.u (u = running sum of the candidates' normalised V, Eq. 2-3), stored per (head, slot): the
//    next eviction ranks from them instead of re-reading V.
#include <hip/hip_ext.h>

#include <algorithm>

#include "adsa_internal.h"
#include "adsa_device.h"

namespace adsa {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Sum over the LPR consecutive lanes that hold one row; every lane of the group gets the sum.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x += dpp_f<0xB1>(x);            // quad_perm [1,0,3,2]
  x += dpp_f<0x4E>(x);            // quad_perm [2,3,0,1]
  x += dpp_f<0x141>(x);           // row_half_mirror: the other quad of the 8-lane group
  if (LPR >= 16) x += dpp_f<0x140>(x);   // row_mirror: the other half of the 16-lane row
  if (LPR >= 32) x += __shfl_xor(x, 16, kWave);
  return x;
}

template <int EB> struct Elems;
template <> struct Elems<2> {      // bf16: 8 values per 16-byte vector
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xFFFF0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xFFFF0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xFFFF0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xFFFF0000u);
  }
};
template <> struct Elems<4> {      // fp32: 4 values per 16-byte vector
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};

constexpr int kBurst = 512;        // bytes of a token that a workgroup of several heads takes

// chunk c of a list of cnt (<= ADSA_MAX_CAP) tokens split evenly over nc (<= kMaxChunks) chunks
__device__ __forceinline__ int chunk_begin(int cnt, int c, int nc) { return (int)(((unsigned)cnt * (unsigned)c) / (unsigned)nc); }

struct AttendArgs {
  adsa_seq* seqs;
  const int32_t* sel_idx;
  const int32_t* sel_cnt;
  const char* q;
  const char* k_new;
  const char* v_new;
  char* out;
  float* lse;
  float* logits;        // [n_seq][n_heads][lg_stride]   scaled logits, log2 units (split launches)
  float* part_ml;       // [n_seq][n_heads][n_chunks][2]
  float* part_acc;      // [n_seq][n_heads][n_chunks][D]
  int n_heads, sel_cap, lg_stride, chunk_max, cap;
  int accumulate, append, advance;     // advance: see kAdvance
  int new_f32;                         // k_new / v_new are fp32 although the cache is bf16: round as they enter
  int vcos_fused;
  long long slot_stride_b, head_stride_b;
  float scale_log2;     // softmax scale * log2(e)
};

// DIRECT: the list of a (sequence, head) is not split (grid.x == 1): the workgroup finishes its heads alone.
// The arguments the first round trip needs come first, as plain scalars: the build asks for leading kernel
// arguments to be preloaded into scalar registers at wave launch, so those loads can leave at once, without
// waiting for a scalar load of the argument block (which would also wait for the sequence record's).
// HT > 1: the workgroup takes HT heads, the lane groups of a wave-load being the HT heads of RPW / HT tokens.
template <int EB, int D, int HT, int U, int NW, bool VF, bool DIRECT>
__global__ __launch_bounds__(NW * kWave) void k_attend(adsa_seq* seqs_arg, const int32_t* sel_idx_arg, const int32_t* sel_cnt_arg,
                                                      const char* q_arg, const char* k_new_arg, const char* v_new_arg,
                                                      int heads_and_flags, int sel_cap_arg, AttendArgs A) {
  constexpr int kAttThreads = NW * kWave;           // the waves of the workgroup share one token chunk
  constexpr int EPL = Elems<EB>::N;                 // elements per lane
  constexpr int LPR = D / EPL;                      // lanes per row
  constexpr int RPW = kWave / LPR / HT;             // tokens per wave-load
  static_assert(HT == 1 || (DIRECT && !VF && RPW * HT * LPR == kWave), "several heads: whole lists only");
  constexpr int PF = 1024 / kAttThreads;            // score read-modify-writes a thread starts early
  extern __shared__ float s_logit[];                // logits [HT][chunk_max] ([2][chunk_max] for VF), then
                                                    // the chunk's slot list int [chunk_max]
  // merge: the lane groups of a wave meet in registers, the waves through these (one state per wave)
  __shared__ float s_wm[NW * HT], s_wl[NW * HT];
  __shared__ __attribute__((aligned(16))) float s_wacc[NW * HT * D];

  const int chunk = DIRECT ? 0 : blockIdx.x, b = blockIdx.z;
  const int n_chunks = DIRECT ? 1 : gridDim.x;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // (only 14 dwords of arguments are preloaded: the two flags the first trip needs ride on the head count)
  const int n_heads = heads_and_flags & 0xFFFF, sel_cap = sel_cap_arg;
  // token and head of this lane's row within a wave-load, 16-byte piece of the row (heads past the last repeat it)
  const int dl = lane % LPR, ts = lane / LPR / HT, hs = HT == 1 ? 0 : lane / LPR % HT;
  const int head0 = blockIdx.y * HT, head = HT == 1 ? head0 : min(head0 + hs, n_heads - 1), heads_here = HT == 1 ? 1 : min(HT, n_heads - head0);

  // ---- first round trip: everything that depends on the kernel arguments only -- the count, the
  // sequence record, q and (when the list is not split, so its chunk starts at 0) the first slots of
  // the loop and the slots whose score words this thread updates at the end.  The record and the
  // count are pinned here so that they cannot drift behind the count test below.
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)(seqs_arg + b);
  const int cnt_raw = ((const gint*)sel_cnt_arg)[b];
  gchar* const k_base = (gchar*)sqp->k;
  gchar* const v_base = (gchar*)sqp->v;
  gfloat* const score = (gfloat*)sqp->score;
  const int pending = sqp->pending_slot;
  gfloat* const u_state = VF ? (gfloat*)sqp->vcos_u : nullptr;
  const gint* idx = (const gint*)sel_idx_arg + (size_t)b * sel_cap;
  const size_t row_off = ((size_t)b * n_heads + head) * D * EB + dl * 16;
  const gchar* const q_g = (const gchar*)q_arg;
  const gchar* const k_new_g = (const gchar*)k_new_arg;
  const gchar* const v_new_g = (const gchar*)v_new_arg;
  gchar* const out_g = (gchar*)A.out;
  gfloat* const lse_g = (gfloat*)A.lse;
  const uint4 qr = load16(q_g + row_off);
  // The wave takes the RPW-token units wave, wave + NW, ... of the chunk, in that order; unit number k of the
  // wave holds, for this lane, token (wave + k * NW) * RPW + ts.  slot_a[u]: slot of unit u; slot_nx[u]: of the unit
  // that takes ring position u next.  pf_slot: the whole list (its first PF * threads entries), one entry per
  // thread and round: staged in LDS below so that the loop finds its slots there instead of in global memory.
  // (These loads need nothing but preloaded arguments: they leave before anything waits for a scalar load.)
  int slot_a[U], slot_nx[U];
  int pf_slot[PF];
  if constexpr (DIRECT) {
#pragma unroll
    for (int u = 0; u < U; ++u) slot_a[u] = idx[min((wave + u * NW) * RPW + ts, sel_cap - 1)];
#pragma unroll
    for (int k = 0; k < PF; ++k) pf_slot[k] = idx[min(tid + k * kAttThreads, sel_cap - 1)];
  }
  // the query token's own K/V row (Section 4.2 append), as this launch attends and stores it: every lane keeps
  // its 16-byte piece in registers; fp32 rows of a bf16 cache are rounded once, here
  const bool append = (heads_and_flags & 0x10000) != 0, new_f32 = (heads_and_flags & 0x20000) != 0;
  uint4 nk = make_uint4(0u, 0u, 0u, 0u), nv = nk;
  if (append) {
    if (EB == 2 && new_f32) {
      const size_t off32 = ((size_t)b * n_heads + head) * D * 4 + dl * 32;
      nk = pack8_bf16(k_new_g + off32);
      nv = pack8_bf16(v_new_g + off32);
    } else {
      nk = load16(k_new_g + row_off);
      nv = load16(v_new_g + row_off);
    }
  }
  pin_uniform(cnt_raw); pin_uniform(k_base); pin_uniform(v_base); pin_uniform(score); pin_uniform(pending);
  if constexpr (VF) pin_uniform(u_state);
  // (the remaining arguments the loop needs: fetched in the same batch of scalar loads, not after it)
  pin_uniform(A.cap); pin_uniform(A.chunk_max); pin_uniform(A.slot_stride_b); pin_uniform(A.head_stride_b);
  pin_uniform(A.scale_log2); pin_uniform(A.accumulate);

  const int cnt = min(cnt_raw, sel_cap);
  if (cnt <= 0) {                                   // inactive or rejected sequence: zero-filled row
    if (chunk == 0) {
      const size_t row = (size_t)b * n_heads + head0;
      for (int o = tid; o < heads_here * D; o += kAttThreads) {
        if (EB == 4) reinterpret_cast<gfloat*>(out_g)[row * D + o] = 0.0f;
        else reinterpret_cast<ADSA_GLOBAL uint16_t*>(out_g)[row * D + o] = 0;
        if (o % D == 0) lse_g[row + o / D] = 0.0f;
      }
      if (head0 == 0 && tid == 0) advance_empty(sqp, A.advance);
    }
    return;
  }
  const int t_begin = DIRECT ? 0 : chunk_begin(cnt, chunk, n_chunks);
  const int t_end = DIRECT ? cnt : chunk_begin(cnt, chunk + 1, n_chunks);
  if (t_begin >= t_end) return;                     // fewer tokens than chunks
  const int len = t_end - t_begin;
  int* const s_idx = reinterpret_cast<int*>(s_logit + (VF ? 2 : HT) * A.chunk_max);   // the chunk's slot list (filled below)
  if constexpr (!DIRECT) {
#pragma unroll
    for (int u = 0; u < U; ++u) slot_a[u] = idx[t_begin + min((wave + u * NW) * RPW + ts, len - 1)];
  }
  // the slot adsa_select reserved for the query token (Section 4.2 append), if this launch fills it
  const int new_slot = (append && pending < A.cap) ? pending : -1;

  float pf_old[PF];
  float qf[EPL];
  Elems<EB>::unpack(qr, qf);
#pragma unroll
  for (int e = 0; e < EPL; ++e) qf[e] *= A.scale_log2;
  const long long lane_off = (long long)head * A.head_stride_b + dl * 16;
  gchar* kb = k_base + lane_off;
  gchar* vb = v_base + lane_off;
  // VF: this lane's columns of u for its head, and the two score rows of the head
  float uf[EPL];
  gfloat* vrows = nullptr;
  bool vf_on = false;
  if constexpr (VF) {
    vf_on = u_state != nullptr;
#pragma unroll
    for (int e = 0; e < EPL; ++e) uf[e] = vf_on ? u_state[(size_t)head * D + dl * EPL + e] : 0.0f;
    vrows = score + (size_t)(2 * head) * A.cap;
  }

  float m = -INFINITY, l = 0.0f, acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.0f;

  // Rolling gather: U units (row pairs per lane) are in flight per wave; as soon as the oldest has arrived it is
  // folded into the lane's online-softmax state and its registers are given to the next unit's loads, so the
  // number of outstanding requests stays constant instead of draining once per batch.
  {
    const int n_units = (len + RPW - 1) / RPW;
    const int n_mine = n_units > wave ? (n_units - wave + NW - 1) / NW : 0;       // units of this wave
    uint4 kr[U], vr[U];
    int tok[U];                                     // token (chunk-relative) in flight at ring position u; >= len: none
    bool fresh[U];                                  // ring position u stands for the query token's own row
#pragma unroll
    for (int u = 0; u < U; ++u) { kr[u] = make_uint4(0u, 0u, 0u, 0u); vr[u] = kr[u]; tok[u] = len; fresh[u] = false; }
    auto issue = [&](int u, int slot_raw, int token) {
      const int slot = min(max(slot_raw, 0), A.cap - 1);      // never touch memory outside the cache
      const long long off = (long long)slot * A.slot_stride_b;
      const bool is_new = slot == new_slot;         // the query token itself: its row is in registers (nk, nv)
      const bool live = token < len && !is_new;     // else (also past the end of the chunk) re-read q's row: cached
      kr[u] = load_stream16(live ? kb + off : q_g + row_off);
      vr[u] = load_stream16(live ? vb + off : q_g + row_off);
      tok[u] = token;
      fresh[u] = is_new;
    };
    auto fold = [&](int u) {
      const bool on = tok[u] < len;
      const uint4 kx = fresh[u] ? nk : kr[u], vx = fresh[u] ? nv : vr[u];
      float kf[EPL];
      Elems<EB>::unpack(kx, kf);
      float d = 0.0f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) d = fmaf(qf[e], kf[e], d);
      d = row_sum<LPR>(d);
      const float z = on ? d : -INFINITY;
      if (A.accumulate && dl == 0 && on) s_logit[hs * A.chunk_max + tok[u]] = z;
      const float m_new = fmaxf(m, z);
      const float corr = (m == -INFINITY) ? 0.0f : fast_exp2(m - m_new);     // (l and acc are 0 while m is -inf)
      const float pr = on ? fast_exp2(z - m_new) : 0.0f;
      float vf[EPL];
      Elems<EB>::unpack(vx, vf);
      l = fmaf(l, corr, pr);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = fmaf(acc[e], corr, pr * vf[e]);
      m = m_new;
      if constexpr (VF) {                           // Eq. 2-3 bookkeeping of this row: |v_h|^2 and v_h . u_h
        float dv = 0.0f, sv = 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) { dv = fmaf(vf[e], uf[e], dv); sv = fmaf(vf[e], vf[e], sv); }
        dv = row_sum<LPR>(dv);
        sv = row_sum<LPR>(sv);
        if (dl == 0 && on) { s_logit[tok[u]] = sv; s_logit[A.chunk_max + tok[u]] = dv; }
      }
      // the state is demanded HERE, and no memory access may cross: the unit is folded completely before the
      // loads that reuse its ring position are issued, and no later unit's arithmetic is pulled in front of it
      // (left to itself the compiler gathers all the logits of a trip first and so waits for the whole ring)
      static_assert(EPL == 4 || EPL == 8, "elements per lane");
      if constexpr (EPL == 8)
        asm volatile("" : "+v"(m), "+v"(l), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]),
                     "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]) : : "memory");
      else
        asm volatile("" : "+v"(m), "+v"(l), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : : "memory");
    };
    // unit k of the wave lives at ring position k % U: units 0 .. U-1 are requested here, trip t folds units
    // tU .. tU+U-1 and requests the units one ring revolution later, the last trip only folds.  (Units past
    // the wave's last one re-read the q row, which is cached by then.)
    auto refill = [&](int u, int k, int slot_raw) { // ring position u <- unit k; fetch the slot of unit k + U
      const int token = (wave + k * NW) * RPW + ts;
      issue(u, slot_raw, token);
      slot_nx[u] = s_idx[min(token + U * NW * RPW, len - 1)];
      asm volatile("" : : : "memory");             // requests leave in ring order (the wait counts rely on it)
      __builtin_amdgcn_sched_barrier(0);            // ... and before the next unit's arithmetic, which waits for ITS rows
    };
    const int n_trips = (n_mine + U - 1) / U;
    // The first revolution's rows are requested at once, from the slots the first round trip brought in registers ...
#pragma unroll
    for (int u = 0; u < U; ++u) {
      issue(u, slot_a[u], (wave + u * NW) * RPW + ts);
      asm volatile("" : : : "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
    // ... and while they are on their way the chunk's slot list goes to LDS (clamped to the cache: nothing below
    // ever leaves it), where the later revolutions and the score update find it
    if constexpr (DIRECT) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        const int j = tid + k * kAttThreads;
        if (j < len) s_idx[j] = min(max(pf_slot[k], 0), A.cap - 1);
      }
      for (int j = tid + PF * kAttThreads; j < len; j += kAttThreads) s_idx[j] = min(max(idx[j], 0), A.cap - 1);
    } else {
      for (int j = tid; j < len; j += kAttThreads) s_idx[j] = min(max(idx[t_begin + j], 0), A.cap - 1);
    }
    __syncthreads();
    // thread i of the final score update serves tokens i, i + threads, ...; start the first PF reads now
    if (DIRECT && HT == 1 && A.accumulate) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        const int i = tid + k * kAttThreads;
        pf_old[k] = 0.0f;
        if (i < len) {
          pf_slot[k] = s_idx[i];
          pf_old[k] = score[(size_t)head * A.cap + pf_slot[k]];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) slot_nx[u] = s_idx[min((wave + (u + U) * NW) * RPW + ts, len - 1)];
    asm volatile("" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);
    int k_next = U;
    for (int trip = 1; trip < n_trips; ++trip) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        fold(u);
        refill(u, k_next + u, slot_nx[u]);
      }
      k_next += U;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) fold(u);
  }
  // ---- merge, step 1 (registers): the RPW lane groups of a wave that worked on the same head bring their
  // states to the wave's maximum and add them up across lanes; every lane ends up with the wave's state.
  if constexpr (RPW > 1) {
    float M = m;
#pragma unroll
    for (int x = LPR * HT; x < kWave; x <<= 1)
      M = x == 8 ? xor_max<8>(M) : x == 16 ? xor_max<16>(M) : xor_max<32>(M);
    const float sc = (m == -INFINITY) ? 0.0f : fast_exp2(m - M);     // a group that saw no token weighs 0
    l *= sc;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] *= sc;
#pragma unroll
    for (int x = LPR * HT; x < kWave; x <<= 1) {
      l = x == 8 ? xor_sum<8>(l) : x == 16 ? xor_sum<16>(l) : xor_sum<32>(l);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = x == 8 ? xor_sum<8>(acc[e]) : x == 16 ? xor_sum<16>(acc[e]) : xor_sum<32>(acc[e]);
    }
    m = M;
  }
  // ---- step 2 (LDS): one state per wave; after ONE barrier every thread works out the
  // normaliser itself, the first D threads each finish one output element
  if (ts == 0) {
    if (dl == 0) { s_wm[wave * HT + hs] = m; s_wl[wave * HT + hs] = l; }
    float4* dst = reinterpret_cast<float4*>(&s_wacc[(wave * HT + hs) * D + dl * EPL]);
#pragma unroll
    for (int e = 0; e < EPL; e += 4) dst[e / 4] = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
  }
  __syncthreads();
  // Section 4.2: the query token's row enters the cache (nothing in this launch reads it from there)
  if (new_slot >= 0 && chunk == n_chunks - 1 && wave == 0 && ts == 0 && hs < heads_here) {
    const long long off = (long long)new_slot * A.slot_stride_b;
    store16(kb + off, nk);
    store16(vb + off, nv);
  }
  if constexpr (HT > 1) {
    // ---- several heads: a thread finishes output elements of one head after the other, then adds its tokens' probabilities to
    // all the heads' score rows
    __shared__ float s_lse2[HT];
    for (int o = tid; o < heads_here * D; o += kAttThreads) {
      const int h = o / D, d = o - h * D;
      float w[NW], M = -INFINITY, L = 0.0f, a = 0.0f;
#pragma unroll
      for (int k = 0; k < NW; ++k) { w[k] = s_wm[k * HT + h]; M = fmaxf(M, w[k]); }
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        w[k] = (w[k] == -INFINITY) ? 0.0f : fast_exp2(w[k] - M);
        L = fmaf(s_wl[k * HT + h], w[k], L);
        a = fmaf(s_wacc[(k * HT + h) * D + d], w[k], a);
      }
      const float val = __fdividef(a, L);
      const size_t row = (size_t)b * n_heads + head0 + h;
      if (EB == 4) reinterpret_cast<gfloat*>(out_g)[row * D + d] = val;
      else reinterpret_cast<ADSA_GLOBAL uint16_t*>(out_g)[row * D + d] = (uint16_t)f32_to_bf16_rne(val);
      if (d == 0) { s_lse2[h] = M + __log2f(L); lse_g[row] = s_lse2[h] * kLn2; }
    }
    if (A.accumulate) {
      __syncthreads();
      float lse2[HT];
#pragma unroll
      for (int h = 0; h < HT; ++h) lse2[h] = s_lse2[min(h, heads_here - 1)];
      for (int i = tid; i < len; i += kAttThreads) {
        gfloat* const at = score + (size_t)head0 * A.cap + s_idx[i];
        float old[HT];
#pragma unroll
        for (int h = 0; h < HT; ++h) old[h] = at[(size_t)min(h, heads_here - 1) * A.cap];
#pragma unroll
        for (int h = 0; h < HT; ++h)
          if (h < heads_here) at[(size_t)h * A.cap] = old[h] + fast_exp2(s_logit[h * A.chunk_max + i] - lse2[h]);
      }
    }
    if (head0 == 0 && tid == 0) advance_step(sqp, A.advance);
    return;
  }
  // log2-domain normaliser of the whole workgroup, worked out by every thread from the waves' states
  float wgt[NW], M = -INFINITY, L = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) { wgt[w] = s_wm[w]; M = fmaxf(M, wgt[w]); }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wgt[w] = (wgt[w] == -INFINITY) ? 0.0f : fast_exp2(wgt[w] - M);       // empty wave: weight 0
    L = fmaf(s_wl[w], wgt[w], L);
  }
  const size_t row = (size_t)b * n_heads + head;
  if (tid < D) {
    static_assert(D <= kAttThreads, "one output element per thread");
    float a = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) a = fmaf(s_wacc[w * D + tid], wgt[w], a);
    if constexpr (DIRECT) {
      const float val = __fdividef(a, L);
      if (EB == 4) reinterpret_cast<gfloat*>(out_g)[row * D + tid] = val;
      else reinterpret_cast<ADSA_GLOBAL uint16_t*>(out_g)[row * D + tid] = (uint16_t)f32_to_bf16_rne(val);
      if (tid == 0) lse_g[row] = (M + __log2f(L)) * kLn2;
    } else {
      const size_t pidx = row * n_chunks + chunk;
      A.part_acc[pidx * D + tid] = a;
      if (tid == 0) { A.part_ml[pidx * 2] = M; A.part_ml[pidx * 2 + 1] = L; }
    }
  }

  if constexpr (VF) {
    // |v_h|^2 and v_h.u_h of this chunk's tokens, left in LDS by the loop (the barrier above ordered them)
    if (vf_on) {
      int j0 = tid;
      if constexpr (DIRECT) {                       // the first slots were fetched before the loop
#pragma unroll
        for (int k = 0; k < PF; ++k) {
          const int j = tid + k * kAttThreads;
          if (j < len) {
            const int slot = min(max(pf_slot[k], 0), A.cap - 1);
            vrows[slot] = s_logit[j];
            vrows[A.cap + slot] = s_logit[A.chunk_max + j];
          }
        }
        j0 = tid + PF * kAttThreads;
      }
      for (int j = j0; j < len; j += kAttThreads) {
        const int slot = s_idx[j];
        vrows[slot] = s_logit[j];
        vrows[A.cap + slot] = s_logit[A.chunk_max + j];
      }
    }
  }
  if constexpr (DIRECT) {
    // -------- this head's attention mass: score[head][slot] += p, from the logits still in LDS
    if (A.accumulate) {
      const float lse2 = M + __log2f(L);
      gfloat* const srow = score + (size_t)head * A.cap;
#pragma unroll
      for (int k = 0; k < PF; ++k) {                // reads were started before the loop
        const int i = tid + k * kAttThreads;
        if (i < len) srow[pf_slot[k]] = pf_old[k] + fast_exp2(s_logit[i] - lse2);
      }
      constexpr int B = 4;                          // longer lists: batches of reads, so that their latencies overlap
      for (int i0 = tid + PF * kAttThreads; i0 < len; i0 += B * kAttThreads) {
        float old[B];
        int slot[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
          slot[k] = s_idx[min(i0 + k * kAttThreads, len - 1)];
          old[k] = srow[slot[k]];
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
          const int i = i0 + k * kAttThreads;
          if (i < len) srow[slot[k]] = old[k] + fast_exp2(s_logit[i] - lse2);
        }
      }
    }
    // last act on a sequence (one thread; no other workgroup reads step): VF marks the score rows as the
    // next step's if u was (tags kept as floats behind u); then the step may advance.  (Written out here:
    // handing the kernel's argument struct to a helper by reference made every variant slower.)
    if (head == 0 && tid == 0) {
      if constexpr (VF) {
        if (u_state) {
          gfloat* tags = u_state + (size_t)A.n_heads * D;
          const float want = (float)(sqp->step + 2);
          tags[1] = tags[0] == want ? want : 0.0f;
        }
      }
      advance_step(sqp, A.advance);
    }
    return;
  } else {
    // -------- several chunks: this workgroup's partial and logits are in the workspace; k_attend_finish, the next kernel
    // on the stream, merges them (the launch boundary orders the two and makes the stores visible on every XCD)
    if (A.accumulate) {
      float* const lg = A.logits + row * A.lg_stride + t_begin;
      for (int i = tid; i < len; i += kAttThreads) lg[i] = s_logit[i];
    }
  }
}

// Second half of a split launch: grid (token slice, head, sequence).  Every workgroup works out the head's softmax
// normaliser from the chunks' (m, l), in chunk order; slice 0 merges the partial outputs and writes out / lse; every
// slice adds the probabilities of its kFinishTokens tokens to the head's score row.
constexpr int kFinishThreads = 256, kFinishTokens = 4 * kFinishThreads;
template <int EB, int D>
__global__ __launch_bounds__(kFinishThreads) void k_attend_finish(AttendArgs A, int n_chunks) {
  const int slice = blockIdx.x, head = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)(A.seqs + b);
  const int cnt = min(((const gint*)A.sel_cnt)[b], A.sel_cap);
  gfloat* const score = (gfloat*)sqp->score;
  gfloat* const u_state = A.vcos_fused ? (gfloat*)sqp->vcos_u : nullptr;
  if (cnt <= 0 || slice * kFinishTokens >= cnt) return;      // (inactive sequences: zero rows, already written)
  const size_t row = (size_t)b * A.n_heads + head;
  const gfloat* const ml = (const gfloat*)A.part_ml + row * n_chunks * 2;
  const gfloat* const acc = (const gfloat*)A.part_acc + row * n_chunks * D;
  const gfloat* const lg = (const gfloat*)A.logits + row * A.lg_stride;
  const gint* const idx = (const gint*)A.sel_idx + (size_t)b * A.sel_cap;
  // chunks beyond a short list hold nothing (their workspace words are stale)
  const bool merge = slice == 0 && tid < D;
  float mc[kMaxChunks], lc[kMaxChunks], ac[kMaxChunks];
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    const bool on = c < n_chunks && chunk_begin(cnt, c, n_chunks) < chunk_begin(cnt, c + 1, n_chunks);
    mc[c] = on ? ml[2 * c] : -INFINITY;
    lc[c] = on ? ml[2 * c + 1] : 0.0f;
    ac[c] = (on && merge) ? acc[(size_t)c * D + tid] : 0.0f;
  }
  constexpr int B = kFinishTokens / kFinishThreads;
  float z[B], old[B];
  int slot[B];
  if (A.accumulate) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int j = min(slice * kFinishTokens + u * kFinishThreads + tid, cnt - 1);
      slot[u] = min(max(idx[j], 0), A.cap - 1);
      z[u] = lg[j];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) old[u] = score[(size_t)head * A.cap + slot[u]];
  }
  float M = -INFINITY, L = 0.0f;
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) M = fmaxf(M, mc[c]);
#pragma unroll
  for (int c = 0; c < kMaxChunks; ++c) {
    mc[c] = (mc[c] == -INFINITY) ? 0.0f : fast_exp2(mc[c] - M);       // from here on: the chunk's weight
    L = fmaf(lc[c], mc[c], L);
  }
  const float lse2 = M + __log2f(L);
  if (merge) {
    float a = 0.0f;
#pragma unroll
    for (int c = 0; c < kMaxChunks; ++c) a = fmaf(ac[c], mc[c], a);
    const float val = __fdividef(a, L);
    const size_t oi = row * D + tid;
    if (EB == 4) reinterpret_cast<gfloat*>((gchar*)A.out)[oi] = val;
    else reinterpret_cast<ADSA_GLOBAL uint16_t*>((gchar*)A.out)[oi] = (uint16_t)f32_to_bf16_rne(val);
    if (tid == 0) ((gfloat*)A.lse)[row] = lse2 * kLn2;
  }
  if (A.accumulate) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int j = slice * kFinishTokens + u * kFinishThreads + tid;
      if (j < cnt) score[(size_t)head * A.cap + slot[u]] = old[u] + fast_exp2(z[u] - lse2);
    }
  }
  if (slice == 0 && head == 0 && tid == 0) {                 // last act on the sequence: see k_attend
    if (u_state) {
      gfloat* tags = u_state + (size_t)A.n_heads * D;
      const float want = (float)(sqp->step + 2);
      tags[1] = tags[0] == want ? want : 0.0f;
    }
    advance_step(sqp, A.advance);
  }
}

template <int EB, int D, int HT, int NW, bool VF, bool DIRECT>
hipError_t launch_attend_w(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  // Row pairs in flight per lane.  us with 2 | 3 | 4 | 6 | 8, bf16: 768 pairs x 647 tokens x 64 22.6 | 22.2 | 22.3 | 22.8 | 23.3; 128 x
  // 1159 x 128 19.4 | 17.5 | 17.6 | 18.0 | 19.1; 40 x 427 x 64 5.8 | 5.8 | 5.6 | 7.0 | 6.4; fp32 63 x 433 x 128 13.0 | 11.3 | 11.5 | 12.2 |
  // 13.1; only 320 x 427 x 64, whose lists fill 3.3 revolutions of 4, is better off with 3: 9.9 | 9.6 | 10.2 | 11.4 | 11.3.
  constexpr int U = 4;
  const size_t lds = (size_t)((VF ? 2 : HT) + 1) * plan.chunk_max * sizeof(float);      // logits rows + the slot list
  dim3 grid(plan.n_chunks, (A.n_heads + HT - 1) / HT, n_seq);
  // (a split launch is two kernels: the start event belongs to the first, the stop event to the second)
  const int hf = A.n_heads | (A.append ? 0x10000 : 0) | (A.new_f32 ? 0x20000 : 0);
  if (ev_start && ev_stop)
    hipExtLaunchKernelGGL((k_attend<EB, D, HT, U, NW, VF, DIRECT>), grid, dim3(NW * kWave), (uint32_t)lds, st, ev_start,
                          DIRECT ? ev_stop : nullptr, 0, A.seqs, A.sel_idx, A.sel_cnt, A.q, A.k_new, A.v_new, hf, A.sel_cap, A);
  else
    hipLaunchKernelGGL((k_attend<EB, D, HT, U, NW, VF, DIRECT>), grid, dim3(NW * kWave), lds, st,
                       A.seqs, A.sel_idx, A.sel_cnt, A.q, A.k_new, A.v_new, hf, A.sel_cap, A);
  if constexpr (!DIRECT) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 fgrid(A.accumulate ? (A.sel_cap + kFinishTokens - 1) / kFinishTokens : 1, A.n_heads, n_seq);
    if (ev_start && ev_stop)
      hipExtLaunchKernelGGL((k_attend_finish<EB, D>), fgrid, dim3(kFinishThreads), 0, st, nullptr, ev_stop, 0, A, plan.n_chunks);
    else
      hipLaunchKernelGGL((k_attend_finish<EB, D>), fgrid, dim3(kFinishThreads), 0, st, A, plan.n_chunks);
  }
  return hipGetLastError();
}

template <int EB, int D, bool VF>
hipError_t launch_attend_v(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  if constexpr (!VF && kBurst > D * EB) {
    if (plan.heads > 1) return launch_attend_w<EB, D, kBurst / (D * EB), 4, VF, true>(A, plan, n_seq, st, ev_start, ev_stop);
  }
  if (plan.n_chunks > 1) return launch_attend_w<EB, D, 1, 8, VF, false>(A, plan, n_seq, st, ev_start, ev_stop);
  if (plan.waves == 8) return launch_attend_w<EB, D, 1, 8, VF, true>(A, plan, n_seq, st, ev_start, ev_stop);
  return launch_attend_w<EB, D, 1, 4, VF, true>(A, plan, n_seq, st, ev_start, ev_stop);
}

template <int EB, int D>
hipError_t launch_attend_t(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (A.vcos_fused) return launch_attend_v<EB, D, true>(A, plan, n_seq, st, ev_start, ev_stop);
  return launch_attend_v<EB, D, false>(A, plan, n_seq, st, ev_start, ev_stop);
}

__global__ void k_zero_words(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

}  // namespace

// Chunks per list the workspace has room for.  adsa_workspace_bytes() is part of what callers size and keep their memory
// by (and what adsa_step_static's limit is compared with), so it does not follow the launch rule of make_attend_plan:
// batches of fewer than 96 (sequence, head group) pairs -- a group being the heads one 1 KB wave-load covers in a
// [slot][head][D] cache -- have room for at least as many chunks as any list there is split into.
static int heads_per_group(const adsa_params& p) {
  const bool slot_major = p.kv_slot_stride >= p.kv_head_stride;
  return slot_major && p.q_per_kv <= 1 ? 1024 / (p.head_dim * elem_bytes(p)) : 1;
}
static int head_groups(const adsa_params& p) { return (p.n_heads + heads_per_group(p) - 1) / heads_per_group(p); }
static int reserved_chunks(const adsa_params& p) {
  const long long pairs = (long long)p.n_seq * head_groups(p);
  long long nc = 1;
  if (pairs < 96) nc = std::min<long long>({(768 + pairs - 1) / pairs, std::max(p.sel_cap / 32, 1), kMaxChunks});
  const int lds_rows = (p.score_mode == ADSA_SCORE_VCOS_FUSED ? 2 : heads_per_group(p)) + 1;
  while (nc < kMaxChunks && (size_t)lds_rows * ((p.sel_cap + nc - 1) / nc + 1) * sizeof(float) > 40 * 1024) ++nc;
  return (int)nc;
}

AttendPlan make_attend_plan(const adsa_params& p) {
  AttendPlan a;
  if (p.q_per_kv > 1) {      // grouped queries: one workgroup per (sequence, cache head, chunk of whole 16-token tiles)
    const long long wgs = (long long)p.n_seq * p.n_heads;
    // 8 waves, but 4 where there is more than one workgroup per CU and the lists are short, or the logits and the waves'
    // tiles of two 8-wave workgroups do not fit a CU and those of two 4-wave ones do.  Measured, 4 | 8 waves: 256 pairs x 649 x 128,
    // G = 8 20.1 | 17.6 us; 512 31.6 | 30.9; 512 x 649 x 64 19.0 | 17.8; 384 x 300 x 128 15.3 | 15.9; 640 x 200 x 64 10.9 | 12.0;
    // 512 x 649 x 128 with G = 16 (two fit with 4) 33.8 | 37.3; 390 x 1230 x 128 in 2336 slots (one fits either way) 58.7 | 46.3.
    const bool four = !gqa_two_fit(gqa_lds_bytes(p, 8, 1)) && gqa_two_fit(gqa_lds_bytes(p, 4, 1));
    a.waves = wgs >= 384 && (p.sel_cap < 448 || four) ? 4 : 8;
    // Lists are split only when they must be (the logits of a whole list, all G queries, do not fit in LDS even
    // with 4 waves) or when it was measured to pay: long lists (>= 2560 slots) of at most 32 (sequence, cache head)
    // pairs, 8 pairs x 2700 x 128 16.7 us in 16 chunks; merged by the last of them to arrive it was 25, whole 41.
    // Hence: as many chunks as fit the LDS limit, and more only while the launch stays near 128 workgroups.
    int nc = 1;
    const bool must = gqa_lds_bytes(p, 4, 1) > kGqaMaxLds;
    if (must || (p.sel_cap >= 2560 && wgs <= 32)) {
      while (nc < kMaxChunks && gqa_lds_bytes(p, 4, nc) > kGqaMaxLds) ++nc;
      int more = (int)((128 + wgs - 1) / wgs);
      if (more > p.sel_cap / 160) more = p.sel_cap / 160;
      if (more > kMaxChunks) more = kMaxChunks;
      if (nc < more) nc = more;
    }
    while (nc == 1 && a.waves > 4 && gqa_lds_bytes(p, a.waves, 1) > kGqaMaxLds) a.waves /= 2;
    if (nc > 1) a.waves = 4;
    a.n_chunks = a.reserved_chunks = nc;
    a.heads = 1;
    a.chunk_max = gqa_logit_stride(p, nc);
    return a;
  }
  // One workgroup per (sequence, head): 8 waves up to one pair per CU, 4 from two on; in between 8 where the lists together
  // are long (80 MB), for the waves that then wait side by side, and 4 where starting the workgroups is a good part of
  // the launch.  Measured, us with 4 | 8 | 16 waves, bf16: 320 pairs x 457 tokens x 64 (37 MB) 10.6 | 11.1 | 15.4;
  // 400 x 650 x 64 (67 MB) 14.6 | 14.9 | 20.6; 480 x 700 x 64 (86 MB) 17.8 | 16.7; 288 x 1300 x 64 (96 MB) 24.6 | 23.3;
  // 400 x 700 x 128 (143 MB) 26.8 | 25.9; 768 x 200 x 64 9.6 | 10.6 | 19.9; 768 x 649 x 64 22.6 | 22.7 | 32.3;
  // 256 x 650 x 128 16.2 | 15.8 | 17.0; 192 x 650 x 64 9.3 | 8.5 | 10.9; 128 x 4000 x 128 60.3 | 53.0 | 52.4;
  // 40 x 400 x 64 6.3 | 5.9 | 7.2; fp32: 288 x 300 x 128 (88 MB) 21.0 | 20.3; 400 x 300 x 128 22.9 | 22.1.  Lists that the
  // rings of 4 waves hold at once (32 KB) gain nothing from more of them: 16 pairs x 64 tokens x 64 3.7 | 4.3, 256 x 128 x 64
  // 4.3 | 4.9, 16 x 32 x 128 fp32 3.3 | 3.8, fused 64 x 64 x 128 4.8 | 6.5; 16 x 192 x 64 (48 KB) 4.4 | 4.5, fp32 16 x 48 x 128 4.2 | 3.9.
  const long long pairs = (long long)p.n_seq * p.n_heads;
  const long long b_list = (long long)p.sel_cap * 2 * p.head_dim * elem_bytes(p);
  a.waves = pairs >= 512 || b_list <= (32 << 10) || (pairs > 256 && pairs * b_list < (80ll << 20)) ? 4 : 8;
  // Splitting a list costs a second launch, ~3 us.  What it can save: a workgroup alone streams ~55 GB/s (8 or 16 waves
  // alike), the chip ~5.5 TB/s, as much as ~100 workgroups.  So a list of b bytes on each of `pairs` workgroups is split
  // when b * (1 - max(pairs / 100, 1 / chunks)) is more than 230 KB, ~4 us; into 8-wave chunks of about 64 KB that
  // together occupy every CU.  Measured, us whole | split: 8 pairs x 256 KB 8.0 | 8.7; 20 x 205 KB 7.4 | 9.2;
  // 16 x 384 KB 11.9 | 9.6; 8 x 512 KB 13.4 | 9.4; 8 x 2 MB 44 | 11.6; 32 x 1 MB 24.6 | 12.6; 32 x 4 MB 84.7 | 27.1;
  // 80 x 384 KB 12.8 | 12.8; 64 x 154 KB 7.1 | 9.8.  (One launch whose last workgroup to arrive merges, behind a
  // device-scope release / acquire, took 12 us for 8 x 512 KB, 58 for 32 x 4 MB and 17.5 for 40 lists of 102 KB, which
  // take 5.9 us whole.)
  // 64 KB is what the rings of 8 waves hold at once: where the CUs allow it a chunk has no more, so that none ends in a
  // second, nearly empty revolution (2 x 300 KB fused: 11.2 with 4 chunks, 9.9 with 5; 2 x 300 KB plain 9.5 and 8.3).  Rows of the
  // fused V-cosine form take longer, so their line is 175 KB of such chunks: 2 x 200 KB 9.4 | 9.8, 2 x 250 KB 10.5 | 9.6,
  // 16 x 300 KB 12.4 | 10.4.
  const bool fused = p.score_mode == ADSA_SCORE_VCOS_FUSED;
  const long long full = b_list / (64 << 10), snug = (b_list + (64 << 10) - 1) / (64 << 10);
  auto chunks = [](long long n) { return n > kMaxChunks ? (long long)kMaxChunks : n < 1 ? 1ll : n; };
  long long nc = chunks(std::min(full, (256 + pairs - 1) / pairs));
  const long long snug_nc = pairs * snug <= 256 ? chunks(snug) : nc;
  if (fused) nc = snug_nc;
  const long long hidden = pairs * nc > 100 ? pairs * nc : 100;          // b_list * (1 - max(pairs / 100, 1 / nc)), in units of 1 / (100 nc)
  if (pairs >= 96 || b_list * (100 * nc - hidden) <= (fused ? 175000ll : 230000ll) * 100 * nc) nc = 1;
  else nc = snug_nc;
  // the logits (two rows of them for the fused V-cosine form) and the slot list of a chunk must fit in LDS
  const int lds_rows = (fused ? 2 : 1) + 1;
  while (nc < kMaxChunks && (size_t)lds_rows * ((p.sel_cap + nc - 1) / nc + 1) * sizeof(float) > 40 * 1024) ++nc;
  a.n_chunks = (int)nc;
  // Heads per workgroup over a [slot][head][D] cache: 512 bytes of a token from 384 such workgroups of 4 waves on, which then keep
  // the chip busy with a quarter or half of the workgroups and visit each page a quarter or half as often.  bf16, us with one
  // head | 512 bytes (all of a 1 KB burst in one wave-load): 41 x 48 heads x 64, 810 tokens 79.2 | 64.7 (65.1); 509 x 24 x 64, 165
  // tokens 101 | 86 (85); 44 x 48 x 64, 39 tokens 10.4 | 8.8 (9.3); 13 x 64 x 128, 879 tokens 68 | 61 (63); fp32 209 x 36 x 64, 150
  // tokens 98 | 92 (94); below the line 32 x 36 x 64, 706 tokens 38 | 44 (51); 26 x 20 x 64, 687 tokens 21.7 | 23.0 (49);
  // 8 x 12 x 64, 300 tokens 5.8 against 11.6 for the burst.  Heads that do not divide by HT leave lanes idle: 259 x 9 x 64, 439
  // tokens 44 | 50, so only short lists, whose workgroups are mostly start and end, take them: 863 x 7 x 64, 52 tokens 23 | 17, 451 x 7 x 64, 61 tokens 14.3 | 11.9.
  // Rows of 512 bytes have nothing to gain.
  const int ht = p.kv_slot_stride > p.kv_head_stride ? kBurst / (p.head_dim * elem_bytes(p)) : 1;
  const long long groups = (p.n_heads + ht - 1) / ht;
  const bool fits = p.n_heads % ht == 0 || (b_list <= (32 << 10) && 100 * groups * ht <= 115ll * p.n_heads);
  a.heads = !fused && nc == 1 && ht > 1 && p.n_seq * groups >= 384 && fits && (size_t)(ht + 1) * (p.sel_cap + 1) * sizeof(float) <= 40 * 1024 ? ht : 1;
  if (a.heads > 1) a.waves = 4;
  a.reserved_chunks = reserved_chunks(p);
  a.chunk_max = (p.sel_cap + a.n_chunks - 1) / a.n_chunks + 1;
  return a;
}

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

Workspace make_workspace(const adsa_params& p, const AttendPlan& plan) {
  Workspace w;
  size_t off = 0;
  const bool split = plan.reserved_chunks > 1;
  const size_t hq = (size_t)p.n_heads * (p.q_per_kv > 1 ? p.q_per_kv : 1);      // rows of out / logits / partials per sequence
  w.lg_stride = p.q_per_kv > 1 ? gqa_global_logit_stride(p) : (int)align_up((size_t)p.sel_cap, 4);
  off = align_up(off + sizeof(int32_t) * (size_t)p.n_seq * head_groups(p), 256);
  w.head_bytes = off;
  w.logits_off = off;
  if (split) off = align_up(off + sizeof(float) * (size_t)p.n_seq * hq * w.lg_stride, 256);
  w.part_ml_off = off;
  if (split) off = align_up(off + sizeof(float) * (size_t)p.n_seq * hq * plan.reserved_chunks * 2, 256);
  w.part_acc_off = off;
  if (split) off = align_up(off + sizeof(float) * (size_t)p.n_seq * hq * plan.reserved_chunks * p.head_dim, 256);
  w.plan_off = off;
  off = align_up(off + sizeof(int32_t) * (size_t)p.n_seq * 4, 256);
  w.vcos_off = off;
  w.vcos_u_off = off;
  w.vcos_s_off = off;
  if (is_vcos(p)) {
    off = align_up(off + sizeof(float) * (size_t)p.n_seq * p.cap, 256);
    w.vcos_u_off = off;
    off = align_up(off + sizeof(float) * (size_t)p.n_seq * vcos_tiles(p.cap) * p.n_heads * p.head_dim, 256);
    w.vcos_s_off = off;
    if (p.score_mode == ADSA_SCORE_VCOS_FUSED) off = align_up(off + sizeof(float) * (size_t)p.n_seq * p.cap, 256);
  }
  w.total = off;
  return w;
}

hipError_t launch_workspace_init(char* ws, const Workspace& w, hipStream_t st) {
  const size_t words = w.head_bytes / 4;
  hipLaunchKernelGGL(k_zero_words, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st,
                     reinterpret_cast<uint32_t*>(ws), words);
  return hipGetLastError();
}

hipError_t launch_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q,
                         const void* k_new, const void* v_new, const int32_t* sel_idx, const int32_t* sel_cnt,
                         void* out, float* lse, char* ws, const Workspace& w, bool accumulate, bool append,
                         int advance, bool new_f32, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (p.q_per_kv > 1)
    return launch_attend_gqa(p, plan, seqs, q, k_new, v_new, sel_idx, sel_cnt, out, lse, ws, w, accumulate, append,
                             advance, new_f32, st, ev_start, ev_stop);
  AttendArgs A;
  A.seqs = seqs; A.q = (const char*)q; A.k_new = (const char*)k_new; A.v_new = (const char*)v_new;
  A.sel_idx = sel_idx; A.sel_cnt = sel_cnt; A.out = (char*)out; A.lse = lse;
  A.logits = reinterpret_cast<float*>(ws + w.logits_off);
  A.part_ml = reinterpret_cast<float*>(ws + w.part_ml_off);
  A.part_acc = reinterpret_cast<float*>(ws + w.part_acc_off);
  A.n_heads = p.n_heads; A.sel_cap = p.sel_cap; A.lg_stride = w.lg_stride;
  A.chunk_max = plan.chunk_max; A.cap = p.cap;
  A.accumulate = accumulate ? 1 : 0; A.append = append ? 1 : 0; A.advance = advance;
  A.new_f32 = (new_f32 && append) ? 1 : 0;
  A.vcos_fused = p.score_mode == ADSA_SCORE_VCOS_FUSED ? 1 : 0;
  const int eb = elem_bytes(p);
  A.slot_stride_b = (long long)p.kv_slot_stride * eb;
  A.head_stride_b = (long long)p.kv_head_stride * eb;
  const float scale = p.softmax_scale != 0.0f ? p.softmax_scale : 1.0f / sqrtf((float)p.head_dim);
  A.scale_log2 = scale * kLog2e;
  const int key = eb * 1000 + p.head_dim;
  if (key == 2064) return launch_attend_t<2, 64>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 2128) return launch_attend_t<2, 128>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 4064) return launch_attend_t<4, 64>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 4128) return launch_attend_t<4, 128>(A, plan, p.n_seq, st, ev_start, ev_stop);
  return hipErrorInvalidValue;
}

}  // namespace adsa
