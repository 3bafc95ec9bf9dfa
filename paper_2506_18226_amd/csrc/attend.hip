// Gather flash-decode of the ADSA decode path (gfx950): Eq. 5's gather fused with softmax
// attention over the selected slots, plus the cache append (Section 4.2) and the per-head
// attention-mass update, in ONE launch.
//
//  k_attend<EB, D, HT, U, NW, VF, DIRECT, WIDE, RANK, PLAN> : grid (token chunk, HT heads, sequence), NW waves.
//    HT = 1: a 16-byte-per-lane streaming load of one wave covers RPW = 64 / (D*EB/16) consecutive tokens of ONE head.
//    That holds for [slot][head][D] caches too: a row is 128 bytes or more, whole cache lines, so a workgroup that
//    walks one head's rows at a stride fetches nothing it does not use.  But it visits every page of the sequence for its
//    128 or 256 bytes a token, and so do the workgroups of the other heads: large launches over such caches take
//    512 bytes of a token (HT heads) per workgroup; the rule and its figures stand in make_attend_plan.
//    q.k is reduced over the lanes of a row with DPP; every lane keeps an online-softmax state (m, l, acc) in
//    registers, fp32, log2 domain.  The lane groups of a wave merge in registers (DPP and 16-/32-lane
//    swaps), the waves through one small LDS record each.
//    With one chunk per (sequence, head) the workgroup writes out / lse itself and adds the probabilities it produced
//    to its OWN head's row of score[].  Except with PLAN no workgroup ever talks to another one of its launch.
//    With several chunks, each writes a partial and the scaled logits to the workspace and a second kernel,
//    k_attend_finish, merges them and updates the scores.
//    VF (ADSA_SCORE_VCOS_FUSED): every V row that streams through also yields its head's share of |v|^2
//    and of v.u (u = running sum of the candidates' normalised V, Eq. 2-3), stored per (head, slot): the
//    next eviction ranks from them instead of re-reading V.
//    RANK: the ranking of a small decode step too.  The workgroup leaves score[], pos and the record as they are and writes the new scores of
//    its head, of all resident slots, to the workspace; k_step_finish, the next kernel, puts them in place.
//    PLAN: the eviction plans of larger steps too, by the last workgroup of a sequence that closed a row, from scores that the sequence's other
//    workgroups have just stored, on any XCD.  What orders this is the hardware alone: score[] is stored and loaded with scope agent, past
//    the L2s; a thread's stores are acknowledged (s_waitcnt vmcnt(0)) and its workgroup's threads have met before the relaxed ticket
//    is drawn, and nothing is loaded before the last one has come back.  A plain store or load of score[] of such a sequence, in the
//    update or in plan_row_end, would be a race; pos, the record and the list come from earlier launches and are read plainly.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "adsa_rank.h"

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
  if (LPR >= 32) x = xor_sum<16>(x);
  return x;
}

// 16 bytes of a row as fp32 values, and their dot product with the lane's piece of q.  bf16: two products per instruction
// (v_dot2, fp32 sums), so q stays as it arrived and the softmax scale is applied to the sum; fp32: q is scaled beforehand.
template <int EB> struct Elems;
template <> struct Elems<2> {      // bf16: 8 values per 16-byte vector
  static constexpr int N = 8;
  uint32_t q[4];
  __device__ __forceinline__ Elems(const uint4& r, float) : q{r.x, r.y, r.z, r.w} {}
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xFFFF0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xFFFF0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xFFFF0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xFFFF0000u);
  }
  __device__ __forceinline__ float dot(const uint4& r) const {
    const uint32_t k[4] = {r.x, r.y, r.z, r.w};
    float d = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q[i]), __builtin_bit_cast(bf16x2, k[i]), d, false);
    return d;
  }
  static __device__ __forceinline__ float scaled(float d, float scale) { return d * scale; }
};
template <> struct Elems<4> {      // fp32: 4 values per 16-byte vector
  static constexpr int N = 4;
  float q[4];
  __device__ __forceinline__ Elems(const uint4& r, float scale) {
    unpack(r, q);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] *= scale;
  }
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ __forceinline__ float dot(const uint4& r) const {
    float k[4], d = 0.0f;
    unpack(r, k);
#pragma unroll
    for (int i = 0; i < 4; ++i) d = fmaf(q[i], k[i], d);
    return d;
  }
  static __device__ __forceinline__ float scaled(float d, float) { return d; }
};

// max(a, b, c) of which none is a signalling NaN (fmaxf would first quiet each of them)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// acc = acc * c + x where acc is kept (left to itself the compiler lets x's register become the sum and copies all of them back
// wherever the pairs of a last revolution are left out)
__device__ __forceinline__ void rescale_add(float& acc, float c, float x) { asm("v_fma_f32 %0, %0, %1, %2" : "+v"(acc) : "v"(c), "v"(x)); }
// a raw list entry inside the cache: no lane touches memory outside it
__device__ __forceinline__ int clamp_slot(int raw, int last) {
  int r;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(raw), "s"(last));
  return r;
}
constexpr float kLowest = -3.4028234663852886e38f;     // the running maximum of a state that has seen no token: z - kLowest is never NaN

// Entry of the staged list: the slot, or a negative number of it where it is not attended in the loop (see RowBuffer).
constexpr int kUnattended = ~ADSA_MAX_CAP;
__device__ __forceinline__ int list_entry(int slot, bool attended) { return slot ^ (attended ? 0 : kUnattended); }
__device__ __forceinline__ int slot_of(int entry) { return entry < 0 ? entry ^ kUnattended : entry; }

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
  int n_heads, sel_cap, lg_stride, cap;
  int accumulate, append, advance;     // advance: see kAdvance
  int new_f32;                         // k_new / v_new are fp32 although the cache is bf16: round as they enter
  int vcos_fused;
  long long slot_stride_b, head_stride_b;
  uint32_t stride24;    // slot_stride_b where a workgroup's rows can be reached with 32-bit offsets (see short_offsets), else 0
  float scale_log2;     // softmax scale * log2(e)
};

// What a workgroup needs when its rows are summed (or, WIDE, for 64-bit offsets): a block of 16 dwords behind the leading arguments.
struct AttendTail {
  char* out;
  float* lse;
  float* logits;
  float* part_ml;
  float* part_acc;
  int lg_stride, advance;
  long long slot_stride_b, unused;
};
static_assert(sizeof(AttendTail) == 64, "one dword per lane of a 16-lane row");

// The same for a launch that ranks for itself (RANK).
struct RankTail {
  char* out;
  float* lse;
  float* vals;          // [n_seq][n_heads][cap]   the resident slots' scores after this step's attention
  int32_t* plan;        // [n_seq][4]   see k_step_finish
  int total, W, R, w, recent_m;
  float inv_w;
  int unused[2];
};
static_assert(sizeof(RankTail) == 64 && offsetof(RankTail, out) == offsetof(AttendTail, out) && offsetof(RankTail, lse) == offsetof(AttendTail, lse), "one dword per lane of a 16-lane row");

// The same for a launch that plans the evictions of row ends (PLAN).
struct PlanTail {
  char* out;
  float* lse;
  int32_t* plan;        // [n_seq][4]   { ticket, then old n_res; first slot that moves; did compact; new n_res }, zeroed by k_select
  int32_t* keep_map;    // [n_seq][cap]
  int W, R, total, advance;
  float inv_w;
  int recent_m, unused[2];
};
static_assert(sizeof(PlanTail) == 64 && offsetof(PlanTail, out) == offsetof(AttendTail, out) && offsetof(PlanTail, lse) == offsetof(AttendTail, lse) &&
              offsetof(PlanTail, advance) == offsetof(AttendTail, advance), "one dword per lane of a 16-lane row");

// Section 4.2's per-row plan of one sequence whose scores this launch's workgroups have just stored (k_compact_plan on which scores
// are kept and where): keep map, positions, plan words and record.  The cache and score rows are moved by the next kernel on the stream.
// (8 rows at once: 12 with 3 slots a thread cost 9 to 19 registers, a step of 300 x 24 x 600 191.8 -> 194.4 us, 32 x 24 39.2 -> 38.5.)
template <int NT, int S>
__device__ __forceinline__ void plan_row_end(RankShared& sh, ADSA_GLOBAL adsa_seq& sq, int s, int rows, int cap, const GridWidth& grid, int R, int recent_m,
                                             gint* plan, gint* map) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), n = sq.n_res;
  gint* const pos = (gint*)sq.pos;
  const QueryCell cell = make_query_cell(sq, s, grid, R, 0, recent_m);
  int idx[S], posv[S];
  float rank[S];
  rank_clear<NT>(sh);
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = min(u * NT + tid, n - 1);
    posv[u] = elem(pos, idx[u]);
  }
  rank_values<S, S == 1 ? 24 : 8, true>((const gfloat*)sq.score, rows, cap, idx, rank);
  uint32_t key[S], restm = 0, in = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (u * NT + tid < n) in |= 1u << u;
    if (((in >> u) & 1u) && evict_class(cell, posv[u]) == 1) restm |= 1u << u;
    key[u] = order_key(rank[u], true);
  }
  const Stats st = block_stats<NT, S>(sh, key, restm, false);
  const uint32_t B = (uint32_t)effective_budget(sq, s);
  uint32_t T, need_eq;
  top_threshold<NT, S>(sh, key, restm, st, B < st.n_cand ? B : st.n_cand, &T, &need_eq);
  uint32_t sure = in & ~restm, eq = 0, dest[S], n_new;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (((restm >> u) & 1u) && key[u] > T) sure |= 1u << u;
    if (((restm >> u) & 1u) && key[u] == T) eq |= 1u << u;
  }
  const uint32_t take = place_kept<NT, S>(sh, sure, eq, need_eq, dest, &n_new);
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int i = u * NT + tid;
    const bool kept = (take >> u) & 1u;
    if ((in >> u) & 1u) map[i] = kept ? (int32_t)dest[u] : -1;
    if (kept && dest[u] != (uint32_t)i) pos[dest[u]] = posv[u];
    const unsigned long long gone = __ballot(((in >> u) & 1u) && !kept);
    if (gone != 0 && lane == 0) atomicMin(&sh.first, (uint32_t)(u * NT + wave_id() * kWave + __ffsll((long long)gone) - 1));
  }
  __syncthreads();                                  // (sh.first is complete)
  if (tid == 0) {
    plan[0] = n; plan[1] = (int)min(sh.first, (uint32_t)n); plan[2] = 1; plan[3] = (int32_t)n_new;
    sq.n_res = (int32_t)n_new;
    sq.compacted = 1;
  }
}

// DIRECT: the list of a (sequence, head) is not split (grid.x == 1): the workgroup finishes its heads alone.
// The build asks for leading kernel arguments to be preloaded into scalar registers at wave launch, and 14 dwords of them are.
// Everything up to the sums is in those 14 (addresses have 48 bits, so six of them take 9 dwords): the first round trip is then
// the count, the record, the list, q and the query token's row, and nothing waits for the argument block, whose scalar load
// takes longer (0.85 us) than those and could not be told from them by a wait count.  The block's rest is fetched by a vector
// load behind the first rows' and read from its lanes at the end.
//   heads_flags: heads | append << 16 | fp32 rows << 17 | accumulate << 18 | upper 5 bits of the head stride << 19 | chunks << 24;
//   caps: cap | sel_cap << 16
// HT > 1: the workgroup takes HT heads, the lane groups of a wave-load being the HT heads of RPW / HT tokens.
// RANK > 0: one launch of a decode step of few (sequence, head) pairs instead of k_select and this one.  Every workgroup of a sequence
// ranks its slots, RANK per thread, for itself, with the append planned, and attends the list it gets, which needs no trip through
// memory.  It only reads the record, pos and score, which the sequence's other workgroups may be reading still: what changes of
// them goes to the workspace, for k_step_finish, the next kernel on the stream (the first head's workgroup writes sel_idx, sel_cnt and
// the plan; a rejected record is marked here, which is what the others find too).
// PLAN > 0: k_compact_plan's work at a row end, by the sequence's last workgroup to end, PLAN slots per thread, while other sequences are
// still attended.  A sequence that closed a row stores its scores with scope agent and draws tickets; the others pay for nothing, and
// nobody waits.  A score's store and load with scope agent meet behind the L2s; the store has been acknowledged (vmcnt) before the ticket is
// drawn, and the loads leave after the last ticket has come back, so no cache is written back or invalidated for it.
// The record's step stays, since workgroups that start later tell a row end from it: the next kernel advances it.
template <int EB, int D, int HT, int U, int NW, bool VF, bool DIRECT, bool WIDE, int RANK = 0, int PLAN = 0>
__global__ __launch_bounds__(NW * kWave) void k_attend(uint32_t seqs_lo, uint32_t idx_lo, uint32_t cnt_lo, uint32_t q_lo, uint32_t kn_lo,
                                                      uint32_t vn_lo, uint32_t seqs_idx_hi, uint32_t cnt_q_hi, uint32_t kn_vn_hi,
                                                      uint32_t heads_flags, uint32_t caps, uint32_t stride24, uint32_t head_stride16,
                                                      float scale_log2, std::conditional_t<(RANK > 0), RankTail, std::conditional_t<(PLAN > 0), PlanTail, AttendTail>> T) {
  constexpr int kAttThreads = NW * kWave;           // the waves of the workgroup share one token chunk
  constexpr int EPL = Elems<EB>::N;                 // elements per lane
  constexpr int LPR = D / EPL;                      // lanes per row
  constexpr int RPW = kWave / LPR / HT;             // tokens per wave-load
  static_assert(HT == 1 || (DIRECT && !VF && RPW * HT * LPR == kWave), "several heads: whole lists only");
  static_assert(RANK == 0 || (HT == 1 && DIRECT && !VF && !WIDE), "ranking: whole lists of one head");
  static_assert(PLAN == 0 || (RANK == 0 && HT == 1 && DIRECT && !VF && !WIDE), "plans: whole lists of one head");
  constexpr int kSlots = RANK > 0 ? RANK : 1;       // slots per thread of the ranking
  constexpr int PF = 4;                             // list entries a thread fetches, and score read-modify-writes it starts, early
  constexpr int kRev = NW * U * RPW;                // tokens of one ring revolution of the workgroup
  extern __shared__ int s_ent[];                    // the chunk's slot list [n_ent], then logits [HT][n_ent] ([2][n_ent] for VF)
  __shared__ int s_new[NW];
  // merge: the lane groups of a wave meet in registers, the waves through these (one state per wave)
  __shared__ float s_wm[NW * HT], s_wl[NW * HT];
  __shared__ __attribute__((aligned(16))) float s_wacc[NW * HT * D];

  const int chunk = DIRECT ? 0 : blockIdx.x, b = blockIdx.z;
  const int n_chunks = DIRECT ? 1 : heads_flags >> 24;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n_heads = heads_flags & 0xFFFF, sel_cap = caps >> 16, cap = caps & 0xFFFF;
  const bool append = (heads_flags & 0x10000) != 0, new_f32 = EB == 2 && (heads_flags & 0x20000) != 0, accumulate = (heads_flags & 0x40000) != 0;
  // token and head of this lane's row within a wave-load, 16-byte piece of the row (heads past the last repeat it)
  const int dl = lane % LPR, ts = lane / LPR / HT, hs = HT == 1 ? 0 : lane / LPR % HT;
  const int head0 = blockIdx.y * HT, head = HT == 1 ? head0 : min(head0 + hs, n_heads - 1), heads_here = HT == 1 ? 1 : min(HT, n_heads - head0);

  // ---- first round trip: everything that depends on the kernel arguments only -- the count, the
  // sequence record, q and (when the list is not split, so its chunk starts at 0) the first slots of
  // the loop and the slots whose score words this thread updates at the end.  The record and the
  // count are pinned here so that they cannot drift behind the count test below.
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)address(seqs_lo, seqs_idx_hi & 0xFFFF) + b;
  int cnt = 0, pending = -1;
  if constexpr (RANK == 0) {
    cnt = ((const gint*)address(cnt_lo, cnt_q_hi & 0xFFFF))[b];
    pending = sqp->pending_slot;
  }
  gchar* const k_base = (gchar*)sqp->k;
  gchar* const v_base = (gchar*)sqp->v;
  gfloat* const score = (gfloat*)sqp->score;
  // (RANK: the rest of the record, as the ranking needs it)
  const int step = RANK > 0 || PLAN > 0 ? sqp->step : 0, status_in = RANK > 0 ? sqp->status : 0;
  const gint* const pos = RANK > 0 ? (const gint*)sqp->pos : nullptr;
  const BudgetOf budget(*sqp);
  const int n_keep_prefix = RANK > 0 ? sqp->n_keep_prefix : 0;
  int n_res = RANK > 0 ? sqp->n_res : 0;
  gfloat* const u_state = VF ? (gfloat*)sqp->vcos_u : nullptr;
  __builtin_amdgcn_sched_barrier(0);                // (the scalar loads leave first: the rows need them and the first slots)
  const gint* const idx_row = (const gint*)address(idx_lo, seqs_idx_hi >> 16) + (size_t)b * sel_cap;
  const size_t row_off = ((size_t)b * n_heads + head) * D * EB + dl * 16;
  // The wave takes the RPW-token units wave, wave + NW, ... of the chunk, in that order; unit number k of the
  // wave holds, for this lane, token (wave + k * NW) * RPW + ts.  slot_a[u]: slot of unit u.  pf_slot: the whole list
  // (its first PF * threads entries), one entry per thread and round: staged in LDS below, where the loop finds its slots.
  // (These loads need nothing but preloaded arguments: they leave before anything waits for a scalar load.)
  int slot_a[U];
  int pf_slot[PF];
  const SlotList list(idx_row, sel_cap);
  const int unit0 = wave * RPW + ts;                // this lane's token of the wave's first unit
  uint32_t tail = 0u;                               // lane i (modulo 16): dword i of T
  auto load_tail = [&] {
    tail = ((const ADSA_GLOBAL uint32_t*)((const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr() + kLeadBytes))[lane % 16];
  };
  auto tail_word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)tail, i); };
  auto tail_address = [&](size_t at) { return address(tail_word(at / 4), tail_word(at / 4 + 1)); };
  if constexpr (RANK > 0) load_tail();
  else if constexpr (DIRECT) {
#pragma unroll
    for (int u = 0; u < U; ++u) slot_a[u] = list[unit0 + u * NW * RPW];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < PF; ++k) pf_slot[k] = list[tid + k * kAttThreads];
  }
  const uint4 qr = load16((const gchar*)address(q_lo, cnt_q_hi >> 16) + row_off);
  // the query token's own K/V row (Section 4.2 append): the last wave, which has the fewest units, attends and stores it, 16 bytes of
  // K and V per lane.
  // fp32 rows of a bf16 cache (twice as many bytes) are rounded once, when they are used
  uint4 nk[4 / EB], nv[4 / EB];
  if (append && wave == NW - 1) {
    const gchar* const k_new_g = (const gchar*)address(kn_lo, kn_vn_hi & 0xFFFF) + (new_f32 ? 2 * row_off : row_off);
    const gchar* const v_new_g = (const gchar*)address(vn_lo, kn_vn_hi >> 16) + (new_f32 ? 2 * row_off : row_off);
    nk[0] = load16(k_new_g);
    nv[0] = load16(v_new_g);
    if constexpr (EB == 2)
      if (new_f32) { nk[1] = load16(k_new_g + 16); nv[1] = load16(v_new_g + 16); }
  }
  pin_uniform(cnt); pin_uniform(k_base); pin_uniform(v_base); pin_uniform(score); pin_uniform(pending);
  if constexpr (VF) pin_uniform(u_state);

  cnt = min(cnt, sel_cap);
  // ---- RANK: k_select's part, of which this thread keeps the places of its slots and their old scores of this head
  uint32_t dest[kSlots], take = 0;
  float old_score[kSlots];
  int n_ranked = 0;                                  // resident slots, the query token's included
  if constexpr (RANK > 0) {
    constexpr int NT = kAttThreads, S = kSlots;
    __shared__ __align__(16) RankShared sh;
    rank_clear<NT>(sh);
    const bool active = step >= 0 && status_in == 0, sane = n_res >= 0 && n_res <= cap, full = step >= 1 && n_res >= cap;
    const int slot_new = step >= 1 ? n_res : -1;     // the end of the cache: where the query token goes
    const int n = slot_new + 1 > 0 ? slot_new + 1 : n_res;
    n_ranked = n;
    int idx[S], posv[S];
    float rank[S];
#pragma unroll
    for (int u = 0; u < S; ++u) { idx[u] = min(u * NT + tid, n - 1); posv[u] = 0; rank[u] = old_score[u] = 0.0f; dest[u] = 0; }
    const bool reads = active && sane && !full && n > 0;      // (an empty sequence's pointers may be null)
    if (reads) {
#pragma unroll
      for (int u = 0; u < S; ++u) { posv[u] = elem(pos, idx[u]); old_score[u] = elem(score + (size_t)head * cap, idx[u]); }
    }
    __builtin_amdgcn_sched_barrier(0);               // (what follows while these are on their way: before them it costs 1 % of a small step)
    // As in k_select, the ranks need not be read where the budget covers every position that can be a candidate; here every head's workgroup
    // would read every head's scores.  adsa_step of 1 sequence x 900 tokens x 64 that attends them all, us with three launches | with them
    // read | with this rule: 24 heads 12.5 | 12.8 | 11.5, 48 heads 12.7 | 14.7 | 11.7, 95 heads 13.6 | 18.8 | 12.1.
    const uint32_t B = (uint32_t)effective_budget(budget, step);
    const bool ranked = reads && (int)B < min(n, budget.grid_origin + step - 1 - n_keep_prefix);
    if (__builtin_expect(ranked, 1)) rank_values<S, S == 1 ? 24 : 12>(score, n_heads, cap, idx, rank);
    const int total = (int)tail_word(offsetof(RankTail, total) / 4);
    uint32_t reject = !active ? 0u : !sane || step > total ? ADSA_SEQ_BAD_STATE : full ? ADSA_SEQ_CACHE_FULL : 0u;
    if (active && reject == 0) {
      const GridWidth grid = {(int)tail_word(offsetof(RankTail, W) / 4), __uint_as_float(tail_word(offsetof(RankTail, inv_w) / 4))};
      struct { int grid_origin, n_keep_prefix; } cell_of = {budget.grid_origin, n_keep_prefix};
      const QueryCell cell = make_query_cell(cell_of, step, grid, (int)tail_word(offsetof(RankTail, R) / 4), (int)tail_word(offsetof(RankTail, w) / 4),
                                             (int)tail_word(offsetof(RankTail, recent_m) / 4));
      uint32_t key[S], candm = 0, fixedm = 0;
      bool bad = false;
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int i = u * NT + tid, c = i == slot_new ? 0 : select_class(cell, posv[u]);
        key[u] = order_key(rank[u], true);
        bad |= i < n && c < 0;
        if (i < n && c == 1) candm |= 1u << u;
        if (i < n && c != 1) fixedm |= 1u << u;
        if (i == slot_new) old_score[u] = 0.0f;      // a new slot starts at 0
      }
      Stats st = block_stats<NT, S>(sh, key, candm, bad);
      if (__builtin_expect(!ranked && B < st.n_cand, 0)) {                // (uniform) positions were not distinct after all
        rank_values<S, S == 1 ? 24 : 12>(score, n_heads, cap, idx, rank);
#pragma unroll
        for (int u = 0; u < S; ++u) key[u] = order_key(rank[u], true);
        __syncthreads();
        st = block_stats<NT, S>(sh, key, candm, bad);
      }
      if (st.bad) reject = ADSA_SEQ_BAD_STATE;
      else {
        uint32_t thr, need_eq, sure = fixedm, eq = 0, count;
        top_threshold<NT, S>(sh, key, candm, st, min(B, st.n_cand), &thr, &need_eq);
#pragma unroll
        for (int u = 0; u < S; ++u) {
          if (((candm >> u) & 1u) && key[u] > thr) sure |= 1u << u;
          if (((candm >> u) & 1u) && key[u] == thr) eq |= 1u << u;
        }
        take = place_kept<NT, S>(sh, sure, eq, need_eq, dest, &count);
        gint* const out = const_cast<gint*>(idx_row);
#pragma unroll
        for (int u = 0; u < S; ++u)
          if (((take >> u) & 1u) && dest[u] < (uint32_t)sel_cap) {
            const int slot = u * NT + tid;
            s_ent[dest[u]] = list_entry(slot, slot != slot_new);
            if (head0 == 0) elem(out, dest[u]) = slot;
          }
        if (count > (uint32_t)sel_cap) reject = ADSA_SEQ_SEL_OVERFLOW;
        else cnt = (int)count;
      }
    }
    pending = reject == 0 && active ? slot_new : -1;
    gint* const plan = (gint*)tail_address(offsetof(RankTail, plan)) + 4 * b;
    if (head0 == 0 && tid == 0) {
      *reinterpret_cast<ADSA_GLOBAL u32x4*>(plan) = u32x4{0u, (uint32_t)(active && reject == 0 ? step : -1), (uint32_t)n, (uint32_t)cnt};
      ((gint*)address(cnt_lo, cnt_q_hi & 0xFFFF))[b] = cnt;
      if (reject != 0) sqp->status = status_in | (int)reject;
      if (!active || reject != 0) sqp->pending_slot = -1;
    }
  }
  if (cnt <= 0) {                                   // inactive or rejected sequence: zero-filled row
    if (chunk == 0) {
      const size_t row = (size_t)b * n_heads + head0;
      for (int o = tid; o < heads_here * D; o += kAttThreads) {
        if (EB == 4) ((gfloat*)T.out)[row * D + o] = 0.0f;
        else ((ADSA_GLOBAL uint16_t*)T.out)[row * D + o] = 0;
        if (o % D == 0) ((gfloat*)T.lse)[row + o / D] = 0.0f;
      }
      if constexpr (RANK == 0)
        if (head0 == 0 && tid == 0) advance_empty(sqp, T.advance);
    }
    return;
  }
  const int t_begin = DIRECT ? 0 : chunk_begin(cnt, chunk, n_chunks);
  const int t_end = DIRECT ? cnt : chunk_begin(cnt, chunk + 1, n_chunks);
  if (t_begin >= t_end) return;                     // fewer tokens than chunks
  const int len = t_end - t_begin;
  // The chunk's slot list, one entry per token (filled below), and entries of no token up to one revolution past the last unit.
  // Those and the query token's own are not attended in the loop.  The last word of a row of logits takes what belongs to no token.
  const int n_ent = ((len + kRev - 1) / kRev + 1) * kRev, dump = n_ent - 1;
  float* const s_logit = reinterpret_cast<float*>(s_ent + n_ent);
  if constexpr (!DIRECT) {
#pragma unroll
    for (int u = 0; u < U; ++u) slot_a[u] = list[t_begin + unit0 + u * NW * RPW];
#pragma unroll
    for (int k = 0; k < PF; ++k) pf_slot[k] = list[t_begin + tid + k * kAttThreads];
  }
  // the slot adsa_select reserved for the query token (Section 4.2 append), if this launch fills it
  const int new_slot = (append && pending < cap) ? pending : -1;

  const Elems<EB> qv(qr, scale_log2);
  long long stride_b = (long long)stride24;
  if constexpr (WIDE) stride_b = T.slot_stride_b;
  const long long head_stride_b = (long long)address(head_stride16, (heads_flags >> 19) & 0x1F) * 16;
  const long long lane_off = (long long)head * head_stride_b + dl * 16;
  gchar* const kb = k_base + lane_off;
  gchar* const vb = v_base + lane_off;
  // VF: this lane's columns of u for its head, and the two score rows of the head
  float uf[EPL];
  gfloat* vrows = nullptr;
  bool vf_on = false;
  if constexpr (VF) {
    vf_on = u_state != nullptr;
#pragma unroll
    for (int e = 0; e < EPL; ++e) uf[e] = vf_on ? u_state[(size_t)head * D + dl * EPL + e] : 0.0f;
    vrows = score + (size_t)(2 * head) * cap;
  }

  float pf_old[PF];
  float m = kLowest, l = 0.0f, acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.0f;

  // Rolling gather: U units (row pairs per lane) are in flight per wave.  Two units at a time are folded into the lane's
  // online-softmax state, which is brought to a new maximum once for both; a register quad is given to the load one
  // revolution ahead as soon as its contents are used (the K quads after the dot products, the V quads after the sums), so the
  // number of outstanding requests stays nearly constant instead of draining once per batch.
  // Small launches are bound by what this loop issues: 40 lists of 427 x 64 on 8 waves each keep a SIMD with 2 waves busy for
  // all of the 2.7 us between the slot list and the merge when a unit takes 102 issue slots (one unit at a time: a rescale per
  // unit, products of 64 bits for addresses, q.k on unpacked values, selects of the query token's row).  It took 54 with two units per
  // rescale and 32-bit addresses, and the launch 4.9 us instead of 5.6; 51 since what is not attended arrives as zeros instead of being
  // masked, with no copies of the sums behind the loop, no branches where the list is staged, and the outputs and the query token given
  // to the last wave: 4.90 -> 4.72 us; 16 x 130 x 64 fp32 3.88 -> 3.73, 320 x 427 x 64 8.86 -> 8.75, 128 x 1159 x 128 16.4 -> 16.2, 768 x
  // 640 x 64, which HBM bounds, 21.0 -> 20.9.  (16 waves for few pairs: 0.65 - 0.94 of the speed, their launch and first trip cost more
  // than the shorter loop saves.)
  {
    uint4 kr[U], vr[U];
    int ent[U], nxt[U];                             // entries of the units in flight at the ring positions; of those that take them next
    const int n_units = (len + RPW - 1) / RPW;
    const int n_mine = n_units > wave ? (n_units - wave + NW - 1) / NW : 0;       // units of this wave
    const int n_trips = max((n_mine + U - 1) / U, 1);
    // Requests leave in the order the program has them (the wait counts rely on it), and before the arithmetic that follows.
    auto in_order = [] {
      asm volatile("" : : : "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // Entries that are not attended read zeros without an access (RowBuffer; an entry that is a slot is at most the offset of its
    // row).  WIDE: they read slot 0 and are masked when they are folded.
    const RowBuffer ku(k_base + (long long)head0 * head_stride_b), vu(v_base + (long long)head0 * head_stride_b);       // uniform
    const uint32_t lane32 = (uint32_t)(head - head0) * (uint32_t)head_stride_b + (uint32_t)dl * 16u;
    auto load = [&](const RowBuffer& rows, const gchar* own, int e) -> uint4 {
      if constexpr (!WIDE) return rows[max(__umul24((uint32_t)e, stride24) + lane32, (uint32_t)e)];
      else return load_stream16(own + (long long)max(e, 0) * stride_b);
    };
    auto entry = [&](int j, int slot) { return list_entry(slot, j < len && slot != new_slot); };
    if constexpr (RANK > 0) {                      // the list is in LDS already, but for the entries of no token
      for (int j = cnt + tid; j < n_ent; j += kAttThreads) s_ent[j] = list_entry(0, false);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) slot_a[u] = s_ent[unit0 + u * NW * RPW];
    }
    // prologue: the pattern of a steady-state trip, so that the loop's wait counts match
#pragma unroll
    for (int u = 0; u < U; u += 2) {
#pragma unroll
      for (int i = u; i < u + 2; ++i) {
        ent[i] = RANK > 0 ? slot_a[i] : entry(unit0 + i * NW * RPW, clamp_slot(slot_a[i], cap - 1));
      }
      kr[u] = load(ku, kb, ent[u]);
      kr[u + 1] = load(ku, kb, ent[u + 1]);
      in_order();
      vr[u] = load(vu, vb, ent[u]);
      vr[u + 1] = load(vu, vb, ent[u + 1]);
      in_order();
    }
    // ... and while these rows are on their way the chunk's slot list goes to LDS
    if constexpr (RANK == 0) {
      load_tail();
      int new_at = 0;                               // 1 + list position of the query token's slot, if this thread stages it
      auto stage = [&](int j, int slot) {
        s_ent[j] = entry(j, slot);
        new_at = slot == new_slot && j < len ? j + 1 : new_at;
      };
#pragma unroll
      for (int k = 0; k < PF; ++k)
        if (k * kAttThreads < n_ent) {                // (uniform; n_ent is a multiple of the revolution, not of the threads)
          const int j = tid + k * kAttThreads;
          pf_slot[k] = clamp_slot(pf_slot[k], cap - 1);
          if (j < n_ent) stage(j, pf_slot[k]);
        }
      for (int j = tid + PF * kAttThreads; j < n_ent; j += kAttThreads) stage(j, clamp_slot(list[t_begin + j], cap - 1));
      if (new_slot >= 0) {                          // (uniform)
        const unsigned long long who = __ballot(new_at != 0);
        const int at = who ? __builtin_amdgcn_readlane(new_at, __ffsll((long long)who) - 1) : 0;
        if (lane == 0) s_new[wave] = at;
      }
      __syncthreads();
    }
    // thread i of the final score update serves tokens i, i + threads, ...; start the first PF reads now
    if (RANK == 0 && DIRECT && HT == 1 && accumulate) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        pf_old[k] = 0.0f;
        if (k * kAttThreads < len) pf_old[k] = *(const gfloat*)((const gchar*)(score + (size_t)head * cap) + (uint32_t)pf_slot[k] * 4u);
      }
    }
    // Section 4.2: the query token's row enters the cache, and, if its slot is in the list, one lane group (per head) of the
    // last wave starts its state with it, from the registers that hold it (no lane reads that row from memory)
    if (new_slot >= 0 && wave == NW - 1) {
      if constexpr (EB == 2)
        if (new_f32) {
          // (converted here, not where the compiler would like to: next to the loads, whose return it would wait for)
          asm volatile("" : "+v"(nk[1].x), "+v"(nk[1].y), "+v"(nk[1].z), "+v"(nk[1].w), "+v"(nv[1].x), "+v"(nv[1].y), "+v"(nv[1].z), "+v"(nv[1].w));
          nk[0] = pack8_bf16(nk[0], nk[1]);
          nv[0] = pack8_bf16(nv[0], nv[1]);
        }
      int at = cnt;                                 // RANK: the newest slot ends the list
      if constexpr (RANK == 0) {
        const int news = s_new[lane % NW];
        const unsigned long long who = __ballot(news != 0);
        at = who ? __builtin_amdgcn_readlane(news, __ffsll((long long)who) - 1) : 0;
      }
      const bool mine = ts == 0;
      if (mine && hs < heads_here && chunk == n_chunks - 1) {
        const long long off = (long long)new_slot * stride_b;
        store16(kb + off, nk[0]);
        store16(vb + off, nv[0]);
      }
      if (at > 0) {
        float z = Elems<EB>::scaled(row_sum<LPR>(qv.dot(nk[0])), scale_log2), vf[EPL];
        Elems<EB>::unpack(nv[0], vf);
        m = mine ? z : m;
        l = mine ? 1.0f : 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = mine ? vf[e] : 0.0f;
        if constexpr (VF) {
          float dv = 0.0f, sv = 0.0f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) { dv = fmaf(vf[e], uf[e], dv); sv = fmaf(vf[e], vf[e], sv); }
          dv = row_sum<LPR>(dv);
          sv = row_sum<LPR>(sv);
          if (mine) { s_logit[at - 1] = sv; s_logit[n_ent + at - 1] = dv; }
        } else {
          if (mine) s_logit[hs * n_ent + at - 1] = z;
        }
      }
    }
    const int* next = s_ent + (wave + U * NW) * RPW + ts;    // entries of the units one revolution ahead
    float* zpos = s_logit + (VF ? 0 : hs * n_ent) + wave * RPW + ts;
    float* const zdump = s_logit + (VF ? 0 : hs * n_ent) + dump;
#pragma unroll
    for (int u = 0; u < U; ++u) nxt[u] = next[u * NW * RPW];
    in_order();

    // units u and u + 1 of the ring; refill: their registers go to the units one revolution ahead
    auto fold = [&](int u, auto refill) {
      constexpr bool kRefill = decltype(refill)::value;
      const int ea = ent[u], eb = ent[u + 1];
      float da = qv.dot(kr[u]), db = qv.dot(kr[u + 1]);
      asm volatile("" : "+v"(da), "+v"(db) : : "memory");
      if constexpr (kRefill) {
        kr[u] = load(ku, kb, nxt[u]);
        kr[u + 1] = load(ku, kb, nxt[u + 1]);
        in_order();
      }
      da = Elems<EB>::scaled(row_sum<LPR>(da), scale_log2);
      db = Elems<EB>::scaled(row_sum<LPR>(db), scale_log2);
      const bool on_a = ea >= 0, on_b = eb >= 0;
      const float za = on_a ? da : -INFINITY, zb = on_b ? db : -INFINITY;
      float* const at_a = on_a ? zpos + u * NW * RPW : zdump;
      float* const at_b = on_b ? zpos + (u + 1) * NW * RPW : zdump;
      if constexpr (!VF) { *at_a = za; *at_b = zb; }         // (the lanes of a row write the same word)
      const float m_new = max3(m, za, zb);
      const float corr = fast_exp2(m - m_new), pa = fast_exp2(za - m_new), pb = fast_exp2(zb - m_new);
      m = m_new;
      l = fmaf(l, corr, pa + pb);
      uint4 xa = vr[u], xb = vr[u + 1];
      if constexpr (WIDE) {                         // (what a masked entry read may be anything: 0 times it need not be 0)
        xa = make_uint4(on_a ? xa.x : 0u, on_a ? xa.y : 0u, on_a ? xa.z : 0u, on_a ? xa.w : 0u);
        xb = make_uint4(on_b ? xb.x : 0u, on_b ? xb.y : 0u, on_b ? xb.z : 0u, on_b ? xb.w : 0u);
      }
      float va[EPL], vc[EPL];
      Elems<EB>::unpack(xa, va);
      Elems<EB>::unpack(xb, vc);
#pragma unroll
      for (int e = 0; e < EPL; ++e) rescale_add(acc[e], corr, fmaf(pb, vc[e], pa * va[e]));
      if constexpr (VF) {                         // Eq. 2-3 bookkeeping of these rows: |v_h|^2 and v_h . u_h
        float dva = 0.0f, sva = 0.0f, dvb = 0.0f, svb = 0.0f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          dva = fmaf(va[e], uf[e], dva); sva = fmaf(va[e], va[e], sva);
          dvb = fmaf(vc[e], uf[e], dvb); svb = fmaf(vc[e], vc[e], svb);
        }
        dva = row_sum<LPR>(dva); sva = row_sum<LPR>(sva);
        dvb = row_sum<LPR>(dvb); svb = row_sum<LPR>(svb);
        at_a[0] = sva; at_b[0] = svb;
        at_a[n_ent] = dva; at_b[n_ent] = dvb;
      }
      // the state is demanded HERE, and no memory access may cross: the units are folded completely before the loads that
      // reuse their registers are issued, and no later unit's arithmetic is pulled in front of them (left to itself the
      // compiler gathers all the logits of a trip first and so waits for the whole ring)
      static_assert(EPL == 4 || EPL == 8, "elements per lane");
      if constexpr (EPL == 8)
        asm volatile("" : "+v"(m), "+v"(l), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]),
                     "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]) : : "memory");
      else
        asm volatile("" : "+v"(m), "+v"(l), "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]) : : "memory");
      if constexpr (kRefill) {
        vr[u] = load(vu, vb, nxt[u]);
        vr[u + 1] = load(vu, vb, nxt[u + 1]);
        ent[u] = nxt[u]; ent[u + 1] = nxt[u + 1];
        nxt[u] = next[(u + U) * NW * RPW]; nxt[u + 1] = next[(u + 1 + U) * NW * RPW];
        in_order();
      }
    };
    for (int trip = 1; trip < n_trips; ++trip) {
#pragma unroll
      for (int u = 0; u < U; u += 2) fold(u, std::true_type());
      next += kRev;
      zpos += kRev;
    }
    // the last revolution; pairs without a unit of this wave are left out (wave-uniform)
#pragma unroll
    for (int u = 0; u < U; u += 2)
      if ((n_trips - 1) * U + u < n_mine) fold(u, std::false_type());
  }
  // ---- merge, step 1 (registers): the RPW lane groups of a wave that worked on the same head bring their states to the wave's
  // maximum and add them up across lanes.  The normaliser's sum goes to every lane; of the output, a swap of 32- or 16-lane
  // halves adds two elements at once and leaves one of them in each half, so that a lane ends up with kLeft elements from e0 on.
  constexpr int kGroups0 = LPR * HT;                 // lanes from one group of a head to its next
  constexpr int kLeft = EPL >> ((kGroups0 <= 32 ? 1 : 0) + (kGroups0 <= 16 ? 1 : 0));
  int e0 = 0;
  if constexpr (RPW > 1) {
    float M = m;
#pragma unroll
    for (int x = kGroups0; x < kWave; x <<= 1) M = x == 8 ? xor_max<8>(M) : x == 16 ? xor_max<16>(M) : xor_max<32>(M);
    const float sc = fast_exp2(m - M);              // 0 for a group that saw no token, unless no group did (then l and acc are 0)
    l *= sc;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] *= sc;
#pragma unroll
    for (int x = kGroups0; x < kWave; x <<= 1) l = x == 8 ? xor_sum<8>(l) : x == 16 ? xor_sum<16>(l) : xor_sum<32>(l);
    auto fold_halves = [&](auto width, int n) {     // acc[0 .. n) <- per half: acc[i] + its partner's, acc[i + n] in the upper half
#pragma unroll
      for (int i = 0; i < EPL / 2; ++i)
        if (i < n) {
          const uint32_t lo = __float_as_uint(acc[i]), hi = __float_as_uint(acc[i + n]);
          const u32x2 r = decltype(width)::value == 32 ? __builtin_amdgcn_permlane32_swap(lo, hi, false, false)
                                                       : __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
          acc[i] = __uint_as_float(r.x) + __uint_as_float(r.y);
        }
      e0 += (lane & decltype(width)::value) ? n : 0;
    };
    fold_halves(std::integral_constant<int, 32>(), EPL / 2);
    if constexpr (kGroups0 <= 16) fold_halves(std::integral_constant<int, 16>(), EPL / 4);
    if constexpr (kGroups0 <= 8) {
#pragma unroll
      for (int i = 0; i < kLeft; ++i) acc[i] = xor_sum<8>(acc[i]);
    }
    m = M;
  }
  // ---- step 2 (LDS): one state per wave; after ONE barrier every thread works out the
  // normaliser itself, the first D threads each finish one output element
  if (ts == 0 && dl == 0) { s_wm[wave * HT + hs] = m; s_wl[wave * HT + hs] = l; }
  {
    float* const dst = &s_wacc[(wave * HT + hs) * D + dl * EPL + e0];         // (lanes that hold the same elements write the same)
    if constexpr (kLeft == 4) *reinterpret_cast<float4*>(dst) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    else if constexpr (kLeft == 2) *reinterpret_cast<float2*>(dst) = make_float2(acc[0], acc[1]);
    else *dst = acc[0];
  }
  __syncthreads();
  gchar* const out_g = (gchar*)tail_address(offsetof(AttendTail, out));
  gfloat* const lse_g = (gfloat*)tail_address(offsetof(AttendTail, lse));
  const int advance = RANK > 0 ? kAdvanceNone : (int)tail_word(offsetof(AttendTail, advance) / 4);
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
        w[k] = fast_exp2(w[k] - M);
        L = fmaf(s_wl[k * HT + h], w[k], L);
        a = fmaf(s_wacc[(k * HT + h) * D + d], w[k], a);
      }
      const float val = __fdividef(a, L);
      const size_t row = (size_t)b * n_heads + head0 + h;
      if (EB == 4) reinterpret_cast<gfloat*>(out_g)[row * D + d] = val;
      else reinterpret_cast<ADSA_GLOBAL uint16_t*>(out_g)[row * D + d] = (uint16_t)f32_to_bf16_rne(val);
      if (d == 0) { s_lse2[h] = M + __log2f(L); lse_g[row] = s_lse2[h] * kLn2; }
    }
    if (accumulate) {
      __syncthreads();
      float lse2[HT];
#pragma unroll
      for (int h = 0; h < HT; ++h) lse2[h] = s_lse2[min(h, heads_here - 1)];
      for (int i = tid; i < len; i += kAttThreads) {
        gfloat* const at = score + (size_t)head0 * cap + slot_of(s_ent[i]);
        float old[HT];
#pragma unroll
        for (int h = 0; h < HT; ++h) old[h] = at[(size_t)min(h, heads_here - 1) * cap];
#pragma unroll
        for (int h = 0; h < HT; ++h)
          if (h < heads_here) at[(size_t)h * cap] = old[h] + fast_exp2(s_logit[h * n_ent + i] - lse2[h]);
      }
    }
    if (head0 == 0 && tid == 0) advance_step(sqp, advance);
    return;
  }
  // log2-domain normaliser of the whole workgroup, worked out by every wave from the waves' states: lane w (modulo NW) weighs wave w
  static_assert(NW == 4 || NW == 8, "reductions over 4 or 8 lanes");
  const float wm = s_wm[lane % NW];
  float M = max2(wm, dpp_f<0xB1>(wm));
  M = max2(M, dpp_f<0x4E>(M));
  if constexpr (NW == 8) M = max2(M, dpp_f<0x141>(M));
  const float weight = fast_exp2(wm - M);           // (a wave that saw no token: 0, or l and acc are 0)
  float L = s_wl[lane % NW] * weight;
  L += dpp_f<0xB1>(L);
  L += dpp_f<0x4E>(L);
  if constexpr (NW == 8) L += dpp_f<0x141>(L);
  const size_t row = (size_t)b * n_heads + head;
  const int d = tid - (kAttThreads - D);            // output element: the last waves have the fewest tokens of the score update
  if (d >= 0) {
    static_assert(D <= kAttThreads, "one output element per thread");
    float w[NW], part[NW], a = 0.0f;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      w[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(weight), k));
      part[k] = s_wacc[k * D + d];
    }
    __builtin_amdgcn_sched_barrier(0);              // (each product right behind its weight's readlane would wait for it)
#pragma unroll
    for (int k = 0; k < NW; ++k) a = fmaf(part[k], w[k], a);
    if constexpr (DIRECT) {
      const float val = __fdividef(a, L);
      if (EB == 4) reinterpret_cast<gfloat*>(out_g)[row * D + d] = val;
      else reinterpret_cast<ADSA_GLOBAL uint16_t*>(out_g)[row * D + d] = (uint16_t)f32_to_bf16_rne(val);
      if (d == 0) lse_g[row] = (M + __log2f(L)) * kLn2;
    } else {
      const size_t pidx = row * n_chunks + chunk;
      ((gfloat*)tail_address(offsetof(AttendTail, part_acc)))[pidx * D + d] = a;
      gfloat* const ml = (gfloat*)tail_address(offsetof(AttendTail, part_ml)) + pidx * 2;
      if (d == 0) { ml[0] = M; ml[1] = L; }
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
            const int slot = pf_slot[k];
            vrows[slot] = s_logit[j];
            vrows[cap + slot] = s_logit[n_ent + j];
          }
        }
        j0 = tid + PF * kAttThreads;
      }
      for (int j = j0; j < len; j += kAttThreads) {
        const int slot = slot_of(s_ent[j]);
        vrows[slot] = s_logit[j];
        vrows[cap + slot] = s_logit[n_ent + j];
      }
    }
  }
  if constexpr (DIRECT) {
    // -------- this head's attention mass: score[head][slot] += p, from the logits still in LDS
    if constexpr (RANK > 0) {
      gfloat* const vals = (gfloat*)tail_address(offsetof(RankTail, vals)) + row * cap;
      const float lse2 = M + __log2f(L);
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        const uint32_t slot = u * kAttThreads + tid;
        const float p = ((take >> u) & 1u) ? fast_exp2(s_logit[((take >> u) & 1u) ? dest[u] : 0u] - lse2) : 0.0f;
        if (slot < (uint32_t)n_ranked) elem(vals, slot) = ((take >> u) & 1u) ? old_score[u] + p : old_score[u];
      }
    } else if (accumulate) {
      const float lse2 = M + __log2f(L);
      gfloat* const srow = score + (size_t)head * cap;
      bool closes = false;                          // PLAN: the sequence closed a row
      if constexpr (PLAN > 0) {
        int col = 0;
        const int W = (int)tail_word(offsetof(PlanTail, W) / 4);
        if (step >= 1) GridWidth{W, __uint_as_float(tail_word(offsetof(PlanTail, inv_w) / 4))}.row(step - 1, &col);
        closes = step >= 1 && step <= (int)tail_word(offsetof(PlanTail, total) / 4) && col == W - 1;
      }
      auto put = [&](gfloat* at, float sum) {
        if (PLAN > 0 && closes) __hip_atomic_store(at, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else *at = sum;
      };
#pragma unroll
      for (int k = 0; k < PF; ++k) {                // reads were started before the loop
        const int i = tid + k * kAttThreads;
        if (k * kAttThreads < len) {                // (uniform)
          const float sum = pf_old[k] + fast_exp2(s_logit[min(i, len - 1)] - lse2);
          if (i < len) put((gfloat*)((gchar*)srow + (uint32_t)pf_slot[k] * 4u), sum);
        }
      }
      constexpr int B = 4;                          // longer lists: batches of reads, so that their latencies overlap
      for (int i0 = tid + PF * kAttThreads; i0 < len; i0 += B * kAttThreads) {
        float old[B];
        int slot[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
          slot[k] = slot_of(s_ent[min(i0 + k * kAttThreads, len - 1)]);
          old[k] = srow[slot[k]];
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
          const int i = i0 + k * kAttThreads;
          if (i < len) put(srow + slot[k], old[k] + fast_exp2(s_logit[i] - lse2));
        }
      }
      if constexpr (PLAN > 0) {
        if (!closes) return;
        __shared__ __align__(16) RankShared sh;
        __shared__ int s_last;
        gint* const plan = (gint*)tail_address(offsetof(PlanTail, plan)) + 4 * b;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this thread's scores are where every XCD sees them ...
        __syncthreads();                                       // ... and so are the workgroup's: it may draw its ticket
        if (tid == 0) s_last = __hip_atomic_fetch_add((int*)plan, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_heads - 1;
        __syncthreads();
        if (!s_last) return;
        const GridWidth grid = {(int)tail_word(offsetof(PlanTail, W) / 4), __uint_as_float(tail_word(offsetof(PlanTail, inv_w) / 4))};
        plan_row_end<kAttThreads, PLAN>(sh, *sqp, step, n_heads, cap, grid, (int)tail_word(offsetof(PlanTail, R) / 4),
                                        (int)tail_word(offsetof(PlanTail, recent_m) / 4), plan, (gint*)tail_address(offsetof(PlanTail, keep_map)) + (size_t)b * cap);
        return;
      }
    }
    // last act on a sequence (one thread; no other workgroup reads step): VF marks the score rows as the
    // next step's if u was (tags kept as floats behind u); then the step may advance.  (Written out here:
    // handing the kernel's argument struct to a helper by reference made every variant slower.)
    if (RANK == 0 && head == 0 && tid == 0) {
      if constexpr (VF) {
        if (u_state) {
          gfloat* tags = u_state + (size_t)n_heads * D;
          const float want = (float)(sqp->step + 2);
          tags[1] = tags[0] == want ? want : 0.0f;
        }
      }
      advance_step(sqp, advance);
    }
    return;
  } else {
    // -------- several chunks: this workgroup's partial and logits are in the workspace; k_attend_finish, the next kernel
    // on the stream, merges them (the launch boundary orders the two and makes the stores visible on every XCD)
    if (accumulate) {
      gfloat* const lg = (gfloat*)tail_address(offsetof(AttendTail, logits)) + row * tail_word(offsetof(AttendTail, lg_stride) / 4) + t_begin;
      for (int i = tid; i < len; i += kAttThreads) lg[i] = s_logit[i];
    }
  }
}

// Second half of a split launch: grid (token slice, head, sequence).  Every workgroup works out the head's softmax
// normaliser from the chunks' (m, l), in chunk order; slice 0 merges the partial outputs and writes out / lse; every
// slice adds the probabilities of its kFinishTokens tokens to the head's score row.
constexpr int kFinishThreads = 256, kFinishTokens = 4 * kFinishThreads;
template <int EB, int D>
__global__ __launch_bounds__(kFinishThreads) void k_attend_finish(
    uint32_t seqs_lo, uint32_t idx_lo, uint32_t cnt_lo, uint32_t out_lo, uint32_t lse_lo, uint32_t lg_lo, uint32_t ml_lo, uint32_t acc_lo,
    uint32_t seqs_idx_hi, uint32_t cnt_out_hi, uint32_t lse_lg_hi, uint32_t ml_acc_hi, uint32_t caps, uint32_t flags) {
  const int n_heads = flags & 0x1FF, advance = (flags >> 18) & 3, n_chunks = flags >> 24, cap = caps & 0xFFFF, sel_cap = caps >> 16;
  const bool accumulate = (flags & 0x10000) != 0, vcos_fused = (flags & 0x20000) != 0;
  const int slice = blockIdx.x, head = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)address(seqs_lo, seqs_idx_hi & 0xFFFF) + b;
  const int cnt = min(((const gint*)address(cnt_lo, cnt_out_hi & 0xFFFF))[b], sel_cap);
  gfloat* const score = (gfloat*)sqp->score;
  gfloat* const u_state = vcos_fused ? (gfloat*)sqp->vcos_u : nullptr;
  if (cnt <= 0 || slice * kFinishTokens >= cnt) return;      // (inactive sequences: zero rows, already written)
  const size_t row = (size_t)b * n_heads + head;
  const gfloat* const ml = (const gfloat*)address(ml_lo, ml_acc_hi & 0xFFFF) + row * n_chunks * 2;
  const gfloat* const acc = (const gfloat*)address(acc_lo, ml_acc_hi >> 16) + row * n_chunks * D;
  const gfloat* const lg = (const gfloat*)address(lg_lo, lse_lg_hi >> 16) + row * ((sel_cap + 3) / 4 * 4);
  const gint* const idx = (const gint*)address(idx_lo, seqs_idx_hi >> 16) + (size_t)b * sel_cap;
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
  if (accumulate) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int j = min(slice * kFinishTokens + u * kFinishThreads + tid, cnt - 1);
      slot[u] = min(max(idx[j], 0), cap - 1);
      z[u] = lg[j];
    }
#pragma unroll
    for (int u = 0; u < B; ++u) old[u] = score[(size_t)head * cap + slot[u]];
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
    if (EB == 4) reinterpret_cast<gfloat*>((gchar*)address(out_lo, cnt_out_hi >> 16))[oi] = val;
    else reinterpret_cast<ADSA_GLOBAL uint16_t*>((gchar*)address(out_lo, cnt_out_hi >> 16))[oi] = (uint16_t)f32_to_bf16_rne(val);
    if (tid == 0) ((gfloat*)address(lse_lo, lse_lg_hi & 0xFFFF))[row] = lse2 * kLn2;
  }
  if (accumulate) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int j = slice * kFinishTokens + u * kFinishThreads + tid;
      if (j < cnt) score[(size_t)head * cap + slot[u]] = old[u] + fast_exp2(z[u] - lse2);
    }
  }
  if (slice == 0 && head == 0 && tid == 0) {                 // last act on the sequence: see k_attend
    if (u_state) {
      gfloat* tags = u_state + (size_t)n_heads * D;
      const float want = (float)(sqp->step + 2);
      tags[1] = tags[0] == want ? want : 0.0f;
    }
    advance_step(sqp, advance);
  }
}

template <int EB, int D, int HT, int NW, bool VF, bool DIRECT, bool WIDE>
hipError_t launch_attend_w(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  // Row pairs in flight per lane.  us with 2 | 3 | 4 | 6 | 8, bf16: 768 pairs x 647 tokens x 64 22.6 | 22.2 | 22.3 | 22.8 | 23.3; 128 x
  // 1159 x 128 19.4 | 17.5 | 17.6 | 18.0 | 19.1; 40 x 427 x 64 5.8 | 5.8 | 5.6 | 7.0 | 6.4; fp32 63 x 433 x 128 13.0 | 11.3 | 11.5 | 12.2 |
  // 13.1; only 320 x 427 x 64, whose lists fill 3.3 revolutions of 4, is better off with 3: 9.9 | 9.6 | 10.2 | 11.4 | 11.3.
  constexpr int U = 4;
  constexpr int kRev = NW * U * (kWave * 16 / (D * EB) / HT);                           // tokens of a ring revolution
  const size_t entries = (size_t)((plan.chunk_max - 1 + kRev - 1) / kRev + 1) * kRev;
  const size_t lds = ((VF ? 2 : HT) + 1) * entries * sizeof(float);                     // the slot list + logits rows
  dim3 grid(plan.n_chunks, (A.n_heads + HT - 1) / HT, n_seq);
  const uint32_t flags = A.n_heads | (A.append ? 0x10000 : 0) | (A.new_f32 ? 0x20000 : 0) | (A.accumulate ? 0x40000 : 0) | (uint32_t)(A.head_stride_b >> 36 & 0x1F) << 19 |
                         plan.n_chunks << 24;
  const AttendTail T = {A.out, A.lse, A.logits, A.part_ml, A.part_acc, A.lg_stride, A.advance, A.slot_stride_b, 0};
  // (a split launch is two kernels: the start event belongs to the first, the stop event to the second)
  auto launch = [&](auto go) {
    go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.q), lo32(A.k_new), lo32(A.v_new), hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.q), hi16s(A.k_new, A.v_new),
       flags, (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, A.stride24, (uint32_t)(A.head_stride_b / 16), A.scale_log2, T);
  };
  if (ev_start && ev_stop)
    launch([&](auto... args) {
      hipExtLaunchKernelGGL((k_attend<EB, D, HT, U, NW, VF, DIRECT, WIDE>), grid, dim3(NW * kWave), (uint32_t)lds, st, ev_start,
                            DIRECT ? ev_stop : nullptr, 0, args...);
    });
  else
    launch([&](auto... args) { hipLaunchKernelGGL((k_attend<EB, D, HT, U, NW, VF, DIRECT, WIDE>), grid, dim3(NW * kWave), lds, st, args...); });
  if constexpr (!DIRECT) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 fgrid(A.accumulate ? (A.sel_cap + kFinishTokens - 1) / kFinishTokens : 1, A.n_heads, n_seq);
    const uint32_t fflags = A.n_heads | (A.accumulate ? 0x10000 : 0) | (A.vcos_fused ? 0x20000 : 0) | (uint32_t)A.advance << 18 | plan.n_chunks << 24;
    auto finish = [&](auto go) {
      go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.out), lo32(A.lse), lo32(A.logits), lo32(A.part_ml), lo32(A.part_acc),
         hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.out), hi16s(A.lse, A.logits), hi16s(A.part_ml, A.part_acc),
         (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, fflags);
    };
    if (ev_start && ev_stop)
      finish([&](auto... args) { hipExtLaunchKernelGGL((k_attend_finish<EB, D>), fgrid, dim3(kFinishThreads), 0, st, nullptr, ev_stop, 0, args...); });
    else
      finish([&](auto... args) { hipLaunchKernelGGL((k_attend_finish<EB, D>), fgrid, dim3(kFinishThreads), 0, st, args...); });
  }
  return hipGetLastError();
}

// A decode step's ranking and attention in one launch (rank_in_attend), S slots per thread.
template <int EB, int D, int NW, int S>
hipError_t launch_ranked(const AttendArgs& A, const RankTail& T, const AttendPlan& plan, int n_seq, hipStream_t st, hipEvent_t ev_start,
                         hipEvent_t ev_stop) {
  constexpr int U = 4, kRev = NW * U * (kWave * 16 / (D * EB));
  const size_t entries = (size_t)((plan.chunk_max - 1 + kRev - 1) / kRev + 1) * kRev, lds = 2 * entries * sizeof(float);
  const dim3 grid(1, A.n_heads, n_seq), block(NW * kWave);
  const uint32_t flags = A.n_heads | 0x10000 | (A.new_f32 ? 0x20000 : 0) | 0x40000 | (uint32_t)(A.head_stride_b >> 36 & 0x1F) << 19 | 1u << 24;
  auto launch = [&](auto go) {
    go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.q), lo32(A.k_new), lo32(A.v_new), hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.q), hi16s(A.k_new, A.v_new),
       flags, (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, A.stride24, (uint32_t)(A.head_stride_b / 16), A.scale_log2, T);
  };
  if (ev_start && ev_stop)
    launch([&](auto... args) { hipExtLaunchKernelGGL((k_attend<EB, D, 1, U, NW, false, true, false, S>), grid, block, (uint32_t)lds, st, ev_start, ev_stop, 0, args...); });
  else
    launch([&](auto... args) { hipLaunchKernelGGL((k_attend<EB, D, 1, U, NW, false, true, false, S>), grid, block, lds, st, args...); });
  return hipGetLastError();
}

// An attention launch that plans the evictions of row ends (plan_in_attend), S slots per thread.
template <int EB, int D, int S>
hipError_t launch_planned(const AttendArgs& A, const PlanTail& T, const AttendPlan& plan, int n_seq, hipStream_t st, hipEvent_t ev_start,
                          hipEvent_t ev_stop) {
  constexpr int U = 4, NW = 4, kRev = NW * U * (kWave * 16 / (D * EB));
  const size_t entries = (size_t)((plan.chunk_max - 1 + kRev - 1) / kRev + 1) * kRev, lds = 2 * entries * sizeof(float);
  const dim3 grid(1, A.n_heads, n_seq), block(NW * kWave);
  const uint32_t flags = A.n_heads | 0x10000 | (A.new_f32 ? 0x20000 : 0) | 0x40000 | (uint32_t)(A.head_stride_b >> 36 & 0x1F) << 19 | 1u << 24;
  auto launch = [&](auto go) {
    go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.q), lo32(A.k_new), lo32(A.v_new), hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.q), hi16s(A.k_new, A.v_new),
       flags, (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, A.stride24, (uint32_t)(A.head_stride_b / 16), A.scale_log2, T);
  };
  if (ev_start && ev_stop)
    launch([&](auto... args) { hipExtLaunchKernelGGL((k_attend<EB, D, 1, U, NW, false, true, false, 0, S>), grid, block, (uint32_t)lds, st, ev_start, ev_stop, 0, args...); });
  else
    launch([&](auto... args) { hipLaunchKernelGGL((k_attend<EB, D, 1, U, NW, false, true, false, 0, S>), grid, block, lds, st, args...); });
  return hipGetLastError();
}

template <int EB, int D, bool VF, bool WIDE>
hipError_t launch_attend_v(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  if constexpr (!VF && kBurst > D * EB) {
    if (plan.heads > 1) return launch_attend_w<EB, D, kBurst / (D * EB), 4, VF, true, WIDE>(A, plan, n_seq, st, ev_start, ev_stop);
  }
  if (plan.n_chunks > 1) return launch_attend_w<EB, D, 1, 8, VF, false, WIDE>(A, plan, n_seq, st, ev_start, ev_stop);
  if (plan.waves == 8) return launch_attend_w<EB, D, 1, 8, VF, true, WIDE>(A, plan, n_seq, st, ev_start, ev_stop);
  return launch_attend_w<EB, D, 1, 4, VF, true, WIDE>(A, plan, n_seq, st, ev_start, ev_stop);
}

template <int EB, int D>
hipError_t launch_attend_t(const AttendArgs& A, const AttendPlan& plan, int n_seq, hipStream_t st,
                           hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (A.vcos_fused) return plan.wide ? launch_attend_v<EB, D, true, true>(A, plan, n_seq, st, ev_start, ev_stop) : launch_attend_v<EB, D, true, false>(A, plan, n_seq, st, ev_start, ev_stop);
  return plan.wide ? launch_attend_v<EB, D, false, true>(A, plan, n_seq, st, ev_start, ev_stop) : launch_attend_v<EB, D, false, false>(A, plan, n_seq, st, ev_start, ev_stop);
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

// Whether a lane reaches every row of its workgroup's heads with a 24-bit product and a 32-bit offset: rows up to 16 MB apart
// whose cache spans less than 4 GB less the offsets that stand for no row (all dense caches: at most 8192 slots of 128 KB).  Others -- a slot that holds every sequence
// and layer of a model, say -- take the form with 64-bit offsets, 4 to 8 registers more, by the same launch rule: one form of it with 8
// waves and one head for all of them took 64 sequences x 24 x 64, rows 18 MB apart, 700 tokens from 56 us to 68, 60 tokens from 9.6 to 14.2.
static bool short_offsets(const adsa_params& p, int heads) {
  const long long eb = elem_bytes(p), slot_b = p.kv_slot_stride * eb;
  return slot_b < (1ll << 24) && (p.cap - 1) * slot_b + (heads - 1) * p.kv_head_stride * eb + p.head_dim * eb <= (long long)kRowBufferBytes;
}

// K and V bytes of the longest list that 4 waves read as fast as 8: see make_attend_plan.
static long long short_list(const adsa_params& p) { return (p.score_mode == ADSA_SCORE_VCOS_FUSED ? 32ll : 72ll) << 10; }

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
    a.wide = false;
    a.chunk_max = gqa_logit_stride(p, nc);
    return a;
  }
  // One workgroup per (sequence, head): 8 waves up to one pair per CU, 4 from two on; in between 8 where the lists together
  // are long (80 MB), for the waves that then wait side by side, and 4 where starting the workgroups is a good part of
  // the launch.  Measured, us with 4 | 8 waves, bf16: 320 pairs x 427 tokens x 64 (35 MB) 9.0 | 9.2; 260 x 698 x 64 12.0 | 12.6;
  // 400 x 698 x 64 (71 MB) 13.7 | 14.0; 480 x 746 x 64 (92 MB) 16.8 | 16.5; 288 x 1394 x 64 (103 MB) 23.3 | 22.7; 400 x 746 x 128
  // (153 MB) 25.6 | 25.4; 768 x 228 x 64 9.9 | 10.7; 768 x 647 x 64 21.3 | 21.5; 256 x 698 x 128 16.0 | 16.1; 192 x 698 x 64 8.0 | 7.8;
  // 40 x 400 x 64 6.3 | 5.9 and 128 x 4000 x 128 60 | 53 (with an earlier loop; 16 waves 7.2 and 52); fp32: 288 x 323 x 128 20.5 |
  // 20.7; 400 x 323 x 128 22.8 | 22.3.  Lists that the rings of 4 waves hold twice over (72 KB) are read in one more revolution than with
  // 8, which costs less than the start and the merge of 4 more waves: 16 pairs x 130 tokens x 64 3.3 | 3.5, 200 3.7 | 3.9, 240 3.85 |
  // 3.94, 300 (82 KB) 4.24 | 4.20; 64 x 200 x 64 3.9 | 4.0; 240 x 130 x 64 4.2 | 4.2, 240 5.0 | 5.3, 300 5.6 | 5.6; 128 x 110 x 128 4.2 |
  // 4.3, 140 (82 KB) 4.5 | 4.5; 30 x 80 x 128 fp32 4.1 | 4.2; 96 x 200 x 64 [slot][head][D] 4.1 | 4.2.  (The line of the fused V-cosine
  // form is the 32 KB of one revolution.)
  const long long pairs = (long long)p.n_seq * p.n_heads;
  const long long b_list = (long long)p.sel_cap * 2 * p.head_dim * elem_bytes(p);
  a.waves = pairs >= 512 || b_list <= short_list(p) || (pairs > 256 && pairs * b_list < (80ll << 20)) ? 4 : 8;
  // Splitting a list costs a second launch, ~2.5 us, and is worth it where one workgroup's bytes are what the launch lasts: from about
  // 330 KB on, a little more where more pairs share the memory's rate.  Into 8-wave chunks of 64 KB, what their rings hold at once (so
  // that none ends in a second, nearly empty revolution), or as many as leave no CU with two, which then lasts as long as those: 24
  // pairs x 804 KB in 10 chunks 10.6, in 11 11.8; 40 x 504 KB in 6 10.1, in 7 11.5; 92 x 704 KB in 2 17.0, in 3 20.7; [slot][head][D]
  // 40 x 745 KB x 128 in 6 11.2, in 7 13.2.  Measured, us whole | split, bf16 x 64: 1 pair x 300 KB 6.0 | 7.1, 350 KB 6.6 | 7.3
  // (slot-major 7.6 | 7.3), 400 KB 8.4 | 7.3; 2 pairs x 300 KB 7.7 | 7.5, 350 KB 8.6 | 7.7; 4 x 260 KB 6.2 | 7.6, 404 KB 9.1 | 7.8; 8 x
  // 325 KB 7.9 | 8.0, 357 KB 8.6 | 8.1; 24 x 325 KB 8.8 | 8.6, 404 KB 10.5 | 8.9; 48 x 325 KB 9.2 | 9.5, 404 KB 11.0 | 10.0; 64 x 325
  // KB 9.4 | 10.0, 404 KB 11.3 | 10.5, 704 KB 18.4 | 13.6; 80 x 504 KB 14.1 | 12.8, 1 MB 25.7 | 19.7; 92 x 704 KB 19.8 | 17.0; fp32 x
  // 128 1 x 350 KB 7.5 | 6.7, 8 x 341 KB 7.9 | 7.5.  All of these lists are full; host code knows only what they can hold.  With half
  // of it, 48 pairs x 500 KB 7.9 | 9.2, 750 KB 10.7 | 10.0; 80 x 500 KB 8.4 | 9.8, 1 MB 14.5 | 13.6.  (One launch whose last workgroup
  // to arrive merges, behind a device-scope release / acquire, took 12 us for 8 x 512 KB.) Rows of the fused V-cosine form take longer,
  // so their line is lower: 2 x 207 KB 7.1 | 7.5, 263 KB 7.8 | 7.6; 8 x 207 KB 7.2 | 7.7, 263 KB 8.1 | 7.9; 32 x 263 KB 8.7 | 8.5; 64 x
  // 327 KB 10.5 | 9.7; 92 x 507 KB 15.2 | 13.6.
  const bool fused = p.score_mode == ADSA_SCORE_VCOS_FUSED;
  const long long line = (fused ? 240 + pairs / 2 : 330 + pairs) << 10, snug = (b_list + (64 << 10) - 1) / (64 << 10);
  long long nc = 1;
  if (pairs < 96 && b_list > line) nc = std::min<long long>({snug, 256 / pairs, kMaxChunks});
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
  a.wide = !short_offsets(p, a.heads);
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

static AttendArgs attend_args(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q, const void* k_new, const void* v_new,
                              const int32_t* sel_idx, const int32_t* sel_cnt, void* out, float* lse, char* ws, const Workspace& w,
                              bool accumulate, bool append, int advance, bool new_f32) {
  AttendArgs A;
  A.seqs = seqs; A.q = (const char*)q; A.k_new = (const char*)k_new; A.v_new = (const char*)v_new;
  A.sel_idx = sel_idx; A.sel_cnt = sel_cnt; A.out = (char*)out; A.lse = lse;
  A.logits = reinterpret_cast<float*>(ws + w.logits_off);
  A.part_ml = reinterpret_cast<float*>(ws + w.part_ml_off);
  A.part_acc = reinterpret_cast<float*>(ws + w.part_acc_off);
  A.n_heads = p.n_heads; A.sel_cap = p.sel_cap; A.lg_stride = w.lg_stride;
  A.cap = p.cap;
  A.accumulate = accumulate ? 1 : 0; A.append = append ? 1 : 0; A.advance = advance;
  A.new_f32 = (new_f32 && append) ? 1 : 0;
  A.vcos_fused = p.score_mode == ADSA_SCORE_VCOS_FUSED ? 1 : 0;
  const int eb = elem_bytes(p);
  A.slot_stride_b = (long long)p.kv_slot_stride * eb;
  A.head_stride_b = (long long)p.kv_head_stride * eb;
  A.stride24 = plan.wide ? 0u : (uint32_t)A.slot_stride_b;
  const float scale = p.softmax_scale != 0.0f ? p.softmax_scale : 1.0f / sqrtf((float)p.head_dim);
  A.scale_log2 = scale * kLog2e;
  return A;
}

hipError_t launch_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q,
                         const void* k_new, const void* v_new, const int32_t* sel_idx, const int32_t* sel_cnt,
                         void* out, float* lse, char* ws, const Workspace& w, bool accumulate, bool append,
                         int advance, bool new_f32, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (p.q_per_kv > 1)
    return launch_attend_gqa(p, plan, seqs, q, k_new, v_new, sel_idx, sel_cnt, out, lse, ws, w, accumulate, append,
                             advance, new_f32, st, ev_start, ev_stop);
  const AttendArgs A = attend_args(p, plan, seqs, q, k_new, v_new, sel_idx, sel_cnt, out, lse, ws, w, accumulate, append, advance, new_f32);
  const int eb = elem_bytes(p);
  const int key = eb * 1000 + p.head_dim;
  if (key == 2064) return launch_attend_t<2, 64>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 2128) return launch_attend_t<2, 128>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 4064) return launch_attend_t<4, 64>(A, plan, p.n_seq, st, ev_start, ev_stop);
  if (key == 4128) return launch_attend_t<4, 128>(A, plan, p.n_seq, st, ev_start, ev_stop);
  return hipErrorInvalidValue;
}

// Whether adsa_step's ranking, attention and eviction are two launches (k_attend with RANK, k_step_finish) instead of three.  The
// ranking is repeated by every head's workgroup, so it is for steps whose launches are chains of latencies anyway: those whose workspace
// has room for the scores that the second kernel puts in place, which is what lists of fewer than 96 head groups may be split into.
// adsa_step, us with three launches | with two (GPU time; a launch less is 2.4 us of the host's beside it), inside a row and where all
// sequences close one: 1 sequence x 16 heads x 64 fp32, 124 tokens 10.2 | 8.2, 16.0 | 13.5; 7 x 9 x 128 [slot][head][D], 401 tokens 13.5 |
// 12.2, 17.2 | 15.6; 3 x 24 x 64, 536 tokens 13.7 | 12.4, 28.6 | 23.3; 4 x 20 x 64 in 1000 slots 14.8 | 13.6, 32.4 | 28.8; 95 x 1 x 64
// 12.8 | 11.3, 24.6 | 20.4; 20 x 16 x 64 [slot][head][D] (320 pairs, 40 groups) 19.3 | 18.5, 38.7 | 34.2.
// Many heads of one sequence, all of whose workgroups read all score rows, change nothing: 1 x 48 heads x 64, 525 of 1000 slots 15.4 | 14.1, 35.8
// | 29.4; 1 x 95 19.3 | 18.0, 51.8 | 39.3; 1 x 256 [slot][head][D] 34.6 | 33.5, 113 | 80, 336 of 500 slots 31.0 | 22.0.
bool rank_in_attend(const adsa_params& p, const AttendPlan& plan, const Workspace& w) {
  return one_launch_compact(p) && p.score_mode == ADSA_SCORE_ATTN_MASS && p.q_per_kv <= 1 && plan.n_chunks == 1 && plan.heads == 1 && !plan.wide &&
         p.cap <= 1024 && sizeof(float) * p.n_seq * p.n_heads * p.cap <= w.plan_off - w.logits_off;
}

hipError_t launch_ranked_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q, const void* k_new, const void* v_new,
                                int32_t* sel_idx, int32_t* sel_cnt, void* out, float* lse, char* ws, const Workspace& w, bool new_f32,
                                hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const AttendArgs A = attend_args(p, plan, seqs, q, k_new, v_new, sel_idx, sel_cnt, out, lse, ws, w, true, true, kAdvanceNone, new_f32);
  const RankTail T = {A.out, A.lse, A.logits, reinterpret_cast<int32_t*>(ws + w.plan_off), p.grid_h * p.grid_w, p.grid_w, p.win_rows_back,
                      p.win_col_radius, p.win_recent_m, 1.0f / (float)p.grid_w, {}};
  auto go = [&](auto waves, auto slots) {
    constexpr int NW = decltype(waves)::value, S = decltype(slots)::value;
    switch (elem_bytes(p) * 1000 + p.head_dim) {
      case 2064: return launch_ranked<2, 64, NW, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 2128: return launch_ranked<2, 128, NW, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 4064: return launch_ranked<4, 64, NW, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 4128: return launch_ranked<4, 128, NW, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      default: return hipErrorInvalidValue;
    }
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 2> two;
  const std::integral_constant<int, 4> four;
  const std::integral_constant<int, 8> eight;
  // 4 waves up to 256 slots, one a thread, however long a row is: adsa_step with 8 waves | 4, 16 pairs x 124 tokens x 64 fp32 8.7 | 8.2 us, 40 x
  // 241 x 128 bf16 9.9 | 9.6, 84 x 242 x 128 fp32 12.5 | 12.2; with two slots a thread, 40 x 237 x 64 in 500 slots, 9.8 | 10.1.
  if (p.cap <= 256) return go(four, one);
  return p.cap <= 512 ? go(eight, one) : go(eight, two);
}

// Whether adsa_step's attention launch plans the evictions too, which leaves select, attention and move: steps that are too large for
// one_launch_compact, with 4 waves a list and up to three slots a thread (more rank in larger workgroups).  adsa_step, us with four
// launches | with three: 64 sequences x 24 heads x 600 slots, no row end 41.6 | 39.9, 2 at one 47.9 | 44.0; 128 x 8 x 250 20.9 | 19.0, 5 at one
// 25.9 | 23.5; 200 x 8 x 700 43.5 | 41.7, 8 at one 55.2 | 49.4; 160 x 24 x 600 86.9 | 85.3, 6 at one 104 | 98.
// Where all sequences close a row at once it takes longer from some 1500 pairs on: a sequence's last workgroup to end plans, that is one of the
// XCD that is behind, which falls further behind for it and draws the next sequence's last ticket too (293 of 381 plans, 883 of 1000).  Up
// to 4096 pairs that is 3 % of one step of a row's, most of which gain: 64 x 24 x 600 95 | 98, 128 x 24 x 600 168 | 173, 500 x 8 x 250 102 | 106,
// 250 x 16 x 400 x 128 299 | 298.  Beyond them it is up to 20 %, for 1 to 2 % inside a row: 200 x 48 x 300 240 | 261 and 111 | 109, 400 x 48 x 300
// 460 | 517 and 210 | 208, 1000 x 24 x 130 276 | 336 and 135 | 132, 1000 x 16 x 300 419 | 466 and 192 | 192.
bool plan_in_attend(const adsa_params& p, const AttendPlan& plan) {
  return p.evict_policy == ADSA_EVICT_ROW_END && p.score_mode == ADSA_SCORE_ATTN_MASS && p.q_per_kv <= 1 && !one_launch_compact(p) && plan.n_chunks == 1 &&
         plan.heads == 1 && plan.waves == 4 && !plan.wide && p.cap <= 768 && (long long)p.n_seq * p.n_heads <= 4096;
}

hipError_t launch_planned_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q, const void* k_new, const void* v_new,
                                 int32_t* sel_idx, int32_t* sel_cnt, void* out, float* lse, int32_t* keep_map, char* ws, const Workspace& w, bool new_f32,
                                 hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const AttendArgs A = attend_args(p, plan, seqs, q, k_new, v_new, sel_idx, sel_cnt, out, lse, ws, w, true, true, kAdvanceNone, new_f32);
  const PlanTail T = {A.out, A.lse, reinterpret_cast<int32_t*>(ws + w.plan_off), keep_map, p.grid_w, p.win_rows_back, p.grid_h * p.grid_w, kAdvanceNone,
                      1.0f / (float)p.grid_w, p.win_recent_m, {}};
  auto go = [&](auto slots) {
    constexpr int S = decltype(slots)::value;
    switch (elem_bytes(p) * 1000 + p.head_dim) {
      case 2064: return launch_planned<2, 64, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 2128: return launch_planned<2, 128, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 4064: return launch_planned<4, 64, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      case 4128: return launch_planned<4, 128, S>(A, T, plan, p.n_seq, st, ev_start, ev_stop);
      default: return hipErrorInvalidValue;
    }
  };
  return p.cap <= 256 ? go(std::integral_constant<int, 1>()) : p.cap <= 512 ? go(std::integral_constant<int, 2>()) : go(std::integral_constant<int, 3>());
}

}  // namespace adsa
