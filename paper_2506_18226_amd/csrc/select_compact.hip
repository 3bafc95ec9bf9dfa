// Partition + ranking kernels of the ADSA decode path (gfx950).
//
//  k_select        : Eq. 1 partition of the resident slots, Eq. 4 ranking of the candidates as a
//                    threshold found by narrowing histograms, lowest-slot tie-break, and the
//                    ascending attended-slot list.  It can plan for the query token's append
//                    (Section 4.2: new tokens go to the end of the cache) that the attention
//                    launch performs, so the ranking never waits for the token's K/V.
//  k_compact_plan  : Section 4.2 in per-row form: keep flags (prefix, last R rows, top-B of the
//                    rest), ballot/prefix-sum keep map, in-place move of pos[] and, where they are few, the score rows; or
//                    Section 4.2 as written (evict the one most redundant candidate when full), closing
//                    the hole in order or leaving it to the incoming token.  (Larger adsa_step batches: k_attend with PLAN does it.)
//  k_compact_move  : in-place, order-preserving move of the surviving K and V rows, and of the score rows where kMovedWithCache says so or
//                    the attention launch has planned, whose records it advances.
//  k_compact_step  : the per-row plan and move of a small decode step in one launch.
//  k_step_finish   : the same after an attention launch that ranked for itself, with the scores, the record and the query token's
//                    position, which that launch left alone.
//
// One workgroup owns one sequence in the first two kernels.  Its slots live in registers, S per thread (slot = u * NT +
// thread), from the one read of the score array to the last write: what crosses threads is a histogram, at most 64
// keys and one pair of counts per wave.  Both kernels are chains of dependent latencies (record -> scores -> a handful
// of barriers -> stores) rather than work, so the number of barriers and of memory round trips is what they are built around.
#include <type_traits>

#include "adsa_rank.h"

namespace adsa {
namespace {

// (512 x 8 and 512 x 16 need 130 registers, two more than let a second workgroup share the CU: held to four waves per SIMD.  One slot
// per thread and 24 rows in flight need 104 if the addresses of all rows are kept; held to seven waves per SIMD it is 66: 1112 sequences x 26
// rows x 231 slots 8.4 us instead of 9.3, 1348 x 8 x 185 7.2 instead of 8.1.  k_compact_plan likewise, 72 instead of 94: 1759 x 1 x 240 6.0 instead of 7.4.
// 256 x 3 for many sequences: 78 instead of 82, six waves instead of five, with which 1536 sequences are resident at once: x 8 rows 11.5 -> 10.3 us.)
template <int NT, int S, int RB = rank_batch(S)>
__global__ __launch_bounds__(NT, S >= 8 ? 4 : S == 1 ? 7 : S == 3 && RB == 8 ? 6 : 1) void k_select(
    uint32_t seqs_lo, uint32_t idx_lo, uint32_t cnt_lo, uint32_t tickets_lo, uint32_t seqs_idx_hi, uint32_t cnt_tickets_hi, uint32_t caps,
    uint32_t flags, int total, int W, int R, int w, int recent_m, float inv_w) {
  __shared__ __align__(16) RankShared sh;
  const int b = blockIdx.x, tid = threadIdx.x;
  gseq& sq = ((gseq*)address(seqs_lo, seqs_idx_hi & 0xFFFF))[b];
  gint* const sel_cnt = (gint*)address(cnt_lo, cnt_tickets_hi & 0xFFFF);
  const RankFlags F(flags);                                  // a: plan the append; b: there are tickets
  const bool plan_append = F.a;
  const int cap = caps & 0xFFFF, sel_cap = caps >> 16;
  const gint* const pos = (const gint*)sq.pos;
  gfloat* const score = (gfloat*)sq.score;
  const int s = sq.step;
  int n = sq.n_res;
  const int status_in = sq.status;
  const BudgetOf budget(sq);                                 // (loaded with the rest of the record, whether it is needed or not)
  rank_clear<NT>(sh);                                        // (while the record is on its way)
  if (F.b && tid < 4) ((gint*)address(tickets_lo, cnt_tickets_hi >> 16))[4 * b + tid] = 0;       // for this step's eviction
  if (s < 0 || status_in != 0) { if (tid == 0) { sel_cnt[b] = 0; sq.pending_slot = -1; } return; }
  if (n < 0 || n > cap || s > total) {
    if (tid == 0) { sq.status = status_in | ADSA_SEQ_BAD_STATE; sel_cnt[b] = 0; sq.pending_slot = -1; }
    return;
  }
  // Section 4.2: the query token goes to the end of the cache (or, with ADSA_EVICT_REUSE_SLOT, into
  // the slot the last eviction freed).  When the append itself happens later in this step (inside
  // the attention launch), plan for it: that slot, always local, score 0.
  const int hole = F.policy == ADSA_EVICT_REUSE_SLOT ? sq.hole - 1 : -1;     // freed slot or -1
  int slot_new = -1;
  if (plan_append && s >= 1) {
    if (hole >= 0 && hole < n) slot_new = hole;
    else {
      if (n + 1 > cap) {
        if (tid == 0) { sq.status = status_in | ADSA_SEQ_CACHE_FULL; sel_cnt[b] = 0; sq.pending_slot = -1; }
        return;
      }
      slot_new = n;
      n += 1;
    }
  }

  // ---- Eq. 1: partition, keys into registers
  const QueryCell cell = make_query_cell(sq, s, GridWidth{W, inv_w}, R, w, recent_m);
  // The streaming policies attend everything resident (context == cache, Tables 1-2).  Otherwise the B best candidates are attended:
  // their ranks need not be read where B covers every position that can be one (positions are distinct), as in the first B steps of
  // an image and for a budget of the whole context: 8 sequences x 16 rows x 8000 slots 8.5 us without the 4 MB of scores, 13.7 with.
  const bool streaming = F.policy != ADSA_EVICT_ROW_END;
  const uint32_t B_row = streaming ? 0u : (uint32_t)effective_budget(budget, s);
  bool ranked = !streaming && (int)B_row < min(n, cell.P + cell.jq - cell.n_keep_prefix);
  int idx[S], posv[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = min(u * NT + tid, n - 1);
    posv[u] = n > 0 ? elem(pos, idx[u]) : 0;                 // (an empty sequence's pointers may be null)
  }
  const bool largest = keep_largest_of(F.mode);
  uint32_t key[S], candm = 0, fixedm = 0, B;
  bool bad = false;
  Stats st;
  auto classify = [&] {
    float rank[S];
#pragma unroll
    for (int u = 0; u < S; ++u) rank[u] = 0.0f;
    if (n > 0 && ranked) rank_values<S, RB>(score, F.rows, cap, idx, rank);
    candm = fixedm = 0;
    int cls[S];
    if (recent_m > 0) {                                      // (uniform; issue slots count where many sequences stream: 1536 x 632 slots 6.2 -> 5.9 us)
#pragma unroll
      for (int u = 0; u < S; ++u) cls[u] = select_class_1d(cell, posv[u]);
    } else {
#pragma unroll
      for (int u = 0; u < S; ++u) cls[u] = select_class(cell, posv[u]);
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const int i = u * NT + tid;
      const bool in = i < n, planned = i == slot_new;        // the slot the query token will occupy
      const bool freed = i == hole && !planned;              // evicted, not yet reused: nobody attends it
      const int c = (planned || freed) ? 0 : cls[u];
      key[u] = order_key(rank[u], largest);
      bad |= in && c < 0;
      if (in && c == 1) candm |= 1u << u;
      if (in && c != 1 && !freed) fixedm |= 1u << u;
    }
    st = block_stats<NT, S>(sh, key, candm, bad);
    B = streaming ? st.n_cand : B_row;
  };
  classify();
  if (!ranked && B < st.n_cand) {                            // (uniform) positions were not distinct after all
    ranked = true;
    __syncthreads();
    classify();
  }
  if (st.bad) {
    if (tid == 0) { sq.status = status_in | ADSA_SEQ_BAD_STATE; sel_cnt[b] = 0; sq.pending_slot = -1; }
    return;
  }

  // ---- Eq. 4: threshold of the top-B candidates
  uint32_t T, need_eq;
  top_threshold<NT, S>(sh, key, candm, st, B < st.n_cand ? B : st.n_cand, &T, &need_eq);

  // ---- ascending slot list
  uint32_t sure = fixedm, eq = 0, dest[S], cnt;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (((candm >> u) & 1u) && key[u] > T) sure |= 1u << u;
    if (((candm >> u) & 1u) && key[u] == T) eq |= 1u << u;
  }
  const uint32_t take = place_kept<NT, S>(sh, sure, eq, need_eq, dest, &cnt);
  gint* const out = (gint*)address(idx_lo, seqs_idx_hi >> 16) + (size_t)b * sel_cap;
#pragma unroll
  for (int u = 0; u < S; ++u)
    if (((take >> u) & 1u) && dest[u] < (uint32_t)sel_cap) elem(out, dest[u]) = u * NT + tid;
  const bool ok = cnt <= (uint32_t)sel_cap;
  const bool reserve = ok && slot_new >= 0;          // commit the planned append: the slot now holds the query token
  if (reserve)
    for (int r = tid; r < F.rows; r += NT) score[(size_t)r * cap + slot_new] = 0.0f;
  if (tid == 0) {
    if (!ok) { sq.status = status_in | ADSA_SEQ_SEL_OVERFLOW; sel_cnt[b] = 0; sq.pending_slot = -1; }
    else {
      sel_cnt[b] = (int32_t)cnt;
      sq.pending_slot = reserve ? slot_new : -1;
      if (reserve) {
        sq.pos[slot_new] = sq.grid_origin + s - 1;
        sq.n_res = n;
        if (slot_new == hole) sq.hole = 0;
      }
    }
  }
}

// In-place, order-preserving move of pos[] and every score row: all sources of a batch of rows have arrived in registers
// before the barrier, all destinations are written after it.  (pos has been in registers since the classification.)
// Rows per batch: as many as leave the kernels around it their residency.  k_compact_plan with 2 slots per thread, us with 8 | 12 |
// 16 | 24 rows (74 | 94 | 122 | 160 registers): 900 slots, 66 sequences x 24 rows 10.1 | 10.2 | 10.4 | 10.0, 514 x 24
// 20.8 | 23.4 | 25.3 | 30.1, 516 x 8 12.1 | 14.4 | 15.5 | 23.2, 1538 x 24 53 | 54 | 56 | 66.  (That was with every row in the plan; where
// kMovedWithCache leaves it up to 11, it asks for other batches.)
template <int NT, int S, int kRowBatch = S == 2 ? 8 : S <= 3 ? 24 : S == 4 ? 8 : 4>
__device__ __forceinline__ void move_scores(gfloat* score, gint* pos, int rows, int cap, uint32_t moves, const uint32_t (&dest)[S],
                                            const int (&posv)[S]) {
  const int tid = threadIdx.x;
  for (int r0 = 0; r0 < rows; r0 += kRowBatch) {
    float sv[S][kRowBatch];
#pragma unroll
    for (int u = 0; u < S; ++u)
      if ((moves >> u) & 1u) {
#pragma unroll
        for (int k = 0; k < kRowBatch; ++k) sv[u][k] = score[(size_t)min(r0 + k, rows - 1) * cap + u * NT + tid];
      }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (int u = 0; u < S; ++u)
      if ((moves >> u) & 1u) {
        if (r0 == 0) pos[dest[u]] = posv[u];
#pragma unroll
        for (int k = 0; k < kRowBatch; ++k)
          if (r0 + k < rows) score[(size_t)(r0 + k) * cap + dest[u]] = sv[u][k];
      }
  }
}

// From 12 score rows on, in caches of more than 128 slots, k_compact_move's workgroups move them, one a head's, and k_compact_plan, one workgroup
// a sequence, is over a round trip or more sooner.  An eviction (us, plan | move): 5 sequences x 46 heads x 1100 slots 31.2 | 24.6, 2 x 59 x 5500
// 38.7 | 34.7, 3 x 30 x 340 18.6 | 16.6, 52 x 28 x 600 57.1 | 53.3, 20 shapes by 1.05; a step of 64 x 24 x 600 with 2 sequences at a row end
// 54.0 | 52.6.  Fewer rows and shorter lists cost the plan less than those workgroups: one row, 4 x 9 x 6600 37.2 | 39.1, 443 x 1 x 377 fp32
// 23.9 | 24.7; 6 rows, 81 x 6 x 253 17.8 | 18.5; 8, a step of 200 x 8 x 250 34.2 | 34.5; 60 slots, 83 x 43 fp32 37.0 | 39.2, 406 x 12 30.2 | 31.4.
// With more than 128 sequences the plan launch is no chain that the chip idles through any more, and finds the rows it has just ranked in its L2:
// there it keeps fewer than 24 rows, and all of them in caches of 257 to 384 slots, which the move takes in a tile of 512.  All sequences at a
// row end, as the layers of one model are, plan | move: 400 sequences x 16 x 300 102 | 106, 1000 x 16 x 300 239 | 253, 800 x 12 x 300 147 | 153; by (plan /
// move) 400 x 24 x 300 0.98, 700 x 12 x 480 0.98, 700 x 20 x 450 0.98, but 128 x 16 x 300 1.01, 400 x 24 x 512 1.04, 400 x 32 x 600 1.02, 160 x 24 x 700 1.03,
// 512 x 24 x 696 1.01.  (One in 20 at a row end: the move is ahead everywhere, by 1.02 to 1.2.)
constexpr int kMovedWithCache = 12, kPlanRowsCap = 128, kPlanRowsSeqs = 128, kManyRows = 24;

// plan[b] = { old n_res, first slot that moves, did compact, new n_res }
template <int NT, int S, int RB = rank_batch(S)>
__global__ __launch_bounds__(NT, S == 1 ? 7 : 1) void k_compact_plan(
    uint32_t seqs_lo, uint32_t map_lo, uint32_t plan_lo, uint32_t vs_lo, uint32_t seqs_map_hi, uint32_t plan_vs_hi, uint32_t cap_arg, uint32_t flags,
    int total, int W, int R, int recent_m, float inv_w, int dim) {
  __shared__ __align__(16) RankShared sh;
  constexpr int NW = NT / kWave;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), cap = (int)cap_arg;
  gseq& sq = ((gseq*)address(seqs_lo, seqs_map_hi & 0xFFFF))[b];
  gint* const plan = (gint*)address(plan_lo, plan_vs_hi & 0xFFFF);
  const RankFlags F(flags);                                  // a: advance the step; b: the move takes the score rows along
  const bool advance_step = F.a;
  gint* const pos = (gint*)sq.pos;
  gfloat* const score = (gfloat*)sq.score;
  const int s = sq.step, n = sq.n_res;
  const bool active = s >= 0 && sq.status == 0;
  const QueryCell cell = make_query_cell(sq, s, GridWidth{W, inv_w}, R, 0, recent_m);      // (streaming: a 1-D window, which has no radius)
  // per-row policy: act when the query token closed a grid row; streaming policy (Section 4.2 as
  // written): act when the cache is full and a token is about to be inserted
  const bool streaming = F.policy != ADSA_EVICT_ROW_END;
  const bool reuse = F.policy == ADSA_EVICT_REUSE_SLOT;
  const bool row_end = active && n >= 0 && n <= cap &&
                       (streaming ? (s >= 1 && s <= total && n == cap && !(reuse && sq.hole != 0))
                                  : is_row_end(cell, s, total));
  if (!row_end) {
    if (tid == 0) {
      plan[4 * b + 0] = 0; plan[4 * b + 1] = 0; plan[4 * b + 2] = 0; plan[4 * b + 3] = n;
      if (active) { sq.compacted = 0; if (advance_step) sq.step = s + 1; }
    }
    return;
  }
  const bool largest = keep_largest_of(F.mode), fused = F.mode == ADSA_SCORE_VCOS_FUSED;
  int idx[S], posv[S];
  float rank[S], dot[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = min(u * NT + tid, n - 1);
    posv[u] = n > 0 ? elem(pos, idx[u]) : 0;                       // (an empty sequence's pointers may be null)
    rank[u] = dot[u] = 0.0f;
  }
  rank_clear<NT>(sh);
  // Fused form: Eq. 3 from what the last attention launch left per (head, slot): S_i = (v^_i.u - v^_i.v^_i)/(N-1) with
  // |v_i|^2 and v_i.u summed over the heads' rows (ascending).  If those rows do not belong to this
  // step, the two-pass computation has just written S_i to the workspace instead.
  bool rows_ok = false;
  if (fused && n > 0) {
    const gfloat* tags = sq.vcos_u ? (const gfloat*)sq.vcos_u + dim : nullptr;
    rows_ok = tags && tags[1] == (float)(s + 1);
    if (rows_ok) rank_pairs<S>(score, F.rows / 2, cap, idx, rank, dot);
    else {
#pragma unroll
      for (int u = 0; u < S; ++u) rank[u] = elem((const gfloat*)address(vs_lo, plan_vs_hi >> 16) + (size_t)b * cap, idx[u]);
    }
  } else if (n > 0) {
    rank_values<S, RB>(score, F.rows, cap, idx, rank);
  }
  uint32_t key[S], restm = 0, in = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    // streaming: the partition of the incoming query (its local region must survive)
    const int c = streaming ? (select_class(cell, posv[u]) == 1 ? 1 : 0) : evict_class(cell, posv[u]);
    if (u * NT + tid < n) in |= 1u << u;
    if (((in >> u) & 1u) && c == 1) restm |= 1u << u;
    key[u] = fused ? 0u : order_key(rank[u], largest);
  }
  Stats st = block_stats<NT, S>(sh, key, restm, false);
  if (fused) {                                               // the keys need N, the number of candidates
    const float inv_nm1 = st.n_cand > 1 ? 1.0f / (float)(st.n_cand - 1) : 0.0f;
#pragma unroll
    for (int u = 0; u < S; ++u) {
      const float ss = rank[u], inv = 1.0f / fmaxf(sqrtf(ss), 1e-8f);
      key[u] = order_key(rows_ok ? (dot[u] * inv - ss * inv * inv) * inv_nm1 : rank[u], false);
    }
    st = block_stats<NT, S, 1>(sh, key, restm, false);
  }
  gint* const map = (gint*)address(map_lo, seqs_map_hi >> 16) + (size_t)b * cap;
  if (reuse) {
    // Evict the candidate ranked last -- smallest key, among equals the newest position -- and leave
    // everything where it is: the freed slot goes to the incoming token.
    uint32_t newest = 0;
#pragma unroll
    for (int u = 0; u < S; ++u)
      if (((restm >> u) & 1u) && key[u] == st.kmin) newest = max(newest, (uint32_t)posv[u] + 1u);
    newest = wave_max(newest);
    if (lane == 0) sh.newest[wave_id()] = newest;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) newest = max(newest, sh.newest[w]);
    if (st.n_cand > 0) {
#pragma unroll
      for (int u = 0; u < S; ++u) {
        const int i = u * NT + tid;
        const bool victim = ((restm >> u) & 1u) && key[u] == st.kmin && (uint32_t)posv[u] + 1u == newest;
        if (i < n) map[i] = victim ? -1 : i;
        if (victim) sq.hole = i + 1;
      }
    }
    if (tid == 0) {
      plan[4 * b + 0] = n; plan[4 * b + 1] = n; plan[4 * b + 2] = 0; plan[4 * b + 3] = n;
      sq.compacted = st.n_cand > 0 ? 1 : 0;
      if (advance_step) sq.step = s + 1;
    }
    return;
  }
  uint32_t B = (uint32_t)effective_budget(sq, s);
  if (streaming) B = st.n_cand > 0 ? st.n_cand - 1 : 0;      // all candidates but the one ranked last
  uint32_t T, need_eq;
  top_threshold<NT, S>(sh, key, restm, st, B < st.n_cand ? B : st.n_cand, &T, &need_eq);
  uint32_t sure = in & ~restm, eq = 0, dest[S], n_new;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (((restm >> u) & 1u) && key[u] > T) sure |= 1u << u;
    if (((restm >> u) & 1u) && key[u] == T) eq |= 1u << u;
  }
  const uint32_t take = place_kept<NT, S>(sh, sure, eq, need_eq, dest, &n_new);
  // first slot whose content changes: the first one that is dropped.  Everything before it stays put.  (Positions have been in registers
  // since before the ranking's barriers.)
  uint32_t moves = 0;
#pragma unroll
  for (int u = S - 1; u >= 0; --u) {
    const int i = u * NT + tid;
    const bool kept = (take >> u) & 1u;
    if ((in >> u) & 1u) map[i] = kept ? (int32_t)dest[u] : -1;
    if (kept && dest[u] != (uint32_t)i) moves |= 1u << u;
    const unsigned long long gone = __ballot(((in >> u) & 1u) && !kept);
    if (gone != 0 && lane == 0) atomicMin(&sh.first, (uint32_t)(u * NT + wave_id() * kWave + __ffsll((long long)gone) - 1));
  }
  // (Batches: for fewer than 12 rows 11 at once where they cost no workgroup its place on the CU, 8 and 4 where they would; for more 24 where
  // they do not.  With 11 for 2 slots per thread, 90 registers instead of 68, the plan of 516 sequences x 1 row x 900 slots and its move took
  // 43.4 us instead of 40.1, 1500 x 1 x 400 10.9 instead of 9.5.)
  constexpr int kFew = S == 1 || S == 3 ? kMovedWithCache - 1 : S <= 4 ? 8 : 4, kMany = S == 1 || S == 3 ? 24 : kFew;
  if (!F.b && (kFew == kMany || F.rows < kMovedWithCache)) move_scores<NT, S, kFew>(score, pos, F.rows, cap, moves, dest, posv);
  else if (!F.b) move_scores<NT, S, kMany>(score, pos, F.rows, cap, moves, dest, posv);
  else {
#pragma unroll
    for (int u = 0; u < S; ++u)
      if ((moves >> u) & 1u) pos[dest[u]] = posv[u];
    __syncthreads();                                         // (sh.first is complete)
  }
  if (tid == 0) {
    plan[4 * b + 0] = n; plan[4 * b + 1] = (int)min(sh.first, (uint32_t)n); plan[4 * b + 2] = 1; plan[4 * b + 3] = (int32_t)n_new;
    sq.n_res = (int32_t)n_new;
    sq.compacted = 1;
    if (advance_step) sq.step = s + 1;
  }
}

// grid = (row slices, 2 {K,V}, n_seq).  A workgroup owns a 128-byte column slice of every row
// of one cache and walks the rows that move in ascending tiles: load survivors -> wait, barrier -> store (a tile's destinations
// are at most its sources and below the next tile's).  Bound by the copy: ROWS rows per thread in flight, and since nothing
// reads a row again before the next step's attention, streaming loads and stores.  A tile ends with a wait for its last load, so the
// best tile is the whole list; but ROWS cost registers (30 with 4 rows, 59 with 8, 107 with 16, 151 with 24, 199 with 32) and most workgroups
// of most steps find nothing to move and are over when they have been launched.  So: as many rows as the capacity needs up to 24, and 32
// for launches that are resident with them at once, two workgroups per CU.  An eviction, plan included, us with 16 | 24 | 32 rows: full lists,
// 4 sequences x 32 heads x 4000 slots - | 65.3 | 60.8, 300 x 24 x 1000 585 | 579 | 567, 64 x 16 x 4000 196 | 202 | 195, 162 x 1 x 7631 fp32 114 | 104 | 123;
// 180 tokens in caches of 1500 slots, 300 x 20 69 | 76 | 95, 64 x 20 27.2 | 29.0 | 33.0; no row end, 300 x 16 x 1000 17.2 | 18.1 | 19.9, 150 x 24 x 2000
// 19.8 | 20.5 | 21.8.  The pass of 512 x 24 x 696, 1.05 GB moved: 230.6 us with 24 rows, 234.6 with 16 (20 more with ordinary accesses).
// Short lists: 350 sequences x 33 heads x 64 bf16, us with 16 rows | the ROWS of the rule: 100 slots 86.9 | 55.1, 128 slots 93.3 | 64.5 (4 rows),
// 140 slots 97.8 | 77.1, 256 slots 134.6 | 132.4 (8 rows).
// The strides come as a struct, which is not preloaded: each preloaded argument delays the launch of every wave, and 80 000
// workgroups with nothing to move took 27.4 us with 12 dwords of them, 23.0 with 8.  The record is asked for with the plan's words: one
// round trip less where rows move (64 x 24 x 696, 4 of them at a row end, 25.2 -> 24.0 us), 0.8 us more for 512 sequences of which none does.
// SCORES: the score rows move along.  Up to 16 registers more (36, 64, 114, 163, 215) and a branch between the map and
// the rows, which moves of cache rows alone do not pay for: us with one form for both | with two (rows left to the plan), 300 sequences x 24
// rows x 100 slots 41.9 | 40.0, 300 x 16 x 128 35.1 | 32.9, 600 x 1 x 250 15.4 | 15.0, 16 x 16 x 128 fp32 10.9 | 10.2.
// ADVANCE: the records advance too, after an attention launch that planned.  The two more words of the record are asked for by these launches
// alone: with nothing to move, 512 sequences x 24 rows x 696 slots 18.9 | 18.0, 300 x 24 x 1000 14.4 | 13.9, 261 x 48 x 435 20.2 | 19.0.
constexpr int kSliceLanes = 8;
struct MoveStrides { long long slot_b, head_b; };
template <int ROWS, bool SCORES, bool ADVANCE>
__global__ __launch_bounds__(kMoveThreads) void k_compact_move(const adsa_seq* seqs, const int32_t* keep_map, const int32_t* plan,
                                                              int part_bits, int cap, MoveStrides stride) {
  constexpr int kPass = kMoveThreads / kSliceLanes;
  const int b = blockIdx.z, head = blockIdx.x >> part_bits, part = blockIdx.x & ((1 << part_bits) - 1);
  const int4 pl = reinterpret_cast<const int4*>(plan)[b];
  gseq& sq = ((gseq*)seqs)[b];
  gchar* const cache = (gchar*)(blockIdx.y == 0 ? sq.k : sq.v);
  const int step = ADVANCE ? sq.step : -1, status = ADVANCE ? sq.status : 0;
  asm volatile("" : : "s"(cache));                           // (asked for together with the plan's words, not after them)
  if constexpr (ADVANCE) asm volatile("" : : "s"(step), "s"(status));
  const int n_old = pl.x, first = pl.y;
  if (ADVANCE && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && step >= 0 && status == 0) {   // (no other workgroup uses these)
    if (pl.z == 0) sq.compacted = 0;
    sq.step = step + 1;
  }
  if (pl.z == 0 || first >= n_old) return;
  const int row_in_pass = threadIdx.x / kSliceLanes, lane = threadIdx.x % kSliceLanes;
  gchar* const base = cache + (long long)head * stride.head_b + (part * kSliceLanes + lane) * 16;
  const gint* const map = (const gint*)keep_map + (size_t)b * cap;
  // one workgroup per head also moves the head's score row (attention mass: a row per cache head), where the plan leaves it: see kMovedWithCache
  constexpr int kTile = kPass * ROWS, SLOTS = (kTile + kMoveThreads - 1) / kMoveThreads;
  const bool scores = SCORES && blockIdx.y == 0 && part == 0;
  gfloat* const score = (gfloat*)sq.score + (size_t)head * cap;
  for (int t0 = first; t0 < n_old; t0 += kTile) {
    uint4 val[ROWS];
    int dst[ROWS], sdst[SLOTS];
    float sval[SLOTS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) dst[u] = elem(map, (uint32_t)min(t0 + u * kPass + row_in_pass, n_old - 1));
    if (scores) {
#pragma unroll
      for (int u = 0; u < SLOTS; ++u) {
        const int k = u * kMoveThreads + (int)threadIdx.x, i = min(t0 + k, n_old - 1);
        sdst[u] = elem(map, (uint32_t)i);
        sval[u] = elem(score, (uint32_t)i);
        if (t0 + k >= n_old || k >= kTile || sdst[u] == i) sdst[u] = -1;
      }
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int i = t0 + u * kPass + row_in_pass;
      if (i >= n_old || dst[u] == i) dst[u] = -1;            // (past the end, or stays where it is)
      if (dst[u] >= 0) val[u] = load_stream16(base + (long long)i * stride.slot_b);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this thread's rows are in registers ...
    __syncthreads();                                         // ... and so are everybody's, before any of them is overwritten
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
      if (dst[u] >= 0) store_stream16(base + (long long)dst[u] * stride.slot_b, val[u]);
    if (scores) {
#pragma unroll
      for (int u = 0; u < SLOTS; ++u)
        if (sdst[u] >= 0) elem(score, (uint32_t)sdst[u]) = sval[u];
    }
  }
}

// This workgroup's column slice (blockIdx.x: those of K, then those of V) of the rows first .. n, moved in place by the map in LDS.
template <int NT, int ROWS>
__device__ __forceinline__ void move_slice(gchar* kb, gchar* vb, int n_heads, int part_bits, int first, int n, const int* s_map, MoveStrides stride) {
  const int tid = threadIdx.x, per_cache = n_heads << part_bits;
  const bool is_v = (int)blockIdx.x >= per_cache;
  const int slice = (int)blockIdx.x - (is_v ? per_cache : 0), head = slice >> part_bits, part = slice & ((1 << part_bits) - 1);
  constexpr int kPass = NT / kSliceLanes;
  const int row_in_pass = tid / kSliceLanes, piece = tid % kSliceLanes;
  gchar* const base = (is_v ? vb : kb) + (long long)head * stride.head_b + (part * kSliceLanes + piece) * 16;
  for (int t0 = first; t0 < n; t0 += kPass * ROWS) {
    uint4 val[ROWS];
    int dst[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int i = t0 + u * kPass + row_in_pass;
      dst[u] = s_map[min(i, n - 1)];
      if (i >= n || dst[u] == i) dst[u] = -1;
      if (dst[u] >= 0) val[u] = load_stream16(base + (long long)i * stride.slot_b);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // as in k_compact_move
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
      if (dst[u] >= 0) store_stream16(base + (long long)dst[u] * stride.slot_b, val[u]);
  }
}

// The row-end eviction of one decode step in ONE launch: grid (column slices of K, then of V; sequence).  The attention launch
// before it has advanced the record (kAdvanceActive), so a workgroup whose sequence did not close a row leaves at once and
// touches nothing.  Every workgroup of a sequence that did works out the ranking for itself (from L2, all at the same time)
// and moves its slice of the rows with the map in its LDS; the one that draws the last ticket -- by then all of them have the
// scores and positions they need in registers -- moves pos[] and the score rows and writes the keep map and the record.
// Nothing waits for another workgroup.
template <int NT, int S, int RB = rank_batch(S)>
__global__ __launch_bounds__(NT) void k_compact_step(
    uint32_t seqs_lo, uint32_t map_lo, uint32_t tickets_lo, uint32_t seqs_map_hi, uint32_t tickets_hi, int part_bits, int cap, uint32_t flags,
    int total, int W, int R, int recent_m, float inv_w, int n_heads, long long slot_stride_b, long long head_stride_b) {
  __shared__ __align__(16) RankShared sh;
  __shared__ int s_map[NT * S];
  __shared__ int s_last;
  constexpr int kRows = 16 * kMoveThreads / NT;              // (whole lists up to 2048 slots, 32 rows: 32 x 16 x 1900 at a row end 86 -> 93 us)
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1);
  const RankFlags F(flags);
  gseq& sq = ((gseq*)address(seqs_lo, seqs_map_hi & 0xFFFF))[b];
  gint* const pos = (gint*)sq.pos;
  gfloat* const score = (gfloat*)sq.score;
  gchar* const kb = (gchar*)sq.k;
  gchar* const vb = (gchar*)sq.v;
  const int s = sq.step - 1, n = sq.n_res;                   // s: the step that has just been attended
  const QueryCell cell = make_query_cell(sq, s, GridWidth{W, inv_w}, R, 0, recent_m);
  if (s < 0 || sq.status != 0 || n < 0 || n > cap || !is_row_end(cell, s, total)) return;
  int idx[S], posv[S];
  float rank[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = min(u * NT + tid, n - 1);
    posv[u] = n > 0 ? elem(pos, idx[u]) : 0;                       // (an empty sequence's pointers may be null)
    rank[u] = 0.0f;
  }
  rank_clear<NT>(sh);
  if (n > 0) rank_values<S, RB>(score, F.rows, cap, idx, rank);
  const bool largest = keep_largest_of(F.mode);
  uint32_t key[S], restm = 0, in = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (u * NT + tid < n) in |= 1u << u;
    if (((in >> u) & 1u) && evict_class(cell, posv[u]) == 1) restm |= 1u << u;
    key[u] = order_key(rank[u], largest);
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
  uint32_t moves = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int i = u * NT + tid;
    const bool kept = (take >> u) & 1u;
    s_map[i] = kept ? (int)dest[u] : -1;
    if (kept && dest[u] != (uint32_t)i) moves |= 1u << u;
    const unsigned long long gone = __ballot(((in >> u) & 1u) && !kept);
    if (gone != 0 && lane == 0) atomicMin(&sh.first, (uint32_t)(u * NT + wave_id() * kWave + __ffsll((long long)gone) - 1));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this thread has read what it needs of the scores and positions ...
  __syncthreads();                                           // ... and so has the workgroup: it may draw its ticket
  if (tid == 0) s_last = __hip_atomic_fetch_add((int*)address(tickets_lo, tickets_hi) + 4 * b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;

  move_slice<NT, kRows>(kb, vb, n_heads, part_bits, (int)min(sh.first, (uint32_t)n), n, s_map, MoveStrides{slot_stride_b, head_stride_b});
  __syncthreads();                                           // s_last is there (also when no row moves)
  if (!s_last) return;

  gint* const map = (gint*)address(map_lo, seqs_map_hi >> 16) + (size_t)b * cap;
#pragma unroll
  for (int u = 0; u < S; ++u)
    if ((in >> u) & 1u) map[u * NT + tid] = ((take >> u) & 1u) ? (int32_t)dest[u] : -1;
  move_scores<NT, S>(score, pos, F.rows, cap, moves, dest, posv);
  if (tid == 0) {
    sq.n_res = (int32_t)n_new;
    sq.compacted = 1;
  }
}

// The second kernel of a small decode step, after a k_attend that ranked for itself: grid (column slices of K, then of V; sequence).
// What that launch's workgroups only read is changed here: the scores, which it left in vals ([n_seq][score rows][cap]), and the
// record; at a row end also what k_compact_step does, on those scores.  plan[b] = { tickets, step or -1 if there is nothing to do,
// resident slots with the query token's, attended slots }; where none is attended there are no vals.  No workgroup reads what another one writes: step and count come from the
// plan, scores from vals, and the positions, which the last to draw a ticket moves, are in registers before one is drawn.
// Most steps close no row: the new scores, the plan and the record are one round trip then, the scores' stores the rest.
template <int NT, int S, int RB = rank_batch(S)>
__global__ __launch_bounds__(NT) void k_step_finish(uint32_t seqs_lo, uint32_t map_lo, uint32_t plan_lo, uint32_t vals_lo, uint32_t seqs_map_hi,
                                                    uint32_t plan_vals_hi, uint32_t cap_heads_bits, int total, int W, int R, int recent_m,
                                                    float inv_w, MoveStrides stride) {
  __shared__ __align__(16) RankShared sh;
  __shared__ int s_map[NT * S];
  __shared__ int s_last;
  constexpr int kRows = 16 * kMoveThreads / NT;
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & (kWave - 1);
  const int cap = cap_heads_bits & 0xFFFF, n_heads = (cap_heads_bits >> 16) & 0x1FF, part_bits = cap_heads_bits >> 25;
  gint* const plan = (gint*)address(plan_lo, plan_vals_hi & 0xFFFF) + 4 * b;
  const int s = plan[1], n = plan[2], attended = plan[3];
  gseq& sq = ((gseq*)address(seqs_lo, seqs_map_hi & 0xFFFF))[b];
  gint* const pos = (gint*)sq.pos;
  gfloat* const score = (gfloat*)sq.score;
  gchar* const kb = (gchar*)sq.k;
  gchar* const vb = (gchar*)sq.v;
  const QueryCell cell = make_query_cell(sq, s, GridWidth{W, inv_w}, R, 0, recent_m);
  const gfloat* const vals = (const gfloat*)address(vals_lo, plan_vals_hi >> 16) + (size_t)b * n_heads * cap;
  const bool head_here = (int)blockIdx.x < n_heads;
  float val[S];
#pragma unroll
  for (int u = 0; u < S; ++u) val[u] = head_here ? elem(vals + (size_t)blockIdx.x * cap, min(u * NT + tid, cap - 1)) : 0.0f;
  if (s < 0) return;
  const int slot_new = s >= 1 ? n - 1 : -1, pos_new = cell.P + s - 1;
  if (!is_row_end(cell, s, total)) {
    if (head_here && attended > 0) {                         // (none: step 0 of candidates without a budget; that launch left vals alone)
#pragma unroll
      for (int u = 0; u < S; ++u)
        if (u * NT + tid < n) elem(score + (size_t)blockIdx.x * cap, u * NT + tid) = val[u];
    }
    if (blockIdx.x == 0 && tid == 0) {
      if (slot_new >= 0) pos[slot_new] = pos_new;
      sq.n_res = n; sq.step = s + 1; sq.compacted = 0; sq.pending_slot = slot_new;
    }
    return;
  }
  // ---- a row end (s >= 1, so there is a query token)
  int idx[S], posv[S];
  float rank[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    idx[u] = min(u * NT + tid, n - 1);
    posv[u] = elem(pos, idx[u]);
  }
  rank_clear<NT>(sh);
  rank_values<S, RB>(vals, n_heads, cap, idx, rank);
  uint32_t key[S], restm = 0, in = 0;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int i = u * NT + tid;
    if (i == slot_new) posv[u] = pos_new;
    if (i < n) in |= 1u << u;
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
    const bool kept = (take >> u) & 1u;
    s_map[u * NT + tid] = kept ? (int)dest[u] : -1;
    const unsigned long long gone = __ballot(((in >> u) & 1u) && !kept);
    if (gone != 0 && lane == 0) atomicMin(&sh.first, (uint32_t)(u * NT + wave_id() * kWave + __ffsll((long long)gone) - 1));
  }
  // A head's scores move from vals, one workgroup a row: every slot below n_new is some kept slot's destination, those from there on
  // hold what the attention left them.
  if (head_here) {
    gfloat* const row = score + (size_t)blockIdx.x * cap;
#pragma unroll
    for (int u = 0; u < S; ++u) {
      if ((take >> u) & 1u) elem(row, dest[u]) = val[u];
      if (((in >> u) & 1u) && u * NT + tid >= (int)n_new) elem(row, u * NT + tid) = val[u];
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // as in k_compact_step: all positions are read, the ticket may be drawn
  __syncthreads();
  if (tid == 0) s_last = __hip_atomic_fetch_add((int*)plan, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  move_slice<NT, kRows>(kb, vb, n_heads, part_bits, (int)min(sh.first, (uint32_t)n), n, s_map, stride);
  __syncthreads();                                           // s_last is there (also when no row moves)
  if (!s_last) return;

  gint* const map = (gint*)address(map_lo, seqs_map_hi >> 16) + (size_t)b * cap;
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int i = u * NT + tid;
    if (!((in >> u) & 1u)) continue;
    const bool kept = (take >> u) & 1u;
    map[i] = kept ? (int32_t)dest[u] : -1;
    if (kept && (i == slot_new || dest[u] != (uint32_t)i)) pos[dest[u]] = posv[u];
    if (i == slot_new && i >= (int)n_new) pos[i] = posv[u];
  }
  if (tid == 0) { sq.n_res = (int32_t)n_new; sq.step = s + 1; sq.compacted = 1; sq.pending_slot = slot_new; }
}

}  // namespace

template <int NT, int... REST>
static constexpr int rank_threads() { return NT; }

#define ADSA_RANK_LAUNCH(KERNEL, SHAPE, ...)                                                                 \
  do {                                                                                                       \
    hipLaunchKernelGGL((KERNEL<SHAPE>), dim3(p.n_seq), dim3(rank_threads<SHAPE>()), 0, st, __VA_ARGS__); \
    return hipGetLastError();                                                                                \
  } while (0)
#define ADSA_SHAPE(...) __VA_ARGS__

// Threads and slots per thread of a ranking workgroup, by the slots a sequence can have.  k_select, us at 256x3 | 512x2 |
// 1024x1: 64 sequences x 24 rows x 696 slots 7.6 | 7.2 | 7.4; 1536 x 24 x 696 20.3 | 20.6 | 37.7; 1536 x 8 x 696
// 12.3 | 15.1 | 35; at 256x4 | 512x2: 64 x 24 x 696 8.3 | 7.2; at 512x4 | 1024x2: 200 x 16 x 2000 11.1 | 11.4.  (One
// workgroup of 256 threads with keys in LDS and a 4-pass radix select: 12.4, 27.3, 18.1 and 19.4 us.)  With 3 slots per
// thread, batches of 12 score rows instead of 8 put 25 rows in flight for 28 more registers: k_select 64 x 24 rows
// 7.9 -> 7.3 us, 576 x 20 10.9 -> 10.5, but 1536 x 8 rows 12.2 -> 14.2 for the residency lost: below 1024 sequences only.
// Above 2048 slots residency decides as soon as there are more sequences than CUs: a workgroup of 1024 threads, or of 512 with
// more than 128 registers, has a CU to itself.  us for 16 sequences x 24 score rows, 1024 x 1, 1024 x 24 (in brackets keys in LDS,
// 256 threads): 3072 slots at 512x6 11.8, 23.6, 58.9, at 1024x4 13.2, 39.6, 76.9 (28.1, 26.3, 73.2); 3100 at 512x8 14.0, 26.3,
// 62.3, at 1024x4 13.3, 40.2, 78.3 (31.3, 28.1, 74.6); 6144 at 512x12 19.6, 38.1, 131.6, at 1024x6 18.2, 50.6, 146.7, at 1024x8
// 21.3, 58.6, 160.9 (50.5, 51.6, 155.3); 6200 at 512x16 23.9, 46.2, 139.2, at 1024x8 21.6, 58.8, 158.1 (53.3, 53.2, 152.4).
// (All of these with the arguments in a block and integer divisions by the grid width; with preloaded arguments and without divisions every
// shape gained: 64 x 24 x 696 6.1 -> 5.7, 1536 x 24 x 696 20.5 -> 19.9, 8 x 16 x 8000 18.5 -> 17.5, 400 x 8 x 5000 27.3 -> 25.8.)
hipError_t launch_select(const adsa_params& p, adsa_seq* seqs, int32_t* sel_idx, int32_t* sel_cnt,
                         bool plan_append, int32_t* tickets, hipStream_t st) {
#define ADSA_SELECT(...)                                                                                                                        \
  ADSA_RANK_LAUNCH(k_select, ADSA_SHAPE(__VA_ARGS__), lo32(seqs), lo32(sel_idx), lo32(sel_cnt), lo32(tickets), hi16s(seqs, sel_idx),             \
                   hi16s(sel_cnt, tickets), (uint32_t)p.cap | (uint32_t)p.sel_cap << 16, rank_flags(p, plan_append, tickets != nullptr),         \
                   p.grid_h * p.grid_w, p.grid_w, p.win_rows_back, p.win_col_radius, p.win_recent_m, inv_width(p))
  if (p.cap <= 256) ADSA_SELECT(256, 1);
  if (p.cap <= 512) ADSA_SELECT(256, 2);
  if (p.cap <= 768 && p.n_seq < 1024) ADSA_SELECT(256, 3, 12);
  if (p.cap <= 768) ADSA_SELECT(256, 3);
  if (p.cap <= 1024) ADSA_SELECT(512, 2);
  if (p.cap <= 2048) ADSA_SELECT(512, 4);
  if (p.cap <= 3072) ADSA_SELECT(512, 6);
  if (p.n_seq <= 256) {
    if (p.cap <= 4096) ADSA_SELECT(1024, 4);
    if (p.cap <= 6144) ADSA_SELECT(1024, 6);
    ADSA_SELECT(1024, 8);
  }
  if (p.cap <= 4096) ADSA_SELECT(512, 8);
  if (p.cap <= 6144) ADSA_SELECT(512, 12, 1);
  ADSA_SELECT(512, 16, 1);
}

// (Rows of the fused V-cosine form, two a head, never move: slots are reused.)
static bool moved_with_cache(const adsa_params& p) {
  return score_rows(p) >= kMovedWithCache && p.cap > kPlanRowsCap &&
         (p.n_seq <= kPlanRowsSeqs || (score_rows(p) >= kManyRows && (p.cap <= 256 || p.cap > 384)));
}

// k_compact_plan: 512 sequences x 24 rows x 696 slots at a row end 15.3 us (32.7 with keys in LDS), 512 x 48 rows x 632 of the
// fused V-cosine form 13.6 us (36.9: its loop over the heads waited for every pair of rows).  It needs more registers than
// k_select (512x8 and 512x12 above 128), so above 3072 slots the workgroups of 1024 threads stay ahead at any number of
// sequences.  Nothing dropped, 16 sequences x 24 rows, 1024 x 1, 1024 x 24: 3072 slots at 512x6 12.3, 17.2, 77.5, at 1024x4 12.5, 26.7,
// 92.4; 4096 at 1024x4 12.5, 28.8, 118, at 512x8 14.8, 32.5, 120; 6144 at 1024x6 16.5, 35.7, 167, at 1024x8 20.9, 43.5, 185,
// at 512x12 19.5, 46.1, 178.  (1024x8 keeps 28 bytes of a thread's state in scratch memory.)
static hipError_t launch_compact_plan(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, int32_t* plan,
                                      bool advance_step, const float* vcos_s, hipStream_t st) {
#define ADSA_PLAN(...)                                                                                                                          \
  ADSA_RANK_LAUNCH(k_compact_plan, ADSA_SHAPE(__VA_ARGS__), lo32(seqs), lo32(keep_map), lo32(plan), lo32(vcos_s), hi16s(seqs, keep_map),          \
                   hi16s(plan, vcos_s), (uint32_t)p.cap, rank_flags(p, advance_step, moved_with_cache(p)), p.grid_h * p.grid_w, p.grid_w, p.win_rows_back, \
                   p.win_recent_m, inv_width(p), p.n_heads * p.head_dim)
  if (p.cap <= 256) ADSA_PLAN(256, 1);
  if (p.cap <= 512) ADSA_PLAN(256, 2);
  if (p.cap <= 768) ADSA_PLAN(256, 3, 12);
  if (p.cap <= 1024) ADSA_PLAN(512, 2);
  if (p.cap <= 2048) ADSA_PLAN(512, 4);
  if (p.cap <= 3072) ADSA_PLAN(512, 6);
  if (p.cap <= 4096) ADSA_PLAN(1024, 4);
  if (p.cap <= 6144) ADSA_PLAN(1024, 6);
  ADSA_PLAN(1024, 8);
}

// column slices of a head row (128, 256 or 512 bytes), as a power of two
static int slice_bits(const adsa_params& p) {
  const int slices = p.head_dim * elem_bytes(p) / (kSliceLanes * 16);
  return slices == 1 ? 0 : slices == 2 ? 1 : 2;
}
static long long row_bytes(const adsa_params& p, int64_t stride) { return (long long)stride * elem_bytes(p); }

// One launch instead of two saves a small step ~2.5 us of launching and, most steps closing no row, an empty kernel.  Its ranking
// is repeated by every workgroup, so a large launch pays for it at a row end.  adsa_step, us with two launches | with one:
// 4 sequences x 20 heads (160 workgroups) 17.9 | 16.1 inside a row, 28.3 | 28.6 at its end; 16 x 20 (640) 24.6 | 22.9, 39.8 | 40.0;
// 64 x 24 (3072) 57 | 55, 94 | 105.  So: up to 1024 workgroups, lists up to 2048 slots (the map in LDS), rankings
// that need no pass over V.
bool one_launch_compact(const adsa_params& p) {
  return p.evict_policy == ADSA_EVICT_ROW_END && !is_vcos(p) && p.cap <= 2048 &&
         ((long long)p.n_seq * p.n_heads * 2 << slice_bits(p)) <= 1024;
}

hipError_t launch_compact_step(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, int32_t* tickets, hipStream_t st) {
  const dim3 grid((2 * p.n_heads) << slice_bits(p), p.n_seq);
#define ADSA_STEP_LAUNCH(NT, ...)                                                                            \
  do {                                                                                                       \
    hipLaunchKernelGGL((k_compact_step<NT, __VA_ARGS__>), grid, dim3(NT), 0, st, lo32(seqs), lo32(keep_map), lo32(tickets), hi16s(seqs, keep_map), \
                       hi16s(tickets, nullptr), slice_bits(p), p.cap, rank_flags(p, false, false), p.grid_h * p.grid_w, p.grid_w, p.win_rows_back,   \
                       p.win_recent_m, inv_width(p), p.n_heads, row_bytes(p, p.kv_slot_stride), row_bytes(p, p.kv_head_stride));                   \
    return hipGetLastError();                                                                                \
  } while (0)
  if (p.cap <= 256) ADSA_STEP_LAUNCH(256, 1);
  if (p.cap <= 512) ADSA_STEP_LAUNCH(256, 2);
  if (p.cap <= 768) ADSA_STEP_LAUNCH(256, 3, 12);
  if (p.cap <= 1024) ADSA_STEP_LAUNCH(512, 2);
  if (p.cap <= 2048) ADSA_STEP_LAUNCH(512, 4);
  return hipErrorInvalidValue;
}

hipError_t launch_step_finish(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, char* ws, const Workspace& w, hipStream_t st) {
  const dim3 grid((2 * p.n_heads) << slice_bits(p), p.n_seq);
  const char *const plan = ws + w.plan_off, *const vals = ws + w.logits_off;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, lo32(seqs), lo32(keep_map), lo32(plan), lo32(vals), hi16s(seqs, keep_map), hi16s(plan, vals),
                       (uint32_t)p.cap | (uint32_t)p.n_heads << 16 | (uint32_t)slice_bits(p) << 25, p.grid_h * p.grid_w, p.grid_w, p.win_rows_back,
                       p.win_recent_m, inv_width(p), MoveStrides{row_bytes(p, p.kv_slot_stride), row_bytes(p, p.kv_head_stride)});
    return hipGetLastError();
  };
  if (p.cap <= 256) return launch(k_step_finish<256, 1>, 256);
  if (p.cap <= 512) return launch(k_step_finish<256, 2>, 256);
  if (p.cap <= 768) return launch(k_step_finish<256, 3, 12>, 256);
  if (p.cap <= 1024) return launch(k_step_finish<512, 2>, 512);
  return hipErrorInvalidValue;
}

static hipError_t launch_move(const adsa_params& p, const adsa_seq* seqs, const int32_t* keep_map, const int32_t* plan, bool scores, bool advance, hipStream_t st) {
  const dim3 grid(p.n_heads << slice_bits(p), 2, p.n_seq);
  constexpr int rows_per_pass = kMoveThreads / kSliceLanes;
  const bool resident = (long long)grid.x * grid.y * grid.z <= 2 * 256;
  auto of_rows = [&](auto with_scores, auto with_records) {
    constexpr bool S = decltype(with_scores)::value, A = decltype(with_records)::value;
    constexpr int kLeast = S && !A ? 8 : 4, kMost = A ? 24 : 32;                        // (see moved_with_cache and plan_in_attend)
    return p.cap <= kLeast * rows_per_pass ? k_compact_move<kLeast, S, A> : p.cap <= 8 * rows_per_pass ? k_compact_move<8, S, A>
         : p.cap <= 16 * rows_per_pass ? k_compact_move<16, S, A> : p.cap <= 24 * rows_per_pass || !resident ? k_compact_move<24, S, A>
         : k_compact_move<kMost, S, A>;
  };
  const std::true_type yes;
  const std::false_type no;
  auto move = advance ? of_rows(yes, yes) : scores ? of_rows(yes, no) : of_rows(no, no);
  hipLaunchKernelGGL(move, grid, dim3(kMoveThreads), 0, st, seqs, keep_map,
                     plan, slice_bits(p), p.cap, MoveStrides{row_bytes(p, p.kv_slot_stride), row_bytes(p, p.kv_head_stride)});
  return hipGetLastError();
}

hipError_t launch_compact(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, char* ws,
                          const Workspace& w, bool advance_step, hipStream_t st) {
  int32_t* plan = reinterpret_cast<int32_t*>(ws + w.plan_off);
  const float* vcos_s = p.score_mode == ADSA_SCORE_VCOS_FUSED ? reinterpret_cast<const float*>(ws + w.vcos_s_off) : nullptr;
  hipError_t e = launch_compact_plan(p, seqs, keep_map, plan, advance_step, vcos_s, st);
  if (e != hipSuccess || p.evict_policy == ADSA_EVICT_REUSE_SLOT) return e;     // slot reuse moves no row
  return launch_move(p, seqs, keep_map, plan, moved_with_cache(p), false, st);
}

hipError_t launch_step_move(const adsa_params& p, adsa_seq* seqs, const int32_t* keep_map, char* ws, const Workspace& w, hipStream_t st) {
  return launch_move(p, seqs, keep_map, reinterpret_cast<int32_t*>(ws + w.plan_off), true, true, st);
}

}  // namespace adsa
