// Internal declarations shared by the translation units of the ADSA HIP library:
// launch plan (how the attended set is split over workgroups), workspace layout,
// and the kernel launchers the C-ABI layer calls.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "adsa.h"

namespace adsa {

constexpr int kWave = 64;
constexpr int kMoveThreads = 256;
constexpr int kMaxChunks = 16;         // a list is split over at most this many workgroups

// Attend launch plan: a workgroup handles (sequence, head or heads, token chunk).
struct AttendPlan {
  int n_chunks;         // token chunks per list; every sequence splits its own count evenly
  int chunk_max;        // upper bound of tokens in one chunk, + 1
  int reserved_chunks;  // chunks per list the workspace has room for (>= n_chunks)
  int waves;            // waves per attend workgroup: 4 or 8
  int heads;            // heads per attend workgroup: 1, or 512 bytes' worth of a token of a [slot][head][D] cache
  bool wide;            // rows further apart than 32-bit offsets from 24-bit products reach
};

// Rows of adsa_seq.score: one accumulator per head for ATTN_MASS (the rank of a slot is their sum),
// a single row otherwise.
static inline int score_rows(const adsa_params& p) {
  if (p.score_mode == ADSA_SCORE_VCOS_FUSED) return 2 * p.n_heads;    // per head: |v|^2 share, v.u share
  return p.score_mode == ADSA_SCORE_ATTN_MASS ? p.n_heads : 1;
}
// Eq. 2-3 ranking in either form
static inline bool is_vcos(const adsa_params& p) {
  return p.score_mode == ADSA_SCORE_VCOS || p.score_mode == ADSA_SCORE_VCOS_FUSED;
}
constexpr int kVcosTags = 4;      // floats after u in adsa_seq.vcos_u: [0] 1 + step u belongs to, [1] 1 + step the score rows belong to

// Workspace layout (byte offsets from a 256-byte aligned base).
struct Workspace {
  size_t head_bytes;       // leading bytes that adsa_workspace_init zeroes; no kernel uses them, but they are part of the size
                           // and of the offsets callers' workspaces were made for
  size_t logits_off;       // float [n_seq][n_heads][lg_stride]  scaled logits in log2 units of split lists; or, over this and the two
                           //                      regions below, the new scores [n_seq][n_heads][cap] of a step in two launches
  size_t part_ml_off;      // float [n_seq][n_heads][n_chunks][2]   (m, l) per chunk
  size_t part_acc_off;     // float [n_seq][n_heads][n_chunks][head_dim]
  size_t plan_off;         // int32 [n_seq][4]   compaction: old n_res, first moved slot, did, new n_res (word 0: tickets where workgroups draw them)
  size_t vcos_off;         // float [n_seq][cap]   inverse V norms of the candidates (0 = not a candidate)
  size_t vcos_u_off;       // float [n_seq][ceil(cap/64)][n_heads*head_dim]   per-tile partial sums of v^
  size_t vcos_s_off;       // float [n_seq][cap]   Eq. 3's S_i of the two-pass computation when score[] holds
                           //                      the fused form's rows (ADSA_SCORE_VCOS_FUSED)
  size_t total;
  int lg_stride;           // sel_cap rounded up to a multiple of 4
};

AttendPlan make_attend_plan(const adsa_params& p);
Workspace make_workspace(const adsa_params& p, const AttendPlan& plan);

static inline int elem_bytes(const adsa_params& p) { return p.dtype == ADSA_F32 ? 4 : 2; }

// What an attention launch does to the record when it is done with a sequence.
enum : int {
  kAdvanceNone = 0,
  kAdvance = 1,            // step += 1 for every sequence it attended
  kAdvanceActive = 2       // step += 1 and compacted = 0 for every active sequence, also one without an attended token: the
                           // bookkeeping of a step whose eviction kernel, next on the stream, then only touches row ends
};

// Kernel launchers (each returns hipGetLastError() of its launch).
hipError_t launch_workspace_init(char* ws, const Workspace& w, hipStream_t st);
// tickets: NULL, or the plan words that launch_compact_step or launch_planned_attend counts in, which the launch clears
hipError_t launch_select(const adsa_params& p, adsa_seq* seqs, int32_t* sel_idx, int32_t* sel_cnt,
                         bool plan_append, int32_t* tickets, hipStream_t st);
hipError_t launch_vcos(const adsa_params& p, adsa_seq* seqs, bool for_compaction, char* ws,
                       const Workspace& w, hipStream_t st);
int vcos_tiles(int cap);
struct VcosPlan {
  bool split;      // a workgroup of the first pass takes a part of 256 slots instead of all of them
  int n_parts;     // partials of u per sequence
  int tile;        // slots per workgroup of the second pass: 64, 128 or 256
};
VcosPlan make_vcos_plan(const adsa_params& p);
// ADSA_SCORE_VCOS_FUSED, after the eviction plan: u <- u - evicted row + the row that turns candidate next step
// (or a fresh sum when u does not belong to this step)
hipError_t launch_vcos_advance(const adsa_params& p, adsa_seq* seqs, hipStream_t st);
bool vcos_fused_fits(const adsa_params& p);
hipError_t launch_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q,
                         const void* k_new, const void* v_new, const int32_t* sel_idx, const int32_t* sel_cnt,
                         void* out, float* lse, char* ws, const Workspace& w, bool accumulate, bool append,
                         int advance, bool new_f32, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop);
// grouped-query path (q_per_kv >= 2): matrix-core kernel, one workgroup per (sequence, cache head, chunk of the list)
constexpr size_t kGqaMaxLds = 128 * 1024;     // dynamic LDS one workgroup may ask for
static inline bool gqa_two_fit(size_t lds) { return 2 * (lds + 2048) <= 160 * 1024; }      // on a CU, static words included
int gqa_logit_stride(const adsa_params& p, int n_chunks);
int gqa_global_logit_stride(const adsa_params& p);
size_t gqa_lds_bytes(const adsa_params& p, int waves, int n_chunks);
hipError_t launch_attend_gqa(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q,
                             const void* k_new, const void* v_new, const int32_t* sel_idx,
                             const int32_t* sel_cnt, void* out, float* lse, char* ws, const Workspace& w,
                             bool accumulate, bool append, int advance, bool new_f32, hipStream_t st,
                             hipEvent_t ev_start, hipEvent_t ev_stop);
hipError_t launch_compact(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, char* ws,
                          const Workspace& w, bool advance_step, hipStream_t st);
// The row-end eviction of a whole decode step in one launch (where one_launch_compact says so): after an attention launch with
// kAdvanceActive, `tickets` cleared by the step's launch_select.
bool one_launch_compact(const adsa_params& p);
// A larger step's attention with the eviction plans of its row ends, and the move after it, which advances the records.  The plan words
// must be zero before (launch_select's tickets).
bool plan_in_attend(const adsa_params& p, const AttendPlan& plan);
hipError_t launch_planned_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q, const void* k_new, const void* v_new,
                                 int32_t* sel_idx, int32_t* sel_cnt, void* out, float* lse, int32_t* keep_map, char* ws, const Workspace& w, bool new_f32,
                                 hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop);
hipError_t launch_step_move(const adsa_params& p, adsa_seq* seqs, const int32_t* keep_map, char* ws, const Workspace& w, hipStream_t st);
hipError_t launch_compact_step(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, int32_t* tickets, hipStream_t st);
// A step of few pairs in two launches (where rank_in_attend says so): the attention launch ranks for itself and leaves in the workspace
// what launch_step_finish does to the record, pos and score, at a row end with the eviction.
bool rank_in_attend(const adsa_params& p, const AttendPlan& plan, const Workspace& w);
hipError_t launch_ranked_attend(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q, const void* k_new, const void* v_new,
                                int32_t* sel_idx, int32_t* sel_cnt, void* out, float* lse, char* ws, const Workspace& w, bool new_f32,
                                hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop);
hipError_t launch_step_finish(const adsa_params& p, adsa_seq* seqs, int32_t* keep_map, char* ws, const Workspace& w, hipStream_t st);
// once per device, before the first launch there: kernels that may ask for more than 64 KB of dynamic LDS
hipError_t gqa_prepare_kernels();
hipError_t vcos_prepare_kernels();

}  // namespace adsa

// What the launch rules decide for parameters p, for tests that have to know which way a call goes (host only; not in adsa.h).
extern "C" {
struct adsa_launch_plan {
  int32_t chunks, waves, heads;       // attention: chunks per list, waves and heads per workgroup
  int32_t eviction;                   // a row end of adsa_step: 0 k_compact_plan and _move, 1 k_compact_step, 2 k_step_finish, 3 the attention and _move
  int32_t vcos_split, vcos_tile;      // V-cosine passes
  int32_t wide;                       // attention: the form with 64-bit offsets
};
int adsa_plan_of(const adsa_params* p, adsa_launch_plan* out);
int adsa_step_launches(const adsa_params* p);      // kernels of an adsa_step that evicts by rows and has no pass over V: 2, 3 or 4; else 0
}
