// TopK-V redundancy score of the ADSA decode path (gfx950): Eq. 2-3, the mean pairwise cosine
// similarity of a candidate's V vector (all heads concatenated) to the other candidates.
//
// The N x N cosine matrix is never formed.  With v^_i = v_i / max(|v_i|, 1e-8) and
// u = sum_j v^_j over the candidates,  S_i = (v^_i . u - v^_i . v^_i) / (N - 1): two streaming
// passes over the candidates' V rows instead of O(N^2 D) work.
//
//  k_vcos_norm_usum : grid (256 slots or a part of them, sequence).  The candidates of 256 slots are listed in LDS; a wave holds
//                     a slot's whole row in registers: inverse norm by a wave reduction, then the normalised row is
//                     added to the wave's column sums; the waves' sums are added in LDS into a partial of u
//                     (no atomics, every row read once).
//  k_vcos_score     : grid (slot tile, sequence).  Every lane sums its columns of the partials of u into registers,
//                     then a wave per slot takes the dot product and writes S_i into
//                     score[slot] (non-candidate slots keep their score).
//
// The order of u's sums does not depend on the launch, so that a sequence's scores are the same bits in whatever batch it is
// ranked.  Entry k of the list of 256 slots belongs to part k mod 4; a part is cut into 4 runs of equal length (at most 16 rows),
// a run is summed in ascending order, the runs in order make the part, the parts in order the group's sum, and the groups are
// added in order.  A large launch gives a workgroup a whole group (a wave per part: together they walk the list), a small one a
// part (a wave per run).  (The last group of a capacity that is no multiple of 256 has a part per 64 slots: that is the room
// the workspace has.)
//
// Both are bound by the stream of V rows.  A wave keeps a ring of U rows in flight (16 bytes per lane and load, so 3 loads
// for a row of 24 heads x 64 bf16).  256 sequences x 535 candidates of that shape, 420 MB a pass: 79 and 75 us (5.3 and
// 5.6 TB/s); one row of 8-byte loads at a time, the next one asked for after its reduction, took 168 and 184 us.
#include <type_traits>

#include "adsa_device.h"
#include "adsa_internal.h"
#include "adsa_partition.h"

namespace adsa {
namespace {

constexpr int kVcThreads = 256;
constexpr int kVcWaves = kVcThreads / kWave;
constexpr int kVcTile = 64;                 // slots per partial of u the workspace has room for
constexpr int kVcGroup = kVcThreads;        // slots that are listed and summed together
constexpr int kVcParts = kVcGroup / kVcTile, kVcPartRuns = 4;
static_assert(kVcWaves == kVcParts && kVcWaves == kVcPartRuns, "a wave per part or per run");
constexpr int kVcMaxDim = 8192;             // n_heads * head_dim limit

// What the two passes work on, unpacked from the preloaded kernel arguments (kVcosParams; see k_attend on what a load of the
// argument block costs: a launch that finds nothing to do is over before it would arrive).
struct VcosArgs {
  gseq* seqs;
  float* inv_norm;      // [n_seq][cap]
  float* u_part;        // [n_seq][n_parts][dim]: a partial of u per group, or per part of a group (split)
  float* s_out;         // [n_seq][cap] where S_i goes when score[] holds the fused form's rows, else NULL
  int n_heads, head_dim, cap, split, n_parts;     // split: a workgroup of the first pass takes a part of a group
  int tile;                                       // slots per workgroup of the second pass: 64, 128 or 256
  int for_compaction, evict_policy;
  int total, R, w, recent_m;
  GridWidth grid;
};
struct VcosStrides { long long slot_b, head_b; };
// dims: cap | partials << 16;  flags: heads | D == 128 << 9 | split << 10 | tile / 64 << 11 | for an eviction << 14 | policy << 15
#define kVcosParams                                                                                                             \
  uint32_t seqs_lo, uint32_t inv_lo, uint32_t up_lo, uint32_t s_lo, uint32_t seqs_inv_hi, uint32_t up_s_hi, uint32_t dims,     \
      uint32_t flags, int total, int W, int R, int w, int recent_m, float inv_w, VcosStrides strides
#define kVcosUnpack                                                                                                             \
  {(gseq*)address(seqs_lo, seqs_inv_hi & 0xFFFF), reinterpret_cast<float*>(address(inv_lo, seqs_inv_hi >> 16)), \
   reinterpret_cast<float*>(address(up_lo, up_s_hi & 0xFFFF)), reinterpret_cast<float*>(address(s_lo, up_s_hi >> 16)),         \
   (int)(flags & 0x1FF), (flags & 0x200) ? 128 : 64, (int)(dims & 0xFFFF), (int)((flags >> 10) & 1), (int)(dims >> 16),         \
   (int)((flags >> 11) & 7) * 64, (int)((flags >> 14) & 1), (int)((flags >> 15) & 3), total, R, w, recent_m, {W, inv_w}}

// sum over the wave: DPP inside the 16-lane rows, then lane 15 -> next row and lane 31 -> upper half; uniform result
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float x) {
  x = dpp_add<0x111, 0xF>(x); x = dpp_add<0x112, 0xF>(x); x = dpp_add<0x114, 0xF>(x); x = dpp_add<0x118, 0xF>(x);
  x = dpp_add<0x142, 0xA>(x); x = dpp_add<0x143, 0xC>(x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), kWave - 1));
}

__device__ __forceinline__ float4 load_f4(const gfloat* p) {
  const uint4 x = load16((const gchar*)p);
  return make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
}

// candidate test (false for inactive sequences / non row-end compaction)
__device__ __forceinline__ bool vcos_candidate(const VcosArgs& A, const QueryCell& c, int pos) {
  if (A.for_compaction && A.evict_policy == ADSA_EVICT_ROW_END) return evict_class(c, pos) == 1;
  return select_class(c, pos) == 1;     // also the streaming eviction: the incoming query's partition
}

__device__ __forceinline__ bool vcos_active(const VcosArgs& A, const QueryCell& cell, const gseq& sq) {
  if (sq.step < 0 || sq.status != 0 || sq.n_res < 0 || sq.n_res > A.cap) return false;
  if (sq.step > A.total) return false;
  if (!A.for_compaction) return true;
  if (A.evict_policy == ADSA_EVICT_REUSE_SLOT && sq.hole != 0) return false;     // room was made already
  if (A.s_out && sq.vcos_u && ((const gfloat*)sq.vcos_u)[A.n_heads * A.head_dim + 1] == (float)(sq.step + 1))
    return false;                                       // the attention launch left this step's numbers
  if (A.evict_policy != ADSA_EVICT_ROW_END) return sq.step >= 1 && sq.n_res == A.cap;
  return is_row_end(cell, sq.step, A.total);
}

// A concatenated V row as a wave holds it: lane l has the 16-byte pieces l, l + 64, ... (G of them at most; pieces past the
// row's end read piece 0 and count as zero).
template <int EB, int G>
struct Row {
  static constexpr int EPL = 16 / EB;        // elements per piece
  static constexpr int U = G == 1 ? 8 : G == 2 ? 6 : G == 3 ? 4 : G == 4 ? 3 : G <= 8 ? 2 : 1;     // rows in flight per wave
  const gchar* p[G];
  bool on[G];
  int col[G];                                // first column of the piece

  __device__ __forceinline__ Row(const void* v, int n_heads, int head_dim, long long head_stride_b) {
    const int lane = threadIdx.x & (kWave - 1), per_head = head_dim * EB / 16, pieces = n_heads * per_head;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int c = lane + g * kWave;
      on[g] = c < pieces;
      const int cc = on[g] ? c : 0, head = cc / per_head;
      col[g] = cc * EPL;
      p[g] = (const gchar*)v + (long long)head * head_stride_b + (cc - head * per_head) * 16;
    }
  }
  __device__ __forceinline__ void load(long long off, uint4 (&x)[G]) const {
#pragma unroll
    for (int g = 0; g < G; ++g) x[g] = load16(p[g] + off);
  }
  __device__ __forceinline__ void unpack(const uint4 (&x)[G], float (&f)[G][EPL]) const {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint32_t w[4] = {x[g].x, x[g].y, x[g].z, x[g].w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t v = on[g] ? w[k] : 0u;
        if constexpr (EB == 4) f[g][k] = __uint_as_float(v);
        else { f[g][2 * k] = __uint_as_float(v << 16); f[g][2 * k + 1] = __uint_as_float(v & 0xFFFF0000u); }
      }
    }
  }
};

// Calls use(k, row) for entries first, first + step, ... below m of the slots listed in s_row, with U rows in flight.
template <int EB, int G, int U = Row<EB, G>::U, typename Use>
__device__ __forceinline__ void for_rows(const Row<EB, G>& row, long long slot_stride_b, const int* s_row, int first, int step, int m, Use use) {
  if (first >= m) return;
  uint4 x[U][G];
  auto request = [&](int u, int k) {         // (entries past the last re-read it)
    row.load((long long)__builtin_amdgcn_readfirstlane(s_row[min(k, m - 1)]) * slot_stride_b, x[u]);
    asm volatile("" : : : "memory");         // requests leave in ring order
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int u = 0; u < U; ++u) request(u, first + u * step);
  for (int k = first; k < m; k += U * step) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ku = k + u * step;
      if (ku < m) {
        float f[G][Row<EB, G>::EPL];
        row.unpack(x[u], f);
        use(ku, f);
      }
      request(u, ku + U * step);
    }
  }
}

// Lists the slots of [s0, s1) that `member` accepts, ascending, in s_row (one slot per thread); returns their number.
template <typename Member>
__device__ __forceinline__ int list_rows(int* s_row, int* s_cnt, int s0, int s1, Member member) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int i = s0 + tid;
  const bool c = i < s1 && member(i);
  const unsigned long long m = __ballot(c);
  if (lane == 0) s_cnt[wave] = __popcll(m);
  __syncthreads();
  int base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kVcWaves; ++w) {
    const int t = s_cnt[w];
    if (w < wave) base += t;
    total += t;
  }
  if (c) s_row[base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = i;
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(total);
}

template <int EB, int G>
__global__ __launch_bounds__(kVcThreads) void k_vcos_norm_usum(kVcosParams) {
  const VcosArgs A = kVcosUnpack;
  extern __shared__ __align__(16) float s_acc[];        // [kVcWaves][dim]
  __shared__ int s_row[kVcThreads], s_cnt[kVcWaves];
  __shared__ float s_inv[kVcThreads];
  constexpr int EPL = 16 / EB;
  const int part = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const gseq& sq = A.seqs[b];
  const QueryCell cell = make_query_cell(sq, sq.step, A.grid, A.R, A.w, A.recent_m);
  if (!vcos_active(A, cell, sq)) return;
  const int group = A.split ? part / kVcParts : part;
  const int n = sq.n_res, s0 = group * kVcGroup;
  if (s0 >= n) return;
  const int s1 = min(n, s0 + kVcGroup), dim = A.n_heads * A.head_dim;
  const gint* const pos = (const gint*)sq.pos;
  gfloat* const inv_norm = (gfloat*)A.inv_norm + (size_t)b * A.cap;
  const int m = list_rows(s_row, s_cnt, s0, s1, [&](int i) {
    const bool c = vcos_candidate(A, cell, pos[i]);
    if (!c) inv_norm[i] = 0.0f;                          // marks "not a candidate"
    return c;
  });
  // this wave's entries: my_part + parts * t, t from the first run's begin to the last one's end (all four runs of a part, or one)
  const int parts = min(kVcParts, (A.cap - s0 + kVcTile - 1) / kVcTile), my_part = A.split ? part % kVcParts : wave;
  const int n_part = my_part < parts ? (m - my_part + parts - 1) / parts : 0;
  auto run_begin = [&](int r) { return my_part + parts * (n_part * r / kVcPartRuns); };
  int r = A.split ? wave : 0;
  const int k0 = run_begin(r), k1 = run_begin(A.split ? r + 1 : kVcPartRuns);
  const Row<EB, G> row(sq.v, A.n_heads, A.head_dim, strides.head_b);
  float acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.0f;
  float* const mine = s_acc + (size_t)wave * dim;        // the sum of this wave's runs so far
  if (k0 == k1)
    for (int c = lane; c < dim / 4; c += kWave) reinterpret_cast<float4*>(mine)[c] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  int end = k0;                                          // of run r
  while (end == k0 && k0 < k1) end = run_begin(++r);     // (short lists have empty runs)
  bool more = false;
  for_rows(row, strides.slot_b, s_row, k0, parts, min(k1, m), [&](int k, const float (&f)[G][EPL]) {
    float ss = 0.0f;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) ss = fmaf(f[g][e], f[g][e], ss);
    ss = wave_sum(ss);
    const float inv = 1.0f / fmaxf(sqrtf(ss), 1e-8f);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(f[g][e], inv, acc[g][e]);
    if (lane == 0) s_inv[k] = inv;
    if (k + parts == end) {                                // (wave-uniform) the run is complete
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (row.on[g]) {
#pragma unroll
          for (int e = 0; e < EPL; e += 4) {
            float4* const at = reinterpret_cast<float4*>(mine + row.col[g] + e);
            float4 t = make_float4(acc[g][e], acc[g][e + 1], acc[g][e + 2], acc[g][e + 3]);
            if (more) { const float4 o = *at; t.x = o.x + t.x; t.y = o.y + t.y; t.z = o.z + t.z; t.w = o.w + t.w; }
            *at = t;
            acc[g][e] = acc[g][e + 1] = acc[g][e + 2] = acc[g][e + 3] = 0.0f;
          }
        }
      more = true;
      while (end == k + parts && end < k1) end = run_begin(++r);
    }
  });
  __syncthreads();
  if (tid < m && (!A.split || tid % parts == my_part)) inv_norm[s_row[tid]] = s_inv[tid];
  gchar* const up = (gchar*)((gfloat*)A.u_part + ((size_t)b * A.n_parts + part) * (size_t)dim);
  for (int c = tid; c < dim / 4; c += kVcThreads) {
    float4 t = reinterpret_cast<const float4*>(s_acc)[c];
#pragma unroll
    for (int w = 1; w < kVcWaves; ++w) {
      const float4 o = reinterpret_cast<const float4*>(s_acc + (size_t)w * dim)[c];
      t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
    }
    store16(up + c * 16, make_uint4(__float_as_uint(t.x), __float_as_uint(t.y), __float_as_uint(t.z), __float_as_uint(t.w)));
  }
}

// The sequences are walked in the opposite order of the first pass: what that read last is still in the memory-side cache.
template <int EB, int G>
__global__ __launch_bounds__(kVcThreads) void k_vcos_score(kVcosParams) {
  const VcosArgs A = kVcosUnpack;
  __shared__ int s_row[kVcThreads], s_cnt[kVcWaves], s_n[kVcWaves];
  __shared__ float s_inv[kVcThreads], s_res[kVcThreads];       // by slot of the tile; by entry of s_row
  constexpr int EPL = 16 / EB;
  const int tile = gridDim.x - 1 - blockIdx.x, b = gridDim.y - 1 - blockIdx.y, tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  gseq& sq = A.seqs[b];
  if (!vcos_active(A, make_query_cell(sq, sq.step, A.grid, A.R, A.w, A.recent_m), sq)) return;
  const int n = sq.n_res, s0 = tile * A.tile;
  if (s0 >= n) return;
  const int s1 = min(n, s0 + A.tile), dim = A.n_heads * A.head_dim;
  const int parts_used = A.split ? min((n + kVcGroup - 1) / kVcGroup * kVcParts, A.n_parts) : (n + kVcGroup - 1) / kVcGroup;
  const gfloat* const invs = (const gfloat*)A.inv_norm + (size_t)b * A.cap;
  int my = 0;
  for (int i = tid; i < n; i += kVcThreads) my += invs[i] != 0.0f;
  const Row<EB, G> row(sq.v, A.n_heads, A.head_dim, strides.head_b);
  const gfloat* const up = (const gfloat*)A.u_part + (size_t)b * A.n_parts * (size_t)dim;
  float uu[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) uu[g][e] = 0.0f;
  for (int t = 0; t < parts_used; t += A.split ? kVcParts : 1) {      // groups in order, a group's own parts first
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPL; e += 4) {
        const gfloat* const at = up + (size_t)t * dim + row.col[g] + e;
        float4 x = load_f4(at);
        if (A.split) {
          float4 y[kVcParts];
#pragma unroll
          for (int j = 1; j < kVcParts; ++j) y[j] = load_f4(at + (size_t)min(j, parts_used - 1 - t) * dim);
#pragma unroll
          for (int j = 1; j < kVcParts; ++j)
            if (t + j < parts_used) { x.x += y[j].x; x.y += y[j].y; x.z += y[j].z; x.w += y[j].w; }
        }
        if (row.on[g]) { uu[g][e] += x.x; uu[g][e + 1] += x.y; uu[g][e + 2] += x.z; uu[g][e + 3] += x.w; }
      }
  }
  for (int d = 32; d >= 1; d >>= 1) my += __shfl_xor(my, d, kWave);
  if (lane == 0) s_n[wave] = my;
  const int m = list_rows(s_row, s_cnt, s0, s1, [&](int i) {
    const float inv = invs[i];
    s_inv[i - s0] = inv;
    return inv != 0.0f;
  });
  int N = 0;
#pragma unroll
  for (int w = 0; w < kVcWaves; ++w) N += s_n[w];
  gfloat* const out = A.s_out ? (gfloat*)A.s_out + (size_t)b * A.cap : (gfloat*)sq.score;
  for_rows(row, strides.slot_b, s_row, __builtin_amdgcn_readfirstlane(wave), kVcWaves, m, [&](int k, const float (&f)[G][EPL]) {
    float dot = 0.0f, ss = 0.0f;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) { dot = fmaf(f[g][e], uu[g][e], dot); ss = fmaf(f[g][e], f[g][e], ss); }
    dot = wave_sum(dot);
    ss = wave_sum(ss);
    const float inv = s_inv[s_row[k] - s0];
    // remove the i == j term (1 for a normal row, 0 for a zero row) and average over the others
    const float self = ss * inv * inv;
    if (lane == 0) s_res[k] = N > 1 ? (dot * inv - self) / (float)(N - 1) : 0.0f;
  });
  __syncthreads();
  if (tid < m) out[s_row[tid]] = s_res[tid];
}

// ADSA_SCORE_VCOS_FUSED: bring u to the candidate set of the NEXT step, after this step's eviction plan and
// before its attention launch (which takes every row's dot product with u).  One workgroup per sequence.
// If u belongs to this step: subtract the evicted row, add the rows that turn from local to candidate
// (normally the one token that leaves the 1-D window).  Otherwise: a fresh sum over the next step's
// candidates.  (512 | 1536 sequences of 632 slots, two rows each: 8.1 | 14.8 us; 8.6 | 16.2 with a ring of 4 rows and the list
// beside the sums in LDS, 10.9 with 256 slots listed at a time and u requested last, 18.3 with every row read twice.)
// The slots that join or leave are listed 1024 at a time; wave w takes entries w, w+4, ... in ascending order into
// its own registers, and the waves' sums are added to u in wave order, so the result does not depend on timing.
constexpr int kAdvRounds = 4;                           // slots per thread and list
// (a ring of one row: two rows are all there is to read in most steps, and the registers of a deeper one would cost residency)
template <int EB, int G>
__global__ __launch_bounds__(kVcThreads) void k_vcos_advance(adsa_seq* seqs, uint32_t heads_d, int cap, int total, int W, int R, int w,
                                                             int recent_m, float inv_w, long long slot_stride_b, long long head_stride_b) {
  extern __shared__ __align__(16) float s_acc[];        // the list (slots, then signs), after it [kVcWaves][dim]
  constexpr int EPL = 16 / EB, kRounds = kAdvRounds;
  __shared__ int s_cnt[kRounds][kVcWaves];
  int* const s_row = reinterpret_cast<int*>(s_acc);
  float* const s_sign = s_acc + kRounds * kVcThreads;   // by entry of s_row
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  gseq& sq = ((gseq*)seqs)[b];
  gfloat* const U = (gfloat*)sq.vcos_u;
  if (sq.step < 0 || sq.status != 0 || U == nullptr) return;
  const int s = sq.step, n = sq.n_res, n_heads = heads_d & 0xFFFF, head_dim = heads_d >> 16, dim = n_heads * head_dim;
  if (n < 0 || n > cap) return;
  gfloat* const tags = U + dim;
  if (s + 1 > total) {                    // no later step evicts
    if (tid == 0) tags[0] = 0.0f;
    return;
  }
  const gint* const pos = (const gint*)sq.pos;
  const int victim = sq.hole - 1;                       // slot freed by this step's eviction, or -1
  const QueryCell now = make_query_cell(sq, s, GridWidth{W, inv_w}, R, w, recent_m);
  const QueryCell next = make_query_cell(sq, s + 1, GridWidth{W, inv_w}, R, w, recent_m);
  const Row<EB, G> row(sq.v, n_heads, head_dim, head_stride_b);
  const bool incremental = tags[0] == (float)(s + 1);   // u is the sum over THIS step's candidates
  float acc[G][EPL];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[g][e] = 0.0f;
  // (u itself is needed last, but requested now: with two rows to move this kernel is nothing but memory round trips)
  constexpr int kOld = G * EPL / kVcWaves > 0 ? G * EPL / kVcWaves : 1;     // dim <= G * 64 * EPL
  float old[kOld];
#pragma unroll
  for (int k = 0; k < kOld; ++k) old[k] = U[min(tid + k * kVcThreads, dim - 1)];
  for (int base = 0; base < n; base += kRounds * kVcThreads) {
    int posv[kRounds];
    float sign[kRounds];
    unsigned long long member[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) posv[r] = pos[min(base + r * kVcThreads + tid, n - 1)];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      // what happens to each slot: +1 joins u, -1 leaves it, 0 nothing
      const int i = base + r * kVcThreads + tid;
      const bool cand_next = select_class(next, posv[r]) == 1;
      sign[r] = 0.0f;
      if (incremental) {
        const bool cand_now = select_class(now, posv[r]) == 1;
        if (i == victim) sign[r] = cand_now ? -1.0f : 0.0f;
        else if (cand_next && !cand_now) sign[r] = 1.0f;
      } else if (cand_next && i != victim) sign[r] = 1.0f;
      if (i >= n) sign[r] = 0.0f;
      member[r] = __ballot(sign[r] != 0.0f);
      if (lane == 0) s_cnt[r][wave] = __popcll(member[r]);
    }
    __syncthreads();
    int m = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {                 // ascending slots: round, wave, lane
      int at = m;
#pragma unroll
      for (int w = 0; w < kVcWaves; ++w) {
        const int t = s_cnt[r][w];
        if (w < wave) at += t;
        m += t;
      }
      if (sign[r] != 0.0f) {
        at += __builtin_amdgcn_mbcnt_hi((uint32_t)(member[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)member[r], 0u));
        s_row[at] = base + r * kVcThreads + tid;
        s_sign[at] = sign[r];
      }
    }
    m = __builtin_amdgcn_readfirstlane(m);
    __syncthreads();
    for_rows<EB, G, 1>(row, slot_stride_b, s_row, wave, kVcWaves, m, [&](int k, const float (&f)[G][EPL]) {
      float ss = 0.0f;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) ss = fmaf(f[g][e], f[g][e], ss);
      const float c = s_sign[k] / fmaxf(sqrtf(wave_sum(ss)), 1e-8f);
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] = fmaf(f[g][e], c, acc[g][e]);
    });
    __syncthreads();                                    // the list is free for the next 1024 slots
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
    if (row.on[g]) {
#pragma unroll
      for (int e = 0; e < EPL; e += 4)
        *reinterpret_cast<float4*>(s_acc + (size_t)wave * dim + row.col[g] + e) = make_float4(acc[g][e], acc[g][e + 1], acc[g][e + 2], acc[g][e + 3]);
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOld; ++k) {
    const int c = tid + k * kVcThreads;
    if (c >= dim) break;
    float t = incremental ? old[k] : 0.0f;
#pragma unroll
    for (int w = 0; w < kVcWaves; ++w) t += s_acc[(size_t)w * dim + c];
    U[c] = t;
  }
  if (tid == 0) tags[0] = (float)(s + 2);               // u now belongs to step s + 1
}

// Calls f(EB, G) as compile-time constants: G pieces of 16 bytes per lane hold a concatenated row.
template <typename F>
hipError_t with_row_shape(const adsa_params& p, F f) {
  const int pieces = p.n_heads * p.head_dim * elem_bytes(p) / 16, g = (pieces + kWave - 1) / kWave;
  auto pick = [&](auto eb) {
    if (g <= 1) return f(eb, std::integral_constant<int, 1>());
    if (g <= 2) return f(eb, std::integral_constant<int, 2>());
    if (g <= 3) return f(eb, std::integral_constant<int, 3>());
    if (g <= 4) return f(eb, std::integral_constant<int, 4>());
    if (g <= 6) return f(eb, std::integral_constant<int, 6>());
    if (g <= 8) return f(eb, std::integral_constant<int, 8>());
    if (g <= 16) return f(eb, std::integral_constant<int, 16>());
    if constexpr (decltype(eb)::value == 4) return f(eb, std::integral_constant<int, 32>());
    else return hipErrorInvalidValue;
  };
  return elem_bytes(p) == 4 ? pick(std::integral_constant<int, 4>()) : pick(std::integral_constant<int, 2>());
}

}  // namespace

int vcos_tiles(int cap) { return (cap + kVcTile - 1) / kVcTile; }

VcosPlan make_vcos_plan(const adsa_params& p) {
  // As large a tile as still gives every CU two workgroups: the second pass reads every partial of u in each workgroup
  // (256 sequences x 692 slots: 154 us both passes with tiles of 256, 177 with 128; taking 128 or 64 sequences at a time so that
  // the second pass finds them in the memory-side cache costs more in short launches than it saves: 192 and 256 us).
  VcosPlan v;
  v.tile = kVcGroup;
  while (v.tile > kVcTile && (long long)p.n_seq * ((p.cap + v.tile - 1) / v.tile) < 512) v.tile /= 2;
  // First pass: a workgroup per part for launches of few groups, where a workgroup per group leaves the chip short of rows in
  // flight; whole groups write and read a quarter of the partials, which counts more the longer a row is.  Both passes, time of
  // groups / time of parts over 120 random shapes, rows under 2 KB | longer ones: 100-200 groups 1.32 | 0.97, 200-350 1.16 | 1.00,
  // 350-500 1.13 | 0.92, 640-800 1.05 | 1.00, 800-1200 1.01 | 0.93; 768 groups of 24 x 64 bf16 156 us | 170.
  const int groups = (p.cap + kVcGroup - 1) / kVcGroup;
  v.split = (long long)p.n_seq * groups < (p.n_heads * p.head_dim * elem_bytes(p) < 2048 ? 640 : 320);
  v.n_parts = v.split ? vcos_tiles(p.cap) : groups;
  return v;
}

// Which parameters ADSA_SCORE_VCOS_FUSED takes: those whose four sums of u and a byte per slot fit 64 KB.  A limit of the interface
// (adsa.h states it), not what k_vcos_advance asks for: its sums, or its list of 8 KB, are always within it.
bool vcos_fused_fits(const adsa_params& p) {
  return sizeof(float) * (size_t)p.n_heads * p.head_dim * kVcWaves + (((size_t)p.cap + 15) / 16) * 16 <= 64 * 1024;
}

hipError_t launch_vcos_advance(const adsa_params& p, adsa_seq* seqs, hipStream_t st) {
  if (!vcos_fused_fits(p)) return hipErrorInvalidValue;
  return with_row_shape(p, [&](auto eb, auto g) {
    constexpr int EB = decltype(eb)::value, G = decltype(g)::value;
    if constexpr (G * 16 / EB <= 64) {                  // (longer rows: refused above)
      const size_t list = 2 * sizeof(int) * kAdvRounds * kVcThreads, sums = sizeof(float) * (size_t)p.n_heads * p.head_dim * kVcWaves;
      hipLaunchKernelGGL((k_vcos_advance<EB, G>), dim3(p.n_seq), dim3(kVcThreads), list > sums ? list : sums, st, seqs, (uint32_t)p.n_heads | (uint32_t)p.head_dim << 16,
                         p.cap, p.grid_h * p.grid_w, p.grid_w, p.win_rows_back, p.win_col_radius, p.win_recent_m, 1.0f / (float)p.grid_w,
                         (long long)p.kv_slot_stride * elem_bytes(p), (long long)p.kv_head_stride * elem_bytes(p));
      return hipGetLastError();
    } else return hipErrorInvalidValue;
  });
}

hipError_t launch_vcos(const adsa_params& p, adsa_seq* seqs, bool for_compaction, char* ws,
                       const Workspace& w, hipStream_t st) {
  const int dim = p.n_heads * p.head_dim;
  if (dim > kVcMaxDim) return hipErrorInvalidValue;
  const float* const inv_norm = reinterpret_cast<float*>(ws + w.vcos_off);
  const float* const u_part = reinterpret_cast<float*>(ws + w.vcos_u_off);
  const float* const s_out = p.score_mode == ADSA_SCORE_VCOS_FUSED ? reinterpret_cast<float*>(ws + w.vcos_s_off) : nullptr;
  const VcosPlan vp = make_vcos_plan(p);
  const uint32_t flags = p.n_heads | (p.head_dim == 128 ? 1u << 9 : 0u) | (vp.split ? 1u << 10 : 0u) | (uint32_t)(vp.tile / 64) << 11 |
                         (for_compaction ? 1u << 14 : 0u) | (uint32_t)p.evict_policy << 15;
  const VcosStrides strides = {(long long)p.kv_slot_stride * elem_bytes(p), (long long)p.kv_head_stride * elem_bytes(p)};
  const dim3 grid1(vp.n_parts, p.n_seq), grid2((p.cap + vp.tile - 1) / vp.tile, p.n_seq);
  auto launch = [&](auto kernel, const dim3& grid, size_t lds) {
    hipLaunchKernelGGL(kernel, grid, dim3(kVcThreads), lds, st, lo32(seqs), lo32(inv_norm), lo32(u_part), lo32(s_out), hi16s(seqs, inv_norm),
                       hi16s(u_part, s_out), (uint32_t)p.cap | (uint32_t)vp.n_parts << 16, flags, p.grid_h * p.grid_w, p.grid_w, p.win_rows_back,
                       p.win_col_radius, p.win_recent_m, 1.0f / (float)p.grid_w, strides);
    return hipGetLastError();
  };
  return with_row_shape(p, [&](auto eb, auto g) {
    constexpr int EB = decltype(eb)::value, G = decltype(g)::value;
    // (64..128 KB of LDS, above the default per-launch limit: allowed once per device by vcos_prepare_kernels)
    const hipError_t e = launch(k_vcos_norm_usum<EB, G>, grid1, sizeof(float) * (size_t)dim * kVcWaves);
    return e == hipSuccess ? launch(k_vcos_score<EB, G>, grid2, 0) : e;
  });
}

// Rows of 4096 elements need 64 KB of dynamic LDS (4 waves' sums) beside the static words, rows of 8192 (the limit) 128 KB: more
// than a launch may ask for by default.  Allowed here, once per device, at the library's first use of that device.
hipError_t vcos_prepare_kernels() {
  const void* kernels[] = {reinterpret_cast<const void*>(&k_vcos_norm_usum<2, 8>), reinterpret_cast<const void*>(&k_vcos_norm_usum<2, 16>),
                           reinterpret_cast<const void*>(&k_vcos_norm_usum<4, 16>), reinterpret_cast<const void*>(&k_vcos_norm_usum<4, 32>),
                           reinterpret_cast<const void*>(&k_vcos_advance<2, 8>), reinterpret_cast<const void*>(&k_vcos_advance<4, 16>)};
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace adsa
