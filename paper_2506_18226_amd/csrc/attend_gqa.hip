// Grouped-query gather flash-decode of the ADSA decode path (gfx950): Eq. 5's gather + softmax
// attention when G = 2..16 query heads share one cache head.  Every K/V row read from HBM now
// meets G queries, so the two products are small dense contractions and run on the matrix cores
// (v_mfma_f32_16x16x16_bf16, fp32 accumulation); the kernel is still bound by the HBM stream.
//
//  k_attend_gqa<D, NW, SPLIT, R> : grid (cache head, sequence), NW waves.  The list is cut into 16-token tiles,
//  dealt round-robin to the waves of the workgroup (a fixed assignment: results are reproducible bit
//  for bit; claiming tiles from a counter was measured no faster), and each wave runs its own online
//  softmax:
//    S[t][g] = K[t] . q[g]   K rows are fetched with coalesced 16-byte loads and staged through a
//            wave-private LDS tile (the MFMA operand layout wants lane%16 = token; a global load in
//            that shape would touch 16 rows per quarter wave), then multiplied with the G (<= 16)
//            query rows held in registers.  The product comes out with lane%16 = query and 4
//            consecutive tokens per lane: exactly the operand layout of the next product, so the
//            probabilities never leave the registers.  The scaled logits (log2 units) are also kept
//            in LDS, [G][list], for the score update.
//    out[g][:] += 2^(S - m[g]) V[t]   V rows come straight from HBM in operand layout: a lane loads the
//            same D/16 columns of 4 tokens and transposes the 4 x D/16 block in registers (the
//            contraction runs over tokens).  P is split into two bf16 halves (hi + lo) so that the
//            product carries ~16 mantissa bits of the probabilities.  When a query's running maximum
//            m[g] grows, the accumulators are rescaled (factors fetched across lanes).
//    Each wave keeps one to four tiles (R) in flight: it waits for the OLDEST tile's K rows only (in-order wait
//    counts; a tile is always requested as its K loads followed by its V loads, with no branch in between),
//    multiplies it and refills its registers with the tile one ring revolution later.  Loads take a uniform base
//    and a 32-bit lane offset; the query token's own slot is read like any other and replaced from registers.
//    The first round trip (count, sequence record, q, slot list, the query token's row) depends on preloaded
//    kernel arguments only, and leaves before anything waits for a scalar load.
//    At the end the waves' (m, l, partial out) are merged through LDS in wave order, the workgroup writes
//    out / lse for its G query heads and adds the probabilities of all G queries, summed in ascending head
//    order, to its OWN cache head's row of score[]: no workgroup talks to another.
#include <hip/hip_ext.h>

#include <type_traits>

#include "adsa_internal.h"
#include "adsa_device.h"

namespace adsa {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ s16x4 as_bf16x4(uint32_t lo, uint32_t hi) {
  const u32x2 v = {lo, hi};
  return __builtin_bit_cast(s16x4, v);
}

__device__ __forceinline__ f32x4 mfma_bf16(s16x4 a, s16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Lanes of one wave hand data to each other through LDS: LDS instructions of a wave execute in
// issue order, so only the compiler has to be kept from moving accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// c ? a : b by components (a ternary on the structs themselves would select between their ADDRESSES and
// keep both in memory)
__device__ __forceinline__ uint4 pick16(bool c, const uint4& a, const uint4& b) {
  return make_uint4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}

// 2 or 4 dwords of a V row: streaming (nontemporal) or plain
template <int W, bool stream>
__device__ __forceinline__ void vload(const gchar* p, uint32_t* w) {
  if constexpr (W == 2) {
    u32x2 v;
    if constexpr (stream) v = __builtin_nontemporal_load(reinterpret_cast<const ADSA_GLOBAL u32x2*>(p));
    else v = *reinterpret_cast<const ADSA_GLOBAL u32x2*>(p);
    w[0] = v.x; w[1] = v.y;
  } else {
    uint4 v;
    if constexpr (stream) v = load_stream16(p);
    else v = load16(p);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  }
}

// lane g's value, g uniform
__device__ __forceinline__ float lane_f(float x, int g) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), g)); }

// Tiles in flight per wave.  8 KB of loads: with no more registers than that (124 and, at D = 128, the limit of 128) two 8-wave workgroups share a CU, and one
// hides the other's first trip, merge and stores (48 x 8 lists x 300 tokens x 128: 15.7 us with 1 tile, 19.2 with 2; 32 x 8 x 649
// x 64 11.4 with 1 or 2, 12.9 with 4).  Where there is one 8-wave workgroup per CU anyway it makes no difference: 32 x 8 x 649 x 128
// 17.6 with 1, 17.9 with 2, 19.3 with 3.
constexpr int ring(int D) { return D == 64 ? 2 : 1; }
// A 4-wave workgroup that has a CU to itself (its logits fill the LDS) needs twice the depth: 79 x 2 lists x 1330 tokens x 128,
// G = 16, 34.7 us with 1 tile, 27.7 with 2; 20 x 2 x 1313 x 128, G = 4, 28.6 and 22.9.
constexpr int deep_ring(int D) { return 2 * ring(D); }

struct GqaArgs {
  adsa_seq* seqs;
  const char* q;
  const char* k_new;
  const char* v_new;
  const int32_t* sel_idx;
  const int32_t* sel_cnt;
  char* out;
  float* lse;
  float* logits;        // [n_seq][n_heads * G][lg_global]  scaled logits, log2 units (split launches)
  float* part_ml;       // [n_seq][n_heads * G][n_chunks][2]
  float* part_acc;      // [n_seq][n_heads * G][n_chunks][D]
  int lg_global;        // row stride of logits
  int n_heads, G, sel_cap, cap;
  int accumulate, append, advance;
  int new_f32;          // k_new / v_new are fp32 although the cache is bf16: round as they enter
  long long slot_stride_b, head_stride_b;
  float scale_log2;
};

// What a workgroup needs when its rows are summed: a block of 16 dwords behind the leading arguments.
struct GqaTail {
  char* out;
  float* lse;
  float* logits;
  float* part_ml;
  float* part_acc;
  int lg_global, advance;
  int unused[4];
};
static_assert(sizeof(GqaTail) == 64, "one dword per lane of a 16-lane row");

// Everything up to the sums is in the 14 dwords of leading arguments that are preloaded into scalar registers at wave launch (see
// k_attend): heads_flags: heads | G << 9 | append << 16 | fp32 rows << 17 | accumulate << 18 | upper 5 bits of the head stride << 19
// | chunks << 24;  caps: cap | sel_cap << 16.
// SPLIT: the list of a (sequence, cache head) is cut into gridDim.z chunks of whole 16-token tiles, one workgroup
// each; every workgroup leaves a partial and its logits in the workspace and k_gqa_finish merges them in chunk order.
// R: tiles in flight per wave (a ring: the oldest is multiplied, then refilled).
// (held to the 128 registers that let two 8-wave workgroups share a CU, but for the deep rings)
template <int D, int NW, bool SPLIT, int R>
__global__ __launch_bounds__(NW * kWave, R > ring(D) ? 1 : 4) void k_attend_gqa(uint32_t seqs_lo, uint32_t idx_lo, uint32_t cnt_lo, uint32_t q_lo,
                                                          uint32_t kn_lo, uint32_t vn_lo, uint32_t seqs_idx_hi, uint32_t cnt_q_hi,
                                                          uint32_t kn_vn_hi, uint32_t heads_flags, uint32_t caps, uint32_t stride32,
                                                          uint32_t head_stride16, float scale_log2, GqaTail T) {
  constexpr int kThreads = NW * kWave;
  constexpr int ROWB = D * 2 + 16;          // bytes of a staged K row (padded against bank conflicts)
  constexpr int LPR = D / 8;                // lanes per K row with 16-byte loads
  constexpr int RPL = kWave / LPR;          // rows per wave-load
  constexpr int LT = 16 / RPL;              // wave-loads per 16-token tile
  constexpr int NC = D / 16;                // 16-wide chunks of the q.k contraction
  constexpr int EV = D / 16;                // V columns a lane holds per token
  constexpr int VW = EV / 2;                // dwords of V a lane loads per token
  constexpr int PF = 2048 / kThreads;              // slot-list entries a thread fetches in the first round trip
  extern __shared__ __align__(16) char smem[];
  __shared__ float s_wm[NW][16], s_wl[NW][16];

  const int hk = blockIdx.x, b = blockIdx.y;
  const int chunk = SPLIT ? blockIdx.z : 0, n_chunks = SPLIT ? heads_flags >> 24 : 1;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r = lane & 15, kg = lane >> 4;                 // matrix-operand role of this lane
  const int n_heads = heads_flags & 0x1FF, G = (heads_flags >> 9) & 0x1F, sel_cap = caps >> 16, cap = caps & 0xFFFF;
  const bool append = (heads_flags & 0x10000) != 0, cvt = (heads_flags & 0x20000) != 0, keep_logits = (heads_flags & 0x40000) != 0;
  const int HQ = n_heads * G;

  // ---- first round trip: the count and the sequence record (scalar loads), q, the whole slot list (one entry per
  // thread and round) and the query token's own K/V row as this launch attends and stores it -- everything that
  // depends on the kernel arguments only.  The record and the count are pinned so that they cannot drift behind
  // the count test below, into a second, dependent trip.
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)address(seqs_lo, seqs_idx_hi & 0xFFFF) + b;
  const int cnt_raw = ((const gint*)address(cnt_lo, cnt_q_hi & 0xFFFF))[b];
  gchar* const k_rec = (gchar*)sqp->k;
  gchar* const v_rec = (gchar*)sqp->v;
  gfloat* const score_rec = (gfloat*)sqp->score;
  const int pending = sqp->pending_slot;
  __builtin_amdgcn_sched_barrier(0);                       // (the scalar loads leave first)
  const gint* const idx = (const gint*)address(idx_lo, seqs_idx_hi >> 16) + (size_t)b * sel_cap;
  const SlotList list(idx, sel_cap);
  const gchar* const q_g = (const gchar*)address(q_lo, cnt_q_hi >> 16);
  // q as the B operand of the first product: lane (g = r, kg) holds columns [D/4*kg, D/4*(kg+1)) of query g
  const gchar* const q_row0 = q_g + ((size_t)b * HQ + (size_t)hk * G) * D * 2;        // query 0 of this cache head
  uint4 qx[NC / 2];
#pragma unroll
  for (int c2 = 0; c2 < NC / 2; ++c2) qx[c2] = load16(q_row0 + ((size_t)min(r, G - 1) * D + (D / 4) * kg) * 2 + c2 * 16);
  // The slots of the wave's first R tiles (lane 16 * u + j: token j of tile u) and the whole list (one entry per thread and
  // round) that goes to LDS for the later ones.  (A chunk of a split list starts where the count says: fetched below.)
  static_assert(R <= 4, "16 lanes per tile");
  const int ld_row = lane / LPR, ld_piece = lane - ld_row * LPR;
  const int first_at = (wave + kg * NW) * 16 + r;            // list position of this lane's token
  int slot_first = 0, pf_slot[PF];
  if constexpr (!SPLIT) {
    slot_first = list[first_at];
#pragma unroll
    for (int k = 0; k < PF; ++k) pf_slot[k] = list[tid + k * kThreads];
  }
  // the query token's row (Section 4.2 append); fp32 rows are rounded once, here: every lane keeps the pieces of
  // the rounded row it would load from the cache (K: 16 bytes at ld_piece, V: its EV columns)
  const size_t new_row = ((size_t)b * n_heads + hk) * D;
  uint4 nk = make_uint4(0u, 0u, 0u, 0u);
  uint32_t nv[VW];
#pragma unroll
  for (int i = 0; i < VW; ++i) nv[i] = 0u;
  if (append) {
    const gchar* const kn = (const gchar*)address(kn_lo, kn_vn_hi & 0xFFFF);
    const gchar* const vn = (const gchar*)address(vn_lo, kn_vn_hi >> 16);
    if (cvt) {
      nk = pack8_bf16(kn + (new_row + ld_piece * 8) * 4);
      if constexpr (EV == 8) {
        const uint4 x = pack8_bf16(vn + (new_row + r * 8) * 4);
        nv[0] = x.x; nv[1] = x.y; nv[2] = x.z; nv[3] = x.w;
      } else {
        const uint4 x = load16(vn + (new_row + r * 4) * 4);
        nv[0] = pack2_bf16(__uint_as_float(x.x), __uint_as_float(x.y));
        nv[1] = pack2_bf16(__uint_as_float(x.z), __uint_as_float(x.w));
      }
    } else {
      nk = load16(kn + new_row * 2 + ld_piece * 16);
      vload<VW, false>(vn + new_row * 2 + r * (EV * 2), nv);
    }
  }
  pin_uniform(cnt_raw); pin_uniform(k_rec); pin_uniform(v_rec); pin_uniform(score_rec); pin_uniform(pending);
  const long long head_stride_b = (long long)address(head_stride16, (heads_flags >> 19) & 0x1F) * 16;
  gchar* const k_base = k_rec + hk * head_stride_b;
  gchar* const v_base = v_rec + hk * head_stride_b;
  gfloat* const score = score_rec + (size_t)hk * cap;

  const int cnt = min(cnt_raw, sel_cap);
  if (cnt <= 0) {                                    // inactive or rejected sequence: zero-filled rows
    if (chunk == 0) {
      const size_t row = (size_t)b * HQ + (size_t)hk * G;
      for (int o = tid; o < G * D; o += kThreads) {
        ((ADSA_GLOBAL uint16_t*)T.out)[row * D + o] = 0;
        if (o % D == 0) ((gfloat*)T.lse)[row + o / D] = 0.0f;
      }
      if (hk == 0 && tid == 0) advance_empty(sqp, T.advance);
    }
    return;
  }
  // this workgroup's tiles of the list: all of them, or chunk `chunk` of n_chunks (whole tiles; the last chunk is
  // never empty, chunks beyond the number of tiles are)
  const int tiles_all = (cnt + 15) / 16;
  const int tile_begin = SPLIT ? (int)(((unsigned)tiles_all * (unsigned)chunk) / (unsigned)n_chunks) : 0;
  const int tile_end = SPLIT ? (int)(((unsigned)tiles_all * (unsigned)(chunk + 1)) / (unsigned)n_chunks) : tiles_all;
  if (tile_begin >= tile_end) return;
  const int t_begin = tile_begin * 16;
  const int len = min(cnt, tile_end * 16) - t_begin;           // tokens of this workgroup, numbered from 0 below
  const int n_tiles = tile_end - tile_begin;
  // LDS: per wave a K tile [16][ROWB] that later holds its partial out [G][D], the slots, the logits [G][lgs]
  const int stage_b = max(16 * ROWB, G * D * 4), lgs = n_tiles * 16 + 4;       // (rows 4 words apart modulo the banks)
  char* const s_stage = smem;
  int* const s_slot = reinterpret_cast<int*>(smem + NW * stage_b);
  float* const s_logit = reinterpret_cast<float*>(s_slot + n_tiles * 16);
  s16x4 qb[NC];
#pragma unroll
  for (int c2 = 0; c2 < NC / 2; ++c2) {
    const uint4 x = r < G ? qx[c2] : make_uint4(0u, 0u, 0u, 0u);
    qb[2 * c2] = as_bf16x4(x.x, x.y);
    qb[2 * c2 + 1] = as_bf16x4(x.z, x.w);
  }
  const int new_slot = (append && pending >= 0 && pending < cap) ? pending : -1;

  char* const stage = s_stage + wave * stage_b;      // LDS this wave owns

  // Ring of R tiles per wave.  Ring position u holds unit k of the wave, i.e. tile wave + k * NW, for k = u, u + R, ...
  // A tile is LT K loads and 4 V loads per lane.  Its K registers go to the next tile of the ring position as soon as they
  // are in LDS, its V registers when they are multiplied, always in that order and with no branch in between, so that "the
  // oldest K rows have arrived" is one in-order wait count and a wave has a tile in flight nearly all the time.  (32 x 8 lists
  // x 647 x 128, G = 8: 17.0 us with both requested when the tile was done, 16.4 now; G = 16 on 512 pairs 36.2 and 34.2, on 158 pairs with
  // 1335 tokens 55 and 50.)
  uint4 kr[R][LT];
  uint32_t vr[R][4][VW];
  uint32_t fresh_k[R], fresh_v[R];                   // bit l: K load l, bit i: V load i stands for the query token's own row
  // byte offsets inside one head's rows fit 32 bits (cap <= 8192 slots, rows at most 64 KB apart): the loads then
  // take a uniform base and a 32-bit lane offset, two instructions of address arithmetic instead of a 64-bit product
  const uint32_t k_lane_off = (uint32_t)ld_piece * 16u, v_lane_off = (uint32_t)r * (EV * 2);
  // The query token's own slot is read like any other (valid memory of the cache; the row is stored at the end of
  // this launch) and what arrives is replaced by the row held in registers when the tile is multiplied.
  auto in_order = [] {
    asm volatile("" : : : "memory");                 // requests leave in ring order (the wait counts rely on it)
    __builtin_amdgcn_sched_barrier(0);               // ... and before the arithmetic that follows, which waits for ITS rows
  };
  auto request_k = [&](int u, const int (&sk)[LT]) {
    uint32_t f = 0u;
#pragma unroll
    for (int l = 0; l < LT; ++l) {
      kr[u][l] = load_stream16(k_base + ((uint32_t)sk[l] * stride32 + k_lane_off));
      f |= sk[l] == new_slot ? (1u << l) : 0u;
    }
    fresh_k[u] = f;
    in_order();
  };
  auto request_v = [&](int u, const int (&sv)[4]) {
    uint32_t f = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      vload<VW, true>(v_base + ((uint32_t)sv[i] * stride32 + v_lane_off), vr[u][i]);
      f |= sv[i] == new_slot ? (1u << i) : 0u;
    }
    fresh_v[u] = f;
    in_order();
  };
  auto slots_k = [&](int tile, int (&sk)[LT]) {      // (tiles past the end re-read the last row)
#pragma unroll
    for (int l = 0; l < LT; ++l) sk[l] = s_slot[min(tile * 16 + l * RPL + ld_row, len - 1)];
  };
  auto slots_v = [&](int tile, int (&sv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sv[i] = s_slot[min(tile * 16 + 4 * kg + i, len - 1)];
  };

  uint32_t tail = 0u;                                // lane i (modulo 16): dword i of T
  float m_run = -INFINITY, l_lane = 0.0f;            // online softmax of query g = r (l: this lane's tokens only)
  f32x4 acc[EV];                                     // acc[j][i] = partial out[g = 4*kg + i][d = EV*r + j]
#pragma unroll
  for (int j = 0; j < EV; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // multiplies ring position u, which holds tile `tile`; refill: requests tile `next` for it on the way
  auto fold = [&](int u, int tile, auto refill, int next) {
    constexpr bool kRefill = decltype(refill)::value;
    int sk[LT], sv[4];
    if constexpr (kRefill) { slots_k(next, sk); slots_v(next, sv); }
    if (__any(fresh_k[u] != 0u)) {                   // (rare) the tile holds the query token: its row comes from registers
#pragma unroll
      for (int l = 0; l < LT; ++l) kr[u][l] = pick16(((fresh_k[u] >> l) & 1u) != 0, nk, kr[u][l]);
    }
    wave_lds_sync();                                 // the previous tile's operand reads are issued
#pragma unroll
    for (int l = 0; l < LT; ++l)
      *reinterpret_cast<uint4*>(stage + (l * RPL + ld_row) * ROWB + ld_piece * 16) = kr[u][l];
    if constexpr (kRefill) { in_order(); request_k(u, sk); }
    wave_lds_sync();
    const char* rowp = stage + r * ROWB + kg * (D / 2);     // token r of the tile, this lane's columns
    f32x4 s4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c2 = 0; c2 < NC / 2; ++c2) {
      const uint4 x = *reinterpret_cast<const uint4*>(rowp + c2 * 16);
      s4 = mfma_bf16(as_bf16x4(x.x, x.y), qb[2 * c2], s4);
      s4 = mfma_bf16(as_bf16x4(x.z, x.w), qb[2 * c2 + 1], s4);
    }
    // s4[i] = q[g = r] . K[token tile*16 + 4*kg + i]
    const int t0 = tile * 16 + 4 * kg;
    float z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = (t0 + i < len) ? s4[i] * scale_log2 : -INFINITY;
    if (keep_logits && r < G)
      *reinterpret_cast<float4*>(s_logit + (size_t)r * lgs + t0) = make_float4(z[0], z[1], z[2], z[3]);
    float tm = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
    tm = xor_max<32>(xor_max<16>(tm));               // maximum of query r over the tile (its first token is valid)
    const float m_new = fmaxf(m_run, tm);
    if (__any(m_new > m_run)) {                      // some query's maximum grew: rescale what was summed so far
      const float c = fast_exp2(m_run - m_new);      // 0 for the first tile
      l_lane *= c;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ci = __shfl(c, 4 * kg + i, kWave);     // factor of query 4*kg + i
#pragma unroll
        for (int j = 0; j < EV; ++j) acc[j][i] *= ci;
      }
      m_run = m_new;
    }
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float p = fast_exp2(z[i] - m_run);
      if (r >= G) p = 0.0f;
      l_lane += p;
      hi[i] = __float_as_uint(p) & 0xFFFF0000u;
      lo[i] = __float_as_uint(p - __uint_as_float(hi[i])) >> 16;     // exact difference, truncated
    }
    if (__any(fresh_v[u] != 0u)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int w2 = 0; w2 < VW; ++w2) vr[u][i][w2] = (fresh_v[u] >> i) & 1u ? nv[w2] : vr[u][i][w2];
      }
    }
    const s16x4 a_hi = as_bf16x4((hi[0] >> 16) | hi[1], (hi[2] >> 16) | hi[3]);
    const s16x4 a_lo = as_bf16x4(lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16));
#pragma unroll
    for (int w2 = 0; w2 < VW; ++w2) {
      const uint32_t r0 = vr[u][0][w2], r1 = vr[u][1][w2], r2 = vr[u][2][w2], r3 = vr[u][3][w2];
      // columns 2*w2 (low halves) and 2*w2+1 (high halves) of the 4 tokens
      const s16x4 b_even = as_bf16x4((r0 & 0xFFFFu) | (r1 << 16), (r2 & 0xFFFFu) | (r3 << 16));
      const s16x4 b_odd = as_bf16x4((r0 >> 16) | (r1 & 0xFFFF0000u), (r2 >> 16) | (r3 & 0xFFFF0000u));
      acc[2 * w2] = mfma_bf16(a_hi, b_even, acc[2 * w2]);
      acc[2 * w2] = mfma_bf16(a_lo, b_even, acc[2 * w2]);
      acc[2 * w2 + 1] = mfma_bf16(a_hi, b_odd, acc[2 * w2 + 1]);
      acc[2 * w2 + 1] = mfma_bf16(a_lo, b_odd, acc[2 * w2 + 1]);
    }
    // the tile is multiplied completely before the loads that reuse its ring position are issued
    asm volatile("" : "+v"(m_run), "+v"(l_lane) : : "memory");
    if constexpr (kRefill) request_v(u, sv);
  };

  {
    // wave w takes tiles w, w + NW, ...: a fixed assignment, so results are reproducible bit for bit.  Units
    // 0 .. R-1 are requested here; trip t multiplies units (t-1)R .. tR-1 (all of them real tiles) and requests
    // the units one ring revolution later; the last trip only multiplies, and skips ring positions without a tile.
    const int n_mine = n_tiles > wave ? (n_tiles - wave + NW - 1) / NW : 0;
    const int n_trips = (n_mine + R - 1) / R;
    if constexpr (!SPLIT) {
      // ... from the slots the first round trip brought in registers; the list is staged in LDS while the rows are on their way.
      // Positions past the end of the list re-read the last token's row, as slots_k and slots_v do (0 times another row need not be 0: that
      // row may hold an infinity the list's own sums do not meet there); a tile without a token reads some row and is not multiplied.
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int end = __builtin_amdgcn_readlane(slot_first, 16 * u + min(max(len - 1 - (wave + u * NW) * 16, 0), 15));
        slot_first = kg == u && first_at >= len ? end : slot_first;
      }
      slot_first = min(max(slot_first, 0), cap - 1);
      int sk[R][LT], sv[R][4];
#pragma unroll
      for (int u = 0; u < R; ++u) {
#pragma unroll
        for (int l = 0; l < LT; ++l) sk[u][l] = __shfl(slot_first, 16 * u + l * RPL + ld_row, kWave);
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[u][i] = __shfl(slot_first, 16 * u + 4 * kg + i, kWave);
      }
#pragma unroll
      for (int u = 0; u < R; ++u) { request_k(u, sk[u]); request_v(u, sv[u]); }
    }
  // slots of the list, clamped into the cache, go to LDS (readers clamp their list position to the last token)
  if constexpr (!SPLIT) {
#pragma unroll
    for (int k = 0; k < PF; ++k) {
      const int j = tid + k * kThreads;
      if (j < len) s_slot[j] = min(max(pf_slot[k], 0), cap - 1);
    }
    for (int j = tid + PF * kThreads; j < len; j += kThreads) s_slot[j] = min(max(idx[j], 0), cap - 1);
  } else {
    for (int j = tid; j < len; j += kThreads) s_slot[j] = min(max(idx[t_begin + j], 0), cap - 1);
  }
    // (a vector load behind the first rows': its scalar form would be waited for with the record)
    tail = ((const ADSA_GLOBAL uint32_t*)((const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr() + kLeadBytes))[lane % 16];
    __syncthreads();
    if constexpr (SPLIT) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        int sk[LT], sv[4];
        slots_k(wave + u * NW, sk);
        slots_v(wave + u * NW, sv);
        request_k(u, sk);
        request_v(u, sv);
      }
    }
    int k0 = 0;                                      // unit at ring position 0
    for (int trip = 1; trip < n_trips; ++trip) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        fold(u, wave + (k0 + u) * NW, std::true_type(), wave + (k0 + R + u) * NW);
      }
      k0 += R;
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int tile = wave + (k0 + u) * NW;
      if (tile < n_tiles) fold(u, tile, std::false_type(), 0);             // wave-uniform
    }
  }
  l_lane = xor_sum<32>(xor_sum<16>(l_lane));
  if (lane < 16) { s_wm[wave][lane] = m_run; s_wl[wave][lane] = l_lane; }
  // one slab of partial outputs per wave, merged below with the waves' softmax weights
  wave_lds_sync();                                   // (the slab reuses the wave's K tile)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int g = 4 * kg + i;
    if (g < G) {
      float* dst = reinterpret_cast<float*>(stage) + (size_t)g * D + EV * r;
#pragma unroll
      for (int j = 0; j < EV; ++j) dst[j] = acc[j][i];
    }
  }
  __syncthreads();
  // Every wave works out for itself, lane r for query r: the waves' softmax weights 2^(m_w - M), the normaliser and its
  // logarithm; a query's values are then fetched by lane.  (One wave doing it for all behind a second barrier was slower.)
  float wgt[NW], M = -INFINITY, L = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) { wgt[w] = s_wm[w][r]; M = fmaxf(M, wgt[w]); }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wgt[w] = (wgt[w] == -INFINITY) ? 0.0f : fast_exp2(wgt[w] - M);         // a wave that saw no tile: weight 0
    L = fmaf(s_wl[w][r], wgt[w], L);
  }
  const float lse2 = M + __log2f(L), inv_l = 1.0f / L;
  const size_t hq0 = (size_t)b * HQ + (size_t)hk * G;           // first query head of this cache head
  auto tail_word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)tail, i); };
  auto tail_address = [&](size_t at) { return address(tail_word(at / 4), tail_word(at / 4 + 1)); };
  ADSA_GLOBAL uint16_t* const out = (ADSA_GLOBAL uint16_t*)tail_address(offsetof(GqaTail, out)) + hq0 * D;
  gfloat* const lse = (gfloat*)tail_address(offsetof(GqaTail, lse)) + hq0;
  gfloat* const part_acc = (gfloat*)tail_address(offsetof(GqaTail, part_acc));
  gfloat* const part_ml = (gfloat*)tail_address(offsetof(GqaTail, part_ml));
  const int advance = tail_word(offsetof(GqaTail, advance) / 4);
  for (int o = tid; o < G * D; o += kThreads) {
    const int g = __builtin_amdgcn_readfirstlane(o / D), d = o - g * D;       // (a wave's 64 columns belong to one query)
    float a = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) a = fmaf(reinterpret_cast<const float*>(s_stage + w * stage_b)[o], lane_f(wgt[w], g), a);
    if constexpr (!SPLIT) {
      out[o] = (uint16_t)f32_to_bf16_rne(a * lane_f(inv_l, g));
      if (d == 0) lse[g] = lane_f(lse2, g) * kLn2;
    } else {                                         // this chunk's partial, relative to its own maximum
      const size_t pidx = (hq0 + g) * n_chunks + chunk;
      part_acc[pidx * D + d] = a;
      if (d == 0) { part_ml[pidx * 2] = lane_f(M, g); part_ml[pidx * 2 + 1] = lane_f(L, g); }
    }
  }
  // Section 4.2 append: this cache head's rows of the new token, from the registers that attended them
  if (new_slot >= 0 && wave == 0 && chunk == n_chunks - 1) {
    const long long off = (long long)new_slot * stride32;
    if (ld_row == 0) store16(k_base + off + ld_piece * 16, nk);
    if (kg == 0) {
      if constexpr (VW == 4) store16(v_base + off + r * 16, make_uint4(nv[0], nv[1], nv[2], nv[3]));
      else {
        u32x2 v; v.x = nv[0]; v.y = nv[1];
        *reinterpret_cast<ADSA_GLOBAL u32x2*>(v_base + off + r * 8) = v;
      }
    }
  }

  if constexpr (!SPLIT) {
    // ---------------- attention mass of this cache head: sum over its G queries, ascending
    // Each (cache head, slot) word is touched by exactly one thread of one workgroup per launch, so a
    // no-return hardware add gives the same fp32 sum as a load + store, without waiting for the load
    // (requesting the old values before the loop and storing plainly was measured: not faster).
    if (keep_logits) {
      for (int t = tid; t < len; t += kThreads) {
        float inc = 0.0f;
        for (int g0 = 0; g0 < G; g0 += 8) {          // eight queries' logits in flight together
          float z[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) z[k] = s_logit[(size_t)min(g0 + k, G - 1) * lgs + t];
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (g0 + k < G) inc += fast_exp2(z[k] - lane_f(lse2, g0 + k));
        }
        unsafeAtomicAdd((float*)(score + s_slot[t]), inc);
      }
    }
    if (hk == 0 && tid == 0) advance_step(sqp, advance);     // no other workgroup reads step
  } else {
    // ---------------- several chunks: this workgroup's partial and logits are in the workspace; k_gqa_finish, the next kernel
    // on the stream, merges them (the launch boundary orders the two and makes the stores visible on every XCD)
    if (keep_logits) {
      gfloat* const logits = (gfloat*)tail_address(offsetof(GqaTail, logits));
      const int lg_global = tail_word(offsetof(GqaTail, lg_global) / 4);
      for (int g = 0; g < G; ++g) {
        gfloat* const lg = logits + (hq0 + g) * lg_global + t_begin;
        for (int t = tid; t < len; t += kThreads) lg[t] = s_logit[(size_t)g * lgs + t];
      }
    }
  }
}

// Second half of a split launch: grid (token slice, cache head, sequence).  Thread (g, c) weighs chunk c of query g; slice 0
// merges the partial outputs in chunk order and writes out / lse; every slice adds the probabilities of its tokens, summed over
// the queries in ascending order, to the cache head's score row.
constexpr int kFinishThreads = 256, kFinishTokens = 2 * kFinishThreads;
static_assert(kMaxChunks == 16 && kFinishThreads == 16 * 16, "one thread per (query, chunk), a query's chunks in one 16-lane row");
template <int D>
__global__ __launch_bounds__(kFinishThreads) void k_gqa_finish(
    uint32_t seqs_lo, uint32_t idx_lo, uint32_t cnt_lo, uint32_t out_lo, uint32_t lse_lo, uint32_t lg_lo, uint32_t ml_lo, uint32_t acc_lo,
    uint32_t seqs_idx_hi, uint32_t cnt_out_hi, uint32_t lse_lg_hi, uint32_t ml_acc_hi, uint32_t caps, uint32_t flags) {
  const int n_heads = flags & 0x1FF, G = (flags >> 9) & 0x1F, advance = (flags >> 18) & 3, n_chunks = flags >> 24, cap = caps & 0xFFFF, sel_cap = caps >> 16;
  const int lg_global = (sel_cap + 15) / 16 * 16 + 16;
  const bool accumulate = (flags & 0x10000) != 0;
  __shared__ float s_w[16][kMaxChunks], s_lse2[16], s_l[16];
  const int slice = blockIdx.x, hk = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  ADSA_GLOBAL adsa_seq* const sqp = (ADSA_GLOBAL adsa_seq*)address(seqs_lo, seqs_idx_hi & 0xFFFF) + b;
  const int cnt = min(((const gint*)address(cnt_lo, cnt_out_hi & 0xFFFF))[b], sel_cap);
  if (cnt <= 0 || slice * kFinishTokens >= cnt) return;      // (inactive sequences: zero rows, already written)
  const size_t hq0 = ((size_t)b * n_heads + hk) * G;
  const unsigned tiles = (unsigned)(cnt + 15) / 16;
  auto on = [&](int c) {                                     // chunks without a tile hold nothing (their workspace words are stale)
    return c < n_chunks && (tiles * (unsigned)c) / (unsigned)n_chunks < (tiles * (unsigned)(c + 1)) / (unsigned)n_chunks;
  };
  const gfloat* const ml = (const gfloat*)address(ml_lo, ml_acc_hi & 0xFFFF);
  const gint* const idx = (const gint*)address(idx_lo, seqs_idx_hi >> 16) + (size_t)b * sel_cap;
  const int t0 = slice * kFinishTokens + tid;
  int slot[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) slot[u] = min(max(idx[min(t0 + u * kFinishThreads, cnt - 1)], 0), cap - 1);
  {
    const int g = tid / 16, c = tid % 16;
    const bool have = g < G && on(c);
    const float m = have ? ml[((hq0 + g) * n_chunks + c) * 2] : -INFINITY, l = have ? ml[((hq0 + g) * n_chunks + c) * 2 + 1] : 0.0f;
    float M = m;
#pragma unroll
    for (int x = 1; x < 16; x <<= 1) M = fmaxf(M, __shfl_xor(M, x, kWave));
    const float w = m == -INFINITY ? 0.0f : fast_exp2(m - M);
    float L = 0.0f;
#pragma unroll
    for (int k = 0; k < kMaxChunks; ++k) L = fmaf(__shfl(l, (tid & 48) + k, kWave), __shfl(w, (tid & 48) + k, kWave), L);
    s_w[g][c] = w;
    if (c == 0) { s_lse2[g] = M + __log2f(L); s_l[g] = L; }
  }
  __syncthreads();
  if (slice == 0) {
    ADSA_GLOBAL uint16_t* const out = (ADSA_GLOBAL uint16_t*)address(out_lo, cnt_out_hi >> 16) + hq0 * D;
    for (int o = tid; o < G * D; o += kFinishThreads) {
      const int g = o / D, d = o - g * D;
      const gfloat* const acc = (const gfloat*)address(acc_lo, ml_acc_hi >> 16) + (hq0 + g) * n_chunks * D + d;
      float ac[kMaxChunks], a = 0.0f;
#pragma unroll
      for (int c = 0; c < kMaxChunks; ++c) ac[c] = on(c) ? acc[(size_t)c * D] : 0.0f;
#pragma unroll
      for (int c = 0; c < kMaxChunks; ++c) a = fmaf(ac[c], s_w[g][c], a);
      out[o] = (uint16_t)f32_to_bf16_rne(__fdividef(a, s_l[g]));
      if (d == 0) ((gfloat*)address(lse_lo, lse_lg_hi & 0xFFFF))[hq0 + g] = s_lse2[g] * kLn2;
    }
  }
  if (accumulate) {
    gfloat* const score = (gfloat*)sqp->score + (size_t)hk * cap;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = t0 + u * kFinishThreads;
      if (t >= cnt) continue;
      const gfloat* const lg = (const gfloat*)address(lg_lo, lse_lg_hi >> 16) + hq0 * lg_global + t;
      float inc = 0.0f;
      for (int g0 = 0; g0 < G; g0 += 8) {
        float z[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) z[k] = lg[(size_t)min(g0 + k, G - 1) * lg_global];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (g0 + k < G) inc += fast_exp2(z[k] - s_lse2[g0 + k]);
      }
      unsafeAtomicAdd((float*)(score + slot[u]), inc);
    }
  }
  if (slice == 0 && hk == 0 && tid == 0) advance_step(sqp, advance);
}

template <int D, int NW, bool SPLIT, int R>
hipError_t launch_gqa_w(const GqaArgs& A, int n_seq, int n_chunks, size_t lds, hipStream_t st, hipEvent_t ev_start,
                        hipEvent_t ev_stop) {
  dim3 grid(A.n_heads, n_seq, n_chunks);     // (lists that need more than 64 KB of LDS: see gqa_prepare_kernels)
  const uint32_t flags = A.n_heads | A.G << 9 | (A.append ? 0x10000 : 0) | (A.new_f32 ? 0x20000 : 0) | (A.accumulate ? 0x40000 : 0) | (uint32_t)(A.head_stride_b >> 36 & 0x1F) << 19 | n_chunks << 24;
  const GqaTail T = {A.out, A.lse, A.logits, A.part_ml, A.part_acc, A.lg_global, A.advance, {}};
  // (a split launch is two kernels: the start event belongs to the first, the stop event to the second)
  auto launch = [&](auto go) {
    go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.q), lo32(A.k_new), lo32(A.v_new), hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.q),
       hi16s(A.k_new, A.v_new), flags, (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, (uint32_t)A.slot_stride_b, (uint32_t)(A.head_stride_b / 16),
       A.scale_log2, T);
  };
  if (ev_start && ev_stop)
    launch([&](auto... args) {
      hipExtLaunchKernelGGL((k_attend_gqa<D, NW, SPLIT, R>), grid, dim3(NW * kWave), (uint32_t)lds, st, ev_start, SPLIT ? nullptr : ev_stop, 0, args...);
    });
  else
    launch([&](auto... args) { hipLaunchKernelGGL((k_attend_gqa<D, NW, SPLIT, R>), grid, dim3(NW * kWave), lds, st, args...); });
  if constexpr (SPLIT) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 fgrid(A.accumulate ? (A.sel_cap + kFinishTokens - 1) / kFinishTokens : 1, A.n_heads, n_seq);
    const uint32_t fflags = A.n_heads | A.G << 9 | (A.accumulate ? 0x10000 : 0) | (uint32_t)A.advance << 18 | n_chunks << 24;
    auto finish = [&](auto go) {
      go(lo32(A.seqs), lo32(A.sel_idx), lo32(A.sel_cnt), lo32(A.out), lo32(A.lse), lo32(A.logits), lo32(A.part_ml), lo32(A.part_acc),
         hi16s(A.seqs, A.sel_idx), hi16s(A.sel_cnt, A.out), hi16s(A.lse, A.logits), hi16s(A.part_ml, A.part_acc),
         (uint32_t)A.cap | (uint32_t)A.sel_cap << 16, fflags);
    };
    if (ev_start && ev_stop)
      finish([&](auto... args) { hipExtLaunchKernelGGL((k_gqa_finish<D>), fgrid, dim3(kFinishThreads), 0, st, nullptr, ev_stop, 0, args...); });
    else
      finish([&](auto... args) { hipLaunchKernelGGL((k_gqa_finish<D>), fgrid, dim3(kFinishThreads), 0, st, args...); });
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_gqa_d(const GqaArgs& A, const AttendPlan& plan, int n_seq, size_t lds, hipStream_t st, hipEvent_t e0,
                        hipEvent_t e1) {
  if (plan.n_chunks > 1) return launch_gqa_w<D, 4, true, ring(D)>(A, n_seq, plan.n_chunks, lds, st, e0, e1);     // split lists: 4 waves
  if (plan.waves == 8) return launch_gqa_w<D, 8, false, ring(D)>(A, n_seq, 1, lds, st, e0, e1);
  if (!gqa_two_fit(lds)) return launch_gqa_w<D, 4, false, deep_ring(D)>(A, n_seq, 1, lds, st, e0, e1);
  return launch_gqa_w<D, 4, false, ring(D)>(A, n_seq, 1, lds, st, e0, e1);
}

}  // namespace

// Dynamic LDS above the default 64 KB per-launch limit has to be allowed per kernel, once per device; that is done
// here, at the library's first use of a device, not next to a launch (where it would also sit inside a captured graph).
hipError_t gqa_prepare_kernels() {
  const int lim = (int)kGqaMaxLds;
  const void* kernels[] = {
      reinterpret_cast<const void*>(&k_attend_gqa<64, 4, false, ring(64)>), reinterpret_cast<const void*>(&k_attend_gqa<64, 8, false, ring(64)>),
      reinterpret_cast<const void*>(&k_attend_gqa<128, 4, false, ring(128)>), reinterpret_cast<const void*>(&k_attend_gqa<128, 8, false, ring(128)>),
      reinterpret_cast<const void*>(&k_attend_gqa<64, 4, false, deep_ring(64)>), reinterpret_cast<const void*>(&k_attend_gqa<128, 4, false, deep_ring(128)>),
      reinterpret_cast<const void*>(&k_attend_gqa<64, 4, true, ring(64)>), reinterpret_cast<const void*>(&k_attend_gqa<128, 4, true, ring(128)>)};
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lim);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}


// row stride of the logits one workgroup keeps in LDS: the tokens of its chunk (whole tiles) + one tile of slack
int gqa_logit_stride(const adsa_params& p, int n_chunks) {
  const int tiles = (p.sel_cap + 15) / 16;
  return ((tiles + n_chunks - 1) / n_chunks) * 16 + 16;
}
// row stride of the logits in the workspace (split launches)
int gqa_global_logit_stride(const adsa_params& p) { return (p.sel_cap + 15) / 16 * 16 + 16; }

// LDS each wave owns: a staged K tile [16][D*2+16 bytes], reused for its partial output [G][D] floats
static size_t gqa_stage_bytes(const adsa_params& p) {
  const size_t tile = (size_t)16 * (p.head_dim * 2 + 16), part = (size_t)p.q_per_kv * p.head_dim * sizeof(float);
  return tile > part ? tile : part;
}

size_t gqa_lds_bytes(const adsa_params& p, int waves, int n_chunks) {
  const size_t lgs = (size_t)gqa_logit_stride(p, n_chunks);
  return ((size_t)p.q_per_kv + 1) * lgs * sizeof(float) + (size_t)waves * gqa_stage_bytes(p);
}

hipError_t launch_attend_gqa(const adsa_params& p, const AttendPlan& plan, adsa_seq* seqs, const void* q,
                             const void* k_new, const void* v_new, const int32_t* sel_idx,
                             const int32_t* sel_cnt, void* out, float* lse, char* ws, const Workspace& w,
                             bool accumulate, bool append, int advance, bool new_f32, hipStream_t st,
                             hipEvent_t ev_start, hipEvent_t ev_stop) {
  if (p.dtype != ADSA_BF16 || p.q_per_kv < 2 || p.q_per_kv > 16) return hipErrorInvalidValue;
  if (plan.n_chunks < 1 || plan.n_chunks > kMaxChunks) return hipErrorInvalidValue;
  GqaArgs A;
  A.seqs = seqs; A.q = (const char*)q; A.k_new = (const char*)k_new; A.v_new = (const char*)v_new;
  A.sel_idx = sel_idx; A.sel_cnt = sel_cnt; A.out = (char*)out; A.lse = lse;
  A.logits = reinterpret_cast<float*>(ws + w.logits_off);
  A.part_ml = reinterpret_cast<float*>(ws + w.part_ml_off);
  A.part_acc = reinterpret_cast<float*>(ws + w.part_acc_off);
  A.lg_global = gqa_global_logit_stride(p);
  A.n_heads = p.n_heads; A.G = p.q_per_kv; A.sel_cap = p.sel_cap; A.cap = p.cap;
  A.accumulate = accumulate ? 1 : 0; A.append = append ? 1 : 0; A.advance = advance;
  A.new_f32 = (new_f32 && append) ? 1 : 0;
  A.slot_stride_b = (long long)p.kv_slot_stride * 2;
  A.head_stride_b = (long long)p.kv_head_stride * 2;
  const float scale = p.softmax_scale != 0.0f ? p.softmax_scale : 1.0f / sqrtf((float)p.head_dim);
  A.scale_log2 = scale * kLog2e;
  const size_t lds = gqa_lds_bytes(p, plan.waves, plan.n_chunks);
  if (lds > kGqaMaxLds) return hipErrorInvalidValue;
  if (p.head_dim == 64) return launch_gqa_d<64>(A, plan, p.n_seq, lds, st, ev_start, ev_stop);
  if (p.head_dim == 128) return launch_gqa_d<128>(A, plan, p.n_seq, lds, st, ev_start, ev_stop);
  return hipErrorInvalidValue;
}

}  // namespace adsa
