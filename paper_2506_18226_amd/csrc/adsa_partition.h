// Device-side statement of the cache partition (Section 4.1, Eq. 1) and of the rows the per-row
// eviction protects (Section 4.2), shared by the ranking and the V-cosine kernels.
#pragma once

#include "adsa.h"

namespace adsa {

// j / W and j mod W for 0 <= j < 2^24 without an integer division (some 25 instructions a slot): inv_w is 1 / W rounded to the
// nearest float, so the product is less than 1 away from the quotient (by 2^-23 of it, at most 0.67 where 1 / W is inexact).
struct GridWidth {
  int W;
  float inv_w;
  __device__ __forceinline__ int row(int j, int* col) const {
    int q = (int)((float)j * inv_w), c = j - q * W;
    if (c < 0) { c += W; --q; }
    if (c >= W) { c -= W; ++q; }
    *col = c;
    return q;
  }
};

// Geometry of one sequence's query for its current decode step s, as ranges of image indices j = pos - P.
struct QueryCell {
  int P;              // grid origin (absolute position of image token 0)
  int n_keep_prefix;  // pinned leading positions
  int jq;             // image index of the query token (s - 1)
  int col, w;         // its column; column radius of the window
  int local_from;     // from here on everything is local: the query's row, or the recent_m most recent tokens (1-D window)
  int above_from;     // from here on local within w columns: the R rows above (2-D window only)
  int keep_from, keep_to;      // what an eviction at this step's row end protects: the last R rows, or the m - 1 most recent tokens (the
                               // next row's first query, jq + 1, reaches back furthest, to j > jq + 1 - m)
  GridWidth grid;
};

// (Seq: adsa_seq, in whatever address space)
template <typename Seq>
__device__ __forceinline__ QueryCell make_query_cell(const Seq& sq, int s, const GridWidth& grid, int R, int w, int recent_m) {
  QueryCell c;
  c.P = sq.grid_origin; c.n_keep_prefix = sq.n_keep_prefix; c.jq = s - 1; c.w = w; c.grid = grid;
  int r = 0;
  c.col = 0;
  if (s >= 1) r = grid.row(c.jq, &c.col);
  if (recent_m > 0) {
    c.local_from = c.jq - recent_m + 1;
    c.above_from = c.keep_to = 0x7FFFFFFF;
    c.keep_from = c.jq + 2 - recent_m;
  } else {
    c.local_from = r * grid.W;
    c.above_from = R >= r ? 0 : (r - R) * grid.W;
    c.keep_from = R > r ? 0 : (r - R + 1) * grid.W;
    c.keep_to = (r + 1) * grid.W - 1;
  }
  return c;
}

// Attention-time partition: 0 = pinned prefix or local window (always attended), 1 = candidate
// ("previous"), -1 = entry newer than the query (malformed state).
__device__ __forceinline__ int select_class(const QueryCell& c, int pos) {
  const int j = pos - c.P;
  int col;
  (void)c.grid.row(j, &col);                         // (of no meaning where j is no image index, and not used there)
  const int d = col - c.col, dc = d < 0 ? -d : d;
  const bool local = j >= c.local_from || (j >= c.above_from && dc <= c.w);
  const int image = j > c.jq ? -1 : local ? 0 : 1;
  return pos < c.n_keep_prefix ? 0 : pos < c.P ? 1 : image;
}

// The same for a cell whose window is the 1-D one, which has no columns.
__device__ __forceinline__ int select_class_1d(const QueryCell& c, int pos) {
  const int j = pos - c.P;
  return pos < c.n_keep_prefix ? 0 : pos < c.P ? 1 : j > c.jq ? -1 : j >= c.local_from ? 0 : 1;
}

// Eviction-time partition at the end of a row: 0 = pinned prefix or a token some window of the next row needs, 1 = competes for
// the budget.
__device__ __forceinline__ int evict_class(const QueryCell& c, int pos) {
  const int j = pos - c.P;
  return pos < c.n_keep_prefix || (pos >= c.P && j >= c.keep_from && j <= c.keep_to) ? 0 : 1;
}

// s: the step the cell was made for; total: image tokens of the grid
__device__ __forceinline__ bool is_row_end(const QueryCell& c, int s, int total) {
  return s >= 1 && s <= total && c.col == c.grid.W - 1;
}

// The fields of a record that a budget follows from.
struct BudgetOf {
  int grid_origin, budget, budget_num, budget_den;
  template <typename Seq>
  __device__ __forceinline__ explicit BudgetOf(const Seq& q) : grid_origin(q.grid_origin), budget(q.budget), budget_num(q.budget_num), budget_den(q.budget_den) {}
};

// Budget of a step: floor((P + s) * num / den) within [0, ADSA_MAX_CAP], or the given number.  (A 64-bit division is some 150
// instructions; a quotient below 8192 is found by a float one to within 1.)
template <typename Seq>
__device__ __forceinline__ int effective_budget(const Seq& q, int s) {
  if (q.budget_den <= 0) return q.budget < 0 ? 0 : q.budget > ADSA_MAX_CAP ? ADSA_MAX_CAP : q.budget;
  const long long x = ((long long)q.grid_origin + s) * q.budget_num, den = q.budget_den;
  if (x <= 0) return 0;
  if (x >= den * ADSA_MAX_CAP) return ADSA_MAX_CAP;
  const int b = (int)((float)x / (float)den);
  return b * den > x ? b - 1 : (b + 1) * den <= x ? b + 1 : b;
}

}  // namespace adsa
