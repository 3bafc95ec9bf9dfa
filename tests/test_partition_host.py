"""The partition header the ranking and V-cosine kernels share, compiled for the CPU: its division-free rows and columns, classes and
budgets against plain integer arithmetic over all the forms it accepts."""
import os
import subprocess

import pytest

from paper_2506_18226_amd import build as B

SOURCE = r"""
#include <cstdio>
#include <cstdint>
#include <cstdlib>
#include <random>
#define __device__
#define __forceinline__ inline
#include "adsa_partition.h"
using namespace adsa;

static int ref_select(long pos, long P, long nkp, long jq, long W, long R, long w, long m) {
  if (pos < nkp) return 0;
  if (pos < P) return 1;
  const long j = pos - P;
  if (j > jq) return -1;
  if (m > 0) return j > jq - m ? 0 : 1;
  const long r = jq / W, col = jq % W, rj = j / W, dc = labs(j % W - col);
  return rj == r || (rj >= r - R && rj < r && dc <= w) ? 0 : 1;
}
static int ref_evict(long pos, long P, long nkp, long jq, long W, long R, long m) {
  if (pos < nkp) return 0;
  if (pos >= P) {
    const long j = pos - P, r = jq / W, rj = j / W;
    if (m > 0) return j > jq + 1 - m ? 0 : 1;
    if (rj >= r - R + 1 && rj <= r) return 0;
  }
  return 1;
}
static long ref_budget(const adsa_seq& q, long s) {
  __int128 b = q.budget;
  if (q.budget_den > 0) b = ((__int128)((long)q.grid_origin + s) * q.budget_num) / q.budget_den;
  return b < 0 ? 0 : b > ADSA_MAX_CAP ? ADSA_MAX_CAP : (long)b;
}

int main() {
  std::mt19937_64 g(5);
  auto r = [&](long lo, long hi) { return lo + (long)(g() % (unsigned long)(hi - lo + 1)); };
  long checked = 0;
  // every column count up to 300 and larger ones, up to the largest grid: around every multiple of W that is tried
  for (long W = 1; W <= 1l << 24; W = W < 300 ? W + 1 : W + r(1, W / 2)) {
    const GridWidth grid{(int)W, 1.0f / (float)W};
    for (int t = 0; t < 4000; ++t) {
      const long k = t < 40 ? (1l << 24) / W - t : r(0, (1l << 24) / W), j0 = k * W;
      for (long j = j0 - 2; j <= j0 + 2; ++j) {
        if (j < 0 || j >= 1l << 24) continue;
        int col;
        if (grid.row((int)j, &col) != j / W || col != j % W) { printf("row W=%ld j=%ld\n", W, j); return 1; }
        ++checked;
      }
    }
  }
  for (int t = 0; t < 400000; ++t) {
    const long W = r(1, t % 3 ? 40 : 300), H = r(1, 60), P = r(0, 50), nkp = t % 5 ? P : r(0, P), s = r(0, H * W), R = r(0, 4) ? r(0, 3) : r(0, 100), w = r(0, 3) ? r(0, W) : 0x7FFFFFFF;
    const long m = r(0, 2) ? 0 : r(1, 2 * W);
    adsa_seq q = {};
    q.grid_origin = (int)P; q.n_keep_prefix = (int)nkp;
    const QueryCell c = make_query_cell(q, (int)s, GridWidth{(int)W, 1.0f / (float)W}, (int)R, (int)w, (int)m);
    if (is_row_end(c, (int)s, (int)(H * W)) != (s >= 1 && s <= H * W && (s - 1) % W == W - 1)) { printf("row end\n"); return 1; }
    for (int i = 0; i < 12; ++i) {
      const long pos = i < 6 ? r(0, P + H * W) : P + s - 1 + r(-2 * W, 3);
      if (pos < 0) continue;
      if (s >= 1 && select_class(c, (int)pos) != ref_select(pos, P, nkp, s - 1, W, R, w, m)) { printf("select pos=%ld s=%ld W=%ld R=%ld w=%ld m=%ld\n", pos, s, W, R, w, m); return 1; }
      if (s >= 1 && m > 0 && select_class_1d(c, (int)pos) != select_class(c, (int)pos)) { printf("1-D class pos=%ld s=%ld m=%ld\n", pos, s, m); return 1; }
      if (s < 1 && pos >= P && select_class(c, (int)pos) != (pos < nkp ? 0 : -1)) { printf("select at s = 0\n"); return 1; }
      if (s >= 1 && evict_class(c, (int)pos) != ref_evict(pos, P, nkp, s - 1, W, R, m)) { printf("evict pos=%ld s=%ld W=%ld R=%ld m=%ld\n", pos, s, W, R, m); return 1; }
      ++checked;
    }
    q.budget = (int)r(-5, 20000);
    q.budget_num = (int)(t % 7 ? r(0, 40) : r(-2147483647l - 1, 2147483647l));
    q.budget_den = (int)(t % 4 == 0 ? r(-2, 0) : t % 7 ? r(1, 40) : r(1, 2147483647l));
    if (t % 11 == 0) { q.budget_num = q.budget_den = 2147483647; }
    if (effective_budget(q, (int)s) != ref_budget(q, s)) { printf("budget P=%ld s=%ld %d/%d: %d, not %ld\n", P, s, q.budget_num, q.budget_den, effective_budget(q, (int)s), ref_budget(q, s)); return 1; }
  }
  for (long den = 1; den <= 300; ++den)                      // exact quotients and their neighbours
    for (long x = 0; x <= 8300; ++x)
      for (int d = -1; d <= 1; ++d) {
        adsa_seq q = {};
        q.grid_origin = (int)(x * den + d); q.budget_num = 1; q.budget_den = (int)den;
        if (effective_budget(q, 0) != ref_budget(q, 0)) { printf("budget %ld/%ld\n", x * den + d, den); return 1; }
      }
  printf("ok %ld\n", checked);
  return 0;
}
"""


@pytest.mark.parametrize("flags", [["-O2"], ["-O0", "-ffp-contract=off"]])
def test_classes_rows_and_budgets(tmp_path, flags):
    src, exe = tmp_path / "partition.cpp", tmp_path / "partition"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", *flags, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout
