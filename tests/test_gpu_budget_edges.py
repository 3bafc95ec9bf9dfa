"""Selection where the budget covers every position that can be a candidate (the scores are then not read), one below it, at the
number of candidates and one below that; with pinned and unpinned prefixes, both windows, fractional budgets, and positions that are
not distinct, where more entries than positions compete after all.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd import workloads as WL
from paper_2506_18226_amd.batch import LayerBatch

from common import oracle_cfg
from test_gpu_parity import DEV, load_state, params_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,s", [(200, 130), (700, 600), (1500, 1333), (5000, 4321)])
@pytest.mark.parametrize("pinned,recent_m", [(True, 0), (False, 0), (True, 9)])
def test_budgets_around_the_number_of_candidates(cap, s, pinned, recent_m):
    rng = np.random.default_rng(cap + recent_m)
    W, P = 16, cap - s - 20
    nkp = P if pinned else P // 2
    wl = WL.get_workload("tiny", n_heads=1, head_dim=64, grid_h=(s + W - 1) // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    n = P + s - 7
    pos = np.sort(rng.choice(P + s, size=n, replace=False)).astype(np.int32)
    twice = pos.copy()                                          # positions of which some are there twice
    twice[1::5] = twice[0::5][: len(twice[1::5])]
    k, v = (rng.standard_normal((n, 1, 64), dtype=np.float32) for _ in range(2))
    score = rng.integers(0, 50, n).astype(np.float32)
    reach = P + s - 1 - nkp                                     # positions that can be candidates
    budgets = [0, 1, s // 2, reach - 1, reach, reach + 1, n - 1, n, 8192]
    # the exact number of candidates, from the oracle's own partition
    cfg0 = oracle_cfg(wl, P=P, budget=8192, score_mode=B.SCORE_EXT_LARGEST, cap=cap, n_keep_prefix=nkp)
    cfg0.win_recent_m = recent_m
    kept = oracle.select(cfg0, pos, score, None, s)[0].size
    cfg1 = oracle_cfg(wl, P=P, budget=0, score_mode=B.SCORE_EXT_LARGEST, cap=cap, n_keep_prefix=nkp)
    cfg1.win_recent_m = recent_m
    cand = kept - oracle.select(cfg1, pos, score, None, s)[0].size
    budgets += [cand - 1, cand, cand + 1]
    cases = [(p, Bud) for p in (pos, twice) for Bud in budgets]
    params = params_for(wl, len(cases), cap, score_mode=B.SCORE_EXT_LARGEST)
    params.win_recent_m = recent_m
    batch = LayerBatch(params, DEV)
    states = []
    for b, (p, Bud) in enumerate(cases):
        cfg = oracle_cfg(wl, P=P, budget=Bud, score_mode=B.SCORE_EXT_LARGEST, cap=cap, n_keep_prefix=nkp)
        cfg.win_recent_m = recent_m
        states.append((cfg, oracle.CacheState.from_arrays(cfg, k, v, p, score)))
        load_state(batch, b, states[b][1], cfg, s)
        batch.seqs_host[b]["n_keep_prefix"] = nkp
        if Bud and b % 3 == 0:                                  # the same number as a fraction of P + s
            batch.seqs_host[b]["budget_num"], batch.seqs_host[b]["budget_den"] = Bud, P + s
    batch.upload_seqs()
    batch.select()
    torch.cuda.synchronize()
    sel, cnt = batch.sel_idx.cpu().numpy(), batch.sel_cnt.cpu().numpy()
    assert (batch.read_seqs()["status"] == 0).all()
    for b, (cfg, st) in enumerate(states):
        ref, _ = oracle.select(cfg, st.pos[:n], st.score[:n], None, s)
        assert cnt[b] == ref.size and np.array_equal(sel[b, :ref.size], ref), (b, cases[b][1])
