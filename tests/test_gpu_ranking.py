"""The ranking kernels at the edges of their workgroup shapes, on scores that take every way through the threshold search: one
value, ties that outnumber a wave, consecutive floats, all exponents with infinities, and a long tail beside a dense cluster."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd import workloads as WL
from paper_2506_18226_amd.batch import LayerBatch

from common import oracle_cfg, plan_of
from test_gpu_parity import DEV, load_state, params_for

pytestmark = pytest.mark.gpu


def score_patterns(rng, n):
    ulps = (np.float32(1.5).view(np.uint32) + rng.permutation(n).astype(np.uint32)).view(np.float32)
    wide = np.ldexp(rng.standard_normal(n), rng.integers(-140, 120, n)).astype(np.float32)
    wide[rng.random(n) < 0.02] = np.inf
    wide[rng.random(n) < 0.02] = -np.inf
    wide[rng.random(n) < 0.05] = -0.0
    cluster = np.where(rng.random(n) < 0.9, 1.0 + rng.integers(0, 5, n) * 2.0 ** -23, rng.random(n) * 1e6).astype(np.float32)
    return [np.zeros(n, np.float32), rng.integers(0, 3, n).astype(np.float32), ulps, wide, cluster,
            rng.gamma(2.0, 0.5, n).astype(np.float32)]


@pytest.mark.parametrize("cap", [65, 255, 256, 257, 512, 513, 768, 769, 1024, 1025, 2048, 2049, 4096, 4097, 8192])
def test_ranking_at_workgroup_edges(cap):
    """select and the row-end eviction given the same scores: lists, keep maps, moved pos / score / K / V bit-exact."""
    rng = np.random.default_rng(cap)
    W, P = 16, cap % 16 + 16
    s = cap - P                                              # every grid row so far is resident, the last one just closed
    wl = WL.get_workload("tiny", n_heads=1, head_dim=64, grid_h=s // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    k, v = (rng.standard_normal((cap, 1, 64), dtype=np.float32) for _ in range(2))
    pos = np.arange(cap, dtype=np.int32)
    cases = [(sc, Bud) for sc in score_patterns(rng, cap) for Bud in (1, s // 3, s - 2 * W - 1)]
    params = params_for(wl, len(cases), cap, score_mode=B.SCORE_EXT_LARGEST)
    batch = LayerBatch(params, DEV)
    states = []
    for b, (sc, Bud) in enumerate(cases):
        cfg = oracle_cfg(wl, P=P, budget=Bud, score_mode=B.SCORE_EXT_LARGEST, cap=cap)
        states.append((cfg, oracle.CacheState.from_arrays(cfg, k, v, pos, sc)))
        load_state(batch, b, states[b][1], cfg, s)
    batch.upload_seqs()
    batch.select()
    batch.compact()
    torch.cuda.synchronize()
    seqs, km, Kd, Vd = batch.read_seqs(), batch.keep_map.cpu().numpy(), batch.k_host(), batch.v_host()
    sel, cnt, posd, scored = (x.cpu().numpy() for x in (batch.sel_idx, batch.sel_cnt, batch.pos, batch.score))
    assert (seqs["status"] == 0).all()
    for b, (cfg, st) in enumerate(states):
        ref, _ = oracle.select(cfg, st.pos[:cap], st.score[:cap], None, s)
        assert cnt[b] == ref.size and np.array_equal(sel[b, :ref.size], ref), b
        ref_map, did = oracle.compact(cfg, st, s)
        n = st.n_res
        assert did and seqs["compacted"][b] == 1 and seqs["n_res"][b] == n, b
        assert np.array_equal(km[b], ref_map), b
        assert np.array_equal(posd[b, :n], st.pos[:n]) and np.array_equal(scored[b, 0, :n], st.score[:n]), b
        assert np.array_equal(Kd[b, :n], st.K[:n]) and np.array_equal(Vd[b, :n], st.V[:n]), b


def test_empty_sequences_touch_no_memory():
    """A record that was never filled (all zero: step 0, no resident slot, null pointers) is ranked without a read."""
    wl = WL.get_workload("tiny", n_heads=2, grid_h=4, grid_w=4, prefix_len=4)
    batch = LayerBatch(params_for(wl, 3, 20), DEV)           # upload_seqs() not called: the device records are zero
    batch.select()
    batch.compact()
    torch.cuda.synchronize()
    assert (batch.sel_cnt.cpu().numpy() == 0).all()


@pytest.mark.parametrize("n_seq,h,D,dtype,cap,layout", [
    (1, 1, 64, "bf16", 70, "head_major"), (3, 4, 64, "f32", 257, "slot_major"), (2, 3, 128, "bf16", 513, "head_major"),
    (2, 2, 128, "f32", 800, "slot_major"), (1, 5, 64, "bf16", 1025, "head_major"), (16, 32, 64, "bf16", 90, "head_major"),
    (17, 32, 64, "bf16", 90, "head_major"), (1, 2, 64, "bf16", 2049, "head_major")])
def test_a_step_evicts_as_select_attend_and_compact_do(n_seq, h, D, dtype, cap, layout, score_mode=None):
    """adsa_step, whose eviction has four forms by the size of the step, against the split-phase calls on a copy of the same state: the
    sequences close a row, stand inside one, are inactive, rejected or empty; everything either of them writes is the same."""
    W, P, R = 10, 7, 1
    H = (cap - P) // W + 3
    rng = np.random.default_rng(cap)
    wl = WL.get_workload("tiny", n_heads=h, head_dim=D, grid_h=H, grid_w=W, prefix_len=P, win_rows_back=R, win_col_radius=2, dtype=dtype)
    batches = [LayerBatch(params_for(wl, n_seq, cap, score_mode=score_mode, layout=layout), DEV) for _ in range(2)]
    rows = ((cap - P) // W - 1) * W                          # whole rows that fit
    for b in range(n_seq):
        s = rows if b % 4 != 1 else rows - 3                 # this step's query token closes the row, or does not
        n = P + s - 1
        k, v = (WL.quantise(wl, rng.standard_normal((n, h, D), dtype=np.float32)) for _ in range(2))
        score = rng.random((h, n)).astype(np.float32)
        for batch in batches:
            batch.set_sequence(b, k=k, v=v, pos=np.arange(n, dtype=np.int32), score=score[:B.score_rows(batch.params)], step=s, grid_origin=P,
                               budget=(5, s, s // 2, s - 3 * W)[b % 4])
            if b == 5:
                batch.seqs_host[b]["step"] = -1              # inactive
            if b == 6:
                batch.seqs_host[b]["status"] = 2             # rejected earlier
            if b == 7:
                batch.seqs_host[b]["n_res"], batch.seqs_host[b]["step"] = 0, 0
    one, two = batches
    # above 2048 slots adsa_step's eviction is the same two launches as adsa_compact's; above 1024 workgroups the attention plans it; up to 1024
    # slots, for whole lists and where the workspace has room for the scores it is k_step_finish; k_compact_step otherwise
    plan = plan_of(one.params)
    own = score_mode is None and n_seq <= 3 and cap <= 1024 and plan.chunks == 1
    assert plan.eviction == (0 if cap > 2048 else 3 if n_seq > 16 else 2 if own else 1)
    for batch in batches:
        batch.seqs_host["compacted"] = 1
        batch.upload_seqs()
    q, kn, vn = (torch.from_numpy(rng.standard_normal((n_seq, h, D), dtype=np.float32)).to(DEV).to(one.tdtype) for _ in range(3))
    one.step(q, kn, vn)
    two.select(B.FLAG_PLAN_APPEND)
    two.attend(q, B.FLAG_APPEND, kn, vn)
    two.compact(B.FLAG_ADVANCE)
    torch.cuda.synchronize()
    for name in ("K", "V", "pos", "score", "out", "lse", "sel_idx", "sel_cnt", "keep_map"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    a, b = one.read_seqs(), two.read_seqs()
    for f in ("n_res", "step", "status", "compacted", "pending_slot", "hole"):
        assert np.array_equal(a[f], b[f]), f
    assert a["compacted"][0] == 1 and a["step"][0] == rows + 1


@pytest.mark.parametrize("rows", [1, 9, 26])
def test_many_sequences_rank_like_few(rows):
    """From 1024 sequences on the ranking keeps fewer score rows in flight: same lists and keep maps as for a small batch."""
    cap, P, W, few = 600, 8, 16, 3
    s = cap - P                                              # 37 whole rows
    wl = WL.get_workload("xl", n_heads=rows, head_dim=64, grid_h=s // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    g = torch.Generator().manual_seed(rows)
    score = torch.randint(0, 40, (few, rows, cap), generator=g).float() / 8
    got = []
    for n_seq in (few, 1030):
        batch = LayerBatch(params_for(wl, n_seq, cap, score_mode=B.SCORE_ATTN_MASS), DEV)
        batch.pos.copy_(torch.arange(cap, dtype=torch.int32).expand(n_seq, cap))
        batch.score.copy_(score[torch.arange(n_seq) % few])
        h = batch.seqs_host
        h["n_res"], h["step"], h["grid_origin"], h["n_keep_prefix"] = cap, s, P, P
        h["budget"] = 100 + 150 * (np.arange(n_seq) % few)
        batch.upload_seqs()
        batch.select()
        batch.compact()
        torch.cuda.synchronize()
        n_res = batch.read_seqs()["n_res"]
        got.append((batch.sel_idx.cpu(), batch.sel_cnt.cpu(), batch.keep_map.cpu(), torch.from_numpy(n_res.copy()), batch.score.cpu()))
    at = torch.arange(1030) % few
    for a, b in zip(*got):
        assert torch.equal(a[at], b)
    assert len(set(got[0][1].tolist())) == few


@pytest.mark.parametrize("cap", [3072, 3073, 6144, 6145])
def test_ranking_at_the_edges_of_the_wide_shapes(cap):
    test_ranking_at_workgroup_edges(cap)


@pytest.mark.parametrize("cap", [127, 128, 129])             # (256 and 257: above)
def test_rows_move_at_the_edges_of_the_tile_sizes(cap):
    test_ranking_at_workgroup_edges(cap)


@pytest.mark.parametrize("cap", [2049, 3073, 4096, 4097, 6144, 6145, 8192])
def test_more_sequences_than_compute_units_rank_like_few(cap):
    """Above 2048 slots launches of more than 256 sequences use smaller workgroups: same lists and keep maps as for a small batch."""
    rng = np.random.default_rng(cap)
    W, P = 16, cap % 16 + 16
    s = cap - P
    wl = WL.get_workload("tiny", n_heads=1, head_dim=64, grid_h=s // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    patterns = score_patterns(rng, cap)
    few = len(patterns)
    got = []
    for n_seq in (few, 259):
        batch = LayerBatch(params_for(wl, n_seq, cap, score_mode=B.SCORE_EXT_LARGEST), DEV)
        at = torch.arange(n_seq) % few
        batch.pos.copy_(torch.arange(cap, dtype=torch.int32).expand(n_seq, cap))
        batch.score.copy_(torch.from_numpy(np.stack(patterns))[at][:, None])
        h = batch.seqs_host
        h["n_res"], h["step"], h["grid_origin"], h["n_keep_prefix"] = cap, s, P, P
        h["budget"] = s // 3 + at.numpy()
        batch.upload_seqs()
        batch.select()
        batch.compact()
        torch.cuda.synchronize()
        n_res = torch.from_numpy(batch.read_seqs()["n_res"].copy())
        got.append([x.cpu() for x in (batch.sel_idx, batch.sel_cnt, batch.keep_map, n_res, batch.score, batch.pos)])
    for a, b in zip(*got):
        assert torch.equal(a[at].view(torch.int32), b.view(torch.int32))
    assert (got[0][1] > s // 3).all()


@pytest.mark.parametrize("cap", [256, 512, 768, 1024, 2048])
def test_a_step_evicts_lists_that_fill_its_tile(cap):
    test_a_step_evicts_as_select_attend_and_compact_do(2, 3, 64, "bf16", cap, "head_major")


@pytest.mark.parametrize("cap", [256, 512, 768, 1024])
def test_a_step_of_given_scores_evicts_lists_that_fill_its_tile(cap):
    """Scores of the caller's leave these lists to k_compact_step."""
    test_a_step_evicts_as_select_attend_and_compact_do(2, 3, 64, "bf16", cap, "head_major", B.SCORE_EXT_LARGEST)


@pytest.mark.parametrize("heads", [11, 12, 13])
@pytest.mark.parametrize("cap,D,layout", [(128, 64, "head_major"), (129, 128, "slot_major"), (513, 64, "slot_major"), (770, 128, "head_major"),
                                          (1100, 64, "head_major"), (4200, 64, "head_major")])
def test_score_rows_move_with_the_cache_rows(heads, cap, D, layout):
    """From 12 heads and 129 slots on each head's workgroup of the cache move takes its score row along: every row where the keep map puts it, what
    is beyond the list and sequences with nothing to move untouched (all of the tensors is compared: rows only move down)."""
    P, W, n_seq = 8 + (cap - 8) % 16, 16, 5
    s = cap - P
    wl = WL.get_workload("xl", n_heads=heads, head_dim=D, grid_h=s // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    g = torch.Generator().manual_seed(cap + heads)
    batch = LayerBatch(params_for(wl, n_seq, cap, score_mode=B.SCORE_ATTN_MASS, layout=layout), DEV)
    before = {"score": torch.randint(0, 40, batch.score.shape, generator=g).float() / 8, "pos": torch.arange(cap, dtype=torch.int32).expand(n_seq, cap),
              "K": torch.randn(batch.K.shape, generator=g).to(batch.K.dtype), "V": torch.randn(batch.V.shape, generator=g).to(batch.V.dtype)}
    for name, x in before.items():
        getattr(batch, name).copy_(x)
    h = batch.seqs_host
    h["n_res"], h["step"], h["grid_origin"], h["n_keep_prefix"] = cap, s, P, P
    h["budget"] = [s // 5, s // 2, 0, s, s - 2 * W - 1]
    h["step"][3] = s - 1                                     # no row end
    batch.upload_seqs()
    batch.compact()
    torch.cuda.synchronize()
    seqs, km = batch.read_seqs(), batch.keep_map.cpu()
    slot_axis = 1 if layout == "head_major" else 0           # (of one sequence's [heads][cap][D] or [cap][heads][D])
    for b in range(n_seq):
        n = int(seqs["n_res"][b])
        kept = torch.arange(cap) if b == 3 else (km[b] >= 0).nonzero()[:, 0]
        assert kept.numel() == n and (n < cap) == (b != 3), b
        assert b == 3 or torch.equal(km[b][kept], torch.arange(n, dtype=torch.int32)), b
        for name, axis in (("pos", 0), ("score", 1), ("K", slot_axis), ("V", slot_axis)):
            want, now = before[name][b].clone(), getattr(batch, name)[b].cpu()
            want.narrow(axis, 0, n).copy_(before[name][b].index_select(axis, kept))
            assert torch.equal(now, want), (b, name)


@pytest.mark.parametrize("rows", [11, 12, 26])
@pytest.mark.parametrize("cap", [120, 200, 300, 400, 700, 1500])
def test_many_sequences_move_their_scores_like_few(cap, rows):
    """From 129 sequences on the plan of an eviction moves fewer than 24 score rows itself, and in caches of 257 to 384 slots all of them: as the
    cache move does for a small batch."""
    P, W, few = cap % 16 + 16, 16, 3
    s = cap - P
    wl = WL.get_workload("xl", n_heads=rows, head_dim=64, grid_h=s // W, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=2)
    g = torch.Generator().manual_seed(cap + rows)
    score = torch.randint(0, 40, (few, rows, cap), generator=g).float() / 8
    got = []
    for n_seq in (few, 129):
        batch = LayerBatch(params_for(wl, n_seq, cap, score_mode=B.SCORE_ATTN_MASS), DEV)
        at = torch.arange(n_seq) % few
        batch.pos.copy_(torch.arange(cap, dtype=torch.int32).expand(n_seq, cap))
        batch.score.copy_(score[at])
        h = batch.seqs_host
        h["n_res"], h["step"], h["grid_origin"], h["n_keep_prefix"] = cap, s, P, P
        h["budget"] = [0, s // 3, s - 2 * W - 1] * (n_seq // few)
        batch.upload_seqs()
        batch.compact()
        torch.cuda.synchronize()
        got.append([x.cpu() for x in (batch.keep_map, torch.from_numpy(batch.read_seqs()["n_res"].copy()), batch.score, batch.pos)])
    for a, b in zip(*got):
        assert torch.equal(a[at], b)
    assert len(set(got[0][1].tolist())) == few
