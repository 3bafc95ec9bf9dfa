"""The V-cosine kernels over the row lengths a wave can hold (1 .. 32 pieces of 16 bytes per lane) and around the edges of their
slot tiles: Eq. 3's scores, the eviction they lead to and the running sum u, against the oracle's pairwise definition and
64-bit sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd import workloads as WL
from paper_2506_18226_amd.batch import LayerBatch

from common import oracle_cfg, plan_of
from test_gpu_parity import DEV, LAYOUTS, params_for

pytestmark = pytest.mark.gpu


def rows(wl, rng, n):
    return WL.quantise(wl, rng.standard_normal((n, wl.n_heads, wl.head_dim), dtype=np.float32) + 0.3)


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("h,D,dtype,n_seq,n", [
    (1, 64, "bf16", 2, 65), (9, 64, "bf16", 2, 64), (24, 64, "bf16", 2, 129), (13, 128, "bf16", 2, 63), (41, 64, "bf16", 2, 200),
    (32, 128, "bf16", 1, 257), (33, 128, "bf16", 1, 130), (64, 128, "bf16", 1, 70), (5, 64, "f32", 2, 255), (11, 128, "f32", 1, 100),
    (32, 128, "f32", 1, 66), (64, 128, "f32", 1, 65), (2, 64, "bf16", 300, 300), (3, 64, "f32", 200, 513)])
def test_vcos_scores_over_row_lengths_and_tiles(h, D, dtype, n_seq, n, layout):
    rng = np.random.default_rng(n)
    P, W = 3, 16
    wl = WL.get_workload("tiny", n_heads=h, head_dim=D, grid_h=40, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=1,
                         dtype=dtype, score_mode=WL.SCORE_VCOS)
    s = n - P + 1                                            # the query token itself is not resident yet
    v = rows(wl, rng, n)
    v[n // 2] = 0.0                                          # a zero row counts as similar to nothing
    batch = LayerBatch(params_for(wl, n_seq, n + 1, layout=layout), DEV)
    b_of = [0, n_seq - 1]
    for b in range(n_seq):
        batch.seqs_host[b]["step"] = -1
    for b in set(b_of):
        batch.set_sequence(b, k=v, v=v, pos=np.arange(n, dtype=np.int32), score=None, step=s, grid_origin=P, budget=7)
    batch.upload_seqs()
    batch.select()
    torch.cuda.synchronize()
    assert (batch.read_seqs()["status"] == 0).all()
    cfg = oracle_cfg(wl, budget=7, cap=n + 1)
    cand = np.nonzero(oracle.classify(cfg, np.arange(n, dtype=np.int32), s) == 2)[0].astype(np.int32)
    ref = oracle.vcos(cfg, v, cand)
    for b in set(b_of):
        got = batch.score[b, 0].cpu().numpy()
        assert np.allclose(got[cand], ref, rtol=1e-4, atol=2e-6), b           # fp32 sums of up to 8192 x 513 terms
        others = np.setdiff1d(np.arange(n), cand)
        assert (got[others] == 0).all(), b


@pytest.mark.parametrize("h,D,dtype,cap", [(1, 64, "bf16", 300), (9, 64, "bf16", 1100), (24, 64, "bf16", 632), (13, 128, "bf16", 70),
                                           (41, 64, "bf16", 90), (31, 128, "bf16", 300), (3, 64, "f32", 257), (31, 128, "f32", 80)])
def test_running_sum_starts_and_moves_on(h, D, dtype, cap):
    """ADSA_SCORE_VCOS_FUSED: after a first (cold) eviction u is the sum over the next step's candidates; after a further step
    it has lost the evicted row and gained the row that left the window."""
    rng = np.random.default_rng(cap)
    P, W, m = 5, 40, 6
    wl = WL.get_workload("tiny", n_heads=h, head_dim=D, grid_h=40, grid_w=W, prefix_len=P, dtype=dtype)
    params = B.make_params(n_seq=2, n_heads=h, head_dim=D, grid_h=40, grid_w=W, win_rows_back=0, win_col_radius=0, cap=cap,
                           dtype=B.F32 if dtype == "f32" else B.BF16, score_mode=B.SCORE_VCOS_FUSED, win_recent_m=m,
                           evict_policy=B.EVICT_REUSE_SLOT)
    batch = LayerBatch(params, DEV)
    s = cap - P + 1
    vs = [rows(wl, rng, cap + 2) for _ in range(2)]
    for b in range(2):
        batch.set_sequence(b, k=vs[b][:cap], v=vs[b][:cap], pos=np.arange(cap, dtype=np.int32), score=None, step=s, grid_origin=P)
    batch.upload_seqs()
    alive = [dict(enumerate(vs[b][:cap].astype(np.float64).reshape(cap, -1))) for b in range(2)]     # position -> row
    for t in range(2):
        batch.compact()
        torch.cuda.synchronize()
        seqs, u = batch.read_seqs(), batch.vcos_u.cpu().numpy()
        for b in range(2):
            unit = {p: r / max(np.linalg.norm(r), 1e-8) for p, r in alive[b].items()}
            cand = [p for p in unit if P <= p <= P + s + t - 1 - m]
            total = sum(unit[p] for p in cand)
            S = {p: unit[p] @ total - unit[p] @ unit[p] for p in cand}
            victim = max(S, key=S.get)
            slot = int(seqs["hole"][b]) - 1
            assert batch.pos[b, slot].item() == victim, (t, b)
            del alive[b][victim]
            want = sum(unit[p] for p in unit if p != victim and P <= p <= P + s + t - m)
            assert np.abs(u[b, :h * D] - want).max() <= 2e-5, (t, b)          # fp32 sums of up to 1100 terms of at most 1
            alive[b][cap + t] = vs[b][cap + t].astype(np.float64).reshape(-1)
        new = torch.from_numpy(np.stack([vs[b][cap + t] for b in range(2)])).to(DEV).to(batch.tdtype)
        batch.select(B.FLAG_PLAN_APPEND)
        batch.attend(new, B.FLAG_APPEND | B.FLAG_ADVANCE, new, new)


@pytest.mark.parametrize("h,D,dtype,cap,layout", [(3, 64, "bf16", 700, "head_major"), (24, 64, "bf16", 513, "slot_major"),
                                                  (9, 128, "f32", 330, "head_major"), (2, 64, "f32", 257, "head_major"),
                                                  (5, 64, "bf16", 64, "slot_major")])
def test_scores_do_not_depend_on_the_batch(h, D, dtype, cap, layout):
    """A sequence's Eq. 3 scores are the same bits whether it is ranked alone or in a batch, at its edges or inside: the launch
    is cut differently for few, some and many sequences, the sums are not."""
    rng = np.random.default_rng(cap)
    P, W = 3, 16
    wl = WL.get_workload("tiny", n_heads=h, head_dim=D, grid_h=50, grid_w=W, prefix_len=P, win_rows_back=1, win_col_radius=1,
                         dtype=dtype, score_mode=WL.SCORE_VCOS)
    lens = [cap - 1, cap // 2 + 1, cap - 40]
    vs = [rows(wl, rng, n) for n in lens]
    groups = (cap + 255) // 256
    got, ways = [], set()
    for n_seq in (3, 500 // groups, 600 // groups, 700 // groups):
        batch = LayerBatch(params_for(wl, n_seq, cap, layout=layout), DEV)
        plan = plan_of(batch.params)
        ways.add((plan.vcos_split, plan.vcos_tile))
        batch.seqs_host["step"] = -1
        at = [0, n_seq // 2, n_seq - 1]
        for b, n, v in zip(at, lens, vs):
            batch.set_sequence(b, k=v, v=v, pos=np.arange(n, dtype=np.int32), score=None, step=n - P + 1, grid_origin=P, budget=7)
        batch.upload_seqs()
        batch.select()
        torch.cuda.synchronize()
        got.append(batch.score[at, 0].cpu())
        assert all(torch.count_nonzero(x) > 1 for x in got[-1])
    assert all(torch.equal(got[0], x) for x in got[1:])
    assert {(1, 64), (0, 256)} < ways and (cap == 64 or any(tile == 128 for _, tile in ways))      # every way was taken
