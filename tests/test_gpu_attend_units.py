"""The attention kernel's units: list lengths around a wave-load, a pair of them, a ring revolution and the entries fetched
early; the query token's slot at every kind of place in the list; rows that are not attended hold NaN, so that no lane without a
token may let what it read reach a result, in every form of the kernel (whole and split lists, one head and several, with the fused
V-cosine rows, 32- and 64-bit offsets).  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd import workloads as WL
from paper_2506_18226_amd.batch import to_device

from common import oracle_cfg, plan_of
from test_gpu_parity import DEV, check_out, lse_tol

pytestmark = pytest.mark.gpu


def run_case(n_heads, D, dtype, layout, cap, lens, slot_stride=None, new_f32=False, fused=False):
    """One attention launch over len(lens) sequences whose caches hold NaN wherever nothing may be read from.  slot_stride
    (elements): the caches lie inside one another, K and V of all sequences between two slots."""
    n_seq, sel_cap = len(lens), max(lens)
    wl = WL.get_workload("tiny", n_heads=n_heads, head_dim=D, grid_h=96, grid_w=96, prefix_len=8, dtype=dtype)
    rng = np.random.default_rng(11)
    k, v = (WL.quantise(wl, rng.standard_normal((cap, n_heads, D), dtype=np.float32)) for _ in range(2))
    q = WL.quantise(wl, rng.standard_normal((n_seq, n_heads, D), dtype=np.float32))
    kn, vn = (rng.standard_normal((n_seq, n_heads, D), dtype=np.float32) for _ in range(2))
    kq, vq = WL.quantise(wl, kn), WL.quantise(wl, vn)
    code, tdt = (B.F32, torch.float32) if dtype == "f32" else (B.BF16, torch.bfloat16)
    p = B.make_params(n_seq=n_seq, n_heads=n_heads, head_dim=D, grid_h=96, grid_w=96, win_rows_back=1, win_col_radius=2, dtype=code,
                      score_mode=B.SCORE_VCOS_FUSED if fused else B.SCORE_ATTN_MASS, evict_policy=B.EVICT_REUSE_SLOT if fused else 0,
                      win_recent_m=4 if fused else 0, cap=cap, sel_cap=sel_cap, layout=layout, kv_slot_stride=slot_stride,
                      kv_head_stride=cap * slot_stride if slot_stride and layout == "head_major" else None)
    span, row = (cap - 1) * p.kv_slot_stride + (n_heads - 1) * p.kv_head_stride + D, n_heads * D
    if slot_stride:
        pool = torch.full((span + 2 * n_seq * row,), float("nan"), dtype=tdt, device=DEV)
        K, V = ([pool[(2 * b + j) * row:] for b in range(n_seq)] for j in range(2))
    else:
        K, V = (torch.full((n_seq, span), float("nan"), dtype=tdt, device=DEV) for _ in range(2))
    view = lambda x, b: torch.as_strided(x[b], (cap, n_heads, D), (p.kv_slot_stride, p.kv_head_stride, 1), x[b].storage_offset())
    score = rng.random((n_seq, B.score_rows(p), cap)).astype(np.float32)
    score_d = torch.from_numpy(score).to(DEV)
    u = rng.standard_normal((n_seq, row + 4)).astype(np.float32)
    u[:, row:] = [602.0, 0.0, 0.0, 0.0]                          # u belongs to the next step
    u_d = torch.from_numpy(u).to(DEV)
    pos = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(n_seq, 1)
    seqs = np.zeros(n_seq, dtype=B.SEQ_DTYPE)
    sels, news = [], []
    sel_idx = torch.full((n_seq, sel_cap), cap + 7, dtype=torch.int32, device=DEV)      # (past a list: nothing that may be used)
    for b, n in enumerate(lens):
        pool_b = np.arange(1, cap) if n < cap and b % 2 else np.arange(cap)             # every other list leaves slot 0 out
        sel = np.sort(rng.choice(pool_b, size=n, replace=False)).astype(np.int32)
        outside = np.setdiff1d(np.arange(cap), sel)
        # the query token's slot: first, middle, last of the list; outside it (its row is stored all the same); none
        new = [int(sel[0]), int(sel[n // 2]), int(sel[-1]), int(outside[-1]) if len(outside) else -1, -1][b % 5]
        rows = torch.from_numpy(sel[sel != new].astype(np.int64)).to(DEV)
        for x, host in ((K, k), (V, v)):
            view(x, b)[rows] = to_device(host[sel[sel != new]], code, DEV)
        sel_idx[b, :n] = torch.from_numpy(sel).to(DEV)
        seqs[b]["k"], seqs[b]["v"] = K[b].data_ptr(), V[b].data_ptr()
        seqs[b]["pos"], seqs[b]["score"] = pos[b].data_ptr(), score_d[b].data_ptr()
        seqs[b]["vcos_u"] = u_d[b].data_ptr() if fused else 0
        seqs[b]["n_res"], seqs[b]["step"], seqs[b]["pending_slot"] = cap, 600, new
        sels.append(sel)
        news.append(new)
    seqs_d = torch.from_numpy(seqs.view(np.uint8).reshape(-1).copy()).to(DEV)
    cnt = torch.tensor(lens, dtype=torch.int32, device=DEV)
    out = torch.zeros((n_seq, n_heads, D), dtype=tdt, device=DEV)
    lse = torch.zeros((n_seq, n_heads), device=DEV)
    ws = torch.full((B.adsa_workspace_bytes(p),), 0xFF, dtype=torch.uint8, device=DEV)  # (NaN in every float)
    new_rows = [torch.from_numpy(x).to(DEV) if new_f32 else to_device(x, code, DEV) for x in ((kn, vn) if new_f32 else (kq, vq))]
    B.adsa_attend(p, seqs_d, to_device(q, code, DEV), sel_idx, cnt, out, lse, ws,
                  B.FLAG_APPEND | B.FLAG_ADVANCE | (B.FLAG_NEW_F32 if new_f32 else 0), *new_rows)
    torch.cuda.synchronize()
    out, lse, got = out.float().cpu().numpy(), lse.cpu().numpy(), score_d.cpu().numpy()
    steps = seqs_d.cpu().numpy().view(B.SEQ_DTYPE)["step"]
    cfg = oracle_cfg(wl, budget=cap, cap=cap)
    for b, n in enumerate(lens):
        kb, vb, new, what = k.copy(), v.copy(), news[b], f"len={n} b={b}"
        if new >= 0:
            kb[new], vb[new] = kq[b], vq[b]
            for x, new_row in ((K, kq), (V, vq)):
                assert np.array_equal(view(x, b)[new].float().cpu().numpy(), new_row[b]), what
        ro, rl, probs = oracle.attend(cfg, kb, vb, q[b], sels[b], want_probs=True)
        check_out(wl, out[b], ro, what)
        assert np.abs(lse[b] - rl).max() <= lse_tol(wl), what
        want, tol = score[b].copy(), dict(rtol=1e-5, atol=1e-6)
        if fused:                                               # |v|^2 and v.u: fp32 sums of D products, a few 1e-7 of their terms
            vs = vb[sels[b]].astype(np.float64)
            want[0::2, sels[b]] = (vs ** 2).sum(-1).T
            want[1::2, sels[b]] = (vs * u[b, :row].reshape(n_heads, D)).sum(-1).T
            tol["atol"] = 1e-4
            assert u_d[b, row + 1] == 602.0                     # the rows are the next step's
        else:
            want[:, sels[b]] += np.asarray(probs, dtype=np.float32).reshape(n_heads, n)
        assert np.allclose(got[b], want, **tol), what
        assert steps[b] == 601
    return p


@pytest.mark.parametrize("n_heads,D,dtype,layout,cap,lens,waves", [
    # waves per workgroup, tokens of a wave-load -> tokens of a revolution: 8 x 8 x 4 = 256
    (3, 64, "bf16", "head_major", 700, [1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 512, 513, 700], 8),
    (2, 128, "bf16", "slot_major", 300, [1, 3, 4, 5, 8, 127, 128, 129, 256, 257, 300], 8),
    (3, 64, "bf16", "slot_major", 128, [1, 7, 8, 9, 31, 32, 33, 64, 96, 127, 128], 4),
    (2, 64, "f32", "head_major", 400, [1, 3, 4, 5, 127, 128, 129, 384, 385, 400], 8),
    (2, 128, "f32", "head_major", 200, [1, 2, 3, 4, 63, 64, 65, 128, 199, 200], 8),
    (2, 128, "f32", "slot_major", 32, [1, 2, 3, 16, 31, 32], 4),
    # entries beyond those fetched early (4 per thread), with 8 waves and with 4
    (9, 64, "bf16", "head_major", 2200, [2047, 2048, 2049, 2200, 1, 2047, 2048, 2049, 2200, 1030, 1024, 5], 8),
    (24, 64, "bf16", "head_major", 1100, [1023, 1024, 1025, 1100, 1, 8] + [16 * i + 3 for i in range(20)], 4),
])
def test_lengths_around_the_units(n_heads, D, dtype, layout, cap, lens, waves):
    p = run_case(n_heads, D, dtype, layout, cap, lens)
    plan = plan_of(p)
    assert (plan.waves, plan.chunks, plan.heads) == (waves, 1, 1)


@pytest.mark.parametrize("D,lens", [(64, [1, 40, 41, 300, 399, 400]), (128, [2, 100, 255, 256, 257])])
def test_fp32_rows_enter_through_the_wave_that_attends_them(D, lens):
    run_case(2, D, "bf16", "head_major", 400, lens, new_f32=True)


def few(n):                                                      # lists of a launch of many short ones
    return [1 + 7 * i % n for i in range(23)] + [n]


@pytest.mark.parametrize("n_heads,D,dtype,layout,cap,lens,fused,plan", [       # plan: chunks, waves, heads per workgroup
    (2, 128, "f32", "head_major", 1100, [1, 15, 16, 17, 1099, 1100], False, (16, 8, 1)),
    (5, 128, "bf16", "slot_major", 1500, [1, 5, 6, 7, 1024, 1025, 1499, 1500], False, (6, 8, 1)),
    (64, 64, "bf16", "slot_major", 80, few(77), False, (1, 4, 4)),
    (64, 128, "bf16", "slot_major", 80, few(60)[12:], False, (1, 4, 2)),
    (65, 64, "f32", "slot_major", 70, few(60)[11:], False, (1, 4, 2)),          # (the last workgroup has one head)
    (3, 64, "bf16", "head_major", 300, [1, 7, 8, 9, 255, 256, 257, 300], True, (1, 8, 1)),
    (3, 128, "f32", "head_major", 32, [1, 2, 3, 31, 32], True, (1, 4, 1)),
    (2, 128, "bf16", "head_major", 500, [1, 4, 5, 6, 499, 500], True, (4, 8, 1)),
])
def test_every_form_with_rows_that_may_not_be_used(n_heads, D, dtype, layout, cap, lens, fused, plan):
    got = plan_of(run_case(n_heads, D, dtype, layout, cap, lens, fused=fused))
    assert (got.chunks, got.waves, got.heads, got.wide) == (*plan, 0)


@pytest.mark.parametrize("n_heads,D,dtype,layout,cap,lens,fused,plan", [
    (2, 64, "bf16", "slot_major", 24, [1, 9, 24], False, (1, 4, 1)),
    (2, 128, "f32", "slot_major", 20, [3, 20], False, (1, 4, 1)),
    (2, 128, "bf16", "slot_major", 300, [300, 1, 299], False, (1, 8, 1)),       # 15 MB apart, over more than 4 GB
    (3, 128, "f32", "slot_major", 400, [1, 5, 6, 7, 399, 400], False, (7, 8, 1)),
    (64, 64, "bf16", "slot_major", 300, few(77), False, (1, 4, 4)),
    (64, 128, "bf16", "slot_major", 280, few(60)[12:], False, (1, 4, 2)),
    (64, 64, "f32", "slot_major", 280, few(60)[12:], False, (1, 4, 2)),
    (1, 64, "bf16", "head_major", 300, [1, 8, 256, 257, 299, 300], True, (1, 8, 1)),
    (2, 64, "f32", "head_major", 40, [1, 4, 39, 40], True, (1, 4, 1)),
    (1, 128, "f32", "head_major", 300, [1, 4, 5, 6, 299, 300], True, (5, 8, 1)),
])
def test_slots_further_apart_than_24_bit_products_reach(n_heads, D, dtype, layout, cap, lens, fused, plan):
    """Rows of a token of a larger structure: 16 MB apart, or a little less over more than 4 GB."""
    stride = (15 << 20) if cap >= 300 else (16 << 20) + 4096
    got = plan_of(run_case(n_heads, D, dtype, layout, cap, lens, slot_stride=stride // (4 if dtype == "f32" else 2), fused=fused))
    assert (got.chunks, got.waves, got.heads, got.wide) == (*plan, 1)
    torch.cuda.empty_cache()
