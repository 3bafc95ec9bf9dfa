"""Attention over lists that are cut into chunks (few (sequence, head) pairs with long lists): list lengths around the
number of chunks and around the token slices of the merging kernel, the query token's row entering the cache inside the last
chunk, the step advancing once, and the fused V-cosine rows; against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd import workloads as WL
from paper_2506_18226_amd.batch import LayerBatch, to_device, to_host

from common import oracle_cfg, plan_of, rank_host
from test_gpu_parity import DEV, check_out, lse_tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_heads,D,dtype,layout,fused,lens,chunks", [
    (2, 128, "f32", "head_major", False, [1, 2, 15, 16, 17, 1023, 1024, 1100], 16),
    (2, 64, "bf16", "slot_major", False, [3, 16, 33, 1025, 2048, 2049, 4100, 4200], 16),
    (5, 128, "bf16", "slot_major", False, [1, 5, 6, 7, 511, 1024, 1025, 1500], 6),
    (6, 128, "bf16", "slot_major", False, [1, 6, 7, 8, 1025, 1500], 7),
    (2, 128, "f32", "head_major", True, [1, 15, 16, 17, 1023, 1024, 1099, 1100], 16),    # |v|^2 and v.u rows of every chunk
    (2, 128, "bf16", "head_major", True, [1, 4, 5, 6, 255, 256, 499, 500], 4),           # the fused form's earlier line
])
def test_split_lists_and_their_merge(n_heads, D, dtype, layout, fused, lens, chunks):
    n_tok, n_seq = max(lens), len(lens)
    wl = WL.get_workload("tiny", n_heads=n_heads, head_dim=D, grid_h=72, grid_w=72, prefix_len=8, dtype=dtype)
    rng = np.random.default_rng(7)
    k, v = (WL.quantise(wl, rng.standard_normal((n_tok, n_heads, D), dtype=np.float32)) for _ in range(2))
    k, q, kn, vn = k / 4, *(WL.quantise(wl, rng.standard_normal((n_seq, n_heads, D), dtype=np.float32)) for _ in range(3))
    params = B.make_params(n_seq=n_seq, n_heads=n_heads, head_dim=D, grid_h=72, grid_w=72, win_rows_back=1, win_col_radius=2,
                           dtype=B.F32 if dtype == "f32" else B.BF16, cap=n_tok, layout=layout,
                           score_mode=B.SCORE_VCOS_FUSED if fused else B.SCORE_ATTN_MASS,
                           evict_policy=B.EVICT_REUSE_SLOT if fused else 0, win_recent_m=4 if fused else 0)
    assert plan_of(params).chunks == chunks
    batch = LayerBatch(params, DEV)
    sels, score = [], rng.random((n_seq, n_tok)).astype(np.float32)
    for b, n in enumerate(lens):
        sel = np.sort(rng.choice(n_tok, size=n, replace=False)).astype(np.int32)
        sels.append(sel)
        batch.set_sequence(b, k=k, v=v, pos=np.arange(n_tok, dtype=np.int32), score=None if fused else score[b], step=600,
                           grid_origin=8, budget=n_tok)
        batch.seqs_host[b]["pending_slot"] = sel[n // 2]       # the query token's slot: somewhere in the list
        batch.sel_idx[b, :n] = torch.from_numpy(sel).to(DEV)
    batch.upload_seqs()
    batch.sel_cnt.copy_(torch.tensor(lens, dtype=torch.int32))
    if fused:
        u = rng.standard_normal((n_seq, n_heads * D + 4)).astype(np.float32)
        u[:, n_heads * D:] = [602.0, 0.0, 0.0, 0.0]            # u belongs to the next step
        batch.vcos_u.copy_(torch.from_numpy(u))
    qd, kd, vd = (to_device(x, params.dtype, DEV) for x in (q, kn, vn))
    batch.attend(qd, B.FLAG_APPEND | B.FLAG_ADVANCE, kd, vd)
    torch.cuda.synchronize()
    out, lse, seqs = to_host(batch.out), batch.lse.cpu().numpy(), batch.read_seqs()
    rank, rows, Kd, Vd = rank_host(batch), batch.score.cpu().numpy(), batch.k_host(), batch.v_host()
    cfg = oracle_cfg(wl, budget=n_tok, cap=n_tok)
    for b, n in enumerate(lens):
        kb, vb, new = k.copy(), v.copy(), sels[b][n // 2]
        kb[new], vb[new] = kn[b], vn[b]
        assert np.array_equal(Kd[b], kb) and np.array_equal(Vd[b], vb) and seqs["step"][b] == 601
        ro, rl, probs = oracle.attend(cfg, kb, vb, q[b], sels[b], want_probs=True)
        check_out(wl, out[b], ro, f"len={n}")
        assert np.abs(lse[b] - rl).max() <= lse_tol(wl), n
        if not fused:
            assert np.allclose(rank[b], oracle.accumulate(cfg, score[b], sels[b], probs), rtol=1e-5, atol=1e-6), n
            continue
        vs = vb[sels[b]].astype(np.float64)                    # fp32 sums of D <= 128 products: a few 1e-7 of their terms
        sq, dot = (vs ** 2).sum(-1), (vs * u[b, :n_heads * D].reshape(n_heads, D)).sum(-1)
        assert np.allclose(rows[b, 0::2][:, sels[b]].T, sq, rtol=1e-5)
        assert np.allclose(rows[b, 1::2][:, sels[b]].T, dot, rtol=1e-5, atol=1e-4)
        assert batch.vcos_u[b, n_heads * D + 1] == 602.0       # the rows are the next step's


def test_timing_hook_counts_a_split_launch_once():
    """A split launch is two kernels; the benchmark's hook counts it as one, with a time."""
    params = B.make_params(n_seq=1, n_heads=2, head_dim=64, grid_h=72, grid_w=72, win_rows_back=1, win_col_radius=2, dtype=B.BF16,
                           score_mode=B.SCORE_ATTN_MASS, cap=4200)
    assert plan_of(params).chunks > 1
    batch = LayerBatch(params, DEV)
    batch.seqs_host["n_res"], batch.seqs_host["step"] = 4200, 600
    batch.upload_seqs()
    batch.sel_idx[0] = torch.arange(4200, dtype=torch.int32, device=DEV)
    batch.sel_cnt.fill_(4200)
    q = torch.ones((1, 2, 64), dtype=torch.bfloat16, device=DEV)
    batch.attend(q)
    B.adsa_profile_enable(True)
    for _ in range(3):
        batch.attend(q)
    torch.cuda.synchronize()
    n, ms = B.adsa_profile_read()
    B.adsa_profile_enable(False)
    assert n == 3 and 0.0 < ms < 100.0
