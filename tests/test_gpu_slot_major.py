"""Attention over large batches in [slot][head][D] caches, where a workgroup takes the heads of 512 bytes of a token: against 64-bit
sums, over lists from empty to full, head counts that leave a group partly filled, and the query token's row on its way in."""
import numpy as np
import pytest
import torch

from paper_2506_18226_amd import binding as B
from paper_2506_18226_amd.batch import LayerBatch

from common import plan_of
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,h,D,dtype,cap,new_f32,accumulate,heads", [
    (100, 16, 64, "bf16", 130, False, True, 4),              # lists longer than a ring revolution
    (200, 7, 64, "bf16", 128, True, True, 4),                # the second group of 4 has 3 heads
    (97, 16, 64, "bf16", 2000, False, False, 4),             # close to the LDS limit, no score update
    (193, 4, 128, "bf16", 97, False, True, 2), (130, 6, 64, "f32", 75, False, True, 2), (130, 7, 64, "f32", 64, False, True, 2),
    (95, 16, 64, "bf16", 130, False, True, 1), (200, 7, 64, "bf16", 129, False, True, 1)])
def test_heads_that_share_a_workgroup(n_seq, h, D, dtype, cap, new_f32, accumulate, heads):
    params = B.make_params(n_seq=n_seq, n_heads=h, head_dim=D, grid_h=100, grid_w=100, win_rows_back=1, win_col_radius=2,
                           dtype=B.F32 if dtype == "f32" else B.BF16, cap=cap, layout="slot_major", score_mode=B.SCORE_ATTN_MASS)
    assert plan_of(params).heads == heads
    batch = LayerBatch(params, DEV)
    gen = torch.Generator(device=DEV).manual_seed(cap)
    for x in (batch.K, batch.V):
        x.normal_(generator=gen)
    q = torch.randn((n_seq, h, D), generator=gen, device=DEV).to(batch.tdtype)
    new = [torch.randn((n_seq, h, D), generator=gen, device=DEV).to(torch.float32 if new_f32 else batch.tdtype) for _ in range(2)]
    batch.score.uniform_(generator=gen)
    old = batch.score.clone()
    rng = np.random.default_rng(cap)
    lens = rng.integers(1, cap + 1, n_seq)
    lens[:6] = [1, 2, 5, 63, cap, 0][: min(6, n_seq)]
    lens = np.minimum(lens, cap)
    sel = np.zeros((n_seq, cap), np.int32)
    for b, n in enumerate(lens):
        sel[b, :n] = np.sort(rng.choice(cap, n, replace=False))
    pending = np.array([s[n // 3] if n else -1 for s, n in zip(sel, lens)], np.int32)
    s = batch.seqs_host
    s["n_res"], s["step"], s["pending_slot"] = cap, 40, pending
    batch.upload_seqs()
    batch.sel_idx.copy_(torch.from_numpy(sel))
    batch.sel_cnt.copy_(torch.from_numpy(lens.astype(np.int32)))
    flags = B.FLAG_APPEND | B.FLAG_ADVANCE | (B.FLAG_NEW_F32 if new_f32 else 0) | (0 if accumulate else B.FLAG_NO_ACCUMULATE)
    K0, V0 = batch.K.clone(), batch.V.clone()
    batch.attend(q, flags, *new)
    torch.cuda.synchronize()
    for b in range(n_seq):                                   # the caches as the launch has to leave them
        if lens[b]:
            K0[b, pending[b]], V0[b, pending[b]] = new[0][b].to(batch.tdtype), new[1][b].to(batch.tdtype)
    assert torch.equal(batch.K, K0) and torch.equal(batch.V, V0)
    assert (batch.read_seqs()["step"] == np.where(lens > 0, 41, 40)).all()
    # D and list sums in fp32: a few 1e-7 of terms of magnitude 1; bf16 rounds the output once
    out_rel, out_abs = (2.0 ** -8, 1e-4) if dtype == "bf16" else (0.0, 1e-5)
    for b in range(n_seq):
        n = int(lens[b])
        if n == 0:
            assert not batch.out[b].any() and not batch.lse[b].any() and torch.equal(batch.score[b], old[b])
            continue
        idx = torch.from_numpy(sel[b, :n].astype(np.int64)).to(DEV)
        z = (K0[b, idx].double() * q[b].double()).sum(-1).T / D ** 0.5                 # [h][n]
        p = torch.softmax(z, -1)
        ref = (p[:, :, None] * V0[b, idx].double().transpose(0, 1)).sum(1)
        assert ((batch.out[b].double() - ref).abs() <= out_rel * ref.abs() + out_abs).all(), (b, n)
        assert (batch.lse[b].double() - torch.logsumexp(z, -1)).abs().max() <= (1e-4 if dtype == "bf16" else 1e-5), (b, n)
        want = old[b].double()
        if accumulate:
            want[:, idx] += p
        assert torch.allclose(batch.score[b].double(), want, rtol=1e-5, atol=1e-6), (b, n)
