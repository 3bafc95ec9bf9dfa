"""adsa_step of few (sequence, head) pairs, which ranks inside the attention launch and leaves the changes of the record, pos and score to a
second one, against the same step as adsa_select, adsa_attend and adsa_compact: lists, keep maps, records, positions and cache rows bit
by bit, over capacities around the numbers of slots per thread, row ends, images that begin, and records that have to be refused."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2506_18226_amd import binding as B

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu

FIELDS = ("n_res", "step", "status", "compacted", "pending_slot", "hole")


def make(n_seq, n_heads, D, dtype, layout, cap, sel_cap, W, R, new_f32, seed, recent_m=0):
    """A batch of ragged states: pinned prefixes, older tokens, the last rows; every third sequence at a row's end; the last ones are an
    empty image, an inactive record, a full cache, a position newer than the query, a list longer than sel_cap and a step past the image."""
    rng = np.random.default_rng(seed)
    H, tdt = 40, torch.float32 if dtype == B.F32 else torch.bfloat16
    p = B.make_params(n_seq=n_seq, n_heads=n_heads, head_dim=D, grid_h=H, grid_w=W, win_rows_back=R, win_col_radius=2, dtype=dtype,
                      score_mode=B.SCORE_ATTN_MASS, cap=cap, sel_cap=sel_cap, layout=layout, win_recent_m=recent_m)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    shape = (n_seq, n_heads, cap, D) if layout == "head_major" else (n_seq, cap, n_heads, D)
    K, V = randn(*shape).to(tdt), randn(*shape).to(tdt)
    score = torch.rand((n_seq, n_heads, cap), generator=gen, device=DEV)
    score[:, :, ::5] = score[:, :, :1]                           # ties
    pos = torch.full((n_seq, cap), -7, dtype=torch.int32)
    seqs = np.zeros(n_seq, dtype=B.SEQ_DTYPE)
    odd = {n_seq - 1 - k: what for k, what in enumerate(("empty", "inactive", "full", "newer", "long", "past"))} if n_seq > 8 else {}
    for b in range(n_seq):
        P = int(rng.integers(1, min(40, cap // 4)))
        s = int(rng.integers(2, 12)) * W if b % 3 == 0 else int(rng.integers(1, 12 * W))
        what = odd.get(b, "")
        P, s = (0, 0) if what == "empty" else (P, s)
        jq = s - 1
        first = max(0, jq // W - R) * W
        if recent_m:
            first = max(0, jq - max(recent_m, W))
        recent, older = np.arange(first, max(jq, 0)), np.arange(0, first)
        if what == "long":                                       # (a prefix that fills the cache but for the query token)
            P, older = cap - 1 - len(recent), older[:0]
        room = cap - 1 - P - len(recent)
        assert room >= 0
        kept = np.sort(rng.permutation(older)[:int(rng.integers(0, room + 1))])
        if what == "full":
            kept = older[:0]
        image = np.concatenate([kept, recent])
        n = P + len(image)
        pos[b, :n] = torch.from_numpy(np.concatenate([np.arange(P), P + image]).astype(np.int32))
        budget = int(rng.integers(0, max(2, sel_cap - min(P, 40) - (R + 1) * W - 1)))
        if what == "full":
            pos[b, n:] = P + jq - 1
            n = cap
        if what == "newer":
            pos[b, n - 1] = P + jq + 1
        if what == "long":
            budget = cap
        q = seqs[b]
        q["k"], q["v"], q["pos"], q["score"] = K[b].data_ptr(), V[b].data_ptr(), 0, score[b].data_ptr()
        q["n_res"], q["step"], q["grid_origin"], q["n_keep_prefix"], q["budget"] = n, s, P, max(0, P - b % 3), budget
        if b % 4 == 1 and not what:
            q["budget_num"], q["budget_den"] = 1, 9
        if what == "inactive":
            q["step"] = -1
        if what == "past":
            q["step"] = H * W + 1
        q["pending_slot"], q["compacted"] = 5, 1
    pos = pos.to(DEV)
    seqs["pos"] = [pos[b].data_ptr() for b in range(n_seq)]
    q, kn, vn = randn(n_seq, n_heads, D).to(tdt), randn(n_seq, n_heads, D), randn(n_seq, n_heads, D)
    if not new_f32:
        kn, vn = kn.to(tdt), vn.to(tdt)
    return p, dict(K=K, V=V, score=score, pos=pos, seqs=seqs), (q, kn, vn)


def run(p, st, inputs, flags, one_call):
    """The step on a copy of the state."""
    st = {k: v.clone() if torch.is_tensor(v) else v.copy() for k, v in st.items()}
    for name, key in (("K", "k"), ("V", "v"), ("pos", "pos"), ("score", "score")):
        st["seqs"][key] = [st[name][b].data_ptr() for b in range(p.n_seq)]
    seqs = torch.from_numpy(st["seqs"].view(np.uint8).reshape(-1).copy()).to(DEV)
    q, kn, vn = inputs
    out, lse = torch.full_like(q, float("nan")), torch.full((p.n_seq, p.n_heads), float("nan"), device=DEV)
    idx = torch.full((p.n_seq, p.sel_cap), -3, dtype=torch.int32, device=DEV)
    cnt = torch.full((p.n_seq,), -3, dtype=torch.int32, device=DEV)
    km = torch.full((p.n_seq, p.cap), -9, dtype=torch.int32, device=DEV)
    ws = torch.full((B.adsa_workspace_bytes(p),), 0xFF, dtype=torch.uint8, device=DEV)
    if one_call:
        B.adsa_step(p, seqs, q, kn, vn, out, lse, idx, cnt, km, ws, flags)
    else:
        B.adsa_select(p, seqs, idx, cnt, flags=B.FLAG_PLAN_APPEND)
        B.adsa_attend(p, seqs, q, idx, cnt, out, lse, ws, B.FLAG_APPEND | flags, kn, vn)
        B.adsa_compact(p, seqs, km, ws, B.FLAG_ADVANCE)
    torch.cuda.synchronize()
    st["seqs"] = seqs.cpu().numpy().view(B.SEQ_DTYPE).reshape(-1)
    return {**st, "out": out.float(), "lse": lse, "idx": idx, "cnt": cnt, "km": km}


@pytest.mark.parametrize("n_seq,n_heads,D,dtype,layout,cap,sel_cap,W,R,new_f32,recent_m,launches", [
    (18, 3, 64, B.BF16, "head_major", 256, 150, 9, 1, True, 0, 2),       # 1, 1 | 2, 1 | 3, 2 | 2 x 512, 2 slots per thread
    (12, 7, 64, B.BF16, "slot_major", 257, 200, 11, 2, False, 0, 2),
    (9, 4, 128, B.BF16, "slot_major", 512, 301, 13, 1, False, 0, 2),
    (13, 5, 128, B.F32, "head_major", 513, 260, 12, 1, False, 0, 2),
    (10, 9, 64, B.F32, "head_major", 768, 330, 17, 1, False, 0, 2),
    (3, 26, 64, B.BF16, "head_major", 769, 500, 24, 2, False, 0, 2),     # more score rows than one batch
    (2, 20, 64, B.BF16, "head_major", 1024, 700, 28, 1, False, 0, 2),
    (11, 1, 64, B.F32, "head_major", 300, 299, 14, 1, False, 0, 2),
    (10, 3, 64, B.BF16, "head_major", 290, 200, 10, 1, False, 7, 2),     # the 1-D window
    (10, 3, 64, B.BF16, "head_major", 1025, 200, 10, 1, False, 0, 3),
    (12, 9, 64, B.BF16, "head_major", 257, 200, 10, 1, False, 0, 3),     # no room for the new scores
])
def test_a_step_in_two_launches_is_select_attend_and_compact(n_seq, n_heads, D, dtype, layout, cap, sel_cap, W, R, new_f32, recent_m, launches):
    lib = B.load_library()
    for seed in (1, 2, 3):
        p, st, inputs = make(n_seq, n_heads, D, dtype, layout, cap, sel_cap, W, R, new_f32, seed, recent_m)
        assert lib.adsa_step_launches(C.byref(p)) == launches
        flags = B.FLAG_NEW_F32 if new_f32 else 0
        got, want = (run(p, st, inputs, flags, one) for one in (True, False))
        assert (want["seqs"]["compacted"] == 1).any() and (want["seqs"]["step"] == st["seqs"]["step"] + 1).any()
        if n_seq > 8:
            assert len(set(want["seqs"]["status"])) >= 4        # none, bad state, cache full, list overflow
        for f in FIELDS:
            assert np.array_equal(got["seqs"][f], want["seqs"][f]), f
        assert torch.equal(got["cnt"], want["cnt"])
        for k in ("idx", "km", "K", "V", "pos"):
            assert torch.equal(got[k], want[k]), k
        # The same fp32 terms summed over 4 waves or 8 (1e-6 at most), and each side's rounding to bf16, 8 significant bits: up to 2^-8 of
        # the value, so two neighbouring results are up to 2^-7 apart
        tol = 2.0 ** -7 if dtype == B.BF16 else 1e-5
        assert ((got["out"] - want["out"]).abs() <= tol * want["out"].abs() + 1e-5).all()
        assert torch.allclose(got["lse"], want["lse"], rtol=1e-6, atol=1e-5)
        assert torch.allclose(got["score"], want["score"], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n_seq,n_heads,D,dtype,layout,cap,sel_cap,W,R,new_f32,recent_m,launches", [
    (60, 9, 64, B.BF16, "head_major", 256, 150, 9, 1, True, 0, 3),       # 1 | 2, 2 | 3, 3 slots per thread
    (30, 9, 128, B.BF16, "slot_major", 257, 200, 11, 2, False, 0, 3),
    (40, 13, 64, B.BF16, "head_major", 512, 301, 13, 1, False, 0, 3),
    (45, 12, 64, B.F32, "head_major", 513, 260, 12, 1, False, 0, 3),
    (33, 8, 128, B.F32, "head_major", 768, 300, 17, 1, False, 0, 3),
    (20, 27, 64, B.BF16, "head_major", 600, 500, 24, 2, False, 0, 3),    # more score rows than three batches
    (513, 1, 64, B.BF16, "head_major", 300, 200, 10, 1, False, 0, 3),    # one ticket
    (300, 2, 64, B.BF16, "head_major", 290, 200, 10, 1, False, 7, 3),    # the 1-D window
    (70, 8, 64, B.BF16, "head_major", 769, 300, 10, 1, False, 0, 4),
])
def test_a_step_that_plans_in_its_attention_is_select_attend_and_compact(n_seq, n_heads, D, dtype, layout, cap, sel_cap, W, R, new_f32, recent_m, launches):
    """Larger steps: the last workgroup of a sequence that closed a row plans its eviction, from scores that the others have just
    stored.  The arithmetic is that of the three calls: everything is the same, bit by bit."""
    lib = B.load_library()
    for seed in (1, 2, 3):
        p, st, inputs = make(n_seq, n_heads, D, dtype, layout, cap, sel_cap, W, R, new_f32, seed, recent_m)
        assert lib.adsa_step_launches(C.byref(p)) == launches
        flags = B.FLAG_NEW_F32 if new_f32 else 0
        got, want = (run(p, st, inputs, flags, one) for one in (True, False))
        assert (want["seqs"]["compacted"] == 1).sum() > n_seq // 5 and (want["seqs"]["step"] == st["seqs"]["step"] + 1).any()
        assert len(set(want["seqs"]["status"])) >= 4
        for f in FIELDS:
            assert np.array_equal(got["seqs"][f], want["seqs"][f]), f
        for k in ("cnt", "idx", "km", "K", "V", "pos", "score", "out", "lse"):
            assert torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("n_seq,n_heads,D,dtype,layout,cap,sel_cap,launches", [
    (9, 4, 64, B.BF16, "head_major", 120, 100, 2),
    (10, 3, 64, B.F32, "slot_major", 290, 200, 2),
    (9, 5, 128, B.BF16, "head_major", 700, 500, 2),
    (2, 20, 64, B.BF16, "head_major", 1024, 700, 2),
    (12, 9, 64, B.BF16, "head_major", 257, 200, 3),                      # ranked by a launch of its own
    (60, 9, 64, B.BF16, "head_major", 256, 150, 3),                      # planned by the attention
])
def test_a_step_before_the_first_token_leaves_scores_that_nobody_attends(n_seq, n_heads, D, dtype, layout, cap, sel_cap, launches):
    """Step 0, a condition that is not pinned: its tokens are candidates, and with an effective budget of 0 none is attended.  The record
    advances; the scores stay, beside sequences that attend some or all of theirs, whatever the workspace holds."""
    p, st, inputs = make(n_seq, n_heads, D, dtype, layout, cap, sel_cap, 10, 1, False, 1)
    assert B.load_library().adsa_step_launches(C.byref(p)) == launches
    none = []
    for b in range(n_seq):
        P = (1, 30)[b % 2]
        num, den, budget, pinned = ((0, 0, 0, 0), (1, P + 1, 7, 0), (1, 2, 0, 0), (0, 0, 0, P))[b // 2 % 4]
        q = st["seqs"][b]
        q["n_res"], q["step"], q["grid_origin"], q["n_keep_prefix"], q["status"] = P, 0, P, pinned, 0
        q["budget"], q["budget_num"], q["budget_den"] = budget, num, den
        st["pos"][b, :P] = torch.arange(P, dtype=torch.int32)
        if pinned == 0 and (P * num // den if den else budget) == 0:
            none.append(b)
    got, want = (run(p, st, inputs, 0, one) for one in (True, False))
    some = [b for b in range(n_seq) if b not in none]
    assert none and (some or n_seq == 2)
    assert (got["cnt"][none] == 0).all() and (got["out"][none] == 0).all() and (got["cnt"][some] > 0).all()
    assert torch.equal(got["score"][none], st["score"][none])
    for f in FIELDS:
        assert np.array_equal(got["seqs"][f], want["seqs"][f]), f
    assert (got["seqs"]["step"] == 1).all() and (got["seqs"]["status"] == 0).all()
    for k in ("cnt", "idx", "km", "K", "V", "pos"):
        assert torch.equal(got[k], want[k]), k
    # (fp32 sums over 4 waves or 8: as above)
    assert torch.allclose(got["score"], want["score"], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n_seq,n_heads,D,dtype,layout,cap", [
    (9, 4, 64, B.BF16, "head_major", 200), (9, 5, 64, B.F32, "slot_major", 400), (9, 3, 64, B.BF16, "head_major", 900)])
def test_a_step_whose_budget_covers_every_candidate(n_seq, n_heads, D, dtype, layout, cap):
    """The ranks are not read then, unless positions are not distinct: more candidates than positions they can have, and the budget is no
    longer all of them.  Beside sequences whose candidates are ranked."""
    p, st, inputs = make(n_seq, n_heads, D, dtype, layout, cap, cap, 10, 1, False, 1)
    assert B.load_library().adsa_step_launches(C.byref(p)) == 2
    rng = np.random.default_rng(cap)
    P, s, n = 12, 3, cap - 1
    for b in range(n_seq):
        q = st["seqs"][b]
        q["grid_origin"], q["n_keep_prefix"], q["status"], q["budget_num"], q["budget_den"] = P, 0, 0, 0, 0
        if b % 3 == 2:                                           # 12 positions in all the slots
            q["step"], q["n_res"], q["budget"] = s, n, P + s - 1
            st["pos"][b, :n] = torch.from_numpy(np.sort(rng.integers(0, P, n)).astype(np.int32))
        else:                                                    # distinct ones, all of them or a third attended
            q["step"], q["n_res"], q["budget"] = n - P + 1, n, n if b % 3 == 0 else cap // 3
            st["pos"][b, :n] = torch.arange(n, dtype=torch.int32)
    p.grid_h = 200                                               # (rows enough for the longest of them)
    got, want = (run(p, st, inputs, 0, one) for one in (True, False))
    assert (want["seqs"]["status"] == 0).all() and (want["seqs"]["step"] == st["seqs"]["step"] + 1).all()
    cnt = want["cnt"].cpu().numpy()
    assert (cnt[0::3] == cap).all() and (cnt[1::3] < cap).all() and (cnt[2::3] == P + s - 1 + 1).all()
    for f in FIELDS:
        assert np.array_equal(got["seqs"][f], want["seqs"][f]), f
    for k in ("cnt", "idx", "km", "K", "V", "pos"):
        assert torch.equal(got[k], want[k]), k
    assert torch.allclose(got["score"], want["score"], rtol=1e-5, atol=1e-6)        # (fp32 sums over 4 waves or 8: as above)
