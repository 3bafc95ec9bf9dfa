"""The work this framework is used for, as cases that can be timed and compared.

A case describes the caches of one decode batch (all layers of a model, or several independent layers) somewhere
inside an image and what a program asks of the library there, through `paper_2506_18226_amd`:

  layers  one decode step of a model in split phase: ONE `select_all` for every layer's sequences, one
          `attend_layer` per layer (append + gather attention + score update), `compact_all` if the step closes a row
  step    one `adsa_step` per layer: the one-call form, also for ragged batches whose sequences stand at different
          depths, with different prefixes and budgets
  stream  one decode step under the paper's own cache policy: evict one when full, then append and attend everything
          resident; the cache moves on from pass to pass and starts over when the image is complete
  evict   the row-end eviction + compaction of a batch

The first two forms and `evict` start every pass from a snapshot of the sequence records (a device copy of 96 bytes per
sequence; where a pass evicts, `pos` and `score` too), so a pass can be repeated.  Cache rows that an eviction has moved
stay where they are: any rows serve the next pass.  Shapes are those of the repository's workload list (tiny, xl, xxl, long,
ragged, gqa) and of its tests; values follow its recipes: Gaussian K and V, logits with a standard deviation of
`q_scale`, attention mass that grows with the time a token has been resident (so that an eviction mostly
drops young tokens).  K/V of a pass exceeds the memory-side cache wherever a model's K/V would.
"""
from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda:0"


# --------------------------------------------------------------------------- cases
def _case(name=None, **kw):
    c = dict(kind="layers", n_seq=1, layers=1, heads=16, head_dim=64, q_per_kv=1, dtype="bf16", layout="head_major",
             prefix=120, grid_h=32, grid_w=32, rows_back=1, col_radius=4, recent_m=0, budget=512, budget_den=0,
             score="mass", policy="row_end", step=1, ragged=False, new_f32=False, q_scale=1.0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: one image, the fp32 toy model of the workload list, 8 layers, one adsa_step each
        _case("tiny_steps", kind="step", n_seq=1, layers=8, heads=16, head_dim=64, dtype="f32", prefix=32, grid_h=16,
              grid_w=16, col_radius=2, budget=64, step=200),
        # interactive generation: ONE image under classifier-free guidance (two sequences) with the 36-layer model
        _case("xl_one_image", n_seq=2, layers=36, heads=20, grid_h=24, grid_w=24, col_radius=3, budget=1, budget_den=2,
              step=400),
        # a middling batch of the same model: 16 sequences, half the context kept
        _case("xl_batch", n_seq=16, layers=36, heads=20, grid_h=24, grid_w=24, col_radius=3, budget=1, budget_den=2,
              step=500),
        # the headline configuration deep in the image: 48 layers x 32 sequences (the largest case)
        _case("xxl_batch", n_seq=32, layers=48, heads=24, step=1000, q_scale=2.8),
        # few sequences with long contexts: 64x64 tokens, 32 heads x 128
        _case("long_batch", n_seq=4, layers=8, heads=32, head_dim=128, prefix=256, grid_h=64, grid_w=64, rows_back=2,
              col_radius=8, budget=1024, step=3600),
        # serving: 64 sequences at independent depths, prefixes and budgets, one adsa_step per layer; some close a row
        _case("ragged_serving", kind="step", n_seq=64, layers=4, heads=24, ragged=True),
        # odd sizes: 7 ragged sequences in a [slot][head][D] cache of 9 heads x 128, fp32 rows converted as they enter
        _case("odd_slot_major", kind="step", n_seq=7, layers=6, heads=9, head_dim=128, layout="slot_major", prefix=37,
              grid_h=23, grid_w=29, rows_back=2, col_radius=5, budget=301, ragged=True, new_f32=True),
        # grouped queries: 8 cache heads x 128 with 8 query heads each, 48 layers
        _case("gqa_batch", n_seq=32, layers=48, heads=8, head_dim=128, q_per_kv=8, step=1000, q_scale=2.8),
        # the paper's cache policy: half-length cache, Eq. 2-3 ranking taken along by the attention launch
        _case("stream_fused", kind="stream", n_seq=32, layers=16, heads=24, recent_m=65, score="vcos_fused",
              policy="reuse", step=640),
        # the paper's ranking (Eq. 2-4, two passes over V) under the per-row cache
        _case("vcos_ranking", n_seq=32, layers=8, heads=24, score="vcos", step=700),
        # the row-end eviction of 16 layers x 32 sequences
        _case("row_eviction", kind="evict", n_seq=32, layers=16, heads=24, step=992),
        # the dense baseline the sparse path is compared with: the budget covers the whole 8000-token context
        _case("dense_8k", n_seq=2, layers=4, heads=16, head_dim=128, prefix=256, grid_h=88, grid_w=88, rows_back=1,
              budget=7744, step=7700),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["layers", "layers", "layers", "step", "step", "gqa", "stream", "vcos", "evict"])
    W = rng.randint(12, 40)
    H = rng.randint(12, 40)
    c = _case(kind=family if family in ("layers", "step", "stream", "evict") else "layers", grid_h=H, grid_w=W,
              prefix=rng.randint(8, 256), rows_back=rng.randint(1, 2), col_radius=rng.randint(2, 8),
              n_seq=_log_int(rng, 1, 64), heads=rng.randint(4, 24), head_dim=rng.choice([64, 64, 128]),
              dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), layout=rng.choice(["head_major", "head_major", "slot_major"]),
              q_scale=rng.choice([1.0, 2.8]), budget=_log_int(rng, 48, 1024))
    if rng.random() < 0.3:
        c["budget"], c["budget_den"] = 1, rng.randint(2, 4)
    c["step"] = rng.randint(W + 1, H * W)
    if c["kind"] == "layers" and rng.random() < 0.8 and c["step"] % W == 0:
        c["step"] -= 1
    if family == "step":
        c["ragged"] = rng.random() < 0.7
    if family == "gqa":
        c["dtype"], c["q_per_kv"], c["heads"] = "bf16", rng.choice([2, 4, 5, 8]), rng.randint(2, 12)
    if c["dtype"] == "bf16":
        c["new_f32"] = rng.random() < 0.25
    if family == "vcos":
        c["score"], c["heads"] = "vcos", min(c["heads"], 2048 // c["head_dim"])
    if family == "stream":
        c["policy"] = rng.choice(["reuse", "reuse", "when_full"])
        c["score"] = rng.choice(["vcos_fused", "vcos_fused", "mass", "vcos"]) if c["policy"] == "reuse" else rng.choice(["mass", "vcos"])
        if c["score"] == "vcos_fused":
            c["layout"] = "head_major"
        c["heads"] = min(c["heads"], 2048 // c["head_dim"])
        c["recent_m"] = rng.randint(2, 2 * W)
        c["budget"], c["budget_den"] = 0, 0
        c["step"] = H * W // 2 + rng.randint(2, H * W // 4)
    if family == "evict":
        c["step"] = W * rng.randint(3, H)
    # as many layers as a pass of 20 MB .. 2 GB of K/V takes, 48 at most
    per_layer = 2 * c["n_seq"] * c["heads"] * c["head_dim"] * _eb(c) * _cap(c)
    target = math.exp(rng.uniform(math.log(2e7), math.log(2e9)))
    c["layers"] = max(1, min(48, int(target / per_layer)))
    return c


# --------------------------------------------------------------------------- geometry
def _eb(c):
    return 4 if c["dtype"] == "f32" else 2


def _max_budget(c):
    L = c["prefix"] + c["grid_h"] * c["grid_w"]
    return L // c["budget_den"] * c["budget"] if c["budget_den"] else c["budget"]


def _cap(c):
    tokens = c["grid_h"] * c["grid_w"]
    if c["kind"] == "stream":
        return c["prefix"] + tokens // 2
    return c["prefix"] + min(tokens, _max_budget(c) + (c["rows_back"] + 1) * c["grid_w"])


def _sel_cap(c):
    if c["kind"] == "stream":
        return _cap(c)
    local = c["grid_w"] + c["rows_back"] * (2 * c["col_radius"] + 1)
    return min(_cap(c), c["prefix"] + local + _max_budget(c))


def _score_rows(c):
    return {"mass": c["heads"], "vcos_fused": 2 * c["heads"]}.get(c["score"], 1)


def _geometry(c, seed):
    """Per sequence (all layers): prefix, budget, step, resident positions before the pass."""
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 77])
    H, W, R, total, cap = c["grid_h"], c["grid_w"], c["rows_back"], c["n_seq"] * c["layers"], _cap(c)
    P, B, S = (np.empty(total, np.int64) for _ in range(3))
    for i in range(total):
        if c["ragged"] and i < c["n_seq"]:
            P[i] = rng.integers(max(1, c["prefix"] // 8), c["prefix"] + 1)
            B[i] = _max_budget(c) * int(rng.integers(1, 5)) // 4
            S[i] = rng.integers(1, H * W + 1)
        elif c["ragged"]:                                  # the layers of one sequence stand at the same step
            P[i], B[i], S[i] = P[i - c["n_seq"]], B[i - c["n_seq"]], S[i - c["n_seq"]]
        else:
            P[i], S[i] = c["prefix"], c["step"]
            B[i] = (P[i] + S[i]) * c["budget"] // c["budget_den"] if c["budget_den"] else c["budget"]
    pos = np.zeros((total, cap), np.int64)
    n = np.empty(total, np.int64)
    for i in range(total):
        jq = int(S[i]) - 1
        last = jq if c["kind"] == "evict" else jq - 1      # newest resident token: the query's own only after its append
        if c["kind"] == "stream":
            recent = np.arange(max(0, last + 1 - c["recent_m"]), last + 1)
            older, keep = np.arange(0, recent[0]), cap - int(P[i]) - recent.size
        else:
            first = max(0, jq // W - R) * W
            recent, older, keep = np.arange(first, last + 1), np.arange(0, first), int(B[i])
        kept = np.sort(rng.permutation(older)[:keep])
        image = np.concatenate([kept, recent])
        n[i] = P[i] + image.size
        pos[i, :n[i]] = np.concatenate([np.arange(P[i]), P[i] + image])
    return dict(P=P, B=B, S=S, pos=pos, n=n)


def _mean_counts(c, seed=0):
    """(attended, resident, candidates) tokens of the pass, averaged over one layer's sequences."""
    one = dict(c, layers=1)
    g = _geometry(one, seed)
    att = res = cand = 0
    W = c["grid_w"]
    for i in range(c["n_seq"]):
        jq, P = int(g["S"][i]) - 1, int(g["P"][i])
        p = g["pos"][i, :g["n"][i]]
        j = p[p >= P] - P
        if c["kind"] == "stream":
            a, k = len(p), int((j <= jq - c["recent_m"]).sum())
        else:
            dr, dc = jq // W - j // W, np.abs(j % W - jq % W)
            local = int(((dr == 0) | ((dr <= c["rows_back"]) & (dc <= c["col_radius"]))).sum())
            k = len(j) - local
            a = P + local + min(k, int(g["B"][i])) + 1
        att, res, cand = att + a, res + len(p) + 1, cand + k
    n = c["n_seq"]
    return att / n, res / n, cand / n


def work(case):
    c = case
    tau = 2 * c["heads"] * c["head_dim"] * _eb(c)          # K and V bytes of a token
    seqs, hq = c["n_seq"] * c["layers"], c["heads"] * c["q_per_kv"]
    rows = _score_rows(c)
    if c["kind"] == "evict":
        moved, n = _evict_counts(c)
        return {"bytes": seqs * (2.0 * moved * tau + n * (4 + 4 * rows) + moved * (4 + 4 * rows) + 4 * n), "flops": float(seqs * n * rows)}
    att, res, cand = _mean_counts(c)
    io = 2 * hq * c["head_dim"] * _eb(c) + 4 * hq + 2 * tau          # q, out, lse, the new row read and stored
    ranks = res * 4                                        # pos
    if c["score"] == "mass":
        ranks += 4 * rows * (att + (0 if c["kind"] == "stream" else res))
    elif c["score"] == "vcos_fused":
        ranks += 4 * rows * 2 * res + 8 * c["heads"] * c["head_dim"]
    else:
        ranks += 4 * res                                   # (the V rows the ranking needs are attended anyway, but for the dropped ones)
        ranks += max(0.0, res - att) * tau / 2
    flops = 4.0 * att * hq * c["head_dim"] + (4.0 * cand * c["heads"] * c["head_dim"] if "vcos" in c["score"] else 0.0)
    return {"bytes": float(seqs * (att * tau + io + ranks + 4 * att)), "flops": float(seqs * flops)}


def _evict_counts(c):
    """(rows that move, resident rows) of one sequence's eviction, averaged over a few sequences."""
    g = _geometry(dict(c, layers=1, n_seq=min(c["n_seq"], 16), ragged=False), 0)
    rng = np.random.default_rng(5)
    moved = n_all = 0
    for i in range(len(g["n"])):
        n, P, jq = int(g["n"][i]), int(g["P"][i]), int(g["S"][i]) - 1
        j = g["pos"][i, :n] - P
        age = np.where(j >= 0, jq - j + 1, jq + 1)
        rank = age * np.exp(0.75 * rng.standard_normal(n))
        rest = np.nonzero((j >= 0) & (j // c["grid_w"] < jq // c["grid_w"] - c["rows_back"] + 1))[0]
        drop = len(rest) - min(len(rest), int(g["B"][i]))
        if drop:
            gone = rest[np.argsort(rank[rest])[:drop]]
            moved += n - int(gone.min()) - drop
        n_all += n
    return moved / len(g["n"]), n_all / len(g["n"])


def tolerance(case):
    if case["kind"] == "evict":
        return "exact"                                     # rows, positions, scores and the keep map are moved, not computed
    if case["dtype"] == "f32" and case["score"] != "vcos_fused":
        t = {"rel": 2e-6, "max": 5e-5}
    else:                                                  # one rounding to bf16 per output element
        t = {"rel": 7e-3, "max": 2e-2}
    if case["score"] != "mass" or case["ragged"] or case["kind"] == "stream" or case["step"] % case["grid_w"] == 0:
        t["differ"] = 4e-3                                 # a near tie of computed scores: one sequence's list, shifted in part
    return t


# --------------------------------------------------------------------------- inputs
class _Inputs:
    """Everything a pass reads, from the seed alone."""

    TOKENS = 16                                            # stream: the incoming tokens repeat after this many steps

    def __init__(self, c, seed):
        self.geo = _geometry(c, seed)
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed * 2 + 1)
        self.c = c
        self.dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def cache(self, K, V):
        """Fills K and V ([layers * n_seq][...], either nesting)."""
        for x in (K, V):
            for i in range(0, x.shape[0], 64):
                x[i:i + 64].normal_(generator=self.gen)

    def rest(self):
        """q, k_new, v_new ([layers][tokens, for a stream][n_seq][heads][D]), score [layers * n_seq][rows][cap], pos."""
        c, g = self.c, self.geo
        T = self.TOKENS if c["kind"] == "stream" else 1
        shape = (c["layers"], T, c["n_seq"])

        def randn(*s):
            return torch.randn(*s, generator=self.gen, device=DEV, dtype=torch.float32)

        q = (randn(*shape, c["heads"] * c["q_per_kv"], c["head_dim"]) * c["q_scale"]).to(self.dtype)
        k = randn(*shape, c["heads"], c["head_dim"])
        v = randn(*shape, c["heads"], c["head_dim"])
        if not c["new_f32"]:
            k, v = k.to(self.dtype), v.to(self.dtype)
        pos = torch.from_numpy(g["pos"]).to(DEV)
        P, S, n = (torch.from_numpy(g[x]).to(DEV)[:, None] for x in ("P", "S", "n"))
        total, cap, rows = pos.shape[0], pos.shape[1], _score_rows(c)
        score = torch.zeros((total, rows, cap), device=DEV)
        if c["score"] == "mass":
            age = torch.where(pos >= P, S - 1 - (pos - P) + 1, S).clamp(min=1).float()
            mass = age / n.float() * torch.exp(0.75 * randn(total, cap))
            score.copy_(mass[:, None] * torch.exp(0.3 * randn(total, rows, cap)))
            score *= (torch.arange(cap, device=DEV)[None] < n)[:, None]
        return q, k, v, score, pos


def prepare(case, seed):
    from paper_2506_18226_amd import binding as B
    from paper_2506_18226_amd.batch import ModelBatch

    c = case
    inp = _Inputs(c, seed)
    p = B.make_params(
        n_seq=c["n_seq"], n_heads=c["heads"], head_dim=c["head_dim"], grid_h=c["grid_h"], grid_w=c["grid_w"],
        win_rows_back=c["rows_back"], win_col_radius=c["col_radius"], dtype=B.F32 if c["dtype"] == "f32" else B.BF16,
        score_mode={"mass": B.SCORE_ATTN_MASS, "vcos": B.SCORE_VCOS, "vcos_fused": B.SCORE_VCOS_FUSED}[c["score"]],
        cap=_cap(c), sel_cap=_sel_cap(c), layout=c["layout"], win_recent_m=c["recent_m"],
        evict_policy={"row_end": B.EVICT_ROW_END, "reuse": B.EVICT_REUSE_SLOT, "when_full": B.EVICT_WHEN_FULL}[c["policy"]],
        q_per_kv=c["q_per_kv"])
    mb = ModelBatch(p, c["layers"], DEV)
    inp.cache(mb.K, mb.V)
    q, k, v, score, pos = inp.rest()
    mb.score.copy_(score)
    mb.pos.copy_(pos)
    g, s = inp.geo, mb.seqs_host
    s["n_res"], s["step"], s["grid_origin"], s["n_keep_prefix"] = g["n"], g["S"], g["P"], g["P"]
    if c["budget_den"] and not c["ragged"]:
        s["budget_num"], s["budget_den"] = c["budget"], c["budget_den"]
    else:
        s["budget"] = g["B"]
    mb.upload_seqs()
    row_ends = bool((g["S"] % c["grid_w"] == 0).any())
    st = {"case": dict(c), "B": B, "mb": mb, "row_ends": row_ends, "seqs0": mb.seqs.clone(),
          "t": 0, "t_end": c["grid_h"] * c["grid_w"] - int(c["step"]) + 1}
    # what a layer's projections leave for the call: one tensor each per layer (and incoming token)
    st["in"] = [[(q[l, t], k[l, t], v[l, t]) for t in range(q.shape[1])] for l in range(c["layers"])]
    if c["kind"] == "step":                                # the layer's rows of the batch's arrays
        n, size = c["n_seq"], B.SEQ_DTYPE.itemsize
        st["rows"] = [(mb.seqs.data_ptr() + b * size, [x[b:b + n] for x in (mb.out, mb.lse, mb.sel_idx, mb.sel_cnt, mb.keep_map)])
                      for b in range(0, n * c["layers"], n)]
    st["state"] = mb.seqs.view(torch.int32).view(-1, 24)[:, 8:20]          # n_res .. reserved of every record
    if row_ends or c["kind"] in ("evict", "stream"):
        st["pos0"], st["score0"] = mb.pos.clone(), mb.score.clone()
    if c["kind"] == "stream":
        for _ in range(2):                                 # the program has been decoding: the running ranking state is warm
            run(st)
    return st


def _restore(st):
    mb = st["mb"]
    mb.seqs.copy_(st["seqs0"])
    if "pos0" in st:
        mb.pos.copy_(st["pos0"])
        mb.score.copy_(st["score0"])


def run(st):
    c, mb, B = st["case"], st["mb"], st["B"]
    new = B.FLAG_NEW_F32 if c["new_f32"] else 0
    if c["kind"] == "stream":
        if st["t"] >= st["t_end"]:                         # the image is complete: start over from the snapshot
            _restore(st)
            if mb.vcos_u is not None:
                mb.vcos_u.zero_()
            st["t"] = 0
        t = st["t"] % _Inputs.TOKENS
        st["t"] += 1
        mb.compact_all()
        mb.select_all(B.FLAG_PLAN_APPEND)
        for l in range(c["layers"]):
            mb.attend_layer(l, *st["in"][l][t], B.FLAG_APPEND | B.FLAG_ADVANCE | new)
    elif c["kind"] == "evict":
        _restore(st)
        mb.compact_all(B.FLAG_ADVANCE)
    elif c["kind"] == "step":
        _restore(st)
        for l in range(c["layers"]):
            seqs, rows = st["rows"][l]
            B.adsa_step(mb.layer_params, seqs, *st["in"][l][0], *rows, mb.layer_workspace, new)
    else:
        _restore(st)
        mb.select_all(B.FLAG_PLAN_APPEND)
        flags = B.FLAG_APPEND | new | (0 if st["row_ends"] else B.FLAG_ADVANCE)
        for l in range(c["layers"]):
            mb.attend_layer(l, *st["in"][l][0], flags)
        if st["row_ends"]:
            mb.compact_all(B.FLAG_ADVANCE)
    out = {"K": mb.K, "V": mb.V, "pos": mb.pos, "score": mb.score, "keep_map": mb.keep_map, "state": st["state"]}
    if c["kind"] != "evict":
        out.update(out=mb.out, lse=mb.lse, sel_idx=mb.sel_idx, sel_cnt=mb.sel_cnt)
    if mb.vcos_u is not None:
        out["vcos_u"] = mb.vcos_u
    return out


# --------------------------------------------------------------------------- the same in 64 bits, plain torch
def _attend64(q, K, V, mask, G):
    """q [n][h*G][D], K and V [n][h][cap][D], mask [n][cap] -> out, lse, probabilities summed over the G queries."""
    n, h, cap, D = K.shape
    z = torch.matmul(q.double().view(n, h, G, D), K.transpose(2, 3)) / math.sqrt(D)
    z = z.masked_fill(~mask[:, None, None, :], float("-inf"))
    lse = torch.logsumexp(z, dim=-1)
    p = torch.exp(z - lse[..., None])
    return torch.matmul(p, V).reshape(n, h * G, D), lse.reshape(n, h * G), p.sum(2)


def _vcos64(V, cand):
    """Mean cosine of every candidate's V row (heads concatenated) to the other candidates: [n][cap]."""
    n, h, cap, D = V.shape
    x = V.permute(0, 2, 1, 3).reshape(n, cap, h * D)
    x = x / x.norm(dim=-1, keepdim=True).clamp(min=1e-8) * cand[..., None]
    N = cand.sum(1, keepdim=True)
    S = (torch.matmul(x, x.sum(1)[..., None])[..., 0] - (x * x).sum(-1)) / (N - 1).clamp(min=1)
    return S * (N > 1)


def exact(case, seed):
    c = case
    if c["kind"] == "evict":
        return None
    inp = _Inputs(c, seed)
    cap, n, h, D, G, L = _cap(c), c["n_seq"], c["heads"], c["head_dim"], c["q_per_kv"], c["layers"]
    hm = c["layout"] == "head_major"
    Kc = torch.empty((n * L, h, cap, D) if hm else (n * L, cap, h, D), device=DEV, dtype=inp.dtype)
    Vc = torch.empty_like(Kc)
    inp.cache(Kc, Vc)
    q, kn, vn, score, pos = inp.rest()
    kn, vn = kn.to(inp.dtype), vn.to(inp.dtype)
    geo = {k: torch.from_numpy(inp.geo[k]).to(DEV) for k in ("P", "B", "S", "n")}
    outs, lses, scores = [], [], []
    with_score = c["kind"] != "stream" and not bool((inp.geo["S"] % c["grid_w"] == 0).any())
    for l in range(L):
        sl = slice(l * n, (l + 1) * n)
        K, V = (x[sl] if hm else x[sl].transpose(1, 2) for x in (Kc, Vc))
        K, V = K.double().contiguous(), V.double().contiguous()
        P, B, S, cnt = (geo[k][sl] for k in ("P", "B", "S", "n"))
        ps = pos[sl].clone()
        sc = score[sl].clone()
        rows, slots = torch.arange(n, device=DEV), torch.arange(cap, device=DEV)
        if c["kind"] == "stream":
            mass = sc.double()
            for t in range(3):                             # two steps before the pass, and the pass
                jq = S + t - 1
                j = ps - P[:, None]
                cand = (j >= 0) & (j <= (jq - c["recent_m"])[:, None])
                if c["score"] == "mass":
                    victim = mass.sum(1).masked_fill(~cand, float("inf")).argmin(1)
                else:
                    victim = _vcos64(V, cand).masked_fill(~cand, float("-inf")).argmax(1)
                K[rows, :, victim], V[rows, :, victim] = kn[l, t].double(), vn[l, t].double()
                ps[rows, victim] = P + jq
                mask = torch.ones((n, cap), dtype=torch.bool, device=DEV)
                o, z, p = _attend64(q[l, t], K, V, mask, G)
                if c["score"] == "mass":
                    mass[rows, :, victim] = 0
                    mass += p
        else:
            K[rows, :, cnt], V[rows, :, cnt] = kn[l, 0].double(), vn[l, 0].double()
            ps[rows, cnt] = P + S - 1
            sc[rows, :, cnt] = 0
            live = slots[None] <= cnt[:, None]
            jq, j, W = (S - 1)[:, None], ps - P[:, None], c["grid_w"]
            dr, dc = jq // W - j // W, (j % W - jq % W).abs()
            local = (j >= 0) & ((dr == 0) | ((dr > 0) & (dr <= c["rows_back"]) & (dc <= c["col_radius"])))
            cand = live & (j >= 0) & ~local
            if c["score"] == "mass":                       # the rank is the fp32 sum of the rows in ascending order
                rank = sc[:, 0].clone()
                for r in range(1, h):
                    rank += sc[:, r]
            else:
                rank = -_vcos64(V, cand)
            order = torch.sort(rank.masked_fill(~cand, float("-inf")), dim=1, descending=True, stable=True).indices
            place = torch.empty_like(order)
            place.scatter_(1, order, slots[None].expand_as(order))
            mask = (live & ~cand) | (cand & (place < B[:, None]))
            o, z, p = _attend64(q[l, 0], K, V, mask, G)
            if with_score:
                scores.append(sc.double() + p if c["score"] == "mass" else -rank * cand)
        outs.append(o)
        lses.append(z)
    ranked = c["score"] == "vcos" and c["kind"] != "stream"          # which of two near ties is attended is not a value
    if ranked and not with_score:
        return None
    return {"out": None if ranked else torch.cat(outs), "lse": None if ranked else torch.cat(lses),
            "score": torch.cat(scores) if with_score else None}
