"""What the attention launch rule promises, over random parameters (host code only)."""
import ctypes as C
import random

from paper_2506_18226_amd import binding as B

from common import plan_of


def test_chunks_leave_no_compute_unit_with_two_and_do_not_depend_on_the_nesting():
    rng, split = random.Random(3), 0
    for _ in range(20000):
        n_seq, n_heads, cap = rng.randint(1, 24), rng.randint(1, 12), rng.randint(100, 4000)
        D, dtype = rng.choice((64, 128)), rng.choice((B.F32, B.BF16))
        plans = [plan_of(B.make_params(n_seq=n_seq, n_heads=n_heads, head_dim=D, grid_h=64, grid_w=64, win_rows_back=1, win_col_radius=2,
                                       dtype=dtype, score_mode=B.SCORE_ATTN_MASS, cap=cap, layout=layout))
                 for layout in ("head_major", "slot_major")]
        what = (n_seq, n_heads, cap, D, dtype)
        assert plans[0].chunks == plans[1].chunks, what
        if plans[0].chunks > 1:                                 # (lists of up to 4000 slots fit the LDS whole)
            split += 1
            assert n_seq * n_heads < 96 and n_seq * n_heads * plans[0].chunks <= 256, what
    assert split > 2000


def test_one_and_two_pairs_split_where_more_do():
    for pairs in (1, 2):
        for D, dtype, eb in ((64, B.BF16, 2), (128, B.BF16, 2), (64, B.F32, 4), (128, B.F32, 4)):
            for layout in ("head_major", "slot_major"):
                plan = lambda kb: plan_of(B.make_params(n_seq=1, n_heads=pairs, head_dim=D, grid_h=64, grid_w=64, win_rows_back=1, win_col_radius=2,
                                                        dtype=dtype, score_mode=B.SCORE_ATTN_MASS, cap=(kb << 10) // (2 * D * eb), layout=layout))
                assert plan(325).chunks == 1 and plan(340).chunks == 6 and plan(420).chunks == 7


def test_caches_of_wide_strides_are_launched_like_dense_ones():
    rng, several, short = random.Random(4), 0, 0
    for _ in range(20000):
        kw = dict(n_seq=rng.randint(1, 200), n_heads=rng.choice((1, 2, 8, 24, 32, 40)), head_dim=rng.choice((64, 128)), grid_h=64, grid_w=64,
                  win_rows_back=1, win_col_radius=2, dtype=rng.choice((B.F32, B.BF16)), score_mode=B.SCORE_ATTN_MASS, cap=rng.randint(100, 4000),
                  layout="slot_major")
        kw["sel_cap"] = rng.randint(1, kw["cap"])
        if kw["n_heads"] == 1:
            kw["kv_head_stride"] = 16 << 20                     # (rows of one head: both nestings; this way head_major for both)
        dense, wide = plan_of(B.make_params(**kw)), plan_of(B.make_params(**kw, kv_slot_stride=1 << 24))
        assert (dense.chunks, dense.waves, dense.heads) == (wide.chunks, wide.waves, wide.heads), kw
        assert (dense.wide, wide.wide) == (0, 1), kw
        several += wide.heads > 1
        short += wide.waves == 4
    assert several > 1000 and short > 1000


def test_32_bit_offsets_end_where_the_unattended_ones_begin():
    """Offsets from 2^32 - 2 * 8192 on stand for no row: a cache whose rows end there is reached with 32 bits, one byte more and it is not."""
    limit, n = (1 << 32) - 2 * B.MAX_CAP, 513                  # 512 strides and a row of 128 bytes
    for stride, wide in (((limit - 128) // 512 // 16 * 16, 0), ((limit - 128) // 512 // 16 * 16 + 16, 1)):
        p = B.make_params(n_seq=1, n_heads=1, head_dim=64, grid_h=64, grid_w=64, win_rows_back=1, win_col_radius=2, dtype=B.BF16,
                          score_mode=B.SCORE_ATTN_MASS, cap=n, layout="slot_major", kv_slot_stride=stride // 2, kv_head_stride=64)
        assert (n - 1) * stride + 128 <= limit if not wide else (n - 1) * stride + 128 > limit
        assert plan_of(p).wide == wide


def test_only_steps_of_up_to_4096_pairs_plan_in_their_attention():
    """The workgroups that plan gather on one XCD, which a row end of a large batch would wait for."""
    lib = B.load_library()
    for n_heads, n_seq in ((24, 170), (48, 85), (8, 512), (1, 4096)):
        for n, launches in ((n_seq, 3), (n_seq + 1, 4)):
            p = B.make_params(n_seq=n, n_heads=n_heads, head_dim=64, grid_h=40, grid_w=24, win_rows_back=1, win_col_radius=2, dtype=B.BF16,
                              score_mode=B.SCORE_ATTN_MASS, cap=300, layout="head_major")
            assert lib.adsa_step_launches(C.byref(p)) == launches, (n, n_heads)
