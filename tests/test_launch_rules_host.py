"""What the attention launch rule promises of split lists, over random parameters (host code only)."""
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
