"""The CPython module between binding.py and the C entry points: what it takes for a pointer, what it refuses, and that the codes
of refused calls come back as before.  Every call here is refused by its arguments; nothing is launched."""
import ctypes as C

import pytest
import torch

from paper_2506_18226_amd import binding as B


def params(**kw):
    base = dict(n_seq=2, n_heads=4, head_dim=64, grid_h=4, grid_w=4, win_rows_back=1, win_col_radius=1, dtype=B.BF16,
                score_mode=B.SCORE_ATTN_MASS, cap=40)
    return B.make_params(**dict(base, **kw))


def entry_points(p, x, ws):
    s = dict(stream=0)
    return [lambda: B.adsa_select(p, x, x, x, ws, **s), lambda: B.adsa_attend(p, x, x, x, x, x, x, ws, 0, x, x, **s),
            lambda: B.adsa_compact(p, x, x, ws, **s), lambda: B.adsa_step(p, x, x, x, x, x, x, x, x, x, ws, **s),
            lambda: B.adsa_step_static(p, x, x, x, x, x, x, x, x, x, **s)]


@pytest.mark.parametrize("pointer", [None, 0, torch.zeros(8), (torch.zeros(8), 16), (0, 0), 1 << 40])
def test_every_entry_point_refuses_bad_parameters(pointer):
    for call in entry_points(params(n_seq=0), pointer, None):
        with pytest.raises(B.AdsaError) as e:
            call()
        assert e.value.code == -2 and str(e.value).startswith("adsa_")


def test_null_pointers_and_a_missing_workspace_are_seen_as_such():
    for call in entry_points(params(), None, torch.zeros(8)):
        with pytest.raises(B.AdsaError) as e:
            call()
        assert e.value.code == -1
    with pytest.raises(B.AdsaError) as e:                       # 64 bytes of workspace: refused by its size
        B.adsa_compact(params(), 1 << 40, 1 << 40, (torch.zeros(64), 0)[0], stream=0)
    assert e.value.code in (-4, -6)


@pytest.mark.parametrize("null", [(None, 96), (0, 4096)])
def test_an_offset_makes_no_pointer_of_null(null):
    """Otherwise valid calls, one pointer after the other missing."""
    x, q = 1 << 40, dict(stream=0)
    calls = [(3, lambda a: B.adsa_select(params(), *a, torch.zeros(8), **q)), (2, lambda a: B.adsa_compact(params(), *a, torch.zeros(8), **q)),
             (6, lambda a: B.adsa_attend(params(), *a, torch.zeros(8), **q)), (8, lambda a: B.adsa_attend(params(), *a[:6], torch.zeros(8), 8, *a[6:], **q)),
             (9, lambda a: B.adsa_step(params(), *a, torch.zeros(8), **q)), (9, lambda a: B.adsa_step_static(params(), *a, **q))]
    for n, call in calls:
        for i in range(n):
            with pytest.raises(B.AdsaError) as e:
                call([null if k == i else x for k in range(n)])
            assert e.value.code == -1


@pytest.mark.parametrize("bad", [1.5, "x", (0, 1.5), ((0, 0), 0), (0, 1, 2), object()])
def test_what_is_no_pointer_is_refused(bad):
    for call in entry_points(params(n_seq=0), bad, None):
        with pytest.raises((TypeError, AttributeError)):
            call()


@pytest.mark.parametrize("bad", [False, True, 0, 1 << 40, "x"])
def test_a_workspace_is_a_tensor_or_none(bad):
    s, p = dict(stream=0), params(n_seq=0)
    for call in (lambda: B.adsa_select(p, 0, 0, 0, bad, **s), lambda: B.adsa_attend(p, 0, 0, 0, 0, 0, 0, bad, **s),
                 lambda: B.adsa_compact(p, 0, 0, bad, **s), lambda: B.adsa_step(p, 0, 0, 0, 0, 0, 0, 0, 0, 0, bad, **s)):
        with pytest.raises(AttributeError):
            call()


@pytest.mark.parametrize("bad", [None, 0, b"\0" * 200, C.c_int(3), C.create_string_buffer(200)])
def test_parameters_of_another_type_are_refused(bad):
    with pytest.raises(TypeError):
        B.adsa_select(bad, 0, 0, 0, None, stream=0)


def test_flags_and_stream_are_integers():
    with pytest.raises(TypeError):
        B.adsa_select(params(n_seq=0), 0, 0, 0, None, flags=1.5, stream=0)
    with pytest.raises((TypeError, AttributeError)):
        B.adsa_select(params(n_seq=0), 0, 0, 0, None, stream="x")
