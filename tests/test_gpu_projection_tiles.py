"""The projection's work-groups where they can go wrong: the body that a ragged last token tile takes (64, 128, 192 or 256
tokens, one row more and less), one or two heads per work-group and both in one launch, an odd number of heads (the last
pair holds one), reductions shorter and longer than the rings of copies; axis splits whose borders fall inside a lane's two
rotation pairs, and empty axes."""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn


def _check(n, heads, c_in, per_head):
    print("projection tiles n=%d heads=%d c_in=%d per_head=%s" % (n, heads, c_in, per_head), flush=True)
    cfg = W.ChunkConfig("QB", 17 + n, heads, 30, 50, start_frame=3, n_frames=1, first_kv_frame=3, token_offset=7, n_local=n)
    group = cfg.head_dim if per_head else cfg.n_heads * cfg.head_dim
    inp = W.make_inputs(cfg)
    pin = W.make_projection_inputs(cfg, c_in=c_in)
    ref = Hn.oracle_projected(cfg, pin, inp, norm_group=group)
    got = Hn.hip_projected(cfg, pin, inp, norm_group=group)
    for name, r in zip(("q", "k", "v"), ref):
        Hn.assert_close(name, got[name], r)
    assert got["untouched_ok"], "rows outside [dst, dst+n) were written"
    again = Hn.hip_projected(cfg, pin, inp, norm_group=group)
    for name in ("q", "k", "v"):
        np.testing.assert_array_equal(got[name], again[name])


# one head per work-group: bodies of 64, 128, 192 and 256 tokens; 1 to 6 reduction steps
@pytest.mark.gpu
@pytest.mark.parametrize("n,c_in", [(63, 64), (64, 128), (65, 192), (127, 256), (128, 320), (129, 384), (192, 64), (193, 128),
                                    (255, 192), (256, 320), (257, 256), (449, 64)])
@pytest.mark.parametrize("per_head", [False, True], ids=["normHD", "normD"])
def test_one_head(n, c_in, per_head):
    _check(n, 3, c_in, per_head)


# two heads per work-group (more than 128 pairs of heads and token tiles), the last pair of 129 heads of q, k and v holds one
@pytest.mark.gpu
@pytest.mark.parametrize("n,heads,c_in", [(257, 43, 64), (320, 43, 128), (385, 43, 192), (449, 43, 256), (540, 40, 640),
                                          (577, 43, 576), (769, 31, 320)])
@pytest.mark.parametrize("per_head", [False, True], ids=["normHD", "normD"])
def test_two_heads(n, heads, c_in, per_head):
    _check(n, heads, c_in, per_head)


# a round of two heads per work-group and the rest in one head each
@pytest.mark.gpu
@pytest.mark.parametrize("n,heads,c_in", [(1100, 40, 64), (1281, 37, 128)])
@pytest.mark.parametrize("per_head", [False, True], ids=["normHD", "normD"])
def test_both_in_one_launch(n, heads, c_in, per_head):
    _check(n, heads, c_in, per_head)


# The epilogue reads two neighbouring table entries at a time and the second by itself where it lies on the next axis: at an odd
# number of time pairs, of time and height pairs, of both, at an axis of one pair; empty axes
@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(44, 42, 42), (42, 44, 42), (42, 42, 44), (46, 2, 80), (2, 126, 0), (126, 0, 2), (0, 126, 2), (0, 2, 126),
                                  (128, 0, 0), (0, 128, 0), (0, 0, 128)], ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("n,heads", [(67, 3), (257, 43)])
@pytest.mark.parametrize("per_head", [False, True], ids=["normHD", "normD"])
def test_axis_splits(dims, n, heads, per_head):
    print("projection axis split %s n=%d heads=%d per_head=%s" % (dims, n, heads, per_head), flush=True)
    cfg = W.ChunkConfig("QX", 5 + n, heads, 5, 9, start_frame=3, n_frames=6, first_kv_frame=3, token_offset=7, n_local=n, dims=dims)
    group = cfg.head_dim if per_head else cfg.n_heads * cfg.head_dim
    inp = W.make_inputs(cfg)
    pin = W.make_projection_inputs(cfg, c_in=64)
    ref = Hn.oracle_projected(cfg, pin, inp, norm_group=group)
    got = Hn.hip_projected(cfg, pin, inp, norm_group=group)
    for name, r in zip(("q", "k", "v"), ref):
        Hn.assert_close(name, got[name], r)
    assert got["untouched_ok"], "rows outside [dst, dst+n) were written"
