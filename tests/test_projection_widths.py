"""Which tile width the projection takes, and the 192-token tiles at their edges.  Where both widths take the same rounds, as
at most sizes here, they are taken for reductions of more than 512 only, so of at least 9 steps: the first step, steady ones
and the last four (two with two heads per work-group), at an odd and an even number of them, so that W's and x's rings end at
different places.  The 256-token ones are what the short reductions of test_gpu_projection.py run."""
import numpy as np
import pytest

import paper_2603_06664_amd as P
from paper_2603_06664_amd import workloads as W

import harness as Hn


@pytest.mark.parametrize("n,heads,c_in,width", [
    (200, 2, 256, 256), (600, 2, 256, 256), (600, 3, 384, 256), (1, 1, 64, 256),       # one round, short reduction
    (129, 40, 320, 256), (540, 40, 192, 256), (257, 40, 64, 256),
    (600, 8, 1024, 192), (600, 12, 1536, 192), (24, 40, 5120, 192), (585, 5, 5120, 192),   # one round of both
    (585, 40, 5120, 192), (4680, 5, 5120, 192), (1320, 16, 2048, 192),                 # two rounds of both
    (1560, 12, 1536, 256), (4680, 12, 1536, 256), (18720, 12, 1536, 256), (4680, 40, 5120, 256)])
def test_width_rule(n, heads, c_in, width):
    assert P.crope_qkv_project_tile_tokens(n, heads, c_in) == width


# Ragged against 192 by one row more and less, one row alone, two tiles and three; against the bodies of the last tile (64, 128, 192
# tokens) and the 16, 32 and 48 tokens that a wave has in them with one head per work-group; the last one in pairs of heads
@pytest.mark.gpu
@pytest.mark.parametrize("n,heads,c_in", [(1, 2, 576), (95, 3, 640), (97, 2, 704), (191, 2, 576), (192, 2, 640),
                                          (193, 2, 704), (383, 5, 576), (385, 2, 640), (540, 40, 576),
                                          (17, 2, 576), (63, 3, 640), (64, 2, 704), (65, 2, 576), (127, 3, 640), (128, 2, 704), (129, 2, 576),
                                          (144, 2, 640), (145, 3, 704), (241, 2, 576), (320, 3, 640)])
@pytest.mark.parametrize("per_head", [False, True], ids=["normHD", "normD"])
@pytest.mark.parametrize("bias", [False, True], ids=["nobias", "bias"])
def test_192_token_tiles(n, heads, c_in, per_head, bias):
    print("projection 192-token tiles n=%d heads=%d c_in=%d per_head=%s bias=%s" % (n, heads, c_in, per_head, bias),
          flush=True)
    assert P.crope_qkv_project_tile_tokens(n, heads, c_in) == 192
    cfg = W.ChunkConfig("QM", 91 + n, heads, 20, 30, start_frame=3, n_frames=1, first_kv_frame=3, token_offset=11,
                        n_local=n)
    group = cfg.head_dim if per_head else cfg.n_heads * cfg.head_dim
    inp = W.make_inputs(cfg)
    pin = W.make_projection_inputs(cfg, c_in=c_in)
    ref = Hn.oracle_projected(cfg, pin, inp, norm_group=group, use_bias=bias)
    got = Hn.hip_projected(cfg, pin, inp, norm_group=group, use_bias=bias, x_pad=0 if bias else 24)
    for name, r in zip(("q", "k", "v"), ref):
        Hn.assert_close(name, got[name], r)
    assert got["untouched_ok"], "rows outside [dst, dst+n) were written"
    again = Hn.hip_projected(cfg, pin, inp, norm_group=group, use_bias=bias, x_pad=0 if bias else 24)
    for name in ("q", "k", "v"):
        np.testing.assert_array_equal(got[name], again[name])
