"""Unsplit calls of the 256-query shape that ask for no log-sum-exp: they do without the sum of the unrounded
probabilities, which also took part in the denominator's fallback and in the range check.  (The limited calls here are
too small for that shape and run in 128-query work-groups.)"""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


def _run(P, q, k, v, folded, want_lse, limits=None):
    import torch
    n_q, H = q.shape[:2]
    n_keys = k.shape[0]
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = W.f32_to_bf16_bits(q * c), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(kb), Hn.to_dev_bf16(vb)
    out = torch.empty_like(qd)
    lse = torch.empty((H, n_q), dtype=torch.float32, device="cuda") if want_lse else None
    scale = P.CROPE_SCALE_FOLDED if folded else Hn.SCALE
    if limits is None:
        P.chunk_attention_planned(qd, n_q, H, kd, vd, n_keys, [(0, n_keys)], scale, (8, 1), out, lse)
    else:
        lim = torch.from_numpy(limits.astype(np.int32)).cuda()
        P.chunk_attention_limited(qd, n_q, H, kd, vd, n_keys, [(0, n_keys)], scale, lim, out, lse)
    torch.cuda.synchronize()
    return Hn.bits_to_f64(Hn.dev_bits(out)), (Hn.bits_to_f64(qb) / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb))


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2603_06664_amd as pkg
    return pkg


@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("n_q,n_keys", [(1, 1), (17, 31), (64, 33), (65, 128), (255, 129), (257, 385), (300, 640)])
def test_matches_the_oracle(P, n_q, n_keys, folded):
    import oracle
    print("no lse: n_q %d n_keys %d folded %d" % (n_q, n_keys, folded), flush=True)
    rng = np.random.default_rng(7 * n_q + n_keys)
    q, k, v = (rng.standard_normal((n, 2, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    got, ref = _run(P, q, k, v, folded, False)
    Hn.assert_close("o", got, oracle.attention(*ref, Hn.SCALE)[0])
    limits = 1 + (np.arange(n_q) * 11) % n_keys
    got, ref = _run(P, q, k, v, folded, False, limits)
    want = np.empty_like(got)
    for lim in np.unique(limits):
        rows = limits == lim
        want[rows] = oracle.attention(ref[0][rows], ref[1][:lim], ref[2][:lim], Hn.SCALE)[0]
    Hn.assert_close("o limited", got, want)


@pytest.mark.parametrize("folded", [False, True])
def test_second_run(P, folded):
    """Keys whose scores are some 200 powers of two above those of the first block."""
    import oracle
    rng = np.random.default_rng(3)
    q, k, v = (rng.standard_normal((n, 2, 128)).astype(np.float32) for n in (200, 300, 300))
    k[70:] *= 50.0
    got, ref = _run(P, q, k, v, folded, False)
    Hn.assert_close("o", got, oracle.attention(*ref, Hn.SCALE)[0])


@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("what", ["nan", "inf", "huge"])
def test_one_query_does_not_reach_another(P, folded, what):
    """A query with NaN, infinite or overflowing scores: every other row is what it is without it (rounding of a
    second run apart), and a NaN or infinite query's own row is NaN, as with the log-sum-exp."""
    rng = np.random.default_rng(11)
    q, k, v = (rng.standard_normal((n, 2, 128)).astype(np.float32) for n in (256, 500, 500))
    clean = _run(P, q, k, v, folded, False)[0]
    bad = [5, 21, 100, 255]
    q2 = q.copy()
    q2[bad, :, 3] = {"nan": np.nan, "inf": np.inf, "huge": 3e4}[what]
    got = _run(P, q2, k, v, folded, False)[0]
    with_lse = _run(P, q2, k, v, folded, True)[0]
    others = np.setdiff1d(np.arange(256), bad)
    # two roundings of the probabilities against different references: a few bf16 half-ulps of the output
    Hn.assert_close("other rows", got[others], clean[others])
    if what != "huge":
        assert np.all(np.isnan(got[bad]))
    assert np.array_equal(np.isnan(got), np.isnan(with_lse))
    ok = ~np.isnan(got)
    assert np.max(np.abs(got[ok] - with_lse[ok])) <= 2e-2
