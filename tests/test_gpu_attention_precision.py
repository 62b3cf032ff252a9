"""What the attention kernels keep exactly: a softmax that one key takes all of returns that key's V."""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2603_06664_amd as pkg
    return pkg


def attend(P, plan, qb, kb, vb, folded, segs=None):
    """bf16 bits in, (bf16 bits of the output, lse) out"""
    import torch
    n_q, H, n_rows = qb.shape[0], qb.shape[1], kb.shape[0]
    segs = segs or [(0, n_rows)]
    n_keys = sum(n for _, n in segs)
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(kb), Hn.to_dev_bf16(vb)
    out = torch.empty_like(qd)
    lse = torch.empty((H, n_q), dtype=torch.float32, device="cuda")
    wsb = P.chunk_attention_planned_workspace_bytes(n_q, H, n_keys, plan)
    ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device="cuda")
    P.chunk_attention_planned(qd, n_q, H, kd, vd, n_rows, segs, P.CROPE_SCALE_FOLDED if folded else Hn.SCALE, plan, out,
                              lse, ws, wsb)
    torch.cuda.synchronize()
    return Hn.dev_bits(out), lse.cpu().numpy()


def folded_q(P, q, folded):
    return W.f32_to_bf16_bits(q * np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else q)


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("gain,v_scale", [(3.0, 1.0), (3.0, 2.0 ** 90), (7.0, 1.0), (7.0, 2.0 ** 40), (9.0, 2.0 ** 100)])
def test_single_key_softmax_returns_its_value(P, waves, splits, folded, gain, v_scale):
    """Query i's own key 40 + i scores gain * |q|^2 * scale, at least 34 above the rest: all other weights together
    are below 1e-10.  Its probability is no bf16 number, but the same rounded value stands in numerator and
    denominator, so the output is V of that key times 1 +- a few 2^-24, which rounds to V's own bits.  Against
    the first 32 keys it is about 2^49, 2^114, 2^147: with a large V the product, and with the largest gain the
    probability itself, leaves fp32's range unless the reference follows."""
    print("single key waves %d splits %d folded %d gain %g v %g" % (waves, splits, folded, gain, v_scale), flush=True)
    H, n_q, n_keys = 2, 200, 300
    rng = np.random.default_rng(77)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    q = W.bf16_bits_to_f32(W.f32_to_bf16_bits(q))
    k[40:40 + n_q] = gain * q
    vb = W.f32_to_bf16_bits(v * np.float32(v_scale))
    got, _ = attend(P, (waves, splits), folded_q(P, q, folded), W.f32_to_bf16_bits(k), vb, folded)
    wrong = np.mean(got != vb[40:40 + n_q])
    assert wrong == 0, "%.1f %% of the outputs are not V" % (100 * wrong)


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("folded", [False, True])
def test_nan_query_leaves_the_others_alone(P, waves, splits, folded):
    import oracle
    print("nan query waves %d splits %d folded %d" % (waves, splits, folded), flush=True)
    H, n_q, n_keys = 2, 130, 200
    rng = np.random.default_rng(78)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    qb, kb, vb = folded_q(P, q, folded), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    c = float(np.float32(P.crope_folded_q_scale(Hn.SCALE))) if folded else 1.0
    o_ref, lse_ref = oracle.attention(Hn.bits_to_f64(qb) / c, Hn.bits_to_f64(kb), Hn.bits_to_f64(vb), Hn.SCALE)
    qb[70, 1, 3] = 0x7FC1
    out, lse = attend(P, (waves, splits), qb, kb, vb, folded)
    out = Hn.bits_to_f64(out)
    assert np.all(np.isnan(out[70, 1])) and np.isnan(lse[1, 70])
    out[70, 1], lse[1, 70] = o_ref[70, 1], lse_ref[1, 70]
    Hn.assert_close("o", out, o_ref)
    assert np.max(np.abs(lse - lse_ref)) <= 2e-5 * np.max(np.abs(lse_ref))


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("n_q", [70, 300])
def test_second_run_over_a_wrapped_ring(P, waves, splits, n_q):
    """Scores that outgrow the first keys' by some 2^300, in three segments, two of them shorter than a tile."""
    import oracle
    print("second run, ring, waves %d splits %d n_q %d" % (waves, splits, n_q), flush=True)
    H, segs = 2, [(500, 100), (20, 45), (100, 330)]
    rng = np.random.default_rng(79)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, 600, 600))
    k[520:] *= 50.0
    k[:500] *= 50.0
    qb, kb, vb = W.f32_to_bf16_bits(q), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    rows = np.concatenate([np.arange(a, a + n) for a, n in segs])
    hidden = np.setdiff1d(np.arange(600), rows)
    kb[hidden] = vb[hidden] = 0x7FC1
    out, lse = attend(P, (waves, splits), qb, kb, vb, False, segs)
    o_ref, lse_ref = oracle.attention(Hn.bits_to_f64(qb), Hn.bits_to_f64(kb)[rows], Hn.bits_to_f64(vb)[rows], Hn.SCALE)
    Hn.assert_close("o", Hn.bits_to_f64(out), o_ref)
    # fp32 scores of magnitude s carry an error of a few 2^-24 * s
    assert np.max(np.abs(lse - lse_ref) / np.maximum(1.0, np.abs(lse_ref))) <= 2e-5
