"""The merge of the partial results at every number of key splits, each of which has a kernel of its own; query counts
that leave the last work-group of the merge and the last wave of the attention partly empty; key ranges of very unlike weight;
both scale conventions; strided outputs."""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn


@pytest.mark.gpu
@pytest.mark.parametrize("splits", range(2, 17))
@pytest.mark.parametrize("n_q,waves", [(1, 4), (67, 4), (33, 8), (259, 8)])
@pytest.mark.parametrize("folded", [False, True], ids=["scale", "folded"])
def test_matches_the_oracle(splits, n_q, waves, folded):
    import torch
    import oracle
    import paper_2603_06664_amd as P
    print("merge: splits %d n_q %d waves %d folded %d" % (splits, n_q, waves, folded), flush=True)
    H, n_keys = 3, 64 * 2 * splits - 5   # two units of 64 keys in every range, the last one ragged
    rng = np.random.default_rng(splits + 100 * n_q)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    k *= np.take([4.0, 0.25, 2.0, 1.0], np.arange(n_keys) // 128 % 4)[:, None, None].astype(np.float32)   # one factor per range
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = (W.f32_to_bf16_bits(x) for x in (q * c, k, v))
    q_ref, k_ref, v_ref = Hn.bits_to_f64(qb) / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb)
    qd, kd, vd = (Hn.to_dev_bf16(x) for x in (qb, kb, vb))
    plan = (waves, splits)
    assert P.chunk_attention_choose_plan(n_q, H, n_keys, plan) == plan
    wide = torch.zeros((n_q, H + 1, 136), dtype=torch.bfloat16, device="cuda")
    out = wide[:, :H, :128]
    lse = torch.empty((H, n_q), dtype=torch.float32, device="cuda")
    ws = torch.empty(P.chunk_attention_planned_workspace_bytes(n_q, H, n_keys, plan), dtype=torch.uint8, device="cuda")
    scale = P.CROPE_SCALE_FOLDED if folded else Hn.SCALE
    P.chunk_attention_planned(qd, n_q, H, kd, vd, n_keys, [(0, n_keys)], scale, plan, out, lse, ws)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attention(q_ref, k_ref, v_ref, Hn.SCALE)[:2]
    # what the ranges weigh: the lightest and the heaviest of the first two differ by a factor of e^3 and more
    first, second = (oracle.attention(q_ref, k_ref[r], v_ref[r], Hn.SCALE)[1] for r in (slice(0, 128), slice(128, 256)))
    assert np.median(first - second) >= 3.0
    Hn.assert_close("o", Hn.bits_to_f64(Hn.dev_bits(out.contiguous())), ref)
    assert np.max(np.abs(lse.cpu().numpy() - ref_lse)) <= 2e-2
    assert not wide[:, H:].any() and not wide[:, :, 128:].any()
