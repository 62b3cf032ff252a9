"""Calls and last work-groups of few queries, whose one or two waves store without the way through LDS that more take (up to 48 of
128, 64 in a split key range), and one query more: strided outputs, whole and split key ranges, with and without the log-sum-exp."""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("n_q", [1, 31, 32, 33, 48, 49, 64, 65, 129, 160, 161, 176, 177, 192, 193])
@pytest.mark.parametrize("with_lse", [False, True], ids=["nolse", "lse"])
def test_matches_the_oracle(n_q, splits, with_lse):
    import torch
    import oracle
    import paper_2603_06664_amd as P
    print("few queries: n_q %d splits %d lse %d" % (n_q, splits, with_lse), flush=True)
    H, n_keys, plan = 2, 201 * splits, (4, splits)
    rng = np.random.default_rng(n_q + 1000 * splits)
    q, k, v = (W.f32_to_bf16_bits(rng.standard_normal((n, H, 128)).astype(np.float32)) for n in (n_q, n_keys, n_keys))
    qd, kd, vd = (Hn.to_dev_bf16(x) for x in (q, k, v))
    wide = torch.full((n_q + 40, H + 1, 136), 7.0, dtype=torch.bfloat16, device="cuda")
    out = wide[:n_q, :H, :128]
    lse = torch.full((H, n_q + 40), 7.0, dtype=torch.float32, device="cuda").view(-1) if with_lse else None
    ws = torch.empty(max(16, P.chunk_attention_planned_workspace_bytes(n_q, H, n_keys, plan)), dtype=torch.uint8, device="cuda")
    P.chunk_attention_planned(qd, n_q, H, kd, vd, n_keys, [(0, n_keys)], Hn.SCALE, plan, out, lse, ws)
    torch.cuda.synchronize()
    ref, ref_lse = oracle.attention(*(Hn.bits_to_f64(x) for x in (q, k, v)), Hn.SCALE)[:2]
    Hn.assert_close("o", Hn.bits_to_f64(Hn.dev_bits(out.contiguous())), ref)
    assert (wide[n_q:] == 7).all() and (wide[:, H:] == 7).all() and (wide[:, :, 128:] == 7).all()
    if with_lse:
        got = lse.cpu().numpy()
        assert np.max(np.abs(got[:H * n_q].reshape(H, n_q) - ref_lse)) <= 2e-2
        assert (got[H * n_q:] == 7).all()
