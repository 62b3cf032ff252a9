"""Both work-group shapes of the attention kernel at the edges of their tiles (blocks of 32 keys,
tiles of 64 and 128, 32-query groups, 128- and 256-query work-groups), and the second run that a
work-group makes when its sums outgrow the reference taken from the first 32 keys."""
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


def _case(P, waves, splits, n_q, n_keys, folded, limits=None, jump_at=None, H=2):
    import torch
    import oracle
    print("case waves %d splits %d n_q %d n_keys %d folded %d limited %d jump %s"
          % (waves, splits, n_q, n_keys, folded, limits is not None, jump_at), flush=True)
    rng = np.random.default_rng(1000 * n_q + n_keys)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    if jump_at is not None:      # from this key on, scores of about +-200 powers of two
        k[jump_at:] *= 50.0
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = W.f32_to_bf16_bits(q * c), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    cap = n_keys + 70            # rows behind the visible ones hold NaN: nothing may read them into a result
    pad = np.full((70, H, 128), 0x7FC1, dtype=np.uint16)
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(np.concatenate([kb, pad])), Hn.to_dev_bf16(np.concatenate([vb, pad]))
    out = torch.empty_like(qd)
    lse = torch.empty((H, n_q), dtype=torch.float32, device="cuda")
    scale = P.CROPE_SCALE_FOLDED if folded else Hn.SCALE
    q_ref, kf, vf = Hn.bits_to_f64(qb) / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb)
    if limits is None:
        plan = (waves, splits)
        wsb = P.chunk_attention_planned_workspace_bytes(n_q, H, n_keys, plan)
        ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device="cuda")
        P.chunk_attention_planned(qd, n_q, H, kd, vd, cap, [(0, n_keys)], scale, plan, out, lse, ws, wsb)
        o_ref, lse_ref = oracle.attention(q_ref, kf, vf, Hn.SCALE)
    else:
        P.chunk_attention_limited(qd, n_q, H, kd, vd, cap, [(0, n_keys)], scale,
                                  torch.from_numpy(limits.astype(np.int32)).cuda(), out, lse)
        o_ref, lse_ref = np.empty_like(q_ref), np.empty((H, n_q))
        for lim in np.unique(limits):
            rows = limits == lim
            o_ref[rows], lse_ref[:, rows] = oracle.attention(q_ref[rows], kf[:lim], vf[:lim], Hn.SCALE)
    torch.cuda.synchronize()
    Hn.assert_close("o", Hn.bits_to_f64(Hn.dev_bits(out)), o_ref)
    # fp32 scores of magnitude s carry an error of a few 2^-24 * s
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref) / np.maximum(1.0, np.abs(lse_ref))) <= 2e-5


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("n_keys", [1, 31, 32, 33, 64, 65, 127, 128, 129, 192, 256, 257, 383, 640])
def test_key_edges(P, waves, n_keys):
    for folded in (False, True):
        _case(P, waves, 1, 65, n_keys, folded)
    _case(P, waves, 2, 33, n_keys, True)


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("n_q", [1, 32, 33, 64, 127, 128, 129, 193, 256, 257])
def test_query_edges(P, waves, n_q):
    _case(P, waves, 1, n_q, 300, True)
    _case(P, waves, 3, n_q, 450, False)


@pytest.mark.parametrize("n_keys", [90, 300, 512])
@pytest.mark.parametrize("folded", [False, True])
def test_second_run(P, n_keys, folded):
    for waves in (4, 8):
        for splits in (1, 2):
            _case(P, waves, splits, 140, n_keys, folded, jump_at=70)
    # limits below, inside and beyond the keys that jump
    limits = np.minimum(n_keys, 1 + (np.arange(300) * 7) % (n_keys + 20))
    _case(P, 0, 0, 300, n_keys, folded, limits=limits, jump_at=70)


@pytest.mark.parametrize("H", [1, 5, 8, 12])
def test_limited_work_order(P, H):
    """Every (head, query tile) is worked off once, whatever the head count leaves over on the 8 XCDs; limits
    that rise with the query, fall with it, and neither."""
    n = 600
    i = np.arange(n)
    for limits in (1 + i, n - i, 1 + (i * 37) % n):
        _case(P, 0, 0, n, n, True, limits=limits, H=H)
