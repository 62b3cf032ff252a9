"""Per-query limits in the 256-query work-groups, which take over once there are enough of them: the work order over
heads and tiles, unmasked tiles up to each wave's smallest limit, masked ones behind it, key ranges that end at the
work-group's largest limit, and the second run; with and without the log-sum-exp (two instances of the loop)."""
import numpy as np
import pytest

from paper_2603_06664_amd import workloads as W

import harness as Hn

pytestmark = pytest.mark.gpu
H = 40


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2603_06664_amd as pkg
    return pkg


def _limits(kind, n_q, n_keys):
    i = np.arange(n_q)
    return {"rising": np.maximum(1, np.minimum(n_keys, (i // 90 + 1) * n_keys * 90 // n_q)),
            "falling": np.maximum(1, n_keys - i * n_keys // n_q),
            "inside": 1 + (i * 37) % n_keys,
            "first tile": 1 + (i * 5) % min(n_keys, 120),
            "beyond": n_keys + i % 3}[kind]


def _case(P, n_q, n_keys, kind, folded, want_lse, jump_at=None):
    import torch
    import oracle
    print("limited, 256 queries per work-group: n_q %d n_keys %d limits %s folded %d lse %d jump %s"
          % (n_q, n_keys, kind, folded, want_lse, jump_at), flush=True)
    assert P.chunk_attention_choose_plan(n_q, H, n_keys, (0, 1))[0] == 8
    rng = np.random.default_rng(1000 * n_q + n_keys)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for n in (n_q, n_keys, n_keys))
    if jump_at is not None:   # from this key on, scores of about +-200 powers of two
        k[jump_at:] *= 50.0
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = W.f32_to_bf16_bits(q * c), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    pad = np.full((70, H, 128), 0x7FC1, dtype=np.uint16)   # rows behind the visible ones hold NaN
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(np.concatenate([kb, pad])), Hn.to_dev_bf16(np.concatenate([vb, pad]))
    limits = _limits(kind, n_q, n_keys)
    out = torch.empty_like(qd)
    lse = torch.empty((H, n_q), dtype=torch.float32, device="cuda") if want_lse else None
    P.chunk_attention_limited(qd, n_q, H, kd, vd, n_keys + 70, [(0, n_keys)], P.CROPE_SCALE_FOLDED if folded else Hn.SCALE,
                              torch.from_numpy(limits.astype(np.int32)).cuda(), out, lse)
    torch.cuda.synchronize()
    got = Hn.bits_to_f64(Hn.dev_bits(out))
    # every query tile of every head: the edges of its waves, and a stride that meets every lane of a column
    rows = np.unique(np.concatenate([np.arange(0, n_q, 17), *(np.arange(0, n_q, 64) + d for d in (0, 1, 15, 16, 63)), [n_q - 1]]))
    rows = rows[rows < n_q]
    q_ref, kf, vf = Hn.bits_to_f64(qb) / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb)
    o_ref, lse_ref = np.empty((len(rows), H, 128)), np.empty((H, len(rows)))
    lim = np.minimum(limits[rows], n_keys)
    for x in np.unique(lim):
        at = np.nonzero(lim == x)[0]
        o_ref[at], lse_ref[:, at] = oracle.attention(q_ref[rows[at]], kf[:x], vf[:x], Hn.SCALE)
    Hn.assert_close("o", got[rows], o_ref)
    assert np.all(np.isfinite(got))
    if want_lse:   # fp32 scores of magnitude s carry an error of a few 2^-24 * s
        e = np.abs(lse.cpu().numpy()[:, rows] - lse_ref) / np.maximum(1.0, np.abs(lse_ref))
        assert np.max(e) <= 2e-5


@pytest.mark.parametrize("want_lse", [False, True])
@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("n_q,n_keys", [(800, 127), (769, 129), (1000, 417)])
def test_matches_the_oracle(P, n_q, n_keys, folded, want_lse):
    for kind in ("rising", "falling", "inside", "first tile", "beyond"):
        _case(P, n_q, n_keys, kind, folded, want_lse)


@pytest.mark.parametrize("want_lse", [False, True])
@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("n_keys", [300, 400, 520])
def test_second_run(P, n_keys, folded, want_lse):
    """An odd and an even number of tiles, and one that leaves every V buffer last: the offsets are reset."""
    for kind in ("rising", "inside"):
        _case(P, 800, n_keys, kind, folded, want_lse, jump_at=70)
