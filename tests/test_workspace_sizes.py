"""A workspace of a size that chunk_attention once asked for is still taken where the present division wants
more: the call runs the fastest division that fits."""
import ctypes

import numpy as np
import pytest

from paper_2603_06664_amd import binding as B

EWORKSPACE = -5
ROW = 130 * 4   # bytes of a query's partial result

# n_q, heads, keys, splits at that time (1 = no workspace)
ONCE = [(545, 44, 15519, 1), (351, 37, 44483, 2), (897, 7, 1794, 2), (4680, 5, 32760, 2), (18720, 12, 131040, 1), (10800, 12, 75600, 2), (9048, 29, 108576, 1),
        (17160, 38, 102960, 1)]


def _bytes(n_q, heads, splits):
    return 0 if splits == 1 else splits * heads * n_q * ROW


def _call(n_q, heads, keys, workspace_bytes, waves=None):
    """The result code with addresses that no kernel ever sees: there is no GPU where this runs."""
    lib = B._load()
    s = B._Strides(heads * 128, 128)
    seg = (B._Segment * 1)(B._Segment(0, keys))
    p = 0x10000
    head = (p, s, n_q, heads, p, p, s, keys, seg, 1, ctypes.c_float(0.1))
    tail = (p, s, None, p if workspace_bytes else None, workspace_bytes, None)
    if waves is None:
        return lib.chunk_attention(*head, *tail)
    return lib.chunk_attention_planned(*head, ctypes.byref(B._Plan(waves, 0)), *tail)


@pytest.fixture
def no_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("made-up addresses: only where no kernel can run")


@pytest.mark.parametrize("n_q,heads,keys,splits", ONCE)
def test_former_size_is_taken(no_gpu, n_q, heads, keys, splits):
    import paper_2603_06664_amd as P
    once = _bytes(n_q, heads, splits)
    assert _call(n_q, heads, keys, once) != EWORKSPACE
    assert _call(n_q, heads, keys, max(once, P.chunk_attention_workspace_bytes(n_q, heads, keys))) != EWORKSPACE
    if once:
        assert _call(n_q, heads, keys, once - 1) == EWORKSPACE
        assert _call(n_q, heads, keys, 0) == EWORKSPACE


def test_pinned_plans(no_gpu):
    """With a pinned work-group size the same holds; a pinned number of splits needs all of its bytes."""
    import paper_2603_06664_amd as P
    size = (4680, 5, 32760)
    assert _call(*size, _bytes(4680, 5, 2), waves=8) != EWORKSPACE
    for plan in ((4, 3), (8, 3), (0, 5)):
        need = P.chunk_attention_planned_workspace_bytes(*size, plan)
        assert need == _bytes(4680, 5, plan[1])
    lib = B._load()
    s = B._Strides(5 * 128, 128)
    seg = (B._Segment * 1)(B._Segment(0, 32760))
    for have, code in ((_bytes(4680, 5, 3) - 1, True), (_bytes(4680, 5, 3), False)):
        rc = lib.chunk_attention_planned(0x10000, s, 4680, 5, 0x10000, 0x10000, s, 32760, seg, 1, ctypes.c_float(0.1),
                                         ctypes.byref(B._Plan(8, 3)), 0x10000, s, None, 0x10000, have, None)
        assert (rc == EWORKSPACE) == code


@pytest.mark.gpu
@pytest.mark.parametrize("folded", [False, True])
@pytest.mark.parametrize("n_q,heads,keys,splits", [(897, 7, 1794, 2), (600, 3, 4000, None)])
def test_smaller_workspace_matches_the_oracle(n_q, heads, keys, splits, folded):
    """The call stays inside the workspace that it was given, and its result is the oracle's."""
    import oracle
    import torch
    import harness as Hn
    import paper_2603_06664_amd as P
    from paper_2603_06664_amd import workloads as W
    need = P.chunk_attention_workspace_bytes(n_q, heads, keys)
    have = need if splits is None else _bytes(n_q, heads, splits)
    assert need > 0 and have <= need
    print("workspace of %d bytes for %d: n_q %d heads %d keys %d folded %d" % (have, need, n_q, heads, keys, folded), flush=True)
    rng = np.random.default_rng(n_q + folded)
    q, k, v = (rng.standard_normal((n, heads, 128)).astype(np.float32) for n in (n_q, keys, keys))
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = W.f32_to_bf16_bits(q * c), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(kb), Hn.to_dev_bf16(vb)
    out, lse = torch.empty_like(qd), torch.empty((heads, n_q), dtype=torch.float32, device="cuda")
    ws = torch.full((need + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    P.chunk_attention(qd, n_q, heads, kd, vd, keys, [(0, keys)], P.CROPE_SCALE_FOLDED if folded else Hn.SCALE, out, lse,
                      ws, have)
    torch.cuda.synchronize()
    assert bool((ws[have:] == 0x5a).all())
    o, lse_ref = oracle.attention(Hn.bits_to_f64(qb) / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb), Hn.SCALE)
    Hn.assert_close("o", Hn.bits_to_f64(Hn.dev_bits(out)), o)
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) <= 2e-5 * np.max(np.abs(lse_ref))
