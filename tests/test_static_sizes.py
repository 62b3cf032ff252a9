"""Which sizes chunk_attention_static takes.  The size check comes before the pointer check and the pointers
here are null: a refused size returns CROPE_EWORKSPACE, an accepted one gets past it and ends at the missing
GPU or at the null pointer, in any case before a kernel."""
import ctypes

import numpy as np
import pytest

from paper_2603_06664_amd import binding as B

EWORKSPACE = -5


def _static_call(n_q, n_heads, n_keys):
    lib = B._load()
    s = B._Strides(n_heads * 128, 128)
    seg = (B._Segment * 1)(B._Segment(0, n_keys))
    return lib.chunk_attention_static(None, s, n_q, n_heads, None, None, s, n_keys, seg, 1, ctypes.c_float(0.1), None, s,
                                      None, None)


# taken since the entry point exists, though chunk_attention's present division of them needs more than the buffer
@pytest.mark.parametrize("size", [(10800, 12, 10800), (10800, 12, 75600), (5860, 12, 3330), (2632, 48, 15921),
                                  (4913, 13, 98932), (2671, 24, 171152)])
def test_sizes_that_have_to_be_divided_less(size):
    import paper_2603_06664_amd as P
    assert P.chunk_attention_workspace_bytes(*size) > P.chunk_attention_static_capacity()
    assert _static_call(*size) != EWORKSPACE


@pytest.mark.parametrize("size", [(735, 40, 174155), (475, 50, 80721), (500, 64, 100000), (585, 40, 32760), (1020, 16, 20000)])
def test_sizes_that_fit(size):
    import paper_2603_06664_amd as P
    assert P.chunk_attention_workspace_bytes(*size) <= P.chunk_attention_static_capacity()
    assert _static_call(*size) != EWORKSPACE


@pytest.mark.parametrize("size", [(300, 64, 60000), (300, 64, 50000), (350, 64, 80000), (1200, 64, 30000)])
def test_sizes_that_are_refused(size):
    assert _static_call(*size) == EWORKSPACE


# unsplit now, but too large for the buffer in the divisions before
@pytest.mark.parametrize("size", [(2887, 25, 4442), (9402, 9, 6252), (5237, 15, 5422)])
def test_sizes_whose_present_division_fits(size):
    import paper_2603_06664_amd as P
    assert P.chunk_attention_workspace_bytes(*size) == 0
    assert _static_call(*size) != EWORKSPACE


def test_a_size_whose_workspace_fits_is_never_refused():
    """The rule of the header: a refused size needs more scratch than the buffer holds, and the message says how much."""
    import paper_2603_06664_amd as P
    rng = np.random.default_rng(506)
    refused = 0
    for _ in range(20000):
        size = [int(round(np.exp(rng.uniform(np.log(lo), np.log(hi))))) for lo, hi in ((200, 20000), (2, 64), (500, 175000))]
        if _static_call(*size) != EWORKSPACE:
            continue
        refused += 1
        need = P.chunk_attention_workspace_bytes(*size)
        assert need > P.chunk_attention_static_capacity(), size
        assert "needs %d bytes" % need in B.crope_last_error(), size
    assert refused > 100


@pytest.mark.gpu
@pytest.mark.parametrize("folded", [False, True])
def test_call_divided_less_matches_the_oracle(folded):
    """A 1280x720 chunk of three frames (10800 queries, 12 heads) over itself: unsplit here, split in two by
    chunk_attention; a sample of the query rows against the oracle, all of them against chunk_attention."""
    import oracle
    import torch
    import harness as Hn
    import paper_2603_06664_amd as P
    from paper_2603_06664_amd import workloads as W
    n, H = 10800, 12
    rng = np.random.default_rng(505)
    q, k, v = (rng.standard_normal((n, H, 128)).astype(np.float32) for _ in range(3))
    c = np.float32(P.crope_folded_q_scale(Hn.SCALE)) if folded else np.float32(1.0)
    qb, kb, vb = W.f32_to_bf16_bits(q * c), W.f32_to_bf16_bits(k), W.f32_to_bf16_bits(v)
    qd, kd, vd = Hn.to_dev_bf16(qb), Hn.to_dev_bf16(kb), Hn.to_dev_bf16(vb)
    scale = P.CROPE_SCALE_FOLDED if folded else Hn.SCALE
    out, ref = torch.empty_like(qd), torch.empty_like(qd)
    lse = torch.empty((H, n), dtype=torch.float32, device="cuda")
    wsb = P.chunk_attention_workspace_bytes(n, H, n)
    assert wsb > P.chunk_attention_static_capacity()
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    print("static call divided less, folded %d" % folded, flush=True)
    P.chunk_attention_static(qd, n, H, kd, vd, n, [(0, n)], scale, out, lse)
    P.chunk_attention(qd, n, H, kd, vd, n, [(0, n)], scale, ref, None, ws, wsb)
    torch.cuda.synchronize()
    got = Hn.bits_to_f64(Hn.dev_bits(out))
    Hn.assert_close("o", got, Hn.bits_to_f64(Hn.dev_bits(ref)))
    rows = np.unique(np.concatenate([[0, 127, 128, 255, 256, n - 1], rng.integers(0, n, 18)]))
    o_ref, lse_ref = oracle.attention(Hn.bits_to_f64(qb)[rows] / float(c), Hn.bits_to_f64(kb), Hn.bits_to_f64(vb), Hn.SCALE)
    Hn.assert_close("o", got[rows], o_ref)
    assert np.max(np.abs(lse.cpu().numpy()[:, rows] - lse_ref)) <= 2e-5 * np.max(np.abs(lse_ref))
