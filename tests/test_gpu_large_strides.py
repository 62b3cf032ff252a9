"""Row strides at their limits, where the copies' offsets inside a tile come close to 2^32: the same rows in a compact
buffer give the same bits."""
import pytest

import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2603_06664_amd as pkg
    return pkg


def _normal(gen, *shape):
    import torch
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)


@pytest.mark.parametrize("waves", [4, 8])
def test_cache_rows_2_to_the_24_elements_apart(P, waves):
    import torch
    n_q, H, n_keys, stride = 70, 2, 420, 1 << 24
    print("cache token stride %d, waves %d" % (stride, waves), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(21)
    q, k, v = (_normal(gen, n, H, 128) for n in (n_q, n_keys, n_keys))
    # 130 rows in front of the cache: 4 GB either way of every tile's base belong to this buffer
    arena = torch.empty((130 + n_keys) * stride, dtype=torch.bfloat16, device="cuda")
    k_far = arena.as_strided((n_keys, H, 128), (stride, 128, 1), 130 * stride)
    v_far = arena.as_strided((n_keys, H, 128), (stride, 128, 1), 130 * stride + 1024)
    k_far.copy_(k)
    v_far.copy_(v)
    got = []
    for kc, vc in ((k, v), (k_far, v_far)):
        out, lse = torch.empty_like(q), torch.empty((H, n_q), dtype=torch.float32, device="cuda")
        P.chunk_attention_planned(q, n_q, H, kc, vc, n_keys, [(0, n_keys)], Hn.SCALE, (waves, 1), out, lse)
        torch.cuda.synchronize()
        got.append((out, lse))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("c_in", [64, 320])
def test_projection_rows_2_to_the_22_elements_apart(P, c_in):
    import torch
    from paper_2603_06664_amd import devutil
    n, H, stride = 300, 2, 1 << 22
    print("projection token stride %d, c_in %d" % (stride, c_in), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(22)
    desc, tab = devutil.make_table()
    gain = torch.ones(H * 128, device="cuda")
    x, w = _normal(gen, n, c_in), _normal(gen, 3 * H * 128, c_in)
    x_far = torch.empty(n * stride, dtype=torch.bfloat16, device="cuda").as_strided((n, c_in), (stride, 1))
    x_far.copy_(x)
    got = []
    for rows in (x, x_far):
        q, k, v = (torch.empty((n, H, 128), dtype=torch.bfloat16, device="cuda") for _ in range(3))
        P.crope_qkv_project_norm_rotate_append(desc, tab, rows, w, None, c_in, gain, gain, 1e-6, 128, n, H, 10, 30, 0, 0, q, k, v,
                                               n, 0)
        torch.cuda.synchronize()
        got.append((q, k, v))
    assert all(torch.equal(a, b) for a, b in zip(*got))
