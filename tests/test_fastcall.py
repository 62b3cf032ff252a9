"""The extension that marshals the per-chunk calls hands the library what ctypes would hand it: the same values for
every kind of argument that it takes itself, and the same exceptions for those that it leaves to ctypes."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_06664_amd import binding as B

NAMES = ["crope_qk_norm_rotate_append", "crope_qk_norm_rotate_append_qscaled", "chunk_attention", "chunk_attention_planned",
         "chunk_attention_static", "chunk_attention_limited", "crope_qkv_project_norm_rotate_append"]


def _value(x):
    if isinstance(x, ctypes.Structure):
        return tuple(getattr(x, f) for f, _ in x._fields_)
    return x


class Recorder:
    """A library whose functions note their arguments."""

    def __init__(self, real):
        self.calls, self.keep = [], []
        for name in NAMES:
            f = getattr(real, name)
            types = list(f.argtypes)

            def note(*args, name=name):
                vals = [_value(a) for a in args]
                if name == "chunk_attention_planned" or name.startswith("chunk_attention"):
                    n = vals[9]
                    vals[8] = [(args[8][i].start, args[8][i].len) for i in range(n)]
                if name == "chunk_attention_planned":
                    vals[11] = (0, 0) if not args[11] else (args[11][0].waves, args[11][0].splits)
                if isinstance(args[0], ctypes.POINTER(B._Desc)):
                    vals[0] = _value(args[0][0])
                self.calls.append((name, vals))
                return 0

            cb = ctypes.CFUNCTYPE(ctypes.c_int, *types)(note)
            cb.argtypes = types
            self.keep.append(cb)
            setattr(self, name, cb)


class NoFast:
    def __getattr__(self, _):
        return lambda *a: NotImplemented


@pytest.fixture
def both(monkeypatch):
    """run(f): the calls or the exception of f through the extension and through ctypes."""
    real = B._load()
    rec = Recorder(real)
    fast = B._load_fastcall(rec)
    plain = []
    watched = type("Watched", (), {n: staticmethod(lambda *a, f=getattr(fast, n): plain.append(f(*a)) or plain[-1])
                                   for n in ("append", "append_qscaled", "attention", "attention_planned",
                                             "attention_static", "attention_limited", "project")})
    monkeypatch.setattr(B, "_lib", rec)

    def run(f):
        out = []
        for mod in (watched, NoFast()):
            monkeypatch.setattr(B, "_fast", mod)
            rec.calls.clear()
            try:
                f()
                out.append(list(rec.calls))
            except Exception as e:
                out.append((type(e), str(e)))
        assert out[0] == out[1]
        return out[0], plain[-1] is not NotImplemented
    yield run
    B._load_fastcall(real)   # the extension's addresses are the process's: back to the library's


def _t(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype)


def _tensors(H=3, n=5, cap=9):
    fused = _t(n, 3, H, 128)
    return dict(tab=_t(64, dtype=torch.float32), q=fused[:, 0], k=fused[:, 1], v=fused[:, 2], g=_t(H * 128, dtype=torch.float32),
                qo=_t(n, H, 128), kc=_t(cap, H, 128), vc=_t(cap, H, 128), out=_t(n, H + 1, 128)[:, 1:],
                lse=_t(H, n, dtype=torch.float32), ws=torch.zeros(4096, dtype=torch.uint8), lim=_t(n, dtype=torch.int32))


def _append(t, scaled, desc=B.TableDesc(), eps=1e-6, dst=4, stream=7, **over):
    t = {**t, **over}
    args = [desc, t["tab"], t["q"], t["k"], t["v"], t["g"], t["g"], eps, 384, 5, 3, 2, 3, 1, 0]
    tail = [t["qo"], t["kc"], t["vc"], 9, dst]
    if scaled:
        return lambda: B.crope_qk_norm_rotate_append_qscaled(*args, 0.127, *tail, stream=stream)
    return lambda: B.crope_qk_norm_rotate_append(*args, *tail, stream=stream)


def _attend(t, kind, n_q=5, segs=((0, 4), (6, 3)), scale=0.25, lse=True, ws=True, plan=(8, 2), stream=None, **over):
    t = {**t, **over}
    head = [t["q"], n_q, 3, t["kc"], t["vc"], 9, segs if isinstance(segs, np.ndarray) else list(segs), scale]
    lse = t["lse"] if lse else None
    w = t["ws"] if ws else None
    return {"": lambda: B.chunk_attention(*head, t["out"], lse, w, stream=stream),
            "planned": lambda: B.chunk_attention_planned(*head, plan, t["out"], lse, w, 1000, stream=stream),
            "static": lambda: B.chunk_attention_static(*head, t["out"], lse, stream=stream),
            "limited": lambda: B.chunk_attention_limited(*head, t["lim"], t["out"], lse, stream=stream)}[kind]


def _project(t, bias=True, x=None, w=None, ws=True):
    x = _t(5, 2, 128)[:, 0] if x is None else x
    w = _t(9 * 128, 128) if w is None else w
    b = _t(9 * 128, dtype=torch.float32) if bias else None
    return lambda: B.crope_qkv_project_norm_rotate_append(B.TableDesc(), t["tab"], x, w, b, 128, t["g"], t["g"], 1e-6, 128, 5, 3,
                                                          2, 3, 1, 0, t["qo"], t["kc"], t["vc"], 9, 4,
                                                          t["ws"] if ws else None, stream=11)


def test_plain_arguments_take_the_extension(both):
    t = _tensors()
    cases = [_append(t, s) for s in (False, True)] + [_project(t), _project(t, bias=False, ws=False)]
    cases += [_attend(t, k, lse=a, ws=w) for k in ("", "planned", "static", "limited") for a in (True, False) for w in (True, False)]
    cases += [_attend(t, "planned", plan=None), _attend(t, "", segs=[(2, 7)], scale=0.0), _attend(t, "", segs=[])]
    cases += [_append(t, True, desc=B.TableDesc(theta=500.0, max_t=64, dim_t=40, dim_h=44, dim_w=44))]
    for f in cases:
        calls, fast = both(f)
        assert fast and len(calls) == 1, calls


class Fake:
    def __init__(self, shape, bad=False):
        self.shape, self.bad = shape, bad

    def data_ptr(self):
        return 0x10000

    def dim(self):
        return len(self.shape)

    def stride(self, i):
        return [self.shape[1] * 128, 128, 2 if self.bad else 1][i]


def test_other_arguments_take_ctypes(both):
    t = _tensors()
    f32 = np.float32(0.25)
    cases = [_append(t, True, eps=f32), _append(t, True, dst=np.int64(4)), _append(t, False, eps=1),
             _append(t, False, k=_t(5, 3, 128)),                     # q, k, v must share strides
             _append(t, False, q=_t(5, 384)), _append(t, False, qo=_t(5, 3, 256)[:, :, ::2]),
             _append(t, False, vc=_t(9, 4, 128)[:, 1:]), _append(t, True, tab=None), _append(t, True, q=Fake((5, 3, 128))),
             _append(t, False, stream=type("S", (), {"cuda_stream": 5})(), q=Fake((5, 3, 128), True)),
             _append(t, False, dst=1 << 70), _append(t, False, dst="4"), _append(t, False, desc=None),
             _append(t, False, desc=B.TableDesc(theta=10000)),
             _attend(t, "", segs=np.array([[0, 4], [6, 3]])), _attend(t, "", segs=[[0, 4]]), _attend(t, "", segs=[(0, 4.7)]),
             _attend(t, "", segs=[(0, 1)] * 20), _attend(t, "static", n_q=True), _attend(t, "static", scale=1), _attend(t, "limited", lim=None),
             _attend(t, "", n_q=1 << 40), _attend(t, "", out=Fake((5, 3, 128))),
             _project(t, x=_t(5, 2, 128)), _project(t, x=_t(128, 5).t()), _project(t, w=_t(128, 9 * 128).t())]
    for i, f in enumerate(cases):
        _, fast = both(f)
        assert not fast, i


def test_a_tensor_without_storage_is_refused_as_before(both):
    t = _tensors()

    def f(row):
        _append(t, False, tab=row)()
        return row
    both(lambda: torch.func.vmap(f)(torch.zeros(2, 4)))
