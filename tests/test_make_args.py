"""What make_args puts into the fields of Args (host only): strides of other layouts, scale arrays in every form that is taken and
the memory that they are read from, and what is refused."""
import ctypes

import numpy as np
import pytest

from paper_2511_21513_amd import binding

FORMS = {
    "float32": lambda x: x,
    "read-only": lambda x: np.frombuffer(x.tobytes(), dtype=np.float32),
    "float64": lambda x: x.astype(np.float64),
    "other byte order": lambda x: x.astype(">f4"),
    "list": lambda x: x.tolist(),
    "strided": lambda x: np.repeat(x, 2)[::2],
    "column": lambda x: x.reshape(-1, 1),
}


@pytest.fixture(scope="module")
def ia():
    return binding.IntAttn(device=-1)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("per_head", [False, True])
def test_fields(ia, form, per_head):
    torch = pytest.importorskip("torch")
    B, Hq, Hkv, L, Lk, d = 2, 6, 3, 5, 9, 64
    q = torch.zeros((B, L, Hq, d + 16), dtype=torch.int8)[..., :d].transpose(1, 2)
    k, v = (torch.zeros((B, Hkv, Lk, d), dtype=torch.int8) for _ in range(2))
    out, sums = torch.zeros((B, Hq, L, d), dtype=torch.int8), torch.zeros((B, Hq, L), dtype=torch.int32)
    want = [np.arange(1, (n if per_head else 1) + 1, dtype=np.float32) / 64 for n in (Hq, Hkv, Hkv, Hq)]
    given = [FORMS[form](x) for x in want]
    a, keep = ia.make_args(q, k, v, out, *given, causal=1, per_head=per_head, row_sum=sums)
    assert (a.B, a.Hq, a.Hkv, a.L, a.Lkv, a.d, a.causal, a.scale_mode, a.q_block, a.k_block) == (B, Hq, Hkv, L, Lk, d, 1, int(per_head), 0, 0)
    for name, t in (("q", q), ("k", k), ("v", v), ("out", out)):
        assert getattr(a, name) == t.data_ptr() and tuple(getattr(a, name + "_stride")) == t.stride()[:3]
    assert (a.dbg_row_max, a.dbg_row_sum, a.dbg_acc) == (None, sums.data_ptr(), None)
    for name, x, y in zip(("scale_q", "scale_k", "scale_v", "scale_out"), want, keep):
        assert getattr(a, name) == y.ctypes.data and y.dtype == np.float32
        assert np.array_equal(np.ctypeslib.as_array((ctypes.c_float * x.size).from_address(getattr(a, name))), x)
    if form == "float32":  # read where it lies, not copied
        assert all(x is y for x, y in zip(given, keep))
    assert ia.make_args(q, k, v, out, *given[:3], per_head=per_head)[0].scale_out is None


def test_refused(ia):
    torch = pytest.importorskip("torch")
    q, k, s = torch.zeros((1, 4, 8, 64), dtype=torch.int8), torch.zeros((1, 2, 8, 64), dtype=torch.int8), np.ones(1, np.float32)
    for bad in (dict(q_block=2), dict(k_block=2), dict(per_head=True), dict(device_scales=True)):
        with pytest.raises((ValueError, AttributeError)):
            ia.make_args(q, k, k, q, s, s, s, **bad)
    with pytest.raises(ValueError):
        ia.make_args(q, k, k[:, :1], q, s, s, s)
    with pytest.raises(ValueError):
        ia.make_args(q, k, k, torch.zeros((1, 4, 8, 128), dtype=torch.int8)[..., ::2], s, s, s)
    with pytest.raises(AttributeError):
        ia.make_args(q, k, k, q, None, s, s)
