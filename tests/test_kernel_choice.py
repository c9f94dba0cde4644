"""Which kernels serve a call (intattn_kernel_choice, host only): both sides of each rule of the automatic choice."""
import ctypes

import numpy as np
import pytest

from paper_2511_21513_amd import binding

SPLIT, SHORT = 6, 7


def choice(ia, B, Hq, Hkv, L, Lkv, d, causal, *, c_int=5203, scale_mode=0, dynamic=False, q_block=0, k_block=0):
    a = binding.Args()
    a.B, a.Hq, a.Hkv, a.L, a.Lkv, a.d, a.causal = B, Hq, Hkv, L, Lkv, d, int(causal)
    a.q, a.k, a.v, a.out = 16, 32, 48, 64  # (not read)
    for name in ("q_stride", "k_stride", "v_stride", "out_stride"):
        setattr(a, name, (ctypes.c_int64 * 3)(d, d, d))
    s_k = 0.03
    scales = [np.full(Hq, s, dtype=np.float32) for s in (6.6 * d**0.5 / (s_k * c_int), s_k, 0.02, 0.004)]
    a.scale_q, a.scale_k, a.scale_v, a.scale_out = (s.ctypes.data for s in scales)
    a.scale_mode, a.q_block, a.k_block = scale_mode, q_block, k_block
    return ia.kernel_choice(a, dynamic)


@pytest.fixture(scope="module")
def ia():
    return binding.IntAttn(device=-1)


CASES = [
    # B, Hq, Hkv, L, Lkv, d, causal, kernel
    (1, 1, 1, 128, 128, 64, False, 3),
    (1, 32, 8, 8192, 8192, 128, True, 5),
    (8, 32, 32, 256, 256, 128, False, 1),
    # few query tiles against many keys
    (1, 32, 8, 509, 7001, 128, True, SPLIT),
    (1, 1, 1, 8192, 8192, 64, True, SPLIT),
    (1, 16, 16, 1024, 1024, 128, True, 3),
    # all scores in registers: enough heads, and enough blocks of 32 rows against variant 3
    (16, 8, 8, 197, 197, 64, False, SHORT),
    (15, 8, 8, 197, 197, 64, False, 3),
    (16, 8, 8, 192, 192, 64, False, 3),
    (16, 8, 8, 96, 96, 64, True, SHORT),
    (16, 8, 8, 64, 64, 64, True, 3),
    (16, 8, 8, 96, 200, 64, True, 3),
    (48, 8, 8, 32, 32, 64, False, SHORT),
    (128, 12, 12, 256, 256, 64, False, SHORT),
    (128, 12, 12, 257, 257, 64, False, 1),
    (128, 12, 12, 256, 256, 128, False, 1),
    # one decoded token
    (1, 32, 8, 1, 1024, 128, True, 9),
    (1, 32, 8, 1, 1023, 128, True, 3),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B{}Hq{}Hkv{}L{}Lk{}d{}c{:d}".format(*c[:7]))
def test_automatic_choice(ia, case):
    *shape, want = case
    got, split_rows, split_pv = choice(ia, *shape)
    assert got == want
    assert (split_rows >= 1 and 1 <= split_pv <= 16) if want == SPLIT else (split_rows, split_pv) == (0, 0)


def test_forms_that_a_rule_does_not_take(ia):
    chunk, short = (1, 32, 8, 509, 7001, 128, True), (128, 12, 12, 197, 197, 64, False)
    assert choice(ia, *chunk, scale_mode=1, dynamic=True)[0] == SPLIT
    assert choice(ia, *chunk, scale_mode=2, dynamic=True, q_block=64)[0] == SPLIT
    for L, causal, want in ((1500, True, 3), (2048, True, 3), (2049, True, 1), (1024, False, 3), (1025, False, 1)):
        assert choice(ia, 1, 32, 32, L, L, 64, causal, scale_mode=2, dynamic=True, q_block=1)[0] == want, (L, causal)
    assert choice(ia, *chunk, scale_mode=3, dynamic=True, q_block=64, k_block=64)[0] == 3
    assert choice(ia, *short, scale_mode=1)[0] == SHORT
    assert choice(ia, *short, dynamic=True)[0] == 1  # device-resident scales
    assert choice(ia, *short, c_int=2**25 + 1)[0] == 1  # a threshold past 2^24
    wide = binding.IntAttn(device=-1, lut_bits=6)
    assert choice(wide, *chunk)[0] == 3 and choice(wide, *short)[0] == 1
    for variant in (1, 2, 3, 4, 5):
        fixed = binding.IntAttn(device=-1, variant=variant)
        assert choice(fixed, *chunk)[0] == variant and choice(fixed, *short)[0] == variant
    four = binding.IntAttn(device=-1, variant=10)
    assert choice(four, 1, 32, 8, 1, 1024, 128, True)[0] == 10


def test_what_a_forward_refuses_is_refused(ia):
    for bad in (dict(d=96), dict(L=0), dict(Hkv=3), dict(Lkv=4)):
        shape = dict(B=1, Hq=4, Hkv=2, L=8, Lkv=8, d=64, causal=True)
        shape.update(bad)
        with pytest.raises(binding.IntAttnError):
            choice(ia, **shape)
    with pytest.raises(binding.IntAttnError):
        choice(ia, 1, 4, 2, 8, 8, 64, True, scale_mode=2, q_block=4)  # host scales have no groups of rows
