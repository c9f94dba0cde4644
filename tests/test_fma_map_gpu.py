"""The index map of the tiled kernels as one single-precision fma on the score accumulator read as a float: thresholds at both
ends of its range, around the table's steps, and past it (a head without a factor takes the map in double), with
scores at the ends of theirs; bit-compared with the oracle."""
import numpy as np
import pytest

from test_parity_gpu import torch_mod  # noqa: F401

D = 64


def scales_for(c_int):
    """(s_q, s_k) whose threshold round(6.6 sqrt(64) / (s_q s_k)) is c_int."""
    s_k = np.float32(0.03)
    s_q = np.float32(6.6 * 8.0 / (float(s_k) * c_int))
    assert int(np.floor(6.6 / ((float(s_q) * float(s_k)) / 8.0) + 0.5)) == c_int
    return s_q, s_k


def has_factor(c, top):
    """Whether a float near top / c serves: rint(x r) == ceil(top x / c - 1/2) on both sides of every step."""
    k = np.arange(top, dtype=np.int64)
    below = ((2 * k + 1) * c) // (2 * top)
    x = np.concatenate([below, np.minimum(below + 1, c), [0, c]])
    want = -((c - 2 * top * x) // (2 * c))
    quotient = np.float32(top / c).view(np.int32)
    products = [(x.astype(np.float64) * float((quotient - np.int32(u)).view(np.float32))).astype(np.float32) for u in (1, 2, 0, 3, 4, -1)]
    return any((np.rint(y).astype(np.int64) == want).all() for y in products)


def without_factor(top):
    return next(c for c in range(300001, 400000) if not has_factor(c, top))


@pytest.mark.parametrize("top", [1, 7, 31, 63])
def test_small_and_usual_thresholds_have_a_factor(top):
    rng = np.random.default_rng(top)
    for c in [*range(1, 130), *(int(x) for x in np.exp(rng.uniform(np.log(130), np.log(60000), 300)))]:
        assert has_factor(c, top), c


@pytest.mark.parametrize("lut_bits", [1, 3, 5, 6])
def test_factors_of_the_library(lut_bits):
    """The library reports a factor exactly where there is one (an exhaustive search of its first thresholds without one), and each
    serves every distance in [0, c_int]."""
    from paper_2511_21513_amd import binding

    ia = binding.IntAttn(device=-1, lut_bits=lut_bits)
    top = (1 << lut_bits) - 1
    rng = np.random.default_rng(lut_bits)
    cs = [*range(1, 130), 2 * top - 1, 2 * top, 445, 5203, 28794, 47011, 55064, 74999, 131071, 200003,
          *(int(x) for x in np.exp(rng.uniform(np.log(130), np.log(2.0**22), 150))), (1 << 22) - 1, 1 << 22, (1 << 25) + 1]
    for c in cs:
        mode, bits, add, sh = ia.derive_index_map(c, 9)
        assert mode == (9 if c < 1 << 22 and has_factor(c, top) else 0), c
        if mode == 9:
            assert add == 0 and sh == 0
            x = np.arange(c + 1, dtype=np.int64)  # distances
            products = ((c - x).astype(np.float64) * float(np.uint32(bits).view(np.float32))).astype(np.float32)
            np.testing.assert_array_equal(top - np.rint(products).astype(np.int64), (2 * top * x + c) // (2 * c))
    first = {5: 208508, 6: 104204}.get(lut_bits)
    if first:
        assert next(c for c in range(1, 300000) if ia.derive_index_map(c, 9)[0] != 9) == first
        assert not has_factor(first, top)


THRESHOLDS = {
    "smallest": [1, 2, 3, 30],
    "steps": [31, 62, 63, 445],
    "usual": [5203, 28794, 47011, 55064],
    "large": [74999, 131071, 200003],
    "last": [(1 << 22) - 1],
    "past": [1 << 22, 5203],
    "none": [None, 5203, 1],
}


@pytest.mark.gpu
@pytest.mark.parametrize("lut_bits", [5, 6])
@pytest.mark.parametrize("variant, causal, lq, lk", [(1, True, 161, 161), (2, False, 97, 131), (4, True, 129, 300), (5, True, 161, 161),
                                                     (5, False, 65, 257), (5, True, 33, 191), (0, True, 40, 1900)])
@pytest.mark.parametrize("which", THRESHOLDS)
def test_host_and_device_scales_bit_exact(torch_mod, oracle, which, variant, causal, lq, lk, lut_bits):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    c_ints = [without_factor((1 << lut_bits) - 1) if c is None else c for c in THRESHOLDS[which]]
    H = len(c_ints)
    print(f"thresholds {c_ints} variant {variant} {lq} x {lk}", flush=True)
    rng = np.random.default_rng(lk)
    q, k, v = (rng.integers(-128, 128, (1, H, n, D), dtype=np.int8) for n in (lq, lk, lk))
    q[:, :, ::7], k[:, :, ::11], k[:, :, 5::13] = -128, -128, 127  # scores of 2^20 and -127 2^13 in one row
    q[:, :, 1::5] //= 16  # and rows whose scores lie close together
    s_q, s_k = (np.array(x, dtype=np.float32) for x in zip(*(scales_for(c) for c in c_ints)))
    s_v, s_o = np.full(H, 0.02, dtype=np.float32), np.full(H, 0.004, dtype=np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=causal, per_head=True, lut_bits=lut_bits)["out"]
    ia = binding.IntAttn(device=0, variant=variant, lut_bits=lut_bits)
    tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
    got = ia.forward(tq, tk, tv, s_q, s_k, s_v, s_o, causal=causal, per_head=True)
    out = torch.full_like(tq, 99)
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=causal, per_head=True, device_scales=True)
    ia.forward_dynamic_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0
    assert int((got.cpu().numpy() != want).sum()) == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()
