"""The index map in double precision, for thresholds without a single-precision factor: exact by rational arithmetic at both sides
of every step (host only); which kernels serve calls that need it, for all heads or for some; and on the GPU, with logits at the
steps themselves and ties among them, against the oracle in every kernel that holds it."""
import math
import struct
from fractions import Fraction

import numpy as np
import pytest

from test_fma_map_gpu import has_factor, without_factor
from test_kernel_choice import SHORT, SPLIT, choice
from test_mixed_heads import mixed_args
from test_parity_gpu import torch_mod  # noqa: F401


def steps(c, top):
    """Distances on both sides of every step of round(delta top / c), and the ends."""
    at = [-(-(2 * k - 1) * c // (2 * top)) for k in range(1, top + 1)]
    return sorted({0, min(c, 1 << 22)} | {d for t in at for d in (t - 1, t, t + 1) if 0 <= d <= min(c, 1 << 22)})


@pytest.mark.parametrize("top", [1, 3, 7, 15, 31, 63])
def test_form_is_exact(top):
    rng = np.random.default_rng(top)
    cs = [*range(1, 70), 62 * 4000, 126 * 3000, 255, 256, 257, (1 << 22), (1 << 24) - 1, 1 << 24, (1 << 24) + 1, 31 << 20, 63 << 20, (1 << 28) + 2, (1 << 29) + 1, 1 << 30,
          *(int(x) for x in np.exp(rng.uniform(np.log(70), np.log(2**30), 60)))]
    for c in cs:
        q = math.nextafter(top / c, math.inf) if hasattr(math, "nextafter") else float(np.nextafter(top / c, np.inf))
        r = q - math.ldexp(q, -31 if c <= 1 << 24 else -31 - bin(top).count("1"))
        for delta in steps(c, top):
            y = Fraction(c - delta) * Fraction(r) + Fraction(1, 2)
            place = int(Fraction(round(y * 2**32), 2**32))  # half to even, then the integer part
            assert place == top - (2 * top * delta + c) // (2 * c), (c, delta)
        if c > top:  # the form without a conversion adds 2^20 + 1/2 - 2^52 r, which has to be a double
            b = 1048576.5 - 4503599627370496.0 * r
            assert Fraction(b) == Fraction(1048576.5) - 2**52 * Fraction(r)
            scaled = 1048576.5 * 2.0**45 - 4503599627370496.0 * (r * 2.0**45)  # the same 2^45 times as large
            assert Fraction(scaled) == 2**45 * Fraction(b)
    assert struct.pack(">d", 2.0**65)[:4] == bytes.fromhex("44000000") and (0x44000000 << 7) % 2**32 == 0


def test_small_thresholds_have_a_factor():
    """The head of a mixed call that is mapped in double has a threshold above the last table index."""
    for top in (1, 3, 7, 15, 31, 63):
        assert all(has_factor(c, top) for c in range(1, 2 * top + 2))


def test_short_sequences_keep_their_kernel():
    from paper_2511_21513_amd import binding

    none = without_factor(31)
    ia = binding.IntAttn(device=-1)
    for c in (none, 648522, 1 << 24):
        assert choice(ia, 128, 12, 12, 197, 197, 64, False, c_int=c)[0] == SHORT
    args, keep = mixed_args(1536, 197, 64, False, [5203, none, 47011])
    assert ia.kernel_choice(args)[0] == SHORT


# B, Hq, Hkv, Lq, Lk, d, causal, variant, kernel (None: not asked)
SHAPES = [
    (1, 4, 2, 161, 161, 64, True, 1, None), (1, 4, 4, 97, 300, 128, False, 1, None), (1, 4, 2, 70, 300, 64, False, 2, None), (1, 4, 2, 161, 161, 64, True, 3, None),
    (1, 4, 4, 40, 300, 128, False, 3, None), (1, 4, 2, 140, 300, 128, True, 4, None), (1, 4, 2, 140, 300, 64, True, 5, None), (1, 4, 4, 70, 2100, 128, True, 5, None),
    (1, 4, 2, 33, 3000, 128, False, 0, SPLIT), (1, 4, 1, 1, 1100, 128, True, 9, 9), (1, 4, 2, 3, 1100, 64, True, 10, 10),
    (96, 4, 4, 70, 100, 64, False, 0, SHORT), (48, 4, 4, 130, 200, 64, True, 0, SHORT), (104, 4, 4, 33, 240, 64, False, 0, SHORT),
]
C_INTS = {
    "none": [None], "past 2^22": [1 << 22], "ties": [62 * 63 * 100], "2^24": [1 << 24], "2^25": [(1 << 25) + 2], "2^30": [1 << 30],
    "heads": [None, 5203, 1, 62 * 63 * 200], "heads past 2^23": [47011, 1 << 27, None, 30],
}


@pytest.mark.gpu
@pytest.mark.parametrize("which", C_INTS)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{:d}v{}".format(*s[:8]))
@pytest.mark.parametrize("lut_bits", [5, 6])
def test_logits_at_the_steps_bit_exact(torch_mod, oracle, lut_bits, shape, which):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, Hq, Hkv, lq, lk, d, causal, variant, kernel = shape
    if lut_bits == 6 and kernel in (SHORT, SPLIT):
        pytest.skip("tables of at most 32 entries")
    top = (1 << lut_bits) - 1
    c_ints = [without_factor(top) if c is None else c for c in C_INTS[which]]
    per_head = len(c_ints) > 1
    n, nk = (Hq, Hkv) if per_head else (1, 1)
    print(f"thresholds {c_ints} {shape} b {lut_bits}", flush=True)
    ia = binding.IntAttn(device=0, variant=variant, lut_bits=lut_bits)
    s_k = np.full(nk, 0.0003, dtype=np.float32)
    s_q = np.array([6.6 * d**0.5 / (float(s_k[0]) * c_ints[h % len(c_ints)]) for h in range(n)], dtype=np.float32)
    s_v, s_o = np.full(nk, 0.02, dtype=np.float32), np.full(n, 0.001, dtype=np.float32)
    c_got = [ia.derive_params(float(s_q[h % n]), float(s_k[0]), 0.02, 0.001, d)[0] for h in range(Hq)]
    assert all(abs(c_got[h] - c_ints[h % len(c_ints)]) <= c_ints[h % len(c_ints)] * 2**-23 for h in range(Hq))
    # every row of Q is 127 but for a 1 in the last channel, so that a key can be given any score: the greatest less a distance at a
    # step.  KV heads serve the steps of their query heads in turn; the keys that remain are random.
    rng = np.random.default_rng(lk)
    q = np.full((B, Hq, lq, d), 127, dtype=np.int8)
    q[..., d - 1] = 1
    k = rng.integers(-128, 128, (B, Hkv, lk, d)).astype(np.int8)
    v = rng.integers(-128, 128, (B, Hkv, lk, d)).astype(np.int8)
    most = 127 * 127 * (d - 1) + 63
    for kv in range(Hkv):
        want = sorted({x for h in range(kv * Hq // Hkv, (kv + 1) * Hq // Hkv) for x in steps(c_got[h], top) if x <= 2 * most - 255})
        want = [want[i] for i in np.linspace(0, len(want) - 1, min(len(want), lk - lq + 1 if causal else lk)).round().astype(int)]
        for i, delta in enumerate(want):
            score = most - delta
            last = (score + 63) % 127 - 63
            rest = (score - last) // 127
            assert rest * 127 + last == score
            row = np.full(d - 1, rest // (d - 1))
            row[: rest - (d - 1) * (rest // (d - 1))] += 1  # (127 (d - 1) at most)
            k[:, kv, i, : d - 1], k[:, kv, i, d - 1] = row, last
            assert np.abs(row).max() <= 127
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=causal, per_head=per_head, lut_bits=lut_bits, taps=True, threads=16)
    tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
    for device_scales in (False, True):
        out = torch.full_like(tq, 99)
        sums = torch.full((B, Hq, lq), -1, dtype=torch.int32, device="cuda")
        args, keep = ia.make_args(tq, tk, tv, out, *(sc if device_scales else (s_q, s_k, s_v, s_o)), causal=causal, per_head=per_head,
                                  device_scales=device_scales, row_sum=sums)
        if kernel and not device_scales and max(c_got) <= 1 << 24:
            assert ia.kernel_choice(args)[0] == kernel
        (ia.forward_dynamic_args if device_scales else ia.forward_args)(args, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert int((sums.cpu().numpy() != want["row_sum"]).sum()) == 0, device_scales
        assert int((out.cpu().numpy() != want["out"]).sum()) == 0, device_scales
    ia.close()


@pytest.mark.gpu
@pytest.mark.parametrize("variant, d, causal", [(1, 64, True), (2, 128, False), (3, 64, False), (3, 128, True), (4, 64, False), (5, 128, True), (5, 64, False)])
def test_row_groups_of_any_threshold_bit_exact(torch_mod, oracle, variant, d, causal):  # noqa: F811
    """A threshold from 1 to 2^30 for every 8 query rows, in one wave."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(d + variant)
    lq, lk, qb = 150, 200, 8
    q, k, v = (rng.integers(-128, 128, (1, h, n, d), dtype=np.int8) for h, n in ((4, lq), (2, lk), (2, lk)))
    q[:, :, 3::7] //= 32
    c = np.exp(rng.uniform(0, np.log(2.0**30), (1, 4, -(-lq // qb))))
    c[0, :, :5] = [1, 31, 62, 1 << 24, 1 << 30]
    s_k = np.full(2, 0.0003, dtype=np.float32)
    s_q = (6.6 * d**0.5 / (0.0003 * c)).astype(np.float32)
    s_v, s_o = np.full(2, 0.02, dtype=np.float32), np.full(s_q.shape, 0.001, dtype=np.float32)
    want = oracle.forward_row_groups(q, k, v, s_q, s_k, s_v, s_o, q_block=qb, causal=causal)["out"]
    tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
    out = torch.full_like(tq, 99)
    ia = binding.IntAttn(device=0, variant=variant)
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=causal, device_scales=True, q_block=qb)
    ia.forward_dynamic_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()
