"""Calls with a scale for each head of which some have no single-precision index factor: those heads alone are mapped in double
precision.  Which kernels serve such a call (host only), and every kernel against the oracle."""
import ctypes

import numpy as np
import pytest

from test_fma_map_gpu import scales_for, without_factor
from test_parity_gpu import torch_mod  # noqa: F401


def mixed_args(H, L, d, causal, c_ints):
    from paper_2511_21513_amd import binding

    a = binding.Args()
    a.B, a.Hq, a.Hkv, a.L, a.Lkv, a.d, a.causal, a.scale_mode = 1, H, H, L, L, d, int(causal), 1
    a.q, a.k, a.v, a.out = 16, 32, 48, 64  # (not read)
    for name in ("q_stride", "k_stride", "v_stride", "out_stride"):
        setattr(a, name, (ctypes.c_int64 * 3)(d, d, d))
    s = [np.array([6.6 * d**0.5 / (0.03 * c_ints[h % len(c_ints)]) for h in range(H)], dtype=np.float32), *(np.full(H, x, dtype=np.float32) for x in (0.03, 0.02, 0.004))]
    a.scale_q, a.scale_k, a.scale_v, a.scale_out = (x.ctypes.data for x in s)
    return a, s


@pytest.mark.parametrize("d, L, heads, causal, want", [(128, 197, 74, False, 1), (128, 1025, 29, True, 5), (64, 1024, 81, True, 5)])
def test_one_head_without_a_factor_leaves_the_choice_alone(d, L, heads, causal, want):
    from paper_2511_21513_amd import binding

    ia = binding.IntAttn(device=-1)
    for c_ints in ([5203], [5203, without_factor(31), 47011]):
        args, keep = mixed_args(heads, L, d, causal, c_ints)
        assert ia.kernel_choice(args)[0] == want, c_ints


@pytest.mark.gpu
@pytest.mark.parametrize("variant, lq, lk, causal", [(0, 150, 150, True), (1, 150, 333, False), (2, 150, 150, True), (3, 150, 333, True), (4, 150, 333, False), (5, 150, 333, True),
                                                     (0, 33, 3000, True), (9, 1, 1100, True), (10, 2, 1100, True)])
def test_bit_exact(torch_mod, oracle, variant, lq, lk, causal):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    c_ints = [5203, without_factor(31), 1, 1 << 23, 61, 47011]
    rng = np.random.default_rng(variant)
    q, k, v = (rng.integers(-128, 128, (2, 6, n, 64), dtype=np.int8) for n in (lq, lk, lk))
    q[:, :, 1::3] //= 16
    s_q, s_k = (np.array(x, dtype=np.float32) for x in zip(*(scales_for(c) for c in c_ints)))
    s_v, s_o = np.full(6, 0.02, dtype=np.float32), np.full(6, 0.002, dtype=np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=causal, per_head=True, threads=16)["out"]
    ia = binding.IntAttn(device=0, variant=variant)
    got = ia.forward(*(torch.from_numpy(x).cuda() for x in (q, k, v)), s_q, s_k, s_v, s_o, causal=causal, per_head=True)
    torch.cuda.synchronize()
    assert int((got.cpu().numpy() != want).sum()) == 0
    ia.close()


@pytest.mark.gpu
@pytest.mark.parametrize("variant, lq, lk, causal", [(2, 12, 59, False), (2, 47, 3, False), (2, 150, 150, False), (2, 300, 333, True), (1, 47, 59, False), (4, 47, 159, False)])
@pytest.mark.parametrize("which", [[None], [5203], [None, 26, 18295], [2, 764260, 2980995]], ids=str)
def test_rows_that_fill_a_wave_in_part_at_head_dimension_128(torch_mod, oracle, which, variant, lq, lk, causal):  # noqa: F811
    """Waves of which some rows lie outside the problem, thresholds of both maps, scales on the host and in device memory."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    H, d = 12, 128
    rng = np.random.default_rng(lk)
    c_ints = [without_factor(31) if c is None else c for c in which]
    q, k, v = (rng.integers(-128, 128, (1, H, n, d), dtype=np.int8) for n in (lq, lk, lk))
    q[:, :, 1::3] //= 16
    s_k = np.full(H, 0.0003, dtype=np.float32)
    s_q = np.array([6.6 * d**0.5 / (0.0003 * c_ints[h % len(c_ints)]) for h in range(H)], dtype=np.float32)
    s_v, s_o = np.full(H, 0.02, dtype=np.float32), np.full(H, 0.002, dtype=np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=causal, per_head=True, threads=16)["out"]
    ia = binding.IntAttn(device=0, variant=variant)
    tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
    for device_scales in (False, True):
        out = torch.full_like(tq, 99)
        args, keep = ia.make_args(tq, tk, tv, out, *(sc if device_scales else (s_q, s_k, s_v, s_o)), causal=causal, per_head=True, device_scales=device_scales)
        (ia.forward_dynamic_args if device_scales else ia.forward_args)(args, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0, device_scales
    ia.close()
