"""The index map that the device picks for thresholds it learns from device-resident scales: the factor of the fma map that it
searches, the map in double precision where a head has none, and the single-precision map of key groups on both sides of
its limit; bit-compared with the oracle."""
import numpy as np
import pytest

from test_fma_map_gpu import without_factor
from test_parity_gpu import key_group_forward, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

D = 64


def scales_for(c_int):
    """(s_q, s_k) whose threshold round(6.6 sqrt(64) / (s_q s_k)) is c_int."""
    s_k = np.float32(0.03)
    s_q = np.float32(6.6 * 8.0 / (float(s_k) * c_int))
    got = int(np.floor(6.6 / ((float(s_q) * float(s_k)) / 8.0) + 0.5))
    assert got == c_int
    return s_q, s_k


def qkv(rng, B, H, L):
    return [rng.integers(-127, 128, (B, H, L, D), dtype=np.int8) for _ in range(3)]


THRESHOLDS = [
    [5203],                          # per tensor: one wave derives for every head
    [47011],
    [None],                          # no single-precision factor
    [900, 5203, 33, 12000, 1],
    [5203, 47011, 30011, 61, 55064],
    [5203, None, 47011],             # one head without a factor: that one in double precision
    [5203, 47011] * 9,
    [5203, 47011] * 17,
    [5203] * 33 + [None, 2**25 + 1],
]


@pytest.mark.parametrize("variant", [0, 1, 3, 4, 5, 9], ids=lambda v: f"variant{v}")
@pytest.mark.parametrize("which", range(len(THRESHOLDS)))
def test_device_scales_bit_exact(torch_mod, oracle, which, variant):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    c_ints = [without_factor(31) if c is None else c for c in THRESHOLDS[which]]
    per_head = len(c_ints) > 1
    H, L, lq = (len(c_ints) if per_head else 2), 161, (1 if variant == 9 else 161)
    print(f"case {c_ints} variant {variant}", flush=True)
    rng = np.random.default_rng(which)
    q, k, v = qkv(rng, 1, H, L)
    q = np.ascontiguousarray(q[:, :, L - lq:])
    s_q, s_k = (np.array(x, dtype=np.float32) for x in zip(*(scales_for(c) for c in c_ints)))
    s_v = np.full(len(c_ints), 0.02, dtype=np.float32)
    s_o = np.full(len(c_ints), 0.004, dtype=np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=True, per_head=per_head)["out"]
    assert np.abs(want).max() > 5
    ia = binding.IntAttn(device=0, variant=variant)
    tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
    out = torch.full_like(tq, 99)
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=True, per_head=per_head, device_scales=True)
    ia.forward_dynamic_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


@pytest.mark.parametrize("lut_bits", [5, 6])
@pytest.mark.parametrize("variant", [1, 3], ids=lambda v: f"variant{v}")
@pytest.mark.parametrize("k_block", [0, 1, 32, 64])
def test_single_precision_map_on_both_sides_of_its_limit(torch_mod, oracle, k_block, variant, lut_bits):  # noqa: F811
    """Groups whose thresholds lie at, below and above the limit of the single-precision map, small ones among them; waves
    with one kind only and waves with both."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    limit = 75000 if lut_bits == 5 else 37000
    rng = np.random.default_rng(k_block + variant)
    L, qb = 161, 16
    q, k, v = qkv(rng, 1, 2, L)
    targets = [limit - 1, limit, limit + 1, 1, 62, 5203, limit - 7, 3 * limit, limit // 2, 2**20, 100]
    s_q = np.zeros((1, 2, len(targets)), dtype=np.float32)
    for i, c in enumerate(targets):
        s_q[0, 0, i], s_k0 = scales_for(c)
        s_q[0, 1, i] = scales_for(max(1, min(c, limit)))[0]
    s_v = np.full(2, 0.02, dtype=np.float32)
    s_o = np.full((1, 2, len(targets)), 0.004, dtype=np.float32)
    ia = binding.IntAttn(device=0, variant=variant, lut_bits=lut_bits)
    if k_block:
        nkb = -(-L // k_block)
        s_k = np.full((1, 2, nkb), s_k0, dtype=np.float32)
        s_k[0, :, 1::3] *= np.float32(0.5)
        want = oracle.forward_groups(q, k, v, s_q, s_k, s_v, s_o, q_block=qb, k_block=k_block, causal=True, lut_bits=lut_bits)["out"]
        out, _, status = key_group_forward(torch, ia, q, k, v, s_q, s_k, s_v, s_o, True, qb, k_block)
    else:
        s_k = np.full(2, s_k0, dtype=np.float32)
        want = oracle.forward_row_groups(q, k, v, s_q, s_k, s_v, s_o, q_block=qb, causal=True, lut_bits=lut_bits)["out"]
        tq, tk, tv, *sc = (torch.from_numpy(x).cuda() for x in (q, k, v, s_q, s_k, s_v, s_o))
        res = torch.full_like(tq, 99)
        args, keep = ia.make_args(tq, tk, tv, res, *sc, causal=True, device_scales=True, q_block=qb)
        ia.forward_dynamic_args(args, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        out, status = res.cpu().numpy(), ia.dynamic_status()
    assert status == 0 and int((out != want).sum()) == 0
    ia.close()
