"""The table of constants that a workgroup of the kernels with the keys split over waves keeps for key groups: up to 64 blocks of
keys, where it takes the workgroup past 64 KiB of LDS at a head dimension of 128, and one block more, which goes without;
compared with the oracle."""
import pytest

from test_parity_gpu import key_group_forward, key_group_problem, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lut_bits", [5, 6])
@pytest.mark.parametrize("lq, lk, d, causal, kb", [(40, 1280, 128, True, 32),   # 40 blocks
                                                   (33, 2016, 128, False, 32),  # 63
                                                   (40, 2048, 128, True, 32), (33, 4050, 128, False, 64), (40, 2037, 64, True, 32),  # 64
                                                   (40, 2049, 128, True, 32), (33, 4097, 128, False, 64), (40, 2049, 64, False, 32)])  # 65
def test_bit_exact_around_the_limit(torch_mod, oracle, lq, lk, d, causal, kb, lut_bits):  # noqa: F811
    from paper_2511_21513_amd import binding

    print(f"case {lq} x {lk} d {d} causal {causal} k_block {kb} b {lut_bits}", flush=True)
    q, k, v, s_q, s_k, s_v, s_o = key_group_problem(lk, 1, 2, 1, lq, lk, d, 16, kb, True)
    want = oracle.forward_groups(q, k, v, s_q, s_k, s_v, s_o, q_block=16, k_block=kb, causal=causal, lut_bits=lut_bits, taps=True)
    ia = binding.IntAttn(device=0, variant=3, lut_bits=lut_bits)
    out, taps, status = key_group_forward(torch_mod, ia, q, k, v, s_q, s_k, s_v, s_o, causal, 16, kb)
    ia.close()
    assert status == 0
    for key in ("row_sum", "acc"):
        assert int((taps[key] != want[key]).sum()) == 0, key
    assert int((out != want["out"]).sum()) == 0
