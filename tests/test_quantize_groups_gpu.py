"""Quantizer with a scale per block of rows: teams of 16 lanes, a wave and a workgroup, groups that are held and groups that are
read twice, partial last groups and padded rows; the two-pass quantizer on few and many rounds a workgroup.  Bit-compared with
the oracle."""
import numpy as np
import pytest

from test_parity_gpu import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

TYPES = {"float32": np.float32, "float16": np.float16}


def source(torch, rng, B, H, L, d, dtype, pad):
    x = (rng.standard_normal((B, H, L, d + pad)) * np.exp(rng.normal(0, 1, (B, H, L, 1)))).astype(TYPES[dtype])
    return x[..., :d], torch.from_numpy(x).cuda()[..., :d]


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("L, d, q_block", [(37, 64, 1), (37, 128, 2), (9, 128, 3), (50, 64, 5), (70, 128, 31), (70, 128, 32), (70, 128, 33), (300, 64, 64),
                                           (260, 128, 128), (260, 128, 129), (700, 128, 300), (130, 8, 1), (20, 136, 7)])
def test_row_groups(torch_mod, oracle, L, d, q_block, dtype, pad):  # noqa: F811
    from paper_2511_21513_amd import binding

    x, tx = source(torch_mod, np.random.default_rng(L + d), 2, 3, L, d, dtype, pad)
    ia = binding.IntAttn(device=0)
    got, scales = ia.quantize(tx, q_block=q_block)
    torch_mod.cuda.synchronize()
    want, want_scales = oracle.quantize_row_groups(np.ascontiguousarray(x).astype(np.float32), q_block)
    assert np.array_equal(scales.cpu().numpy().reshape(-1), np.asarray(want_scales, dtype=np.float32).reshape(-1))
    assert np.array_equal(got.cpu().numpy(), want)
    ia.close()


@pytest.mark.parametrize("B, H, L, d, per_head", [(1, 1, 5, 64, False), (1, 8, 1024, 128, True), (2, 24, 1366, 128, False), (3, 32, 2050, 128, True)])
def test_two_passes(torch_mod, oracle, B, H, L, d, per_head):  # noqa: F811
    from paper_2511_21513_amd import binding

    x, tx = source(torch_mod, np.random.default_rng(L), B, H, L, d, "float16", 0)
    ia = binding.IntAttn(device=0)
    got, scales = ia.quantize(tx, per_head=per_head)
    torch_mod.cuda.synchronize()
    want, want_scales = oracle.quantize(x.astype(np.float32), per_head=per_head)
    assert np.array_equal(scales.cpu().numpy().reshape(-1), np.asarray(want_scales, dtype=np.float32).reshape(-1))
    assert np.array_equal(got.cpu().numpy(), want)
    ia.close()
