"""Sweeps A+B with one and with two row blocks a wave, on both sides of the rule between them, and staged tiles of 128 keys
that end inside and at the edge of a part of 64; bit-compared with the oracle."""
import numpy as np
import pytest

from test_parity_gpu import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d, causal, lq, lk", [
    (128, True, 300, 2048), (128, True, 300, 2049), (128, True, 2049, 2049), (128, False, 257, 191), (128, False, 64, 193), (128, True, 129, 129),
    (64, True, 300, 2049), (64, False, 127, 64), (64, False, 33, 65), (64, True, 128, 320),
])
def test_bit_exact(torch_mod, oracle, d, causal, lq, lk):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    print(f"{lq} x {lk} d {d} causal {causal}", flush=True)
    rng = np.random.default_rng(lk)
    q, k, v = (np.clip(rng.normal(0, 30, (1, h, n, d)).round(), -127, 127).astype(np.int8) for h, n in ((2, lq), (1, lk), (1, lk)))
    s = [np.array([x], dtype=np.float32) for x in (0.03, 0.03, 0.02, 0.004)]
    want = oracle.forward(q, k, v, *s, causal=causal)["out"]
    ia = binding.IntAttn(device=0, variant=5)
    got = ia.forward(*(torch.from_numpy(x).cuda() for x in (q, k, v)), *s, causal=causal)
    torch.cuda.synchronize()
    assert np.abs(want).max() > 5 and int((got.cpu().numpy() != want).sum()) == 0
    ia.close()
