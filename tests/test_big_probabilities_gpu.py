"""Rows whose probabilities pass 127, the largest signed byte the matrix cores take: one dominant key (P = 255), two equal
ones (128 each), and row sums on both sides of the bound up to which a kernel looks for them (510 | 511); bit-compared with
the oracle."""
import numpy as np
import pytest

from test_parity_gpu import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

# table indices of a row's live keys (all others are clipped); LUT_hat[0] = 255, [26] = [27] = 1, [24] = 2
ROWS = {"one": [0], "two equal": [0, 0], "sum 511": [0, 0, 27], "sum 512": [0, 0, 24], "three equal": [0, 0, 0], "one and a near one": [0, 1],
        "one and many": [0] + [20] * 20, "flat": [0] * 60}


@pytest.mark.parametrize("d, variant, heads, causal, lq, lk", [
    (64, 1, 2, True, 70, 70), (64, 2, 2, False, 70, 133), (64, 3, 2, True, 70, 70), (64, 4, 2, False, 70, 133), (64, 5, 2, True, 140, 333), (64, 0, 128, True, 130, 130),
    (64, 0, 128, False, 33, 200), (128, 1, 2, False, 70, 133), (128, 3, 2, True, 70, 70), (128, 5, 2, True, 300, 300), (128, 5, 2, False, 33, 70), (128, 0, 8, True, 40, 3000),
])
def test_bit_exact(torch_mod, oracle, d, variant, heads, causal, lq, lk):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    print(f"d {d} variant {variant} heads {heads} {lq} x {lk}", flush=True)
    rng = np.random.default_rng(lk + heads)
    q, k = (np.zeros((1, heads, n, d), dtype=np.int8) for n in (lq, lk))
    q[..., 0] = 100  # scores are 100 k[0]; the threshold 3100 makes an index of every step of k[0]
    k[..., 0] = -100
    for h in range(heads):
        live = list(ROWS.values())[h % len(ROWS)]
        first = 0 if h % 3 == 0 else min(lk - len(live), 31 + h)  # from the first key on, or across a block of 32
        k[0, h, first:first + len(live), 0] = 60 - np.array(live)
    v = rng.integers(-128, 128, (1, heads, lk, d), dtype=np.int8)
    s_k = np.float32(0.03)
    s_q = np.float32(6.6 * np.sqrt(d) / (float(s_k) * 3100))
    s = [np.array([x], dtype=np.float32) for x in (s_q, s_k, 0.02, 0.02)]
    want = oracle.forward(q, k, v, *s, causal=causal)["out"]
    ia = binding.IntAttn(device=0, variant=variant)
    got = ia.forward(*(torch.from_numpy(x).cuda() for x in (q, k, v)), *s, causal=causal)
    torch.cuda.synchronize()
    assert np.abs(want).max() > 100 and int((got.cpu().numpy() != want).sum()) == 0
    ia.close()
