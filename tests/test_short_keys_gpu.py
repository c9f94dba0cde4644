"""The kernel for short key sequences (d = 64, at most 256 keys, scores held in registers), taken by the automatic variant:
edges of its 32-key sub-tiles and of its register layouts, partly filled waves and workgroups, masks, strides and table sizes;
row maxima, row sums, accumulators and bytes of the oracle."""
import numpy as np
import pytest

from test_kernel_choice import SHORT
from test_parity_gpu import rect_forward, rect_problem, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Lq, Lkv, causal, per_head: enough heads that the shape is served by this kernel
SHAPES = [(170, 6, 6, lk, lk, causal, False) for lk in (33, 128, 129, 197, 224, 225, 256) for causal in (False, True)] + [
    (1030, 1, 1, 1, 1, False, False),
    (130, 8, 2, 31, 32, True, True),      # one partly filled wave
    (70, 16, 4, 100, 250, True, True),    # fewer query rows than keys
    (200, 6, 3, 300, 200, False, True),   # more query rows than one workgroup takes
    (64, 17, 17, 515, 97, False, False),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}c{}ph{}".format(*[int(x) for x in s]))
def test_short_keys_bit_exact(torch_mod, oracle, shape):  # noqa: F811
    from paper_2511_21513_amd import binding

    B, Hq, Hkv, lq, lk, causal, per_head = shape
    print(f"case {shape}", flush=True)
    base, q, k, v = rect_problem(lq + 7 * lk, 2, Hq, Hkv, lq, lk, 64, causal, per_head)
    q[0, 0, 0], k[0, 0, 0], v[0, 0, 0] = -128, -128, -128
    q, k, v = (np.ascontiguousarray(np.tile(x, (B // 2, 1, 1, 1))) for x in (q, k, v))
    want = oracle.forward(q[:2], k[:2], v[:2], base.s_q, base.s_k, base.s_v, None, causal=causal, per_head=per_head, taps=True, threads=16)
    ia = binding.IntAttn(device=0)
    tensors = [torch_mod.from_numpy(x) for x in (q, k, v)]
    args, _ = ia.make_args(*tensors, torch_mod.empty_like(tensors[0]), base.s_q, base.s_k, base.s_v, None, causal=causal, per_head=per_head)
    args.q, args.k, args.v, args.out = 16, 32, 48, 64  # (not read)
    assert ia.kernel_choice(args)[0] == SHORT
    got = rect_forward(torch_mod, ia, base, q, k, v)
    ia.close()
    for key in ("row_max", "row_sum", "acc", "out"):
        for part in range(0, q.shape[0], 2):
            assert int((got[key][part:part + 2] != want[key]).sum()) == 0, (key, part)


@pytest.mark.parametrize("lut_bits", [1, 3, 5])
def test_short_keys_fused_projection_layout_bit_exact(torch_mod, oracle, lut_bits):  # noqa: F811
    """Q, K and V as slices of one [B, L, 3, H, d] tensor, the output as [B, L, H, d]; bytes around the rows stay."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, H, L = 90, 12, 145
    base, q, k, v = rect_problem(3, 2, H, H, L, L, 64, False)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=False, lut_bits=lut_bits, threads=16)["out"]
    qkv = torch.from_numpy(np.stack([np.tile(x, (B // 2, 1, 1, 1)).transpose(0, 2, 1, 3) for x in (q, k, v)], axis=2)).cuda()
    out = torch.full((B, L, H, 96), 7, dtype=torch.int8, device="cuda")
    ia = binding.IntAttn(device=0, lut_bits=lut_bits)
    q, k, v = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    dst = out[..., 16:80].permute(0, 2, 1, 3)
    assert ia.kernel_choice(ia.make_args(q, k, v, dst, base.s_q, base.s_k, base.s_v, None, causal=False)[0])[0] == SHORT
    ia.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=False, out=dst)
    torch.cuda.synchronize()
    ia.close()
    got = out.cpu().numpy()
    assert (got[..., :16] == 7).all() and (got[..., 80:] == 7).all()
    got = got[..., 16:80].transpose(0, 2, 1, 3)
    for part in range(0, B, 2):
        assert int((got[part:part + 2] != want).sum()) == 0, part
