"""Sweep C as a launch of its own (variant 4, and the automatic choice with a table of 64 entries) builds its probability tables from
a LUT_hat that the first wave of a workgroup puts into LDS.  Contexts with different tables take turns, each on a first call, so that
a wave that read it too early would find another context's; compared with the oracle."""
import numpy as np
import pytest

import workloads
from test_parity_gpu import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lut_bits, variant, B, d, causal", [(5, 4, 1, 64, True), (6, 4, 1, 64, False), (6, 0, 16, 64, True), (5, 4, 1, 128, True), (6, 4, 1, 128, True)])
def test_contexts_with_different_tables_take_turns(torch_mod, oracle, lut_bits, variant, B, d, causal):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    H, L = 8, 1000
    p = workloads.random_problem(d + lut_bits, B, H, H, L, d, causal, per_head=True, spread=1.2)
    s_o = (p.s_v * 0.05).astype(np.float32)
    q, k, v = (torch.from_numpy(x).cuda() for x in (p.q, p.k, p.v))
    clips = (6.6, 2.0, 9.0)
    want = [torch.from_numpy(oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, s_o, causal=causal, per_head=True, lut_bits=lut_bits, clip=c, threads=16)["out"]).cuda()
            for c in clips]
    assert not torch.equal(want[0], want[1]) and not torch.equal(want[0], want[2])
    for rep in range(12):
        ia = binding.IntAttn(device=0, variant=variant, lut_bits=lut_bits, clip=clips[rep % 3])
        args, keep = ia.make_args(q, k, v, torch.empty_like(q), p.s_q, p.s_k, p.s_v, s_o, causal=causal, per_head=True)
        assert ia.kernel_choice(args)[0] == 4
        got = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=causal, per_head=True)
        torch.cuda.synchronize()
        assert int((got != want[rep % 3]).sum()) == 0, rep
        ia.close()
