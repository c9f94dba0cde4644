"""The two layouts of the tables in the kernel for short key sequences: both sides of the rule (more than 128 keys and workgroups
of four waves), partly filled and idle waves, bit-compared with the oracle."""
import pytest

from test_kernel_choice import SHORT
from test_parity_gpu import rect_problem, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads, lq, lk", [(800, 64, 64), (200, 128, 128), (200, 129, 129), (200, 128, 200), (300, 96, 200), (400, 33, 256),
                                           (200, 97, 130), (130, 161, 161)])
def test_both_layouts(torch_mod, oracle, heads, lq, lk, causal):  # noqa: F811
    from paper_2511_21513_amd import binding

    base, q, k, v = rect_problem(lq + lk, 1, heads, heads, lq, lk, 64, causal)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=causal, threads=16)["out"]
    tq, tk, tv = (torch_mod.from_numpy(x).cuda() for x in (q, k, v))
    out = torch_mod.empty_like(tq)
    ia = binding.IntAttn(device=0)
    args, keep = ia.make_args(tq, tk, tv, out, base.s_q, base.s_k, base.s_v, None, causal=causal)
    assert ia.kernel_choice(args)[0] == SHORT
    ia.forward_args(args, torch_mod.cuda.current_stream().cuda_stream)
    torch_mod.cuda.synchronize()
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()
