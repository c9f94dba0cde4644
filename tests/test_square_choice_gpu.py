"""The second look at square problems in the automatic choice: both sides of each rule (host only), and on the GPU a problem of
each new kind against the oracle, also with scales in device memory and captured on a context that holds no memory."""
import numpy as np
import pytest

from test_kernel_choice import choice
from test_parity_gpu import rect_problem, torch_mod  # noqa: F401

RULES = [
    # heads, L, d, causal, kernel
    (73, 197, 128, False, 3), (74, 197, 128, False, 1),        # 511 and 518 workgroups of 32 rows
    (74, 197, 128, True, 3),
    (256, 197, 128, True, 1), (257, 197, 128, True, 5), (511, 197, 128, True, 5), (512, 197, 128, True, 5),
    (64, 1024, 128, True, 1), (65, 1024, 128, True, 5), (28, 1025, 128, True, 3), (29, 1025, 128, True, 5),
    (32, 2048, 128, True, 5), (31, 2049, 128, True, 1),
    (256, 197, 128, False, 1), (257, 197, 128, False, 5), (384, 197, 128, False, 5), (385, 197, 128, False, 1),
    (128, 767, 128, False, 5), (129, 767, 128, False, 1), (129, 768, 128, False, 5), (127, 1024, 128, False, 5), (600, 197, 128, False, 1),
    (50, 1024, 64, False, 3), (51, 1024, 64, False, 5), (80, 1024, 64, True, 3), (81, 1024, 64, True, 5),
    (149, 384, 64, True, 3), (150, 384, 64, True, 1), (266, 384, 64, True, 1), (267, 384, 64, True, 5), (512, 384, 64, True, 5),
    (266, 384, 64, False, 1), (267, 384, 64, False, 5), (342, 384, 64, False, 1),
]


@pytest.mark.parametrize("case", RULES, ids=lambda c: "H{}L{}d{}c{:d}".format(*c[:4]))
def test_rules(case):
    from paper_2511_21513_amd import binding

    heads, L, d, causal, want = case
    ia = binding.IntAttn(device=-1)
    assert choice(ia, 1, heads, heads, L, L, d, causal)[0] == want
    assert choice(ia, 1, heads, heads, L, L, d, causal, dynamic=True)[0] == want
    # what the rules leave alone: rectangles, maps in double precision, groups of rows
    old = 1 if heads * -(-L // 128) > 256 and not (d == 64 and L >= 1024) else 3
    if heads * -(-L // 128) < 1024:
        assert choice(ia, 1, heads, heads, L, L, d, causal, c_int=2**25 + 1)[0] == old
        assert choice(ia, 1, heads, heads, L, L + 1, d, causal)[0] == old


@pytest.mark.gpu
@pytest.mark.parametrize("heads, L, d, causal, kernel", [(74, 197, 128, False, 1), (257, 131, 128, True, 5), (512, 193, 128, True, 5), (29, 1025, 128, True, 5),
                                                         (257, 130, 128, False, 5), (51, 1025, 64, False, 5), (81, 1024, 64, True, 5),
                                                         (100, 300, 64, True, 3), (270, 300, 64, True, 5), (270, 300, 64, False, 5)])
def test_bit_exact_and_captured_without_memory(torch_mod, oracle, heads, L, d, causal, kernel):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    base, q, k, v = rect_problem(heads + L, 1, heads, heads, L, L, d, causal)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=causal, threads=16)["out"]
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    out = torch.empty_like(tq)
    stream = lambda: torch.cuda.current_stream().cuda_stream  # noqa: E731
    ia = binding.IntAttn(device=0)
    args, keep = ia.make_args(tq, tk, tv, out, base.s_q, base.s_k, base.s_v, None, causal=causal)
    assert ia.kernel_choice(args)[0] == kernel
    workgroups = heads * -(-L // 128)
    if workgroups <= 256 or (d == 64 and L >= 1024):  # served by the kernels that take no memory before, and so when captured first
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ia.forward_args(args, stream())
        for _ in range(3):
            out.fill_(55)
            graph.replay()
            torch.cuda.synchronize()
            assert int((out.cpu().numpy() != want).sum()) == 0
    out.fill_(55)
    ia.forward_args(args, stream())
    torch.cuda.synchronize()
    assert int((out.cpu().numpy() != want).sum()) == 0
    scales = [torch.from_numpy(np.ascontiguousarray(s, dtype=np.float32)).cuda() for s in (base.s_q, base.s_k, base.s_v)]
    out.fill_(55)
    args, keep = ia.make_args(tq, tk, tv, out, *scales, None, causal=causal, device_scales=True)
    assert ia.kernel_choice(args, dynamic=True)[0] == kernel
    ia.forward_dynamic_args(args, stream())
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()
