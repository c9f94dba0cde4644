"""What a context has to hold before a forward runs: nothing for the kernels of a single launch, and a call captured on a context
that holds nothing allocates nothing, whatever its shape, runs in one launch where two would need a workspace, and gives the
oracle's bytes."""
import pytest

from test_parity_gpu import rect_problem, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, H, L, d, causal, variant, lut_bits, kernel of an eager call
    (1, 40, 900, 128, True, 0, 5, 1),    # the 128-row single launch
    (1, 74, 197, 128, False, 0, 5, 1),   # the same by the second look at square problems
    (1, 40, 200, 64, True, 2, 5, 2),
    (1, 257, 131, 128, True, 0, 5, 5),   # 1 -> 5 by the second look
    (1, 51, 1025, 64, False, 0, 5, 5),   # 3 -> 5
    (16, 8, 1000, 64, True, 0, 5, 5),    # 1024 workgroups of 128 rows: 5 by the first choice
    (16, 8, 1000, 64, True, 0, 6, 4),    # the same with a table of 64 entries
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}H{}L{}d{}c{:d}v{}b{}".format(*s[:7]))
def test_first_call(torch_mod, oracle, shape):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, H, L, d, causal, variant, lut_bits, kernel = shape
    print(f"case {shape}", flush=True)
    base, q, k, v = rect_problem(H + L, B, H, H, L, L, d, causal)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=causal, lut_bits=lut_bits, threads=16)["out"]
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    out = torch.full_like(tq, 55)

    def fresh():
        ia = binding.IntAttn(device=0, variant=variant, lut_bits=lut_bits)
        args, keep = ia.make_args(tq, tk, tv, out, base.s_q, base.s_k, base.s_v, None, causal=causal)
        assert ia.kernel_choice(args)[0] == kernel
        return ia, args, keep

    ia, args, keep = fresh()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ia.forward_args(args, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        out.fill_(55)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0
    del graph
    ia.close()

    ia, args, keep = fresh()
    free = torch.cuda.mem_get_info()[0]
    out.fill_(55)
    ia.forward_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert int((out.cpu().numpy() != want).sum()) == 0
    if kernel in (1, 2):
        assert torch.cuda.mem_get_info()[0] == free
    ia.close()

    ia, args, keep = fresh()  # a reservation has room for whichever kernels serve the call
    ia.reserve(args)
    free = torch.cuda.mem_get_info()[0]
    out.fill_(55)
    ia.forward_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()
