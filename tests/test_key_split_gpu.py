"""The tiled path with the keys split over several workgroups (few query tiles against many keys, automatic variant),
bit-compared with the CPU oracle; and the mapping of work to XCDs for group counts that do not divide by eight."""
import numpy as np
import pytest

from test_fma_map_gpu import scales_for, without_factor
from test_kernel_choice import SPLIT
from test_parity_gpu import rect_forward, rect_problem, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, Hq, Hkv, Lq, Lkv, d, causal, per_head
    (1, 1, 1, 32, 16384, 64, True, False),     # one partly filled query tile, every range a single tile long
    (1, 1, 1, 257, 9001, 128, True, False),    # ragged rows and keys, the diagonal in the last range only
    (1, 4, 1, 129, 8192, 64, False, True),     # no mask, whole tiles
    (1, 3, 3, 200, 8190, 128, True, True),     # three groups over eight XCDs
    (2, 2, 1, 513, 7001, 128, True, False),
    (1, 1, 1, 4096, 4096, 128, True, False),   # the first query tiles have fewer key tiles than there are ranges: empty ranges
    (1, 1, 1, 8192, 8192, 64, True, False),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{}ph{}".format(*[int(x) for x in s]))
def test_key_split_bit_exact(torch_mod, oracle, shape):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, Hq, Hkv, lq, lk, d, causal, per_head = shape
    print(f"case {shape}", flush=True)
    ia = binding.IntAttn(device=0)
    base, q, k, v = rect_problem(900 + lq, B, Hq, Hkv, lq, lk, d, causal, per_head)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=causal, per_head=per_head, taps=True, threads=16)
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    kernel, split_rows, split_pv = ia.kernel_choice(ia.make_args(tq, tk, tv, torch.empty_like(tq), base.s_q, base.s_k, base.s_v, None, causal=causal,
                                                                 per_head=per_head)[0])
    assert kernel == SPLIT and split_rows > 1 and split_pv > 1
    got = rect_forward(torch, ia, base, q, k, v)
    for key in ("row_max", "row_sum", "acc", "out"):
        assert int((got[key] != want[key]).sum()) == 0, key
    # the same scales in device memory
    sc = [torch.from_numpy(np.ascontiguousarray(s, dtype=np.float32)).to(dev) for s in (base.s_q, base.s_k, base.s_v)]
    out = torch.empty_like(tq)
    args, keep = ia.make_args(tq, tk, tv, out, *sc, None, causal=causal, per_head=per_head, device_scales=True)
    assert ia.kernel_choice(args, dynamic=True)[0] == SPLIT
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want["out"]).sum()) == 0
    ia.close()


@pytest.mark.parametrize("lut_bits, c_int, scheme", [(3, 5203, 9), (5, 47011, 9), (5, None, 0), (5, 2**25 + 1, 0)],
                         ids=["table of 8", "fma", "double", "double past 2^24"])
def test_key_split_tables_and_index_maps_bit_exact(torch_mod, oracle, lut_bits, c_int, scheme):  # noqa: F811
    """Tables of fewer than 32 entries, and both index maps; also as the device picks them."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    c_int = without_factor(31) if c_int is None else c_int
    assert binding.IntAttn(device=-1, lut_bits=lut_bits).derive_index_map(c_int, 9)[0] == scheme
    base, q, k, v = rect_problem(77, 1, 2, 1, 129, 9001, 64, True)
    s_q, s_k = (np.array([x], dtype=np.float32) for x in scales_for(c_int))
    s_v, s_o = np.array([0.02], dtype=np.float32), np.array([0.004], dtype=np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=True, lut_bits=lut_bits, threads=16)["out"]
    ia = binding.IntAttn(device=0, lut_bits=lut_bits)
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    for device_scales in (False, True):
        out = torch.full_like(tq, 99)
        sc = [torch.from_numpy(x).cuda() if device_scales else x for x in (s_q, s_k, s_v, s_o)]
        args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=True, device_scales=device_scales)
        assert ia.kernel_choice(args, dynamic=device_scales)[0] == SPLIT
        (ia.forward_dynamic_args if device_scales else ia.forward_args)(args, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0, device_scales
    ia.close()


def test_key_split_row_groups_bit_exact(torch_mod, oracle):  # noqa: F811
    """A scale and an output scale per block of query rows: every row's own requantization after the ranges meet."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    ia = binding.IntAttn(device=0)
    base, q, k, v = rect_problem(31, 1, 2, 1, 100, 8200, 128, True, per_head=True)
    rng = np.random.default_rng(5)
    s_q = (base.s_q[None, :, None] * rng.uniform(0.3, 2.5, size=(1, 2, 15))).astype(np.float32)
    s_o = (base.s_v[[0, 0]][None, :, None] * rng.uniform(0.02, 0.2, size=(1, 2, 15))).astype(np.float32)
    want = oracle.forward_row_groups(q, k, v, s_q, base.s_k, base.s_v, s_o, q_block=7, causal=True)["out"]
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    sc = [torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in (s_q, base.s_k, base.s_v, s_o)]
    out = torch.empty_like(tq)
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=True, device_scales=True, q_block=7)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


@pytest.mark.parametrize("variant", [1, 3, 5], ids=lambda v: f"variant{v}")
@pytest.mark.parametrize("heads", [(1, 1, 1), (1, 6, 2), (1, 12, 12), (3, 9, 3), (1, 8, 4), (257, 1, 1)], ids=str)
def test_group_counts_over_xcds_bit_exact(torch_mod, oracle, heads, variant):  # noqa: F811
    from paper_2511_21513_amd import binding

    B, Hq, Hkv = heads
    ia = binding.IntAttn(device=0, variant=variant)
    base, q, k, v = rect_problem(60 + B + Hq, B, Hq, Hkv, 150 if B < 100 else 33, 150 if B < 100 else 33, 64, True)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=True, threads=16)["out"]
    assert int((rect_forward(torch_mod, ia, base, q, k, v, taps=False)["out"] != want).sum()) == 0
    ia.close()


def test_key_split_workspace_reserved_ahead_and_under_capture(torch_mod, oracle):  # noqa: F811
    """A chunk after a reservation for a longer prompt allocates nothing; a capture on a context without a workspace runs
    (unsplit) instead of allocating."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    base, q, k, v = rect_problem(77, 1, 2, 1, 129, 9001, 128, True)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=True, threads=16)["out"]
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    out = torch.empty_like(tq)
    ia = binding.IntAttn(device=0)
    args, keep = ia.make_args(tq, tk, tv, out, base.s_q, base.s_k, base.s_v, None, causal=True)
    longer = torch.zeros((1, 2, 9001, 128), dtype=torch.int8, device="cuda")
    ia.reserve(ia.make_args(longer, tk, tv, torch.empty_like(longer), base.s_q, base.s_k, base.s_v, None, causal=True)[0])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ia.forward_args(args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()

    ia = binding.IntAttn(device=0)
    out.fill_(55)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ia.forward_args(args, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        out.fill_(55)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


def test_captured_launches_stay_valid_when_the_room_for_split_keys_grows(torch_mod, oracle):  # noqa: F811
    """Graphs captured after an eager call, of a problem that splits its keys and of one that uses the workspace; then eager
    calls that split and need more room: what the graphs were recorded with is still theirs."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    ia = binding.IntAttn(device=0)
    stream = lambda: torch.cuda.current_stream().cuda_stream  # noqa: E731

    def call(B, Hq, Hkv, lq, lk, d, kernel):
        base, q, k, v = rect_problem(lq, B, Hq, Hkv, lq, lk, d, True)
        tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
        out = torch.empty_like(tq)
        args, keep = ia.make_args(tq, tk, tv, out, base.s_q, base.s_k, base.s_v, None, causal=True)
        assert ia.kernel_choice(args)[0] == kernel
        ia.forward_args(args, stream())
        torch.cuda.synchronize()
        return args, out, out.cpu().numpy(), (tq, tk, tv, keep), (base, q, k, v)

    graphs = []
    for shape in ((1, 2, 1, 129, 9001, 128, SPLIT), (1, 40, 40, 900, 900, 128, 1)):
        args, out, want, keep, problem = call(*shape)
        if shape[-1] == SPLIT:
            base, q, k, v = problem
            assert int((want != oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=True, threads=16)["out"]).sum()) == 0
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ia.forward_args(args, stream())
        graphs.append((graph, out, want, keep))
    for shape in ((1, 2, 1, 513, 9001, 128, SPLIT), (1, 8, 2, 513, 12000, 128, SPLIT)):
        call(*shape)
        filler = [torch.full((1 << 20,), 77, dtype=torch.int32, device="cuda") for _ in range(8)]
        for graph, out, want, _ in graphs:
            out.fill_(55)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert int((out.cpu().numpy() != want).sum()) == 0
        assert all(int((x != 77).sum()) == 0 for x in filler)
    ia.close()
