"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  The whole pipeline is integer, so the bar is bit-exact: zero mismatching
bytes in the INT8 output, and equal int32 row max / row sum / accumulator taps."""
import functools

import numpy as np
import pytest

import workloads as inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_mod():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X (torch.cuda.is_available() is False)")
    return torch


# kernel variants: 0 = automatic choice; 1, 2 = one launch (32 / 64 query rows per wave); 4 = two
# launches (sweeps A+B, then sweep C) with the phase-ordered kernels; 5 = sweep C's own kernel; 9 = the split-key kernels (few query rows against many keys) wherever
# (Hq / Hkv) * L <= 31, else as 0
@pytest.fixture(scope="module", params=[0, 1, 2, 3, 4, 5, 9], ids=lambda v: f"variant{v}")
def ia(torch_mod, request):
    from paper_2511_21513_amd import binding

    ctx = binding.IntAttn(device=0, variant=request.param)
    yield ctx
    ctx.close()


@functools.lru_cache(maxsize=2)
def cached_problem(name):
    return inputs.make_problem(name)


def gpu_forward(torch, ia, p, s_o=None, taps=False):
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    r = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=p.causal, per_head=p.per_head, taps=taps)
    torch.cuda.synchronize()
    if taps:
        return {k_: v_.cpu().numpy() for k_, v_ in r.items()}
    return {"out": r.cpu().numpy()}


def check_full(torch, ia, oracle, p, s_o=None, taps=True, threads=16):
    got = gpu_forward(torch, ia, p, s_o, taps=taps)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, s_o, causal=p.causal, per_head=p.per_head,
                          taps=taps, threads=threads)
    if taps:
        for key in ("row_max", "row_sum", "acc"):
            bad = int((got[key] != want[key]).sum())
            assert bad == 0, f"{p.name}: {bad} mismatching {key} entries"
    bad = int((got["out"] != want["out"]).sum())
    assert bad == 0, f"{p.name}: {bad} mismatching output bytes of {want['out'].size}"
    return got


SHAPES = [
    # B, Hq, Hkv, L, d, causal, per_head
    (1, 1, 1, 1, 64, False, False),
    (1, 1, 1, 1, 128, True, False),
    (2, 2, 1, 31, 64, True, False),
    (1, 2, 2, 32, 128, False, False),
    (1, 3, 3, 33, 64, False, False),
    (2, 4, 2, 97, 128, True, True),
    (1, 2, 1, 128, 64, True, False),
    (1, 2, 2, 129, 128, False, True),
    (1, 4, 1, 197, 64, False, False),
    (1, 2, 2, 300, 128, True, False),
    (1, 1, 1, 515, 64, True, False),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B{}Hq{}Hkv{}L{}d{}c{}ph{}".format(*[int(x) for x in s]))
def test_small_shapes_bit_exact(torch_mod, ia, oracle, shape):
    B, Hq, Hkv, L, d, causal, per_head = shape
    print(f"case {shape}", flush=True)
    p = inputs.random_problem(100 + L + d, B, Hq, Hkv, L, d, causal, per_head=per_head, spread=1.5)
    check_full(torch_mod, ia, oracle, p)
    s_o = inputs.calibrated_out_scale(p)
    check_full(torch_mod, ia, oracle, p, s_o)


@pytest.mark.parametrize("scale,d", [(0.5, 64), (0.05, 64), (0.004, 64), (0.002, 64), (0.0005, 64), (0.01, 128),
                                     (0.004, 128)])
def test_clip_threshold_range_bit_exact(torch_mod, ia, oracle, scale, d):
    """Thresholds from a handful (coarse index steps) to far beyond the reach of the 24-bit and
    fp32 schemes (the kernels' fp64 index map), with and without the clip binding."""
    p = inputs.random_problem(7, 1, 2, 2, 160, d, True)
    p.s_q = np.asarray([scale], dtype=np.float32)
    p.s_k = np.asarray([scale], dtype=np.float32)
    print("c_int", oracle.c_int(6.6, p.s_q[0], p.s_k[0], d), flush=True)
    check_full(torch_mod, ia, oracle, p)


def test_adversarial_rows_bit_exact(torch_mod, ia, oracle):
    """Zero queries (all logits equal: P = round(255/n), zero beyond n = 510), a dominant key
    (one-hot rows, P = 255 >= 128 exercises the unsigned-probability path), extreme int8
    values including -128, and saturating outputs."""
    rng = np.random.default_rng(5)
    L, d = 640, 64
    q = rng.integers(-128, 128, size=(1, 4, L, d)).astype(np.int8)
    k = rng.integers(-128, 128, size=(1, 2, L, d)).astype(np.int8)
    v = rng.integers(-128, 128, size=(1, 2, L, d)).astype(np.int8)
    q[0, 0] = 0                # equal logits
    k[0, 0, 17] = 127
    q[0, 1] = 127              # key 17 dominates head 1 (KV head 0)
    q[0, 2, ::2] = -128
    k[0, 1, ::3] = -128
    v[0, 1, ::5] = -128
    for causal in (False, True):
        p = inputs.Problem("adversarial", 1, 4, 2, L, d, causal, False, q, k, v,
                           np.asarray([0.02], np.float32), np.asarray([0.03], np.float32), np.asarray([0.05], np.float32))
        got = check_full(torch_mod, ia, oracle, p)
        assert not got["out"][0, 0, 600 if not causal else 639].any()
        check_full(torch_mod, ia, oracle, p, np.asarray([0.002], np.float32))  # saturates at +-127


def test_strided_views_bit_exact(torch_mod, ia, oracle):
    """Tensors laid out [B, L, H, d] in memory (a transposed view) must give the same bytes."""
    torch = torch_mod
    p = inputs.random_problem(9, 2, 4, 2, 150, 64, True)
    dev = torch.device("cuda:0")
    mk = lambda x: torch.from_numpy(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).to(dev).permute(0, 2, 1, 3)
    q, k, v = mk(p.q), mk(p.k), mk(p.v)
    out = torch.empty((2, 150, 4, 64), dtype=torch.int8, device=dev).permute(0, 2, 1, 3)
    ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, causal=True, out=out)
    torch.cuda.synchronize()
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, causal=True)["out"]
    assert int((out.cpu().numpy() != want).sum()) == 0


def test_config1_single_head(torch_mod, ia, oracle):
    p = inputs.make_problem("c1_single_head")
    check_full(torch_mod, ia, oracle, p)
    check_full(torch_mod, ia, oracle, p, inputs.calibrated_out_scale(p))


def test_config2_vit(torch_mod, ia, oracle):
    p = inputs.make_problem("c2_vit_b16")
    check_full(torch_mod, ia, oracle, p)
    check_full(torch_mod, ia, oracle, p, inputs.calibrated_out_scale(p), taps=False)


def test_config3_llm_prefill_2k(torch_mod, ia, oracle):
    p = inputs.make_problem("c3_llm_prefill_2k")
    check_full(torch_mod, ia, oracle, p)
    check_full(torch_mod, ia, oracle, p, inputs.calibrated_out_scale(p), taps=False)


def check_sampled(torch, ia, oracle, p, s_o, heads, n_rows, seed):
    """Full-size problem in the benchmark's launch configuration; the oracle recomputes sampled
    query rows one by one (always including the first and last rows and a tile boundary)."""
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    out = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=p.causal, per_head=p.per_head)
    torch.cuda.synchronize()
    rng = np.random.default_rng(seed)
    for (b, h) in heads:
        rows = np.unique(np.concatenate([[0, 1, 127, 128, p.L - 1, p.L - 129], rng.integers(0, p.L, n_rows)])).astype(np.int32)
        want = oracle.rows(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, s_o, b=b, hq=h, rows=rows, causal=p.causal,
                           per_head=p.per_head)
        got = out[b, h].cpu().numpy()[rows]
        bad = int((got != want["out"]).sum())
        assert bad == 0, f"{p.name} b={b} h={h}: {bad} mismatching bytes on sampled rows"
    return out


def test_config4_gqa_prefill_8k_sampled(torch_mod, ia, oracle):
    p = cached_problem("c4_gqa_prefill_8k")
    s_o = inputs.calibrated_out_scale(p, sample_rows=16)
    heads = [(0, 0), (0, 5), (0, 17), (0, 31)]
    out = check_sampled(torch_mod, ia, oracle, p, s_o, heads, 24, 4)
    assert int(out.abs().max()) > 20  # the calibrated scale makes the bytes informative
    check_sampled(torch_mod, ia, oracle, p, None, heads[:2], 8, 5)


def test_config5_batched_prefill_4k_sampled(torch_mod, ia, oracle):
    p = cached_problem("c5_batched_prefill_4k")
    s_o = inputs.calibrated_out_scale(p, sample_rows=8)
    heads = [(0, 0), (3, 7), (9, 30), (15, 31)]
    check_sampled(torch_mod, ia, oracle, p, s_o, heads, 16, 6)


def test_long_ragged_sequence_sampled(torch_mod, ia, oracle):
    """L far beyond the benchmark sizes and not a multiple of any tile (70001 = 546 * 128 + 113):
    hundreds of key tiles per row, row sums beyond 2^16, a ragged last tile in every sweep."""
    p = inputs.random_problem(31, 1, 2, 1, 70001, 64, True, spread=1.2)
    check_sampled(torch_mod, ia, oracle, p, None, [(0, 0), (0, 1)], 12, 7)
    p = inputs.random_problem(32, 1, 1, 1, 33333, 128, False, spread=1.0)
    check_sampled(torch_mod, ia, oracle, p, inputs.calibrated_out_scale(p, sample_rows=8), [(0, 0)], 12, 8)


def fp64_reference_out(p, s_o):
    """fp64 softmax attention of the dequantized inputs, in units of s_O (not rounded)."""
    g = p.Hq // p.Hkv
    out = np.zeros((p.B, p.Hq, p.L, p.d))
    for b in range(p.B):
        for h in range(p.Hq):
            kv = h // g
            sq = float(p.s_q[h] if p.per_head else p.s_q[0])
            sk = float(p.s_k[kv] if p.per_head else p.s_k[0])
            sv = float(p.s_v[kv] if p.per_head else p.s_v[0])
            so = float(s_o[h] if p.per_head else s_o[0])
            a = (p.q[b, h].astype(np.float64) * sq) @ (p.k[b, kv].astype(np.float64) * sk).T / np.sqrt(p.d)
            if p.causal:
                a = np.where(np.tril(np.ones((p.L, p.L), dtype=bool)), a, -np.inf)
            a -= a.max(axis=1, keepdims=True)
            w = np.exp(a)
            w /= w.sum(axis=1, keepdims=True)
            out[b, h] = w @ (p.v[b, kv].astype(np.float64) * sv) / so
    return out


@pytest.mark.parametrize("shape", [(1, 2, 2, 197, 64, False, False), (2, 4, 2, 333, 128, True, True),
                                   (1, 2, 1, 1100, 128, True, False)],
                         ids=lambda s: "B{}Hq{}Hkv{}L{}d{}c{}ph{}".format(*[int(x) for x in s]))
def test_quantonly_comparator_close_to_fp64(torch_mod, ia, shape):
    """The conventional INT8 comparator (dequantize -> fp32 softmax -> requantize P to INT8 x127) is
    not an exact integer function; it must stay within the error its 7-bit probabilities allow:
    each P entry is off by at most 1/254 of the row's largest weight, so the output error is
    bounded by n_keys/254 * max|V_hat| * s_V/s_O in the worst case and is far smaller on
    average.  Checked: mean error below one output step and no outliers beyond 6 steps."""
    torch = torch_mod
    B, Hq, Hkv, L, d, causal, per_head = shape
    p = inputs.random_problem(500 + L, B, Hq, Hkv, L, d, causal, per_head=per_head, spread=1.5)
    s_o = inputs.calibrated_out_scale(p)
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    got = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=causal, per_head=per_head, quantonly=True)
    torch.cuda.synchronize()
    ref = fp64_reference_out(p, s_o)
    err = np.abs(got.cpu().numpy().astype(np.float64) - np.clip(ref, -127, 127))
    assert err.mean() < 1.0, err.mean()
    assert err.max() <= 6.0, err.max()


def test_stages_compose_to_the_forward(torch_mod, oracle):
    """Stage 1 (sweeps A+B) followed by stage 2 (sweep C) gives the bytes of the
    one-call forward; a single-launch variant refuses to be cut."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    dev = torch.device("cuda:0")
    p = inputs.random_problem(21, 2, 4, 2, 300, 128, True)
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=True)["out"]
    for variant in (4, 5):
        ia = binding.IntAttn(device=0, variant=variant)
        out = torch.zeros_like(q)
        args, keep = ia.make_args(q, k, v, out, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=False)
        ia.forward_stage(args, 1)
        torch.cuda.synchronize()
        assert not out.any(), "stage 1 must not write the output"
        ia.forward_stage(args, 2)
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0
        ia.close()
    ia = binding.IntAttn(device=0, variant=1)
    args, keep = ia.make_args(q, k, v, torch.zeros_like(q), p.s_q, p.s_k, p.s_v, None, causal=True, per_head=False)
    with pytest.raises(binding.IntAttnError):
        ia.forward_stage(args, 2)
    ia.close()


QUANT_CASES = [
    # B, H, L, d, dtype, per_head
    (1, 1, 1, 8, "float32", False),
    (2, 3, 37, 64, "float16", False),
    (2, 3, 37, 64, "bfloat16", True),
    (1, 5, 1000, 128, "float32", True),
    (3, 2, 513, 72, "float16", True),
    (1, 8, 4096, 128, "bfloat16", False),
]


@pytest.mark.parametrize("case", QUANT_CASES, ids=lambda c: "B{}H{}L{}d{}{}ph{}".format(*c[:5], int(c[5])))
def test_quantizer_bit_exact(torch_mod, oracle, case):
    """The on-GPU dynamic quantizer (Sec. 2.1, Eq. quant) against the oracle: INT8 bytes and fp32
    scales must be identical (fp16 / bf16 inputs are widened exactly on both sides)."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, H, L, d, dtype, per_head = case
    print(f"case {case}", flush=True)
    rng = np.random.default_rng(B * 1000 + L)
    x = (rng.standard_t(4, size=(B, H, L, d)) * rng.uniform(0.05, 20.0, size=(1, H, 1, 1))).astype(np.float32)
    xt = torch.from_numpy(x).to("cuda:0").to(getattr(torch, dtype))
    ia = binding.IntAttn(device=0)
    xq, s = ia.quantize(xt, per_head)
    torch.cuda.synchronize()
    want_q, want_s = oracle.quantize(xt.float().cpu().numpy(), per_head)
    np.testing.assert_array_equal(s.cpu().numpy(), want_s)
    assert int((xq.cpu().numpy() != want_q).sum()) == 0
    ia.close()


def test_quantizer_edge_cases(torch_mod, oracle):
    """All-zero tensor (floored scale), exact ties (scale exactly 1), a strided [B, L, H, d] view
    in and out, and the same context reused with more groups."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    ia = binding.IntAttn(device=0)
    z = torch.zeros((1, 2, 5, 16), device="cuda:0", dtype=torch.float16)
    zq, zs = ia.quantize(z, per_head=True)
    want_q, want_s = oracle.quantize(z.float().cpu().numpy(), True)
    np.testing.assert_array_equal(zs.cpu().numpy(), want_s)
    assert not zq.any()
    t = torch.zeros((1, 1, 1, 8), device="cuda:0")
    t[0, 0, 0] = torch.tensor([127.0, 0.5, 1.5, 2.5, -0.5, -1.5, -2.5, 126.5])
    tq, ts = ia.quantize(t)
    assert ts.item() == 1.0 and tq[0, 0, 0].tolist() == [127, 0, 2, 2, 0, -2, -2, 126]
    rng = np.random.default_rng(77)
    x = rng.standard_normal((2, 150, 6, 64)).astype(np.float32)  # [B, L, H, d] in memory
    xv = torch.from_numpy(x).to("cuda:0").permute(0, 2, 1, 3)
    out = torch.empty((2, 150, 6, 64), dtype=torch.int8, device="cuda:0").permute(0, 2, 1, 3)
    xq, s = ia.quantize(xv, per_head=True, out=out)
    torch.cuda.synchronize()
    want_q, want_s = oracle.quantize(np.ascontiguousarray(x.transpose(0, 2, 1, 3)), True)
    np.testing.assert_array_equal(s.cpu().numpy(), want_s)
    assert int((xq.cpu().numpy() != want_q).sum()) == 0
    ia.close()


def test_quantizer_feeds_the_forward(torch_mod, oracle):
    """fp16 Q, K, V -> on-GPU quantizer -> forward: the same bytes as the oracle quantizer
    followed by the oracle forward."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(78)
    B, Hq, Hkv, L, d = 1, 4, 2, 300, 64
    qf = torch.from_numpy(rng.standard_normal((B, Hq, L, d)).astype(np.float32)).to("cuda:0").half()
    kf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to("cuda:0").half()
    vf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to("cuda:0").half()
    ia = binding.IntAttn(device=0)
    (q, sq), (k, sk), (v, sv) = (ia.quantize(t) for t in (qf, kf, vf))
    out = ia.forward(q, k, v, sq.cpu().numpy(), sk.cpu().numpy(), sv.cpu().numpy(), causal=True)
    torch.cuda.synchronize()
    oq, osq = oracle.quantize(qf.float().cpu().numpy())
    ok, osk = oracle.quantize(kf.float().cpu().numpy())
    ov, osv = oracle.quantize(vf.float().cpu().numpy())
    want = oracle.forward(oq, ok, ov, osq, osk, osv, None, causal=True)["out"]
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


# ---------------------------------------------------------------- forward with device-resident scales

def dynamic_forward(torch, ia, p, s_o=None):
    """intattn_forward_dynamic with the problem's scales copied to the GPU; returns (out, status)."""
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    scales = [torch.from_numpy(np.ascontiguousarray(s, dtype=np.float32)).to(dev) if s is not None else None
              for s in (p.s_q, p.s_k, p.s_v, s_o)]
    out = torch.empty_like(q)
    args, keep = ia.make_args(q, k, v, out, *scales, causal=p.causal, per_head=p.per_head, device_scales=True)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    return out.cpu().numpy(), ia.dynamic_status()


DYN_SHAPES = [
    # B, Hq, Hkv, L, d, causal, per_head, scale multiplier on s_q (moves c_int between the schemes)
    (1, 1, 1, 1, 64, False, False, 1.0),
    (2, 4, 2, 97, 128, True, True, 1.0),
    (1, 4, 1, 197, 64, False, False, 0.01),
    (1, 2, 2, 300, 128, True, False, 1e-4),
    (1, 6, 2, 515, 64, True, True, 1.0),
]


@pytest.mark.parametrize("shape", DYN_SHAPES, ids=lambda s: "B{}Hq{}Hkv{}L{}d{}c{}ph{}x{}".format(*s))
def test_dynamic_forward_bit_exact(torch_mod, ia, oracle, shape):
    """Scales in device memory, parameters derived by a kernel: the same bytes as the oracle computes
    from the same scale values, for every kernel variant, with and without an output scale."""
    B, Hq, Hkv, L, d, causal, per_head, mul = shape
    print(f"case {shape}", flush=True)
    p = inputs.random_problem(300 + L + d, B, Hq, Hkv, L, d, causal, per_head=per_head, spread=1.5)
    p.s_q = (p.s_q * mul).astype(np.float32)
    for s_o in (None, inputs.calibrated_out_scale(p)):
        got, status = dynamic_forward(torch_mod, ia, p, s_o)
        want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, s_o, causal=p.causal, per_head=p.per_head)["out"]
        assert status == 0
        assert int((got != want).sum()) == 0


def test_dynamic_forward_mixed_schemes(torch_mod, ia, oracle):
    """Per-head scales that put some heads in reach of the fp32 index map and others beyond it:
    each head is served by exactly one of the two launches of a kernel."""
    p = inputs.random_problem(41, 2, 8, 4, 260, 64, True, per_head=True, spread=1.5)
    p.s_q = (p.s_q * np.asarray([1, 1e-2, 1, 1e-3, 3e-3, 1, 2e-5, 1], dtype=np.float32)).astype(np.float32)
    cs = [oracle.c_int(6.6, p.s_q[h], p.s_k[h // 2], 64) for h in range(8)]
    print("c_int per head", cs, flush=True)
    assert min(cs) < 300000 and max(cs) > 2**24
    got, status = dynamic_forward(torch_mod, ia, p)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True)["out"]
    assert status == 0
    assert int((got != want).sum()) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("d,causal", [(64, True), (128, True), (128, False)], ids=lambda v: str(v))
def test_host_scales_mixed_schemes_in_sweep_c(torch_mod, oracle, d, causal):
    """Per-head host scales with thresholds below 62, of hundreds and of tens of thousands in one call of the two-launch path:
    every tap and the output equal the oracle's, also on a second call and after the scales change."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    p = inputs.random_problem(43, 2, 8, 4, 700, d, causal, per_head=True, spread=1.2)
    ia = binding.IntAttn(device=0, variant=5)
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    base = np.float32(np.sqrt(6.6 * np.sqrt(d) / 900.0))  # s_q = s_k = base: c_int = 900
    for mult in ([1, 1, 18, 1, 1, 0.03, 1, 1], [1, 20, 1, 1, 1, 1, 1, 1], [1] * 8):  # c_int 900; 50 and 30000; 45
        s_q = (base * np.asarray(mult, dtype=np.float32)).astype(np.float32)
        s_k = np.full(4, base, dtype=np.float32)
        cs = [oracle.c_int(6.6, s_q[h], s_k[h // 2], d) for h in range(8)]
        print("c_int per head", cs, flush=True)
        want = oracle.forward(p.q, p.k, p.v, s_q, s_k, p.s_v, None, causal=causal, per_head=True, taps=True, threads=8)
        for rep in range(2):
            got = ia.forward(q, k, v, s_q, s_k, p.s_v, None, causal=causal, per_head=True, taps=True)
            torch.cuda.synchronize()
            for key in ("row_max", "row_sum", "acc", "out"):
                assert int((got[key].cpu().numpy() != want[key]).sum()) == 0, (mult, rep, key)
    ia.close()


def test_dynamic_forward_on_the_workload_configs(torch_mod, oracle):
    """Two of the workload configurations in full, through the automatic variant."""
    from paper_2511_21513_amd import binding

    ia = binding.IntAttn(device=0)
    for name in ("c2_vit_b16", "c3_llm_prefill_2k"):
        p = inputs.make_problem(name)
        got, status = dynamic_forward(torch_mod, ia, p)
        want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=p.causal, per_head=p.per_head)["out"]
        assert status == 0 and int((got != want).sum()) == 0, name
    ia.close()


def test_dynamic_forward_reports_unusable_scales(torch_mod, oracle):
    """A zero, negative, infinite or NaN scale cannot come back as a return code (the host never
    reads it): the status word says so, nothing faults, and the next good call clears it."""
    from paper_2511_21513_amd import binding

    ia = binding.IntAttn(device=0)
    assert ia.dynamic_status() == 0  # before any call
    p = inputs.random_problem(43, 1, 4, 2, 130, 64, False, per_head=True)
    good = p.s_q.copy()
    for bad in (0.0, -1.0, np.inf, np.nan):
        p.s_q = good.copy()
        p.s_q[2] = bad
        got, status = dynamic_forward(torch_mod, ia, p)
        assert status == 1
        # the other heads are untouched by it
        p.s_q = good.copy()
        want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=False, per_head=True)["out"]
        keep = [0, 1, 3]
        assert int((got[:, keep] != want[:, keep]).sum()) == 0
        assert not got[:, 2].any()  # defined output for the head with the unusable scale: all zeros
    p.s_q = good
    got, status = dynamic_forward(torch_mod, ia, p)
    assert status == 0 and int((got != want).sum()) == 0
    ia.close()


@pytest.mark.parametrize("scale", [0.0371, 1.0, 3.0e-3, 777.7], ids=lambda v: f"s{v}")
def test_quantizer_quotients_next_to_half_integers_bit_exact(torch_mod, oracle, scale):
    """Elements whose quotient x / s lies on, or a few units in the last place beside, k + 1/2 for
    every k in -127..126 (where a shortcut for the division would round differently from the IEEE
    quotient), plus exact integers and random fill: the bytes of the oracle quantizer."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    s = np.float32(scale)
    amax = np.float32(127.0) * s  # the group maximum; s = amax / 127 may differ from `scale` in the last place
    s_eff = np.float32(amax / np.float32(127.0))
    vals = []
    for k in range(-127, 127):
        c = np.float32(np.float32(k + 0.5) * s_eff)
        x = c
        for _ in range(6):
            x = np.nextafter(x, np.float32(-np.inf), dtype=np.float32)
        for _ in range(13):
            vals.append(x)
            x = np.nextafter(x, np.float32(np.inf), dtype=np.float32)
        vals.append(np.float32(np.float32(k) * s_eff))
    vals = np.asarray(vals, dtype=np.float32)
    rng = np.random.default_rng(7)
    n = 2 * 2 * 64 * 64
    x = (rng.uniform(-1, 1, n).astype(np.float32) * amax).astype(np.float32)
    x[: vals.size] = vals
    x[-1] = amax
    x[-2] = -amax
    x = x.reshape(2, 2, 64, 64)
    tx = torch.from_numpy(x).to("cuda:0")
    ia = binding.IntAttn(device=0)
    for kw in (dict(), dict(per_head=True), dict(q_block=16)):
        got, sc = ia.quantize(tx, **kw)
        torch.cuda.synchronize()
        if "q_block" in kw:
            want, wsc = oracle.quantize_row_groups(x, 16)
        else:
            want, wsc = oracle.quantize(x, per_head=bool(kw))
        assert int((sc.cpu().numpy().reshape(-1) != wsc.reshape(-1)).sum()) == 0, kw
        assert int((got.cpu().numpy() != want).sum()) == 0, kw
    ia.close()


def test_quantizer_batch_equals_separate_calls_and_the_oracle(torch_mod, oracle):
    """intattn_quantize_batch on three tensors of different shapes, element types and scale modes (a
    ragged tail, a strided source): the bytes and scales of the oracle quantizer, tensor by tensor."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(101)
    dev = torch.device("cuda:0")
    xq = torch.from_numpy((rng.standard_normal((2, 6, 333, 128)) * 3.0).astype(np.float32)).to(dev).half()
    xk = torch.from_numpy((rng.standard_normal((2, 2, 1000, 128)) * np.asarray([1.0, 7.0])[None, :, None, None]).astype(np.float32)).to(dev)
    wide = torch.from_numpy(rng.standard_normal((2, 2, 77, 80)).astype(np.float32)).to(dev).bfloat16()
    xv = wide[:, :, :, :64]  # rows 160 bytes apart, 128 used
    ia = binding.IntAttn(device=0)
    outs, scs = ia.quantize_batch([xq, xk, xv], per_head=[False, True, True])
    torch.cuda.synchronize()
    for x, o, s, ph in zip((xq, xk, xv), outs, scs, (False, True, True)):
        want, wsc = oracle.quantize(x.float().cpu().numpy(), per_head=ph)
        assert int((s.cpu().numpy() != wsc).sum()) == 0
        assert int((o.cpu().numpy() != want).sum()) == 0
        single, ssc = ia.quantize(x, per_head=ph)
        torch.cuda.synchronize()
        assert torch.equal(single, o) and torch.equal(ssc, s)
    with pytest.raises(binding.IntAttnError):
        ia.quantize_batch([xq] * 5)
    ia.close()


def test_quantizer_to_dynamic_forward_without_host_reads(torch_mod, oracle):
    """fp16 Q, K, V -> on-GPU quantizer (per head) -> dynamic forward, all enqueued before the
    first synchronization: the bytes of the oracle quantizer followed by the oracle forward."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(79)
    B, Hq, Hkv, L, d = 2, 4, 2, 333, 128
    dev = torch.device("cuda:0")
    qf = torch.from_numpy(rng.standard_normal((B, Hq, L, d)).astype(np.float32)).to(dev).half()
    kf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to(dev).half()
    vf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to(dev).half()
    ia = binding.IntAttn(device=0)
    for per_head in (False, True):
        (q, sq), (k, sk), (v, sv) = (ia.quantize(t, per_head=per_head) for t in (qf, kf, vf))
        out = torch.empty_like(q)
        args, keep = ia.make_args(q, k, v, out, sq, sk, sv, None, causal=True, per_head=per_head, device_scales=True)
        ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert ia.dynamic_status() == 0
        oq, osq = oracle.quantize(qf.float().cpu().numpy(), per_head=per_head)
        ok, osk = oracle.quantize(kf.float().cpu().numpy(), per_head=per_head)
        ov, osv = oracle.quantize(vf.float().cpu().numpy(), per_head=per_head)
        want = oracle.forward(oq, ok, ov, osq, osk, osv, None, causal=True, per_head=per_head)["out"]
        assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


# ---------------------------------------------------------------- rectangular shapes (L query rows, Lkv keys)

def rect_problem(seed, B, Hq, Hkv, lq, lk, d, causal, per_head=False):
    """Seeded q [B,Hq,lq,d], k, v [B,Hkv,lk,d] with the value recipe of the square problems."""
    base = inputs.random_problem(seed, B, Hq, Hkv, max(lq, lk), d, causal, per_head=per_head, spread=1.5)
    q = np.ascontiguousarray(base.q[:, :, :lq])
    k = np.ascontiguousarray(base.k[:, :, :lk])
    v = np.ascontiguousarray(base.v[:, :, :lk])
    return base, q, k, v


def rect_forward(torch, ia, base, q, k, v, s_o=None, taps=True):
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    r = ia.forward(tq, tk, tv, base.s_q, base.s_k, base.s_v, s_o, causal=base.causal, per_head=base.per_head, taps=taps)
    torch.cuda.synchronize()
    return {k_: v_.cpu().numpy() for k_, v_ in r.items()} if taps else {"out": r.cpu().numpy()}


RECT_SHAPES = [
    # B, Hq, Hkv, Lq, Lkv, d, causal, per_head
    (1, 1, 1, 1, 1, 64, True, False),
    (2, 4, 2, 1, 300, 128, True, False),      # one decoded token
    (2, 4, 2, 1, 300, 64, False, True),
    (1, 2, 1, 5, 129, 64, True, False),
    (1, 4, 4, 128, 1000, 128, True, False),   # a chunk of a prefill, tile-aligned start ...
    (1, 2, 2, 100, 777, 64, True, True),      # ... and not
    (1, 2, 1, 333, 334, 128, True, False),
    (1, 3, 1, 200, 64, 64, False, False),     # more queries than keys (no mask)
    (1, 2, 2, 40, 515, 128, False, False),
]


@pytest.mark.parametrize("shape", RECT_SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{}ph{}".format(*[int(x) for x in s]))
def test_rectangular_shapes_bit_exact(torch_mod, ia, oracle, shape):
    """L != Lkv: every tap and the output equal the oracle's, for every kernel variant."""
    B, Hq, Hkv, lq, lk, d, causal, per_head = shape
    print(f"case {shape}", flush=True)
    base, q, k, v = rect_problem(500 + lq + lk, B, Hq, Hkv, lq, lk, d, causal, per_head)
    got = rect_forward(torch_mod, ia, base, q, k, v)
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=causal, per_head=per_head, taps=True)
    for key in ("row_max", "row_sum", "acc", "out"):
        assert got[key].shape == want[key].shape
        assert int((got[key] != want[key]).sum()) == 0, key


def test_decode_and_chunked_prefill_at_workload_size(torch_mod, oracle):
    """The GQA prefill workload's heads and key length (32 / 8 heads, 8192 keys, d = 128): one
    decoded token per sequence in full, and the last 2048-row chunk of the prefill on sampled rows,
    through the automatic variant."""
    from paper_2511_21513_amd import binding

    ia = binding.IntAttn(device=0)
    base, q, k, v = rect_problem(77, 1, 32, 8, 2048, 8192, 128, True, per_head=True)
    q1 = np.ascontiguousarray(q[:, :, :1])
    got = rect_forward(torch_mod, ia, base, q1, k, v, taps=False)["out"]
    want = oracle.forward(q1, k, v, base.s_q, base.s_k, base.s_v, None, causal=True, per_head=True, threads=16)["out"]
    assert int((got != want).sum()) == 0
    got = rect_forward(torch_mod, ia, base, q, k, v, taps=False)["out"]
    rng = np.random.default_rng(3)
    for hq in (0, 13, 31):
        rows = np.unique(np.concatenate([[0, 1, 127, 128, 2047], rng.integers(0, 2048, 6)])).astype(np.int32)
        w = oracle.rows(q, k, v, base.s_q, base.s_k, base.s_v, None, b=0, hq=hq, rows=rows, causal=True, per_head=True)
        assert int((got[0, hq][rows] != w["out"]).sum()) == 0, hq
    ia.close()


def test_rectangular_dynamic_forward(torch_mod, oracle):
    """Device-resident scales with L != Lkv."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    ia = binding.IntAttn(device=0)
    dev = torch.device("cuda:0")
    base, q, k, v = rect_problem(91, 2, 4, 2, 7, 260, 64, True, per_head=True)
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    sc = [torch.from_numpy(np.ascontiguousarray(s, dtype=np.float32)).to(dev) for s in (base.s_q, base.s_k, base.s_v)]
    out = torch.empty_like(tq)
    args, keep = ia.make_args(tq, tk, tv, out, sc[0], sc[1], sc[2], None, causal=True, per_head=True, device_scales=True)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    want = oracle.forward(q, k, v, base.s_q, base.s_k, base.s_v, None, causal=True, per_head=True)["out"]
    assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


SPLIT_KEY_SHAPES = [
    # B, Hq, Hkv, Lq, Lkv, d, causal: all take the split-key kernels ((Hq/Hkv) * Lq <= 31)
    (1, 31, 1, 1, 700, 64, True),        # 31 packed rows: the operand's last free row carries the ones
    (2, 12, 2, 5, 1500, 128, True),      # 30 packed rows, masks that differ per query row
    (4, 8, 4, 1, 20000, 128, True),      # 2512 tiles: two tiles per workgroup, odd tile count, ragged last tile
    (24, 8, 8, 2, 5000, 64, False),      # 7680 tiles: seven tiles per workgroup, no mask
    (1, 4, 4, 3, 131071, 64, True),      # the longest key sequence
    (32, 16, 4, 1, 16384, 64, True),     # 16 tiles per workgroup with 4 packed rows: the largest chunk the single launch holds
]


@pytest.mark.parametrize("shape", SPLIT_KEY_SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{}".format(*[int(x) for x in s]))
def test_split_key_kernels_bit_exact(torch_mod, oracle, shape):
    """Few query rows against many keys through the split-key kernels: several tiles per workgroup,
    full and nearly full operand, per-row masks; taps and output equal the oracle's, with host and
    with device-resident scales."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, Hq, Hkv, lq, lk, d, causal = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(lk + lq)
    q = rng.integers(-127, 128, size=(B, Hq, lq, d)).astype(np.int8)
    k = rng.integers(-127, 128, size=(B, Hkv, lk, d)).astype(np.int8)
    v = rng.integers(-127, 128, size=(B, Hkv, lk, d)).astype(np.int8)
    s_v = rng.uniform(0.01, 0.05, Hkv).astype(np.float32)
    s_o = (s_v[np.arange(Hq) // (Hq // Hkv)] * np.float32(0.05)).astype(np.float32)
    s_q0 = rng.uniform(0.004, 0.02, Hq).astype(np.float32)
    s_k0 = rng.uniform(0.004, 0.02, Hkv).astype(np.float32)
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    # thresholds of 10^5..10^6 (one launch with 32-bit scores in LDS) and of a few thousand (one launch, 16-bit
    # distances in LDS; the device-scale entry takes 32-bit scores); variant 10: the four launches
    for variant, mul in ((9, 1.0), (9, 8.0), (10, 8.0)):
        s_q, s_k = (s_q0 * np.float32(mul)).astype(np.float32), (s_k0 * np.float32(mul)).astype(np.float32)
        want = oracle.forward(q, k, v, s_q, s_k, s_v, s_o, causal=causal, per_head=True, taps=True, threads=16)
        ia = binding.IntAttn(device=0, variant=variant)
        for rep in range(2):  # the second call finds the group state as the first one left it
            got = ia.forward(tq, tk, tv, s_q, s_k, s_v, s_o, causal=causal, per_head=True, taps=True)
            torch.cuda.synchronize()
            for key in ("row_max", "row_sum", "acc", "out"):
                assert int((got[key].cpu().numpy() != want[key]).sum()) == 0, (variant, mul, rep, key)
        sc = [torch.from_numpy(x).to(dev) for x in (s_q, s_k, s_v, s_o)]
        out = torch.empty_like(tq)
        args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=causal, per_head=True, device_scales=True)
        ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want["out"]).sum()) == 0, (variant, mul)
        ia.close()


@pytest.mark.gpu
def test_split_key_wait_is_bounded_and_reserve_recovers(torch_mod, oracle, monkeypatch):
    """The one-launch split-key path with its wait bound forced to a single poll: the workgroups of the large
    groups give up instead of waiting, every kernel exits, and after intattn_reserve (which clears the
    counters they left behind) the same context computes the oracle's bytes again."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, Hq, Hkv, lq, lk, d = 1, 4, 4, 3, 131071, 64  # 256 workgroups per (batch, KV head) group
    rng = np.random.default_rng(77)
    q = rng.integers(-127, 128, size=(B, Hq, lq, d)).astype(np.int8)
    k = rng.integers(-127, 128, size=(B, Hkv, lk, d)).astype(np.int8)
    v = rng.integers(-127, 128, size=(B, Hkv, lk, d)).astype(np.int8)
    s_q = rng.uniform(0.03, 0.16, Hq).astype(np.float32)
    s_k = rng.uniform(0.03, 0.16, Hkv).astype(np.float32)
    s_v = rng.uniform(0.01, 0.05, Hkv).astype(np.float32)
    want = oracle.forward(q, k, v, s_q, s_k, s_v, None, causal=True, per_head=True, threads=16)["out"]
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    out = torch.empty_like(tq)
    ia = binding.IntAttn(device=0, variant=9)
    args, keep = ia.make_args(tq, tk, tv, out, s_q, s_k, s_v, None, causal=True, per_head=True)
    stream = torch.cuda.current_stream(dev).cuda_stream
    ia.forward_args(args, stream)
    torch.cuda.synchronize()
    assert int((out.cpu().numpy() != want).sum()) == 0
    print("bound of one poll", flush=True)
    monkeypatch.setenv("INTATTN_SPLITKEY_SPIN_LIMIT", "0")
    ia.forward_args(args, stream)
    torch.cuda.synchronize()  # returns: nothing waits for ever (the output of this call is undefined)
    monkeypatch.delenv("INTATTN_SPLITKEY_SPIN_LIMIT")
    print("reserve, then the full bound again", flush=True)
    ia.reserve(args)
    out.zero_()
    for _ in range(2):
        ia.forward_args(args, stream)
        torch.cuda.synchronize()
        assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


@pytest.mark.gpu
@pytest.mark.parametrize("ratio", [1.0, 1 / 30.0, 1 / 50.0, 1 / 64.0, 1 / 100.0, 1 / 1000.0, 255.0], ids=lambda r: f"so_over_sv_{r:.4g}")
def test_requantization_shift_range_bit_exact(torch_mod, oracle, ratio):
    """Output scales from s_V * 255 down to s_V / 1000: requantization shifts on both sides of 33, where the
    kernels change from the high word of the product to the 64-bit form, and outputs that saturate at +-127;
    tiled kernels, split-key kernels and device-resident scales."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    dev = torch.device("cuda:0")
    p = inputs.random_problem(17, 2, 4, 2, 300, 128, True, per_head=True, spread=1.1)
    s_o = (np.repeat(p.s_v, p.Hq // p.Hkv) * np.float32(ratio)).astype(np.float32)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, s_o, causal=True, per_head=True, threads=8)["out"]
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    for variant in (1, 3, 5):
        ia = binding.IntAttn(device=0, variant=variant)
        got = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=True, per_head=True)
        torch.cuda.synchronize()
        assert int((got.cpu().numpy() != want).sum()) == 0, variant
        sc = [torch.from_numpy(x).to(dev) for x in (p.s_q, p.s_k, p.s_v, s_o)]
        out = torch.empty_like(q)
        args, keep = ia.make_args(q, k, v, out, *sc, causal=True, per_head=True, device_scales=True)
        ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0, ("device scales", variant)
        ia.close()
    q1 = torch.from_numpy(np.ascontiguousarray(p.q[:, :, -2:])).to(dev)
    for variant in (9, 10):
        ia = binding.IntAttn(device=0, variant=variant)
        got = ia.forward(q1, k, v, p.s_q, p.s_k, p.s_v, s_o, causal=True, per_head=True)
        torch.cuda.synchronize()
        assert int((got.cpu().numpy() != want[:, :, -2:]).sum()) == 0, variant
        ia.close()


# ---------------------------------------------------------------- IndexSoftmax as an operator

SOFTMAX_SHAPES = [
    # rows, cols, c_int, causal rows_per_matrix (0: no mask)
    (1, 1, 37, 0), (3, 5, 1, 0), (84, 197, 5203, 0), (64, 256, 55064, 0), (33, 257, 37, 0), (40, 1000, 10**6, 20),
    (5, 2048, 5203, 5), (6, 2049, 2**30, 0), (4, 5000, 445, 2), (3, 16384, 5203, 3), (2, 16385, 28794, 0),
    (2, 70001, 5203, 2),
]


@pytest.mark.parametrize("shape", SOFTMAX_SHAPES, ids=lambda s: "r{}c{}ci{}m{}".format(*s))
def test_index_softmax_operator_bit_exact(torch_mod, oracle, shape):
    """Every row layout of the operator (a wave or a workgroup per row, resident or streamed),
    thresholds served by each index-map scheme, with and without the mask, rows with padding
    between them, and logits at the ends of the int32 range."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rows, cols, ci, rpm = shape
    print(f"case {shape}", flush=True)
    rng = np.random.default_rng(rows * 131 + cols)
    spread = max(4 * ci, 50) if ci < 2**28 else 2**30
    a = rng.integers(-spread, spread, size=(rows, cols), dtype=np.int64).astype(np.int32)
    a[0, :] = 11                         # equal logits
    if cols > 4:
        a[-1, 3] = 2**31 - 1             # the distance to the maximum exceeds 31 bits
        a[-1, 4] = -2**31
    want = oracle.index_softmax(a, ci, rows_per_matrix=rpm, causal=rpm > 0)
    ia = binding.IntAttn(device=0)
    dev = torch.device("cuda:0")
    got = ia.index_softmax(torch.from_numpy(a).to(dev), ci, causal=rpm > 0, rows_per_matrix=rpm)
    torch.cuda.synchronize()
    assert int((got.cpu().numpy() != want).sum()) == 0
    # rows with padding between them (strides that are not the row length)
    pad_c = (cols + 3) // 4 * 4 + 8
    buf = torch.zeros((rows, pad_c), dtype=torch.int32, device=dev)
    buf[:, :cols] = torch.from_numpy(a).to(dev)
    outbuf = torch.full((rows, pad_c), 7, dtype=torch.uint8, device=dev)
    ia.index_softmax(buf[:, :cols], ci, causal=rpm > 0, rows_per_matrix=rpm, out=outbuf[:, :cols])
    torch.cuda.synchronize()
    o = outbuf.cpu().numpy()
    assert int((o[:, :cols] != want).sum()) == 0 and (o[:, cols:] == 7).all()
    ia.close()


# ---------------------------------------------------------------- other table resolutions b and clip bounds c

@pytest.mark.parametrize("bc", [(1, 6.6), (2, 5.5), (3, 6.0), (4, 7.7), (5, 5.5), (5, 7.7), (6, 5.5), (6, 6.6), (6, 7.7)],
                         ids=lambda t: f"b{t[0]}c{t[1]}")
def test_other_lut_bits_and_clip(torch_mod, oracle, bc):
    """The (b, c) settings of the paper's sweep (Sec. 4, table resolution and clip bound): tiled
    kernels in one and in three launches, the split-key kernels, and the operator, against the
    oracle with the same (b, c)."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    b, c = bc
    dev = torch.device("cuda:0")
    p = inputs.random_problem(600 + b, 1, 4, 2, 300, 64, True, per_head=True, spread=1.5)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True, lut_bits=b, clip=c, taps=True)
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    for variant in (1, 2, 3, 4, 5):
        ia = binding.IntAttn(device=0, lut_bits=b, clip=c, variant=variant)
        got = ia.forward(q, k, v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True, taps=True)
        torch.cuda.synchronize()
        for key in ("row_sum", "acc", "out"):
            assert int((got[key].cpu().numpy() != want[key]).sum()) == 0, (variant, key)
        ia.close()
    # scales in device memory: the parameter kernel's search at this table size
    for variant in (1, 3, 5):
        ia = binding.IntAttn(device=0, lut_bits=b, clip=c, variant=variant)
        got, status = dynamic_forward(torch, ia, p)
        assert status == 0 and int((got != want["out"]).sum()) == 0, ("device scales", variant)
        ia.close()
    # one decoded token: the split-key kernels
    ia = binding.IntAttn(device=0, lut_bits=b, clip=c, variant=9)
    q1 = np.ascontiguousarray(p.q[:, :, :1])
    w1 = oracle.forward(q1, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True, lut_bits=b, clip=c)["out"]
    g1 = ia.forward(torch.from_numpy(q1).to(dev), k, v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True)
    torch.cuda.synchronize()
    assert int((g1.cpu().numpy() != w1).sum()) == 0
    # the operator on the logits of head 0
    logits = (p.q[0, 0].astype(np.int64) @ p.k[0, 0].astype(np.int64).T).astype(np.int32)
    ci = oracle.c_int(c, p.s_q[0], p.s_k[0], 64)
    wp = oracle.index_softmax(logits, ci, lut_bits=b, clip=c, rows_per_matrix=300, causal=True)
    gp = ia.index_softmax(torch.from_numpy(logits).to(dev), ci, causal=True, rows_per_matrix=300)
    torch.cuda.synchronize()
    assert int((gp.cpu().numpy() != wp).sum()) == 0
    ia.close()


# ---------------------------------------------------------------- finer quantization groups over query rows

ROW_GROUP_SHAPES = [
    # B, Hq, Hkv, Lq, Lkv, d, causal, q_block, with an output scale per group
    (1, 2, 1, 37, 37, 64, True, 1, False),       # per token
    (2, 4, 2, 150, 150, 128, True, 1, True),
    (1, 4, 4, 300, 300, 64, False, 7, True),     # blocks that straddle waves and tiles
    (1, 2, 2, 260, 260, 128, True, 64, False),
    (2, 2, 1, 40, 333, 64, True, 16, True),      # a chunk of queries against a longer key sequence
]


@pytest.mark.parametrize("shape", ROW_GROUP_SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{}qb{}so{}".format(*[int(x) for x in s]))
def test_row_group_scales_bit_exact(torch_mod, ia, oracle, shape):
    """Scale mode 2 (Sec. 3.3, groups = blocks of query rows, per token at q_block = 1): every row
    follows its group's c_int and requantization; all kernel variants, device-resident scales."""
    torch = torch_mod
    B, Hq, Hkv, lq, lk, d, causal, qb, with_so = shape
    print(f"case {shape}", flush=True)
    base, q, k, v = rect_problem(700 + lq + qb, B, Hq, Hkv, lq, lk, d, causal, per_head=True)
    rng = np.random.default_rng(qb + lq)
    nblk = (lq + qb - 1) // qb
    s_q = (base.s_q[None, :, None] * rng.uniform(0.3, 2.5, size=(B, Hq, nblk))).astype(np.float32)
    s_q[0, 0, 0] *= np.float32(1e-3)  # one group far beyond the reach of the 24-bit and fp32 index maps
    s_o = (base.s_v[np.arange(Hq) // (Hq // Hkv)][None, :, None] * rng.uniform(0.02, 0.2, size=(B, Hq, nblk))).astype(np.float32) if with_so else None
    want = oracle.forward_row_groups(q, k, v, s_q, base.s_k, base.s_v, s_o, q_block=qb, causal=causal, taps=True)
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    sc = [torch.from_numpy(np.ascontiguousarray(x)).to(dev) if x is not None else None for x in (s_q, base.s_k, base.s_v, s_o)]
    out = torch.empty_like(tq)
    taps = {"row_max": torch.zeros((B, Hq, lq), dtype=torch.int32, device=dev),
            "row_sum": torch.zeros((B, Hq, lq), dtype=torch.int32, device=dev),
            "acc": torch.zeros((B, Hq, lq, d), dtype=torch.int32, device=dev)}
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=causal, device_scales=True, q_block=qb, **taps)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0
    for key in ("row_max", "row_sum", "acc"):
        assert int((taps[key].cpu().numpy() != want[key]).sum()) == 0, key
    assert int((out.cpu().numpy() != want["out"]).sum()) == 0


KEY_GROUP_SHAPES = [
    # B, Hq, Hkv, Lq, Lkv, d, causal, q_block, k_block, with an output scale per group of query rows
    (1, 2, 1, 37, 37, 64, True, 1, 1, False),        # per token x per key ("per channel")
    (2, 4, 2, 150, 150, 128, True, 16, 32, True),    # blocks of 32 keys: one group per MFMA sub-tile
    (1, 4, 4, 300, 300, 64, False, 300, 64, True),   # one query scale per head, 64-key blocks, no mask
    (1, 2, 2, 260, 260, 128, True, 64, 7, False),    # key blocks that straddle sub-tiles and tiles
    (2, 2, 1, 40, 333, 64, True, 8, 128, True),      # a chunk of queries against a longer key sequence
    (1, 2, 1, 600, 600, 128, True, 600, 96, False),  # more than 512 keys
    (1, 1, 1, 130, 130, 64, False, 5, 1, True),
]


def key_group_problem(seed, B, Hq, Hkv, lq, lk, d, qb, kb, with_so):
    """INT8 tensors with scales per block of query rows and per block of keys that differ by up to 25x
    (one pair far apart, so that the image of the row maximum leaves a block's 32-bit range)."""
    rng = np.random.default_rng(seed)
    q = rng.integers(-127, 128, (B, Hq, lq, d), dtype=np.int8)
    k = rng.integers(-127, 128, (B, Hkv, lk, d), dtype=np.int8)
    v = rng.integers(-127, 128, (B, Hkv, lk, d), dtype=np.int8)
    nqb, nkb = -(-lq // qb), -(-lk // kb)
    s_q = (0.02 * np.exp(rng.uniform(np.log(0.2), np.log(5.0), size=(B, Hq, nqb)))).astype(np.float32)
    s_k = (0.02 * np.exp(rng.uniform(np.log(0.2), np.log(5.0), size=(B, Hkv, nkb))) / np.sqrt(d / 64)).astype(np.float32)
    if nkb > 1:
        s_k[0, 0, nkb - 1] *= np.float32(1e-6)  # m^(g) of this block lies far above its logits: everything clipped
    s_v = rng.uniform(0.01, 0.03, size=Hkv).astype(np.float32)
    s_o = (s_v[np.arange(Hq) // (Hq // Hkv)][None, :, None] * rng.uniform(0.02, 0.2, size=(B, Hq, nqb))).astype(np.float32) if with_so else None
    return q, k, v, s_q, s_k, s_v, s_o


def key_group_forward(torch, ia, q, k, v, s_q, s_k, s_v, s_o, causal, qb, kb):
    dev = torch.device("cuda:0")
    B, Hq, lq, d = q.shape
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    sc = [torch.from_numpy(np.ascontiguousarray(x)).to(dev) if x is not None else None for x in (s_q, s_k, s_v, s_o)]
    out = torch.full(q.shape, 99, dtype=torch.int8, device=dev)
    taps = {"row_sum": torch.zeros((B, Hq, lq), dtype=torch.int32, device=dev),
            "acc": torch.zeros((B, Hq, lq, d), dtype=torch.int32, device=dev)}
    args, keep = ia.make_args(tq, tk, tv, out, *sc, causal=causal, device_scales=True, q_block=qb, k_block=kb, **taps)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    return out.cpu().numpy(), {key: t.cpu().numpy() for key, t in taps.items()}, ia.dynamic_status()


@pytest.mark.parametrize("shape", KEY_GROUP_SHAPES, ids=lambda s: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{:d}qb{}kb{}so{:d}".format(*s))
def test_key_group_scales_bit_exact(torch_mod, oracle, shape):
    """Scale mode 3 (Sec. 3.3, groups over query rows and over keys; per key at k_block = 1): row
    sums, accumulators and output bytes of the oracle for the same reading, whatever kernel variant
    the context names (the mode runs its own single-launch kernel)."""
    from paper_2511_21513_amd import binding

    B, Hq, Hkv, lq, lk, d, causal, qb, kb, with_so = shape
    print(f"case {shape}", flush=True)
    q, k, v, s_q, s_k, s_v, s_o = key_group_problem(900 + lq + kb, B, Hq, Hkv, lq, lk, d, qb, kb, with_so)
    want = oracle.forward_groups(q, k, v, s_q, s_k, s_v, s_o, q_block=qb, k_block=kb, causal=causal, taps=True)
    for variant in (0, 5):
        ia = binding.IntAttn(device=0, variant=variant)
        out, taps, status = key_group_forward(torch_mod, ia, q, k, v, s_q, s_k, s_v, s_o, causal, qb, kb)
        ia.close()
        assert status == 0
        for key in ("row_sum", "acc"):
            assert int((taps[key] != want[key]).sum()) == 0, (variant, key)
        assert int((out != want["out"]).sum()) == 0, variant
    assert np.abs(want["out"]).max() > 5


def test_key_groups_with_equal_scales_equal_the_per_head_forward(torch_mod, oracle):
    """With one scale value in every group the mode must reproduce the per-head forward (and oracle)."""
    from paper_2511_21513_amd import binding

    p = inputs.random_problem(97, 2, 4, 2, 200, 64, True, per_head=True, spread=1.5)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=True, per_head=True)["out"]
    ia = binding.IntAttn(device=0)
    for qb, kb in ((1, 1), (200, 32), (13, 50)):
        nqb, nkb = -(-200 // qb), -(-200 // kb)
        s_q = np.broadcast_to(p.s_q[None, :, None], (2, 4, nqb)).copy()
        s_k = np.broadcast_to(p.s_k[None, :, None], (2, 2, nkb)).copy()
        out, _, status = key_group_forward(torch_mod, ia, p.q, p.k, p.v, s_q, s_k, p.s_v, None, True, qb, kb)
        assert status == 0 and int((out != want).sum()) == 0, (qb, kb)
    ia.close()


def test_key_groups_report_unusable_scales(torch_mod, oracle):
    """A key block with a zero, negative, infinite or NaN scale: status 1, that KV head's query heads
    all zeros, the other heads as the oracle says; nothing faults."""
    from paper_2511_21513_amd import binding

    B, Hq, Hkv, L, d, qb, kb = 1, 4, 2, 130, 64, 16, 32
    q, k, v, s_q, s_k, s_v, s_o = key_group_problem(5, B, Hq, Hkv, L, L, d, qb, kb, False)
    want = oracle.forward_groups(q, k, v, s_q, s_k, s_v, None, q_block=qb, k_block=kb, causal=True)["out"]
    ia = binding.IntAttn(device=0)
    for bad in (0.0, -1.0, np.inf, np.nan):
        s2 = s_k.copy()
        s2[0, 1, 2] = bad  # KV head 1 serves query heads 2 and 3
        out, _, status = key_group_forward(torch_mod, ia, q, k, v, s_q, s2, s_v, None, True, qb, kb)
        assert status == 1
        assert not out[:, 2:].any() and int((out[:, :2] != want[:, :2]).sum()) == 0
    out, _, status = key_group_forward(torch_mod, ia, q, k, v, s_q, s_k, s_v, None, True, qb, kb)
    assert status == 0 and int((out != want).sum()) == 0
    ia.close()


def test_per_block_quantizers_feed_the_key_group_forward(torch_mod, oracle):
    """fp16 Q quantized per block of 32 query rows and K per block of 64 keys on the GPU (V per head),
    then the forward on those device-resident scales, nothing read by the host in between: the bytes
    of the oracle's per-block quantizer followed by the oracle for groups over both axes."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(89)
    B, Hq, Hkv, L, d, qb, kb = 2, 4, 2, 300, 128, 32, 64
    dev = torch.device("cuda:0")
    qf = torch.from_numpy((rng.standard_normal((B, Hq, L, d)) * rng.uniform(0.2, 5.0, size=(B, Hq, L, 1))).astype(np.float32)).to(dev).half()
    kf = torch.from_numpy((rng.standard_normal((B, Hkv, L, d)) * rng.uniform(0.2, 5.0, size=(B, Hkv, L, 1))).astype(np.float32)).to(dev).half()
    vf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to(dev).half()
    ia = binding.IntAttn(device=0)
    q, sq = ia.quantize(qf, q_block=qb)
    k, sk = ia.quantize(kf, q_block=kb)
    v, sv = ia.quantize(vf, per_head=True)
    out = torch.empty_like(q)
    args, keep = ia.make_args(q, k, v, out, sq, sk, sv, None, causal=True, device_scales=True, q_block=qb, k_block=kb)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0
    oq, osq = oracle.quantize_row_groups(qf.float().cpu().numpy(), qb)
    ok, osk = oracle.quantize_row_groups(kf.float().cpu().numpy(), kb)
    ov, osv = oracle.quantize(vf.float().cpu().numpy(), per_head=True)
    want = oracle.forward_groups(oq, ok, ov, osq, osk, osv, None, q_block=qb, k_block=kb, causal=True)["out"]
    assert int((q.cpu().numpy() != oq).sum()) == 0 and int((k.cpu().numpy() != ok).sum()) == 0
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


@pytest.mark.parametrize("case", [(2, 3, 50, 64, "float16", 1), (1, 2, 77, 128, "float32", 5), (1, 4, 300, 128, "bfloat16", 64),
                                  (2, 2, 33, 8, "float32", 1), (1, 1, 100, 64, "float16", 1000)],
                         ids=lambda c: "B{}H{}L{}d{}{}qb{}".format(*c))
def test_row_group_quantizer_bit_exact(torch_mod, oracle, case):
    """Eq. quant with one scale per block of rows (per token at q_block = 1): bytes and scales equal
    the per-tensor oracle quantizer applied to each block; a wave or a workgroup per group."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, H, L, d, dt, qb = case
    rng = np.random.default_rng(L + d + qb)
    x = (rng.standard_normal((B, H, L, d)) * rng.uniform(0.1, 10.0, size=(B, H, L, 1))).astype(np.float32)
    x[0, 0, 0] = 0.0  # an all-zero token
    tx = torch.from_numpy(x).to("cuda:0").to(getattr(torch, dt))
    ia = binding.IntAttn(device=0)
    got, sc = ia.quantize(tx, q_block=qb)
    torch.cuda.synchronize()
    want, wsc = oracle.quantize_row_groups(tx.float().cpu().numpy(), qb)
    assert sc.shape == wsc.shape
    assert int((sc.cpu().numpy() != wsc).sum()) == 0
    assert int((got.cpu().numpy() != want).sum()) == 0
    ia.close()


def test_per_token_quantizer_feeds_the_row_group_forward(torch_mod, oracle):
    """fp16 Q quantized per token on the GPU, K and V per head, then the forward on those
    device-resident scales: the bytes of the oracle quantizers followed by the row-group oracle."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(83)
    B, Hq, Hkv, L, d = 2, 4, 2, 200, 128
    dev = torch.device("cuda:0")
    qf = torch.from_numpy((rng.standard_normal((B, Hq, L, d)) * rng.uniform(0.2, 5.0, size=(B, Hq, L, 1))).astype(np.float32)).to(dev).half()
    kf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to(dev).half()
    vf = torch.from_numpy(rng.standard_normal((B, Hkv, L, d)).astype(np.float32)).to(dev).half()
    ia = binding.IntAttn(device=0)
    q, sq = ia.quantize(qf, q_block=1)
    (k, sk), (v, sv) = (ia.quantize(t, per_head=True) for t in (kf, vf))
    out = torch.empty_like(q)
    args, keep = ia.make_args(q, k, v, out, sq, sk, sv, None, causal=True, device_scales=True, q_block=1)
    ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
    torch.cuda.synchronize()
    assert ia.dynamic_status() == 0
    oq, osq = oracle.quantize_row_groups(qf.float().cpu().numpy(), 1)
    ok, osk = oracle.quantize(kf.float().cpu().numpy(), per_head=True)
    ov, osv = oracle.quantize(vf.float().cpu().numpy(), per_head=True)
    want = oracle.forward_row_groups(oq, ok, ov, osq, osk, osv, None, q_block=1, causal=True)["out"]
    assert int((out.cpu().numpy() != want).sum()) == 0
    ia.close()


# ---------------------------------------------------------------- seeded random sweep over shapes, modes and variants

def _random_cases(n, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for _ in range(n):
        g = int(rng.choice([1, 1, 2, 4, 8]))
        Hkv = int(rng.integers(1, 4))
        causal = bool(rng.integers(0, 2))
        lk = int(rng.choice([1, 2, 31, 33, 64, 127, 129, 200, 257, 400, 1100]))
        lq = int(rng.integers(1, lk + 1)) if causal else int(rng.choice([1, 3, 32, 65, 130, 300]))
        if rng.integers(0, 3) == 0:
            lq = lk
        cases.append((int(rng.integers(1, 3)), g * Hkv, Hkv, lq, lk, int(rng.choice([64, 128])), causal,
                      int(rng.integers(0, 3)),           # scale mode: per tensor, per head, per block of rows
                      int(rng.choice([1, 3, 32, 50])),   # q_block (mode 2)
                      int(rng.choice([0, 1, 2, 3, 4, 5, 9, 5, 0, 3, 1])),  # kernel variant
                      bool(rng.integers(0, 2)),          # with an output scale
                      float(rng.choice([1.0, 1.0, 0.05, 1e-3]))))  # multiplier on s_q: moves c_int between the schemes
    return cases


@pytest.mark.parametrize("case", _random_cases(48, 2024), ids=lambda c: "B{}Hq{}Hkv{}Lq{}Lk{}d{}c{}m{}qb{}v{}so{}x{}".format(*[int(x) if not isinstance(x, float) else x for x in c]))
def test_random_shapes_modes_variants(torch_mod, oracle, case):
    """A seeded sweep over shapes (square, rectangular, single rows), masks, GQA ratios, scale modes,
    kernel variants and thresholds: host scales through intattn_forward where the mode has them,
    device scales through intattn_forward_dynamic, both against the oracle."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    B, Hq, Hkv, lq, lk, d, causal, mode, qb, variant, with_so, mul = case
    print(f"case {case}", flush=True)
    base, q, k, v = rect_problem(900 + lq + lk + Hq, B, Hq, Hkv, lq, lk, d, causal, per_head=(mode != 0))
    rng = np.random.default_rng(lq * 7 + lk)
    grp = np.arange(Hq) // (Hq // Hkv)
    dev = torch.device("cuda:0")
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    ia = binding.IntAttn(device=0, variant=variant)
    up = lambda x: None if x is None else torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(dev)
    if mode == 2:
        nblk = (lq + qb - 1) // qb
        s_q = (base.s_q[None, :, None] * mul * rng.uniform(0.5, 2.0, size=(B, Hq, nblk))).astype(np.float32)
        s_o = (base.s_v[grp][None, :, None] * rng.uniform(0.02, 0.3, size=(B, Hq, nblk))).astype(np.float32) if with_so else None
        want = oracle.forward_row_groups(q, k, v, s_q, base.s_k, base.s_v, s_o, q_block=qb, causal=causal)["out"]
        out = torch.empty_like(tq)
        args, keep = ia.make_args(tq, tk, tv, out, up(s_q), up(base.s_k), up(base.s_v), up(s_o), causal=causal,
                                  device_scales=True, q_block=qb)
        ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0
    else:
        per_head = mode == 1
        s_q = (base.s_q * mul).astype(np.float32)
        s_o = None
        if with_so:
            s_o = (base.s_v[grp] * 0.1).astype(np.float32) if per_head else (base.s_v * 0.1).astype(np.float32)
        want = oracle.forward(q, k, v, s_q, base.s_k, base.s_v, s_o, causal=causal, per_head=per_head)["out"]
        got = ia.forward(tq, tk, tv, s_q, base.s_k, base.s_v, s_o, causal=causal, per_head=per_head)
        torch.cuda.synchronize()
        assert int((got.cpu().numpy() != want).sum()) == 0, "host scales"
        out = torch.empty_like(tq)
        args, keep = ia.make_args(tq, tk, tv, out, up(s_q), up(base.s_k), up(base.s_v), up(s_o), causal=causal,
                                  per_head=per_head, device_scales=True)
        ia.forward_dynamic_args(args, torch.cuda.current_stream(dev).cuda_stream)
        torch.cuda.synchronize()
        assert ia.dynamic_status() == 0 and int((out.cpu().numpy() != want).sum()) == 0, "device scales"
    ia.close()


def test_parameter_cache_follows_the_scales(torch_mod, oracle):
    """The context keeps the parameters derived from the last call's host scales; a call with other
    scales (any one value, the output scale appearing or disappearing, the scale mode) must not
    see them."""
    from paper_2511_21513_amd import binding

    torch = torch_mod
    p = inputs.random_problem(123, 1, 4, 2, 140, 64, True, per_head=True, spread=1.5)
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in (p.q, p.k, p.v))
    ia = binding.IntAttn(device=0)
    s_o = inputs.calibrated_out_scale(p)
    sq2 = p.s_q.copy()
    sq2[3] *= np.float32(1.0000001) if sq2[3] * np.float32(1.0000001) != sq2[3] else np.float32(1.001)
    runs = [(p.s_q, None, True), (p.s_q, None, True), (sq2, None, True), (p.s_q, s_o, True), (p.s_q, None, True),
            (p.s_q[:1], None, False), (p.s_q, None, True)]
    for s_q, so, per_head in runs:
        sk, sv = (p.s_k, p.s_v) if per_head else (p.s_k[:1], p.s_v[:1])
        so_ = so if per_head or so is None else so[:1]
        got = ia.forward(q, k, v, s_q, sk, sv, so_, causal=True, per_head=per_head)
        torch.cuda.synchronize()
        want = oracle.forward(p.q, p.k, p.v, s_q, sk, sv, so_, causal=True, per_head=per_head)["out"]
        assert int((got.cpu().numpy() != want).sum()) == 0
    ia.close()


# ---------------------------------------------------------------- sweep C on rows with large and small sums
@pytest.mark.parametrize("case", [
    # L, d, causal, spread, per_head: flat logits make the row sums large, so that only the first eight table
    # entries of a row can give a nonzero probability
    (1500, 128, True, 0.6, False), (1500, 64, False, 0.6, True), (2048, 64, True, 1.0, False),
    (900, 128, True, 0.35, False), (700, 128, False, 2.0, False),
], ids=lambda c: "L{}d{}c{}s{}ph{}".format(c[0], c[1], int(c[2]), c[3], int(c[4])))
def test_short_table_path_bit_exact(torch_mod, oracle, case):
    """Rows whose sum of E_hat exceeds 510 * LUT_hat[8], rows below it, and waves and workgroups that mix both:
    every tap and every output byte against the oracle, on diagonal (masked) and ragged tiles too."""
    from paper_2511_21513_amd import binding

    L, d, causal, spread, per_head = case
    p = inputs.random_problem(77, 1, 4, 2, L, d, causal, per_head=per_head, spread=spread)
    want = oracle.forward(p.q, p.k, p.v, p.s_q, p.s_k, p.s_v, None, causal=causal, per_head=per_head, taps=True, threads=8)
    n_short = int((want["row_sum"] > 510 * 46).sum())
    print(f"case {case}: {n_short} of {want['row_sum'].size} rows above the short-table threshold", flush=True)
    if spread < 2.0:
        assert n_short > want["row_sum"].size // 5  # the case does exercise the path
    ia = binding.IntAttn(device=0, variant=5)
    check_full(torch_mod, ia, oracle, p)
    check_full(torch_mod, ia, oracle, p, inputs.calibrated_out_scale(p), taps=False)
    ia.close()


def test_short_table_path_on_the_headline_distribution(torch_mod, oracle):
    """Four query heads of the long-context GQA workload at a ragged length: small threshold, late rows with large sums,
    early rows with small ones."""
    from paper_2511_21513_amd import binding

    p = inputs.make_problem("c4_gqa_prefill_8k", Hq=4, Hkv=1, L=5000)
    s_o = inputs.calibrated_out_scale(p, sample_rows=16)
    for variant in (0, 5):
        ia = binding.IntAttn(device=0, variant=variant)
        check_full(torch_mod, ia, oracle, p, s_o, taps=False)
        ia.close()
    ia = binding.IntAttn(device=0, variant=5)
    got = check_full(torch_mod, ia, oracle, p)
    ia.close()
    assert int((got["row_sum"] > 510 * 46).sum()) > got["row_sum"].size // 4
