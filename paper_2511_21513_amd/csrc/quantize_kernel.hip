// Dynamic symmetric INT8 quantizer in front of the attention path (Sec. 2.1, Eq. quant) for gfx950:
//   s_X = max|X| / 127 per tensor (or per head index, Sec. 3.3),  X_hat = clamp(round(X / s_X), -127, 127).
// fp32, fp16 or bf16 in, INT8 and the fp32 scales (device memory) out.  Two passes over the input,
// both bound by HBM: (1) max|X| of each workgroup's part of a (b, h) slice, 16-byte loads, reduced
// per wave and per workgroup and stored (no atomics: two thousand updates of one word cost more
// than reading the tensor); (2) every workgroup reduces the partial maxima of its group, then one
// IEEE fp32 division per element (done as a multiplication where that provably rounds alike, see quantize8),
// nearest integer with ties to even (v_rndne_f32), eight INT8 results per 8-byte store.  Up to four tensors (Q, K, V) share the two launches: a flat grid whose
// workgroups find their tensor from cumulative counts.  The second pass walks the grid backwards, so
// that it starts in what the first pass left in the caches.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace {

constexpr int QNT = 256;   // threads per workgroup
constexpr int QITEMS = 4;  // 8-element items per thread in flight
constexpr int QLOOP_MAX = 4; // rounds of QITEMS items per thread in the second pass, which share one reduction of the partial maxima
// Workgroups that the second pass is cut into where the tensors allow: six a compute unit.  (Always four rounds: Q, K, V of 2 x
// 2048 tokens, 32 / 8 heads, fp16, 29.7 us for both passes, now 28.0; V of 1024 tokens, 8 heads, 14.7 -> 8.7; 3 x 100 tokens, 8
// heads, 10.3 -> 7.7.  3072 workgroups: 29.7, 8.7, 7.8.)
constexpr int64_t QWGS = 1536;
constexpr int RHOLD = 8;   // items per thread that quantize_rows_kernel holds between its two passes

// eight consecutive elements of a row as they are in memory, and as fp32 (widening fp16 / bf16 is exact)
template <int DTYPE> struct Raw8 {
    uint4 v[DTYPE == 0 ? 2 : 1];
};
template <int DTYPE> __device__ __forceinline__ Raw8<DTYPE> load_raw8(const uint8_t *p)
{
    Raw8<DTYPE> r;
    r.v[0] = *(const uint4 *)p;
    if constexpr (DTYPE == 0) r.v[1] = *(const uint4 *)(p + 16);
    return r;
}
template <int DTYPE> __device__ __forceinline__ void widen8(const Raw8<DTYPE> &raw, float (&x)[8])
{
    const uint32_t w[4] = {raw.v[0].x, raw.v[0].y, raw.v[0].z, raw.v[0].w};
    if constexpr (DTYPE == 0) {
        const uint32_t u[4] = {raw.v[1].x, raw.v[1].y, raw.v[1].z, raw.v[1].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(w[i]), x[4 + i] = __uint_as_float(u[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (DTYPE == 1) {
                x[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] & 0xffffu));
                x[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] >> 16));
            } else {
                x[2 * i] = __uint_as_float(w[i] << 16);
                x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
            }
        }
    }
}
template <int DTYPE> __device__ __forceinline__ void load8(const uint8_t *p, float (&x)[8])
{
    widen8<DTYPE>(load_raw8<DTYPE>(p), x);
}

// Eight elements to INT8: q = clamp(rint(x / s), -127, 127) with x / s the IEEE fp32 quotient and rint to nearest,
// ties to even -- two words of four bytes.  The division is replaced by a multiplication wherever that provably gives
// the same integer: with r = fl(1 / s) (one IEEE division per group) and t = fl(x r), t differs from fl(x / s) by at
// most |x / s| * 3 * 2^-24 (1 + 2^-23) < 2.3e-5 (|x / s| <= 127.5: x is an element of the group whose maximum defines
// s), so whenever t is farther than 2^-14 from every half-integer, t and fl(x / s) lie strictly between the same two
// half-integers and round to the same integer.  Items with an element closer than that (about 1 in 25 for random data)
// take the division itself; the branch is per item of eight elements.
__device__ __forceinline__ void quantize8(const float (&x)[8], float s, float r, uint32_t (&w)[2])
{
    float t[8];
    bool near = false;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        t[i] = x[i] * r;
        const float f = t[i] - __builtin_floorf(t[i]); // in [0, 1]
        near |= __builtin_fabsf(f - 0.5f) < 6.103515625e-05f;
    }
    if (near) {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = x[i] / s; // IEEE division
    }
    w[0] = w[1] = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float q = __builtin_rintf(t[i]); // nearest integer, ties to even
        q = fminf(fmaxf(q, -127.0f), 127.0f);
        w[i / 4] |= ((uint32_t)(int)q & 0xffu) << (8 * (i % 4));
    }
}

// Byte offsets of item `it` (eight elements) inside a (b, h) slice.  Rows that follow each other
// without gaps need no division; the host checked that the item count fits 31 bits.
template <int ES>
__device__ __forceinline__ void item_offsets(const QuantParams &p, uint32_t it, uint32_t ipr, int64_t &so, int64_t &dofs)
{
    if (p.ss[2] == (int64_t)p.d * ES && p.ds[2] == (int64_t)p.d) { // wave-uniform
        so = (int64_t)it * 8 * ES;
        dofs = (int64_t)it * 8;
    } else {
        const uint32_t row = it / ipr, c = it - row * ipr;
        so = (int64_t)row * p.ss[2] + (int64_t)c * 8 * ES;
        dofs = (int64_t)row * p.ds[2] + (int64_t)c * 8;
    }
}

// Tensor and position of a workgroup in the flat grid of a batch: workgroups [first[i], first[i + 1])
// belong to tensor i and are numbered x-fastest inside it.
struct BatchSlot {
    int ti;
    uint32_t bx, by;
};
__device__ __forceinline__ BatchSlot batch_slot(const QuantBatch &qb, uint32_t lin, const uint32_t (&gx)[4])
{
    int ti = 0;
#pragma unroll
    for (int i = 1; i < 4; ++i)
        if (i < qb.n && lin >= qb.first[i]) ti = i;
    const uint32_t rel = lin - qb.first[ti];
    return BatchSlot{ti, rel % gx[ti], rel / gx[ti]};
}

// by = b * H + h; bx walks the (L * d / 8) items of that slice.
template <int DTYPE>
__device__ __forceinline__ void absmax_body(const QuantParams &p, uint32_t bx, uint32_t gdx, uint32_t by)
{
    constexpr int ES = DTYPE == 0 ? 4 : 2;
    __shared__ float wmax[QNT / 64];
    const int bh = (int)by, b = bh / p.H, h = bh % p.H;
    const uint8_t *src = (const uint8_t *)p.src + (int64_t)b * p.ss[0] + (int64_t)h * p.ss[1];
    const int ipr = p.d / 8; // items per row
    const int64_t items = (int64_t)p.L * ipr;
    float m = 0.0f;
    // grid-stride walk, QITEMS loads in flight per thread
    for (int64_t base = (int64_t)bx * QNT + threadIdx.x; base < items; base += (int64_t)gdx * QNT * QITEMS) {
        float x[QITEMS][8];
#pragma unroll
        for (int j = 0; j < QITEMS; ++j) {
            const int64_t it = base + (int64_t)j * gdx * QNT;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[j][i] = 0.0f;
            if (it < items) {
                int64_t so, dofs;
                item_offsets<ES>(p, (uint32_t)it, (uint32_t)ipr, so, dofs);
                load8<DTYPE>(src + so, x[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < QITEMS; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(x[j][i]));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < QNT / 64; ++w) m = fmaxf(m, wmax[w]);
        p.partial[(int64_t)bh * gdx + bx] = m;
    }
}

__global__ __launch_bounds__(QNT) void absmax_kernel(const QuantBatch qb)
{
    uint32_t gx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) gx[i] = (uint32_t)qb.t[i].n_partial;
    const BatchSlot sl = batch_slot(qb, blockIdx.x, gx);
    const QuantParams &p = qb.t[sl.ti];
    if (p.dtype == 0) absmax_body<0>(p, sl.bx, gx[sl.ti], sl.by);
    else if (p.dtype == 1) absmax_body<1>(p, sl.bx, gx[sl.ti], sl.by);
    else absmax_body<2>(p, sl.bx, gx[sl.ti], sl.by);
}

template <int DTYPE>
__device__ __forceinline__ void quantize_body(const QuantParams &p, int loops, uint32_t bx, uint32_t by)
{
    constexpr int ES = DTYPE == 0 ? 4 : 2;
    const int bh = (int)by, b = bh / p.H, h = bh % p.H;
    const int g = p.per_head ? h : 0;
    // max|X| of the group from the partial maxima: slices (b', h') with h' = h, or all slices
    __shared__ float wmax[QNT / 64];
    float m = 0.0f;
    if (p.per_head) {
        for (int i = threadIdx.x; i < p.B * p.n_partial; i += QNT)
            m = fmaxf(m, p.partial[((int64_t)(i / p.n_partial) * p.H + h) * p.n_partial + i % p.n_partial]);
    } else {
        for (int i = threadIdx.x; i < p.B * p.H * p.n_partial; i += QNT) m = fmaxf(m, p.partial[i]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < QNT / 64; ++w) m = fmaxf(m, wmax[w]);
    const float amax = fmaxf(m, 1e-12f);
    const float s = amax / 127.0f; // one IEEE fp32 division
    const float rs = 1.0f / s;     // and its reciprocal, for quantize8
    if (bx == 0 && threadIdx.x == 0 && b == 0 && (p.per_head || h == 0)) p.scales[g] = s;
    const uint8_t *src = (const uint8_t *)p.src + (int64_t)b * p.ss[0] + (int64_t)h * p.ss[1];
    int8_t *dst = p.dst + (int64_t)b * p.ds[0] + (int64_t)h * p.ds[1];
    const int ipr = p.d / 8;
    const int64_t items = (int64_t)p.L * ipr;
    for (int r = 0; r < loops; ++r) {
        // QITEMS loads in flight per thread, then the arithmetic and the stores
        float x[QITEMS][8];
        int64_t dofs[QITEMS];
        bool live[QITEMS];
#pragma unroll
        for (int j = 0; j < QITEMS; ++j) {
            const int64_t it = ((int64_t)(bx * (uint32_t)loops + r) * QITEMS + j) * QNT + threadIdx.x;
            live[j] = it < items;
            dofs[j] = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[j][i] = 0.0f;
            if (live[j]) {
                int64_t so;
                item_offsets<ES>(p, (uint32_t)it, (uint32_t)ipr, so, dofs[j]);
                load8<DTYPE>(src + so, x[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < QITEMS; ++j) {
            uint32_t w[2];
            quantize8(x[j], s, rs, w);
            if (live[j]) *(uint2 *)(dst + dofs[j]) = make_uint2(w[0], w[1]);
        }
    }
}

__global__ __launch_bounds__(QNT) void quantize_kernel(const QuantBatch qb)
{
    uint32_t gx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) gx[i] = qb.gx[i];
    const BatchSlot sl = batch_slot(qb, qb.first[qb.n] - 1u - blockIdx.x, gx); // backwards through the grid
    const QuantParams &p = qb.t[sl.ti];
    if (p.dtype == 0) quantize_body<0>(p, qb.loops, sl.bx, sl.by);
    else if (p.dtype == 1) quantize_body<1>(p, qb.loops, sl.bx, sl.by);
    else quantize_body<2>(p, qb.loops, sl.bx, sl.by);
}

// One scale per block of q_block rows of a (b, h) slice (Sec. 3.3; per token at q_block = 1).  A
// group is small, so one team (16 lanes up to 256 elements, a wave up to 4096, else the workgroup) takes it
// whole: max|X| over the group, then the same arithmetic as above.
template <int DTYPE, int NTHR>
__global__ __launch_bounds__(QNT) void quantize_rows_kernel(const QuantParams p)
{
    constexpr int ES = DTYPE == 0 ? 4 : 2;
    __shared__ float wmax[QNT / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = tid % NTHR; // NTHR == QNT: the workgroup is the team; 64: a wave; 16: a quarter of a wave
    const int nblk = (p.L + p.q_block - 1) / p.q_block;
    const int64_t gi = (int64_t)blockIdx.x * (QNT / NTHR) + tid / NTHR;
    if (gi >= (int64_t)p.B * p.H * nblk) return; // a whole team (of a wave or less: no barrier below)
    const int blk = (int)(gi % nblk), bh = (int)(gi / nblk), b = bh / p.H, h = bh % p.H;
    const int r0 = blk * p.q_block, r1 = min(p.L, r0 + p.q_block);
    const int ipr = p.d / 8, items = (r1 - r0) * ipr;
    const uint8_t *src = (const uint8_t *)p.src + (int64_t)b * p.ss[0] + (int64_t)h * p.ss[1] + (int64_t)r0 * p.ss[2];
    int8_t *dst = p.dst + (int64_t)b * p.ds[0] + (int64_t)h * p.ds[1] + (int64_t)r0 * p.ds[2];
    auto offsets = [&](int it, int64_t &so, int64_t &dofs) __attribute__((always_inline)) {
        item_offsets<ES>(p, (uint32_t)it, (uint32_t)ipr, so, dofs);
    };
    float m = 0.0f;
    auto take = [&](const Raw8<DTYPE> &r) __attribute__((always_inline)) {
        float x[8];
        widen8<DTYPE>(r, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(x[i]));
    };
    auto load = [&](int it) __attribute__((always_inline)) {
        int64_t so, dofs;
        offsets(it, so, dofs);
        return load_raw8<DTYPE>(src + so);
    };
    float s = 0.0f, rs = 0.0f;
    auto scale = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int o = NTHR < 64 ? NTHR / 2 : 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        if (NTHR == QNT) {
            if (lane == 0) wmax[wave] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < QNT / 64; ++w) m = fmaxf(m, wmax[w]);
        }
        s = fmaxf(m, 1e-12f) / 127.0f; // one IEEE fp32 division
        rs = 1.0f / s;                 // and its reciprocal, for quantize8
        if (t == 0) p.scales[gi] = s;
    };
    auto put = [&](int it, const Raw8<DTYPE> &r) __attribute__((always_inline)) {
        float x[8];
        widen8<DTYPE>(r, x);
        uint32_t w[2];
        quantize8(x, s, rs, w);
        int64_t so, dofs;
        offsets(it, so, dofs);
        *(uint2 *)(dst + dofs) = make_uint2(w[0], w[1]);
    };
    // Groups of up to RHOLD items a thread are read once, all of them in flight, and held as they are; larger ones are read
    // again, from the caches.  (With one load in flight and two reads: 32 x 1024 rows of 128 in blocks of 128 rows 9.6 us, now
    // 7.0; with a test before each load 8.1.)
    auto hold = [&](auto count) __attribute__((always_inline)) {
        constexpr int N = decltype(count)::value;
        Raw8<DTYPE> raw[N];
#pragma unroll
        for (int j = 0; j < N; ++j) raw[j] = load(min(t + j * NTHR, items - 1)); // past the end: the last item once more
#pragma unroll
        for (int j = 0; j < N; ++j) take(raw[j]);
        scale();
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (t + j * NTHR < items) put(t + j * NTHR, raw[j]);
    };
    if (items <= NTHR) hold(std::integral_constant<int, 1>{});
    else if (items <= 2 * NTHR) hold(std::integral_constant<int, 2>{});
    else if (items <= 4 * NTHR) hold(std::integral_constant<int, 4>{});
    else if (items <= RHOLD * NTHR) hold(std::integral_constant<int, RHOLD>{});
    else {
#pragma unroll 4
        for (int it = t; it < items; it += NTHR) take(load(it));
        scale();
        for (int it = t; it < items; it += NTHR) put(it, load(it));
    }
}

template <int DTYPE>
int launch_rows(const QuantParams &p, hipStream_t st)
{
    const int64_t groups = (int64_t)p.B * p.H * ((p.L + p.q_block - 1) / p.q_block);
    if ((int64_t)p.q_block * p.d <= 256) // one or two items a thread; per token most of a wave would idle (2048 tokens, 32 heads, d 128: 39 -> 11.5 us)
        hipLaunchKernelGGL((quantize_rows_kernel<DTYPE, 16>), dim3((unsigned)((groups + 15) / 16)), dim3(QNT), 0, st, p);
    else if ((int64_t)p.q_block * p.d <= 4096)
        hipLaunchKernelGGL((quantize_rows_kernel<DTYPE, 64>), dim3((unsigned)((groups + 3) / 4)), dim3(QNT), 0, st, p);
    else
        hipLaunchKernelGGL((quantize_rows_kernel<DTYPE, QNT>), dim3((unsigned)groups), dim3(QNT), 0, st, p);
    return (int)hipGetLastError();
}

} // namespace

// Partial maxima per (b, h) slice: about 1024 workgroups in all (four per compute unit, each with 64
// KiB of loads in flight), never more than the slice has work for.
int quantize_partials_per_slice(int B, int H, int L, int d)
{
    const int64_t items = (int64_t)L * (d / 8);
    const int64_t blocks = (items + QNT * QITEMS - 1) / (QNT * QITEMS);
    const int64_t want = (1024 + (int64_t)B * H - 1) / ((int64_t)B * H);
    return (int)(blocks < want ? blocks : want);
}

// n tensors (1..4), each with per_head 0 or 1 and its own partial buffer, in two launches; or one tensor with
// per_head 2 (a scale per block of rows) in one.
int launch_quantize(const QuantParams *ps, int n, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (n < 1 || n > 4) return (int)hipErrorInvalidValue;
    if (ps[0].per_head == 2) {
        if (n != 1) return (int)hipErrorInvalidValue;
        if (ps[0].dtype == 0) return launch_rows<0>(ps[0], st);
        if (ps[0].dtype == 1) return launch_rows<1>(ps[0], st);
        if (ps[0].dtype == 2) return launch_rows<2>(ps[0], st);
        return (int)hipErrorInvalidValue;
    }
    QuantBatch qb;
    memset(&qb, 0, sizeof(qb));
    qb.n = n;
    // Rounds of the second pass: as many as leave QWGS workgroups.
    int64_t rounds = 0;
    for (int i = 0; i < n; ++i)
        rounds += (int64_t)ps[i].B * ps[i].H * (((int64_t)ps[i].L * (ps[i].d / 8) + QNT * QITEMS - 1) / (QNT * QITEMS));
    qb.loops = (int)(rounds / QWGS < 1 ? 1 : (rounds / QWGS > QLOOP_MAX ? QLOOP_MAX : rounds / QWGS));
    uint64_t tot_a = 0, tot_q = 0;
    uint32_t first_a[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < n; ++i) {
        const QuantParams &p = ps[i];
        if (p.per_head == 2 || p.dtype < 0 || p.dtype > 2) return (int)hipErrorInvalidValue;
        qb.t[i] = p;
        const int64_t items = (int64_t)p.L * (p.d / 8);
        const int64_t per_wg = (int64_t)QNT * QITEMS * qb.loops;
        qb.gx[i] = (uint32_t)((items + per_wg - 1) / per_wg);
        first_a[i] = (uint32_t)tot_a;
        qb.first[i] = (uint32_t)tot_q;
        tot_a += (uint64_t)p.n_partial * (uint64_t)(p.B * p.H);
        tot_q += (uint64_t)qb.gx[i] * (uint64_t)(p.B * p.H);
        if (tot_a > 0x7fffffffull || tot_q > 0x7fffffffull) return (int)hipErrorInvalidValue;
    }
    for (int i = n; i <= 4; ++i) first_a[i] = (uint32_t)tot_a, qb.first[i] = (uint32_t)tot_q;
    QuantBatch qa = qb; // the reduction pass: each workgroup walks its part of a slice
    for (int i = 0; i <= 4; ++i) qa.first[i] = first_a[i];
    hipLaunchKernelGGL(absmax_kernel, dim3((unsigned)tot_a), dim3(QNT), 0, st, qa);
    hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)tot_q), dim3(QNT), 0, st, qb);
    return (int)hipGetLastError();
}

} // namespace intattn
