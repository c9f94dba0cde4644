// Per-head kernel parameters from scales that live in DEVICE memory (as the dynamic quantizer
// leaves them), so that quantizer and attention follow each other on a stream without the host
// reading anything back:
//   c_int = round(c * sqrt(d) / (s_Q s_K))                    (Sec. 3.1, Eq. clipping_thr)
//   (M, sh) with M * 2^-sh ~ s_V / (255 s_O), M in [2^30, 2^31)   (output requantization)
//   the factor of the fma map idx = round(x * top / c_int) (ScoreIndex; Sec. 3.1, index map), or, for a head without one, that of
//   the fp64 map.
// The arithmetic is the host's, operation for operation, in IEEE double: products, quotients,
// floor, frexp and the fma are exactly rounded on the GPU as on the CPU, and sqrt(d) comes from the
// host.  One wave per query head, one check point of the index map per lane.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace {

__device__ __forceinline__ bool good_scale(float s) { return s > 0.0f && s < __builtin_inff(); } // false for NaN

// round(x top / c_int), exact: numerator and denominator are integers below 2^38, and a quotient that is no integer lies at
// least 2^-31 from one (its rounding error is below 2^-46)
__device__ __forceinline__ uint32_t exact_index(double x, double c_int, double top)
{
    return (uint32_t)(int)((2.0 * top * x + c_int) / (2.0 * c_int));
}

// c_int (capped at 2^30: beyond 62 * 2 * 128*128*128 every index is 0 anyway) and the requantization
// multiplier of one parameter set; false (and harmless values) when a scale is unusable.
__device__ __forceinline__ bool derive_scalars(float sq, float sk, float sv, float so, double clip, double sqrt_d, HeadParams &hp)
{
    hp.pad[0] = IDX_FP64;
    hp.fma_r = 0;
    bool ok = good_scale(sq) && good_scale(sk) && good_scale(sv) && good_scale(so);
    double c = 1.0;
    if (ok) {
        const double alpha = ((double)sq * (double)sk) / sqrt_d;
        c = __builtin_floor(clip / alpha + 0.5);
        if (!(c >= 1.0)) c = 1.0;
        if (c > 1073741824.0) c = 1073741824.0;
    }
    hp.c_int = (int32_t)c;
    // unusable scales: multiplier 0, i.e. the head's output is all zeros (and its status word is set)
    hp.rq_mult = 0;
    hp.rq_shift = 31;
    if (ok) {
        const double r = (double)sv / (255.0 * (double)so);
        int e = 0;
        const double m = __builtin_frexp(r, &e);
        long long M = __builtin_llround(m * 2147483648.0);
        if (M == 2147483648LL) {
            M = 1073741824LL;
            e += 1;
        }
        const int sh = 31 - e;
        if (!(r > 0.0) || sh < 1 || sh > 62) ok = false;
        else {
            hp.rq_mult = (int32_t)M;
            hp.rq_shift = sh;
        }
    }
    return ok;
}

// the fp64 index map's factor for c_int: the bits of -(the double after top / c_int), low word in
// idx_mul, high word in idx_add
__device__ __forceinline__ uint64_t set_fp64_factor(HeadParams &hp, uint32_t top)
{
    const uint64_t bits = (uint64_t)__double_as_longlong((double)top / (double)(uint32_t)hp.c_int) + 1ull;
    const uint64_t neg = bits ^ 0x8000000000000000ull;
    hp.idx_mul = (uint32_t)neg;
    hp.idx_add = (uint32_t)(neg >> 32);
    hp.idx_shift = 0;
    return bits;
}

// One wave per query head.  Every map in question is a monotone step function, so agreement at x = 0, x = c_int and on
// both sides of each of the (at most 63) steps of the exact map is agreement on all of [0, c_int].  Lane l checks the step to
// index l + 1 for the host's candidates one after another (the first serves 99 % of thresholds) with the arithmetic of the
// kernels.  Bound by the latency of one wave: a chain of double-precision divisions.
__device__ __forceinline__ bool derive_head(const DeriveParams &dp, int h, int lane, HeadParams &hp)
{
    const int si = dp.per_head ? h : 0;
    const int kv = dp.per_head ? h / dp.group : 0;
    const float sq = dp.scale_q[si], sk = dp.scale_k[kv], sv = dp.scale_v[kv];
    const float so = dp.scale_out ? dp.scale_out[si] : sv;
    const bool ok = derive_scalars(sq, sk, sv, so, dp.clip, dp.sqrt_d, hp);

    // t_k = ceil((2 k - 1) c_int / (2 top)), the first x whose index is at least k: a quotient that is no integer lies at
    // least 1 / 126 from one, its rounding error is below 2^-22.  Lanes past the last step hold c_int, whose index is top.
    const uint32_t c_int = (uint32_t)hp.c_int, top = (uint32_t)dp.top;
    const double cd = (double)c_int, topd = (double)top;
    const bool step = (uint32_t)lane < top;
    const int t = step ? (int)__builtin_ceil((2.0 * lane + 1.0) * cd / (2.0 * topd)) : (int)c_int;
    const int at[2] = {t, step ? t - 1 : t}; // (t_1 >= 1, and t_1 - 1 stands for 0)
    uint32_t want[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) want[q] = exact_index((double)at[q], cd, topd);

    if (c_int < (1u << 22)) { // wave-uniform; also for unusable scales, whose c_int is 1
        const uint32_t quotient = __float_as_uint((float)(topd / cd));
#pragma unroll 1
        for (int u = 0; u < 6 && hp.fma_r == 0; ++u) {
            hp.fma_r = quotient - (uint32_t)(u == 0 ? 1 : u == 1 ? 2 : u == 2 ? 0 : u == 3 ? 3 : u == 4 ? 4 : -1);
            ScoreIndex<IDX_FMA> si;
            si.init(hp, 0, top);
            bool match = true;
#pragma unroll
            for (int q = 0; q < 2; ++q) match = match && si.index(si.start() - at[q]) == top - want[q];
            if (!__all(match)) hp.fma_r = 0;
        }
    }
    if (hp.fma_r != 0) hp.pad[0] = IDX_FMA;
    else set_fp64_factor(hp, top);
    return ok;
}

__device__ __forceinline__ void put_head(const DeriveParams &dp, int h, const HeadParams &hp, bool ok)
{
    dp.hp_table[h] = hp;
    dp.status[h] = ok ? 0 : 1;
}

__global__ __launch_bounds__(64) void derive_kernel(const DeriveParams dp)
{
    HeadParams hp;
    const bool ok = derive_head(dp, blockIdx.x, threadIdx.x, hp);
    if (threadIdx.x == 0) put_head(dp, blockIdx.x, hp, ok);
}

// Per-tensor scales: one wave derives the one parameter set and writes it for every head.
__global__ __launch_bounds__(64) void derive_one_kernel(const DeriveParams dp)
{
    HeadParams hp;
    const bool ok = derive_head(dp, 0, threadIdx.x, hp);
    for (int h = threadIdx.x; h < dp.Hq; h += 64) put_head(dp, h, hp, ok);
}

// Parameters per block of q_block query rows (finer quantization groups over the query rows,
// Sec. 3.3): one thread per (batch, head, block); scale_q / scale_out hold one value per block,
// scale_k / scale_v one per KV head.  Every block takes the fp64 index map, which is exact for
// every c_int without a search.
__global__ __launch_bounds__(256) void derive_rows_kernel(const DeriveParams dp)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= dp.n_entries) return;
    const int hq = (int)((e / dp.n_rowblk) % dp.Hq), kv = hq / dp.group;
    // with groups over the key axis too (n_kentries > 0) the key scales are checked by a kernel of their own
    // and c_int is formed per logit in the forward kernel: only the requantization is taken from here
    const float sq = dp.scale_q[e], sk = dp.n_kentries > 0 ? 1.0f : dp.scale_k[kv], sv = dp.scale_v[kv];
    const float so = dp.scale_out ? dp.scale_out[e] : sv;
    HeadParams hp;
    const bool ok = derive_scalars(sq, sk, sv, so, dp.clip, dp.sqrt_d, hp);
    set_fp64_factor(hp, (uint32_t)dp.top);
    dp.row_table[e] = hp;
    if (!ok) dp.status[hq] = 1; // every writer stores the same value
}

// Scales per block of keys, [B * Hkv][n_kblk]: an unusable one marks every query head of its KV head.
__global__ __launch_bounds__(256) void check_key_scales_kernel(const DeriveParams dp)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= dp.n_kentries) return;
    if (good_scale(dp.scale_k[e])) return;
    const int kv = (int)((e / dp.n_kblk) % dp.Hkv);
    for (int g = 0; g < dp.group; ++g) dp.status[kv * dp.group + g] = 1; // every writer stores the same value
}

__global__ __launch_bounds__(256) void zero_status_kernel(int32_t *status, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) status[i] = 0;
}

} // namespace

int launch_derive_rows(const DeriveParams &dp, void *stream)
{
    hipLaunchKernelGGL(zero_status_kernel, dim3((unsigned)((dp.Hq + 255) / 256)), dim3(256), 0, (hipStream_t)stream, dp.status, dp.Hq);
    hipLaunchKernelGGL(derive_rows_kernel, dim3((unsigned)((dp.n_entries + 255) / 256)), dim3(256), 0, (hipStream_t)stream, dp);
    return (int)hipGetLastError();
}

int launch_derive_groups(const DeriveParams &dp, void *stream)
{
    const int e = launch_derive_rows(dp, stream);
    if (e != 0) return e;
    hipLaunchKernelGGL(check_key_scales_kernel, dim3((unsigned)((dp.n_kentries + 255) / 256)), dim3(256), 0, (hipStream_t)stream, dp);
    return (int)hipGetLastError();
}

// One launch: a wave for all heads, or a workgroup of one wave for each.
int launch_derive(const DeriveParams &dp, void *stream)
{
    if (!dp.per_head) hipLaunchKernelGGL(derive_one_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, dp);
    else hipLaunchKernelGGL(derive_kernel, dim3((unsigned)dp.Hq), dim3(64), 0, (hipStream_t)stream, dp);
    return (int)hipGetLastError();
}

} // namespace intattn
