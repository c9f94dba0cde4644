// Per-head kernel parameters from scales that live in DEVICE memory (as the dynamic quantizer
// leaves them), so that quantizer and attention follow each other on a stream without the host
// reading anything back:
//   c_int = round(c * sqrt(d) / (s_Q s_K))                    (Sec. 3.1, Eq. clipping_thr)
//   (M, sh) with M * 2^-sh ~ s_V / (255 s_O), M in [2^30, 2^31)   (output requantization)
//   constants of an exact index map idx = round(x * top / c_int)  (Sec. 3.1, index map): the factor of the fma map
//   (ScoreIndex) for the tiled kernels, and, for those that do not take it, the multiply-high of 24-bit factors where it
//   exists (nearly every threshold up to 60000); else the fp64 map for all.
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
// both sides of each of the (at most 63) steps of the exact map is agreement on all of [0, c_int].  Lane l computes t_k, the
// first x whose index is at least k = l + 1; then every lane tests one candidate of each scheme against all of the steps,
// whose t_k it reads from lane k - 1.  Bound by the latency of one wave: quotients are IEEE double divisions (exact under
// floor and ceil, see below) and the loops hold 32-bit integer operations only.  (With 64-bit integer divisions and
// products, and the steps in LDS: 18.8 us for this kernel, now 8.0.)
__device__ __forceinline__ bool derive_head(const DeriveParams &dp, int h, int lane, HeadParams &hp)
{
    const int si = dp.per_head ? h : 0;
    const int kv = dp.per_head ? h / dp.group : 0;
    const float sq = dp.scale_q[si], sk = dp.scale_k[kv], sv = dp.scale_v[kv];
    const float so = dp.scale_out ? dp.scale_out[si] : sv;
    bool ok = derive_scalars(sq, sk, sv, so, dp.clip, dp.sqrt_d, hp);

    // t_k = ceil((2 k - 1) c_int / (2 top)): a quotient that is no integer lies at least 1 / 126 from one, its rounding
    // error is below 2^-22.  Lanes past the last step hold c_int.
    const uint32_t c_int = (uint32_t)hp.c_int, top = (uint32_t)dp.top;
    const double cd = (double)c_int, topd = (double)top;
    const int t = (uint32_t)lane < top ? (int)__builtin_ceil((2.0 * lane + 1.0) * cd / (2.0 * topd)) : (int)c_int;
    const int at[3] = {t, t - 1, (int)c_int}; // this lane's check points (t >= 1); t_1 - 1 or 0 is checked by lane 0
    uint32_t want[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) want[q] = exact_index((double)at[q], cd, topd);

    // the factor of the IDX_FMA map: the host's candidates with the arithmetic of the kernels
    if (ok && c_int < (1u << 22)) {
        const uint32_t quotient = __float_as_uint((float)(topd / cd));
#pragma unroll 1
        for (int u = 0; u < 6 && hp.fma_r == 0; ++u) {
            hp.fma_r = quotient - (uint32_t)(u == 0 ? 1 : u == 1 ? 2 : u == 2 ? 0 : u == 3 ? 3 : u == 4 ? 4 : -1);
            ScoreIndex<IDX_FMA> si;
            si.init(hp, 0, top);
            bool match = true;
#pragma unroll
            for (int q = 0; q < 3; ++q) match = match && si.index(si.start() - at[q]) == top - want[q];
            if (!__all(match)) hp.fma_r = 0;
        }
    }

    bool found = false;
    if (ok && hp.fma_r != 0) { // wave-uniform
        // (((x << pre) + off) * mul) >> 32 with factors below 2^23: a lane per shift and per one of the two multipliers
        // around top 2^32 / (c_int << pre).  The step to index k confines off to
        // ceil(k 2^32 / mul) - (t << pre) <= off < ceil(k 2^32 / mul) - ((t - 1) << pre); the quotients are kept as
        // quotient and remainder, one addition per step (multipliers below 512 cannot reach the first step).
        const int pre = lane >> 1;
        const bool fits = pre < 23 && ((uint64_t)c_int << pre) < (1ull << 23);
        const int span = fits ? (int)(c_int << pre) : 1;
        const double muld = __builtin_floor(topd * 4294967296.0 / (double)span) + (double)(lane & 1);
        const bool valid = fits && muld >= 512.0 && muld < 8388608.0;
        const int mul = valid ? (int)muld : 512, sh = fits ? pre : 0;
        const int q1 = (int)(4294967296.0 / (double)mul), r1 = (int)(0u - (uint32_t)q1 * (uint32_t)mul); // 2^32 = q1 mul + r1
        int lo = 0, hi = (1 << 23) - 1 - span, quo = 0, rem = 0;
        auto next_quotient = [&]() __attribute__((always_inline)) { // ceil of the next multiple of 2^32 over mul
            quo += q1;
            rem += r1;
            if (rem >= mul) rem -= mul, quo += 1;
            return quo + (rem > 0 ? 1 : 0);
        };
        for (int k = 1; k <= (int)top; ++k) {
            const int base = next_quotient() - (__builtin_amdgcn_readlane(t, k - 1) << sh);
            lo = max(lo, base);
            hi = min(hi, base - 1 + (1 << sh));
        }
        hi = min(hi, next_quotient() - 1 - span);
        const unsigned long long good = __ballot(valid && lo <= hi);
        if (good != 0ull) {
            const int src = __builtin_ctzll(good), pre_s = src >> 1;
            const int lo_s = __shfl(lo, src), hi_s = __shfl(hi, src);
            const uint32_t mul_s = (uint32_t)__shfl(mul, src), off_s = (uint32_t)(lo_s + (hi_s - lo_s) / 2);
            bool match = true; // every check point, with the arithmetic of the kernels
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if ((uint32_t)(((uint64_t)(((uint32_t)at[q] << pre_s) + off_s) * mul_s) >> 32) != want[q]) match = false;
            if (__all(match)) {
                found = true;
                hp.pad[0] = IDX_MULHI24;
                hp.idx_mul = 0u - mul_s;
                hp.idx_add = 0u - off_s;
                hp.idx_shift = pre_s;
            }
        }
    }
    if (!found) {
        // fp64 with r the double after top / c_int: exact for every c_int (the excess of r is under
        // two units in the last place and the fma rounds once, monotonically; values of
        // x*top/c_int + 1/2 that are not integers stay 1/(2 c_int) away from the next integer)
        const double r = -__longlong_as_double((long long)(set_fp64_factor(hp, top)));
        bool match = true;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if ((uint32_t)(int)__builtin_fma(-(double)at[q], r, 0.5) != want[q]) match = false;
        if (!__all(match)) ok = false;
        hp.pad[0] = IDX_FP64;
    }
    if (!ok) hp.rq_mult = 0; // (the fp64 check cannot fail; kept as the last line of defence)
    return ok;
}

// All heads of a call run one index scheme (sweep C one kernel): a launch that serves only some head indices leaves most
// of the chip idle, because the workgroups of a head index share an XCD.  If any head lacks multiply-high
// constants, every head takes the fp64 map (exact for every threshold).
__device__ __forceinline__ void unify_scheme(const DeriveParams &dp, int h)
{
    HeadParams hp = dp.hp_table[h];
    if (hp.pad[0] != IDX_FP64) {
        hp.pad[0] = IDX_FP64;
        set_fp64_factor(hp, (uint32_t)dp.top);
        dp.hp_table[h] = hp;
    }
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

__global__ __launch_bounds__(64) void unify_schemes_kernel(const DeriveParams dp)
{
    bool mixed = false;
    for (int h = threadIdx.x; h < dp.Hq; h += 64) mixed |= dp.hp_table[h].pad[0] == IDX_FP64;
    if (!__any(mixed)) return;
    for (int h = threadIdx.x; h < dp.Hq; h += 64) unify_scheme(dp, h);
}

// Per-tensor scales: one wave derives the one parameter set and writes it for every head.
__global__ __launch_bounds__(64) void derive_one_kernel(const DeriveParams dp)
{
    HeadParams hp;
    const bool ok = derive_head(dp, 0, threadIdx.x, hp);
    for (int h = threadIdx.x; h < dp.Hq; h += 64) put_head(dp, h, hp, ok);
}

// Per-head scales of few heads: one workgroup derives all of them, a wave per head, and settles the scheme.
constexpr int FEW_HEADS = 8;
__global__ __launch_bounds__(64 * FEW_HEADS) void derive_heads_kernel(const DeriveParams dp)
{
    const int lane = threadIdx.x & 63, h = threadIdx.x >> 6;
    HeadParams hp;
    const bool ok = derive_head(dp, h, lane, hp);
    if (lane == 0) put_head(dp, h, hp, ok);
    if (!__syncthreads_or(hp.pad[0] == IDX_FP64)) return;
    __syncthreads(); // (the table written above is visible)
    for (int h = threadIdx.x; h < dp.Hq; h += blockDim.x) unify_scheme(dp, h);
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

// One launch where the heads share their scales or are few (a launch is 2 to 4 us of the stream): one workgroup of a wave per
// head.  More heads take a workgroup each and a second launch for the scheme: the waves of one workgroup share a compute unit
// and its double-precision divisions (8 heads 9.2 us, 16 13.2, 32 in two rounds 23.3, against 8.0 + 1.4 for any number).
int launch_derive(const DeriveParams &dp, void *stream)
{
    if (!dp.per_head) {
        hipLaunchKernelGGL(derive_one_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, dp);
        return (int)hipGetLastError();
    }
    if (dp.Hq <= FEW_HEADS) {
        hipLaunchKernelGGL(derive_heads_kernel, dim3(1), dim3((unsigned)(64 * dp.Hq)), 0, (hipStream_t)stream, dp);
        return (int)hipGetLastError();
    }
    hipLaunchKernelGGL(derive_kernel, dim3((unsigned)dp.Hq), dim3(64), 0, (hipStream_t)stream, dp);
    hipLaunchKernelGGL(unify_schemes_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, dp);
    return (int)hipGetLastError();
}

} // namespace intattn
