// IndexSoftmax as an operator of its own (Sec. 3.1-3.2) on INT32 logits [rows, cols] in device
// memory, UINT8 probabilities out: per row  max -> clip at c_int -> index map -> LUT_hat -> integer
// sum -> P = round(255 E / S).  Bound by HBM: 4 bytes in, 1 byte out per element when the row is
// read once.  A row is handled by a team of 64 lanes (cols <= 2048, four rows per workgroup) or 256
// threads; it stays in registers between the three steps when it fits (cols <= 16384), otherwise
// it is streamed three times (the later passes mostly hit the caches).  The 32 table values and
// the 33 probabilities a row can take live in lanes and are fetched with a lane permute.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace {

__device__ __forceinline__ int32_t wave_max(int32_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o));
    return v;
}
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4))); // 16 bytes at the alignment of a logit

__device__ __forceinline__ bool in_row(int c, int end) { return (uint32_t)c < (uint32_t)end; }

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// NTHR threads per row (64: a wave, no barriers; 256: the workgroup).  NCH > 0: the row is held in
// NCH groups of four logits per thread; NCH == 0: streamed.  MODE: IDX_TOP24 (the index is the top
// byte of a 24-bit multiply-add; thresholds up to several thousand) or IDX_FP64 (every threshold).
// Table indices travel as idx * 4, the byte offset the lane permute takes, so that a lookup is one
// permute: LUT_hat[idx] and later P[idx] live in lane idx.
// ROWS_ANY: any row.  ROWS_WHOLE: no mask, rows of a multiple of four columns, probabilities that start on a word: a group of
// columns lies in the row as a whole or not at all, so that there is no test per column, and the loads of a row have no branch
// between them and are all in flight at once.  (As ROWS_ANY: 8192 rows of 2048 columns 17.4 us, now 14.6; of 8192 columns 62.8
// and 59.2; of 6000 columns 39.5 and 35.4.)  ROWS_SHORT: up to 256 columns, groups from column 0, words or bytes stored as
// the alignment has it; for rows where the lead costs more than it gives (see the launcher).
enum Rows { ROWS_ANY, ROWS_WHOLE, ROWS_SHORT };

// Waves a SIMD that ROWS_WHOLE of long rows is held to: fewer rows in flight stream faster (4096 rows of 16384 columns: 66.7 us
// at five, 63.4 at three; 8192 rows of 7168 columns: 44.6 at eight, 42.8 at five; ROWS_ANY is slower with the limit, 81 against
// 67 us at 8190 columns).
constexpr int max_waves(int nthr, int nch, int rows) { return rows != ROWS_WHOLE || nthr < 256 || nch < 8 ? 8 : (nch < 16 ? 5 : 3); }

template <int NTHR, int NCH, int MODE, int ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, max_waves(NTHR, NCH, ROWS)))) void index_softmax_kernel(const SoftmaxParams p)
{
    __shared__ int32_t red[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = NTHR == 64 ? lane : tid;
    const int64_t row = NTHR == 64 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    if (row >= p.rows) return; // a whole wave of the four-row layout; the 256-thread layout has no spare rows
    const int cols = p.cols;
    const int n_vis = p.causal ? (int)(row % p.rows_per_matrix) + cols - p.rows_per_matrix + 1 : cols;
    const int32_t *src = (const int32_t *)((const uint8_t *)p.logits + row * p.ls);
    uint8_t *dst = p.prob + row * p.ps;
    const HeadParams hp = p.hp;
    const uint32_t c_int = (uint32_t)hp.c_int, top4 = (uint32_t)p.top * 4u;
    const uint32_t lutv = (p.lut[lane >> 2] >> (8 * (lane & 3))) & 0xffu; // LUT_hat[lane] (0 beyond the table; up to 64 entries)
    const double negr = idx_fp64_factor(hp);
    const int mul = (int)hp.idx_mul;

    // Groups of four columns start where the row's probabilities are 4-byte aligned: column 4 g - lead, the first and the
    // last group partly outside the row.  Every store is then one aligned word whatever the strides are, and every load
    // 16 bytes at the 4-byte alignment that logits have anyway.  (Rows of 6001 columns, whose starts fall on every
    // alignment, took four loads and four byte stores a group: 8192 x 6001: 67.9 us, now 47.4, 5.2 TB/s.)
    constexpr bool whole = ROWS == ROWS_WHOLE;
    const int lead = ROWS == ROWS_ANY ? (int)((uintptr_t)dst & 3u) : 0;
    [[maybe_unused]] const bool words = ((uintptr_t)dst & 3u) == 0;
    auto load4 = [&](int c, int32_t (&x)[4]) __attribute__((always_inline)) {
        if (whole || (c >= 0 && c + 3 < n_vis)) {
            const v4i_a4 q = *(const v4i_a4 *)(src + c);
            x[0] = q[0], x[1] = q[1], x[2] = q[2], x[3] = q[3];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = in_row(c + e, n_vis) ? src[c + e] : 0;
        }
    };
    auto team_max = [&](int32_t v) __attribute__((always_inline)) {
        v = wave_max(v);
        if (NTHR == 64) return v;
        if (lane == 0) red[0][wave] = v;
        __syncthreads();
        return max(max(red[0][0], red[0][1]), max(red[0][2], red[0][3]));
    };
    auto team_sum = [&](uint32_t v) __attribute__((always_inline)) {
        v = wave_sum(v);
        if (NTHR == 64) return v;
        if (lane == 0) red[1][wave] = (int32_t)v;
        __syncthreads();
        return (uint32_t)red[1][0] + (uint32_t)red[1][1] + (uint32_t)red[1][2] + (uint32_t)red[1][3];
    };
    // 4 * table index of a visible logit -- Delta = max - A needs 33 bits; as an unsigned difference it is
    // exact, and the clip brings it to at most 2^30
    auto index4 = [&](int32_t x, int32_t m) __attribute__((always_inline)) {
        const uint32_t delta = (uint32_t)m - (uint32_t)x;
        const int tneg = -(int)(delta < c_int ? delta : c_int);
        if (MODE == IDX_TOP24) return (((uint32_t)__mul24(tneg, mul) + hp.idx_add) >> 22) & 0x3fcu;
        return (uint32_t)(int)__builtin_fma((double)tneg, negr, 0.5) << 2;
    };
    // the four indices (times 4) of the group at column c as bytes of one word; a hidden column takes the
    // last table entry, which is 0 by Eq. lut16.  Groups that are visible as a whole skip the selects.
    auto index_word = [&](const int32_t (&x)[4], int32_t m, int c) __attribute__((always_inline)) {
        uint32_t w = 0;
        if (whole || (c >= 0 && c + 3 < n_vis)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) w |= index4(x[e], m) << (8 * e);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) w |= (in_row(c + e, n_vis) ? index4(x[e], m) : top4) << (8 * e);
        }
        return w;
    };
    // lane value `v` of the lanes named by the four bytes of w (byte offsets idx * 4), summed / packed
    auto gather_sum = [&](uint32_t v, uint32_t w) __attribute__((always_inline)) {
        uint32_t acc = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += (uint32_t)__builtin_amdgcn_ds_bpermute((int)((w >> (8 * e)) & 0xffu), (int)v);
        return acc;
    };
    auto gather_pack = [&](uint32_t v, uint32_t w) __attribute__((always_inline)) {
        uint32_t packed = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) packed |= (uint32_t)__builtin_amdgcn_ds_bpermute((int)((w >> (8 * e)) & 0xffu), (int)v) << (8 * e);
        return packed;
    };
    auto store4 = [&](int c, uint32_t packed) __attribute__((always_inline)) {
        if (whole || ((ROWS == ROWS_ANY || words) && c >= 0 && c + 3 < cols)) *(uint32_t *)(dst + c) = packed;
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (in_row(c + e, cols)) dst[c + e] = (uint8_t)(packed >> (8 * e));
    };

    constexpr int NREG = NCH > 0 ? NCH : 1;
    int32_t v[NREG][4];
    int32_t m = INT32_MIN;
    // ---- row max over the visible columns
    if (NCH > 0) {
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int c = (t + NTHR * j) * 4 - lead;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[j][e] = 0;
            if (whole) load4(min(c, cols - 4), v[j]); // (a hidden group: the row's last one again)
            else if (c < n_vis) load4(c, v[j]);
        }
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int c = (t + NTHR * j) * 4 - lead;
            if (whole || (c >= 0 && c + 3 < n_vis)) {
                m = max(max(m, v[j][0]), max(v[j][1], max(v[j][2], v[j][3])));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (in_row(c + e, n_vis)) m = max(m, v[j][e]);
            }
        }
    } else {
        for (int c = t * 4 - lead; c < n_vis; c += NTHR * 4) {
            int32_t x[4];
            load4(c, x);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (in_row(c + e, n_vis)) m = max(m, x[e]);
        }
    }
    m = team_max(m);

    // ---- clip, index map, LUT_hat, row sum; the indices of a resident row are kept as bytes
    uint32_t w[NREG];
    uint32_t sum = 0;
    if (NCH > 0) {
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            // a wave past the last visible column has nothing to look up (the last table entry is 0)
            const int c = (t + NTHR * j) * 4 - lead;
            w[j] = top4 * 0x01010101u;
            if (whole || c - 4 * lane < n_vis) { // wave-uniform
                const uint32_t x = index_word(v[j], m, c);
                if (!whole || c < cols) w[j] = x;
                sum += gather_sum(lutv, w[j]);
            }
        }
    } else {
        // every lane takes part in every permute: the trip count is rounded up for the whole team
        for (int c = t * 4 - lead; c - t * 4 < n_vis; c += NTHR * 4) {
            int32_t x[4] = {0, 0, 0, 0};
            if (c < n_vis) load4(c, x);
            sum += gather_sum(lutv, index_word(x, m, c));
        }
    }
    const uint32_t S = team_sum(sum); // >= 255: the column of the row maximum is visible

    // ---- Eq. uint8-prob: lane l holds the probability of table index l (0 beyond the table)
    const uint32_t ptv = (510u * lutv + S) / (2u * S);
    if (NCH > 0) {
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const int c = (t + NTHR * j) * 4 - lead;
            uint32_t packed = 0; // hidden columns
            if (whole || c - 4 * lane < n_vis) packed = gather_pack(ptv, w[j]); // wave-uniform
            if (c < cols) store4(c, packed);
        }
    } else {
        for (int c = t * 4 - lead; c - t * 4 < cols; c += NTHR * 4) {
            int32_t x[4] = {0, 0, 0, 0};
            if (c < n_vis) load4(c, x);
            const uint32_t packed = gather_pack(ptv, index_word(x, m, c));
            if (c < cols) store4(c, packed);
        }
    }
}

template <int NTHR, int NCH, int ROWS> int launch_rows(const SoftmaxParams &p, hipStream_t st)
{
    const int64_t blocks = NTHR == 64 ? (p.rows + 3) / 4 : p.rows;
    if (p.hp.pad[0] == IDX_TOP24)
        hipLaunchKernelGGL((index_softmax_kernel<NTHR, NCH, IDX_TOP24, ROWS>), dim3((unsigned)blocks), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL((index_softmax_kernel<NTHR, NCH, IDX_FP64, ROWS>), dim3((unsigned)blocks), dim3(256), 0, st, p);
    return (int)hipGetLastError();
}

template <int NTHR, int NCH> int launch_one(const SoftmaxParams &p, bool aligned, hipStream_t st)
{
    if constexpr (NCH > 0 && (NCH & (NCH - 1)) == 0)
        if (aligned && !p.causal && p.cols % 4 == 0) return launch_rows<NTHR, NCH, ROWS_WHOLE>(p, st);
    return launch_rows<NTHR, NCH, ROWS_ANY>(p, st);
}

} // namespace

// rows <= 2^31 - 1 workgroups' worth, 1 <= cols <= 2^29; strides in bytes, logits and their stride multiples of 4; p.hp
// holds c_int and the index-map constants with the scheme in pad[0]: IDX_TOP24 or IDX_FP64.  Rows whose probabilities may
// start off a 4-byte boundary need room for up to three columns more (the lead of their first group).
int launch_index_softmax(const SoftmaxParams &p, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    const bool al = (((uintptr_t)p.prob | (uint64_t)p.ps) & 3u) == 0; // every row of probabilities starts on a word
    const int c = p.cols + (al ? 0 : 3);
    // A lead costs 0.3 us where there is none to find (20000 masked rows of 200: 8.3 us, 8.1 without) or where the rows are too
    // short for their stores to matter (20000 rows of 50: 8.1 and 7.9), and a second group per lane for a column or three where
    // it takes the row past 256 (20000 rows of 254: 10.2 and 8.4).  (Rows of 250 off a word: 8.6 us with it, 9.2 without.)
    if (p.cols <= 256 && (c > 256 || p.cols <= 128 || al) && !(al && !p.causal && p.cols % 4 == 0)) return launch_rows<64, 1, ROWS_SHORT>(p, st);
    if (p.cols <= 2048 && c > 2048) return launch_one<64, 9>(p, al, st); // api.cpp counts workgroups of four rows up to 2048 columns
    if (c <= 256) return launch_one<64, 1>(p, al, st);
    if (c <= 512) return launch_one<64, 2>(p, al, st);
    if (c <= 1024) return launch_one<64, 4>(p, al, st);
    if (c <= 2048) return launch_one<64, 8>(p, al, st);
    if (c <= 4096) return launch_one<256, 4>(p, al, st);
    if (c <= 8192) return launch_one<256, 8>(p, al, st);
    if (c <= 16384) return launch_one<256, 16>(p, al, st);
    if (p.cols <= 16384) return launch_one<256, 17>(p, al, st);
    return launch_one<256, 0>(p, al, st);
}

} // namespace intattn
