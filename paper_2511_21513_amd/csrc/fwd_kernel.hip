// Host side of the forward launches: the kernel variants, the small kernels ahead of and behind split
// keys, and the order of the launches of one forward.  The forward kernel template itself is in
// fwd_kernel_impl.h and is instantiated in fwd_single.hip (all three sweeps in one launch) and
// fwd_split.hip (sweeps A+B, and sweep C, as launches of their own).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace fwdk {
// instantiated explicitly in fwd_single.hip / fwd_split.hip
template <int RB, int KT, int PH>
int launch_shape(const FwdParams &p, int d, int idx_mode, hipStream_t st);
} // namespace fwdk
using fwdk::launch_shape;

namespace sweepc {
template <int D, bool SPLIT>
int launch(const FwdParams &p, int idx_mode, hipStream_t st); // instantiated explicitly in sweep_c_*.hip
} // namespace sweepc

static int launch_sweep_c(const FwdParams &p, int d, int idx_mode, hipStream_t st)
{
    if (d == 64) return p.split_c > 0 ? sweepc::launch<64, true>(p, idx_mode, st) : sweepc::launch<64, false>(p, idx_mode, st);
    if (d == 128) return p.split_c > 0 ? sweepc::launch<128, true>(p, idx_mode, st) : sweepc::launch<128, false>(p, idx_mode, st);
    return (int)hipErrorInvalidValue;
}

namespace {

// Key-split path: the row maxima and row sums that the launches of sweeps A and B accumulate into, at their neutral values.
__global__ __launch_bounds__(256) void neutral_rows_kernel(const FwdParams p, int64_t rows)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= rows) return;
    p.ws_row_max[i] = INT32_MIN;
    p.ws_row_sum[i] = 0;
}

// Key-split path: adds up the partial accumulators of sweep C's ranges and requantizes; a thread takes four channels of a
// row.  Bound by the partials it reads (16 bytes a load).
template <int D>
__global__ __launch_bounds__(256) void finish_split_kernel(const FwdParams p)
{
    const int64_t n4 = (int64_t)p.B * p.Hq * p.L * (D / 4), i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const int64_t r = i / (D / 4); // (b * Hq + hq) * L + row
    const int c4 = (int)(i % (D / 4)), l = (int)(r % p.L), bh = (int)(r / p.L), hq = bh % p.Hq, b = bh / p.Hq;
    v4i acc = {0, 0, 0, 0};
#pragma unroll 4
    for (int s = 0; s < p.split_c; ++s) acc += *(const v4i *)(p.ws_part + 4 * (s * n4 + i));
    HeadParams hp = p.hp_table ? p.hp_table[hq] : p.hp0;
    if (p.row_table) hp = p.row_table[(int64_t)bh * p.n_rowblk + l / p.q_block];
    uint32_t packed = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (p.dbg_acc) p.dbg_acc[4 * i + k] = acc[k];
        packed |= ((uint32_t)requant_any(acc[k], hp.rq_mult, hp.rq_shift) & 0xffu) << (8 * k);
    }
    *(uint32_t *)(p.out + (int64_t)b * p.os[0] + (int64_t)hq * p.os[1] + (int64_t)l * p.os[2] + 4 * c4) = packed;
}

int launch_finish_split(const FwdParams &p, int d, hipStream_t st)
{
    const int64_t n4 = (int64_t)p.B * p.Hq * p.L * (d / 4);
    const dim3 grid((unsigned)((n4 + 255) / 256)), block(256);
    if (d == 64) hipLaunchKernelGGL(finish_split_kernel<64>, grid, block, 0, st, p);
    else if (d == 128) hipLaunchKernelGGL(finish_split_kernel<128>, grid, block, 0, st, p);
    else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

int launch_neutral_rows(const FwdParams &p, hipStream_t st)
{
    const int64_t rows = (int64_t)p.B * p.Hq * p.L;
    hipLaunchKernelGGL(neutral_rows_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st, p, rows);
    return (int)hipGetLastError();
}

} // namespace

// Kernel variants (0 = automatic choice; the others are tuning knobs, all bit-identical):
//   1  one launch, 32 query rows per wave, 64-key tiles     2  one launch, 64 rows per wave
//   3  one launch, a workgroup per 32 query rows with the keys split over its four waves (fwd_splitk.hip)
//   4  two launches: sweeps A+B (32 or 64 rows per wave), then sweep C (32 rows per wave), phase-ordered kernels
//   5  as 4 with sweep C's kernel of its own
//   9, 10  the split-key kernels of decode_kernel.hip (one launch / four launches) whenever the shape allows them, else as 0
// Automatic choice among the tiled kernels (square problems are looked at again by fwd_refine_square), by measurement on shapes from 8 x 12 x 197 to 2 x 32 x 4096 (W = workgroups
// of 128 query rows): W >= 1024 fills the chip with the two-launch path (variant 5), short rows excepted; up to 256 the 128-row kernels
// leave most SIMDs with one long-running wave and the split-key single launch (variant 3) is 1.1 to 2.3 times faster;
// in between variant 3 still wins at d = 64 on long rows, otherwise variant 1 (at d = 128 the four waves of variant 3
// each stream their own K fragments from L2, which costs more than the better fill gains).
int fwd_choose_variant(int variant, int B, int Hq, int L, int Lk, int d, int causal)
{
    if (variant != 0 && variant != 9 && variant != 10) return variant;
    const int nt = (L + 127) / 128;
    const int64_t workgroups = (int64_t)B * Hq * nt;
    // Short key runs (at most three key tiles per query tile on average: up to Lk = 384, or L = Lk = 640 under the
    // causal mask): one launch, which stages K once, beats two (c2 at batch 512: 0.29 against 0.37 ms).
    const int kt2 = causal ? 2 * ((Lk - L + 127) / 128) + nt + 1 : 2 * ((Lk + 127) / 128); // twice the average
    if (workgroups >= 1024) return kt2 <= 6 ? 1 : 5;
    if (workgroups <= 256) return 3;
    return (d == 64 && L >= 1024) ? 3 : 1;
}
// Square problems that neither split their keys nor hold all scores in registers: a second look at variants 1 and 3 around the
// points where one of them starts a further round of workgroups (W = workgroups of 128 rows).  Rectangular ones, whose tiles
// are as long as their keys and not as their rows, keep the choice above.  us, this choice against the one above:
//   d 128: variant 3 holds 512 workgroups of 32 rows at a time and every one is as long without a mask: 1 past that (192 x 197:
//     96 heads 16.2 against 20.0; 1024, 32 heads 38 against 58; at 504 workgroups, 384, 42 heads, 19.3 against 16.0 for 3).
//     Variant 1 holds 512 workgroups: past that 5 with its finer launches (1024 masked, 120 heads 59.9 against 68.7; 197, 330
//     heads 24.0 against 33.2; 4096 without a mask, 17 heads 211 against 259), but not under the mask beyond 2048 keys (4096, 24
//     heads: 161 against 135), nor without one below 768 keys past 768 (384, 310 heads: 49 against 44; 250 heads: 37.7 against 40.0).  Under the mask 5 is
//     ahead for 1025 to 2048 keys already from 257 (2048, 20 heads: 65.8 against 72.4; 1024, 60 heads: 42 both), and for short
//     rows past 1023 too (640, 300 heads: 71 against 86).
//   d 64: variant 3 where the chip is full of it loses to 5, past 640 under the mask (1024, 116 heads: 32.4 against 39.1; 4096, 19
//     heads, W 608: 93.5 against 86.5 for 3) and past 400 without (2048, 28 heads: 60.6 against 72.3; 24 heads, W 384: 57 both).
//     Rows below 1024: 3 up to 448 under the mask (640, 64 heads: 18.1 against 23.7; W 450: 23.2 against 23.8; W 540: 25.1 against 23.9), 5 past 800
//     (640, 192 heads: 27.9 against 35.2; W 750: 25.7 against 25.9 for 1), short rows without a mask past 1023 excepted.
int fwd_refine_square(int variant, int B, int Hq, int L, int d, int causal)
{
    if (variant != 1 && variant != 3) return variant;
    const int64_t heads = (int64_t)B * Hq, w = heads * ((L + 127) / 128);
    if (d == 128) {
        if (variant == 3) return !causal && heads * ((L + 31) / 32) > 512 ? 1 : 3;
        if (causal) return L <= 2048 && w > (L > 1024 ? 256 : 512) ? 5 : 1;
        return w > 512 && w < 1024 && (L >= 768 || w <= 768) ? 5 : 1;
    }
    if (variant == 3) return w > (causal ? 640 : 400) ? 5 : 3;
    if (causal && w <= 448) return 3;
    return w > 800 && (causal || w < 1024) ? 5 : 1;
}
bool fwd_variant_known(int variant) { return variant == 0 || (variant >= 1 && variant <= 5) || variant == 9 || variant == 10; }

// Workgroups per query tile for the key-split path, and whether it pays at all: a model of its time against one of the
// variant (1 or 3) that serves the shape otherwise, in microseconds.  A kernel takes its key tiles times a cost per tile
// times the rounds of 256 compute units, with two rounds as the least (a unit with a single workgroup is bound by latency);
// sweep C also writes and reads the partial accumulators of each range; 24 us for five launches.  The single launches are
// bound by their longest chain of tiles or, once the chip is full, by a cost per 32 x 32 block (variant 3) or by rounds of
// 380 workgroups (variant 1).  It is made to rank the two and errs where a launch is a little over a whole number of rounds
// (509 x 7001, 32 / 8 heads, d 128: 544 workgroups of variant 3, two rounds of 512; it says 161 us, measured 238), for the
// single launch then, as the margins below do.  KV heads do not enter: 32 / 32 and 32 / 8 heads
// measure within 6 % of each other (one pair of 25: 11 %).  Timed on 286 shapes of 1 to 128 heads, 40
// to 8192 rows and 600 to 16384 keys before the fma map: the 105 that it splits took 0.23 to 0.94 of the time of the better of
// variants 1 and 3.  With the fma map, which made all sides faster: 509 x 7001 219 -> 111 us; 128 x 12000, 8 heads, d 64, 103 -> 37;
// 3000 square, 12 heads, d 128, 93 -> 79.  What else a split would serve was not timed.  Small problems lose by it (1024 square, 16 heads,
// d 128: 21 us unsplit, 49 split before the fma map).
KeySplit fwd_key_split(int variant, int B, int Hq, int L, int Lk, int d, int causal)
{
    const int row_lo = causal ? Lk - L : 0, tiles = (Lk + 127) / 128;
    const int64_t rows = (int64_t)B * Hq * L, fixed = 2 * rows; // row maxima and sums
    const int64_t w_ab = (int64_t)B * Hq * fwd_row_tiles(row_lo, L, 256), w_c = (int64_t)B * Hq * fwd_row_tiles(row_lo, L, 128);
    const double seen = causal ? (Lk - 0.5 * L) / Lk : 1.0; // share of the keys that an average row sees
    const double us_tile = d == 128 ? 1.4 : 0.9, us_part = (double)B * Hq * L * d * 8 / 4.0e6;
    double other;
    if (variant == 3) {
        const double blocks = (double)B * Hq * ((L + 31) / 32) * (Lk * seen) / 32;
        other = 8 + std::max(tiles * (d == 128 ? 1.75 : 1.15), blocks * (d == 128 ? 1.42e-3 : 0.58e-3));
    } else {
        other = 12 + tiles * (d == 128 ? 3.8 : 3.3) * std::max(1.0, (double)B * Hq * ((L + 127) / 128) * seen / 380);
    }
    const double worth = (d == 128 ? 0.93 : 0.8) * other;
    if (24 > worth) return KeySplit{0, 0}; // the launches alone take longer
    auto rounds = [&](int64_t w, int s) { return std::max((double)((w * s + 255) / 256) * seen, 2.0) / s * tiles; };
    KeySplit ks = {1, 1};
    double t_ab = 1e30, t_c = 1e30;
    for (int s = 1; s <= 32 && (s == 1 || 2 * s <= tiles); ++s) {
        const double ab = rounds(w_ab, s) * 2 * us_tile + 0.1 * s, c = rounds(w_c, s) * us_tile + us_part * s;
        if (ab < t_ab) t_ab = ab, ks.ab = s;
        if (s <= KEY_SPLIT_MAX_RANGES && s * rows * d + fixed <= KEY_SPLIT_MAX_WORDS && c < t_c) t_c = c, ks.c = s;
    }
    if (24 + t_ab + t_c > worth) return KeySplit{0, 0};
    return ks;
}
// Blocks of 32 query rows of a wave of sweeps A+B.  Two share every K fragment, which saves LDS reads, and a tile is staged
// for 256 rows; one leaves four waves a SIMD instead of three and half the masked work on the diagonal.  d = 64, where a
// fragment is half as long: always one (4 x 4096, causal, 16 heads: 95 against 100 us; 8 x 1024: 30.5 against 38.4; 1 x 8192 the
// same).  d = 128: one up to 2048 keys under the mask (8 x 1024, 32 heads: 47 against 55; 2 x 2048: 45 against 58; 8 x 2048: 160
// against 163), two beyond (2 x 4096: 144 against 145; 1 x 8192: 265 against 276; 16 x 4096: 1020 against 1074) and without a
// mask (1 x 4096: 138 against 142; 4 x 1024 the same).
static int fwd_ab_row_blocks(int d, int causal, int Lk) { return d == 64 || (causal && Lk <= 2048) ? 1 : 2; }

// All scores in registers (fwd_short.hip): up to 256 keys at d = 64, from 128 heads on.  Against variant 3, whose chain is a
// quarter as long, only where more blocks of 32 rows than three for each compute unit are in flight, or, as its waves pad the
// masked half, one under a square mask: 160 heads of 160 x 160 10.2 us against 10.4, 128 of 197 x 197 10.5 against 11.2, masked
// 128 of 96 x 96 8.5 against 8.8, but 128 heads of 96 x 96 8.0 against 7.1 and of 64 x 200, masked, 11.1 against 10.0.  Against
// the 128-row kernels always: 384 heads of 32 x 32 7.2 us against 10.9, 1536 of 197 x 197 48.5 against 74.
bool fwd_short_serves(int variant, int B, int Hq, int L, int Lk, int d, int causal)
{
    if (d != 64 || Lk > 256 || (int64_t)B * Hq < 128) return false;
    return variant != 3 || (int64_t)B * Hq * ((L + 31) / 32) > (causal && L == Lk ? 256 : 768);
}

int fwd_rows_per_block(int variant) { return variant == 2 ? 256 : (variant == 3 ? 32 : 128); }

int launch_fwd(const FwdParams &p_in, int d, int idx_mode, int variant, int stage, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    FwdParams p = p_in;
    const int64_t k_bytes = (int64_t)p.Lk * d; // K of one (batch, KV head) group; V is as large
    p.group_batch = fwd_group_batch(p.B, p.Hkv, 2 * k_bytes); // kernels that stream K and V
    const bool two_launches = variant == 4 || variant == 5;
    if (variant == VARIANT_SHORT) return stage != 0 ? (int)hipErrorNotSupported : launch_fwd_short(p, d, idx_mode, stream);
    if (variant == VARIANT_KEY_SPLIT) {
        if (stage != 0) return (int)hipErrorNotSupported;
        int e = launch_neutral_rows(p, st);
        FwdParams pab = p;
        pab.n_qtiles = fwd_row_tiles(p.row_lo, p.L, 256);
        pab.group_batch = fwd_group_batch(p.B, p.Hkv, k_bytes); // streams K only
        if (e == 0) e = launch_shape<2, 2, 3>(pab, d, idx_mode, st);
        if (e == 0) e = launch_shape<2, 2, 4>(pab, d, idx_mode, st);
        if (e == 0) e = launch_sweep_c(p, d, idx_mode, st);
        return e == 0 ? launch_finish_split(p, d, st) : e;
    }
    if (stage != 0 && !two_launches) return (int)hipErrorNotSupported;
    if (variant == 3) return launch_fwd_splitk(p, d, idx_mode, stream);
    if (variant == 2) return launch_shape<2, 2, 0>(p, d, idx_mode, st);
    if (two_launches) {
        // sweeps A+B leave row max and row sum in the workspace for sweep C
        if (stage != 2) {
            FwdParams pab = p;
            pab.group_batch = fwd_group_batch(p.B, p.Hkv, k_bytes); // streams K only
            const int rb = fwd_ab_row_blocks(d, p.causal, p.Lk);
            pab.n_qtiles = fwd_row_tiles(p.row_lo, p.L, 128 * rb);
            const int e = rb == 1 ? launch_shape<1, 2, 1>(pab, d, idx_mode, st) : launch_shape<2, 2, 1>(pab, d, idx_mode, st);
            if (e != 0 || stage == 1) return e;
        }
        if (variant == 4) return launch_shape<1, 2, 2>(p, d, idx_mode, st);
        return launch_sweep_c(p, d, idx_mode, st);
    }
    return launch_shape<1, 2, 0>(p, d, idx_mode, st);
}

} // namespace intattn
