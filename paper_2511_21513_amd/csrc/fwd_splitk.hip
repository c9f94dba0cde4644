// Fused IntAttention forward for mid-size problems on gfx950 (MI355X): one workgroup per block of 32
// query rows, the KEYS of that block split over the four waves of the workgroup.
//
// With 128-row tiles a problem of a few hundred workgroups leaves most SIMDs with one wave that walks
// every key of its tile three times; the longest tile sets the time.  Here every wave takes every
// fourth 32-key sub-tile of the block's keys (interleaved, so the causal triangle is shared evenly),
// so the longest chain is a quarter as long and there are four times as many workgroups.  The three
// reductions of IndexSoftmax (Sec. 3.1-3.2: row max, row sum of E_hat, P_hat.V_hat) cross the waves
// through LDS once each:
//   sweep A: S^T = K.Q^T of the wave's sub-tiles -> row max -> max over the waves
//   sweep B: S^T again -> clip, index, LUT_hat -> row sum -> sum over the waves -> per-row table
//            P_hat = round(255 E/S) (Eq. uint8-prob), built once per workgroup
//   sweep C: S^T again -> index -> table -> 16 probability bytes per lane = one MFMA B operand of
//            O^T += V^T.P^T -> accumulators added up over the waves in LDS -> requantize, store.
// A wave works alone between the reductions: K fragments come straight from global memory (a lane reads
// the 16 bytes of its key row that its MFMA operand holds; the next sub-tile is requested before this one is
// computed), V sub-tiles go through a wave-private LDS buffer (direct global -> LDS loads, then the
// transposing LDS read), and there is no workgroup barrier inside a sweep.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace {

constexpr int WAVES = 4;
constexpr int NT = WAVES * 64;

// Waves a SIMD (and workgroups a compute unit): at d = 64 three, i.e. 168 registers (143 to 150 in use).  With four, 17 spill
// inside the loops (2048 rows, 16 heads: 24.3 -> 31.8 us; 8 x 12 heads of 197 rows 8.2 -> 11.0); with four and the start values
// added by the vector ALU instead of held for the MFMAs none does, at the same speed as three.  Key groups hold yet
// more (156 at d = 64, under the mask).
constexpr int splitk_waves(int d, int mode) { return d != 64 || mode == IDX_KGROUP ? 2 : 3; }

// How key groups lie against the 32-key sub-tiles: a sub-tile may meet several blocks of keys (constants for each logit), or lies in
// one, whose constants each wave forms, or the workgroup keeps in a table.  An instantiation each: in one kernel
// that decided at run time the first took 5 % longer (24 heads of 700 under the mask, blocks of 7 keys: 92.2 us against 87.1 at d 64,
// 101.7 against 96.7 at d 128; 87.7 and 97.7 before there was a table) and the second 4 % (200 rows of 4096 keys in blocks of
// 32, 16 heads, d 64: 96.8 against 92.5).
enum KeyBlocks { STRADDLING = 0, WHOLE = 1, WHOLE_TABLE = 2 };

template <int D, bool CAUSAL, int MODE, int BLOCKS = STRADDLING>
__global__ __launch_bounds__(NT, splitk_waves(D, MODE)) void fwd_splitk_kernel(const FwdParams p)
{
    constexpr int KB = D / 32;  // 32-wide blocks of the head dimension
    constexpr int CB = D / 32;  // 32-wide blocks of output channels
    constexpr int SUB = 32 * D; // bytes of a 32-key sub-tile
    [[maybe_unused]] constexpr int NBLK = SUB / 1024; // 1 KiB blocks of a sub-tile: one wave-wide 16-byte load each
    [[maybe_unused]] constexpr int CPR = D / 16;      // 16-byte chunks per key row
    [[maybe_unused]] constexpr int RPB = 1024 / D;    // key rows per block

    // wave-private V sub-tiles, two buffers as separate arrays (the compiler tracks each direct-to-LDS load by
    // the array it targets, so reads of one buffer need not wait for loads into the other)
    __shared__ __attribute__((aligned(1024))) int8_t Vw0[WAVES][SUB];
    __shared__ __attribute__((aligned(1024))) int8_t Vw1[WAVES][SUB];
    __shared__ int32_t acc_lds[32][D + 1]; // output accumulators, summed over the waves (rows padded: one bank per row)
    __shared__ int32_t red[2][WAVES][32];                               // per-wave row max / row sum
    __shared__ double red_m[MODE == IDX_KGROUP ? WAVES : 1][32];        // per-wave maximum of the dequantized logits
    __shared__ uint32_t lut_lds[16];
    extern __shared__ __attribute__((aligned(16))) uint32_t PT[]; // [idx][row], NIDX * 32 words; then, under WHOLE_TABLE, 8 bytes [key block][row]

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 31, h = lane >> 5;
    HeadParams hp = p.hp0;
    // asked for with the rest of the work item's parameters, not with vector loads through a selected pointer, whose wait is 0.1
    // to 0.2 us of a small launch
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(hp.c_int), "+s"(hp.idx_mul), "+s"(hp.idx_add), "+s"(hp.rq_mult), "+s"(hp.rq_shift), "+s"(hp.fma_r));
#endif
    const WorkItem wi = fwd_work_item(p, (int)blockIdx.x);
    if (!wi.valid) return; // padding of the XCD-aware grid (uniform for the whole workgroup)
    const int b = wi.b, hq = wi.hq, kvh = wi.kvh, qt = wi.qt + p.row_lo / 32;
    const int bh = b * p.Hq + hq;
    if (p.hp_table) hp = p.hp_table[hq];
    // The rest with the index scheme M as a compile-time constant: MODE, or, under IDX_DEVICE, the one that the parameters
    // derived on the device allow.
    auto body = [&](auto mode_tag) __attribute__((always_inline)) {
    constexpr int M = decltype(mode_tag)::value;
    const int L = p.Lk;
    const int rlo = p.row_lo, rhi = p.row_lo + p.L, LQ = p.L;
    const uint32_t top = (uint32_t)p.top;
    const int NIDX = top < 32 ? 32 : 64;
    // Finer quantization groups (Sec. 3.3): parameters per block of query rows, from the row table; KG: each key block
    // has a scale of its own too, so that the row maximum is taken over the dequantized logits (fp64) and a lane forms the
    // constants of its row for each key block (once per 32-key sub-tile where a sub-tile lies in one block).
    constexpr bool KG = M == IDX_KGROUP;
    const float *skp = KG ? p.sk_blocks + (int64_t)(b * p.Hkv + kvh) * p.n_kblk : nullptr;
    constexpr bool kg_blocks = KG && BLOCKS != STRADDLING, kg_table = KG && BLOCKS == WHOLE_TABLE;
    auto row_hp = [&](int r) __attribute__((always_inline)) {
        const int lr = (r >= p.row_lo && r < p.row_lo + p.L) ? r - p.row_lo : 0;
        return p.row_table[(int64_t)bh * p.n_rowblk + lr / p.q_block];
    };

    const int q0 = qt * 32, row = q0 + n; // the lane's query row (numbering in which row r sees keys <= r)
    const bool row_ok = row >= rlo && row < rhi;
    const int8_t *Qp = p.q + (int64_t)b * p.qs[0] + (int64_t)hq * p.qs[1];
    const int8_t *Kp = p.k + (int64_t)b * p.ks[0] + (int64_t)kvh * p.ks[1];
    const int8_t *Vp = p.v + (int64_t)b * p.vs[0] + (int64_t)kvh * p.vs[1];

    double sq_row = 0.0, Mreal = -__builtin_inf();
    auto scale_q = [&](int r) __attribute__((always_inline)) {
        return (double)p.sq_rows[(int64_t)bh * p.n_rowblk + (r >= rlo && r < rhi ? r - rlo : 0) / p.q_block];
    };
    if constexpr (KG) sq_row = scale_q(row);
    // alpha^(g) of the logit (lane's row, key); keys past the end take the last block's scale
    auto kg_alpha = [&](int key) __attribute__((always_inline)) {
        return (sq_row * (double)skp[min(key, L - 1) / p.k_block]) / p.sqrt_d;
    };

    // LUT_hat by place (see ScoreIndex)
    if (tid < 64) {
        const int idx = ScoreIndex<M>::place(tid, (int)top);
        ((uint8_t *)lut_lds)[tid] = idx >= 0 ? (uint8_t)(p.lut[idx / 4] >> (8 * (idx % 4))) : (uint8_t)0;
    }
    for (int i = tid; i < 32 * (D + 1); i += NT) (&acc_lds[0][0])[i] = 0;

    // Q fragments: row q0 + n, bytes [32 kb + 16 h, +16)
    v4i qf[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        qf[kb] = v4i{0, 0, 0, 0};
        if (row_ok) qf[kb] = *(const v4i *)(Qp + (int64_t)(row - rlo) * p.qs[2] + kb * 32 + h * 16);
    }

    const int kmax = CAUSAL ? min(L, q0 + 32) : L; // keys any row of the block sees
    const int nsub = (kmax + 31) / 32;             // sub-tiles of the block; wave w takes w, w + 4, ...

    // Key groups: the constants of each row for each block of keys, formed once by the workgroup instead of by every wave
    // for every sub-tile and sweep (three double-precision divisions a lane): alpha^(g) for sweep A, then, in the same place,
    // m^(g) and c_int^(g).  (1024 tokens, 32 / 8 heads, d 128, 128-row and 64-key groups: 61 -> 54 us.)
    double *const kt_alpha = (double *)(PT + NIDX * 32);
    v2i *const kt = (v2i *)(PT + NIDX * 32);
    auto kg_blk = [&](int j) __attribute__((always_inline)) { return quotient(j, p.by_k_subtiles); }; // of sub-tile j
    auto each_group = [&](auto f) __attribute__((always_inline)) {
        const int n_entries = (kg_blk(nsub - 1) + 1) * 32;
        for (int e = tid; e < n_entries; e += NT) f(e);
    };
    if constexpr (kg_table) {
        each_group([&](int e) __attribute__((always_inline)) { kt_alpha[e] = (scale_q(q0 + (e & 31)) * (double)skp[e >> 5]) / p.sqrt_d; });
        __syncthreads();
    }

    // K fragments of sub-tile j straight from global memory: key row 32 j + n, bytes [32 kb + 16 h, +16)
    auto load_kf = [&](int j, v4i (&kf)[KB]) __attribute__((always_inline)) {
        // key rows at or past L: the last row is read instead; their scores are hidden keys and never used
        const int key = min(32 * j + n, L - 1);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) kf[kb] = v4i{0, 0, 0, 0};
        if (j < nsub) { // wave-uniform
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) kf[kb] = *(const v4i *)(Kp + (int64_t)key * p.ks[2] + kb * 32 + h * 16);
        }
    };
    v16i start = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}; // what the scores are added to
    auto scores = [&](const v4i (&kf)[KB]) __attribute__((always_inline)) {
        v16i s = start;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[kb], qf[kb], s, 0, 0, 0);
        return s;
    };
    auto visible = [&](int key) { return key < L && (!CAUSAL || key <= row); };
    // wave-uniform: every key of sub-tile j is visible to every row of the block
    auto sub_is_full = [&](int j) { return 32 * j + 32 <= L && (!CAUSAL || 32 * j + 31 <= q0); };

    // The wave's sub-tiles in order, K fragments of the next one requested before this one is computed; the two
    // register sets (and V buffers) alternate statically, so nothing is copied and no wait is forced early.
    // body(j, kf, buffer number); prefetch(j, buffer number) is called with the K request of sub-tile j.
    auto walk = [&](auto prefetch, auto body) __attribute__((always_inline)) {
        v4i kA[KB], kB[KB];
        load_kf(wave, kA);
        prefetch(wave, 0);
        for (int j = wave; j < nsub; j += 2 * WAVES) {
            load_kf(j + WAVES, kB);
            prefetch(j + WAVES, 1);
            body(j, kA, 0);
            if (j + WAVES < nsub) {
                load_kf(j + 2 * WAVES, kA);
                prefetch(j + 2 * WAVES, 0);
                body(j + WAVES, kB, 1);
            }
        }
    };
    auto no_prefetch = [&](int, int) {};

    // ================================================================= sweep A: row max
    int mx = INT32_MIN;
    walk(no_prefetch, [&](int j, const v4i (&kf)[KB], int) __attribute__((always_inline)) {
        const v16i s = scores(kf);
        if constexpr (KG) {
            const bool full = sub_is_full(j);
            if constexpr (kg_blocks) {
                int lmax = INT32_MIN; // no score is INT32_MIN
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (full || visible(32 * j + acc_key(i, h))) lmax = max(lmax, s[i]);
                if (lmax != INT32_MIN) {
                    const double al = kg_table ? kt_alpha[kg_blk(j) * 32 + n] : kg_alpha(32 * j);
                    const double x = al * (double)lmax; // alpha > 0: the block's largest logit
                    Mreal = x > Mreal ? x : Mreal;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = 32 * j + acc_key(i, h);
                    if (full || visible(key)) {
                        const double x = kg_alpha(key) * (double)s[i];
                        Mreal = x > Mreal ? x : Mreal;
                    }
                }
            }
        } else if (sub_is_full(j)) {
#pragma unroll
            for (int i = 0; i < 16; i += 2) mx = max(max(s[i], s[i + 1]), mx);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = visible(32 * j + acc_key(i, h)) ? max(mx, s[i]) : mx;
        }
    });
    mx = max(mx, __shfl_xor(mx, 32));
    if (h == 0) red[0][wave][n] = mx;
    __syncthreads(); // (also: lut_lds and the zeroed accumulators are visible)
    mx = max(max(red[0][0][n], red[0][1][n]), max(red[0][2][n], red[0][3][n]));
    if (!row_ok) mx = 0; // rows outside the problem: zero scores, never stored
    if constexpr (KG) {
        double o = __shfl_xor(Mreal, 32);
        Mreal = o > Mreal ? o : Mreal;
        if (h == 0) red_m[wave][n] = Mreal;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            o = red_m[w][n];
            Mreal = o > Mreal ? o : Mreal;
        }
    }

    ScoreIndex<M> si;
    si.init(M == IDX_ROW64 ? row_hp(row) : hp, KG ? 0 : mx, top);
    [[maybe_unused]] RowIndex &ri = si.ri;
#pragma unroll
    for (int i = 0; i < 16; ++i) start[i] = si.start();
    // Key groups: where every lane's threshold is small enough, the index map runs in fp32 (see RowIndex32), the choice
    // uniform for the wave.
    RowIndex32 ri32;
    bool single = false;
    // Key groups: the constants of the lane's row for the key block of `key`, as in the tiled kernel: c_int^(g) =
    // round(c / alpha^(g)) capped at 2^30, m^(g) = round(M / alpha^(g)) clamped to [-2^22, 2^30 + 2^22], which changes no
    // result (comparisons written so that a NaN from an unusable scale lands on a bound).
    auto kg_group = [&](double al, double M_row) __attribute__((always_inline)) {
        double cd = __builtin_floor(p.clip / al + 0.5);
        cd = cd >= 1.0 ? cd : 1.0;
        cd = cd < 1073741824.0 ? cd : 1073741824.0;
        double md = __builtin_floor(M_row / al + 0.5);
        md = md < 1077936128.0 ? md : 1077936128.0;
        md = md > -4194304.0 ? md : -4194304.0;
        return v2i{(int)md, (int)cd};
    };
    if constexpr (kg_table) {
        each_group([&](int e) __attribute__((always_inline)) { // (a thread meets the entries it wrote)
            double M_row = red_m[0][e & 31];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) {
                const double o = red_m[w][e & 31];
                M_row = o > M_row ? o : M_row;
            }
            kt[e] = kg_group(kt_alpha[e], M_row);
        });
        __syncthreads();
    }
    auto set_double = [&](v2i g) __attribute__((always_inline)) {
        ri.mx = g[0];
        ri.bound = g[0] - g[1];
        const uint64_t bits = (uint64_t)__double_as_longlong((double)top / (double)g[1]) + 1ull; // the double after top / c_int
        ri.negr = __longlong_as_double((long long)(bits ^ 0x8000000000000000ull));
    };
    auto kg_index = [&](int key) __attribute__((always_inline)) {
        const v2i g = kg_table ? kt[kg_blk(key >> 5) * 32 + n] : kg_group(kg_alpha(key), Mreal);
        ri.mx = g[0];
        ri.bound = g[0] - g[1];
        single = __all(ri32.init(g[1], g[0], top));
        if (!single) set_double(g);
    };
    // table places of the sixteen scores of sub-tile j (in place).  Hidden keys (masked: there may be some) take the last
    // table entry, which is 0; with key groups they and logits above their block's image of the maximum are
    // brought to it, and the caller leaves them out.
    const int last = CAUSAL ? min(L - 1, row) : L - 1; // last key the lane's row sees
    auto indices = [&](int j, v16i &s, auto masked_tag) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        if constexpr (!KG) {
            const int lim = last - 32 * j - 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = (int)si.index(!MASKED || acc_key(i, 0) <= lim ? s[i] : si.hidden());
        } else if constexpr (!kg_blocks) {
            // Four logits at a time, whose divisions do not depend on each other, and one choice of map for them.  (One at a time: 87.1 us
            // for 75.7 in the first case above, and 200 rows of 4096 keys, blocks of 48, 16 heads, d 64, where a wave has a SIMD to
            // itself, 467 to 489 with the order that the compiler found, for 324.)
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                v2i g[4];
                RowIndex32 m32[4];
                bool fits = true;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    g[r] = kg_group(kg_alpha(32 * j + acc_key(i + r, h)), Mreal);
                    fits = m32[r].init(g[r][1], g[r][0], top) && fits;
                }
                if (__all(fits)) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[i + r] = (int)m32[r](min(max(s[i + r], g[r][0] - g[r][1]), g[r][0]));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        set_double(g[r]);
                        s[i + r] = (int)ri(min(max(s[i + r], ri.bound), ri.mx));
                    }
                }
            }
        } else {
            kg_index(32 * j);
            if (single) {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[i] = (int)ri32(min(max(s[i], ri.bound), ri.mx));
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[i] = (int)ri(min(max(s[i], ri.bound), ri.mx));
            }
        }
    };

    // ================================================================= sweep B: row sum of E_hat
    const uint8_t *lut_b = (const uint8_t *)lut_lds;
    uint32_t sum = 0;
    walk(no_prefetch, [&](int j, const v4i (&kf)[KB], int) __attribute__((always_inline)) {
        v16i s = scores(kf);
        if (sub_is_full(j)) {
            uint32_t e[16];
            indices(j, s, std::false_type{});
#pragma unroll
            for (int i = 0; i < 16; ++i) e[i] = lut_b[s[i]];
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += e[i];
        } else {
            indices(j, s, std::true_type{});
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t e = lut_b[s[i]];
                sum += !KG || visible(32 * j + acc_key(i, h)) ? e : 0u;
            }
        }
    });
    sum += __shfl_xor(sum, 32);
    if (h == 0) red[1][wave][n] = (int32_t)sum;
    __syncthreads();
    sum = (uint32_t)red[1][0][n] + (uint32_t)red[1][1][n] + (uint32_t)red[1][2][n] + (uint32_t)red[1][3][n];
    const bool big = __any(row_ok && sum <= BIG_ROW_SUM); // wave-uniform, and the same for the four waves
    if (wave == 0 && h == 0 && row_ok) {
        if (!KG && p.dbg_row_max) p.dbg_row_max[(int64_t)bh * LQ + (row - rlo)] = mx;
        if (p.dbg_row_sum) p.dbg_row_sum[(int64_t)bh * LQ + (row - rlo)] = (int32_t)sum;
    }
    // per-row probability table, once per workgroup: PT[place of idx][row] = round(255 LUT_hat[idx] / S)
    for (int e = tid; e < NIDX * 32; e += NT) {
        const int idx = e >> 5, r = e & 31;
        const uint32_t S = (uint32_t)red[1][0][r] + (uint32_t)red[1][1][r] + (uint32_t)red[1][2][r] + (uint32_t)red[1][3][r];
        const uint32_t Sd = q0 + r >= rlo && q0 + r < rhi ? S : 1u << 24; // rows outside the problem: all probabilities 0
        PT[e] = prob_u8(lut_b[idx], Sd, __builtin_amdgcn_rcpf((float)(2u * Sd))); // (LUT_hat is 0 past the table)
    }
    __syncthreads();

    // ================================================================= sweep C: P_hat and P_hat.V_hat
    // V sub-tile j into this wave's buffer `buf`: direct global -> LDS loads, the XOR swizzle applied to the
    // global address; rows at or past L arrive as zeros from the range check of the buffer descriptor
    auto stage_v = [&](int j, int buf) __attribute__((always_inline)) {
        if (j >= nsub) return; // wave-uniform
        const int key0 = 32 * j;
        const int8_t *tb = Vp + (int64_t)key0 * p.vs[2];
        const int64_t rem = (int64_t)(L - key0 - 1) * p.vs[2] + D;
        const uint32_t nrec = rem <= 0 ? 0u : (rem > 0xffffffffll ? 0xffffffffu : (uint32_t)rem);
#if defined(__HIP_DEVICE_COMPILE__) // the host pass has neither the descriptor type nor the builtins
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)tb, 0, (int)nrec, 0x00020000);
#pragma unroll
        for (int blk = 0; blk < NBLK; ++blk) {
            const int key = blk * RPB + lane / CPR, cpos = lane % CPR;
            const int goff = key * (int)p.vs[2] + ((cpos ^ swz_v<D>(key)) << 4); // the host checked 128 * stride < 2^31
            int8_t *dst = (buf ? &Vw1[wave][0] : &Vw0[wave][0]) + blk * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16, goff, 0, 0, 0);
        }
#else
        (void)tb, (void)nrec, (void)buf;
#endif
    };
    // transposing read of V^T fragments: lanes 2j, 2j+1 of a 16-lane group point at the two 8-byte halves of a key row
    const int tr_i = lane & 15, tr_g = (lane >> 4) & 1;
    auto vt_frag = [&](const int8_t *Vb, int cb) __attribute__((always_inline)) {
        v4i a;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int jj = tr_i >> 1;
            const int key = 8 * (2 * r + (jj >> 2)) + 4 * h + (jj & 3);
            const int c16 = 2 * cb + tr_g;
            const int8_t *ptr = Vb + key * D + ((c16 ^ swz_v<D>(key)) << 4) + 8 * (tr_i & 1);
            const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3))) *)ptr);
            a[2 * r] = x[0];
            a[2 * r + 1] = x[1];
        }
        return a;
    };

    v16i o[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cb][i] = 0;
    const uint32_t *pt = PT + n;
    walk(stage_v, [&](int j, const v4i (&kf)[KB], int buf) __attribute__((always_inline)) {
        v16i s = scores(kf);
        const bool full = sub_is_full(j);
        if (full) indices(j, s, std::false_type{});
        else indices(j, s, std::true_type{});
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = (int)pt[s[i] * 32];
        v4i pf, vf[CB];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t pb4[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 4 * g + r;
                pb4[r] = (uint32_t)s[i];
                if (KG && !full) pb4[r] = visible(32 * j + acc_key(i, h)) ? pb4[r] : 0u;
            }
            pf[g] = (int)(((pb4[1] << 8) | pb4[0]) | (((pb4[3] << 8) | pb4[2]) << 16));
        }
        // (the compiler waits for this wave's direct-to-LDS loads into the buffer before the reads below)
        const int8_t *Vb = buf ? &Vw1[wave][0] : &Vw0[wave][0];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) vf[cb] = vt_frag(Vb, cb);
        if (big) add_pv<true>(vf, pf, o);
        else add_pv<false>(vf, pf, o);
    });
    // the accumulators of the four waves meet in LDS: register i of lane (n, h) in channel block cb is
    // row n, channel 32 cb + 8 (i / 4) + 4 h + (i % 4)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) atomicAdd(&acc_lds[n][cb * 32 + 8 * (i >> 2) + 4 * h + (i & 3)], o[cb][i]);
    __syncthreads();

    // ================================================================= epilogue: 8 threads per row
    constexpr int CPT = D / 8; // channels per thread
    const int er = tid >> 3, ec0 = (tid & 7) * CPT, erow = q0 + er;
    if (erow >= rlo && erow < rhi) {
        int8_t *Op = p.out + (int64_t)b * p.os[0] + (int64_t)hq * p.os[1] + (int64_t)(erow - rlo) * p.os[2];
        HeadParams he = KG || M == IDX_ROW64 ? row_hp(erow) : hp;
        if (KG && p.head_status[hq] != 0) he.rq_mult = 0; // an unusable scale somewhere in the head: all zeros
#pragma unroll
        for (int c4 = 0; c4 < CPT; c4 += 4) {
            uint32_t packed = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ch = ec0 + c4 + r;
                const int32_t acc = acc_lds[er][ch];
                if (p.dbg_acc) p.dbg_acc[((int64_t)bh * LQ + (erow - rlo)) * D + ch] = acc;
                packed |= ((uint32_t)requant_any(acc, he.rq_mult, he.rq_shift) & 0xffu) << (8 * r);
            }
            *(uint32_t *)(Op + ec0 + c4) = packed;
        }
    }
    };
    if constexpr (MODE == IDX_DEVICE) {
        if (hp.fma_r != 0) body(std::integral_constant<int, IDX_FMA>{}); // uniform for the workgroup
        else body(std::integral_constant<int, IDX_FP64>{});
    } else {
        body(std::integral_constant<int, MODE>{});
    }
}

// Slots of an XCD whose order is folded, or 0.  Where all workgroups of a causal launch are resident at once, a compute unit
// takes one from each round of 32 and nothing is dealt later: with the longest blocks of rows first in every round, the unit
// with the longest block of the first round also gets the longest of the others (2048 rows, two heads an XCD: 156 sub-tile
// columns against 126 on average).  Reversing every other round evens that out: 1024 rows, 16 heads, d 128: 28.5 -> 25.2 us;
// 4096 rows, 8 heads, d 64: 60.1 -> 56.0; 2048 rows, 16 heads, d 64: 31.2 -> 30.6.  (Sweeps A+B of 512 workgroups gained nothing from it.)
inline int fold_slots(int64_t grid, bool causal, int workgroups_per_cu)
{
    return causal && grid > 256 && grid <= (int64_t)256 * workgroups_per_cu ? (int)(grid / NUM_XCD) : 0;
}

template <int D, bool CAUSAL>
int launch_mode(const FwdParams &p_in, int idx_mode, hipStream_t st)
{
    FwdParams p = p_in;
    const int64_t n_wg = fwd_map_work(p);
    p.map.fold = fold_slots(n_wg, CAUSAL, splitk_waves(D, idx_mode));
    const dim3 grid((unsigned)n_wg), block(NT);
    const unsigned sh = (unsigned)((p.top < 32 ? 32 : 64) * 32 * sizeof(uint32_t)); // the per-row probability table
    if (idx_mode == IDX_FMA)
        hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_FMA>), grid, block, sh, st, p);
    else if (idx_mode == IDX_DEVICE)
        hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_DEVICE>), grid, block, sh, st, p);
    else if (idx_mode == IDX_ROW64)
        hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_ROW64>), grid, block, sh, st, p);
    else if (idx_mode == IDX_KGROUP && p.k_block % 32 != 0)
        hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_KGROUP, STRADDLING>), grid, block, sh, st, p);
    else if (idx_mode == IDX_KGROUP) {
        p.by_k_subtiles = fast_div((uint32_t)(p.k_block / 32));
        // a table of up to 64 blocks of keys, 16 KiB, which leave two workgroups a compute unit at d = 128 (51 KiB without)
        if (p.n_kblk <= 64)
            hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_KGROUP, WHOLE_TABLE>), grid, block, sh + (unsigned)p.n_kblk * 32u * 8u, st, p);
        else
            hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_KGROUP, WHOLE>), grid, block, sh, st, p);
    } else if (idx_mode == IDX_FP64)
        hipLaunchKernelGGL((fwd_splitk_kernel<D, CAUSAL, IDX_FP64>), grid, block, sh, st, p);
    else
        return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

} // namespace

// p.n_qtiles counts 32-row blocks; every parameter mode; no workspace.
int launch_fwd_splitk(const FwdParams &p, int d, int idx_mode, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (d == 64) return p.causal ? launch_mode<64, true>(p, idx_mode, st) : launch_mode<64, false>(p, idx_mode, st);
    if (d == 128) return p.causal ? launch_mode<128, true>(p, idx_mode, st) : launch_mode<128, false>(p, idx_mode, st);
    return (int)hipErrorInvalidValue;
}

} // namespace intattn
