// Fused IntAttention forward for gfx950 (MI355X).
//
// One workgroup = 4 wavefronts; each wavefront owns RB blocks of 32 query rows of one
// (batch, query head).  Keys/values stream through LDS in tiles of BK keys, double
// buffered, one barrier per tile.  Because IndexSoftmax (Sec. 3.1-3.2) needs the exact row
// maximum before any table index and the exact row sum before any probability, the key axis
// is swept three times, recomputing the INT8 score tile each time instead of ever storing
// the L x L matrix:
//   sweep A: S^T = K.Q^T (MFMA)            -> running row max
//   sweep B: S^T again -> clip, index (the row max is folded into per-row constants), LUT_hat ->
//            row sum; then the 2^b distinct probabilities of the row, P_hat = round(255 E/S), go
//            to a per-row table in LDS
//   sweep C: S^T again -> index -> per-row table -> 16 probability bytes per lane, which
//            are exactly one MFMA B operand of O^T += V^T.P^T; then requantize and store.
// Scores are produced transposed (keys x queries) so that each lane owns one query row:
// row max and row sum are in-lane plus one exchange between the two half-waves.
//
// All intermediate magnitudes stay below 2^31 for L < 131072.
//
// LDS tiles are row-major [key][d] with the 16-byte chunks of each row XOR-swizzled so that
// both access patterns are bank-conflict free: K fragments are read with 128-bit loads
// (one key row per lane), V^T fragments with the transposing 64-bit load (eight key rows per
// 16 lanes).  The tiles are filled by buffer loads that write LDS directly.
//
// Within a tile the work is ordered in phases (all fragment reads, all MFMAs, all index
// arithmetic with every table lookup in flight, then the consumers).  This is the kernel for
// small problems (all three sweeps in one launch) and for sweeps A+B of large ones; sweep C of
// large problems has a kernel of its own.  Sweep B takes a tile sub-tile by sub-tile, which leaves room for the start values
// of the IDX_FMA map at three waves a SIMD, and costs two vector instructions, half an addition and a lookup a score
// (1 x 8192, 32 / 8 heads, d 128: sweeps A and B 292 -> 262 us; A alone 118).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace fwdk {

constexpr int WAVES = 4;
constexpr int NT = WAVES * 64;

// The kernel for one work item with the index scheme M as a compile-time constant; the LDS arrays are the kernel's (see
// there), ksp is the number of this workgroup's range of key tiles out of n_split.  A function rather than a lambda in the
// kernel: as a lambda it cost the instantiations with sweep C 13 (d = 64) to 28 (d = 128) registers and 5 to 9 % more
// vector instructions (139 and 221 registers as it is, causal, one launch, fma map).
template <int D, int RB, int KT, bool CAUSAL, int M, int PH>
__device__ __forceinline__ void fwd_body(const FwdParams &p, const WorkItem &wi, const HeadParams &hp, const int ksp, const int n_split,
                                         int8_t *Ks0, int8_t *Ks1, int8_t *Vs0, int8_t *Vs1, uint32_t *PT, uint32_t *lut_lds)
{
    constexpr int KS = KT; // sub-tiles sweep C computes per step: the whole staged tile
    constexpr int KB = D / 32;       // 32-wide blocks of the head dimension
    constexpr int CB = D / 32;       // 32-wide blocks of output channels
    // Sweeps A and B alone stage twice as many keys as they compute at a time: half the barriers and address arithmetic a key
    // (1 x 4096 without a mask, 32 / 8 heads, d 128: 155 -> 137 us; 8 x 1024, causal: 63 -> 56; 1 x 8192: 267 -> 265).
    constexpr int PARTS = PH == 1 || PH == 3 || PH == 4 ? 2 : 1; // computed parts of a staged tile
    constexpr int BK = 32 * KT;      // keys per part
    constexpr int SK = BK * PARTS;   // keys per staged tile
    constexpr int BQ = WAVES * RB * 32;
    constexpr int TILE = SK * D;     // bytes
    constexpr int NBLK = TILE / 1024;                // 1 KiB blocks per tile (one wave-wide 16-byte load each)
    constexpr int JB = (NBLK + WAVES - 1) / WAVES;   // blocks per wave per tile
    constexpr int CPR = D / 16;                      // 16-byte chunks per key row
    constexpr int RPB = 1024 / D;                    // key rows per block

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 31, h = lane >> 5;
    const int b = wi.b, hq = wi.hq, kvh = wi.kvh, qt = wi.qt + p.row_lo / BQ;
    const int bh = b * p.Hq + hq;
    const int L = p.Lk; // keys
    // query rows: [rlo, rhi) of the numbering in which row r sees keys <= r under the causal mask
    const int rlo = p.row_lo, rhi = p.row_lo + p.L, LQ = p.L;
    const uint32_t top = (uint32_t)p.top;
    const int NIDX = top < 32 ? 32 : 64; // table entries allocated per row
    // Finer quantization groups over both axes (Sec. 3.3): the lane's query row has the scale of its block
    // of q_block rows, every key the scale of its block of k_block keys.  alpha^(g) = s_Q^(g) s_K^(g) / sqrt(d)
    // per logit; the row maximum is taken over the dequantized logits (fp64), and each key block measures
    // distances from the image of that maximum in its own integer units.
    constexpr bool KG = M == IDX_KGROUP;
    const float *skp = KG ? p.sk_blocks + (int64_t)(b * p.Hkv + kvh) * p.n_kblk : nullptr;
    const bool kg_blocks = KG && (p.k_block % 32) == 0; // a 32-key sub-tile lies in one key block (uniform)
    double sq_row[RB], Mreal[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        sq_row[rb] = 0.0;
        Mreal[rb] = -__builtin_inf();
    }

    const int q0 = qt * BQ, qw0 = q0 + wave * (RB * 32);
    const int8_t *Qp = p.q + (int64_t)b * p.qs[0] + (int64_t)hq * p.qs[1];
    const int8_t *Kp = p.k + (int64_t)b * p.ks[0] + (int64_t)kvh * p.ks[1];
    const int8_t *Vp = p.v + (int64_t)b * p.vs[0] + (int64_t)kvh * p.vs[1];

    // LUT_hat by place (see ScoreIndex)
    if (tid < 64) {
        const int idx = ScoreIndex<M>::place(tid, (int)top);
        ((uint8_t *)lut_lds)[tid] = idx >= 0 ? (uint8_t)(p.lut[idx / 4] >> (8 * (idx % 4))) : (uint8_t)0;
    }
    if constexpr (KG) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = q0 + wave * (RB * 32) + 32 * rb + n;
            const int lr = (row >= rlo && row < rhi) ? row - rlo : 0;
            sq_row[rb] = (double)p.sq_rows[(int64_t)bh * p.n_rowblk + lr / p.q_block];
        }
    }
    // alpha^(g) of the logit (lane's row of row block rb, key); keys past the end take the last block's scale
    auto kg_alpha = [&](int rb, int key) __attribute__((always_inline)) {
        return (sq_row[rb] * (double)skp[min(key, L - 1) / p.k_block]) / p.sqrt_d;
    };

    // Q fragments: row block rb, row qw0 + 32 rb + n, bytes [32 kb + 16 h, +16); zeros for rows outside the problem.  With all sweeps and
    // two row blocks a wave, where registers run past 256, lanes without a row load the first one and select: around a branch the
    // compiler put a copy of a register that lives on (in the kernel of both index maps, d = 128) where those lanes were still
    // switched off.
    v4i qf[RB][KB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = qw0 + 32 * rb + n;
        const bool row_ok = row >= rlo && row < rhi;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if constexpr (RB == 2 && PH == 0) {
                const v4i x = *(const v4i *)(Qp + (int64_t)(row_ok ? row - rlo : 0) * p.qs[2] + kb * 32 + h * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i) qf[rb][kb][i] = row_ok ? x[i] : 0;
            } else {
                qf[rb][kb] = v4i{0, 0, 0, 0};
                if (row_ok) qf[rb][kb] = *(const v4i *)(Qp + (int64_t)(row - rlo) * p.qs[2] + kb * 32 + h * 16);
            }
        }
    }

    const int kmax = CAUSAL ? min(L, q0 + BQ) : L;
    const int ntiles = (kmax + SK - 1) / SK;
    // this workgroup's staged key tiles [tlo, thi)
    const int tlo = PH == 3 || PH == 4 ? ntiles * ksp / n_split : 0;
    const int thi = PH == 3 || PH == 4 ? ntiles * (ksp + 1) / n_split : ntiles;
    if ((PH == 3 || PH == 4) && tlo >= thi) return; // fewer tiles than ranges (uniform for the workgroup)

    // ---- staging: global -> LDS directly (no registers, no LDS store instructions), a tile ahead.
    // One wave-wide 16-byte load fills 1 KiB of LDS, lane i at byte 16 i: the lane's slot is key row
    // i / CPR of the block at chunk position i % CPR, which under the XOR swizzle holds global chunk
    // (i % CPR) ^ swz(key) -- so the swizzle is applied to the global address.
    int dma_goff_k[JB], dma_goff_v[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        const int key = (wave + WAVES * j) * RPB + lane / CPR, cp = lane % CPR;
        dma_goff_k[j] = key * (int)p.ks[2] + ((cp ^ swz_k<D>(key)) << 4); // the host checked BK * stride < 2^31
        dma_goff_v[j] = key * (int)p.vs[2] + ((cp ^ swz_v<D>(key)) << 4);
    }
    // The loads go through a buffer descriptor that starts at the tile and ends with the last
    // byte of key row L-1, so key rows at or past L come back as zeros from the range check.
    auto dma_tile = [&](const int8_t *base, int64_t stride, const int (&goff)[JB], int t, int8_t *dst)
                        __attribute__((always_inline)) {
        const int8_t *tb = base + (int64_t)t * SK * stride; // wave-uniform
        const int64_t rem = (int64_t)(L - t * SK - 1) * stride + D;
        const uint32_t nrec = rem > 0xffffffffll ? 0xffffffffu : (uint32_t)rem;
#if defined(__HIP_DEVICE_COMPILE__) // the host pass has neither the descriptor type nor the builtins
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)tb, 0, (int)nrec, 0x00020000);
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int blk = wave + WAVES * j;
            if (NBLK % WAVES != 0 && blk >= NBLK) break;    // wave-uniform
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(dst + blk * 1024), 16,
                                                     goff[j], 0, 0, 0);
        }
#else
        (void)tb, (void)nrec, (void)goff, (void)dst;
#endif
    };
    auto dma_k = [&](int t, int8_t *dst) __attribute__((always_inline)) { dma_tile(Kp, p.ks[2], dma_goff_k, t, dst); };
    auto dma_v = [&](int t, int8_t *dst) __attribute__((always_inline)) { dma_tile(Vp, p.vs[2], dma_goff_v, t, dst); };
    // One sweep over the key tiles, whose parts (numbered through) go to body: tile t+1 is requested before tile t is computed; the barrier at
    // the end of a step (which waits for the wave's own loads first) publishes it and frees tile
    // t's buffer.  Unrolled by two so that every buffer is named statically.
    auto sweep = [&](auto with_v, auto body) __attribute__((always_inline)) {
        constexpr bool WITH_V = decltype(with_v)::value;
        dma_k(tlo, Ks0);
        if (WITH_V) dma_v(tlo, Vs0);
        publish_tiles_barrier();
        for (int t = tlo; t < thi; t += 2) {
            if (t + 1 < thi) {
                dma_k(t + 1, Ks1);
                if (WITH_V) dma_v(t + 1, Vs1);
            }
#pragma unroll
            for (int part = 0; part < PARTS; ++part) body(t * PARTS + part, (const int8_t *)Ks0 + part * BK * D, (const int8_t *)Vs0);
            publish_tiles_barrier();
            if (t + 1 < thi) {
                if (t + 2 < thi) {
                    dma_k(t + 2, Ks0);
                    if (WITH_V) dma_v(t + 2, Vs0);
                }
#pragma unroll
                for (int part = 0; part < PARTS; ++part) body((t + 1) * PARTS + part, (const int8_t *)Ks1 + part * BK * D, (const int8_t *)Vs1);
                publish_tiles_barrier();
            }
        }
    };

    // ---- S^T blocks of one tile: KT sub-tiles of 32 keys x RB row blocks, KB chained MFMAs each.
    // The chains are interleaved (kb outermost) so that consecutive MFMAs are independent.
    // All K fragments of the tile are requested before the first MFMA (the scheduling barrier keeps
    // the compiler from re-serialising read -> wait -> MFMA), so one LDS latency is paid per tile.
    auto qk_tile = [&](const int8_t *Kb, int st0, auto &s) __attribute__((always_inline)) {
        constexpr int NS = (int)(sizeof(s) / sizeof(s[0]));
        v4i kf[KB][NS];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int st = 0; st < NS; ++st) {
                const int key = 32 * (st0 + st) + n;
                kf[kb][st] = *(const v4i *)(Kb + key * D + (((2 * kb + h) ^ swz_k<D>(key)) << 4));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int st = 0; st < NS; ++st) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    s[st][rb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[kb][st], qf[rb][kb], s[st][rb], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto read_kf = [&](const int8_t *Kb, int st, v4i (&kf)[KB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int key = 32 * st + n;
            kf[kb] = *(const v4i *)(Kb + key * D + (((2 * kb + h) ^ swz_k<D>(key)) << 4));
        }
    };
    // the scores of one sub-tile, added to `start`
    auto qk_sub = [&](const v4i (&kf)[KB], const v16i (&start)[RB], v16i (&s)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                s[rb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[kb], qf[rb][kb], kb == 0 ? start[rb] : s[rb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto visible = [&](int key, int row) { return key < L && (!CAUSAL || key <= row); };
    // wave-uniform: every key of tile t is visible to every row of this wave (no mask needed)
    auto tile_is_full = [&](int t) { return (t + 1) * BK <= L && (!CAUSAL || (t + 1) * BK - 1 <= qw0); };
    // wave-uniform: no key of tile t is visible to any row of this wave
    auto tile_is_hidden = [&](int t) { return (PARTS > 1 && t * BK >= L) || (CAUSAL && t * BK > qw0 + RB * 32 - 1); };

    // ================================================================= sweep A: row max
    int mx[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) mx[rb] = INT32_MIN;

    // One part of sweep A, sub-tile by sub-tile: the scores of the next sub-tile ahead of the maxima of this one.
    auto tile_a = [&](auto masked_tag, int t, const int8_t *Kb) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        v4i kf[KT][KB];
        v16i s[KT][RB], zero[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) zero[rb][i] = 0;
#pragma unroll
        for (int st = 0; st < KT; ++st) read_kf(Kb, st, kf[st]);
        __builtin_amdgcn_sched_barrier(0);
        auto take = [&](int st) __attribute__((always_inline)) {
            const int klo = t * BK + 32 * st;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int row = qw0 + 32 * rb + n;
                if constexpr (KG) {
                    if (kg_blocks) {
                        int lmax = INT32_MIN; // no score is INT32_MIN
#pragma unroll
                        for (int i = 0; i < 16; ++i)
                            if (!MASKED || visible(klo + acc_key(i, h), row)) lmax = max(lmax, s[st][rb][i]);
                        if (lmax != INT32_MIN) {
                            const double x = kg_alpha(rb, klo) * (double)lmax; // alpha > 0: the block's largest logit
                            Mreal[rb] = x > Mreal[rb] ? x : Mreal[rb];
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int key = klo + acc_key(i, h);
                            if (!MASKED || visible(key, row)) {
                                const double x = kg_alpha(rb, key) * (double)s[st][rb][i];
                                Mreal[rb] = x > Mreal[rb] ? x : Mreal[rb];
                            }
                        }
                    }
                } else if (MASKED) {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        mx[rb] = visible(klo + acc_key(i, h), row) ? max(mx[rb], s[st][rb][i]) : mx[rb];
                } else {
#pragma unroll
                    for (int i = 0; i < 16; i += 2) mx[rb] = max(max(s[st][rb][i], s[st][rb][i + 1]), mx[rb]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int st = 0; st < KT; ++st) {
            qk_sub(kf[st], zero, s[st]);
            if (st > 0) take(st - 1);
        }
        take(KT - 1);
    };

    if constexpr (PH != 2 && PH != 4) {
        sweep(std::false_type{}, [&](int t, const int8_t *Kb, const int8_t *) __attribute__((always_inline)) {
            if (tile_is_full(t)) tile_a(std::false_type{}, t, Kb);
            else if (!tile_is_hidden(t)) tile_a(std::true_type{}, t, Kb);
        });
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) mx[rb] = max(mx[rb], __shfl_xor(mx[rb], 32));
        if constexpr (KG) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const double o = __shfl_xor(Mreal[rb], 32);
                Mreal[rb] = o > Mreal[rb] ? o : Mreal[rb];
            }
        }
    } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = qw0 + 32 * rb + n;
            mx[rb] = (row >= rlo && row < rhi) ? p.ws_row_max[(int64_t)bh * LQ + (row - rlo)] : 0;
        }
    }

    if constexpr (PH == 3) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = qw0 + 32 * rb + n;
            if (h == 0 && row >= rlo && row < rhi) atomicMax(&p.ws_row_max[(int64_t)bh * LQ + (row - rlo)], mx[rb]);
        }
        return;
    }

    // exact index map of each row block's lane row, applied to the accumulators of its scores
    // parameters of the block of query rows that `row` lies in (finer groups over query rows, Sec. 3.3)
    auto row_hp = [&](int row) __attribute__((always_inline)) {
        const int lr = (row >= rlo && row < rhi) ? row - rlo : 0;
        return p.row_table[(int64_t)bh * p.n_rowblk + lr / p.q_block];
    };
    // (start values in double would leave the kernels with sweep C at d = 64 three waves a SIMD instead of four: 140 registers, 126 without)
    ScoreIndex<M, PH == 0 || PH == 2, PH == 0 || M == IDX_ROW64> si[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) si[rb].init(M == IDX_ROW64 ? row_hp(qw0 + 32 * rb + n) : hp, KG ? 0 : mx[rb], top);
    // Key groups: the index constants of the lane's row for the key block of `key` (Sec. 3.3):
    // c_int^(g) = round(c / alpha^(g)) capped at 2^30, m^(g) = round(M / alpha^(g)), the fp64 index map's
    // factor for c_int^(g).  m^(g) is clamped to [-2^22, 2^30 + 2^22]: below every logit / far enough above
    // every logit that the distance exceeds any c_int, so the clamp changes no result and all later
    // arithmetic fits 32 bits (comparisons written so that a NaN from an unusable scale lands on a bound).
    auto kg_index = [&](int rb, int key) __attribute__((always_inline)) {
        const double al = kg_alpha(rb, key);
        double cd = __builtin_floor(p.clip / al + 0.5);
        cd = cd >= 1.0 ? cd : 1.0;
        cd = cd < 1073741824.0 ? cd : 1073741824.0;
        double md = __builtin_floor(Mreal[rb] / al + 0.5);
        md = md < 1077936128.0 ? md : 1077936128.0;
        md = md > -4194304.0 ? md : -4194304.0;
        const int c_int = (int)cd;
        si[rb].ri.mx = (int)md;
        si[rb].ri.bound = si[rb].ri.mx - c_int;
        const uint64_t bits = (uint64_t)__double_as_longlong((double)top / cd) + 1ull; // the double after top / c_int
        si[rb].ri.negr = __longlong_as_double((long long)(bits ^ 0x8000000000000000ull));
    };

    // ================================================================= sweep B: row sum of E_hat
    // transposing read: lanes 2j, 2j+1 of a 16-lane group point at the two 8-byte halves of key
    // row j's 16 channels; lane i of the group receives channel i of the eight rows.
    const int tr_i = lane & 15, tr_g = (lane >> 4) & 1;
    auto vt_frag = [&](const int8_t *Vb, int st, int cb) __attribute__((always_inline)) {
        v4i a;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = tr_i >> 1;
            const int key = 32 * st + 8 * (2 * r + (j >> 2)) + 4 * h + (j & 3);
            const int c16 = 2 * cb + tr_g;
            const int8_t *ptr = Vb + key * D + ((c16 ^ swz_v<D>(key)) << 4) + 8 * (tr_i & 1);
            const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3))) *)ptr);
            a[2 * r] = x[0];
            a[2 * r + 1] = x[1];
        }
        return a;
    };

    const uint8_t *lut_b = (const uint8_t *)lut_lds;
    v16i start[RB]; // what the scores are added to
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 16; ++i) start[rb][i] = si[rb].start();
    uint32_t sum[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) sum[rb] = 0;

    // One tile of sweep B, sub-tile by sub-tile: the scores, their table lookups (in place, all in flight), and, behind the
    // MFMAs of the next sub-tile, their sum.
    auto tile_b = [&](auto masked_tag, int t, const int8_t *Kb) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        v4i kf[KT][KB];
#pragma unroll
        for (int st = 0; st < KT; ++st) read_kf(Kb, st, kf[st]);
        __builtin_amdgcn_sched_barrier(0);
        v16i s[KT][RB];
        auto add_up = [&](int st) __attribute__((always_inline)) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[rb] += (uint32_t)s[st][rb][i];
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int st = 0; st < KT; ++st) {
            qk_sub(kf[st], start, s[st]);
            if (st > 0 && !KG) add_up(st - 1);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int klo = t * BK + 32 * st, row = qw0 + 32 * rb + n;
                if (KG && kg_blocks) kg_index(rb, klo);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = klo + acc_key(i, h);
                    if constexpr (KG) {
                        if (!kg_blocks) kg_index(rb, key);
                        const RowIndex &ri = si[rb].ri;
                        const uint32_t e = lut_b[ri(min(max(s[st][rb][i], ri.bound), ri.mx))];
                        sum[rb] += (!MASKED || visible(key, row)) ? e : 0u;
                    } else {
                        // a hidden key takes the table's last entry, which is 0
                        const int sc = !MASKED || visible(key, row) ? s[st][rb][i] : si[rb].hidden();
                        s[st][rb][i] = (int)lut_b[si[rb].index(sc)];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!KG) add_up(KT - 1);
    };

    if constexpr (PH != 2 && PH != 3) {
        sweep(std::false_type{}, [&](int t, const int8_t *Kb, const int8_t *) __attribute__((always_inline)) {
            if (tile_is_full(t)) tile_b(std::false_type{}, t, Kb);
            else if (!tile_is_hidden(t)) tile_b(std::true_type{}, t, Kb);
        });
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) sum[rb] += __shfl_xor(sum[rb], 32);
    }
    if constexpr (PH == 4) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = qw0 + 32 * rb + n;
            if (h == 0 && row >= rlo && row < rhi) atomicAdd(&p.ws_row_sum[(int64_t)bh * LQ + (row - rlo)], (int32_t)sum[rb]);
        }
        return;
    } else if constexpr (PH == 1) {
        // hand row max and row sum to the second launch
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = qw0 + 32 * rb + n;
            if (h == 0 && row >= rlo && row < rhi) {
                p.ws_row_max[(int64_t)bh * LQ + (row - rlo)] = mx[rb];
                p.ws_row_sum[(int64_t)bh * LQ + (row - rlo)] = (int32_t)sum[rb];
            }
        }
        return;
    } else if constexpr (PH == 2) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = qw0 + 32 * rb + n;
            sum[rb] = (row >= rlo && row < rhi) ? (uint32_t)p.ws_row_sum[(int64_t)bh * LQ + (row - rlo)] : 0u;
        }
        __syncthreads(); // LUT_hat, which the first wave put into LDS, is visible (with sweeps ahead, their barriers do that)
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = qw0 + 32 * rb + n;
        if (row < rlo || row >= rhi) sum[rb] = 1u << 24; // all probabilities 0, never stored
        // per-row probability table: PT[place of idx] = round(255 * LUT_hat[idx] / sum)
        uint32_t *pt = PT + (wave * RB + rb) * NIDX * 32;
        const float inv_2s = __builtin_amdgcn_rcpf((float)(2u * sum[rb]));
        for (int j = 0; j < NIDX / 2; ++j) {
            const int kidx = (NIDX / 2) * h + j;
            pt[kidx * 32 + n] = prob_u8(lut_b[kidx], sum[rb], inv_2s); // by place, like LUT_hat
        }
        if (!KG && p.dbg_row_max && h == 0 && row >= rlo && row < rhi) p.dbg_row_max[(int64_t)bh * LQ + (row - rlo)] = mx[rb];
        if (p.dbg_row_sum && h == 0 && row >= rlo && row < rhi) p.dbg_row_sum[(int64_t)bh * LQ + (row - rlo)] = (int32_t)sum[rb];
    }

    // ================================================================= sweep C: P_hat and P_hat.V_hat
    v16i o[RB][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[rb][cb][i] = 0;

    // One tile of sweep C in phases, separated by scheduling barriers so that each kind of LDS
    // latency is paid once per tile: S^T blocks; all probability lookups (in place, one per score)
    // followed by all V^T fragment reads; packing into MFMA B operands (LDS returns in order, so
    // the lookups land first while the fragments are still in flight).
    auto tile_c = [&](auto masked_tag, int t, const int8_t *Kb, const int8_t *Vb, int st0, v4i (&pf)[KS][RB],
                      v4i (&vf)[KS][CB]) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        v16i s[KS][RB];
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) s[st][rb] = start[rb];
        qk_tile(Kb, st0, s);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const uint32_t *pt = PT + (wave * RB + rb) * NIDX * 32 + n;
                if (kg_blocks) kg_index(rb, t * BK + 32 * (st0 + st));
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = t * BK + 32 * (st0 + st) + acc_key(i, h);
                    if constexpr (KG) {
                        if (!kg_blocks) kg_index(rb, key);
                        const RowIndex &ri = si[rb].ri;
                        s[st][rb][i] = (int)pt[ri(min(max(s[st][rb][i], ri.bound), ri.mx)) * 32];
                        if (MASKED) s[st][rb][i] = visible(key, qw0 + 32 * rb + n) ? s[st][rb][i] : 0;
                    } else { // a hidden key takes the table's last entry, whose probability is 0
                        const int sc = !MASKED || visible(key, qw0 + 32 * rb + n) ? s[st][rb][i] : si[rb].hidden();
                        s[st][rb][i] = (int)pt[si[rb].index(sc) * 32];
                    }
                }
            }
        }
#pragma unroll
        for (int st = 0; st < KS; ++st)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) vf[st][cb] = vt_frag(Vb, st0 + st, cb);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    uint32_t pb4[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) pb4[r] = (uint32_t)s[st][rb][4 * g + r];
                    pf[st][rb][g] = (int)(((pb4[1] << 8) | pb4[0]) | (((pb4[3] << 8) | pb4[2]) << 16));
                }
            }
        }
    };

    sweep(std::true_type{}, [&](int t, const int8_t *Kb, const int8_t *Vb) __attribute__((always_inline)) {
#pragma unroll
        for (int st0 = 0; st0 < KT; st0 += KS) {
            if (tile_is_hidden(t)) continue; // no P_hat of this wave's rows there
            // (the P_hat.V_hat MFMAs follow in one place for both instantiations, so that the output
            // accumulators have a single home)
            v4i pf[KS][RB], vf[KS][CB];
            // wave-uniform: every key of this step is visible to every row of this wave
            const int khi = t * BK + 32 * (st0 + KS);
            if (khi <= L && (!CAUSAL || khi - 1 <= qw0)) tile_c(std::false_type{}, t, Kb, Vb, st0, pf, vf);
            else tile_c(std::true_type{}, t, Kb, Vb, st0, pf, vf);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int st = 0; st < KS; ++st)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) add_pv<true>(vf[st], pf[st][rb], o[rb]);
        }
    });

    // ================================================================= epilogue
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = qw0 + 32 * rb + n;
        if (row < rlo || row >= rhi) continue;
        int8_t *Op = p.out + (int64_t)b * p.os[0] + (int64_t)hq * p.os[1] + (int64_t)(row - rlo) * p.os[2];
        HeadParams he = (M == IDX_ROW64 || KG) ? row_hp(row) : hp;
        if (KG && p.head_status[hq] != 0) he.rq_mult = 0; // an unusable scale somewhere in the head: all zeros
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int ch0 = cb * 32 + 8 * g + 4 * h;
                uint32_t packed = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t acc = o[rb][cb][4 * g + r];
                    if (p.dbg_acc) p.dbg_acc[((int64_t)bh * LQ + (row - rlo)) * D + ch0 + r] = acc;
                    packed |= ((uint32_t)requant_any(acc, he.rq_mult, he.rq_shift) & 0xffu) << (8 * r);
                }
                *(uint32_t *)(Op + ch0) = packed;
            }
        }
    }
}

// PH selects which part of the path this instantiation runs: 0 = all three sweeps in one launch;
// 1 = sweeps A and B only (row max and row sum go to a small workspace: 8 bytes per query row) --
// without the output accumulators it needs far fewer registers, so a wave can own 64 query rows
// (every K fragment read feeds two MFMAs) at three waves per SIMD; 2 = sweep C only, reading that
// workspace; 3 and 4 = sweep A and sweep B over one of FwdParams::split_ab ranges of the keys, for problems whose
// query tiles alone leave compute units idle: row max and row sum meet in the workspace (atomics; the launch ahead of
// these set it to INT32_MIN and 0).
template <int D, int RB, int KT, bool CAUSAL, int MODE, int PH>
__global__ __launch_bounds__(NT, (PH == 1 || PH >= 3) ? (RB == 1 ? 4 : 3) : (RB == 1 ? (KT == 1 ? 3 : 2) : 1)) void fwd_kernel(const FwdParams p)
{
    constexpr bool WITHOUT_C = PH == 1 || PH == 3 || PH == 4; // sweeps A and / or B alone
    constexpr int TILE = 32 * KT * D * (WITHOUT_C ? 2 : 1); // bytes of a staged tile of keys

    // Two buffers per operand, as separate arrays: the compiler tracks each direct-to-LDS load by
    // the array it targets, so reads of one buffer need not wait for loads into the other.
    __shared__ __attribute__((aligned(1024))) int8_t Ks0[TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Ks1[TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Vs0[WITHOUT_C ? 16 : TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Vs1[WITHOUT_C ? 16 : TILE];
    // per-row probability tables, [wave][row block][idx][row]: dynamic shared memory of WAVES * RB * NIDX * 32
    // words, NIDX = 32 or 64 table entries (none for sweeps A+B alone)
    extern __shared__ uint32_t PT[];
    __shared__ uint32_t lut_lds[16];

    int bid = (int)blockIdx.x;
    const int n_split = PH == 3 || PH == 4 ? p.split_ab : 1;
    const int ksp = PH == 3 || PH == 4 ? fwd_split_index(bid, n_split) : 0;
    const WorkItem wi = fwd_work_item(p, bid);
    if (!wi.valid) return; // padding of the XCD-aware grid (uniform for the whole workgroup)
    const HeadParams hp = p.hp_table ? p.hp_table[wi.hq] : p.hp0;
    // MODE, or, under IDX_DEVICE, the scheme that the device-derived parameters name (uniform for the workgroup)
    if constexpr (MODE == IDX_DEVICE) {
        if (hp.fma_r != 0) fwd_body<D, RB, KT, CAUSAL, IDX_FMA, PH>(p, wi, hp, ksp, n_split, Ks0, Ks1, Vs0, Vs1, PT, lut_lds);
        else fwd_body<D, RB, KT, CAUSAL, IDX_FP64, PH>(p, wi, hp, ksp, n_split, Ks0, Ks1, Vs0, Vs1, PT, lut_lds);
    } else {
        fwd_body<D, RB, KT, CAUSAL, MODE, PH>(p, wi, hp, ksp, n_split, Ks0, Ks1, Vs0, Vs1, PT, lut_lds);
    }
}

template <int D, int RB, int KT, bool CAUSAL, int PH>
int launch_mode(const FwdParams &p_in, int idx_mode, hipStream_t st)
{
    FwdParams p = p_in;
    const int n_split = PH == 3 || PH == 4 ? p.split_ab : 1;
    const dim3 grid((unsigned)fwd_map_work(p, n_split)), block(NT);
    // dynamic shared memory: the per-row probability tables (32 or 64 entries of a word per query row)
    const unsigned sh = PH == 1 || PH >= 3 ? 0u : (unsigned)(WAVES * RB * (p.top < 32 ? 32 : 64) * 32 * sizeof(uint32_t));
    if constexpr (PH == 3) { // row maxima: no index map
        hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_FP64, PH>), grid, block, sh, st, p);
    } else if (idx_mode == IDX_DEVICE) { // the scheme is known on the device only
        hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_DEVICE, PH>), grid, block, sh, st, p);
    } else if (idx_mode == IDX_KGROUP) { // groups over the key axis: single-launch kernel only
        if constexpr (RB == 1 && KT == 2 && PH == 0) hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_KGROUP, PH>), grid, block, sh, st, p);
        else return (int)hipErrorInvalidValue;
    } else if (idx_mode == IDX_FMA) {
        hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_FMA, PH>), grid, block, sh, st, p);
    } else if (idx_mode == IDX_ROW64) {
        hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_ROW64, PH>), grid, block, sh, st, p);
    } else {
        hipLaunchKernelGGL((fwd_kernel<D, RB, KT, CAUSAL, IDX_FP64, PH>), grid, block, sh, st, p);
    }
    return (int)hipGetLastError();
}

template <int RB, int KT, int PH>
int launch_shape(const FwdParams &p, int d, int idx_mode, hipStream_t st)
{
    if constexpr (!(RB == 2 && PH == 1)) // sweeps A+B at d = 64 take one row block a wave
        if (d == 64)
            return p.causal ? launch_mode<64, RB, KT, true, PH>(p, idx_mode, st) : launch_mode<64, RB, KT, false, PH>(p, idx_mode, st);
    if (d == 128)
        return p.causal ? launch_mode<128, RB, KT, true, PH>(p, idx_mode, st) : launch_mode<128, RB, KT, false, PH>(p, idx_mode, st);
    return (int)hipErrorInvalidValue;
}

} // namespace fwdk

} // namespace intattn
