// Sweep C of the IntAttention forward as a kernel of its own (gfx950): with the row maxima and row
// sums of E_hat already in a workspace, recompute the INT8 scores, map them through the index
// map and the per-row probability table (Sec. 3.1-3.2: P_hat = round(255 E_hat / S)), multiply
// by V_hat on the matrix cores and requantize (INT8 output).
//
// Same data layout and lane ownership as the generic forward kernel (transposed scores, one query
// row per lane, XOR-swizzled K/V tiles in LDS filled by direct global->LDS loads); a wave owns 32
// query rows and takes the keys in steps of 32: scores, table entries, packing, P.V, each phase whole
// before the next, with the K fragments of the next step requested ahead of P.V.
//
// What bounds it (c = 4-byte LDS bank clocks of a compute unit, per 32 x 32 block of scores and wave, d = 128): the LDS
// pipe serves sixteen table lookups (34 clocks), four K and eight V^T fragment reads (33) and the tile loads (16), 83 in all
// or 330 for the four SIMDs that share it; the matrix cores need 256 cycles of a SIMD, the vector ALU 44 instructions or
// about 250.  No two of them overlap fully, so few instructions and many waves count: with the IDX_FMA map a score costs
// two vector instructions, its share of the packing and one lookup, and the kernel fits three waves a SIMD (168
// registers), four at d = 64, in place of two (232).  Measured against the kernel before it, which held a software pipeline
// inside a wave and tables in registers (1 x 8192, 32 / 8 heads, d 128): 317 -> 267 to 277 us with the card; 16 x 4096, 32 heads, a scale for each
// head: 1545 -> 1162; without a mask, 2 x 2048: 102 -> 84; d 64, 4 x 4096, 16 heads: 121 -> 98.  With this map the pipeline
// takes as long as the phases (271 us at two waves; three spill), tiles of 128 keys or workgroups of six or eight waves
// longer (448, 315).
//
// Tiles are two sub-tiles (64 keys), double buffered per operand; one barrier per tile.  K tiles are cut one sub-tile
// earlier than V tiles (K tile t covers sub-tiles [2 t - 1, 2 t + 1)), so that iteration T reads exactly K tile T + 1 and
// V tile T, and at its top requests K tile T + 2 and V tile T + 1 into the buffers that were read an iteration ago.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace sweepc {

constexpr int WAVES = 4;
constexpr int NT = WAVES * 64;

// SPLIT: every work item is taken by p.split_c workgroups, each with a range of the key tiles.  (An instantiation of its own:
// with the range decided at run time the launches that do not split were 1 % slower.)
template <int D, bool CAUSAL, int MODE, bool SPLIT>
__global__ __launch_bounds__(NT, D == 128 ? 3 : 4) void sweep_c_kernel(const FwdParams p)
{
    constexpr int KB = D / 32;       // 32-wide blocks of the head dimension
    constexpr int CB = D / 32;       // 32-wide blocks of output channels
    constexpr int NSUB = 2;          // 32-key sub-tiles (steps) per tile
    constexpr int BK = 32 * NSUB;    // keys per tile
    constexpr int BQ = WAVES * 32;   // query rows of the workgroup
    constexpr int TILE = BK * D;     // bytes
    constexpr int SUB = 32 * D;      // bytes of a 32-key sub-tile
    constexpr int NBLK = TILE / 1024;
    constexpr int JB = NBLK / WAVES;
    constexpr int CPR = D / 16;
    constexpr int RPB = 1024 / D;
    static_assert(NBLK % WAVES == 0, "every wave requests the same number of blocks");

    __shared__ __attribute__((aligned(1024))) int8_t Ks0[TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Ks1[TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Vs0[TILE];
    __shared__ __attribute__((aligned(1024))) int8_t Vs1[TILE];
    // per-row probability tables of the workgroup as bytes [place of the index][lane][wave]: a table row (one index) is 256
    // bytes, lane l of wave w owns byte 4 l + w of every row -- its own bank, so lookups never conflict.  The address of an
    // entry is (index << 8) + 4 l + w (aligned to 64 KiB: byte 1 of the address is the index alone).  The two lanes that
    // share a query row (l and l + 32) each hold a copy of its table.
    __shared__ __attribute__((aligned(65536))) uint8_t PT[32 * 256];
    __shared__ uint32_t lut_lds[8];

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 31, h = lane >> 5;
    int bid = (int)blockIdx.x;
    const int n_split = SPLIT ? p.split_c : 1;
    const int ksp = SPLIT ? fwd_split_index(bid, n_split) : 0;
    const WorkItem wi = fwd_work_item(p, bid);
    if (!wi.valid) return; // padding of the XCD-aware grid (uniform for the whole workgroup)
    const int b = wi.b, hq = wi.hq, kvh = wi.kvh, qt = wi.qt + p.row_lo / BQ;
    const int bh = b * p.Hq + hq;
    const HeadParams hp = p.hp_table ? p.hp_table[hq] : p.hp0;
    // The rest of the kernel with the index scheme M as a compile-time constant: MODE itself, or, under IDX_DEVICE, the
    // scheme that the parameters derived on the device allow.
    auto body = [&](auto mode_tag) __attribute__((always_inline)) {
    constexpr int M = decltype(mode_tag)::value;
    const int L = p.Lk; // keys
    // query rows: [rlo, rhi) of the numbering in which row r sees keys <= r under the causal mask
    const int rlo = p.row_lo, rhi = p.row_lo + p.L, LQ = p.L;
    // parameters of the block of query rows that `row` lies in (finer groups over query rows, Sec. 3.3)
    auto row_hp = [&](int row) __attribute__((always_inline)) {
        const int lr = (row >= rlo && row < rhi) ? row - rlo : 0;
        return p.row_table[(int64_t)bh * p.n_rowblk + lr / p.q_block];
    };
    const uint32_t top = (uint32_t)p.top;

    const int q0 = qt * BQ;
    const int8_t *Qp = p.q + (int64_t)b * p.qs[0] + (int64_t)hq * p.qs[1];
    const int8_t *Kp = p.k + (int64_t)b * p.ks[0] + (int64_t)kvh * p.ks[1];
    const int8_t *Vp = p.v + (int64_t)b * p.vs[0] + (int64_t)kvh * p.vs[1];

    if (tid < 8) lut_lds[tid] = p.lut[tid];

    const int kmax = CAUSAL ? min(L, q0 + BQ) : L;
    // iterations = V tiles [tlo, thi); K tiles tlo..thi are touched.  Key-split launches take a range of the tiles each and
    // leave partial accumulators; otherwise the range is all of them.
    const int tall = (kmax + BK - 1) / BK;
    const int tlo = tall * ksp / n_split, thi = tall * (ksp + 1) / n_split;

    // ---- staging: direct global -> LDS loads; the XOR swizzle is applied to the global address
    // (lane i of a wave-wide 16-byte load lands at byte 16 i of its 1 KiB block).
    int dma_goff_k[JB], dma_goff_v[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        const int key = (wave + WAVES * j) * RPB + lane / CPR, cp = lane % CPR;
        dma_goff_k[j] = key * (int)p.ks[2] + ((cp ^ swz_k<D>(key)) << 4); // the host checked BK * stride < 2^31
        dma_goff_v[j] = key * (int)p.vs[2] + ((cp ^ swz_v<D>(key)) << 4);
    }
    // The loads go through a buffer descriptor that starts at the tile's first key row and ends
    // with the last byte of key row L-1, so key rows at or past L come back as zeros from the range
    // check.  Blocks below first_blk are skipped (the part of K tile 0 that lies before key 0).
    auto dma_tile = [&](const int8_t *base, int64_t stride, const int (&goff)[JB], int key0, int first_blk, int8_t *dst)
                        __attribute__((always_inline)) {
        const int8_t *tb = base + (int64_t)key0 * stride; // wave-uniform
        const int64_t rem = (int64_t)(L - key0 - 1) * stride + D;
        const uint32_t nrec = rem <= 0 ? 0u : (rem > 0xffffffffll ? 0xffffffffu : (uint32_t)rem); // 0: all of it past L
#if defined(__HIP_DEVICE_COMPILE__) // the host pass has neither the descriptor type nor the builtins
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)tb, 0, (int)nrec, 0x00020000);
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int blk = wave + WAVES * j;
            if (blk < first_blk) continue; // wave-uniform
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(dst + blk * 1024), 16,
                                                     goff[j], 0, 0, 0);
        }
#else
        (void)tb, (void)nrec, (void)goff, (void)dst, (void)first_blk;
#endif
    };
    // K tile t starts one sub-tile before V tile t; the rows of K tile 0 that would lie before key 0 are not requested
    auto dma_k = [&](int t, int8_t *dst) __attribute__((always_inline)) {
        const int key0 = (t * NSUB - 1) * 32;
        dma_tile(Kp, p.ks[2], dma_goff_k, key0, key0 < 0 ? -key0 / RPB : 0, dst);
    };
    auto dma_v = [&](int t, int8_t *dst) __attribute__((always_inline)) { dma_tile(Vp, p.vs[2], dma_goff_v, t * BK, 0, dst); };

    if (tlo < thi) { // (a range of a key-split launch may be empty)
        dma_k(tlo, Ks0);
        dma_v(tlo, Vs0);
        dma_k(tlo + 1, Ks1);
    }

    const int qw0 = q0 + 32 * wave;
    const int row = qw0 + n; // this lane's query row
    const bool valid = row >= rlo && row < rhi;

    // Q fragments: row `row`, bytes [32 kb + 16 h, +16)
    v4i qf[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        qf[kb] = v4i{0, 0, 0, 0};
        if (valid) qf[kb] = *(const v4i *)(Qp + (int64_t)(row - rlo) * p.qs[2] + kb * 32 + h * 16);
    }

    // ---- per-row state from the first launch
    const HeadParams hrow = M == IDX_ROW64 ? row_hp(row) : hp;
    const int mx = valid ? p.ws_row_max[(int64_t)bh * LQ + (row - rlo)] : 0;
    uint32_t sum = valid ? (uint32_t)p.ws_row_sum[(int64_t)bh * LQ + (row - rlo)] : 0u;
    const bool big = __any(valid && sum <= BIG_ROW_SUM); // of any of the wave's rows: wave-uniform
    if (!valid) sum = 1u << 24;                          // rows outside [rlo, rhi): all probabilities 0, never stored
    if (p.dbg_row_max && h == 0 && valid) p.dbg_row_max[(int64_t)bh * LQ + (row - rlo)] = mx;
    if (p.dbg_row_sum && h == 0 && valid) p.dbg_row_sum[(int64_t)bh * LQ + (row - rlo)] = (int32_t)sum;
    ScoreIndex<M> si;
    si.init(hrow, mx, top);

    publish_tiles_barrier(); // LUT_hat, K tiles tlo and tlo + 1, V tile tlo are in LDS

    // per-row probability table: the byte at the place of idx is round(255 * LUT_hat[idx] / sum); each lane of a row's pair
    // computes half of the entries and stores them into both lanes' columns
    const uint32_t lane_base = (uint32_t)(4 * lane + wave);
    {
        const uint8_t *lut_b = (const uint8_t *)lut_lds;
        const float inv_2s = __builtin_amdgcn_rcpf((float)(2u * sum));
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int kidx = 16 * h + j, at = ScoreIndex<M>::place(kidx, (int)top) & 31; // entries past the table go to rows nothing reads
            const uint8_t byte = (uint8_t)prob_u8(lut_b[kidx], sum, inv_2s);
            PT[at * 256 + 4 * n + wave] = byte;
            PT[at * 256 + 4 * (n + 32) + wave] = byte;
        }
    }

    // ---- LDS read addresses (lane constants; sub-tile and buffer go into immediate offsets)
    int kf_off[KB], vf_off[CB];
    {
        const int sw = swz_k<D>(n); // equal for keys n and n + 32
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) kf_off[kb] = n * D + (((2 * kb + h) ^ sw) << 4);
        // transposing read: lanes 2j, 2j+1 of a 16-lane group point at the two 8-byte halves of key
        // row j's 16 channels; lane i of the group receives channel i of the eight rows.
        const int tr_i = lane & 15, tr_g = (lane >> 4) & 1, jj = tr_i >> 1;
        const int key = 8 * (jj >> 2) + 4 * h + (jj & 3); // + 16 for the second half of the operand
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) vf_off[cb] = key * D + (((2 * cb + tr_g) ^ swz_v<D>(key)) << 4) + 8 * (tr_i & 1);
    }
    auto read_kf = [&](const int8_t *Ksub, v4i (&kf)[KB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) kf[kb] = *(const v4i *)(Ksub + kf_off[kb]);
    };
    auto read_vf = [&](const int8_t *Vsub, v4i (&vf)[CB]) __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const v2i x0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3))) *)(Vsub + vf_off[cb]));
            const v2i x1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3))) *)(Vsub + vf_off[cb] + 16 * D));
            vf[cb] = v4i{x0[0], x0[1], x1[0], x1[1]};
        }
    };

    v16i o[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cb][i] = 0;
    v16i s0; // what the scores are added to
#pragma unroll
    for (int i = 0; i < 16; ++i) s0[i] = si.start();
    v4i kf[KB], vf[CB], pf;

    const int last = CAUSAL ? min(L - 1, row) : L - 1; // last key the lane's row sees
    // One step = sub-tile j: kf holds its K fragments and receives those of the next one.
    auto step = [&](auto masked_tag, auto big_tag, int j, const int8_t *Knext, const int8_t *Vcur) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        // no row of the wave sees a key of it, nor of any later one (wave-uniform)
        if (MASKED && (32 * j >= L || (CAUSAL && 32 * j > qw0 + 31))) return;
        v16i s = s0;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[kb], qf[kb], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        read_vf(Vcur, vf);
        __builtin_amdgcn_sched_barrier(0);
        const int lim = last - 32 * j - 4 * h;
        uint32_t l[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int sc = !MASKED || acc_key(i, 0) <= lim ? s[i] : si.hidden();
            l[i] = PT[si.address(sc, lane_base)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint32_t a = __builtin_amdgcn_perm(l[4 * g + 1], l[4 * g], 0x0c0c0400u);
            const uint32_t c = __builtin_amdgcn_perm(l[4 * g + 3], l[4 * g + 2], 0x0c0c0400u);
            pf[g] = (int)__builtin_amdgcn_perm(c, a, 0x05040100u);
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr bool BIG = decltype(big_tag)::value;
        if (!BIG) read_kf(Knext, kf); // (ahead of P.V, which hides the latency; with BIG there are no registers for it)
        __builtin_amdgcn_sched_barrier(0);
        add_pv<BIG>(vf, pf, o);
        __builtin_amdgcn_sched_barrier(0);
        if (BIG) read_kf(Knext, kf);
        __builtin_amdgcn_sched_barrier(0);
    };
    // One iteration = V tile T and K tile T + 1.  With PAR = (T - tlo) & 1: K tile T + 2 replaces K tile T (read an
    // iteration ago) in Ks[PAR], V tile T + 1 replaces V tile T - 1 in Vs[PAR ^ 1].
    auto iteration = [&](auto masked_tag, auto big_tag, int T, int8_t *Kdma, int8_t *Vdma, const int8_t *Krd, const int8_t *Vrd)
                         __attribute__((always_inline)) {
        if (T + 2 <= thi) dma_k(T + 2, Kdma);
        if (T + 1 < thi) dma_v(T + 1, Vdma);
#pragma unroll
        for (int u = 0; u < NSUB; ++u) step(masked_tag, big_tag, NSUB * T + u, Krd + u * SUB, Vrd + u * SUB);
        publish_tiles_barrier(); // K tile T + 2 and V tile T + 1 have landed; every wave is done with tile T
    };

    read_kf(Ks0 + SUB, kf);
    __syncthreads(); // every wave has read K tile tlo before iteration tlo overwrites it with K tile tlo + 2

    // Iterations whose sub-tiles are all fully visible to this wave need no masks (wave-uniform
    // count).  They run in pairs in a loop of their own, every buffer named statically (the compiler
    // then knows which direct-to-LDS load a fragment read depends on) and no branch inside the body;
    // the few remaining iterations take the masked code with the buffers chosen at run time.
    // Every wave of the workgroup passes the same number of barriers: one per iteration, thi - tlo in all.
    const int nfull_sub = CAUSAL ? min(L / 32, (qw0 + 1) / 32) : L / 32;
    const int nhot = min(nfull_sub / NSUB, thi);
    int T = tlo;
    auto hot = [&](auto big_tag) __attribute__((always_inline)) {
#pragma unroll 1
        for (; T + 2 <= nhot; T += 2) {
            iteration(std::false_type{}, big_tag, T, Ks0, Vs1, Ks1, Vs0);
            iteration(std::false_type{}, big_tag, T + 1, Ks1, Vs0, Ks0, Vs1);
        }
    };
    if (big) hot(std::true_type{});
    else hot(std::false_type{});
#pragma unroll 1
    for (; T < thi; ++T) {
        const bool odd = (T - tlo) & 1;
        iteration(std::true_type{}, std::true_type{}, T, odd ? Ks1 : Ks0, odd ? Vs0 : Vs1, odd ? Ks0 : Ks1, odd ? Vs1 : Vs0);
    }

    // Key-split launch: the accumulators of this range, for finish_split_kernel to add up
    if constexpr (SPLIT) {
        if (valid) {
            int32_t *Pp = p.ws_part + ((int64_t)ksp * p.B * p.Hq * LQ + (int64_t)bh * LQ + (row - rlo)) * D;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int ch0 = cb * 32 + 8 * g + 4 * h;
                    v4i a;
#pragma unroll
                    for (int r = 0; r < 4; ++r) a[r] = o[cb][4 * g + r];
                    *(v4i *)(Pp + ch0) = a;
                }
            }
        }
        return;
    }
    // ================================================================= epilogue (Sec. 3.2: requantization)
    // (instantiated for the shift range and for the debug tap, so that the 64 values of a lane meet no branch)
    auto epilogue = [&](auto fast_tag, auto dbg_tag) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(fast_tag)::value, DBG = decltype(dbg_tag)::value;
        int8_t *Op = p.out + (int64_t)b * p.os[0] + (int64_t)hq * p.os[1] + (int64_t)(row - rlo) * p.os[2];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int ch0 = cb * 32 + 8 * g + 4 * h;
                uint32_t packed = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t acc = o[cb][4 * g + r];
                    if (DBG) p.dbg_acc[((int64_t)bh * LQ + (row - rlo)) * D + ch0 + r] = acc;
                    packed |= ((uint32_t)requant<FAST>(acc, hrow.rq_mult, hrow.rq_shift) & 0xffu) << (8 * r);
                }
                *(uint32_t *)(Op + ch0) = packed;
            }
        }
    };
    if (valid) {
        const bool fast = hrow.rq_shift >= 33;
        if (p.dbg_acc) {
            if (fast) epilogue(std::true_type{}, std::true_type{});
            else epilogue(std::false_type{}, std::true_type{});
        } else {
            if (fast) epilogue(std::true_type{}, std::false_type{});
            else epilogue(std::false_type{}, std::false_type{});
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

template <int D, bool CAUSAL, bool SPLIT>
int launch_mode(const FwdParams &p_in, int idx_mode, hipStream_t st)
{
    FwdParams p = p_in;
    const dim3 grid((unsigned)fwd_map_work(p, SPLIT ? p.split_c : 1)), block(NT);
    if (idx_mode == IDX_FMA)
        hipLaunchKernelGGL((sweep_c_kernel<D, CAUSAL, IDX_FMA, SPLIT>), grid, block, 0, st, p);
    else if (idx_mode == IDX_DEVICE)
        hipLaunchKernelGGL((sweep_c_kernel<D, CAUSAL, IDX_DEVICE, SPLIT>), grid, block, 0, st, p);
    else if (idx_mode == IDX_ROW64)
        hipLaunchKernelGGL((sweep_c_kernel<D, CAUSAL, IDX_ROW64, SPLIT>), grid, block, 0, st, p);
    else
        hipLaunchKernelGGL((sweep_c_kernel<D, CAUSAL, IDX_FP64, SPLIT>), grid, block, 0, st, p);
    return (int)hipGetLastError();
}

// p.n_qtiles must count tiles of 128 query rows; p.ws_row_max / ws_row_sum filled.  Instantiated in a source of its own for each D and SPLIT.
template <int D, bool SPLIT>
int launch(const FwdParams &p, int idx_mode, hipStream_t st)
{
    return p.causal ? launch_mode<D, true, SPLIT>(p, idx_mode, st) : launch_mode<D, false, SPLIT>(p, idx_mode, st);
}

} // namespace sweepc

} // namespace intattn
