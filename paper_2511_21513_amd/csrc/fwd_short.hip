// Fused IntAttention forward for short key sequences (at most 256 keys, d = 64: image encoders, short prompts) on gfx950
// (MI355X), where throughput counts (fwd_short_serves): one workgroup per (batch, query head) and 128 query rows, a wave per
// 32 rows.
//
// All scores of a wave's rows fit its registers (16 per 32 keys), so Q.K^T is computed once and the three reductions of
// IndexSoftmax (Sec. 3.1-3.2) run on registers: the score becomes its table index, then its probability, in place.  K and
// V of the head are staged in LDS once; a barrier when they are, and one when K is read where its room is used again.  What bounds it is vector
// instructions per score: against the tiled kernel it saves two of three score computations and one of two index
// computations, and pads rows and keys to 32 only (197 x 197: 224 x 224 scores instead of 256 x 256).  Measured against
// them as they were: 128 x 12 heads of 197 x 197 75.1 -> 46.2 us, 256 x 32 heads of 64 x 64 98 -> 47, 128 x 12 heads of
// 256 x 256 under the mask 78 -> 46.7.  Workgroups of up to eight waves, a whole head each, took 60.5 us on the first: 148
// to 167 registers (five to eight sub-tiles; 103 up to four) leave a compute unit 12 waves, so only one workgroup of
// seven.
//
// Hidden keys take the last table index, whose entry is 0 by Eq. lut16: no part in the sum, probability 0.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernel_common.h"
#include "params.h"

namespace intattn {

namespace {

constexpr int D = 64;
constexpr int MAX_WAVES = 4; // 12 waves fit a compute unit: three workgroups of four, but only one of seven
constexpr int KB = D / 32, CB = D / 32;
[[maybe_unused]] constexpr int CPR = D / 16; // 16-byte chunks per key row
constexpr int RPB = 1024 / D; // key rows per 1 KiB block

// NS: 32-key sub-tiles held (Lk <= 32 NS).  MODE: IDX_FMA, or IDX_DEVICE where every head has its own of IDX_FMA and IDX_FP64.
template <int NS, bool CAUSAL, bool BY_BYTE, int MODE>
__global__ __launch_bounds__(MAX_WAVES * 64, 2) void fwd_short_kernel(const FwdParams p)
{
    __shared__ __attribute__((aligned(1024))) int8_t Ks[NS * 32 * D];
    __shared__ __attribute__((aligned(1024))) int8_t Vs[NS * 32 * D];
    // Tables by place.  BY_BYTE: a row of 256 bytes for each place; lane l of wave w reads byte 4 l + w, so the address is the
    // conversion of the index map put into byte 1 of 4 l + w, with no instruction of its own, and no two lanes of a wave share
    // a bank.  Else LUT_hat by byte and words [place][row], a table for each wave.  The first takes 8 KiB more of LDS where a
    // workgroup has two waves, and a longer fill: 128 x 12 heads of 197 x 197 47.5 us against 48.5, but 256 x 32 heads of 64 x 64
    // 59.4 against 44.5, and at 128 keys they are even (25.8, 26.1), so it serves more than 128
    // keys, in workgroups of four waves, where the LDS is the same.
    __shared__ __attribute__((aligned(256))) uint8_t LT[BY_BYTE ? 32 * 256 : 32];  // LUT_hat
    __shared__ __attribute__((aligned(256))) uint8_t PT[BY_BYTE ? 32 * 256 : 256]; // the probabilities of the lane's row (BY_BYTE)
    extern __shared__ __attribute__((aligned(16))) uint32_t PT_words[];            // else: 32 x 32 words a wave; then its output rows

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, n = lane & 31, h = lane >> 5;
    [[maybe_unused]] const int n_waves = __builtin_amdgcn_readfirstlane((int)blockDim.x >> 6);
    const WorkItem wi = fwd_work_item(p, (int)blockIdx.x);
    if (!wi.valid) return; // padding of the XCD-aware grid (uniform for the whole workgroup)
    const int b = wi.b, hq = wi.hq, kvh = wi.kvh, bh = b * p.Hq + hq;
    const HeadParams hp = p.hp_table ? p.hp_table[hq] : p.hp0;
    const int L = p.Lk, LQ = p.L;
    const uint32_t top = (uint32_t)p.top;
    const int l0 = (wi.qt * MAX_WAVES + wave) * 32, lr = l0 + n; // the lane's row of Q
    const int row = p.row_lo + lr;                               // it sees keys <= row under the causal mask
    const bool row_ok = lr < LQ;
    const int8_t *Qp = p.q + (int64_t)b * p.qs[0] + (int64_t)hq * p.qs[1];

    // K and V straight into LDS; the XOR swizzle is applied to the global address, rows at or past L arrive as zeros from the
    // range check of the buffer descriptor
    auto stage = [&](const int8_t *base, int64_t stride, int8_t *dst, int first, bool is_v) __attribute__((always_inline)) {
        const int64_t bytes = (int64_t)(L - 1) * stride + D; // below 2^32: L <= 256, stride <= 2^24
        const int nblk = ((L + 31) / 32) * 32 / RPB;
#if defined(__HIP_DEVICE_COMPILE__) // the host pass has neither the descriptor type nor the builtins
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)(uint32_t)bytes, 0x00020000);
        for (int blk = first; blk < nblk; blk += n_waves) {
            const int key = blk * RPB + lane / CPR, cpos = lane % CPR;
            const int swz = is_v ? swz_v<D>(key) : swz_k<D>(key);
            const int goff = (int)((uint32_t)key * (uint32_t)stride + (uint32_t)((cpos ^ swz) << 4));
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(dst + blk * 1024), 16, goff, 0, 0, 0);
        }
#else
        (void)base, (void)bytes, (void)nblk, (void)dst, (void)first, (void)is_v;
#endif
    };
    stage(p.k + (int64_t)b * p.ks[0] + (int64_t)kvh * p.ks[1], p.ks[2], Ks, wave, false);
    stage(p.v + (int64_t)b * p.vs[0] + (int64_t)kvh * p.vs[1], p.vs[2], Vs, wave, true);
    // LUT_hat by place (see ScoreIndex)
    if constexpr (!BY_BYTE) {
        if (tid < 32) {
            const int idx = ScoreIndex<IDX_FMA>::place(tid, (int)top);
            LT[tid] = idx >= 0 ? (uint8_t)(p.lut[idx / 4] >> (8 * (idx % 4))) : (uint8_t)0;
        }
    }
    for (int t = tid; BY_BYTE && t < 256; t += 64 * n_waves) { // 32 bytes of a row each
        const int idx = ScoreIndex<IDX_FMA>::place(t >> 3, (int)top);
        const int v = (int)((idx >= 0 ? (p.lut[idx / 4] >> (8 * (idx % 4))) & 0xffu : 0u) * 0x01010101u);
        *(v4i *)(LT + t * 32) = v4i{v, v, v, v};
        *(v4i *)(LT + t * 32 + 16) = v4i{v, v, v, v};
    }
    v4i qf[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        qf[kb] = v4i{0, 0, 0, 0};
        if (row_ok) qf[kb] = *(const v4i *)(Qp + (int64_t)lr * p.qs[2] + kb * 32 + h * 16);
    }
    publish_tiles_barrier();

    // wave-uniform: sub-tiles that hold keys some row of the wave sees, and whether every row sees all of a sub-tile
    const int kmax = l0 >= LQ ? 0 : (CAUSAL ? min(L, p.row_lo + l0 + 32) : L);
    auto live = [&](int st) { return 32 * st < kmax; };
    auto full = [&](int st) { return 32 * st + 32 <= L && (!CAUSAL || 32 * st + 31 <= p.row_lo + l0); };
    auto visible = [&](int key) { return key < L && (!CAUSAL || key <= row); };

    // ---- scores and row max
    v16i s[NS];
    int mx = INT32_MIN;
#pragma unroll
    for (int st = 0; st < NS; ++st) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[st][i] = 0;
        if (!live(st)) continue;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int key = 32 * st + n;
            const v4i kf = *(const v4i *)(Ks + key * D + (((2 * kb + h) ^ swz_k<D>(key)) << 4));
            s[st] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf, qf[kb], s[st], 0, 0, 0);
        }
    }
    if constexpr (BY_BYTE) __syncthreads(); // K is read: the waves' output rows take its place
    if (l0 >= LQ) return;                   // no barrier below
#pragma unroll
    for (int st = 0; st < NS; ++st) {
        if (!live(st)) continue;
        if (full(st)) {
#pragma unroll
            for (int i = 0; i < 16; i += 2) mx = max(max(s[st][i], s[st][i + 1]), mx);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = visible(32 * st + acc_key(i, h)) ? max(mx, s[st][i]) : mx;
        }
    }
    mx = max(mx, __shfl_xor(mx, 32));
    if (!row_ok) mx = 0; // rows outside the problem: zero scores, never stored

    // ---- table places and row sum; the row maximum is known only now, so the start value is added here
    const int last = CAUSAL ? min(L - 1, row) : L - 1; // last key the lane's row sees
    const uint32_t own = (uint32_t)(4 * lane + wave); // the lane's byte of a table row
    uint32_t *PTw = PT_words + wave * 1024;
    uint32_t sum = 0;
    auto places = [&](auto mode_tag) __attribute__((always_inline)) {
        constexpr int M = decltype(mode_tag)::value;
        ScoreIndex<M> si;
        si.init(hp, mx, top);
        // (in double four scores at a time: sixteen hold 16 registers more, and 182 at 256 keys leave a SIMD two waves instead of three)
        auto pause = [&](int i) __attribute__((always_inline)) {
            if (M != IDX_FMA && i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        };
        auto place = [&](int sc) __attribute__((always_inline)) { return (int)(BY_BYTE ? si.address(sc, own) : si.index(sc)); };
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            if (!live(st)) continue;
            if (full(st)) {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[st][i] = place(s[st][i] + si.start()), pause(i);
            } else {
                const int lim = last - 32 * st - 4 * h;
#pragma unroll
                for (int i = 0; i < 16; ++i) s[st][i] = place(acc_key(i, 0) <= lim ? s[st][i] + si.start() : si.hidden()), pause(i);
            }
            uint32_t e[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) e[i] = LT[(uint32_t)s[st][i]];
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += e[i];
        }
    };
    if (MODE == IDX_FMA || hp.fma_r != 0) places(std::integral_constant<int, IDX_FMA>{}); // uniform for the workgroup
    else places(std::integral_constant<int, IDX_FP64>{});
    sum += __shfl_xor(sum, 32);
    const bool big = __any(row_ok && sum <= BIG_ROW_SUM); // wave-uniform
    if (!row_ok) sum = 1u << 24;                          // rows outside the problem: all probabilities 0
    if (h == 0 && row_ok) {
        if (p.dbg_row_max) p.dbg_row_max[(int64_t)bh * LQ + lr] = mx;
        if (p.dbg_row_sum) p.dbg_row_sum[(int64_t)bh * LQ + lr] = (int32_t)sum;
    }

    // ---- the row's probabilities (Eq. uint8-prob) by place; the LDS executes one wave's instructions in order
    // Where a probability may exceed 127 (BIG_ROW_SUM) the wave feeds P - 128 and takes the column sums of V from an operand of
    // all ones.  (Rows this short mostly have a key of that size in every sub-tile or none at all, so taking the top bits
    // apart as add_pv does costs more here: 128 x 12 heads of 197 x 197 with outlier channels 50.3 us.)
    const uint32_t flip = big ? 0x80u : 0u;
    const float inv_2s = __builtin_amdgcn_rcpf((float)(2u * sum));
#pragma unroll 4
    for (int j = 0; j < 16; ++j) {
        const uint32_t pl = (uint32_t)(16 * h + j), row = BY_BYTE ? pl << 8 : pl;
        const uint32_t pr = prob_u8(LT[row], sum, inv_2s) ^ flip; // LUT_hat is 0 past the table
        if constexpr (BY_BYTE) { // half the places each: for this lane and for the other one of its row
            PT[row + own] = (uint8_t)pr;
            PT[row + (own ^ 128u)] = (uint8_t)pr;
        } else {
            PTw[row * 32 + n] = pr;
        }
    }
    v4i pf[NS];
#pragma unroll
    for (int st = 0; st < NS; ++st) {
        pf[st] = v4i{0, 0, 0, 0};
        if (!live(st)) continue;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[st][i] = BY_BYTE ? (int)PT[(uint32_t)s[st][i]] : (int)PTw[s[st][i] * 32 + n];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            pf[st][g] = (int)((((uint32_t)s[st][4 * g + 1] << 8) | (uint32_t)s[st][4 * g]) |
                              ((((uint32_t)s[st][4 * g + 3] << 8) | (uint32_t)s[st][4 * g + 2]) << 16));
    }

    // ---- P_hat.V_hat
    const int tr_i = lane & 15, tr_g = (lane >> 4) & 1, jj = tr_i >> 1;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    v16i o[CB], ocs[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[cb][i] = 0, ocs[cb][i] = 0;
#pragma unroll
    for (int st = 0; st < NS; ++st) {
        if (!live(st)) continue;
        v4i vf[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int key = 32 * st + 8 * (2 * r + (jj >> 2)) + 4 * h + (jj & 3);
                const int8_t *ptr = Vs + key * D + (((2 * cb + tr_g) ^ swz_v<D>(key)) << 4) + 8 * (tr_i & 1);
                const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3))) *)ptr);
                vf[cb][2 * r] = x[0];
                vf[cb][2 * r + 1] = x[1];
            }
        }
        add_pv<false>(vf, pf[st], o);
        if (big) add_pv<false>(vf, ones, ocs);
    }

    // ---- requantize (Sec. 3.2); the wave's 32 rows of 64 bytes meet in what held K or its table, so that stores are 16 bytes a lane.
    // Bits 2 and 3 of a word's number are XORed with bits 2 and 3 of the row's, which spreads the rows over the banks.
    uint32_t *rows = BY_BYTE ? (uint32_t *)Ks + wave * 512 : PTw;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int ch0 = cb * 32 + 8 * g + 4 * h;
            uint32_t packed = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t acc = o[cb][4 * g + r] + 128 * ocs[cb][4 * g + r];
                if (p.dbg_acc && row_ok) p.dbg_acc[((int64_t)bh * LQ + lr) * D + ch0 + r] = acc;
                packed |= ((uint32_t)requant_any(acc, hp.rq_mult, hp.rq_shift) & 0xffu) << (8 * r);
            }
            rows[n * 16 + ((ch0 / 4) ^ (((n >> 2) & 3) << 2))] = packed;
        }
    }
    int8_t *Op = p.out + (int64_t)b * p.os[0] + (int64_t)hq * p.os[1];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int r = q * 16 + lane / 4, c = lane % 4;
        const v4i x = *(const v4i *)(rows + r * 16 + 4 * (c ^ ((r >> 2) & 3)));
        if (l0 + r < LQ) *(v4i *)(Op + (int64_t)(l0 + r) * p.os[2] + c * 16) = x;
    }
}

template <int NS, bool CAUSAL, int MODE>
int launch_mode(const FwdParams &p_in, hipStream_t st)
{
    FwdParams p = p_in;
    const int waves = p.L >= MAX_WAVES * 32 ? MAX_WAVES : (p.L + 31) / 32;
    const dim3 grid((unsigned)fwd_map_work(p)), block((unsigned)(64 * waves));
    if constexpr (NS > 4) {
        if (waves == MAX_WAVES) { // see BY_BYTE
            hipLaunchKernelGGL((fwd_short_kernel<NS, CAUSAL, true, MODE>), grid, block, 0, st, p);
            return (int)hipGetLastError();
        }
    }
    hipLaunchKernelGGL((fwd_short_kernel<NS, CAUSAL, false, MODE>), grid, block, (unsigned)waves * 4096u, st, p);
    return (int)hipGetLastError();
}

template <int NS, bool CAUSAL>
int launch_shape(const FwdParams &p, int idx_mode, hipStream_t st)
{
    return idx_mode == IDX_FMA ? launch_mode<NS, CAUSAL, IDX_FMA>(p, st) : launch_mode<NS, CAUSAL, IDX_DEVICE>(p, st);
}

} // namespace

// d = 64, Lk <= 256, tables of at most 32 entries, host scales, parameters per
// tensor or per head; p.n_qtiles counts tiles of 128 query rows from row 0; no workspace.
int launch_fwd_short(const FwdParams &p, int d, int idx_mode, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (d != D || p.Lk > 256 || p.top > 31 || (idx_mode != IDX_FMA && idx_mode != IDX_FP64 && idx_mode != IDX_DEVICE))
        return (int)hipErrorInvalidValue;
    if (p.Lk <= 128) return p.causal ? launch_shape<4, true>(p, idx_mode, st) : launch_shape<4, false>(p, idx_mode, st);
    if (p.Lk <= 224) return p.causal ? launch_shape<7, true>(p, idx_mode, st) : launch_shape<7, false>(p, idx_mode, st);
    return p.causal ? launch_shape<8, true>(p, idx_mode, st) : launch_shape<8, false>(p, idx_mode, st);
}

} // namespace intattn
