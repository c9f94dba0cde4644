// Device helpers shared by the forward kernels: vector types, the mapping of workgroups to work, the exact index map of Sec. 3.1,
// the MFMA accumulator-to-key map and the LDS chunk swizzles.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "params.h"
#include "work_map.h"

namespace intattn {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------ index map (Sec. 3.1)
// The fp64 scheme's factor -r (its bits are split over idx_mul, low word, and idx_add).
__device__ __forceinline__ double idx_fp64_factor(const HeadParams &hp)
{
    return __builtin_bit_cast(double, ((uint64_t)hp.idx_add << 32) | (uint64_t)hp.idx_mul);
}

// Key groups: the fp64 map applied to RAW scores of one query row (the lane's row), whose constants change from block to block
// of keys: idx = trunc(fma(-Delta', -r, 0.5)) in IEEE fp64, r the double after top/c_int: exact for every c_int.  Call with sc =
// min(max(s, bound), mx); the index is kept inside the table whatever an unusable scale produced.
struct RowIndex {
    int bound; // mx - c_int
    int mx;
    int top;   // 2^b - 1
    double negr;

    __device__ __forceinline__ uint32_t operator()(int sc) const
    {
        return min((uint32_t)(int)__builtin_fma((double)(sc - mx), negr, 0.5), (uint32_t)top);
    }
};

// The index map in single precision for parameters that a lane forms itself: trunc(fma(t, -r, 0.5)), t = -Delta' in
// [-c_int, 0], r the float after fl(top / c_int).  Exact where init() says so, without a search: r exceeds top / c_int by
// more than 0 and less than 3 * 2^-24 of it, so the exact value of the fma is at least v = -t top / c_int + 1/2 and above it
// by less than 3 top 2^-24; its rounding adds at most half a unit in the last place of a value below top + 1 (2^-20 for
// top <= 31, 2^-19 for 63) and is monotone, so an integer v stays on or above itself; any other v lies at least
// 1 / (2 c_int) below the next integer, which is more than the sum of both up to 76900 (top = 31) and 37900 (top = 63).
struct RowIndex32 {
    int mx;
    float negr;
    __device__ __forceinline__ bool init(int c_int, int row_max, uint32_t top)
    {
        mx = row_max;
        negr = -__uint_as_float(__float_as_uint((float)top / (float)c_int) + 1u); // one IEEE division
        return c_int <= (top < 32 ? 75000 : 37000);
    }
    __device__ __forceinline__ uint32_t operator()(int sc) const { return (uint32_t)(int)__builtin_fmaf((float)(sc - mx), negr, 0.5f); }
};

// The map of a score to its place in a table of 2^b entries, for kernels that start the score's MFMAs at start().  Places count
// entries from the end of the table (place = top - idx, 0 where a key is clipped or hidden), key groups apart, whose scores
// are mapped with RowIndex.
//
// IDX_FMA needs neither a clip nor a conversion of the score.  The accumulators of the score's MFMAs start at the bits of
// the float 2^23 + c_int - rowMax, so that a finished one, read as a float f, is 2^23 + x with x = c_int - Delta exactly
// where x >= 0, and below 2^23 where the distance Delta exceeds c_int (|score - rowMax| <= 2^22, c_int < 2^22).  One fma gives
// f r - 2^23 r = x r, rounded once (2^23 r is exact), and the conversion to a byte rounds it to the nearest integer and takes
// negative values to 0.  r is a float just below top / c_int, so that ties (top x / c_int = k + 1/2) go down, as
// top - round-half-up(top Delta / c_int) does; the host (find_fma) or the derivation kernel has proved it at both sides of
// every step.  Rounding and saturation of v_cvt_pk_u8_f32: nearest even, [0, 255].
//
// IDX_FP64 and IDX_ROW64 serve the thresholds c that have no such float, in double.  The accumulators start at c - rowMax, so
// that x = max(accumulator, 0), and one fma gives y = x r + 2^20 + 1/2: 32 bits of y are a fraction, and the low byte of its
// high word is the place, ceil(v) - 1 for v = top x / c + 1/2.  With r = (1 - e) top / c (to within 2^-51 of it) the sum
// before its rounding, which is by at most 2^-33, is v - (v - 1/2) e.  An integer v, a tie, has to land below itself:
// (v - 1/2) e > 2^-33.  Any other v lies at least 1 / (2 c) above the integer that it has to stay on or above: top e <= 1 / (2 c).
//   c <= 2^24: e = 2^-31; a tie's (v - 1/2) e >= 2^-32, and top e < 2^-25.
//   beyond, where no Delta passes 2^22, so that x >= 3/4 c or the key is hidden: e = 2^-31 / (top + 1); a tie has v - 1/2 >= 3/4 top,
//   its (v - 1/2) e >= 3/4 2^-32, and top e < 2^-31 <= 1 / (2 c).
// IDX_FP64 converts nothing: x is the low word of the double 2^52 + x, and 2^20 + 1/2 - 2^52 r is added, which is exact for r < 1.
// A head that it serves has c > top (find_fma finds a float for every smaller one).  IDX_ROW64, whose rows may have any c, converts x.
// (1 x 8192, 32 / 8 heads, d 128, whole calls: 683 us when a score took a clip, a subtraction, two conversions and the fma in double,
// 568 now with IDX_FP64, about 600 with IDX_ROW64's form; IDX_FMA 533, and 640 the fp32 map that served such thresholds before it.  2048
// rows, 16 heads, d 64: 31.9 -> 26.1, IDX_FMA 23.3, the fp32 map 29.9.  509 rows of 7001: 130 -> 112, IDX_FMA 105, the fp32 map 122.)
//
// LATE (in double only): the accumulators start at 0 and c - rowMax is added here, an instruction a score for 16 registers.
// SHIFTED (in double only): r and the addend are held 2^45 times as large, which moves the exponent alone.  The high word is then
// 0x44000000 + place, of which a shift by 7 leaves the place, so the address of an entry in a table with rows of 128 bytes is one
// shift-and-add and not four operations (128 x 12 heads of 197 rows, d 64, a scale for each 128 rows: 81.3 -> 74.7 us; IDX_FP64,
// device scales, 76.8 -> 70.1).  It takes IDX_FP64 two registers more, and kernels that these cost a wave a SIMD, or a spill, go without.
template <int MODE, bool LATE = false, bool SHIFTED = false> struct ScoreIndex {
    static constexpr bool FMA = MODE == IDX_FMA, KG = MODE == IDX_KGROUP;
    static constexpr uint32_t HIGH = SHIFTED ? 0x44000000u : 0x41300000u; // high word of 2^65, of 2^20
    static constexpr double UNIT = SHIFTED ? 35184372088832.0 : 1.0;      // 2^45
    RowIndex ri;
    float r, b;
    double r64, b64;
    int add0;
    // place of entry idx of the table, and the entry at a place (top = 2^b - 1)
    static __device__ __forceinline__ int place(int idx, int top) { return KG ? idx : top - idx; }
    __device__ __forceinline__ void init(const HeadParams &hp, int row_max, uint32_t top_)
    {
        if constexpr (FMA) {
            r = __uint_as_float(hp.fma_r);
            b = r * -8388608.0f;
            add0 = 0x4b000000 + hp.c_int - row_max;
        } else if constexpr (KG) {
            ri.top = (int)top_;
            add0 = 0;
        } else {
            const double q = -idx_fp64_factor(hp); // the double after top / c
            r64 = (q - __builtin_ldexp(q, hp.c_int <= (1 << 24) ? -31 : -31 - (int)__builtin_popcount(top_))) * UNIT;
            if constexpr (MODE == IDX_FP64) { // (a head's: uniform, and so kept in scalar registers)
                const uint64_t bits = __builtin_bit_cast(uint64_t, r64);
                r64 = __builtin_bit_cast(double, ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(bits >> 32)) << 32) |
                                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)bits));
            }
            b64 = 1048576.5 * UNIT - (MODE == IDX_FP64 ? 4503599627370496.0 * r64 : 0.0);
            add0 = hp.c_int - row_max;
        }
    }
    static constexpr bool ADD = LATE && !FMA && !KG;
    __device__ __forceinline__ int start() const { return ADD ? 0 : add0; } // of the score's accumulator
    __device__ __forceinline__ int hidden() const { return FMA ? 0 : -0x7f000000; } // the score of a hidden key (|c - rowMax| <= 2^30 + 2^21)
    __device__ __forceinline__ float steps(int sc) const { return __builtin_fmaf(__uint_as_float((uint32_t)sc), r, b); }
    __device__ __forceinline__ uint32_t steps64(int sc) const // HIGH + place
    {
        const int x = max(ADD ? sc + add0 : sc, 0);
        const double xd = MODE == IDX_FP64 ? __builtin_bit_cast(double, 0x4330000000000000ull | (uint64_t)(uint32_t)x) : (double)x;
        return (uint32_t)__builtin_bit_cast(v2i, __builtin_fma(xd, r64, b64))[1]; // (as a shift of 64 bits it would be joined with the address's)
    }
    __device__ __forceinline__ uint32_t index(int sc) const
    {
        if constexpr (FMA) return __builtin_amdgcn_cvt_pk_u8_f32(steps(sc), 0, 0);
        else return steps64(sc) - HIGH;
    }
    // Offset of the score's entry in a table whose rows (one per place) are 256 bytes apart; lane_base = the lane's offset
    // (< 256) inside a row: the conversion, or a byte permute, writes the place into byte 1.
    __device__ __forceinline__ uint32_t address(int sc, uint32_t lane_base) const
    {
        if constexpr (FMA) return __builtin_amdgcn_cvt_pk_u8_f32(steps(sc), 1, lane_base);
        else return __builtin_amdgcn_perm(steps64(sc), lane_base, 0x03020400u);
    }
};

// The map with the scheme named in the parameters themselves (pad[0]: chosen on the host, or by the derivation kernel for
// device-resident scales), for kernels where the map is not the hot loop: round(min(delta, c_int) * top / c_int) for
// 0 <= delta < 2^23.
struct AnyIndex {
    const HeadParams &hp;
    int c_int, add0, top;
    float r, b;
    bool fma;
    __device__ __forceinline__ AnyIndex(const HeadParams &hp_, int top_)
        : hp(hp_), c_int(hp_.c_int), add0(0x4b000000 + hp_.c_int), top(top_), r(__uint_as_float(hp_.fma_r)), b(r * -8388608.0f), fma(hp_.pad[0] == IDX_FMA)
    {
    }
    // with the fma map: top minus the index, into byte j of w
    __device__ __forceinline__ uint32_t place(int delta, int j, uint32_t w) const
    {
        return __builtin_amdgcn_cvt_pk_u8_f32(__builtin_fmaf(__uint_as_float((uint32_t)(add0 - delta)), r, b), j, w);
    }
    __device__ __forceinline__ uint32_t operator()(int delta) const
    {
        if (fma) return (uint32_t)top - place(delta, 0, 0);
        return (uint32_t)(int)__builtin_fma(-(double)min(delta, c_int), idx_fp64_factor(hp), 0.5);
    }
};

// The barrier that publishes tiles filled by direct-to-LDS loads: a wave's own loads must have landed before
// it signals, because the other waves read what it loaded.  (On this target the compiler also drains every
// counter before s_barrier; the wait is spelled out so that correctness does not rest on that.)
__device__ __forceinline__ void publish_tiles_barrier()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Key (within a 32-key block) held in accumulator register i of a 32x32 MFMA result by a
// lane of half-wave h; the same key sits in byte i of that lane's next B operand.
__device__ __forceinline__ int acc_key(int i, int h) { return 8 * (i >> 2) + 4 * h + (i & 3); }

// Eq. uint8-prob: round-half-up(255 E / S) = floor((510 E + S) / (2 S)) for E <= 255 and 1 <= S < 2^25, without an
// integer division: a single-precision estimate of the quotient (below 256, so off by one at most) corrected against
// the exact products.  inv_2s: the reciprocal of (float)(2 S) to within a few units in the last place (v_rcp_f32).
__device__ __forceinline__ uint32_t prob_u8(uint32_t e, uint32_t S, float inv_2s)
{
    const uint32_t num = 510u * e + S, den = 2u * S;
    uint32_t q = (uint32_t)((float)num * inv_2s);
    if (q * den > num) --q;
    if ((q + 1u) * den <= num) ++q;
    return q;
}

// ------------------------------------------------------------------ P_hat.V_hat (Sec. 3, Eq. pv-link)
// The int8 MFMA is signed x signed and P_hat unsigned.  P_hat = round(255 E / S) <= 127 wherever S > 510, so most rows feed
// their bytes as they are.  The probabilities of a row add up to 255 or little more, so in any other row one or two keys may
// have 128 or more.  The MFMA takes such a byte for P - 256, and where a sub-tile holds one, 256 = 2 + 127 + 127 in its
// place are multiplied by V as well.  (Before, P - 128 went in for every key, and 128 times the column sums of V were added back: a launch of their
// own, 4 to 5 us, or an MFMA more for each of P.V; and a masked key had to pass the matrix cores like any other.)
constexpr uint32_t BIG_ROW_SUM = 510; // a row sum up to which a probability may exceed 127

template <bool BIG, int CB> __device__ __forceinline__ void add_pv(const v4i (&vf)[CB], const v4i pf, v16i (&o)[CB])
{
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[cb], pf, o[cb], 0, 0, 0);
    if constexpr (BIG) {
        // (behind the MFMAs: with a branch ahead of them the compiler moves the accumulators, and spills 80 registers and more)
        if (__any(((pf[0] | pf[1] | pf[2] | pf[3]) & (int)0x80808080u) != 0)) {
            v4i part;
#pragma unroll
            for (int g = 0; g < 4; ++g) part[g] = (int)(((uint32_t)pf[g] >> 6) & 0x02020202u);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[cb], part, o[cb], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) part[g] = (int)(((uint32_t)part[g] << 6) - ((uint32_t)part[g] >> 1)); // 127 in place of 2
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf[cb], part, o[cb], 0, 0, 0);
        }
    }
}

// Output requantization (Sec. 3.2): clamp(floor((acc * M + 2^(sh-1)) / 2^sh), -127, 127) with M < 2^31 and
// 1 <= sh <= 62.  For sh >= 33 (every ratio s_V / (255 s_O) below 1/4) the rounding addend lies wholly in the high
// word of the 64-bit product and the low word cannot change the floor of a division by 2^(sh-32) >= 2, so the
// high word alone gives the same value: multiply-high, add, shift.  FAST is the caller's statement that sh >= 33.
template <bool FAST> __device__ __forceinline__ int requant(int32_t acc, int32_t M, int32_t sh)
{
    int v;
    if (FAST) {
        v = (__mulhi(acc, M) + (1 << (sh - 33))) >> (sh - 32);
    } else {
        const int64_t w = ((int64_t)acc * M + (1ll << (sh - 1))) >> sh;
        v = w > 127 ? 127 : (w < -127 ? -127 : (int)w);
    }
    return v > 127 ? 127 : (v < -127 ? -127 : v);
}

// the same with the form chosen at run time (sh is uniform over a head)
__device__ __forceinline__ int requant_any(int32_t acc, int32_t M, int32_t sh)
{
    return sh >= 33 ? requant<true>(acc, M, sh) : requant<false>(acc, M, sh);
}

// XOR swizzles of the 16-byte chunk index inside a key row.
// K fragments are read with ds_read_b128, lane -> key row, all lanes of a half-wave on the same
// chunk.  The LDS serves 16 consecutive lanes (256 bytes, all 64 banks) per clock, so the 16 rows
// of such a group must land on 16 different 16-byte bank groups: rows 256 bytes apart share
// banks, and the swizzle separates exactly those (measured: 4.2 clocks per wave instruction
// against 7.6 with a swizzle that only separates 8 consecutive rows).
template <int D> __device__ __forceinline__ int swz_k(int key) { return D == 128 ? ((key >> 1) & 7) : ((key >> 2) & 3); }
template <int D> __device__ __forceinline__ int swz_v(int key)
{
    return D == 128 ? ((key & 3) | (((key >> 3) & 1) << 2)) : (((key >> 1) & 1) | (((key >> 3) & 1) << 1));
}

} // namespace intattn
