// Workgroup -> work mapping of the forward kernels.
//
// Workgroups are dealt round-robin to the 8 XCDs (workgroup id mod 8), and each XCD has its own L2.  All query heads that
// share one KV head -- i.e. one (batch, KV head) group -- are therefore sent to the same XCD, so that K and V of the group
// are fetched into one L2 only.  Within an XCD the groups are taken in batches of FwdParams::group_batch groups: inside a
// batch the longest (latest) causal query tiles of all its groups come first, which balances the compute units; the batch is
// sized so that the K and V its workgroups read at the same time fit the XCD's L2 (with the tiles of all 64 groups of an XCD
// interleaved, and no sharing between query heads, sweep C of the batched prefill workload streamed 4.3 TB/s of K and V from
// HBM and was bound by it).
//
// Where B * Hkv is not a multiple of 8, the groups past the last multiple (at most seven) are dealt to all XCDs unit by unit
// (a unit: a query tile of a query head), evenly among the units of the whole groups.  With whole groups only, as many XCDs
// as there are groups left over work on one group more, or alone (4096 rows, 8 / 2 heads, d 128: 414 us, dealt out 123;
// 33 heads, d 128: 243 and 216).  K and V of the groups dealt out pass the L2 of every XCD; no other group's do.  (Cutting every
// group into eight classes of units, one for each XCD, instead: 255 heads of 197 rows, which have fewer units than that, 58 us
// against 19; 33 heads of 4096 rows, d 64, 278 against 184.)  Whole groups only, some XCDs with one less, where an XCD has a
// compute unit for each of its units, so that nothing is left to even out (one head of 128 rows: 6.2 us, dealt out 6.35), and
// where less than 1 / 64 of the chip would idle (255 heads of 4096 rows, d 128: 1282 us, dealt out 1308).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "params.h"

namespace intattn {

constexpr int NUM_XCD = 8; // (a power of two)
constexpr int64_t XCD_L2_BUDGET = 4 << 20; // bytes of K (and V) that a batch of groups may hold in flight: the L2 of an XCD
                                           // (1 to 16 MiB measured within 3 % of each other on the batched prefill workload)
constexpr int XCD_CUS = 32;

// groups per batch for kernels that stream `bytes_per_group` of K (and V) per (batch, KV head) group
inline int fwd_group_batch(int B, int Hkv, int64_t bytes_per_group)
{
    const int64_t gpx = ((int64_t)B * Hkv + NUM_XCD - 1) / NUM_XCD; // groups of an XCD at most
    const int64_t fit = bytes_per_group > 0 ? XCD_L2_BUDGET / bytes_per_group : gpx;
    return (int)std::max<int64_t>(1, std::min(fit, gpx));
}

// floor(n / d) for 0 <= n < 2^31 as a product: with l = ceil(log2 d), mul = ceil(2^(31 + l) / d) fits 32 bits and
// n mul / 2^(31 + l) exceeds n / d by n e / (d 2^(31 + l)), e = d mul - 2^(31 + l) < d <= 2^l: by less than 1 / d.
inline FastDiv fast_div(uint32_t d)
{
    const uint32_t l = d > 1 ? 32 - __builtin_clz(d - 1) : 0;
    return FastDiv{(uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
__host__ __device__ __forceinline__ int quotient(int n, const FastDiv &d) { return (int)(((uint64_t)(uint32_t)n * d.mul) >> d.shift); }

// Fills p.map for p's shape, p.n_qtiles and p.group_batch; returns the number of workgroups.  Every division of the mapping is
// by a number known here.  n_split: workgroups per work item (key-split launches).
inline int64_t fwd_map_work(FwdParams &p, int n_split = 1)
{
    const int groups = p.B * p.Hkv;
    WorkMap &m = p.map;
    m.groups = groups;
    m.units = p.group * p.n_qtiles;
    m.whole = groups / NUM_XCD;
    m.left = groups % NUM_XCD;
    if (m.left > 0 && ((int64_t)(m.whole + 1) * m.units * n_split <= XCD_CUS || (NUM_XCD - m.left) * 64 < NUM_XCD * (m.whole + 1)))
        m.whole += 1, m.left = 0;
    const int64_t dealt = ((int64_t)m.left * m.units + NUM_XCD - 1) / NUM_XCD, slots = dealt + (int64_t)m.whole * m.units;
    // ceil(s m / 2^32) of the first s slots are dealt out, the first one among them: in an XCD's order a dealt-out unit meets
    // whole groups' units of about its length.  For s = slots (below 2^32) that is `dealt`.
    m.dealt_mul = m.whole > 0 && dealt > 0 ? (uint32_t)(((uint64_t)dealt << 32) / slots) : 0;
    p.group_batch = std::min(p.group_batch, std::max(m.whole, 1));
    const FastDiv none = {0, 0}; // quotient 0
    m.by_left = m.left > 0 ? fast_div((uint32_t)m.left) : none;
    m.by_group = fast_div((uint32_t)p.group);
    m.by_hkv = fast_div((uint32_t)p.Hkv);
    m.by_full = fast_div((uint32_t)p.group_batch);
    m.by_batch = m.by_last = none;
    if (p.group_batch < m.whole) { // several batches
        m.by_batch = fast_div((uint32_t)(p.group_batch * m.units));
        m.by_last = fast_div((uint32_t)std::max(m.whole % p.group_batch, 1));
    }
    m.fold = 0;
    return NUM_XCD * slots * n_split;
}

struct WorkItem {
    int b, hq, kvh, qt;
    bool valid;
};

// All of it is scalar and straight-line, and everything it needs is asked for at once: a load in a branch is a latency of the
// scalar cache more at the head of every workgroup.
__host__ __device__ __forceinline__ WorkItem fwd_work_item(const FwdParams &p, int bid)
{
    const WorkMap m = p.map;
    const int g = p.group, gb = p.group_batch, n_qtiles = p.n_qtiles, hkv = p.Hkv;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::"s"(m.groups), "s"(m.whole), "s"(m.left), "s"(m.units), "s"(m.dealt_mul), "s"(m.by_left.mul), "s"(m.by_left.shift),
                 "s"(m.by_group.mul), "s"(m.by_group.shift), "s"(m.by_hkv.mul), "s"(m.by_hkv.shift), "s"(m.by_batch.mul),
                 "s"(m.by_batch.shift), "s"(m.by_full.mul), "s"(m.by_full.shift), "s"(m.by_last.mul), "s"(m.by_last.shift),
                 "s"(m.fold), "s"(g), "s"(gb), "s"(n_qtiles), "s"(hkv), "s"(p.hp_table));
#endif
    const int xcd = bid & (NUM_XCD - 1), plain = bid >> 3, round = plain & ~31;
    // folded order: every other round of an XCD's 32 compute units in reverse
    const int back = round + (32 < m.fold - round ? 32 : m.fold - round) - 1 - (plain - round);
    const int slot = (m.fold > 0 && (round & 32)) ? back : plain;
    const uint64_t scaled = (uint64_t)(uint32_t)slot * m.dealt_mul + 0xffffffffu;
    const int before = (int)(scaled >> 32), upto = (int)((scaled + m.dealt_mul) >> 32); // dealt-out slots below this one, and with it
    const bool dealt = m.whole == 0 || upto > before;
    // a dealt-out unit: round the groups and the XCDs, query head fastest: of 1, 2 or 4 groups an XCD meets one only
    const int t = (m.whole == 0 ? slot : before) * NUM_XCD + xcd, unit = quotient(t, m.by_left);
    // a whole group's: within a batch, query heads of a group fastest (they share K and V), then the groups, then the tiles;
    // the last batch may hold fewer groups
    const int s = slot - before, first = quotient(s, m.by_batch) * gb, rem = s - first * m.units, rest = quotient(rem, m.by_group);
    const bool last = first + gb > m.whole;
    const int rev = last ? quotient(rest, m.by_last) : quotient(rest, m.by_full);
    // tiles in reverse: the longest (latest) first
    const int unit_rev = quotient(unit, m.by_group), qt_rev = dealt ? unit_rev : rev;
    const int hg = dealt ? unit - unit_rev * g : rem - rest * g;
    const int gi = dealt ? m.whole * NUM_XCD + t - unit * m.left : (first + rest - rev * (last ? m.whole - first : gb)) * NUM_XCD + xcd;
    WorkItem w;
    w.valid = dealt ? unit < m.units : gi < m.groups;
    w.b = quotient(gi, m.by_hkv);
    w.kvh = gi - w.b * hkv;
    w.hq = w.kvh * g + hg;
    w.qt = n_qtiles - 1 - qt_rev;
    return w;
}

// Key-split launches: every work item is taken by n_split consecutive workgroups of one XCD, each with a range of the
// item's key tiles.  Returns the range's number and replaces bid by the item's.
__device__ __forceinline__ int fwd_split_index(int &bid, int n_split)
{
    const int xcd = bid % NUM_XCD, slot = bid / NUM_XCD;
    bid = (slot / n_split) * NUM_XCD + xcd;
    return slot % n_split;
}

} // namespace intattn
