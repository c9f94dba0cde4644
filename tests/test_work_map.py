"""The mapping of workgroups to work (csrc/work_map.h), compiled for the host and enumerated: every query tile of every head
is taken exactly once, the XCDs get the same number of work items (where one has more than a compute unit for each, to within
1 / 64), and whole (batch, KV head) groups stay on one XCD."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_21513_amd", "csrc")

MAIN = r"""
#include <stdio.h>
#include <string.h>
#include <set>
#include <tuple>
#include "work_map.h"
using namespace intattn;

// 0, or the number of the check that failed
static int check(int B, int Hkv, int group, int n_qtiles, int batch, int n_split)
{
    FwdParams p;
    memset(&p, 0, sizeof(p));
    p.B = B; p.Hkv = Hkv; p.group = group; p.Hq = Hkv * group; p.n_qtiles = n_qtiles;
    p.group_batch = std::min(batch, fwd_group_batch(B, Hkv, 0));
    const int64_t grid = fwd_map_work(p, n_split) / n_split;
    if (grid % NUM_XCD != 0 || grid * n_split != fwd_map_work(p, n_split)) return 1;
    std::set<std::tuple<int, int, int>> seen;
    std::set<std::pair<int, int>> group_on_xcd;
    int64_t per_xcd[NUM_XCD] = {0};
    for (int64_t bid = 0; bid < grid; ++bid) {
        const WorkItem w = fwd_work_item(p, (int)bid);
        if (!w.valid) continue;
        if (w.b < 0 || w.b >= B || w.hq < 0 || w.hq >= p.Hq || w.qt < 0 || w.qt >= n_qtiles) return 2;
        if (w.kvh != w.hq / group) return 3;
        if (!seen.insert({w.b, w.hq, w.qt}).second) return 4;
        per_xcd[bid % NUM_XCD]++;
        group_on_xcd.insert({w.b * Hkv + w.kvh, (int)(bid % NUM_XCD)});
    }
    if ((int64_t)seen.size() != (int64_t)B * p.Hq * n_qtiles) return 5;
    int64_t lo = per_xcd[0], hi = per_xcd[0];
    for (int64_t n : per_xcd) lo = n < lo ? n : lo, hi = n > hi ? n : hi;
    const int64_t idle = NUM_XCD * hi - (int64_t)seen.size(); // unit slots of the longest XCD that the others do not fill
    if (hi - lo > 1 && hi * n_split > XCD_CUS && idle * 64 >= NUM_XCD * hi) return 6;
    for (int g = 0; g < std::min(p.map.whole * NUM_XCD, B * Hkv); ++g) {
        int n = 0;
        for (int x = 0; x < NUM_XCD; ++x) n += (int)group_on_xcd.count({g, x});
        if (n != 1) return 7;
    }
    return 0;
}

int main()
{
    // quotients at both sides of every multiple near the ends of the range
    for (uint32_t d : {1u, 2u, 3u, 5u, 7u, 8u, 12u, 97u, 1000u, 65537u, (1u << 28) - 1, 1u << 28})
        for (uint64_t k : {0ull, 1ull, 2ull, 0x7fffffffull / d, 0x7fffffffull / d / 2})
            for (int64_t o : {-1, 0, 1}) {
                const int64_t n = (int64_t)(k * d) + o;
                if (n >= 0 && n <= 0x7fffffff && quotient((int)n, fast_div(d)) != (int)(n / d)) return printf("quotient %lld / %u\n", (long long)n, d), 1;
            }
    int cases = 0;
    for (int groups : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 15, 16, 17, 20, 33, 36, 51, 63, 64, 65, 100, 255, 256, 257})
        for (int Hkv : {1, 3, 4})
            for (int group : {1, 3, 4, 8})
                for (int n_qtiles : {1, 2, 5, 16, 33})
                    for (int batch : {1, 2, 3, 1000})
                        for (int n_split : {1, 5}) {
                            if (groups % Hkv) continue;
                            const int bad = check(groups / Hkv, Hkv, group, n_qtiles, batch, n_split);
                            if (bad)
                                return printf("check %d: B %d Hkv %d group %d tiles %d batch %d split %d\n", bad, groups / Hkv, Hkv, group, n_qtiles, batch, n_split), 1;
                            ++cases;
                        }
    printf("%d cases\n", cases);
    return 0;
}
"""


def test_every_work_item_once_and_evenly_over_the_xcds(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-host-only", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert "cases" in r.stdout
