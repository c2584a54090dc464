"""The simulation's 64-bit queue keys at the ends of their fields, on the host:
the key arithmetic is compiled into a small program that walks them."""
import os
import subprocess

import pytest

from paper_2404_03226_amd import build

SRC = r"""
#include <cstdio>
#include <vector>
#include "keys.hpp"
using namespace insp;

struct Entry { uint64_t ia, ie; uint32_t seq; };

// a before b: the order by (first, second, earlier push)
static bool before(const Entry &a, const Entry &b, int rule) {
    if (rule < 2) {
        const uint64_t a0 = rule ? a.ie : a.ia, b0 = rule ? b.ie : b.ia, a1 = rule ? a.ia : a.ie, b1 = rule ? b.ia : b.ie;
        if (a0 != b0) return a0 > b0;
        if (a1 != b1) return a1 > b1;
    }
    return a.seq < b.seq;
}

template <int KK>
static int check(int o0) {
    unsigned long long slot[64];
    Keys<KK> K;
    K.ka = slot;
    K.ke = nullptr;
    K.o0 = o0;
    const uint32_t most = (uint32_t)M21;
    std::vector<Entry> all;
    for (uint64_t ia : {0ull, 1ull, 31ull, 32ull, (unsigned long long)most - 1, (unsigned long long)most})
        for (uint64_t ie : {0ull, 1ull, (unsigned long long)most - 1, (unsigned long long)most})
            for (uint32_t seq : {0u, 1u, most - 1, most}) all.push_back({ia, ie, seq});
    int bad = 0;
    for (const Entry &a : all)
        for (int r = 0; r < 2; r++) {
            K.put(5, K.big(a.ia << 21 | a.ie, a.seq));
            const uint64_t ka = K.lds(5, r);
            if (K.word(5) == 0 || ka == 0) {
                printf("entry (%llu, %llu, %u) reads as an empty slot\n", (unsigned long long)a.ia, (unsigned long long)a.ie, a.seq);
                bad++;
            }
            const int rule = r ? 1 : o0 == 2 ? 2 : 0;
            for (const Entry &b : all) {
                K.put(6, K.big(b.ia << 21 | b.ie, b.seq));
                const bool same = rule == 2 ? a.seq == b.seq : a.ia == b.ia && a.ie == b.ie && a.seq == b.seq;
                if (same ? ka != K.lds(6, r) : before(a, b, rule) != (ka > K.lds(6, r))) bad++;
            }
        }
    K.put(5, 0);
    if (K.lds(5, 0) || K.lds(5, 1)) bad++;
    return bad;
}

// ranks of up to 42 bits, the longest first
static int ranks() {
    int bad = 0;
    Keys<kFixed> K;
    K.o0 = 3;
    uint64_t prev = 0;
    for (uint64_t rank : {0ull, 1ull, (1ull << 32) - 1, 1ull << 32, (1ull << 42) - 1})
        for (uint32_t seq : {(uint32_t)M21, 1u, 0u}) {
            const uint64_t k = K.rule(K.big(rank, seq), 0);
            if (k <= prev) bad++;
            prev = k;
        }
    return bad;
}

int main() {
    const int bad = check<kWide>(0) + check<kWide>(2) + check<kFixed>(0) + check<kFixed>(2) + ranks();
    printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def test_every_entry_has_a_key(tmp_path):
    src = tmp_path / "keys.hip"
    src.write_text(SRC)
    exe = str(tmp_path / "keys")
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    subprocess.check_call([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-I" + build.CSRC, "-o", exe, str(src)])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
