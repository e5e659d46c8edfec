"""The order of additions of the four-sums-at-once exchange of the cubic fits,
lane by lane on the host: every lane of a row ends with the same bits (the
rows of one stencil are then updated with one reflection), and with the sums."""
import os
import subprocess


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2206_14061_amd", "csrc")

HOST = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include "lp_rowsum.h"

struct Row {
    double v[16];
};
static Row operator+(const Row& a, const Row& b)
{
    Row r;
    for (int i = 0; i < 16; ++i) r.v[i] = a.v[i] + b.v[i];
    return r;
}
static Row operator*(const Row& a, const Row& b)
{
    Row r;
    for (int i = 0; i < 16; ++i) r.v[i] = a.v[i] * b.v[i];
    return r;
}
struct Lanes {
    Row pick(int bit, const Row& a, const Row& b) const
    {
        Row r;
        for (int i = 0; i < 16; ++i) r.v[i] = i & bit ? a.v[i] : b.v[i];
        return r;
    }
    // quad permutations (controls below 256) and rotations to the right
    template <int CTRL>
    Row move(const Row& x) const
    {
        static_assert(CTRL < 0x100 || (CTRL > 0x120 && CTRL < 0x130), "known moves");
        Row r;
        for (int i = 0; i < 16; ++i)
            r.v[i] = CTRL < 0x100 ? x.v[(i & ~3) + ((CTRL >> (2 * (i & 3))) & 3)]
                                  : x.v[(i - (CTRL & 15)) & 15];
        return r;
    }
};

int main()
{
    uint64_t seed = 1;
    auto rnd = [&] {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (double)(int64_t)seed / 9.2e18 * std::exp2((int)(seed >> 59) - 16);
    };
    int lanes = 0, off = 0;
    for (int t = 0; t < 2000; ++t) {
        Row d[4], s, f[4];
        const double k = rnd();
        for (int i = 0; i < 16; ++i) {
            s.v[i] = k;
            for (int q = 0; q < 4; ++q) d[q].v[i] = rnd();
        }
        lp::row_sum4(Lanes{}, d, s, f);
        for (int q = 0; q < 4; ++q) {
            long double sum = 0, mag = 0;
            for (int i = 0; i < 16; ++i) {
                sum += d[q].v[i];
                mag += std::fabs(d[q].v[i]);
                lanes += std::memcmp(&f[q].v[i], &f[q].v[0], 8) != 0;
            }
            // four additions and a product, each half an ulp of its magnitude
            off += !(std::fabs((double)(f[q].v[0] - sum * k)) <=
                     5 * 1.2e-16 * (double)(mag * std::fabs(k)));
        }
    }
    std::printf("%d %d\n", lanes, off);
    return 0;
}
"""


def test_every_lane_ends_with_the_same_sums(tmp_path):
    src, exe = tmp_path / "row.cc", tmp_path / "row"
    src.write_text(HOST)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    lanes, off = subprocess.run([str(exe)], check=True, capture_output=True,
                                text=True).stdout.split()
    assert (int(lanes), int(off)) == (0, 0)
