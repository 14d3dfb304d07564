"""Rows of many ids played through the choice of candidates (csrc/candidates.h) on the CPU: the sampled ids are ids of the row, all of
them different and one in each of 1024 equal parts, and of the rows that look for their K largest among candidates next to all find them.

The number of samples above a key of true rank x is binomial in a sample without strata, narrower in one with: a row fails where it is 3
spreads off, once in 700 on either side: of 2 000 rows 6 at the very most, 30 allowed."""
import subprocess

import pytest

import plan_choice

_MAIN = r"""
#include <stdio.h>
#include <string.h>
#include <algorithm>
#include <random>
#include <set>
#include <vector>
#include "candidates.h"
static uint32_t order_key(float z) { uint32_t b; memcpy(&b, &z, 4); return b & 0x80000000u ? ~b : b | 0x80000000u; }
int main() {
    for (uint32_t V = 16385; V <= 65536; V += V < 17000 ? 1 : 97) {
        uint32_t last = 0;
        for (uint32_t t = 0; t < kSamples; ++t) {
            const uint32_t id = sample_id(t, V);
            if (id >= V || (t && id <= last) || (uint64_t)id * kSamples / V > t || (uint64_t)(id + 1) * kSamples / V < t) { printf("sample %u of %u: %u\n", t, V, id); return 1; }
            last = id;
        }
    }
    std::mt19937 rng(1);
    std::normal_distribution<float> n(0.0f, 3.0f);
    int rows = 0, missed = 0, shapes = 0;
    for (uint32_t V : {16385u, 20000u, 32768u, 33000u, 40000u, 65536u}) for (uint32_t K : {50u, 1000u, 2000u, 4000u, 6000u}) {
        if (!candidates_fit(K, V)) continue;
        ++shapes;
        for (int r = 0; r < 2000 / 18; ++r, ++rows) {
            std::vector<uint32_t> key(V), s(kSamples);
            for (auto &k : key) k = order_key(n(rng));
            const uint32_t kmax = *std::max_element(key.begin(), key.end());
            for (uint32_t t = 0; t < kSamples; ++t) s[t] = std::min((kmax - key[sample_id(t, V)]) >> kBin0Shift, (uint32_t)kSelBins - 1);
            std::nth_element(s.begin(), s.begin() + candidate_rank(K, V) - 1, s.end());
            const uint32_t bound = candidate_bound(kmax, s[candidate_rank(K, V) - 1]);
            const uint32_t found = std::count_if(key.begin(), key.end(), [&](uint32_t k) { return k >= bound; });
            missed += found < K || found > kCand;
        }
    }
    printf("%d %d %d\n", shapes, rows, missed);
}
"""


def test_rows_find_their_largest_among_the_candidates(tmp_path):
    (tmp_path / "main.cpp").write_text(_MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", plan_choice.CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    r = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    shapes, rows, missed = (int(x) for x in r.stdout.split())
    assert shapes >= 15 and missed <= 30 * rows // 2000, (shapes, rows, missed)


@pytest.mark.parametrize("V,K,fits", [(65536, 2000, True), (33000, 2000, True), (17000, 2000, True), (65536, 4000, False), (65536, 6000, False),
                                      (16384, 1000, False), (4097, 50, False), (20000, 20000, False)])
def test_which_rows_look_for_candidates(tmp_path, V, K, fits):
    (tmp_path / "main.cpp").write_text('#include "candidates.h"\nint main() { return candidates_fit(%d, %d); }' % (K, V))
    subprocess.run(["g++", "-std=c++17", "-I", plan_choice.CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    assert subprocess.run([str(tmp_path / "main")]).returncode == int(fits)
