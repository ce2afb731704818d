"""The search for a pair split looks at a few counts only: it has to find what looking at all of them finds."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_07103_amd", "csrc")

PROGRAM = r"""
#include <math.h>
#include <stdio.h>
#include <random>
#include "lmkan_split.h"
using namespace lmkan;

static int all(int64_t tiles, int K, int64_t part, int most)
{
    int best = 1;
    double best_us = pair_split_us((tiles + 255) / 256, K, 1, part);
    for (int split = 2; split <= most && K / split >= 4; ++split) {
        const int pairs = (K + split - 1) / split;
        if ((int64_t)(split - 1) * pairs >= K) continue;  // the last split would have none
        const double us = pair_split_us((tiles * split + 255) / 256, pairs, split, part);
        if (us < best_us) best = split, best_us = us;
    }
    return best;
}

int main()
{
    std::mt19937_64 r(1);
    std::uniform_real_distribution<double> u(0, 1);
    int bad = 0, split = 0;
    for (int i = 0; i < 200000; ++i) {
        const int64_t tiles = (int64_t)pow(2, u(r) * (i % 3 ? 9 : 22));
        const int K = i % 10 ? (int)pow(2, u(r) * 11) : 65535 - (int)(u(r) * 65534);
        const int64_t part = u(r) < 0.4 ? 0 : 16 * (int64_t)pow(2, u(r) * 30);
        const int most = u(r) < 0.7 ? K : 1 + (int)(u(r) * 40);
        const int want = all(tiles, K, part, most), got = pair_split_count(tiles, K, part, most);
        split += want > 1;
        if (want != got && bad++ < 5) printf("tiles %ld K %d part %ld most %d: %d, not %d\n", (long)tiles, K, (long)part, most, got, want);
        if (got > 1 && (got > most || (int64_t)(got - 1) * ((K + got - 1) / got) >= K)) ++bad;
    }
    printf("%d bad, %d split\n", bad, split);
    return bad != 0 || split < 50000;
}
"""


def test_the_short_search_finds_the_best_split(tmp_path):
    source, program = tmp_path / "split.cpp", tmp_path / "split"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", str(program), str(source)], check=True)
    got = subprocess.run([str(program)], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout
