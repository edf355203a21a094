"""The split of a captured chunk into launches, by brute force over small chunks and at the
launch bound: every step once, joined launches in whole stretches, the statistics' stretch alone,
and the step hints wherever a launch is of one step."""
import subprocess

from paper_2503_09203_amd import build

MAIN = r"""
#include "graph_split.hpp"
#include <cstdio>
using namespace mgx;
static int check(int n, int K, bool single, bool join, bool stats) {
    const ChunkSplit s{n, K, single, join, stats, 4};
    bool one = false;
    int done = 0, k = 0;
    while (done < n) {
        k = s.next(done);
        if (k < 1 || k > n - done || k > (K > kMaxLaunchSteps ? K : kMaxLaunchSteps)) return 1;
        if (single && k != 1) return 2;
        if (!single && done % K != 0) return 3;              // stretches start at multiples of K
        if (!single && !join && k != (n - done < K ? n - done : K)) return 4;
        if (join && k < 4 && k > K) return 5;
        one = one || k == 1;
        done += k;
    }
    // the last launch ends the last stretch, and holds no other where statistics are taken
    if (stats && !single && k != (n % K ? n % K : K)) return 6;
    return one == s.any_single() ? 0 : 7;
}
int main() {
    for (int single = 0; single < 2; ++single)
        for (int join = 0; join + single < 2; ++join)
            for (int stats = 0; stats < 2; ++stats)
                for (int K = 1; K < 20; ++K)
                    for (int n = 1; n < 70; ++n)
                        for (int far = 0; far < 2; ++far) {
                            if (join && K == 1) continue;
                            const int steps = far ? kMaxLaunchSteps / K * K + n : n;
                            if (int e = check(steps, K, single, join, stats)) {
                                std::printf("fault %d: n %d K %d single %d join %d stats %d\n", e, steps, K, single, join, stats);
                                return 1;
                            }
                        }
    return check(4100, 4097, false, false, true);
}
"""


def test_split_of_a_chunk(tmp_path):
    src = tmp_path / "split.cpp"
    src.write_text(MAIN)
    exe = str(tmp_path / "split")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC, str(src), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
