"""Places of the quarter maxima of large clusters: disjoint, inside the buffer, the largest clusters first - and where a cluster that
one wavefront cannot look through on its own would go without, the rule that chooses that walk says no (CPU: the header is compiled for
the host; no GPU)."""
import pathlib
import shutil
import subprocess

ROOT = pathlib.Path(__file__).resolve().parent.parent

MAIN = r"""
#include <cstdio>
#include <random>
#include "quarters.hpp"
using namespace lorann;
#define REQUIRE(x) do { if (!(x)) { std::printf("%s (trial %d, nq %lld)\n", #x, trial, (long long)nq); return 1; } } while (0)
int main() {
    std::mt19937 rng(7);
    int with = 0, without = 0;
    for (int trial = 0; trial < 400; ++trial) {
        const int L = 1 + (int)(rng() % 300);
        std::vector<int64_t> off(1, 0);
        for (int c = 0; c < L; ++c) {
            const double u = (rng() % 100000) / 1e5;
            const int64_t size = trial % 5 == 0 ? (int64_t)(rng() % 3000) : (int64_t)(2000.0 / (1.0 - 0.9995 * u));     // heavy tail up to 4 000 000
            off.push_back(off.back() + size);
        }
        const QuarterLayout q = lay_out_quarters(off.data(), L);
        for (int64_t nq : {2049ll, 10000ll, 22000ll, 32768ll}) {
            const int64_t groups = quarter_groups(nq), kept = quarter_chunks(q.chunks, nq);
            REQUIRE(groups * kGroupPairs >= nq && kept * groups <= kSubMaxItems && kept <= q.chunks);
            std::vector<char> used((size_t)kept, 0);
            int64_t smallest_with = INT64_MAX, largest_without = 0;
            for (int c = 0; c < L; ++c) {
                const int64_t points = off[c + 1] - off[c], chunks = cluster_chunks(points);
                REQUIRE((q.first[c] >= 0) == (points > kSubMinPoints));
                if (q.first[c] < 0) continue;
                if (q.first[c] + chunks > kept) { largest_without = std::max(largest_without, points); continue; }       // the kernels' condition
                smallest_with = std::min(smallest_with, points);
                for (int64_t k = 0; k < chunks; ++k) { REQUIRE(!used[q.first[c] + k]); used[q.first[c] + k] = 1; }
            }
            REQUIRE(largest_without <= smallest_with);
            const bool wave_walk = quarters_suffice(q, kept);                                                                  // the dispatch rule
            REQUIRE(wave_walk == (largest_without <= kWaveWholePoints));
            (wave_walk ? with : without) += 1;
        }
    }
    if (with < 100 || without < 100) { std::printf("%d with, %d without\n", with, without); return 1; }
    return 0;
}
"""


def test_every_cluster_that_needs_them_has_its_quarter_maxima(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    assert cxx, "a host C++ compiler is needed"
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined,address", "-fno-sanitize-recover=all", "-I",
                    str(ROOT / "paper_2410_18926_amd" / "csrc"), "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    res = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr

