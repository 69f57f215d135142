"""Every buffer request of the one-wavefront candidate walk stays inside the arrays or is answered with zeros (CPU: the offsets'
header is compiled for the host; no GPU)."""
import pathlib
import shutil
import subprocess

ROOT = pathlib.Path(__file__).resolve().parent.parent

# A buffer starts at the cluster's first point and ends at its last; the cluster is the last one of arrays that hold nothing behind it.
# Range check of a raw buffer load: zeros if the vector offset (with the constant one) is not below the record count; otherwise the
# address is vector + scalar offset, whatever the scalar one is.
MAIN = r"""
#include <cstdio>
#include <initializer_list>
#include "walk_offsets.hpp"
using namespace lorann;
static int64_t worst = 0;
static bool sound(int64_t m_c, int own, int64_t base, int stride, int bytes) {
    const int64_t point = base + own;
    if (point - m_c > worst) worst = point - m_c;
    if ((point + 1) * stride > INT32_MAX) return false;                       // the kernel computes in int
    const PieceOffset at = piece_offset(own, (int)base, stride);
    if (at.vector < 0 || at.scalar < 0) return false;
    for (int64_t u = 0; u < stride; u += bytes) {                             // a code is read in several loads
        const int64_t v = (int64_t)at.vector + u, records = m_c * stride;
        const bool zeros = v >= records;
        if (zeros != (point >= m_c)) return false;                            // inside: the point itself, beyond: zeros
        if (!zeros && v + at.scalar + bytes > records) return false;          // past the array
    }
    return true;
}
static int piece(int64_t m_c, int64_t base, bool quarter) {
    for (int lane = 0; lane < 64; ++lane)
        for (int stride : {4, 32, 64})
            if (!sound(m_c, quarter ? quarter_point(lane) : lane, base, stride, stride < 16 ? stride : 16)) {
                std::printf("cluster of %lld points, piece at %lld, lane %d, stride %d\n", (long long)m_c, (long long)base, lane, stride);
                return 1;
            }
    return 0;
}
int main() {
    const int64_t top = kSelectWaveMaxCluster;
    for (int64_t m_c : {int64_t(1), int64_t(7), int64_t(63), int64_t(64), int64_t(65), int64_t(191), int64_t(255), int64_t(256), int64_t(257), int64_t(449),
                        int64_t(1000), int64_t(2048), int64_t(2049), int64_t(41111), top - 1, top}) {
        const int64_t from = m_c > 4096 ? (m_c - 2048) / 256 * 256 : 0;       // (the far end of a large cluster is where it matters)
        for (int b = 0; b < kWalkAhead; ++b) if (piece(m_c, 64 * b, false)) return 1;
        for (int64_t p0 = from; p0 < m_c; p0 += 256)
            for (int b = 0; b < 4; ++b) if (piece(m_c, p0 + 64 * (b + kWalkAhead), false)) return 1;
        // quarters: 512 points per item, quarters 8 apart, two halves each; none left: the cluster's end
        for (int64_t t = from / 512 * 512; t < m_c; t += 512)
            for (int s = 0; s < 4; ++s)
                for (int half = 0; half < 2; ++half) if (piece(m_c, t + 8 * s + half * kQuarterHalf, true)) return 1;
        for (int half = 0; half < 2; ++half) if (piece(m_c, m_c + half * kQuarterHalf, true)) return 1;
    }
    if (worst >= kWalkReach) { std::printf("a request is %lld points beyond the end\n", (long long)worst); return 1; }
    return 0;
}
"""


def test_requests_stay_inside_the_arrays(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    assert cxx, "a host C++ compiler is needed"
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", str(ROOT / "paper_2410_18926_amd" / "csrc"),
                    "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    res = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_the_walk_takes_its_offsets_from_the_header():
    """The kernel's buffer loads all go through piece_offset."""
    text = (ROOT / "paper_2410_18926_amd" / "csrc" / "select_wave.hpp").read_text()
    loads = [l for l in text.splitlines() if "raw_buffer_load" in l]
    assert len(loads) == 4 and all("at.vector" in l and "at.scalar" in l or "at4.vector" in l and "at4.scalar" in l for l in loads)
