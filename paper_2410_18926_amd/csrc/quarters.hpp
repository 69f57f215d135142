// Where the quarter maxima of large clusters (score_mfma.hpp) are kept.  Plain C++: tests/test_quarter_layout.py compiles it for the host.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace lorann {

constexpr int kChunkPoints = 512;                        // points of a scoring work item
constexpr int kGroupPairs = 64;                          // pairs of a scoring work item
constexpr int kSubMinPoints = 2048;                      // smaller clusters have no quarter maxima
constexpr int kWaveWholePoints = 4 * kSubMinPoints;      // the largest cluster that one wavefront may have to look through without them
// Quarter maxima of at most this many work items are kept, 1 KiB each.  A launch of 32 768 queries over 1M points with heavy-tailed norms
// (four clusters beyond kWaveWholePoints, 398 chunks) needs 204 000: candidate selection 901 us, 1771 with four wavefronts per query.
constexpr int64_t kSubMaxItems = 512 * 1024;

inline int64_t cluster_chunks(int64_t points) { return (points + kChunkPoints - 1) / kChunkPoints; }

// The chunks of the clusters beyond kSubMinPoints, one cluster after the other, the LARGEST first: where room is short it is the small
// ones that go without.  A query probes a cluster at most once, so a cluster's pairs make at most ceil(nq / 64) groups, and the maxima of
// (cluster c, chunk k, group g) have their place at (first[c] + k) * ceil(nq / 64) + g.
struct QuarterLayout {
    std::vector<int32_t> first;      // [L] a cluster's first chunk, -1: too small (empty: no cluster is large)
    int64_t chunks = 0;              // of all of them
    int64_t needed = 0;              // of those beyond kWaveWholePoints
};

inline QuarterLayout lay_out_quarters(const int64_t* off, int L) {
    QuarterLayout q;
    q.first.assign((size_t)L, -1);
    std::vector<int32_t> large;
    for (int c = 0; c < L; ++c) if (off[c + 1] - off[c] > kSubMinPoints) large.push_back(c);
    std::stable_sort(large.begin(), large.end(), [&](int32_t a, int32_t b) { return off[a + 1] - off[a] > off[b + 1] - off[b]; });
    for (int32_t c : large) {
        const int64_t points = off[c + 1] - off[c];
        q.first[(size_t)c] = (int32_t)q.chunks;
        q.chunks += cluster_chunks(points);
        if (points > kWaveWholePoints) q.needed = q.chunks;
    }
    return q;
}

inline int64_t quarter_groups(int64_t nq) { return (nq + kGroupPairs - 1) / kGroupPairs; }
// Chunks that keep their maxima in a launch of nq queries (a cluster whose chunks are not all among them has none).
inline int64_t quarter_chunks(int64_t chunks, int64_t nq) { return std::min(chunks, kSubMaxItems / quarter_groups(nq)); }
// One wavefront per query may walk: every cluster that it could not look through on its own has its maxima.
inline bool quarters_suffice(const QuarterLayout& q, int64_t kept) { return q.needed <= kept; }

}  // namespace lorann
