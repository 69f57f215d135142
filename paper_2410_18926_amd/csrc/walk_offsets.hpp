// Byte offsets of the buffer loads of the one-wavefront walk (select_wave.hpp).  Plain C++: tests/test_walk_offsets.py compiles it
// for the host and checks every request of the walk against the arrays.
#pragma once
#include <cstdint>

namespace lorann {

// A raw buffer load's range check compares the VECTOR offset with the buffer's size and returns zeros beyond it; the scalar offset is
// added to the address without being part of the comparison.  So the whole place of a point goes into the vector operand.
struct PieceOffset { int vector, scalar; };
constexpr PieceOffset piece_offset(int own, int base, int stride) { return {(base + own) * stride, 0}; }

// The walk requests pieces before it knows whether the cluster goes on; no request is this many points beyond its end.
constexpr int kWalkReach = 512;
// Points of the largest cluster that one wavefront walks: byte offsets (64 bytes per point at most) stay below 2^31.
constexpr int64_t kSelectWaveMaxCluster = int64_t(1) << 24;
static_assert((kSelectWaveMaxCluster + kWalkReach) * 64 < (int64_t(1) << 31), "byte offsets inside a cluster must fit an int");

// Pieces of 64 points requested ahead of the one that is scored, and how far apart the two halves of a quarter are.
constexpr int kWalkAhead = 3;
constexpr int kQuarterHalf = 256;
// First point of a lane in a quarter's half: eight runs of eight points, 32 apart.
constexpr int quarter_point(int lane) { return (lane >> 3) * 32 + (lane & 7); }

}  // namespace lorann
