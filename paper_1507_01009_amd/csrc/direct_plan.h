// Which kernels form the FP64 direct sums, and how they split the sources: a
// function of the sizes alone (no HIP in here, so a host program can check
// it).
#ifndef TG_DIRECT_PLAN_H
#define TG_DIRECT_PLAN_H

#include <algorithm>
#include <cstdint>

namespace tg {

enum class DirectPath { kFew, kTile, kPlain };

struct DirectPlan {
  DirectPath path;
  int lane_targets;    // tiles: targets to a lane
  int64_t chunk;       // sources of one partial sum
  int64_t nchunks;     // partial sums of a target (1: written as the result)
  bool block_reduce;   // a block per target adds them up (else a thread)
};

constexpr int kTileSrc = 256;            // sources of a tile in LDS

// The few-target kernel takes up to 4096 targets of several segments, which
// have no tiled kernel, and the plain one gives neighbouring lanes targets of
// different segments: 64 systems of 20000 stars with two SMBHs each 24 us in
// 640 blocks against 155, 256 systems of 8192 with one each 22 against 189.
// Of one segment it takes up to kFewTargets targets (a tile costs its block of
// 128 whatever it holds: on 262144 sources 64 targets 48 us against 66, 96
// targets 67 against 69, 128 targets 86 against 69), and more as long as there
// are few pairs, which leave most of the chip without a tile: 128 targets on
// 8192 sources 11.4 us against 19.2, 192 on 32768 23.7 against 28.5; at the
// line 128 on 65536 30.2 against 29.0, 512 on 16384 30.4 against 29.0.
constexpr int64_t kFewTargets = 88, kFewTargetsMax = 4096, kFewPairs = (int64_t)1 << 23;

// Sources per block: 4096, or 1024 where that leaves much of the chip idle,
// up to 384 blocks over all targets, and a target's partial sums are at most
// four to a thread of the second pass (2^20 sources) and fit.  Measured, in us
// with 1024 and with 4096: 131072 sources on one target 9.2 and 12.8 (32
// blocks of 4096), 500000 on two 14.8 and 16.8 (246), at the line 250000 on
// six 18.3 and 17.1 (372) and 131072 on twelve 13.2 and 14.5 (384), beyond it
// 500000 on four 21.4 and 19.9 (492), 250000 on 24 42.0 and 23.3 (1488).
inline int few_span(int64_t part_cap, int64_t n, int64_t nt) {
  const bool idle = (n + 4095) / 4096 * nt <= 384;
  const bool fits = n <= (1 << 20) && (n + 1023) / 1024 * nt * 8 <= part_cap;
  return idle && fits ? 1024 : 4096;
}

// Whether sums of (at most) n sources of a segment on nt targets in all take
// the few-target kernel (part_cap doubles of partial sums).
inline bool few_path(int64_t part_cap, int64_t n, int64_t nt, int nseg) {
  if (nt > kFewTargetsMax || n < 8192) return false;
  if (nseg == 1 && nt > kFewTargets && nt * n >= kFewPairs) return false;
  const int64_t bpt = (n + 4095) / 4096;
  return bpt * nt * 8 <= part_cap && bpt <= 65535;
}

// The tiled kernel's split: chunks of whole tiles, enough for kTileBlocks
// blocks (eight per CU, two rounds of those resident) where the partial sums
// fit.  One target to a lane where two would give less than a block per CU
// (1000 targets on 1000 sources: 19.5 against 26.7 us).
constexpr int64_t kTileBlocks = 2048;

// More targets than one round of tile blocks holds (four to a CU), on few
// sources: two or three of the four waves of such a block have little to do or
// nothing, and a thread per target is faster.  In us by tiles and by threads:
// a million targets on 64 sources 203 and 144, on 80 213 and 178, on 100 241
// and 227; 200000 on 64 53 and 43, on 80 54 and 53, on 100 64 and 65; a round
// or less, 131072 on 64, 24.6 and 25.1, on 100 31 and 38.
constexpr int64_t kTileRound = 1 << 17, kTileMinSrc = 64, kTileMinSrcMany = 96;

// n: sources of the longest segment; nt >= 1 targets in all.
inline DirectPlan direct_plan(int64_t part_cap, int64_t n, int64_t nt, int nseg) {
  if (few_path(part_cap, n, nt, nseg)) {
    const int64_t span = few_span(part_cap, n, nt);
    return {DirectPath::kFew, 1, span, (n + span - 1) / span, true};
  }
  // one segment: tiles, from a wave of targets and of sources on (fewer pairs
  // than that are one launch of the plain kernel either way)
  if (nseg == 1 && nt >= 64 && n >= (nt > kTileRound ? kTileMinSrcMany : kTileMinSrc)) {
    const int64_t tiles = (n + kTileSrc - 1) / kTileSrc;
    const bool two = (nt + 127) / 128 * tiles >= 256;
    const int64_t bx = two ? (nt + 127) / 128 : (nt + 63) / 64;
    int64_t nchunks = std::min((kTileBlocks + bx - 1) / bx, tiles);
    nchunks = std::max<int64_t>(1, std::min(nchunks, part_cap / (8 * nt)));
    const int64_t chunk = (tiles + nchunks - 1) / nchunks * kTileSrc;
    nchunks = (n + chunk - 1) / chunk;
    // a block per target for many chunks, which one thread would add up one
    // after another (64 targets: 16 chunks 21.2 us with threads and 19.0 with
    // blocks, 32 chunks 26.2 and 19.0, 64 chunks 36.5 and 19.0; 8191 targets:
    // 16 chunks 69.5 and 84.5)
    return {DirectPath::kTile, two ? 2 : 1, chunk, nchunks, nchunks > 16};
  }
  // aim for >= 2^16 independent (target, chunk) sums; with part_cap >= 2^19
  // doubles the partials of nt < 2^16 targets always fit at some chunk
  int64_t nchunks = 1, chunk = std::max<int64_t>(n, 1);
  if (nt < 65536 && n > 256) {
    const int64_t want = (65536 + nt - 1) / nt;
    chunk = std::max<int64_t>(256, (n + want - 1) / want);
    nchunks = (n + chunk - 1) / chunk;
    while (nchunks > 1 && nchunks * nt * 8 > part_cap) {
      chunk *= 2;
      nchunks = (n + chunk - 1) / chunk;
    }
  }
  return {DirectPath::kPlain, 1, chunk, nchunks, true};
}

}  // namespace tg

#endif
