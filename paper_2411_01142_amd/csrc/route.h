// How a decode call is divided: SliceMode and its parameters, from what the
// host knows: the batch, the heads, the table's width (mbps) and the compute
// units. The width bounds the lengths and says little else about them (a table
// is as wide as a program's longest context), so it is used only where it makes
// every batch of that width a good one for the division; what depends on the
// lengths is decided on the device. A caller's slice cap is a cap on wavefronts'
// slices.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "neo_internal.h"

namespace neo {

struct Route {
  SliceMode mode;
  int32_t parts;   // kPairs
  int32_t units;   // kUnits
  int32_t grid_y;  // kUnits, kWhole
};

// Times below: device time of a call with 32 / 8 heads on 256 compute units,
// tables as wide as the longest request where no width is given.
//
// Without slices: up to three (request, kv head) pairs per compute unit (in
// planned slices / so: 96 requests of U[50, 150] tokens 16.5 / 13.3 us, of U[500,
// 3000] 114 / 105, of 500 tokens in 200 columns 39.6 / 36.5). Of a batch that it
// reads, the kernel reads 64 lengths a register of every wavefront, and for three
// rounds of workgroups that is worth it up to kThreeRoundsMaxBatch requests (300
// of 500 tokens, two kv heads, 37.3 / 39.7). With four, short pairs lose where
// the device has to choose (128 requests of U[50, 150], 200 columns, 16.4 / 18.3;
// of U[500, 3000] 147 / 138).
constexpr int32_t kPairsPerCu = 3;
constexpr int32_t kThreeRoundsMaxBatch = 2 * kWave;
//
// A pair of at most kPairShortBlocks blocks is not worth a merge (19 blocks: 6.8
// us by one workgroup, 8.3 by two), and any batch of such pairs suits kPairs.
// Wider tables take it where a workgroup still has at most that many blocks (5
// requests of U[50, 150] tokens: 4.9 us so, 5.6 as kUnits, whose lengths are a
// round trip more; 13 of U[100, 1500], up to 47 blocks each: 13.2 and 12.3), or
// twice as many where pairs outnumber half of the compute units, so that none
// can be cut (32 of U[50, 150]: 6.0 so, 6.6 as kWhole); and with one request,
// whose pairs are equal.
//
// Cutting needs compute units to spare: with up to half of them taken, units of
// at most twice an even share of the blocks are enough (kUnits). With more pairs
// none is cut (kWhole).
constexpr int32_t kMaxCus = 256;
static_assert(2 * kMaxCus <= kWholeMaxBatch && kThreeRoundsMaxBatch <= kWholeMaxBatch &&
                  kMaxCus / 2 <= kUnitMaxBatch,
              "the kernels read that many lengths");

// Head slices need whole groups of four kv heads, and pay once every compute
// unit has a few (request, four heads) pairs with some blocks to stream: below
// that a slice is a part of one or two pairs and the cut pairs' partials all
// cross workgroups, where wave slices merge most of them in LDS. Measured, wave
// / head slices: 128 requests of U[512, 2048] tokens (one pair each) 107.6 /
// 109.4 us; with two, 256 of U[512, 2048] 204.8 / 203.5, of U[1000, 2000] 247.7 /
// 246.6, of U[256, 4096] 350 / 341, lognormal 295.7 / 287.1 (dense caches 314.9
// / 311.1); with four, 512 of U[256, 4096] 697 / 681 (64 / 8 heads 681 / 643).
// How large the gain is depends on the card, whose XCDs are unlike: a lognormal
// batch with two pairs each has also measured 288 / 296.
constexpr int32_t kHeadPairsPerCu = 2;
// The kernel takes wave slices when the batch has fewer positions than this per
// compute unit (a pair of n blocks has n + 1). Wave slices / wave slices found
// out on the device / head slices, by positions: 7 (256 requests of U[10, 60]
// tokens) 16.0 / 17.3 / 19.2 us, 15 (512 of them) 24.7 / 25.9 / 27.6, 19 (256 of
// U[50, 200]) 30.0 / 31.4 / 32.4, 28 (384) 42.1 / 43.3 / 42.6, 30 (1024 of U[10,
// 60]) 44.9 / 46.3 / 45.0, 37 (512 of U[50, 200]) 54.1 / - / 53.3, 52 (256, four
// of them of 16000 tokens) 79.7 / - / 75.6. The host takes wave slices at once
// where the table has no room for more.
constexpr int32_t kHeadPositionsPerCu = 24;
constexpr int32_t kHeadWidthPerCu = 64;

inline Route route(int32_t variant, int32_t max_slices, int32_t batch, int32_t hkv, int32_t mbps,
                   int32_t cus) {
  if (variant != NEO_VARIANT_MFMA || max_slices != 0) return {kWaveSlices, 0, 0, 0};
  const int64_t pairs = (int64_t)batch * hkv;
  if (pairs <= (int64_t)kPairsPerCu * cus && cus <= kMaxCus &&
      (pairs <= 2 * (int64_t)cus || batch <= kThreeRoundsMaxBatch || mbps <= kPairShortBlocks)) {
    const int32_t n = (int32_t)pairs;
    const bool uncut = n > cus / 2;
    if (mbps <= kPairShortBlocks || (uncut && n <= cus && mbps <= 2 * kPairShortBlocks))
      return {kPairs, 1, 0, 0};
    // (With a workgroup for every slice, should the device choose wave slices.)
    const int32_t whole = (cus - 1) / hkv + 1;
    if (uncut) return {kWhole, 0, 0, std::max(batch, whole)};
    const int32_t parts = std::min(cus / n, (mbps - 1) / kPairChunk + 1);
    if (batch == 1 || mbps <= kPairShortBlocks * parts) return {kPairs, parts, 0, 0};
    return {kUnits, 0, cus / hkv, whole};
  }
  if (hkv % kHeadsPerSlice == 0) {
    const int64_t groups = pairs / kHeadsPerSlice;
    if (groups >= (int64_t)kHeadPairsPerCu * cus &&
        groups * mbps >= (int64_t)kHeadWidthPerCu * cus)
      return {kHeadSlices, 0, 0, 0};
  }
  return {kWaveSlices, 0, 0, 0};
}

}  // namespace neo
