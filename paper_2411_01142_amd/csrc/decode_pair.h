// The matrix-core family's kernels for small batches, in which a workgroup of
// eight wavefronts takes one (request, kv head) pair or a part of one.
//
// What bounds a small call is its chain of dependent steps, not its bytes. A
// planned call reads every length, finds its slice, reads the block ids, then
// the tiles, writes a partial, counts it, and one wavefront merges a pair's
// partials, up to 128 of them, in as many dependent rounds as its registers
// need. Here eight wavefronts share a workgroup's blocks and merge in LDS, and
// what is left to merge across workgroups is one partial for each of a pair's
// few, merged by a whole workgroup, a head per wavefront.
//
// Three divisions (the host chooses one, from what it knows):
//  kPairs: the host's own, the same workgroups for every pair. Lengths, block
//    ids and query rows are read together.
//  kUnits: pairs cut into units of one size, found from all lengths.
//  kWhole: one workgroup per pair, if all lengths make that a good division.
// The last two must not depend on the table's width, which says little about
// the lengths. They take wave slices instead where the lengths make their own
// division a bad one: a workgroup with far more than its share of the blocks
// reads them alone while the others are done.
//
// One compute unit reads about 77 GB/s of tiles however many of its wavefronts
// ask (2 MB by each of 8 workgroups alone: 27 us with 4, 8 or 16 wavefronts,
// one or two tiles a step). Eight wavefronts with one tile in flight measured
// best: with more prefetch or at the 128 registers of two workgroups per
// compute unit (which spills) calls are 10-60 % longer; with four, equal when
// small and 5 % longer at 512 pairs. Chunks of 16 blocks: with 32, one request
// of 877 tokens takes 9.7 us instead of 7.7.
//
// Measured (device time of a call, planned slices -> here, 32 / 8 heads):
//  kPairs: one request of 877 tokens 12.8 -> 7.8 us, of 50021 59 -> 36; 4
//    requests of U[64, 512] with 32 / 32 heads 9.6 -> 8.1; 64 of U[50, 150]
//    13.3 -> 9.6.
//  kUnits, tables of 500 blocks: 13 requests of U[100, 1500] 15.9 -> 12.3, 5 of
//    U[50, 150] 8.8 -> 5.6, 5 of 8000 tokens 37.0 -> 30.2, one of 8000 among 12
//    of U[75, 150] 31.3 -> 13.6. (Fixed workgroups for every pair: 14.9, 4.9,
//    30.5 and 23.9.)
//  kWhole: 64 of U[512, 2048] 58 -> 51, 64 of 2048 tokens 89 -> 82, 32 of
//    U[100, 1000] 19.7 -> 15.5, 96 of U[500, 3000] 114 -> 105; 512 of U[256,
//    4096] with 8 / 1 heads 102 -> 90.
//    Where it takes wave slices: one of 4096 among 64 of U[75, 150] 20.7 -> 20.7
//    (whole pairs 41.6), 64 lognormal around 500 33.9 -> 33.8 (44.2).
#pragma once

#include "decode_common.h"

namespace neo {

// One head of a pair from the partials of `k` workgroups, the i-th of them in
// workspace slot slot_of(i): the exact log-sum-exp merge in that order. Lane l
// owns dims 2l, 2l + 1.
template <int G, class SlotOf>
__device__ inline float2 merge_parts(const DecodeParams& p, SlotOf slot_of, int32_t k, int h,
                                     int lane) {
  constexpr int kBatch = 16;
  float m = kLowest, z = 0.f, x = 0.f, y = 0.f;
  for (int32_t base = 0; base < k; base += kWave) {
    const int32_t cnt = min(kWave, k - base);
    const float got = load_coherent(p.part_lse + slot_of(base + min(lane, cnt - 1)) * G + h);
    const float lse = lane < cnt ? got : -INFINITY;
    float2 v[kBatch];
    auto load = [&](int32_t i0) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        v[u] = load_coherent2(
            p.part_o + ((size_t)slot_of(base + min(i0 + u, cnt - 1)) * G + h) * kHeadDim + 2 * lane);
    };
    load(0);
    const float mc = fmaxf(m, wave_max_f32(lse));
    const float rescale = __expf(m - mc);  // 0 on the first round
    const float w = __expf(lse - mc);
    m = mc;
    z = z * rescale + wave_sum_f32(w);
    x *= rescale;
    y *= rescale;
    for (int32_t i0 = 0; i0 < cnt; i0 += kBatch) {
      if (i0 > 0) load(i0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (i0 + u >= cnt) break;
        const float wi = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, w), i0 + u));
        x = fmaf(wi, v[u].x, x);
        y = fmaf(wi, v[u].y, y);
      }
    }
  }
  const float inv = 1.f / z;
  return float2{x * inv, y * inv};
}

// The eight wavefronts of a workgroup over its share of pair (b, g): wavefront
// wv computes tiles 0 .. n - 1, the i-th of them block block_of(i); `ids` holds
// the physical ids of the first 64, one per lane. `shares`: wavefronts with
// tiles (the first ones). The pair has k workgroups with tiles, whose partials
// are in slots slot_of(0) .. slot_of(k - 1), this workgroup's in `slot`.
template <class F, int G, class BlockOf, class SlotOf>
__device__ inline void pair_body(const DecodeParams& p, int32_t b, int32_t g, int32_t L, int32_t n,
                                 int shares, int32_t ids, const typename F::Q& q, BlockOf block_of,
                                 int32_t k, int32_t slot, SlotOf slot_of, int lane, int wv) {
  __shared__ float rows[kPairWaves][G * kHeadDim];  // unnormalised, staged as by F::stage
  __shared__ float ms[kPairWaves][G], ls[kPairWaves][G];
  __shared__ int32_t arrived;
  const int32_t* row = p.table + (size_t)b * p.mbps;
  float* out = p.out + ((size_t)b * p.hq + g * G) * kHeadDim;
  if (n > 0) {
    const size_t blk_stride = (size_t)p.blk_stride;
    int32_t base = 0;  // first tile whose id is in ids
    auto tile_off = [&](int32_t i) -> size_t {
      if (i - base >= kWave) {
        base += kWave;
        ids = row[min(block_of(base + lane), p.mbps - 1)];
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // here, not at the join
      }
      const int32_t id = __builtin_amdgcn_readlane(ids, i - base);
      return (size_t)min((uint32_t)id, (uint32_t)(p.num_blocks - 1)) * blk_stride +
             (size_t)g * kTileElems;
    };
    typename F::State st;
    F::init(st);
    typename F::Tile buf[2];
    typename F::Shared sh;
    {
      const size_t off = tile_off(0);
      F::load_tile(buf[0], p.k + off, p.v + off, true, lane);
    }
    for (int32_t i0 = 0; i0 < n; i0 += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int32_t i = i0 + u;
        if (i >= n) break;
        const size_t off = tile_off(min(i + 1, n - 1));
        F::load_tile(buf[u ^ 1], p.k + off, p.v + off, i + 1 < n, lane);
        F::step(st, buf[u], q, L - block_of(i) * kBlock, p.scale_log2, lane, sh);
      }
    }
    F::stage(st, rows[wv], lane);
    const float lt = sum_over_rows(st.l);
    if (lane < G) {
      ms[wv][lane] = st.m;
      ls[wv][lane] = lt;
    }
  }
  __syncthreads();
  for (int h = wv; h < G; h += kPairWaves) {
    float m = kLowest, l = 0.f, x = 0.f, y = 0.f;
    for (int w = 0; w < shares; ++w) m = fmaxf(m, ms[w][h]);
    for (int w = 0; w < shares; ++w) {
      const float e = __builtin_amdgcn_exp2f(ms[w][h] - m);
      const float2 v =
          *reinterpret_cast<const float2*>(rows[w] + h * kHeadDim + ((2 * lane) ^ (4 * h)));
      l = fmaf(e, ls[w][h], l);
      x = fmaf(e, v.x, x);
      y = fmaf(e, v.y, y);
    }
    const float inv = share_inverse(l, k > 1);
    if (k == 1) {
      *reinterpret_cast<float2*>(out + h * kHeadDim + 2 * lane) = float2{x * inv, y * inv};
    } else {
      store_coherent2(p.part_o + ((size_t)slot * G + h) * kHeadDim + 2 * lane, x * inv, y * inv);
      if (lane == 0) store_coherent(p.part_lse + slot * G + h, (m + __log2f(l)) * kLn2);
    }
  }
  if (k == 1) return;
  // Every wavefront's stores are complete before the workgroup is counted; the
  // last workgroup of the pair merges it and leaves the counter at zero.
  const int32_t pair = b * p.hkv + g;
  wait_all_memory();
  __syncthreads();
  if (threadIdx.x == 0) {
    const int32_t old =
        __hip_atomic_fetch_add(p.counters + pair, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == k - 1)
      __hip_atomic_store(p.counters + pair, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    arrived = old;
  }
  __syncthreads();
  if (arrived != k - 1) return;
  for (int h = wv; h < G; h += kPairWaves)
    *reinterpret_cast<float2*>(out + h * kHeadDim + 2 * lane) =
        merge_parts<G>(p, slot_of, k, h, lane);
}

// The output rows of pair (b, g), which has no tokens.
template <int G>
__device__ inline void zero_pair(const DecodeParams& p, int32_t b, int32_t g) {
  float* out = p.out + ((size_t)b * p.hq + g * G) * kHeadDim;
  for (int i = threadIdx.x; i < G * kHeadDim; i += kPairWaves * kWave) out[i] = 0.f;
}

// kPairs. Workgroup (s, g, b) takes chunks s, s + parts, s + 2 parts, ... of
// pair (b, g); in a chunk wavefront w takes tiles w, w + kPairWaves, ...
template <class F, int G>
__device__ inline void pair_driver(const DecodeParams& p) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = uniform(threadIdx.x >> 6);
  const int32_t s = blockIdx.x, g = blockIdx.y, b = blockIdx.z, parts = gridDim.x;
  // Block of this wavefront's i-th tile.
  auto block_of = [&](int32_t i) -> int32_t {
    return kPairChunk * (s + parts * (i / kPairTilesPerWave)) + wv +
           kPairWaves * (i % kPairTilesPerWave);
  };
  // The length, the block ids and the query rows do not wait for one another.
  const int32_t raw = p.lens[b];
  const int32_t ids = p.table[(size_t)b * p.mbps + min(block_of(lane), p.mbps - 1)];
  typename F::Q q;
  F::load_q(q, p.q + ((size_t)b * p.hq + g * G) * kHeadDim, lane);
  const int32_t L = clamp_len(uniform(raw), p.mbps);
  const int32_t nb = (L + kBlock - 1) / kBlock;
  const int32_t chunks = (nb + kPairChunk - 1) / kPairChunk;
  if (s >= chunks) {  // no block for this workgroup
    if (nb == 0 && s == 0) zero_pair<G>(p, b, g);
    return;
  }
  // Tiles of this wavefront: all of the workgroup's chunks but the last are whole.
  const int32_t last = (chunks - 1 - s) / parts;
  const int32_t rem = nb - kPairChunk * (s + parts * last);  // blocks from the last chunk on
  const int32_t n = kPairTilesPerWave * last +
                    min(kPairTilesPerWave, max(0, (rem - wv + kPairWaves - 1) / kPairWaves));
  const int shares = last > 0 ? kPairWaves : min(kPairWaves, rem);
  const int32_t slot0 = (b * p.hkv + g) * parts;
  pair_body<F, G>(p, b, g, L, n, shares, ids, q, block_of, min(parts, chunks), slot0 + s,
                  [&](int32_t i) { return slot0 + i; }, lane, wv);
}

// Blocks that the busiest workgroup of a call without slices may have beyond an
// even share (`even`) of all blocks before wave slices are the better division.
// It reads them while others are done, at 0.106 us each. Wave slices spend about
// 4 us more on plans and ends, stream an even share about 4 % more slowly, and
// merge a pair of `longest` blocks from its cuts at 32 rows a round trip of
// 0.8 us.
constexpr float kLoneBlocks = 40.f;
constexpr float kLoneBlocksOfEven = 0.125f;
constexpr float kLoneBlocksPerRow = 0.25f;
template <int G>
__device__ inline float lone_slack(const DecodeParams& p, float even, int32_t W, int32_t longest) {
  const float slices =
      (float)slice_count(W, p.min_tiles, p.max_slices, p.slice_quantum, kWaveSlices);
  return kLoneBlocks + kLoneBlocksOfEven * even +
         kLoneBlocksPerRow * G * (float)longest * slices / (float)max(W, 1);
}

// Lengths of the first 64 kSets requests, 64 t + lane in raw[t] (past the batch
// the last one's): straight-line code, since a branch would make the compiler
// wait for what is requested after them. Few sets are worth kernels of their own:
// with room for 512 requests, 64 of U[512, 2048] tokens take 52 us instead of 50.5.
template <int kSets>
__device__ inline void load_lens(const DecodeParams& p, int lane, int32_t* raw) {
#pragma unroll
  for (int t = 0; t < kSets; ++t) raw[t] = p.lens[min(kWave * t + lane, p.batch - 1)];
}

// kUnits: every pair is cut into units of S blocks, the last one shorter, and
// the units of all pairs run at once, one per compute unit. A kv head's units
// are numbered alike, request after request, and workgroup (g, v) takes unit v
// of kv head g.
struct Unit {
  int32_t b, L;
  int32_t first, blocks;  // its blocks: first .. first + blocks - 1
  int32_t unit0, units;   // the units of its pair
};
enum UnitFound { kUnitFound, kNoUnit, kBadDivision };

// Unit v. S is the smallest of 64 sizes that gives at most p.units units (the
// grid has one for every request). Every wavefront finds S and the unit by
// itself from all lengths.
template <int G, int kSets>
__device__ inline UnitFound find_unit(const DecodeParams& p, int32_t v, Unit& u, int lane,
                                      const int32_t* raw) {
  int32_t L[kSets], nb[kSets];
  int32_t sum = 0, most = 0, weights = 0;
#pragma unroll
  for (int t = 0; t < kSets; ++t) {
    L[t] = kWave * t + lane < p.batch ? clamp_len(raw[t], p.mbps) : 0;
    nb[t] = (L[t] + kBlock - 1) / kBlock;
    sum += nb[t];
    most = max(most, nb[t]);
    weights += pair_weight(L[t], p.mbps, kWaveSlices);
  }
  const int32_t all = wave_sum_i32(sum), longest = wave_max_i32(most);
  // A pair of at most kPairShortBlocks blocks is not worth a cut (19 blocks: 6.8
  // us by one workgroup, 8.3 by two); should no size fit, none is cut.
  int32_t S = longest;
  if (longest > kPairShortBlocks) {
    // Sizes from an even share of the blocks up to three of them; number 63 cuts
    // nothing. (The counts are fp32 estimates; the exact one follows.)
    const float share = (float)all / (float)p.units;
    auto size_of = [&](int32_t i) -> int32_t {
      const int32_t blocks = (int32_t)(share + share * (float)i * (1.f / 31.f));
      return max(kUnitBlocksMin, (blocks / kPairWaves + 1) * kPairWaves);
    };
    int32_t i = 0;
#pragma unroll
    for (int32_t step = 32; step > 0; step /= 2) {
      const float per_block = __builtin_amdgcn_rcpf((float)size_of(i + step - 1));
      int32_t count = 0;
#pragma unroll
      for (int t = 0; t < kSets; ++t)
        count += nb[t] <= kPairShortBlocks ? nb[t] > 0 : (int32_t)ceilf((float)nb[t] * per_block);
      if (wave_sum_i32(count) > p.units) i += step;
    }
    S = i < 63 ? min(size_of(i), longest) : longest;
    S = uniform(S);
    const int32_t W = wave_sum_i32(weights) * p.hkv;
    const float even = (float)all * (float)p.hkv / (float)p.cus;
    if (uniform((float)S > even + lone_slack<G>(p, even, W, longest))) return kBadDivision;
  }
  int32_t units[kSets], total;
  for (;;) {
    int32_t c = 0;
#pragma unroll
    for (int t = 0; t < kSets; ++t) {
      units[t] = nb[t] <= max(S, kPairShortBlocks) ? nb[t] > 0 : (nb[t] + S - 1) / S;
      c += units[t];
    }
    total = wave_sum_i32(c);
    if (total <= p.units) break;
    S = longest;  // one unit a pair
  }
  if (v >= total) return kNoUnit;
  int32_t before = 0;
#pragma unroll
  for (int t = 0; t < kSets; ++t) {
    const int32_t incl = before + wave_incl_scan_i32(units[t]);
    const uint64_t hit = __ballot(v < incl && v >= incl - units[t]);
    if (hit) {
      const int e = __ffsll((unsigned long long)hit) - 1;
      u.b = kWave * t + e;
      u.L = __builtin_amdgcn_readlane(L[t], e);
      u.units = __builtin_amdgcn_readlane(units[t], e);
      u.unit0 = __builtin_amdgcn_readlane(incl, e) - u.units;
    }
    before = __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  const int32_t blocks = (u.L + kBlock - 1) / kBlock;
  const int32_t part = u.units == 1 ? blocks : S;
  u.first = (v - u.unit0) * part;
  u.blocks = min(part, blocks - u.first);
  return kUnitFound;
}

// Wavefront w of a unit takes its tiles w, w + kPairWaves, ...
template <class F, int G, int kSets>
__device__ inline void unit_driver(const DecodeParams& p) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = uniform(threadIdx.x >> 6);
  const int32_t g = blockIdx.x, v = blockIdx.y;
  int32_t raw[kSets];
  load_lens<kSets>(p, lane, raw);
  const int32_t own = v < p.batch ? p.lens[v] : 1;
  Unit u;
  const UnitFound found = find_unit<G, kSets>(p, v, u, lane, raw);
  if (found == kBadDivision) {
    __shared__ GroupMerge<G> gm;
    const int32_t index = v * p.hkv + g;
    const int32_t workgroups = (p.max_slices + kWavesPerGroup - 1) / kWavesPerGroup;
    if (index >= workgroups || wv >= kWavesPerGroup) return;
    int32_t len0;
    const SliceInfo si = plan_wave_slice<kFused>(p, index, &len0);
    decode_driver<F, G, 1, kFused>(p, gm, index, workgroups, si, len0);
    return;
  }
  if (own <= 0) zero_pair<G>(p, v, g);  // the grid has a workgroup per pair
  if (found == kNoUnit) return;
  auto block_of = [&](int32_t i) -> int32_t { return u.first + wv + kPairWaves * i; };
  const int32_t ids = p.table[(size_t)u.b * p.mbps + min(block_of(lane), p.mbps - 1)];
  typename F::Q q;
  F::load_q(q, p.q + ((size_t)u.b * p.hq + g * G) * kHeadDim, lane);
  const int32_t n = max(0, (u.blocks - wv + kPairWaves - 1) / kPairWaves);
  pair_body<F, G>(p, u.b, g, u.L, n, min(kPairWaves, u.blocks), ids, q, block_of, u.units,
                  v * p.hkv + g, [&](int32_t i) { return (u.unit0 + i) * p.hkv + g; }, lane, wv);
}

// kWhole: one workgroup per pair, longest first where they run in rounds,
// so that short ones fill the ends (index order / longest first: 64 requests of
// U[512, 2048] tokens, 8 kv heads 57.7 / 55.9 us, 40 of them 41.3 / 35.9).
constexpr int kLengthClasses = 16;
constexpr int kWholeSets = kWholeMaxBatch / kWave;  // of 64 requests
// Of kLoneBlocks, what remains where two pairs follow each other on a compute unit:
// a second start costs about 3 us (264 pairs of 32 blocks each, an even share of
// 33: 21.8 us whole, 19.4 in wave slices).
constexpr float kLoneBlocksTwoRounds = 12.f;
// Three rounds are three starts, worth it from this even share on (96 requests of
// U[50, 150] tokens, 20 blocks a compute unit: 16.5 us in wave slices, 16.8 turned
// to them; of 500 tokens, 96 blocks: 39.5 and 36.6).
constexpr float kEvenBlocksThreeRounds = 32.f;

// The request of rank r, longest first to within a sixteenth of the longest
// (ties in index order): a ballot for each of 16 classes, a scan over the
// classes' counts. blocks: of request 64 wv + lane, or with up to 64 requests
// (kOneSet) of request lane, when no wavefront needs another's ballots.
template <bool kOneSet>
__device__ inline int32_t request_of_rank(const DecodeParams& p, int32_t r, int32_t blocks,
                                          int32_t longest, int lane, int wv) {
  const int32_t groups = kOneSet ? 1 : (p.batch + kWave - 1) / kWave;
  const int32_t gr = kOneSet ? 0 : wv;
  uint64_t mine = 0;  // lane k: the members of class k
  if (gr < groups) {
    const float per_width = 1.f / (float)(longest / kLengthClasses + 1);
    const int32_t cls = gr * kWave + lane < p.batch
                            ? max(0, kLengthClasses - 1 - (int32_t)((float)blocks * per_width))
                            : -1;
#pragma unroll
    for (int k = 0; k < kLengthClasses; ++k) {
      const uint64_t m = __ballot(cls == k);
      if (lane == k) mine = m;
    }
  }
  // Entries of 64 requests in the order of their classes; in the one holding
  // rank r, the request with that many members below it.
  auto find = [&](uint64_t m, int32_t before, int32_t* past) -> int32_t {
    const int32_t c = __popcll(m);
    const int32_t incl = before + wave_incl_scan_i32(c);
    *past = __builtin_amdgcn_readlane(incl, kWave - 1);
    const uint64_t hit = __ballot(incl > r);
    if (!hit) return -1;
    const int e = __ffsll((unsigned long long)hit) - 1;
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)m, e);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(m >> 32), e);
    const int32_t want =
        r - (__builtin_amdgcn_readlane(incl, e) - __builtin_amdgcn_readlane(c, e));
    const int32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
    const bool member = ((lane < 32 ? lo : hi) >> (lane & 31)) & 1;
    const uint64_t at = __ballot(member && below == want);
    return e * kWave + __ffsll((unsigned long long)at) - 1;
  };
  int32_t before = 0;
  if constexpr (kOneSet) {
    return max(0, find(mine, 0, &before)) % kWave;
  } else {
    __shared__ uint64_t members[kLengthClasses * kWholeSets];  // [class][64 requests]
    if (gr < groups && lane < kLengthClasses) members[lane * groups + gr] = mine;
    __syncthreads();
    const int32_t entries = groups * kLengthClasses;
    for (int32_t base = 0; base < entries; base += kWave) {
      const int32_t at = find(base + lane < entries ? members[base + lane] : 0, before, &before);
      if (at >= 0) return (base + at / kWave) % groups * kWave + at % kWave;
    }
    return 0;  // not reached: r is below the batch
  }
}

template <class F, int G, bool kRounds, int kSets>
__device__ inline void whole_driver(const DecodeParams& p) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = uniform(threadIdx.x >> 6);
  const int32_t g = blockIdx.x, r = blockIdx.y;
  auto block_of = [&](int32_t i) -> int32_t { return wv + kPairWaves * i; };
  int32_t w[kPlanRegs] = {}, raw[kPlanRegs] = {};  // as plan_slice takes them
  load_lens<kSets>(p, lane, raw);
  const int32_t index = r * p.hkv + g;  // of the workgroup, for wave slices
  const int32_t wave = index * kWavesPerGroup + wv;
  const int32_t len0 = p.lens[min(wave, p.batch - 1)];
  // In one round pair (r, g) is this workgroup's, and its reads do not wait for
  // the lengths.
  int32_t b = min(r, p.batch - 1), ids = 0;
  typename F::Q q;
  if constexpr (!kRounds) {
    ids = p.table[(size_t)b * p.mbps + min(block_of(lane), p.mbps - 1)];
    F::load_q(q, p.q + ((size_t)b * p.hq + g * G) * kHeadDim, lane);
  }
  int32_t nb[kSets], weights = 0, sum = 0, most = 0, own = 0;
#pragma unroll
  for (int t = 0; t < kSets; ++t) {
    raw[t] = kWave * t + lane < p.batch ? raw[t] : 0;
    nb[t] = blocks_of(raw[t], p.mbps);
    w[t] = pair_weight(raw[t], p.mbps, kWaveSlices);
    weights += w[t];
    sum += nb[t];
    most = max(most, nb[t]);
    if (kSets == 1 || t == wv) own = nb[t];
  }
  const int32_t W = wave_sum_i32(weights) * p.hkv;
  const int32_t longest = wave_max_i32(most);
  const float even = (float)wave_sum_i32(sum) * (float)p.hkv / (float)p.cus;
  bool whole = (float)longest <= even + lone_slack<G>(p, even, W, longest);
  if constexpr (kRounds) {
    // Two pairs of more than half of what a compute unit may have must not follow
    // each other on one, nor three of more than a third.
    const int32_t pairs = p.batch * p.hkv;
    const bool two = pairs <= 2 * p.cus;
    const float may = even + kLoneBlocksOfEven * even + (two ? kLoneBlocksTwoRounds : 0.f);
    for (int32_t k = 1; k * p.cus < pairs; ++k) {
      int32_t larger = 0;
#pragma unroll
      for (int t = 0; t < kSets; ++t)
        larger += __popcll(__ballot((float)nb[t] * (float)(k + 1) > may));
      whole = whole && larger * p.hkv <= k * p.cus;
    }
    whole = whole && (two || even >= kEvenBlocksThreeRounds);
  }
  if (uniform(whole)) {
    if (r >= p.batch) return;
    int32_t len;
    if constexpr (kRounds) {
      // (Short pairs are not worth an order: 64 requests of U[50, 150] tokens 9.7
      // us in index order, 11.7 longest first.)
      if (longest > kPairShortBlocks)
        b = uniform(request_of_rank<kSets == 1>(p, r, own, longest, lane, wv));
      len = p.lens[b];
      ids = p.table[(size_t)b * p.mbps + min(block_of(lane), p.mbps - 1)];
      F::load_q(q, p.q + ((size_t)b * p.hq + g * G) * kHeadDim, lane);
    } else {
      len = p.lens[b];
    }
    const int32_t L = clamp_len(uniform(len), p.mbps);
    const int32_t blocks = (L + kBlock - 1) / kBlock;
    if (blocks == 0) {
      zero_pair<G>(p, b, g);
      return;
    }
    const int32_t n = max(0, (blocks - wv + kPairWaves - 1) / kPairWaves);
    pair_body<F, G>(p, b, g, L, n, min(kPairWaves, blocks), ids, q, block_of, 1, 0,
                    [](int32_t) { return 0; }, lane, wv);
    return;
  }
  const int32_t workgroups = (p.max_slices + kWavesPerGroup - 1) / kWavesPerGroup;
  if (index >= workgroups || wv >= kWavesPerGroup) return;
  __shared__ GroupMerge<G> gm;
  const SliceInfo si = plan_slice<kWaveSlices>(p, wave, lane, W, w, raw);
  decode_driver<F, G, 1, kFused>(p, gm, index, workgroups, si, len0);
}

}  // namespace neo
