// The matrix-core family's driver for head slices: a workgroup's slice is a run
// of (request, four kv heads) pairs, and its four wavefronts walk the same
// blocks together, one head each.
//
// Why: HBM bound. The four tiles that a step reads of K (and of V) are one
// 16 KiB run of a block, read by one compute unit at one time, instead of four
// 4 KiB reads at unrelated times. A read probe of 4.6 GB of interleaved caches
// with shuffled blocks measured 7.17 TB/s for one slice per wavefront, 7.33
// for the four heads of a block by one workgroup, 7.41 with a barrier per step
// that keeps the four wavefronts at the same block (two steps in flight: 7.31;
// eight heads by eight wavefronts: 7.33; dense caches: 6.96 one slice per
// wavefront, 6.86 here).
//
// A slice's tiles, whatever pairs they belong to, are one sequence: while a
// tile is computed the next one's loads are in flight, also across the end of
// a pair, and the next pair's query rows and block ids were requested a pair
// earlier. So a pair's end costs its arithmetic, not a drained prefetch and
// three dependent round trips.
//
// The wait counts are the compiler's: on gfx9 loads and stores share one
// in-order counter, and where two paths join it assumes the path with fewer
// operations in flight. So the loop is written as chunks (at most 64 tiles of
// one pair): a chunk's first step follows the chunk switch in straight-line
// code, where the loads of the switch are counted exactly and not waited for;
// the steps after it are the plain loop, in which they are a step old and
// complete.
//
// Measured (one layer, interleaved caches, time of a call; one slice per
// wavefront with results written one by one -> here): 64 / 8 heads, batch 512,
// U[256, 4096]: 681 -> 643 us; 32 / 8 heads, 8 x 32768 among 1016 x U[16, 256]
// tokens: 272 -> 261 us; dense caches, 256 lognormal lengths: 286 -> 282 us.
#pragma once

#include "decode_common.h"

namespace neo {

// s_waitcnt vmcnt(12): everything but the newest tile's loads.
constexpr int kWaitVmcnt12 = 0x0F7C;

// A finished [G][128] fp32 result waits in LDS and leaves in a batch with
// others. Results written one by one, each as soon as it was ready, cost far
// more than their bytes: HBM turns from reading to writing and back for every
// few kilobytes. Measured on 4.6 GB of KV with 67 MB of results (2048
// requests of 544 tokens, 64 / 8 heads): 732 us written at once, 668 us in
// batches with nontemporal whole-line stores (696 us with plain ones), 639 us
// not written at all.
//
// Slots per wavefront: what 128 KiB of LDS hold, one of them kept for staging
// partials.
constexpr int stash_slots(int G) {
  const int n = 128 * 1024 / (kWavesPerGroup * G * kHeadDim * 4) - 1;
  return n > 16 ? 16 : n;
}

// Family provides: Tile, State, Q, Shared; load_q, init, load_tile, step,
// normalise, stage, merge_in_place.
template <class F, int G, Schedule kSched>
__device__ inline void stream_driver(const DecodeParams& p) {
  constexpr bool kMergeHere = kSched == kFused;  // merge cut pairs in this kernel
  constexpr SliceMode kMode = kHeadSlices;
  constexpr int kStash = stash_slots(G);
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = uniform(threadIdx.x >> 6);
  const int wave = blockIdx.x * kWavesPerGroup + wv;
  const int slice = blockIdx.x;
  const int32_t len0 = wave < p.batch ? p.lens[wave] : 0;
  __shared__ float stash[kWavesPerGroup][(kStash + 1) * G * kHeadDim];
  __shared__ int32_t stash_row[kWavesPerGroup][kStash];  // first output row of each slot
  int32_t w[kPlanRegs], raw[kPlanRegs];
  const int32_t W = kSched == kStaged ? p.hdr->total : plan_total<kMode>(p, lane, w, raw);
  if (W < p.head_positions) {
    // Too little for head slices: wave slices, merged in this kernel under every
    // schedule. (The two-kernel launch's combine reads the total alone then.)
    if (kSched == kTwoKernel && wave == 0 && lane == 0) p.hdr->total = W;
    static_assert(sizeof(GroupMerge<G>) <= sizeof(stash), "the merge state takes the stash's place");
    // (Planned anew: reusing the lengths above keeps them in registers and costs
    // the loop below 0.5 %.)
    const SliceInfo si = plan_in_wave<kWaveSlices>(p, wave, lane);
    decode_driver<F, G, 1, kFused>(p, *reinterpret_cast<GroupMerge<G>*>(&stash[0][0]), blockIdx.x,
                                   gridDim.x, si, len0);
    return;
  }
  const SliceInfo si = kSched == kStaged ? read_plan<kMode>(p, slice)
                                         : plan_slice<kMode>(p, slice, lane, W, w, raw);
  zero_empty_rows(p, wave, gridDim.x * kWavesPerGroup, lane, len0);
  if (kSched == kTwoKernel && lane == 0 && wv == 0) record_plan<kMode>(p, si, slice);
  // The plan is the workgroup's: its wavefronts leave together, here and
  // below, and take the same steps (and barriers).
  if ((slice << slice_shift(kMode)) >= si.geo.n) return;

  const Cuts cuts = make_cuts(si.geo, kMode, wv);
  const int32_t hk = pairs_per_request(p.hkv, kMode);
  const size_t blk_stride = (size_t)p.blk_stride;
  auto kv_head = [&](int32_t pair) -> int32_t { return pair * kHeadsPerSlice + wv; };

  // Lengths of 64 requests from lens_base on, one per lane (read beside the
  // first block ids and used after the first tile is requested).
  int32_t lens_base = si.b;
  int32_t lens_v = p.lens[min(lens_base + lane, p.batch - 1)];
  auto length_of = [&](int32_t b) -> int32_t {
    if (b - lens_base >= kWave) {
      lens_base = b;
      lens_v = p.lens[min(b + lane, p.batch - 1)];
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // here, not at the join
    }
    return clamp_len(__builtin_amdgcn_readlane(lens_v, b - lens_base), p.mbps);
  };

  // The segment being computed: tiles [j, jend) of pair g of request b, whose
  // nb blocks start at position first; and the slice's next segment (none:
  // nend == 0), which always starts at block 0.
  int32_t b = si.b, g = si.g;
  int32_t L = si.L >= 0 ? si.L : length_of(b);
  int32_t nb = (L + kBlock - 1) / kBlock;
  int32_t first = si.s0 - si.x + pair_cost(nb, kMode);
  int32_t j = max(0, si.x - pair_cost(nb, kMode));
  int32_t jend = min(nb, si.s1 - first);
  if (jend <= j) return;  // the slice ends before this pair's next tile
  int32_t nxb = 0, nxg = 0, nxL = 0, nxnb = 0, nxfirst = 0, nend = 0;
  auto find_next = [&]() {
    const int32_t pos = first + nb;
    nend = 0;
    nxb = b;
    nxg = g + 1;
    nxL = L;
    nxnb = nb;
    if (nxg == hk) {
      nxg = 0;
      ++nxb;
      if (pos >= si.s1) return;
      for (; nxb < p.batch; ++nxb) {  // past requests with no tokens
        nxL = length_of(nxb);
        nxnb = (nxL + kBlock - 1) / kBlock;
        if (nxnb > 0) break;
      }
      if (nxb >= p.batch) return;
    }
    nxfirst = pos + pair_cost(nxnb, kMode);
    nend = max(0, min(nxnb, si.s1 - nxfirst));
  };

  typename F::Q q, qn;
  F::load_q(q, p.q + ((size_t)b * p.hq + kv_head(g) * G) * kHeadDim, lane);
  // Block ids, one per lane: of the chunk being computed, and of the one after it.
  int32_t cb = j, cend = min(jend, j + kWave);
  int32_t ids = p.table[(size_t)b * p.mbps + min(cb + lane, jend - 1)];
  int32_t ids_next, gnext;
  bool more_next;
  auto load_next_ids = [&]() {
    const bool same = cend < jend;
    more_next = same || nend > 0;
    gnext = same ? g : nxg;
    const int32_t row = same || nend == 0 ? b : nxb;
    const int32_t at = same ? min(cend + lane, jend - 1) : min(lane, max(nend, 1) - 1);
    ids_next = p.table[(size_t)row * p.mbps + at];
  };
  auto load_next_q = [&]() {
    const int32_t qb = nend > 0 ? nxb : b, qg = nend > 0 ? nxg : g;
    F::load_q(qn, p.q + ((size_t)qb * p.hq + kv_head(qg) * G) * kHeadDim, lane);
  };

  typename F::Tile t0, t1;
  typename F::State st;
  F::init(st);
  auto issue = [&](typename F::Tile& t, int32_t id, int32_t pair, bool valid) {
    const size_t off = (size_t)min((uint32_t)id, (uint32_t)(p.num_blocks - 1)) * blk_stride +
                       (size_t)kv_head(pair) * kTileElems;
    F::load_tile(t, p.k + off, p.v + off, valid, lane);
  };
  issue(t0, __builtin_amdgcn_readlane(ids, 0), g, true);
  find_next();
  load_next_ids();
  load_next_q();

  // Slices holding a cut pair's first and last tiles; computed when a segment
  // starts, while its first tile is on its way.
  int32_t c0 = 0, c1 = 0;
  // Last segment cut with exactly one later slice, which handles its share of
  // the pair first: if it has already arrived, this slice will be the last,
  // so it merges straight from registers (no partial of its own, no atomic,
  // one round trip for the other partial). The counter is read a few tiles
  // before the segment ends (late enough that the next slice has usually
  // finished its share, early enough that the read's latency hides behind
  // the remaining tiles) and only looked at after the tiles.
  int32_t seen = 0;
  // An arrival at a cut pair that this slice entered in its middle, counted a
  // step after its partial was stored (by then the stores have completed).
  struct Cut {
    int32_t b, g, first, c0, c1;
  } early{};
  bool early_cut = false, arrive_due = false;
  int32_t early_old = 0;
  int32_t event = -1;  // tile at which one of the two happens
  int32_t check_at = -1;
  auto start_segment = [&]() {
    if (j > 0 || jend < nb) {
      c0 = uniform(cuts.holder(first));
      c1 = uniform(cuts.holder(first + nb - 1));
    }
    check_at = -1;
    seen = 0;
    if constexpr (kMergeHere) {
      if (j == 0 && jend < nb && c1 == slice + 1) check_at = max(j + 2, jend - kMergeCheckAhead);
    }
    event = arrive_due ? j + 1 : check_at;
  };
  start_segment();
  auto arrive_early = [&]() {
    early_old = count_arrival(p, cuts.id(early.c0), lane);
    arrive_due = false;
  };

  __shared__ typename F::Shared shared[kWavesPerGroup];
  int32_t jj = j;
  // One step: the next tile's loads go out, then tile jj is computed.
  auto step = [&](typename F::Tile& cur, typename F::Tile& nxt) {
    __builtin_amdgcn_s_barrier();
    const bool in_chunk = jj + 1 < cend;
    const int32_t id = in_chunk ? __builtin_amdgcn_readlane(ids, (jj + 1 - cb) & (kWave - 1))
                                : __builtin_amdgcn_readlane(ids_next, 0);
    issue(nxt, id, in_chunk ? g : gnext, in_chunk || more_next);
    if constexpr (kMergeHere) {
      if (jj == event) {
        if (arrive_due) {
          // The partial was stored before tile jj's loads were issued.
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          __builtin_amdgcn_s_waitcnt(kWaitVmcnt12);
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          arrive_early();
          event = check_at;
        } else {
          seen = __hip_atomic_load(p.counters + cuts.id(slice), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    F::step(st, cur, q, L - jj * kBlock, p.scale_log2, lane, shared[wv]);
    ++jj;
  };

  int32_t stashed = 0;
  auto flush = [&]() {
    wave_sync_lds();
    for (int s = 0; s < stashed; ++s) {
      const float* slot = &stash[wv][s * G * kHeadDim];
      f32x4_t* rows =
          reinterpret_cast<f32x4_t*>(p.out + (size_t)uniform(stash_row[wv][s]) * kHeadDim);
#pragma unroll
      for (int i = 0; i < (G * 32 + kWave - 1) / kWave; ++i) {
        const int w = i * kWave + lane;  // 16-byte word
        if (G * 32 % kWave == 0 || w < G * 32)
          __builtin_nontemporal_store(
              *reinterpret_cast<const f32x4_t*>(slot + 4 * (w ^ (w >> 5))), rows + w);
      }
    }
    wave_sync_lds();
    stashed = 0;
  };
  auto put_result = [&](int32_t row) {
    F::stage(st, &stash[wv][stashed * G * kHeadDim], lane);
    stash_row[wv][stashed] = row;  // every lane: the same value
    if (++stashed == kStash) flush();
  };
  // A partial leaves as whole lines too, a row per store.
  auto put_partial = [&](int32_t slot, float lse) {
    float* tmp = &stash[wv][kStash * G * kHeadDim];
    wave_sync_lds();
    F::stage(st, tmp, lane);
    wave_sync_lds();
    float* rows = p.part_o + (size_t)slot * G * kHeadDim;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float2 v = *reinterpret_cast<const float2*>(tmp + h * kHeadDim + ((2 * lane) ^ (4 * h)));
      store_coherent2(rows + h * kHeadDim + 2 * lane, v.x, v.y);
    }
    if (lane < G) store_coherent(p.part_lse + slot * G + lane, lse);
  };
  // The computed segment's result.
  auto finish_segment = [&]() {
    const int32_t kvh = kv_head(g);
    const int32_t row = b * p.hq + kvh * G;
    const bool whole = j == 0 && jend == nb;
    const float lse = F::normalise(st, !whole);
    if (whole) {
      put_result(row);
      return;
    }
    if constexpr (kMergeHere) {
      if (__builtin_amdgcn_readfirstlane(seen) == 1) {
        if (lane == 0)
          __hip_atomic_store(p.counters + cuts.id(slice), 0, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        const int slot = cuts.slot_u(slice + 1, first);
        F::merge_in_place(st, lse, p.part_o + (size_t)slot * G * kHeadDim, p.part_lse + slot * G,
                          lane);
        put_result(row);
        return;
      }
    }
    put_partial(partial_slot(cuts.id(slice), si.s0, first), lse);
    if constexpr (kMergeHere) {
      // Count the partial, a step later if more of the slice is to come; the
      // last one to arrive merges the pair.
      if (nend > 0) {
        early = Cut{b, kvh, first, c0, c1};
        early_cut = arrive_due = true;
      } else {
        flush();
        if (arrive_last(p, cuts.id(c0), c1 - c0 + 1, lane))
          merge_cut<G>(p, b, kvh, first, c0, c1, cuts, lane);
      }
    }
  };
  // After a chunk's last tile: false when the slice is done.
  auto next_chunk = [&]() -> bool {
    if (jj == jend) {
      if constexpr (kMergeHere) {
        if (arrive_due) {  // a segment of one tile came after the cut one
          wait_all_memory();
          arrive_early();
        }
      }
      finish_segment();
      if (nend == 0) return false;
      b = nxb;
      g = nxg;
      L = nxL;
      nb = nxnb;
      first = nxfirst;
      j = jj = cb = 0;
      jend = nend;
      q = qn;
      F::init(st);
      find_next();
      start_segment();
    } else {
      cb = cend;
    }
    ids = ids_next;
    cend = min(jend, cb + kWave);
    load_next_q();
    load_next_ids();
    return true;
  };

  bool odd = false;  // which buffer holds tile jj
  do {
    if (!odd) {
      step(t0, t1);
      for (;;) {
        odd = true;
        if (jj == cend) break;
        step(t1, t0);
        odd = false;
        if (jj == cend) break;
        step(t0, t1);
      }
    } else {
      step(t1, t0);
      for (;;) {
        odd = false;
        if (jj == cend) break;
        step(t0, t1);
        odd = true;
        if (jj == cend) break;
        step(t1, t0);
      }
    }
  } while (next_chunk());
  flush();

  if constexpr (kMergeHere) {
    if (early_cut && is_last(p, cuts.id(early.c0), early.c1 - early.c0 + 1, early_old, lane))
      merge_cut<G>(p, early.b, early.g, early.first, early.c0, early.c1, cuts, lane);
  }
}

}  // namespace neo
