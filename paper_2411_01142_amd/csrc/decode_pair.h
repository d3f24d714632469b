// The matrix-core family's kernel for small batches: nothing is planned; the
// `parts` workgroups of each (request, kv head) pair know their blocks from
// their own index.
//
// What bounds a small call is its chain of dependent steps, not its bytes. A
// planned call reads every length, finds its slice, reads the block ids, then
// the tiles, writes a partial, counts it, and one wavefront merges a pair's
// partials, up to 128 of them, in as many dependent rounds as its registers
// need. Here lengths, block ids and query rows are read together, eight
// wavefronts share a workgroup's blocks and merge in LDS, and what is left to
// merge across workgroups is one partial for each of a pair's `parts`, merged
// by a whole workgroup, a head per wavefront.
//
// One compute unit reads about 77 GB/s of tiles however many of its wavefronts
// ask (2 MB by each of 8 workgroups alone: 27 us with 4, 8 or 16 wavefronts,
// one or two tiles a step), which is what `parts` is for. Eight wavefronts
// with one tile in flight measured best: with more prefetch or at the 128
// registers of two workgroups per compute unit (which spills) calls are 10-60 %
// longer; with four, equal when small and 5 % longer at 512 pairs. Chunks of
// 16 blocks: with 32, one request of 877 tokens takes 9.7 us instead of 7.7.
//
// Measured (device time of a call, planned slices -> here, 32 / 8 heads):
// one request of 877 tokens 13.0 -> 7.7 us, of 50021 59 -> 37 us; 4 requests
// of U[64, 512] with 32 / 32 heads 10.0 -> 8.4; 13 of U[100, 1500] 16.5 ->
// 13.8; 64 of U[512, 2048] 65.6 -> 61.0 (128 / 8 heads: 72 -> 59).
#pragma once

#include "decode_common.h"

namespace neo {

// One head of a pair from the partials of `k` workgroups (workspace slots
// slot0 .. slot0 + k - 1): the exact log-sum-exp merge in the order of the
// slots. Lane l owns dims 2l, 2l + 1.
template <int G>
__device__ inline float2 merge_parts(const DecodeParams& p, int32_t slot0, int32_t k, int h,
                                     int lane) {
  constexpr int kBatch = 16;
  float m = kLowest, z = 0.f, x = 0.f, y = 0.f;
  for (int32_t base = 0; base < k; base += kWave) {
    const int32_t cnt = min(kWave, k - base);
    const float got = load_coherent(p.part_lse + (slot0 + base + min(lane, cnt - 1)) * G + h);
    const float lse = lane < cnt ? got : -INFINITY;
    float2 v[kBatch];
    auto load = [&](int32_t i0) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        v[u] = load_coherent2(
            p.part_o + ((size_t)(slot0 + base + min(i0 + u, cnt - 1)) * G + h) * kHeadDim + 2 * lane);
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

// The request of rank r when requests are taken longest first, to within a
// sixteenth of the table's width (ties in index order). Pairs beyond one per
// compute unit run in rounds, and the call ends with the last workgroup: with
// long pairs first the short ones fill the ends. Every workgroup finds its
// request by itself: 64 lengths a wavefront, a ballot for each of 16 classes,
// a scan over the classes' counts; about a microsecond per round. Measured,
// index order / longest first: 64 requests of U[512, 2048] tokens, 8 kv heads
// 57.7 / 55.9 us, of lognormal lengths around 500 33.8 / 28.4, 40 of U[512,
// 2048] 41.3 / 35.9, one of 2000 among 127 of 100 33.5 / 25.0, 128 of nearly
// equal lengths 97.8 / 100.0.
constexpr int kLengthClasses = 16;
__device__ inline int32_t request_of_rank(const DecodeParams& p, int32_t r, int lane, int wv) {
  __shared__ uint64_t members[kLengthClasses * (kMaxOrderedBatch / kWave)];  // [class][64 requests]
  const int32_t groups = (p.batch + kWave - 1) / kWave;
  const int32_t shift = max(0, 28 - __clz(p.mbps));  // mbps >> shift is below 16
  for (int32_t gr = wv; gr < groups; gr += kPairWaves) {
    const int32_t i = gr * kWave + lane;
    const int32_t cls =
        i < p.batch ? kLengthClasses - 1 - (blocks_of(p.lens[i], p.mbps) >> shift) : -1;
    uint64_t mine = 0;
#pragma unroll
    for (int k = 0; k < kLengthClasses; ++k) {
      const uint64_t m = __ballot(cls == k);
      if (lane == k) mine = m;
    }
    if (lane < kLengthClasses) members[lane * groups + gr] = mine;
  }
  __syncthreads();
  const int32_t entries = groups * kLengthClasses;
  int32_t before = 0;
  for (int32_t base = 0; base < entries; base += kWave) {
    const uint64_t m = base + lane < entries ? members[base + lane] : 0;
    const int32_t c = __popcll(m);
    const int32_t incl = before + wave_incl_scan_i32(c);
    const uint64_t hit = __ballot(incl > r);
    if (hit) {
      // The entry holding rank r, and in it the request with that many
      // members below it.
      const int e = __ffsll((unsigned long long)hit) - 1;
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)m, e);
      const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(m >> 32), e);
      const int32_t want =
          r - (__builtin_amdgcn_readlane(incl, e) - __builtin_amdgcn_readlane(c, e));
      const int32_t below = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
      const bool member = ((lane < 32 ? lo : hi) >> (lane & 31)) & 1;
      const uint64_t at = __ballot(member && below == want);
      return (base + e) % groups * kWave + __ffsll((unsigned long long)at) - 1;
    }
    before = __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  return 0;  // not reached: r is below the batch
}

// Workgroup (s, g, b) takes chunks s, s + parts, s + 2 parts, ... of pair
// (b, g); in a chunk wavefront w takes tiles w, w + kPairWaves, ...
template <class F, int G>
__device__ inline void pair_driver(const DecodeParams& p) {
  __shared__ float rows[kPairWaves][G * kHeadDim];  // unnormalised, staged as by F::stage
  __shared__ float ms[kPairWaves][G], ls[kPairWaves][G];
  __shared__ int32_t arrived;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = uniform(threadIdx.x >> 6);
  const int32_t s = blockIdx.x, g = blockIdx.y, parts = gridDim.x;
  const int32_t b =
      p.longest_first ? uniform(request_of_rank(p, blockIdx.z, lane, wv)) : (int32_t)blockIdx.z;
  // Block of this wavefront's i-th tile.
  auto block_of = [&](int32_t i) -> int32_t {
    return kPairChunk * (s + parts * (i / kPairTilesPerWave)) + wv +
           kPairWaves * (i % kPairTilesPerWave);
  };
  // The length, the block ids and the query rows do not wait for one another.
  const int32_t raw = p.lens[b];
  const int32_t* row = p.table + (size_t)b * p.mbps;
  int32_t ids = row[min(block_of(lane), p.mbps - 1)];
  typename F::Q q;
  F::load_q(q, p.q + ((size_t)b * p.hq + g * G) * kHeadDim, lane);
  float* out = p.out + ((size_t)b * p.hq + g * G) * kHeadDim;
  const int32_t L = clamp_len(uniform(raw), p.mbps);
  const int32_t nb = (L + kBlock - 1) / kBlock;
  const int32_t chunks = (nb + kPairChunk - 1) / kPairChunk;
  if (s >= chunks) {  // no block for this workgroup
    if (nb == 0 && s == 0)
      for (int i = threadIdx.x; i < G * kHeadDim; i += kPairWaves * kWave) out[i] = 0.f;
    return;
  }
  // Tiles of this wavefront: all of the workgroup's chunks but the last are whole.
  const int32_t last = (chunks - 1 - s) / parts;
  const int32_t rem = nb - kPairChunk * (s + parts * last);  // blocks from the last chunk on
  const int32_t n = kPairTilesPerWave * last +
                    min(kPairTilesPerWave, max(0, (rem - wv + kPairWaves - 1) / kPairWaves));
  const int shares = last > 0 ? kPairWaves : min(kPairWaves, rem);  // wavefronts with tiles
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
  const int32_t k = min(parts, chunks);  // workgroups with blocks of this pair
  const int32_t pair = b * p.hkv + g;
  const int32_t slot = pair * parts + s;
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
        merge_parts<G>(p, pair * parts, k, h, lane);
}

}  // namespace neo
