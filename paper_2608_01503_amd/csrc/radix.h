// One tile of a stable radix scatter by 8-bit digits (prim.hip: whole arrays; segsort.hip: long segments).
#pragma once

#include "common.h"

namespace lcc {

namespace {

constexpr int RX_TILE = 4096;
constexpr int RX_ITEMS = RX_TILE / BLOCK;  // per thread
constexpr int RX_WAVES = BLOCK / WAVE;

struct RadixLds {
  union {
    uint32_t cnt[RX_WAVES][256];           // items of every digit so far, per wavefront; then first places
    struct { uint64_t k[RX_TILE]; uint32_t v[RX_TILE]; } item;
  };
  uint32_t to[256];                        // position of a digit's run in the output, less its place in the tile
  uint32_t wsum[RX_WAVES];
};

__device__ __forceinline__ void rx_order() {  // the wavefront's own LDS accesses execute in order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// items <= RX_TILE items, load(i, key, val) the i-th; base: where the output run of digit threadIdx.x starts;
// store(at, key, val).  A wavefront takes a quarter of the items, 64 at a time: an item's rank among those of its
// digit is the wavefront's count so far plus the lower lanes with the same digit (ballots over the digit's bits).
// Wavefronts meet only to add up their counts; the items then go through LDS into digit order, so that consecutive
// threads store consecutive positions of a run.
// Bound by memory: 24 bytes an item.  When the whole workgroup ranked 256 items at a time, with four barriers a round and
// the round's loads in between, a pass over 15 M pairs took 186 us, now 88 us (74 us at the rate of a copy); tiles of
// 2048 items 100 us.
template <typename Load, typename Store>
__device__ __forceinline__ void radix_tile(RadixLds& l, int items, int shift, uint32_t base, Load load, Store store) {
  const int t = threadIdx.x, wv = t / WAVE, lane = t & (WAVE - 1);
  const uint64_t below = (1ull << lane) - 1;
  const int rounds = (items + BLOCK - 1) / BLOCK;  // a wavefront's items, in 64s
  const int i0 = wv * rounds * WAVE + lane;
  uint64_t key[RX_ITEMS];
  uint32_t val[RX_ITEMS], at[RX_ITEMS];
#pragma unroll
  for (int r = 0; r < RX_ITEMS; ++r) {
    key[r] = 0;
    val[r] = 0;
    if (r < rounds && i0 + r * WAVE < items) load(i0 + r * WAVE, key[r], val[r]);
  }
#pragma unroll
  for (int k = 0; k < 256 / WAVE; ++k) l.cnt[wv][k * WAVE + lane] = 0;
  rx_order();
#pragma unroll
  for (int r = 0; r < RX_ITEMS; ++r) {
    const bool valid = r < rounds && i0 + r * WAVE < items;
    const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
    uint64_t mask = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      mask &= bit ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(mask & below);
    const uint32_t c = l.cnt[wv][d];
    at[r] = c + rank;
    rx_order();
    if (valid && rank == 0) l.cnt[wv][d] = c + (uint32_t)__popcll(mask);
    rx_order();
  }
  __syncthreads();
  {  // thread t: digit t
    uint32_t c[RX_WAVES], tot = 0;
#pragma unroll
    for (int k = 0; k < RX_WAVES; ++k) { c[k] = l.cnt[k][t]; tot += c[k]; }
    uint32_t inc = tot;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o, WAVE);
      if (lane >= o) inc += y;
    }
    if (lane == WAVE - 1) l.wsum[wv] = inc;
    __syncthreads();
    uint32_t first = inc - tot;
    for (int k = 0; k < wv; ++k) first += l.wsum[k];
    l.to[t] = base - first;
#pragma unroll
    for (int k = 0; k < RX_WAVES; ++k) { l.cnt[k][t] = first; first += c[k]; }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RX_ITEMS; ++r)
    at[r] += l.cnt[wv][(uint32_t)(key[r] >> shift) & 255u];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RX_ITEMS; ++r)
    if (r < rounds && i0 + r * WAVE < items) { l.item.k[at[r]] = key[r]; l.item.v[at[r]] = val[r]; }
  __syncthreads();
  for (int p = t; p < items; p += BLOCK) {
    const uint64_t k = l.item.k[p];
    store((uint32_t)p + l.to[(uint32_t)(k >> shift) & 255u], k, l.item.v[p]);
  }
}

}  // namespace

}  // namespace lcc
