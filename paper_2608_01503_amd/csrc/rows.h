// Row helpers shared by the per-bucket kernels of the local move (lm.hip) and the team kernels (team.hip):
// reductions over groups of lanes, the decision rule, the afterburner's order and pattern, the LDS hash.
#pragma once

#include "common.h"

namespace lcc {

namespace {

// ---------------------------------------------------------------------------------------------------------
// reductions over a group of G lanes (G <= 64: shuffles; G == BLOCK-sized: shuffles + LDS)
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ bool better(int64_t s2, int32_t c2, int64_t s, int32_t c) {
  return s2 > s || (s2 == s && c2 < c);
}

// Partner of butterfly step K (K = 0, 1, ...) inside aligned groups of G lanes.  Groups of at most 16 lanes
// use DPP lane moves (register to register, no LDS): two quad permutations (lane ^ 1, lane ^ 2), the row half
// mirror (lane i of an 8-lane half-row <-> lane 7 - i) and the row mirror (i <-> 15 - i).  The mirror partners
// are not xor partners, but each step pairs every lane with one in the other half of its 2^(K+1)-lane block,
// whose lanes all hold the same value after the earlier steps: an all-reduction of a commutative and
// associative operation gets the same result.  The steps between rows of 16 swap rows (permlane16_swap: the odd rows
// of its first operand with the even rows of its second, permlane32_swap the same with halves), also without LDS:
// with shuffles, two LDS permutes per step and 64-bit value, the chain of a 32-lane argmax was about 600 cycles.
constexpr int DPP_GROUP_STEP[4] = {0xB1, 0x4E, 0x141, 0x140};

template <int G, int K>
__device__ __forceinline__ int32_t gx32(int32_t x) {
  static_assert((1 << K) < G && G <= WAVE, "a step inside the group");
  if constexpr (K < 4) {
    return __builtin_amdgcn_update_dpp(0, x, DPP_GROUP_STEP[K], 0xf, 0xf, false);
  } else if constexpr (K == 4) {
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
    return (int32_t)((threadIdx.x & 16) ? r[0] : r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    return (int32_t)((threadIdx.x & 32) ? r[0] : r[1]);
  }
}
template <int G, int K>
__device__ __forceinline__ int64_t gx64(int64_t x) {
  const int32_t lo = gx32<G, K>((int32_t)(uint32_t)(uint64_t)x);
  const int32_t hi = gx32<G, K>((int32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}

// Lane K of every aligned group of G lanes (G = 4: quad permutation; 8 and 16: row broadcasts; else shuffle).
template <int G, int K>
__device__ __forceinline__ int32_t gbcast32(int32_t x) {
  if constexpr (G == 4) {
    return __builtin_amdgcn_update_dpp(0, x, K | (K << 2) | (K << 4) | (K << 6), 0xf, 0xf, false);
  } else if constexpr (G == 8) {
    const int32_t lo = __builtin_amdgcn_update_dpp(0, x, 0x150 + K, 0xf, 0xf, false);      // row_newbcast:K
    const int32_t hi = __builtin_amdgcn_update_dpp(0, x, 0x150 + K + 8, 0xf, 0xf, false);  // row_newbcast:K+8
    return (threadIdx.x & 8) ? hi : lo;
  } else if constexpr (G == 16) {
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + K, 0xf, 0xf, false);
  } else {
    return __shfl(x, K, G);
  }
}

template <int G, int K = 0>
__device__ __forceinline__ void argmax_steps(int64_t& s, int32_t& c) {
  if constexpr ((1 << K) < G) {
    const int64_t s2 = gx64<G, K>(s);
    const int32_t c2 = gx32<G, K>(c);
    if (better(s2, c2, s, c)) { s = s2; c = c2; }
    argmax_steps<G, K + 1>(s, c);
  }
}
template <int G, int K = 0>
__device__ __forceinline__ int64_t sum_steps(int64_t x) {
  if constexpr ((1 << K) < G) return sum_steps<G, K + 1>(x + gx64<G, K>(x));
  else return x;
}

template <int G>
__device__ __forceinline__ void argmax_reduce(int64_t& s, int32_t& c) {
  if constexpr (G <= WAVE) {
    argmax_steps<G>(s, c);
  } else {
    __shared__ int64_t ss[G / WAVE];
    __shared__ int32_t cc[G / WAVE];
    argmax_reduce<WAVE>(s, c);
    int wv = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0) { ss[wv] = s; cc[wv] = c; }
    __syncthreads();
    s = ss[0]; c = cc[0];
#pragma unroll
    for (int k = 1; k < G / WAVE; ++k)
      if (better(ss[k], cc[k], s, c)) { s = ss[k]; c = cc[k]; }
    __syncthreads();
  }
}

template <int G>
__device__ __forceinline__ int64_t sum_reduce(int64_t x) {
  if constexpr (G <= WAVE) {
    return sum_steps<G>(x);
  } else {
    __shared__ int64_t ss[G / WAVE];
    x = sum_reduce<WAVE>(x);
    int wv = threadIdx.x / WAVE;
    if ((threadIdx.x & (WAVE - 1)) == 0) ss[wv] = x;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int k = 0; k < G / WAVE; ++k) t += ss[k];
    __syncthreads();
    return t;
  }
}

// Destination and candidacy of one vertex from its own score and its best neighbouring cluster
// (Alg. 2: argmax, the empty-cluster rule, the temperature rule w'(v,D) >= (1 - phi) w'(v,C[v])).
// strict != 0 replaces the temperature rule by "the move strictly improves" (node optimality, Sec. V-A).
struct Verdict {
  int32_t d;
  int64_t delta;
  bool cand;
};
__device__ __forceinline__ Verdict decide(int64_t scur, int64_t sbest, int32_t cbest, uint32_t pa, uint32_t pb,
                                          int strict) {
  int32_t d;
  int64_t sd;
  if (scur < 0 && (cbest == INT32_MAX || sbest < 0)) {
    d = D_EMPTY;
    sd = 0;
  } else if (cbest == INT32_MAX) {
    return {D_NONE, 0, false};
  } else {
    d = cbest;
    sd = sbest;
  }
  int64_t delta = sd - scur;
  bool cand = strict ? (delta > 0) : ((__int128)pb * sd >= (__int128)(pb - pa) * scur);
  return {cand ? d : D_NONE, cand ? delta : 0, cand};
}

__device__ __forceinline__ uint32_t hslot(int32_t c, int bits) {
  return ((uint32_t)c * 2654435761u) >> (32 - bits);
}

__device__ __forceinline__ int ceil_log2(int64_t x) {
  int b = 0;
  while (((int64_t)1 << b) < x) ++b;
  return b;
}

// log2 of the LDS hash capacity for a row of degree d: pow2ceil(2 d) << shift slots (at least 2), at most the
// kernel's table of `slots`; the bucket bounds keep 2 d <= slots, so the load factor never exceeds 1/2
__device__ __forceinline__ int table_bits(int64_t d, int shift, int slots) {
  int bits = ceil_log2(2 * d);
  if (bits < 1) bits = 1;
  bits += shift;
  const int cap = ceil_log2(slots);
  return bits < cap ? bits : cap;
}

// Sum of x over the 64 lanes of a fully active wavefront, returned to every lane.  A row-local Hillis-Steele
// scan by DPP row shifts (1, 2, 4, 8), then the two row broadcasts carry rows 0-2 into rows 1-3, so lane 63
// holds the total: register-to-register moves only, no LDS round trips.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  int v = (int)x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ void lds_insert(int32_t* hk, uint32_t* hv, int bits, int32_t c, uint32_t wt) {
  const uint32_t mask = (1u << bits) - 1;
  uint32_t h = hslot(c, bits);
  for (uint32_t probe = 0; probe <= mask; ++probe) {  // the table has room for every distinct key
    int32_t prev = atomicCAS(&hk[h], -1, c);
    if (prev == -1 || prev == c) { atomicAdd(&hv[h], wt); return; }
    h = (h + 1) & mask;
  }
}

struct Best {
  int64_t s;
  int32_t c;
  int64_t own;
  int64_t np;
};

__device__ __forceinline__ Best best_init() { return Best{INT64_MIN, INT32_MAX, 0, 0}; }

// reduction of Best over G lanes (G <= 64) or a block of G threads; the result is valid in lane / thread 0
template <int G, int K = 0>
__device__ __forceinline__ void best_steps(Best& r) {
  if constexpr ((1 << K) < G) {
    const int64_t s2 = gx64<G, K>(r.s);
    const int32_t c2 = gx32<G, K>(r.c);
    r.own += gx64<G, K>(r.own);
    r.np += gx64<G, K>(r.np);
    if (better(s2, c2, r.s, r.c)) { r.s = s2; r.c = c2; }
    best_steps<G, K + 1>(r);
  }
}

template <int G>
__device__ __forceinline__ void best_reduce(Best& r) {
  constexpr int WD = G < WAVE ? G : WAVE;
  best_steps<WD>(r);
  if constexpr (G > WAVE) {
    __shared__ Best sb[G / WAVE];
    if ((threadIdx.x & (WAVE - 1)) == 0) sb[threadIdx.x / WAVE] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 1; k < G / WAVE; ++k) {
        r.own += sb[k].own;
        r.np += sb[k].np;
        if (better(sb[k].s, sb[k].c, r.s, r.c)) { r.s = sb[k].s; r.c = sb[k].c; }
      }
    }
  }
}

// Every lane of the group sees every lane's (cluster, weight) in turn and sums the weights of its own cluster;
// a lane stays leader when no earlier lane holds its cluster.
template <int G, int K = 0>
__device__ __forceinline__ void pair_sweep(int32_t c, int32_t wt, bool has, int gl, int64_t& acc, bool& leader) {
  if constexpr (K < G) {
    const int32_t ck = gbcast32<G, K>(c);
    const int32_t wk = gbcast32<G, K>(wt);
    if (has && ck == c) {
      acc += wk;
      if (K < gl) leader = false;
    }
    pair_sweep<G, K + 1>(c, wt, has, gl, acc, leader);
  }
}

// Orders a wavefront's own LDS accesses around a phase change of its private table: every LDS operation of
// the wavefront has completed (lgkmcnt 0) and the compiler moves no memory access across.  No other wavefront
// is involved, so no workgroup barrier.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt left at their maximum
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sums of equal keys within groups of G lanes of a wavefront (one entry per lane), by electing a leader lane per
// key in LDS: every open lane writes (key, lane) to the slot its key hashes to, reads the slot back, and if its
// key won, adds its weight to the sum of the lane that wrote last; the lanes of keys that lost hash again.  Every
// round settles at least one key per contested slot, so the rounds end (one or two as a rule).  An all-pairs
// sweep of 32 lanes costs 64 LDS permutes and about 350 vector instructions per wavefront whatever the keys are;
// this costs about 8 LDS operations and 40 instructions.
// A wavefront's LDS operations execute in order, so only the compiler is kept from reordering them.
// E entries per lane: groups of at most G E entries.
template <int E>
struct LeaderLds {
  uint64_t slot[2 * WAVE * E];
  uint32_t sum[WAVE * E];
};
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// On return leader[k] is set for one entry per distinct key (among those with has[k]), and wt[k] is that key's sum.
template <int G, int E>
__device__ __forceinline__ void leader_sum(LeaderLds<E>& l, int lane, const int32_t (&key)[E], uint32_t (&wt)[E],
                                           const bool (&has)[E], bool (&leader)[E]) {
  constexpr int BITS = G * E == 8 ? 4 : G * E == 16 ? 5 : G * E == 32 ? 6 : G * E == 64 ? 7 : 8;  // 2 G E slots per group
  static_assert((2 * G * E) == (1 << BITS), "slots of a group");
  const int base = 2 * E * (lane & ~(G - 1));
  uint32_t h[E];
  bool open[E];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    h[k] = (uint32_t)key[k] * 2654435761u;
    open[k] = has[k];
    leader[k] = false;
    l.sum[lane * E + k] = 0;
  }
  for (;;) {
    bool any = open[0];
#pragma unroll
    for (int k = 1; k < E; ++k) any = any || open[k];
    if (!__ballot(any)) break;
#pragma unroll
    for (int k = 0; k < E; ++k)
      if (open[k]) l.slot[base + (int)(h[k] >> (32 - BITS))] = (uint64_t)(uint32_t)(lane * E + k) << 32 | (uint32_t)key[k];
    lds_order();
#pragma unroll
    for (int k = 0; k < E; ++k) {
      if (open[k]) {
        const uint64_t got = l.slot[base + (int)(h[k] >> (32 - BITS))];
        if ((int32_t)(uint32_t)got == key[k]) {
          const int w = (int)(got >> 32);
          atomicAdd(&l.sum[w], wt[k]);
          leader[k] = w == lane * E + k;
          open[k] = false;
        }
      }
      h[k] = (h[k] ^ h[k] >> 15) * 2246822519u + 3266489917u;
    }
    lds_order();
  }
#pragma unroll
  for (int k = 0; k < E; ++k) wt[k] = l.sum[lane * E + k];
}

// u and v are graph-local ids (the level id minus the graph's first id in a union of graphs).
__device__ __forceinline__ bool before(int32_t u, int64_t du, int32_t v, int64_t dv, int64_t tie) {
  const __int128 diff = (__int128)du - dv;  // two deltas below 2^63 each: their difference needs 65 bits
  const __int128 ad = diff < 0 ? -diff : diff;
  if (ad <= tie) return fmix64((uint64_t)(uint32_t)u) < fmix64((uint64_t)(uint32_t)v);
  return diff > 0;
}

__device__ __forceinline__ int ab_pattern(int32_t cv, int32_t dv, int32_t cu, int32_t du) {
  int a = 0;
  if (cv == cu) a += 1;
  else if (dv == cu) a -= 1;
  if (du != D_EMPTY) {
    if (cv == du) a -= 1;
    else if (dv == du) a += 1;
  }
  return a;
}

}  // namespace

}  // namespace lcc
