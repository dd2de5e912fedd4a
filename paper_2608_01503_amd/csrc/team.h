// Teams: workgroups of one launch that run on one XCD and pass through many phases without leaving the device.
//
// On small levels the method is a chain of dependent phases of a few microseconds each, so a launch per phase
// (2.8 us from one kernel to the next, measured with empty kernels) and the host's reads in between (14 us each)
// cost more than the work.  A team runs the phases in one launch.  Its workgroups share one L2, so a phase
// boundary needs no cache write-back: stores are drained (vmcnt 0) into that L2, and data written by other
// workgroups is read with agent-scope loads, which pass by the CU's own L1.  (With agent-scope release and acquire
// fences instead, a boundary of 32 workgroups took 4.6 us where this takes 1.0 us.)
//
// Membership: workgroups are launched over the whole chip.  The first to arrive picks its XCD; the others on that
// XCD join until the first member closes the list (all expected ones are there, or TEAM_WAIT has passed), and
// every workgroup elsewhere or later returns at once.  A member waits only for members, all of which are already
// running, so every wait ends whatever else runs on the device; results do not depend on the number of members.
//
// The kernels use no private memory: parameters are read from the kernel's argument segment where a phase needs
// them (TEAM_PHASE keeps them from being held in registers across phases), and everything is inlined.
#pragma once

#include "common.h"

namespace lcc {

constexpr int TEAM_BLOCK = 1024;            // threads of a workgroup: 16 wavefronts, one workgroup per CU
constexpr int TEAM_WAVES = TEAM_BLOCK / WAVE;
constexpr int TEAM_MAX = 32;                // members: the CUs of an XCD
constexpr int TEAM_GRID = 8 * TEAM_MAX;     // workgroups launched (they spread over the XCDs in turn)
constexpr unsigned long long TEAM_WAIT = 300;  // 3 us of the 100 MHz clock
constexpr int TEAM_VALS = 4;                // values summed at one boundary
constexpr int TEAM_SLOTS = 2;               // control blocks: a launch uses one and clears the next launch's

// One launch's control block (zero when the launch starts).
struct TeamCtl {
  alignas(128) uint32_t xcc;    // 1 + the team's XCD
  alignas(128) uint32_t state;  // TEAM_CLOSED | arrivals
  alignas(128) uint32_t n;      // members, once closed
  // Boundary words, two sets used in turn: a member announces boundary e by writing words e << 32 | payload, two
  // per value it adds to a sum; every member polls the words of all members.  One store and one load carry the
  // arrival and the data.
  alignas(128) uint64_t word[2][TEAM_MAX][2 * TEAM_VALS];
};
constexpr uint32_t TEAM_CLOSED = 0x80000000u;

#ifndef TEAM_KERNARG
#define TEAM_KERNARG __attribute__((address_space(4)))
#endif
// At the start of a phase: nothing read through kp before is kept for it.
#define TEAM_PHASE(kp) asm volatile("" : "+s"(kp))

namespace {

// Loads of data that other members write.
template <typename T>
__device__ __forceinline__ T ald(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Stores to it: an ordinary store instruction that the compiler can neither split nor merge.
template <typename T>
__device__ __forceinline__ void ast(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int uniform32(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uint64_t)x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// Sum over the 64 lanes of a fully active wavefront, returned to every lane: the row scan and row broadcasts of
// wave_sum_u32 on both halves, no LDS round trips.
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t dpp64(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(uint64_t)x, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)x >> 32), CTRL, ROWS, 0xf, false);
  return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t wave_sum64(int64_t x) {
  x += dpp64<0x111, 0xf>(x);
  x += dpp64<0x112, 0xf>(x);
  x += dpp64<0x114, 0xf>(x);
  x += dpp64<0x118, 0xf>(x);
  x += dpp64<0x142, 0xa>(x);
  x += dpp64<0x143, 0xc>(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)x, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), 63);
  return (int64_t)((uint64_t)hi << 32 | lo);
}

struct TeamShared {
  int64_t red[TEAM_VALS][TEAM_WAVES];
  int64_t tot[TEAM_VALS];
  int64_t pre[TEAM_VALS];
  uint32_t wsum[TEAM_WAVES];
  uint32_t rank, n;
};
__shared__ TeamShared team_sh;

struct Sum1 { int64_t a; };
struct Sum2 { int64_t a, b; };
struct Sum3 { int64_t a, b, c; };

struct Team {
  TeamCtl* c;
  int rank, n;        // this workgroup, members (uniform)
  uint32_t epoch;     // the last boundary

  // False: this workgroup is not a member and returns.  Called by all its threads.
  __device__ __forceinline__ bool join(TeamCtl* ctl, TeamCtl* next) {
    c = ctl;
    epoch = 0;
    if (threadIdx.x == 0) {
      team_sh.n = 0;
      const uint32_t x = 1u + __builtin_amdgcn_s_getreg(20 | (3 << 11));  // XCC_ID, bits 3:0
      const uint32_t first = atomicCAS(&ctl->xcc, 0u, x);
      if (first == 0u || first == x) {
        const uint32_t old = atomicAdd(&ctl->state, 1u);
        if (!(old & TEAM_CLOSED) && old < (uint32_t)TEAM_MAX) {
          if (old == 0) {
            const unsigned long long t0 = wall_clock64();
            while (ald(&ctl->state) < (uint32_t)TEAM_MAX && wall_clock64() - t0 < TEAM_WAIT) {}
            const uint32_t f = atomicOr(&ctl->state, TEAM_CLOSED);
            ast(&ctl->n, min(f, (uint32_t)TEAM_MAX));
            next->xcc = next->state = next->n = 0;
          }
          uint32_t m;
          while ((m = ald(&ctl->n)) == 0) {}
          team_sh.rank = old;
          team_sh.n = m;
        }
      }
    }
    __syncthreads();
    n = uniform32((int)team_sh.n);
    rank = n ? uniform32((int)team_sh.rank) : 0;
    if (n && rank == 0)
      for (int k = threadIdx.x; k < (int)(sizeof(next->word) / 8); k += TEAM_BLOCK) (&next->word[0][0][0])[k] = 0;
    return n != 0;
  }

  // Wavefront 0: writes the K words of this member (lane k < K holds word k's payload) and waits for every
  // member's; got[k] = word k of member `lane`.
  template <int K>
  __device__ __forceinline__ void exchange(uint32_t mine, uint32_t (&got)[K]) {
    const int lane = threadIdx.x;
    uint64_t(*w)[2 * TEAM_VALS] = c->word[epoch & 1];
    if (lane < K) ast(&w[rank][lane], (uint64_t)epoch << 32 | mine);
    const int from = lane < n ? lane : 0;
    bool all;
    do {
      all = true;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint64_t x = ald(&w[from][k]);
        got[k] = (uint32_t)x;
        all = all && (uint32_t)(x >> 32) == epoch;
      }
    } while (__ballot(!all));
  }

  // Phase boundary: everything written before it is visible to agent-scope loads after it.
  __device__ __forceinline__ void sync() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    ++epoch;
    if (threadIdx.x < WAVE) {
      uint32_t got[1];
      exchange<1>(0, got);
    }
    asm volatile("" ::: "memory");
    __syncthreads();
  }
  // The same, and plain loads see it too (the CU's L1 is emptied): before reading arrays the team has built with
  // ordinary loads.
  __device__ __forceinline__ void sync_all() {
    sync();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
  }

  template <int K>
  __device__ __forceinline__ void put(int64_t x) {
    const int64_t s = wave_sum64(x);
    if ((threadIdx.x & (WAVE - 1)) == 0) team_sh.red[K][threadIdx.x / WAVE] = s;
  }
  template <int K>
  __device__ __forceinline__ void sums() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    ++epoch;
    if (threadIdx.x < WAVE) {
      const int lane = threadIdx.x;
      int64_t s = 0;  // lanes 2k and 2k + 1: this member's sum of value k
      if (lane < 2 * K) {
#pragma unroll
        for (int w = 0; w < TEAM_WAVES; ++w) s += team_sh.red[lane / 2][w];
      }
      uint32_t got[2 * K];
      exchange<2 * K>(lane & 1 ? (uint32_t)((uint64_t)s >> 32) : (uint32_t)(uint64_t)s, got);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int64_t p = lane < n ? (int64_t)((uint64_t)got[2 * k + 1] << 32 | got[2 * k]) : 0;
        const int64_t tot = wave_sum64(p), pre = wave_sum64(lane < rank ? p : 0);
        if (lane == 0) { team_sh.tot[k] = tot; team_sh.pre[k] = pre; }
      }
    }
    asm volatile("" ::: "memory");
    __syncthreads();
  }
  // Sums over all threads of the team, at a phase boundary; every thread gets them.
  __device__ __forceinline__ Sum1 sum(int64_t a) {
    put<0>(a);
    sums<1>();
    Sum1 r{uniform64(team_sh.tot[0])};
    __syncthreads();
    return r;
  }
  __device__ __forceinline__ Sum2 sum(int64_t a, int64_t b) {
    put<0>(a); put<1>(b);
    sums<2>();
    Sum2 r{uniform64(team_sh.tot[0]), uniform64(team_sh.tot[1])};
    __syncthreads();
    return r;
  }
  __device__ __forceinline__ Sum3 sum(int64_t a, int64_t b, int64_t d) {
    put<0>(a); put<1>(b); put<2>(d);
    sums<3>();
    Sum3 r{uniform64(team_sh.tot[0]), uniform64(team_sh.tot[1]), uniform64(team_sh.tot[2])};
    __syncthreads();
    return r;
  }
  // The same, and the sums over the members of lower rank.
  __device__ __forceinline__ Sum1 sum(int64_t a, Sum1& pre) {
    put<0>(a);
    sums<1>();
    Sum1 r{uniform64(team_sh.tot[0])};
    pre.a = uniform64(team_sh.pre[0]);
    __syncthreads();
    return r;
  }
  __device__ __forceinline__ Sum2 sum(int64_t a, int64_t b, Sum2& pre) {
    put<0>(a); put<1>(b);
    sums<2>();
    Sum2 r{uniform64(team_sh.tot[0]), uniform64(team_sh.tot[1])};
    pre.a = uniform64(team_sh.pre[0]);
    pre.b = uniform64(team_sh.pre[1]);
    __syncthreads();
    return r;
  }

  // Exclusive prefix of x over the threads of this workgroup; *total = its sum.
  __device__ __forceinline__ uint32_t block_excl(uint32_t x, uint32_t& total) {
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o, WAVE);
      if (lane >= o) inc += y;
    }
    if (lane == WAVE - 1) team_sh.wsum[wv] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < TEAM_WAVES; ++w) {
      const uint32_t s = team_sh.wsum[w];
      if (w < wv) before += s;
      tot += s;
    }
    __syncthreads();
    total = (uint32_t)uniform32((int)tot);
    return before + inc - x;
  }

  // this member's share [lo, hi) of m items
  __device__ __forceinline__ int share_lo(int m) const { return (int)((int64_t)m * rank / n); }
  __device__ __forceinline__ int share_hi(int m) const { return (int)((int64_t)m * (rank + 1) / n); }
  __device__ __forceinline__ int threads() const { return n * TEAM_BLOCK; }
};

// This thread's number within its workgroup, recomputed in every phase (values derived from it are not kept
// across phases).
__device__ __forceinline__ int team_tx() {
  int x = threadIdx.x;
  asm volatile("" : "+v"(x));
  return x;
}

}  // namespace

}  // namespace lcc
