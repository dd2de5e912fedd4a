// Small levels: the local move as one launch of a team (team.h).
//
// The same method as lm.hip, with the same integer forms and the same results, laid out for levels whose phases
// take a few microseconds each: counters stay in registers (every member sums the same partials), the moves are
// applied where the afterburner keeps them, cluster sizes are kept beside the weights so that free ids need no
// marking pass, and repeated passes cost nothing.  A level has at most TEAM_ENTRIES entries, so positions are
// 32-bit here.
#include <algorithm>

#include "team.h"
#include "rows.h"

namespace lcc {

namespace {

constexpr int TW_SLOTS = 1024;   // LDS hash of a wavefront (rows of up to TW_ROW entries), 16 of them
constexpr int TW_ROW = TW_SLOTS / 2;
constexpr int TB_SLOTS = 16384;  // LDS hash of the whole workgroup (rows of up to TB_ROW entries)
constexpr int TB_ROW = TB_SLOTS / 2;
constexpr int TD_SLOTS = 32768;  // dense table of cluster ids for longer rows: one pass over the row per 32768 ids
constexpr int AG_SLOTS = 2048;   // LDS table of the cluster-weight changes

union TeamLds {
  struct { int32_t k[TEAM_WAVES][TW_SLOTS]; uint32_t v[TEAM_WAVES][TW_SLOTS]; } wave;
  struct { int32_t k[TB_SLOTS]; uint32_t v[TB_SLOTS]; } blk;
  uint32_t dense[TD_SLOTS];
  struct { int32_t k[AG_SLOTS]; int32_t c[AG_SLOTS]; unsigned long long w[AG_SLOTS]; } agg;
};
static_assert(sizeof(LeaderLds<2>) <= TW_SLOTS * sizeof(int32_t), "a wavefront may use its hash for leaders");
__shared__ TeamLds lds;
__shared__ Best team_best[TEAM_WAVES];

struct TeamArgs {
  TeamCtl* ctl;
  TeamCtl* next;
  int32_t n;
  const int64_t* off;
  const int32_t* idx;
  const int32_t* w;
  const int64_t* vw;
  const int32_t* list;          // vertices by degree bucket, bucket b at [boff[b], boff[b + 1])
  int32_t boff[NBUCKET + 1];
  int32_t hash_shift;
  Score sc;
  const int32_t* cons;
  int32_t* C;
  int32_t* Cout;
  int64_t* W;
  int32_t* cnt;                 // members of every cluster id
  VState* vs;
  uint8_t* empty;
  int32_t *freelist, *movers;
  int64_t sum_w2;
  int32_t singleton, pass_limit, symmetry;
  uint32_t phi_num[MAX_PASSES + 1], phi_den[MAX_PASSES + 1];
  LMSlot* slot;
  uint8_t* used;
  int32_t* rank;
};
typedef const TEAM_KERNARG TeamArgs* KP;

// Changes of the cluster weights and sizes, summed per workgroup.  A slot belongs to the first cluster that
// claims it; changes of other clusters that hash to it go to memory directly.  The return values are the change
// of the sum of squared weights that the update made, modulo 2^64.
__device__ __forceinline__ void agg_clear() {
  for (int s = team_tx(); s < AG_SLOTS; s += TEAM_BLOCK) { lds.agg.k[s] = -1; lds.agg.c[s] = 0; lds.agg.w[s] = 0; }
  __syncthreads();
}
__device__ __forceinline__ uint64_t agg_apply(int64_t* W, int32_t* cnt, int32_t c, int64_t w, int32_t n) {
  atomicAdd(&cnt[c], n);
  const uint64_t old = atomicAdd((unsigned long long*)&W[c], (unsigned long long)w);
  return 2 * old * (uint64_t)w + (uint64_t)w * (uint64_t)w;
}
__device__ __forceinline__ uint64_t agg_add(int64_t* W, int32_t* cnt, int32_t c, int64_t w, int32_t n) {
  static_assert(AG_SLOTS == 1 << 11, "hash width");
  const uint32_t s = ((uint32_t)c * 2654435761u) >> 21;
  const int32_t old = atomicCAS(&lds.agg.k[s], -1, c);
  const bool mine = old == -1 || old == c;
  if (mine) {
    atomicAdd(&lds.agg.w[s], (unsigned long long)w);
    atomicAdd(&lds.agg.c[s], n);
  }
  asm volatile("" ::: "memory");  // the LDS updates above and the memory updates below stay separate instructions
  uint64_t d = 0;
  if (!mine) d = agg_apply(W, cnt, c, w, n);
  return d;
}
__device__ __forceinline__ uint64_t agg_flush(int64_t* W, int32_t* cnt) {
  __syncthreads();
  uint64_t d = 0;
  for (int s = team_tx(); s < AG_SLOTS; s += TEAM_BLOCK)
    if (lds.agg.k[s] >= 0) d += agg_apply(W, cnt, lds.agg.k[s], (int64_t)lds.agg.w[s], lds.agg.c[s]);
  return d;
}

struct TeamAcc {
  int32_t ncand = 0;
  int64_t own = 0;
};

__device__ __forceinline__ void team_finish(KP kp, int32_t v, int32_t cv, int64_t wv, int64_t own, int64_t sbest,
                                            int32_t cbest, int64_t wcv, uint32_t pa, uint32_t pb, TeamAcc& a) {
  const int64_t scur = kp->sc.q * own - kp->sc.p * wv * (wcv - wv);
  const Verdict vd = decide(scur, sbest, cbest, pa, pb, 0);
  VState o;
  o.c = cv;
  o.d = vd.d;
  o.delta = vd.delta;
  kp->vs[v] = o;
  a.ncand += vd.cand ? 1 : 0;
  a.own += own;
}

// Work of a pass over the rows: a wavefront takes 64 / G vertices of a bucket of G-lane groups (G = 4, 8, 16, 32)
// or one longer row at a time.  All buckets form one list of such tasks, the long rows first, dealt to the members
// in turn: a wavefront goes through one dependent chain of loads per task it gets, not one per bucket (with a loop
// per bucket a pass over 27,000 entries took 28 us, most of it six such chains one after the other).
template <typename Op>
__device__ __forceinline__ void team_tasks(const Team& t, KP kp, Op& op) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), lane = tx & (WAVE - 1), wv = uniform32(tx / WAVE);
  const int e0 = kp->boff[1], e1 = kp->boff[2], e2 = kp->boff[3], e3 = kp->boff[4], e4 = kp->boff[NBUCKET];
  const int n4 = e4 - e3, n3 = n4 + (e3 - e2 + 1) / 2, n2 = n3 + (e2 - e1 + 3) / 4, n1 = n2 + (e1 - e0 + 7) / 8,
            n0 = n1 + (e0 + 15) / 16;
  for (int k = wv * t.n + t.rank; k < n0; k += t.n * TEAM_WAVES) {
    if (k < n4) {
      op.wave(kp, uniform32(kp->list[e4 - 1 - k]), lane);  // the longest buckets are at the end of the list
    } else if (k < n3) {
      const int i = e2 + (k - n4) * 2 + lane / 32;
      if (i < e3) op.template group<32>(kp, kp->list[i], lane & 31);
    } else if (k < n2) {
      const int i = e1 + (k - n3) * 4 + lane / 16;
      if (i < e2) op.template group<16>(kp, kp->list[i], lane & 15);
    } else if (k < n1) {
      const int i = e0 + (k - n2) * 8 + lane / 8;
      if (i < e1) op.template group<8>(kp, kp->list[i], lane & 7);
    } else {
      const int i = (k - n1) * 16 + lane / 4;
      if (i < e0) op.template group<4>(kp, kp->list[i], lane & 3);
    }
  }
}

// First pass from singletons: the clusters are the neighbours.
struct SingleOp {
  uint32_t pa, pb;
  TeamAcc a;
  template <int U, int G>
  __device__ __forceinline__ void row(KP kp, int32_t v, int gl) {
    const int64_t wv = kp->vw[v];
    const int e = (int)kp->off[v + 1];
    const int32_t bv = kp->cons ? kp->cons[v] : 0;
    int64_t bs = INT64_MIN;
    int32_t bc = INT32_MAX;
    for (int j0 = (int)kp->off[v] + gl; j0 < e; j0 += U * G) {
      int32_t us[U], ws[U];
      int64_t vu[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int j = j0 + k * G < e ? j0 + k * G : e - 1;
        us[k] = kp->idx[j];
        ws[k] = kp->w[j];
      }
#pragma unroll
      for (int k = 0; k < U; ++k) vu[k] = kp->vw[us[k]];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int64_t s = kp->sc.q * ws[k] - kp->sc.p * wv * vu[k];
        // an entry read again past the end changes nothing
        if ((!kp->cons || kp->cons[us[k]] == bv) && better(s, us[k], bs, bc)) { bs = s; bc = us[k]; }
      }
    }
    argmax_steps<G>(bs, bc);
    if (gl == 0) team_finish(kp, v, v, wv, 0, bs, bc, wv, pa, pb, a);
  }
  template <int G>
  __device__ __forceinline__ void group(KP kp, int32_t v, int gl) { row<1, G>(kp, v, gl); }
  __device__ __forceinline__ void wave(KP kp, int32_t v, int lane) { row<4, WAVE>(kp, v, lane); }
};

// The row [b, e) into an LDS hash, by S lanes of which this is lane x; returns the lane's share of the weight to
// the own cluster cv.  Lanes of a wavefront that hold the same cluster are combined first.
__device__ __forceinline__ int64_t team_insert(KP kp, int b, int e, int x, int S, int32_t cv, int32_t bv, int32_t* hk,
                                               uint32_t* hv, int bits) {
  constexpr int U = 4;
  const int lane = x & (WAVE - 1);
  int64_t own = 0;
  for (int j0 = b + x, jw = uniform32(b + (x - lane)); jw < e; j0 += S * U, jw += S * U) {
    int32_t us[U], cs[U];
    uint32_t ws[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int j = j0 + k * S < e ? j0 + k * S : e - 1;
      us[k] = kp->idx[j];
      ws[k] = (uint32_t)kp->w[j];
    }
#pragma unroll
    for (int k = 0; k < U; ++k) cs[k] = ald(kp->C + us[k]);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const bool ok = j0 + k * S < e && (!kp->cons || kp->cons[us[k]] == bv);
      int32_t key = ok ? cs[k] : -1;
      const uint32_t val = ok ? ws[k] : 0u;
      if (key == cv) { own += val; key = -1; }
#pragma unroll
      for (int round = 0; round < 2; ++round) {
        const uint64_t act = __ballot(key >= 0);
        if (!act) break;
        const int lead = __ffsll((unsigned long long)act) - 1;
        const int32_t lk = __builtin_amdgcn_readlane(key, lead);
        if (__popcll(__ballot(key == lk)) < 2) break;
        const uint32_t part = wave_sum_u32(key == lk ? val : 0u);
        if (lane == lead) lds_insert(hk, hv, bits, lk, part);
        if (key == lk) key = -1;
      }
      if (key >= 0) lds_insert(hk, hv, bits, key, val);
    }
  }
  return own;
}

// slots x, x + S, ... < cap: the best cluster
__device__ __forceinline__ void team_scan(KP kp, const int32_t* hk, const uint32_t* hv, int cap, int x, int S, int64_t wv,
                                          Best& r) {
  constexpr int U = 4;
  for (int s0 = x; s0 < cap; s0 += S * U) {
    int32_t ks[U];
    uint32_t as[U];
    int64_t Ws[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int sl = s0 + k * S;
      ks[k] = sl < cap ? hk[sl] : -1;
      as[k] = sl < cap ? hv[sl] : 0u;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) Ws[k] = ks[k] >= 0 ? ald(kp->W + ks[k]) : 0;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t s = kp->sc.q * (int64_t)as[k] - kp->sc.p * wv * Ws[k];
      if (ks[k] >= 0 && better(s, ks[k], r.s, r.c)) { r.s = s; r.c = ks[k]; }
    }
  }
}

// General pass: the neighbouring clusters and the best of them.
struct EnumOp {
  uint32_t pa, pb;
  TeamAcc a;
  // rows of at most G E entries, E per lane: clusters summed by an all-pairs sweep or by leaders
  template <int G, int E>
  __device__ __forceinline__ void row(KP kp, int32_t v, int gl) {
    const int rb = (int)kp->off[v], d = (int)kp->off[v + 1] - rb;
    const int32_t cv = ald(kp->C + v);
    const int64_t wv = kp->vw[v];
    const int32_t bv = kp->cons ? kp->cons[v] : 0;
    int32_t cs[E];
    uint32_t as[E];
    bool has[E], lead[E];
    int64_t Ws[E], own = 0, bs = INT64_MIN;
    int32_t bc = INT32_MAX;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int j = gl + k * G;
      has[k] = j < d;
      cs[k] = has[k] ? kp->idx[rb + j] : v;
      as[k] = has[k] ? (uint32_t)kp->w[rb + j] : 0u;
      if (kp->cons && kp->cons[cs[k]] != bv) has[k] = false;
    }
#pragma unroll
    for (int k = 0; k < E; ++k) cs[k] = ald(kp->C + cs[k]);
    const int64_t wcv = ald(kp->W + cv);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      if (has[k] && cs[k] == cv) { own += as[k]; has[k] = false; }
      Ws[k] = has[k] ? ald(kp->W + cs[k]) : 0;
    }
    if constexpr (G * E <= 8) {
      int64_t acc = 0;
      lead[0] = has[0];
      pair_sweep<G>(cs[0], (int32_t)as[0], has[0], gl, acc, lead[0]);
      as[0] = (uint32_t)acc;
    } else {
      leader_sum<G, E>(*(LeaderLds<E>*)lds.wave.k[uniform32((int)threadIdx.x / WAVE)], threadIdx.x & (WAVE - 1), cs, as, has, lead);
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int64_t s = kp->sc.q * (int64_t)as[k] - kp->sc.p * wv * Ws[k];
      if (lead[k] && better(s, cs[k], bs, bc)) { bs = s; bc = cs[k]; }
    }
    argmax_steps<G>(bs, bc);
    own = sum_steps<G>(own);
    if (gl == 0) team_finish(kp, v, cv, wv, own, bs, bc, wcv, pa, pb, a);
  }
  template <int G>
  __device__ __forceinline__ void group(KP kp, int32_t v, int gl) { row<G, 1>(kp, v, gl); }
  // longer rows of at most TW_ROW entries: an LDS hash of the wavefront's own
  __device__ __forceinline__ void wave(KP kp, int32_t v, int lane) {
    const int b = (int)kp->off[v], e = (int)kp->off[v + 1];
    if (e - b > TW_ROW) return;  // team_enum_blk
    if (e - b <= 2 * WAVE) return row<WAVE, 2>(kp, v, lane);
    const int wv = uniform32((int)threadIdx.x / WAVE);
    int32_t* tk = lds.wave.k[wv];
    uint32_t* tv = lds.wave.v[wv];
    const int32_t cv = uniform32(ald(kp->C + v));
    const int64_t wvt = kp->vw[v], wcv = ald(kp->W + cv);
    const int bits = table_bits(e - b, kp->hash_shift, TW_SLOTS);
    for (int s = lane; s < (1 << bits); s += WAVE) { tk[s] = -1; tv[s] = 0; }
    wave_lds_sync();
    const int64_t own = team_insert(kp, b, e, lane, WAVE, cv, kp->cons ? kp->cons[v] : 0, tk, tv, bits);
    wave_lds_sync();
    Best r = best_init();
    team_scan(kp, tk, tv, 1 << bits, lane, WAVE, wvt, r);
    argmax_steps<WAVE>(r.s, r.c);
    r.own = wave_sum64(own);
    if (lane == 0) team_finish(kp, v, cv, wvt, r.own, r.s, r.c, wcv, pa, pb, a);
    wave_lds_sync();
  }
};

// longer rows, the workgroup each
__device__ __forceinline__ void team_enum_blk(const Team& t, KP kp, uint32_t pa, uint32_t pb, TeamAcc& a) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), lane = tx & (WAVE - 1), wv = tx / WAVE, end = kp->boff[NBUCKET];
  __syncthreads();
  for (int i = kp->boff[5] + t.rank; i < end; i += t.n) {  // uniform over the workgroup
    const int32_t v = uniform32(kp->list[i]);
    const int b = (int)kp->off[v], e = (int)kp->off[v + 1];
    if (e - b <= TW_ROW) continue;
    const int32_t cv = uniform32(ald(kp->C + v));
    const int32_t bv = kp->cons ? kp->cons[v] : 0;
    const int64_t wvt = kp->vw[v], wcv = ald(kp->W + cv);
    Best r = best_init();
    if (e - b <= TB_ROW) {
      const int bits = table_bits(e - b, kp->hash_shift, TB_SLOTS);
      for (int s = tx; s < (1 << bits); s += TEAM_BLOCK) { lds.blk.k[s] = -1; lds.blk.v[s] = 0; }
      __syncthreads();
      r.own = team_insert(kp, b, e, tx, TEAM_BLOCK, cv, bv, lds.blk.k, lds.blk.v, bits);
      __syncthreads();
      team_scan(kp, lds.blk.k, lds.blk.v, 1 << bits, tx, TEAM_BLOCK, wvt, r);
    } else {  // any length: cluster ids in ranges of TD_SLOTS, a dense table (weights are positive: 0 = absent)
      for (int base = 0; base < kp->n; base += TD_SLOTS) {
        for (int s = tx; s < TD_SLOTS; s += TEAM_BLOCK) lds.dense[s] = 0;
        __syncthreads();
        for (int j = b + tx; j < e; j += TEAM_BLOCK) {
          const int32_t u = kp->idx[j];
          if (kp->cons && kp->cons[u] != bv) continue;
          const int c = ald(kp->C + u) - base;
          if (c < 0 || c >= TD_SLOTS) continue;
          if (c + base == cv) r.own += kp->w[j];
          else atomicAdd(&lds.dense[c], (uint32_t)kp->w[j]);
        }
        __syncthreads();
        for (int s = tx; s < TD_SLOTS; s += TEAM_BLOCK) {
          if (!lds.dense[s]) continue;
          const int64_t x = kp->sc.q * (int64_t)lds.dense[s] - kp->sc.p * wvt * ald(kp->W + base + s);
          if (better(x, base + s, r.s, r.c)) { r.s = x; r.c = base + s; }
        }
        __syncthreads();
      }
    }
    argmax_steps<WAVE>(r.s, r.c);
    r.own = wave_sum64(r.own);
    if (lane == 0) team_best[wv] = r;
    __syncthreads();
    if (tx == 0) {
      for (int k = 1; k < TEAM_WAVES; ++k) {
        r.own += team_best[k].own;
        if (better(team_best[k].s, team_best[k].c, r.s, r.c)) { r.s = team_best[k].s; r.c = team_best[k].c; }
      }
      team_finish(kp, v, cv, wvt, r.own, r.s, r.c, wcv, pa, pb, a);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ VState ald_state(const VState* vs, int32_t v) {
  const uint64_t cd = ald((const uint64_t*)&vs[v]);
  VState s;
  s.c = (int32_t)(uint32_t)cd;
  s.d = (int32_t)(cd >> 32);
  s.delta = ald(&vs[v].delta);
  return s;
}

struct TeamKeep {
  int32_t nm = 0, ne = 0;
  uint64_t dsq = 0;
};

// The verdict on vertex v: C_out follows the state the pass started from when that state was the best so far
// (copy), and a kept move is applied.
__device__ __forceinline__ void team_apply(KP kp, int32_t v, const VState& me, bool keep, bool copy, TeamKeep& k) {
  if (copy) ast(kp->Cout + v, me.c);
  const bool fresh = keep && me.d == D_EMPTY;
  ast(kp->empty + v, (uint8_t)fresh);
  if (!keep) return;
  k.nm += 1;
  k.ne += fresh;
  const int64_t w = kp->vw[v];
  k.dsq += agg_add(kp->W, kp->cnt, me.c, -w, -1);
  if (!fresh) {
    k.dsq += agg_add(kp->W, kp->cnt, me.d, w, 1);
    ast(kp->C + v, me.d);
  }
}

__device__ __forceinline__ bool team_rule(const VState& me, int symmetry, int pass) {
  if (me.d == D_NONE) return false;
  return symmetry == 1 || !(pass & 1) || me.d == D_EMPTY || me.d < me.c;
}

// sum of the afterburner's adjustments over the entries x, x + S, ... of the row [b, e)
template <int U>
__device__ __forceinline__ int64_t team_ab_row(KP kp, int b, int e, int x, int S, int32_t v, const VState& me, int64_t wv) {
  int64_t acc = 0;
  for (int j0 = b + x; j0 < e; j0 += S * U) {
    int32_t us[U], ws[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int j = j0 + k * S < e ? j0 + k * S : e - 1;
      us[k] = kp->idx[j];
      ws[k] = kp->w[j];
    }
    VState os[U];
#pragma unroll
    for (int k = 0; k < U; ++k) os[k] = ald_state(kp->vs, us[k]);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (j0 + k * S < e && os[k].d != D_NONE && before(us[k], os[k].delta, v, me.delta, kp->sc.tie)) {
        const int pat = ab_pattern(me.c, me.d, os[k].c, os[k].d);
        if (pat) acc += (int64_t)pat * (kp->sc.q * ws[k] - kp->sc.p * kp->vw[us[k]] * wv);
      }
    }
  }
  return acc;
}

struct KeepOp {
  int pass;
  bool copy;
  TeamKeep k;
  template <int G>
  __device__ __forceinline__ void group(KP kp, int32_t v, int gl) {
    const VState me = ald_state(kp->vs, v);
    bool keep = false;
    if (kp->symmetry) {
      keep = team_rule(me, kp->symmetry, pass);
    } else if (me.d != D_NONE) {
      const int64_t acc = sum_steps<G>(team_ab_row<1>(kp, (int)kp->off[v], (int)kp->off[v + 1], gl, G, v, me, kp->vw[v]));
      keep = (__int128)me.delta + acc >= 0;
    }
    if (gl == 0) team_apply(kp, v, me, keep, copy, k);
  }
  __device__ __forceinline__ void wave(KP kp, int32_t v, int lane) {
    const int b = (int)kp->off[v], e = (int)kp->off[v + 1];
    if (e - b > TB_ROW) return;  // team_ab_blk
    const VState me = ald_state(kp->vs, v);
    bool keep = false;
    if (kp->symmetry) {
      keep = team_rule(me, kp->symmetry, pass);
    } else if (me.d != D_NONE) {
      const int64_t acc = wave_sum64(team_ab_row<2>(kp, b, e, lane, WAVE, v, me, kp->vw[v]));
      keep = (__int128)me.delta + acc >= 0;
    }
    if (lane == 0) team_apply(kp, v, me, keep, copy, k);
  }
};

// the workgroup per row above TB_ROW entries
__device__ __forceinline__ void team_ab_blk(const Team& t, KP kp, int pass, bool copy, TeamKeep& kk) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), lane = tx & (WAVE - 1), end = kp->boff[NBUCKET];
  for (int i = kp->boff[5] + t.rank; i < end; i += t.n) {  // uniform over the workgroup
    const int32_t v = uniform32(kp->list[i]);
    const int b = (int)kp->off[v], e = (int)kp->off[v + 1];
    if (e - b <= TB_ROW) continue;
    const VState me = ald_state(kp->vs, v);
    int64_t acc = 0;
    if (!kp->symmetry && me.d != D_NONE) acc = team_ab_row<2>(kp, b, e, tx, TEAM_BLOCK, v, me, kp->vw[v]);
    acc = wave_sum64(acc);
    __syncthreads();
    if (lane == 0) team_best[tx / WAVE].own = acc;
    __syncthreads();
    if (tx == 0) {
      for (int k = 1; k < TEAM_WAVES; ++k) acc += team_best[k].own;
      const bool keep = kp->symmetry ? team_rule(me, kp->symmetry, pass) : me.d != D_NONE && (__int128)me.delta + acc >= 0;
      team_apply(kp, v, me, keep, copy, kk);
    }
  }
}

// Movers to a new singleton: the i-th in ascending vertex order takes the i-th id without members.  Every member
// lists its share of the ids and of the movers, at the places that the shares before it leave.
__device__ __forceinline__ void team_empty(Team& t, KP kp, int nm, int64_t& sw2) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), n = kp->n, lo = t.share_lo(n), hi = t.share_hi(n);
  int xf = 0, xe = 0;
  for (int i = lo + tx; i < hi; i += TEAM_BLOCK) {
    xf += ald(kp->cnt + i) == 0;
    xe += ald(kp->empty + i) != 0;
  }
  Sum2 pre;
  t.sum(xf, xe, pre);
  int f = (int)pre.a, e = (int)pre.b;
  for (int i0 = lo; i0 < hi; i0 += TEAM_BLOCK) {  // uniform over the workgroup
    const int i = i0 + tx;
    const uint32_t isf = i < hi && ald(kp->cnt + i) == 0, ise = i < hi && ald(kp->empty + i) != 0;
    uint32_t tot;
    const uint32_t at = t.block_excl(isf | ise << 16, tot);
    const int pf = f + (int)(at & 0xFFFF), pe = e + (int)(at >> 16);
    if (isf && pf < nm) ast(kp->freelist + pf, i);  // no more ids than movers are needed
    if (ise) ast(kp->movers + pe, i);
    f += (int)(tot & 0xFFFF);
    e += (int)(tot >> 16);
  }
  t.sync();
  int64_t d = 0;
  for (int k = t.rank * TEAM_BLOCK + tx; k < nm; k += t.threads()) {
    const int32_t v = ald(kp->movers + k), c = ald(kp->freelist + k);
    const int64_t w = kp->vw[v];
    ast(kp->C + v, c);
    ast(kp->W + c, w);
    ast(kp->cnt + c, 1);
    d += w * w;
  }
  sw2 += t.sum(d).a;
}

// internal weight of a clustering, this thread's share
struct InternalOp {
  const int32_t* C;
  int64_t s;
  template <int G>
  __device__ __forceinline__ void group(KP kp, int32_t v, int gl) {
    const int32_t cv = ald(C + v);
    const int e = (int)kp->off[v + 1];
    for (int j = (int)kp->off[v] + gl; j < e; j += G)
      if (ald(C + kp->idx[j]) == cv) s += kp->w[j];
  }
  __device__ __forceinline__ void wave(KP kp, int32_t v, int lane) { group<WAVE>(kp, v, lane); }
};

// The starting state: cluster weights and sizes of C_out (or singletons), C = C_out.
__device__ __forceinline__ void team_start(Team& t, KP kp) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), n = kp->n, t0 = t.rank * TEAM_BLOCK + tx;
  if (kp->singleton) {
    for (int v = t0; v < n; v += t.threads()) {
      ast(kp->C + v, v);
      ast(kp->Cout + v, v);
      ast(kp->W + v, kp->vw[v]);
      ast(kp->cnt + v, 1);
    }
  } else {
    for (int v = t0; v < n; v += t.threads()) { ast(kp->W + v, (int64_t)0); ast(kp->cnt + v, 0); }
    t.sync();
    agg_clear();
    for (int v = t0; v < n; v += t.threads()) {
      const int32_t c = ald(kp->Cout + v);
      ast(kp->C + v, c);
      agg_add(kp->W, kp->cnt, c, kp->vw[v], 1);
    }
    agg_flush(kp->W, kp->cnt);
  }
  t.sync();
}

// sum of squared cluster weights, this thread's share
__device__ __forceinline__ int64_t team_sw2(const Team& t, KP kp) {
  TEAM_PHASE(kp);
  int64_t sq = 0;
  for (int c = t.rank * TEAM_BLOCK + team_tx(); c < kp->n; c += t.threads()) {
    const int64_t w = ald(kp->W + c);
    sq += w * w;
  }
  return sq;
}

// LocalMovePasses (Alg. 2) from singletons or from C_out (which holds the starting clustering); the result is
// left in C_out.  *slot receives the statistics (plain stores, read after the launch).
__device__ __forceinline__ void team_local_move(Team& t, const KP kp0) {
  KP kp = kp0;
  TEAM_PHASE(kp);
  const bool log = t.rank == 0 && threadIdx.x == 0;
  for (int k = threadIdx.x; t.rank == 0 && k < (int)(sizeof(LMSlot) / 8); k += TEAM_BLOCK) ast((int64_t*)kp->slot + k, (int64_t)0);
  team_start(t, kp);
  int64_t sw2 = 0, I = 0, Nbest = 0, N0 = 0, nL = 0, nM = 0;
  bool first = true, skipped = false;
  const int limit = kp->pass_limit;
  for (int i = 1; i <= limit; ++i) {
    KP kp = kp0;
    TEAM_PHASE(kp);
    const uint32_t pa = kp->phi_num[i], pb = kp->phi_den[i];
    skipped = i >= 2 && nM == 0 && kp->symmetry != 2 && pa == kp->phi_num[i - 1] && pb == kp->phi_den[i - 1];
    if (skipped) {  // repeats the previous pass exactly
      if (log) { LMSlot* s = kp->slot; s->skip[i] = 1; s->nL[i] = nL; s->I[i - 1] = I; s->SW2[i] = sw2; }
      continue;
    }
    const int64_t sq = first ? team_sw2(t, kp) : 0;
    TeamAcc a;
    if (kp->singleton && i == 1) {
      SingleOp op{pa, pb, a};
      team_tasks(t, kp, op);
      a = op.a;
    } else {
      EnumOp op{pa, pb, a};
      team_tasks(t, kp, op);
      a = op.a;
      team_enum_blk(t, kp, pa, pb, a);
    }
    const Sum3 x = t.sum(a.ncand, a.own, sq);
    nL = x.a;
    I = x.b;
    if (first) sw2 = x.c;
    const int64_t N = kp->sc.q * I - kp->sc.p * (sw2 - kp->sum_w2);  // the state this pass starts from
    const bool copy = !first && N > Nbest;
    if (log) { LMSlot* s = kp->slot; s->nL[i] = nL; s->I[i - 1] = I; if (first) s->SW2[0] = sw2; }
    if (first) N0 = N;
    if (first || copy) Nbest = N;
    first = false;
    agg_clear();
    KeepOp ko{i, copy, TeamKeep{}};
    team_tasks(t, kp, ko);
    TeamKeep kk = ko.k;
    team_ab_blk(t, kp, i, copy, kk);
    kk.dsq += agg_flush(kp->W, kp->cnt);
    const Sum3 y = t.sum(kk.nm, kk.ne, (int64_t)kk.dsq);
    nM = y.a;
    sw2 = (int64_t)((uint64_t)sw2 + (uint64_t)y.c);
    if (y.b) team_empty(t, kp, (int)y.b, sw2);
    if (log) { LMSlot* s = kp->slot; s->nM[i] = nM; s->SW2[i] = sw2; }
  }
  bool copy = false;
  if (first) {  // no pass
    const int64_t sq = t.sum(team_sw2(t, kp)).a;
    if (log) kp->slot->SW2[0] = sq;
    N0 = Nbest = -kp->sc.p * (sq - kp->sum_w2);
  } else {
    if (!skipped && nM) {  // the state the last pass left
      InternalOp op{kp->C, 0};
      team_tasks(t, kp, op);
      I = t.sum(op.s).a;
      const int64_t N = kp->sc.q * I - kp->sc.p * (sw2 - kp->sum_w2);
      if (N > Nbest) { Nbest = N; copy = true; }
    }
    if (log) kp->slot->I[kp->pass_limit] = I;
  }
  if (copy) {
    for (int v = t.rank * TEAM_BLOCK + team_tx(); v < kp->n; v += t.threads()) ast(kp->Cout + v, ald(kp->C + v));
    t.sync();
  }
  if (log) { kp->slot->Nbest = Nbest; kp->slot->N0 = N0; }
}

// ranks of the labels in use: rank[c] = labels below c in use, for c in [0, n]; returns their number
__device__ __forceinline__ int team_rank(Team& t, KP kp, const int32_t* lab) {
  TEAM_PHASE(kp);
  const int tx = team_tx(), n = kp->n;
  for (int c = t.rank * TEAM_BLOCK + tx; c < n; c += t.threads()) ast(kp->used + c, (uint8_t)0);
  t.sync();
  for (int v = t.rank * TEAM_BLOCK + tx; v < n; v += t.threads()) ast(kp->used + ald(lab + v), (uint8_t)1);
  t.sync();
  const int lo = t.share_lo(n), hi = t.share_hi(n);
  int x = 0;
  for (int c = lo + tx; c < hi; c += TEAM_BLOCK) x += ald(kp->used + c);
  Sum1 pre;
  const int nc = (int)t.sum(x, pre).a;
  int run = (int)pre.a;
  for (int c0 = lo; c0 < hi; c0 += TEAM_BLOCK) {  // uniform over the workgroup
    const int c = c0 + tx;
    uint32_t tot;
    const uint32_t at = t.block_excl(c < hi ? (uint32_t)ald(kp->used + c) : 0u, tot);
    if (c < hi) ast(kp->rank + c, run + (int)at);
    run += (int)tot;
  }
  if (t.rank == t.n - 1 && tx == 0) ast(kp->rank + n, nc);
  return nc;
}

__global__ __launch_bounds__(TEAM_BLOCK) void k_team_local_move(TeamArgs args) {
  KP kp = (KP)__builtin_amdgcn_kernarg_segment_ptr();
  Team t;
  if (!t.join(kp->ctl, kp->next)) return;
  team_local_move(t, kp);
  const int nc = team_rank(t, kp, kp->Cout);
  if (t.rank == 0 && threadIdx.x == 0) kp->slot->nlab = nc;
}

}  // namespace

// --- host launchers

static TeamCtl* team_ctl(TeamHost& h, TeamCtl** next) {
  TeamCtl* c = h.ctl + h.turn % TEAM_SLOTS;
  *next = h.ctl + (h.turn + 1) % TEAM_SLOTS;
  ++h.turn;
  return c;
}

void team_local_move_launch(const DevGraph& g, const Buckets& b, const LMParams& prm, bool singleton, LMBuffers& bufs,
                            int32_t* C, uint8_t* used, int32_t* rank, TeamHost& th, LMSlot* slot, hipStream_t st) {
  TeamArgs a{};
  a.ctl = team_ctl(th, &a.next);
  a.n = (int32_t)g.n;
  a.off = g.off; a.idx = g.idx; a.w = g.w; a.vw = g.vw;
  a.list = b.list;
  for (int k = 0; k <= NBUCKET; ++k) a.boff[k] = (int32_t)b.off[k];
  a.hash_shift = b.hash_shift;
  a.sc = prm.sc;
  a.cons = prm.cons;
  a.C = bufs.C; a.Cout = C; a.W = bufs.W; a.cnt = bufs.scan_a; a.vs = bufs.vs;
  a.empty = bufs.empty; a.freelist = bufs.freelist; a.movers = bufs.scan_b;
  a.sum_w2 = prm.sum_w2;
  a.singleton = singleton ? 1 : 0;
  a.pass_limit = prm.pass_limit;
  a.symmetry = prm.symmetry;
  for (int i = 0; i <= MAX_PASSES; ++i) { a.phi_num[i] = prm.phi_num[i]; a.phi_den[i] = prm.phi_den[i]; }
  a.slot = slot;
  a.used = used; a.rank = rank;
  k_team_local_move<<<TEAM_GRID, TEAM_BLOCK, 0, st>>>(a);
}

}  // namespace lcc
