// REM scheduler: global-batch replica allocation and micro-batch token
// dispatching on the device, one wavefront per independent problem (layer).
//
// Paper: Sec. 3.2.1 -- the Benefit Score S(e, r_s, r_r, tau), the number of
// tokens a replica of expert e on the receiving rank r_r takes over from the
// sending rank r_s, with tau the mean rank load:
//   min(tau - L_r, T_e, L_s - tau)        if L_r < tau < L_s
//   min(floor((L_s - L_r) / 2), T_e)      if L_r >= tau and L_s > L_r
//   -1                                    otherwise.
// App. B, Alg. 1 -- while a rank has a free replica slot, the least-loaded
// such rank receives a replica of the expert with the largest score; the
// loads and the expert's volume move by that score; a score <= 0 stops it.
// App. B, Alg. 2 -- D passes; each orders the ranks by queue depth (lightest
// first, without re-sorting inside the pass) and lets every rank pull tokens
// through the best of the replicas it holds.
//
// All arithmetic is exact in integers: tau = total / R is kept as its floor tf
// and ceiling tc, with R * L < total <=> L < tc, R * L > total <=> L > tf, and
// the two differences with tau, rounded down to whole tokens, equal to tf - L_r
// and L_s - tc.  An expert's tokens come from its home rank.  Ties: the
// lowest rank index among equally loaded receivers, the lowest expert index
// among equal scores (Alg. 1), the earliest replica (Alg. 2), ranks of equal
// depth by index.  Alg. 2 applies a move only when its score is positive.
//
// Both algorithms are serial chains, one placement after another, so a step's
// latency is all that counts.  A step's searches reduce the values alone, with
// DPP row shifts (no LDS), and find the winner's index with a ballot.  Values
// are 32-bit when the layer's loads sum to less than 2^31 and no volume
// reaches it (token counts of a global batch do), else 64-bit.  8 layers, 256
// experts, 64 ranks, 4 replicas each: allocation 167 -> 35 us, dispatch 239
// -> 45 us (before: 64-bit keys through ds_bpermute, divisions by R in every
// score, and all replicas searched for those of one rank).
#include <algorithm>

#include "common.h"

namespace dol {
namespace {

constexpr int64_t kRemMaxVal = int64_t(1) << 40;  // loads and volumes must be below this
constexpr int64_t kSmall = int64_t(1) << 31;

// T tokens of an expert whose home rank has load Ls, to a rank with load Lr.
template <typename V>
__device__ __forceinline__ V benefit(V T, V Ls, V Lr, V tf, V tc) {
  const V a = min(min((V)(tf - Lr), T), (V)(Ls - tc));
  const V b = min((V)((Ls - Lr) >> 1), T);
  const V below = Ls > tf ? a : (V)-1;  // L_r < tau
  const V above = Ls > Lr ? b : (V)-1;
  return Lr < tc ? below : above;
}

// Value of `v` CTRL-shifted within rows (0x111.. row_shr, 0x142 / 0x143 row
// broadcasts); lanes with no source get `id`.
template <int CTRL>
__device__ __forceinline__ int32_t dpp(int32_t v, int32_t id) {
  return __builtin_amdgcn_update_dpp(id, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ int64_t dpp(int64_t v, int64_t id) {
  const uint32_t lo = (uint32_t)dpp<CTRL>((int32_t)v, (int32_t)id);
  const int32_t hi = dpp<CTRL>((int32_t)(v >> 32), (int32_t)(id >> 32));
  return (int64_t)(((u64)(uint32_t)hi << 32) | lo);
}
__device__ __forceinline__ int32_t lane_value(int32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ int64_t lane_value(int64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, l);
  const int32_t hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return (int64_t)(((u64)(uint32_t)hi << 32) | lo);
}

// Reductions over the wave (every lane active), the result uniform.
template <typename V, typename F>
__device__ __forceinline__ V wave_reduce(V v, V id, F f) {
  v = f(v, dpp<0x111>(v, id));
  v = f(v, dpp<0x112>(v, id));
  v = f(v, dpp<0x114>(v, id));
  v = f(v, dpp<0x118>(v, id));
  v = f(v, dpp<0x142>(v, id));
  v = f(v, dpp<0x143>(v, id));
  return lane_value(v, 63);
}
template <typename V>
struct Lim;
template <>
struct Lim<int32_t> {
  static constexpr int32_t kMax = 0x7FFFFFFF, kMin = -kMax - 1;  // the identities of min and max (fused DPP)
};
template <>
struct Lim<int64_t> {
  static constexpr int64_t kMax = 0x7FFFFFFFFFFFFFFFll, kMin = -kMax - 1;
};
template <typename V>
__device__ __forceinline__ V wave_min(V v) {
  return wave_reduce(v, Lim<V>::kMax, [](V a, V b) { return min(a, b); });
}
// The largest value of lanes 0 to 15.
template <typename V>
__device__ __forceinline__ V row_max(V v) {
  const V id = Lim<V>::kMin;
  v = max(v, dpp<0x111>(v, id));
  v = max(v, dpp<0x112>(v, id));
  v = max(v, dpp<0x114>(v, id));
  v = max(v, dpp<0x118>(v, id));
  return lane_value(v, 15);
}
template <typename V>
__device__ __forceinline__ V wave_max(V v) {
  return wave_reduce(v, Lim<V>::kMin, [](V a, V b) { return max(a, b); });
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor((long long)v, off, 64);
  return v;
}
__device__ __forceinline__ int64_t wave_max_i64(int64_t v) { return wave_max<int64_t>(v); }

// The greedy loop of Alg. 1.  Lane l holds experts l + 64 s (T_e, home rank and
// the home's load) and ranks l + 64 s (load, replicas taken; D for positions
// past R).  Returns the number of placements.
template <typename V, int NE, int NR>
__device__ __forceinline__ int allocate_loop(V (&T)[NE], const int (&home)[NE], V (&Ls)[NE], V (&Ld)[NR],
                                             int (&used)[NR], int R, int D, int64_t total, do_rem_move* mv, int lane) {
  const V tf = (V)(total / R), tc = (V)((total + R - 1) / R);
  const int cap = R * D;
  int n = 0;
  while (n < cap) {
    // the receiver: least-loaded rank with a free slot, lowest index on ties
    V v = Lim<V>::kMax;
#pragma unroll
    for (int s = 0; s < NR; ++s) v = used[s] < D ? min(v, Ld[s]) : v;
    const V Lr = wave_min(v);
    int rr = -1;
#pragma unroll
    for (int s = NR - 1; s >= 0; --s) {
      const u64 m = __ballot(used[s] < D && Ld[s] == Lr);
      if (m != 0ull) rr = 64 * s + __builtin_ctzll(m);
    }
    if (rr < 0) break;  // every rank is full
    // the expert with the largest score, lowest index on ties
    V sc[NE], b = (V)-2;
    if (Lr < tc) {  // wave-uniform: one of benefit()'s two cases for every expert
#pragma unroll
      for (int s = 0; s < NE; ++s) {
        const V x = min(min((V)(tf - Lr), T[s]), (V)(Ls[s] - tc));
        sc[s] = home[s] != rr && Ls[s] > tf ? x : (V)-1;
        b = max(b, sc[s]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < NE; ++s) {
        const V x = min((V)((Ls[s] - Lr) >> 1), T[s]);
        sc[s] = home[s] != rr && Ls[s] > Lr ? x : (V)-1;
        b = max(b, sc[s]);
      }
    }
    const V delta = wave_max(b);
    if (delta <= 0) break;
    int e = 0, rs = 0;
#pragma unroll
    for (int s = NE - 1; s >= 0; --s) {
      const u64 m = __ballot(sc[s] == delta);
      if (m != 0ull) {
        const int l = __builtin_ctzll(m);
        e = 64 * s + l;
        rs = __builtin_amdgcn_readlane(home[s], l);
      }
    }
#pragma unroll
    for (int s = 0; s < NE; ++s) {
      T[s] -= 64 * s + lane == e ? delta : (V)0;
      Ls[s] += home[s] == rr ? delta : home[s] == rs ? (V)-delta : (V)0;
    }
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      const int r = 64 * s + lane;
      Ld[s] += r == rr ? delta : r == rs ? (V)-delta : (V)0;
      used[s] += r == rr ? 1 : 0;
    }
    if (lane == 0) {
      do_rem_move m;
      m.expert = e;
      m.src_rank = rs;
      m.dst_rank = rr;
      m.reserved = 0;
      m.tokens = (int64_t)delta;
      mv[n] = m;
    }
    ++n;
  }
  return n;
}

template <typename V, int NE, int NR>
__device__ __forceinline__ void allocate_layer(const int64_t* Tsh, const int64_t* Lsh, const RankMap& rm, int E, int D,
                                               int64_t total, do_rem_move* mv, int32_t* n_out, int64_t* load_out,
                                               int64_t* tokens_out, int lane) {
  const int R = rm.R;
  V T[NE], Ls[NE], Ld[NR];
  int home[NE], used[NR];
#pragma unroll
  for (int s = 0; s < NE; ++s) {
    const int e = 64 * s + lane;
    home[s] = e < E ? (int)rm.rank[e] : -1;  // no expert: a score of 0 at most, never placed
    T[s] = e < E ? (V)Tsh[e] : (V)0;
    Ls[s] = e < E ? (V)Lsh[home[s]] : (V)0;
  }
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    const int r = 64 * s + lane;
    Ld[s] = r < R ? (V)Lsh[r] : (V)0;
    used[s] = r < R ? 0 : D;
  }
  const int n = allocate_loop<V, NE, NR>(T, home, Ls, Ld, used, R, D, total, mv, lane);
  if (lane == 0) *n_out = n;
  if (load_out != nullptr) {
#pragma unroll
    for (int s = 0; s < NR; ++s)
      if (64 * s + lane < R) load_out[64 * s + lane] = (int64_t)Ld[s];
  }
  if (tokens_out != nullptr) {
#pragma unroll
    for (int s = 0; s < NE; ++s)
      if (64 * s + lane < E) tokens_out[64 * s + lane] = (int64_t)T[s];
  }
}

// Loads the layer's volumes into LDS and checks that every value is in
// [0, 2^40); returns false (wave-uniform) otherwise.
__device__ bool load_tokens(const int64_t* src, int64_t* T, int E, int lane) {
  bool bad = false;
  for (int e = lane; e < E; e += kWave) {
    const int64_t v = src[e];
    bad = bad || v < 0 || v >= kRemMaxVal;
    T[e] = v;
  }
  return __ballot(bad) == 0ull;
}

// Adds every expert's volume to its home rank's load (below 2^50: no overflow).
__device__ void home_loads(const int64_t* T, const RankMap& rm, int E, int64_t* L, int lane) {
  for (int e = lane; e < E; e += kWave)
    atomicAdd(reinterpret_cast<u64*>(&L[rm.rank[e]]), (u64)T[e]);
}

// Alg. 1 for layer blockIdx.x (one wavefront).
template <int NE, int NR>
__global__ __launch_bounds__(kWave) void k_rem_allocate(const int64_t* rank_load, const int64_t* tokens, RankMap rm,
                                                        int E, int D, do_rem_move* moves, int32_t* n_moves,
                                                        int64_t* load_out, int64_t* tokens_out) {
  __shared__ int64_t T[kMaxE];
  __shared__ int64_t Ld[kMaxE];
  const int lane = threadIdx.x, l = blockIdx.x, R = rm.R;
  bool ok = load_tokens(tokens + (int64_t)l * E, T, E, lane);
  for (int r = lane; r < R; r += kWave) Ld[r] = 0;
  __syncthreads();
  if (rank_load != nullptr)
    ok = load_tokens(rank_load + (int64_t)l * R, Ld, R, lane) && ok;
  else
    home_loads(T, rm, E, Ld, lane);
  __syncthreads();
  if (!ok) {
    if (lane == 0) n_moves[l] = -1;
    return;
  }
  int64_t part = 0, top = 0;
  for (int r = lane; r < R; r += kWave) part += Ld[r];
  for (int e = lane; e < E; e += kWave) top = max(top, T[e]);
  const int64_t total = wave_sum_i64(part);
  const bool small = total < kSmall - R && wave_max_i64(top) < kSmall;
  do_rem_move* mv = moves + (int64_t)l * R * D;
  int64_t* lo = load_out != nullptr ? load_out + (int64_t)l * R : nullptr;
  int64_t* to = tokens_out != nullptr ? tokens_out + (int64_t)l * E : nullptr;
  if (small)
    allocate_layer<int32_t, NE, NR>(T, Ld, rm, E, D, total, mv, n_moves + l, lo, to, lane);
  else
    allocate_layer<int64_t, NE, NR>(T, Ld, rm, E, D, total, mv, n_moves + l, lo, to, lane);
}

constexpr int kMaxRep = 4096;  // replicas of a layer

// Orders LDS accesses of the block's one wavefront (its LDS operations execute
// in order, so only the compiler has to keep them so).  __syncthreads would
// also wait for the move's store to memory in every step.
__device__ __forceinline__ void lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// The D passes of Alg. 2.  list: the layer's replicas grouped by rank, packed
// as expert | src << 10 | index << 20; range[r]: rank r's first and past-last
// entry.  A step reads its replicas' T and Q, reduces the scores, and the
// winning lane writes the move; the next step's rank and replicas, which no
// move changes, are read meanwhile.  Returns the number of routes.
template <typename V>
__device__ __forceinline__ int dispatch_passes(V* T, V* Q, u64* order, const uint32_t* range, const uint32_t* list, int R,
                                               int D, int64_t total, do_rem_move* out, int lane) {
  const V tf = (V)(total / R), tc = (V)((total + R - 1) / R);
  int n = 0;
  for (int d = 0; d < D; ++d) {
    const int before = n;
    // ranks by queue depth, ties by index: position = number of smaller keys
    for (int r = lane; r < R; r += kWave) {
      const V q = Q[r];
      int pos = 0;
#pragma unroll 8
      for (int o = 0; o < R; ++o) pos += Q[o] < q || (Q[o] == q && o < r) ? 1 : 0;
      order[pos] = (u64)(uint32_t)r | ((u64)range[r] << 32);
    }
    lds_order();
    // of the coming steps, step j + 2's rank and range and step j + 1's
    // replicas are read while step j runs
    u64 o1 = order[0], o2 = order[min(1, R - 1)];
    uint32_t e1 = list[min((int)((o1 >> 32) & 0xFFFFu) + lane, kMaxRep - 1)];
    for (int j = 0; j < R; ++j) {
      const int r = __builtin_amdgcn_readfirstlane((int)(uint32_t)o1);
      const uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)(o1 >> 32));
      const int lo = (int)(g & 0xFFFFu), hi = (int)(g >> 16);
      uint32_t ent = e1;
      o1 = o2;
      e1 = list[min((int)((o1 >> 32) & 0xFFFFu) + lane, kMaxRep - 1)];
      o2 = order[min(j + 2, R - 1)];
      V Qr = 0, t = 0, q = 0, best = (V)-2;
      uint32_t mine = 0xFFFFFFFFu;
      if (lo < hi) {
        Qr = Q[r];
        for (int i = lo + lane; i - lane < hi; i += kWave) {
          if (i - lane != lo) ent = list[min(i, kMaxRep - 1)];
          const V ti = T[ent & 1023u], qi = Q[(ent >> 10) & 1023u];
          const V s = i < hi ? benefit<V>(ti, qi, Qr, tf, tc) : (V)-2;
          const bool take = s > best || (s == best && (ent >> 20) < (mine >> 20));
          best = take ? s : best;
          mine = take ? ent : mine;
          t = take ? ti : t;
          q = take ? qi : q;
        }
        // replicas in the first 16 lanes: one row's reduction
        const V delta = hi - lo <= 16 ? row_max(best) : wave_max(best);
        if (delta > 0) {
          u64 m = __ballot(best == delta);
          if ((m & (m - 1)) != 0ull) {  // equal scores: the earliest replica
            const int idx = best == delta ? (int)(mine >> 20) : 0x7FFFFFFF;
            const int first = wave_min<int32_t>(idx);
            m = __ballot(idx == first);
          }
          if (lane == __builtin_ctzll(m)) {
            const int e = (int)(mine & 1023u), src = (int)((mine >> 10) & 1023u);
            Q[r] = Qr + delta;
            Q[src] = q - delta;
            T[e] = t - delta;
            do_rem_move o;
            o.expert = e;
            o.src_rank = src;
            o.dst_rank = r;
            o.reserved = 0;
            o.tokens = (int64_t)delta;
            out[n] = o;
          }
          ++n;
        }
      }
      lds_order();
    }
    if (n == before) break;  // nothing moved: every later pass would see the same
  }
  return n;
}

// The D passes for at most 64 ranks with at most kLaneReps replicas each: lane
// j holds the rank at position j of the pass's order and scores all of its
// replicas at once.  The first position at or after the current one with a
// positive score is the pass's next route; positions before it route nothing,
// as they would one after another.  So a pass takes one round per route and one
// more, not one step per rank (64 ranks, 4 replicas each: 81 -> 45 us).  More
// ranks, or more replicas on one, go through dispatch_passes, whose step costs
// the same for any number of them.
constexpr int kLaneReps = 8;
template <typename V>
__device__ __forceinline__ int dispatch_rounds(V* T, V* Q, u64* order, const uint32_t* range, const uint32_t* list,
                                               int R, int D, int64_t total, do_rem_move* out, int lane) {
  const V tf = (V)(total / R), tc = (V)((total + R - 1) / R);
  int n = 0;
  for (int d = 0; d < D; ++d) {
    const int before = n;
    if (lane < R) {
      const V q = Q[lane];
      int pos = 0;
#pragma unroll 8
      for (int o = 0; o < R; ++o) pos += Q[o] < q || (Q[o] == q && o < lane) ? 1 : 0;
      order[pos] = (u64)(uint32_t)lane | ((u64)range[lane] << 32);
    }
    lds_order();
    const u64 o = order[min(lane, R - 1)];
    const int r = (int)(uint32_t)o, lo = (int)((o >> 32) & 0xFFFFu);
    const int cnt = lane < R ? (int)(o >> 48) - lo : 0;
    uint32_t ent[kLaneReps];
    int most = 0;  // replicas of the busiest rank (wave-uniform)
#pragma unroll
    for (int i = 0; i < kLaneReps; ++i) {
      ent[i] = list[min(lo + i, kMaxRep - 1)];
      if (__ballot(cnt > i) != 0ull) most = i + 1;
    }
    u64 open = ~0ull;  // positions not yet passed
    while (true) {
      const V Qr = Q[r];
      V ti[kLaneReps], qi[kLaneReps];
#pragma unroll
      for (int i = 0; i < kLaneReps; ++i)
        if (i < most) {
          ti[i] = T[ent[i] & 1023u];
          qi[i] = Q[(ent[i] >> 10) & 1023u];
        }
      V t = 0, q = 0, best = 0;  // only positive scores count
      uint32_t mine = 0xFFFFFFFFu;
#pragma unroll
      for (int i = 0; i < kLaneReps; ++i)
        if (i < most) {
          const V s = i < cnt ? benefit<V>(ti[i], qi[i], Qr, tf, tc) : (V)-2;
          // equal scores: the earliest replica
          const bool take = s > best || (s == best && s > 0 && (ent[i] >> 20) < (mine >> 20));
          best = take ? s : best;
          mine = take ? ent[i] : mine;
          t = take ? ti[i] : t;
          q = take ? qi[i] : q;
        }
      const u64 m = __ballot(best > 0) & open;
      if (m == 0ull) break;
      const int j = __builtin_ctzll(m);
      if (lane == j) {
        const int e = (int)(mine & 1023u), src = (int)((mine >> 10) & 1023u);
        Q[r] = Qr + best;
        Q[src] = q - best;
        T[e] = t - best;
        do_rem_move o2;
        o2.expert = e;
        o2.src_rank = src;
        o2.dst_rank = r;
        o2.reserved = 0;
        o2.tokens = (int64_t)best;
        out[n] = o2;
      }
      ++n;
      open = j < 63 ? ~0ull << (j + 1) : 0ull;
      lds_order();
    }
    if (n == before) break;  // nothing moved: every later pass would see the same
    lds_order();
  }
  return n;
}

template <typename V>
__device__ __forceinline__ int dispatch_any(bool rounds, V* T, V* Q, u64* order, const uint32_t* range,
                                            const uint32_t* list, int R, int D, int64_t total, do_rem_move* out,
                                            int lane) {
  return rounds ? dispatch_rounds<V>(T, Q, order, range, list, R, D, total, out, lane)
                : dispatch_passes<V>(T, Q, order, range, list, R, D, total, out, lane);
}

// Alg. 2 for layer blockIdx.x (one wavefront).  replicas [L][rep_stride]
// with n_rep[l] valid entries (dst_rank = the rank holding the replica).
__global__ __launch_bounds__(kWave) void k_rem_dispatch(const do_rem_move* replicas, const int32_t* n_rep,
                                                        int rep_stride, const int64_t* tokens, RankMap rm, int E,
                                                        int D, do_rem_move* routes, int32_t* n_routes,
                                                        int64_t* queue_out, int64_t* tokens_out) {
  __shared__ int64_t T[kMaxE];
  __shared__ int64_t Q[kMaxE];
  __shared__ u64 order[kMaxE];
  __shared__ uint32_t range[kMaxE], fill[kMaxE];
  __shared__ uint32_t list[kMaxRep];
  const int lane = threadIdx.x, l = blockIdx.x, R = rm.R;
  bool ok = load_tokens(tokens + (int64_t)l * E, T, E, lane);
  const int nr = n_rep[l];
  ok = ok && nr >= 0 && nr <= rep_stride;
  const do_rem_move* rep = replicas + (int64_t)l * rep_stride;
  for (int r = lane; r < R; r += kWave) {
    Q[r] = 0;
    fill[r] = 0;
  }
  __syncthreads();
  if (ok) {
    bool bad = false;
    for (int i = lane; i < nr; i += kWave) {
      const do_rem_move m = rep[i];
      const bool b = m.expert < 0 || m.expert >= E || m.dst_rank < 0 || m.dst_rank >= R ||
                     m.src_rank != (int)rm.rank[m.expert];
      bad = bad || b;
      if (!b) atomicAdd(&fill[m.dst_rank], 1u);  // replicas per rank
    }
    ok = __ballot(bad) == 0ull;
  }
  if (!ok) {
    if (lane == 0) n_routes[l] = -1;
    return;
  }
  home_loads(T, rm, E, Q, lane);
  __syncthreads();
  // ranges of the ranks in `list`: an exclusive prefix sum of the counts
  uint32_t base = 0;
  bool rounds = R <= kWave;
  for (int r0 = 0; r0 < R; r0 += kWave) {
    const uint32_t c = r0 + lane < R ? fill[r0 + lane] : 0u;
    rounds = rounds && __ballot(c > (uint32_t)kLaneReps) == 0ull;
    uint32_t x = c;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)x, d);
      x += lane >= d ? y : 0u;
    }
    if (r0 + lane < R) {
      range[r0 + lane] = (base + x - c) | ((base + x) << 16);
      fill[r0 + lane] = base + x - c;
    }
    base += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  }
  __syncthreads();
  for (int i = lane; i < nr; i += kWave) {
    const do_rem_move m = rep[i];
    list[atomicAdd(&fill[m.dst_rank], 1u)] = (uint32_t)m.expert | ((uint32_t)m.src_rank << 10) | ((uint32_t)i << 20);
  }
  // entries past the last one are read (never used) up to a wavefront further
  for (int i = nr + lane; i < min(nr + kWave, kMaxRep); i += kWave) list[i] = 0u;
  int64_t part = 0;
  for (int r = lane; r < R; r += kWave) part += Q[r];
  const int64_t total = wave_sum_i64(part);
  do_rem_move* out = routes + (int64_t)l * R * D;
  int n;
  if (total < kSmall - R) {  // every volume and depth is at most the total
    // 32-bit copies in place: each pass of 64 entries is read before it is written below
    int32_t* T32 = reinterpret_cast<int32_t*>(T);
    int32_t* Q32 = reinterpret_cast<int32_t*>(Q);
    __syncthreads();
    for (int e0 = 0; e0 < max(E, R); e0 += kWave) {
      const int32_t a = e0 + lane < E ? (int32_t)T[e0 + lane] : 0;
      const int32_t b = e0 + lane < R ? (int32_t)Q[e0 + lane] : 0;
      __syncthreads();
      T32[e0 + lane] = a;
      Q32[e0 + lane] = b;
      __syncthreads();
    }
    n = dispatch_any<int32_t>(rounds, T32, Q32, order, range, list, R, D, total, out, lane);
    if (queue_out != nullptr)
      for (int r = lane; r < R; r += kWave) queue_out[(int64_t)l * R + r] = Q32[r];
    if (tokens_out != nullptr)
      for (int e = lane; e < E; e += kWave) tokens_out[(int64_t)l * E + e] = T32[e];
  } else {
    __syncthreads();
    n = dispatch_any<int64_t>(rounds, T, Q, order, range, list, R, D, total, out, lane);
    if (queue_out != nullptr)
      for (int r = lane; r < R; r += kWave) queue_out[(int64_t)l * R + r] = Q[r];
    if (tokens_out != nullptr)
      for (int e = lane; e < E; e += kWave) tokens_out[(int64_t)l * E + e] = T[e];
  }
  if (lane == 0) n_routes[l] = n;
}

template <int NE>
void run_allocate(const int64_t* rank_load, const int64_t* tokens, const RankMap& rm, int32_t E, int32_t D, int32_t L,
                  do_rem_move* moves, int32_t* n_moves, int64_t* load_out, int64_t* tokens_out, hipStream_t s) {
  if (rm.R <= kWave)
    hipLaunchKernelGGL((k_rem_allocate<NE, 1>), dim3((unsigned)L), dim3(kWave), 0, s, rank_load, tokens, rm, E, D,
                       moves, n_moves, load_out, tokens_out);
  else
    hipLaunchKernelGGL((k_rem_allocate<NE, kMaxE / kWave>), dim3((unsigned)L), dim3(kWave), 0, s, rank_load, tokens,
                       rm, E, D, moves, n_moves, load_out, tokens_out);
}

}  // namespace

hipError_t launch_rem_allocate(const int64_t* rank_load, const int64_t* tokens, const RankMap& rm, int32_t E,
                               int32_t D, int32_t L, do_rem_move* moves, int32_t* n_moves, int64_t* load_out,
                               int64_t* tokens_out, hipStream_t s) {
  // registers for 64, 128, 256 or 1,024 experts
  if (E <= 64)
    run_allocate<1>(rank_load, tokens, rm, E, D, L, moves, n_moves, load_out, tokens_out, s);
  else if (E <= 128)
    run_allocate<2>(rank_load, tokens, rm, E, D, L, moves, n_moves, load_out, tokens_out, s);
  else if (E <= 256)
    run_allocate<4>(rank_load, tokens, rm, E, D, L, moves, n_moves, load_out, tokens_out, s);
  else
    run_allocate<kMaxE / kWave>(rank_load, tokens, rm, E, D, L, moves, n_moves, load_out, tokens_out, s);
  return hipGetLastError();
}

hipError_t launch_rem_dispatch(const do_rem_move* replicas, const int32_t* n_rep, int32_t rep_stride,
                               const int64_t* tokens, const RankMap& rm, int32_t E, int32_t D, int32_t L,
                               do_rem_move* routes, int32_t* n_routes, int64_t* queue_out, int64_t* tokens_out,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_rem_dispatch, dim3((unsigned)L), dim3(kWave), 0, s, replicas, n_rep, rep_stride, tokens, rm, E,
                     D, routes, n_routes, queue_out, tokens_out);
  return hipGetLastError();
}

}  // namespace dol
