// Host dispatch of the Top-K kernel (topk_kernel.h), the run-time choice of
// its unit schedule, and the MFMA Gram of stored signatures.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <mutex>

#include "topk_kernel.h"

namespace dol {
namespace {

// Process-wide overrides of choices that never change results (do_set_option):
// the Gram kind and the unit schedule.
std::atomic<int> g_opt_gram{0};    // 0: fp4 MFMA, 1: VALU popcount
std::atomic<int> g_opt_sched{-1};  // -1: measured per launch shape, else an index into kSchedCand

int gram_mode() { return g_opt_gram.load(std::memory_order_relaxed) == 1 ? kGramPopc : kGramMfma; }

// Segments on unit boundaries (the condition of the kAligned rows).
bool aligned_segments(const SegTable& tab) {
  for (int i = 0; i < tab.nseg; ++i)
    if (tab.s[i].n % 512 != 0 || tab.s[i].tok_off % 512 != 0) return false;
  return true;
}

// kAligned against kDirect: bf16 at 128 experts -11 %; fp32 at 256 experts
// -8.5 % without signature output and -5 % with it where the stores are cheap
// (halved SGPR spills)
template <typename T, int EP>
hipError_t launch_rows(RowMode mode, const SegTable& tab, const PathArgs& a, Sched sc, hipStream_t s,
                       const ProfEv& pe) {
  if (mode == kAligned) return launch_mode<T, EP, kAligned>(gram_mode(), tab, a, true, sc, s, pe);
  return launch_mode<T, EP, kDirect>(gram_mode(), tab, a, true, sc, s, pe);
}

template <typename T>
hipError_t launch_ep(RowMode mode, const SegTable& tab, const PathArgs& a, Sched sc, hipStream_t s, const ProfEv& pe) {
  if (a.E <= 32) return launch_rows<T, 32>(mode, tab, a, sc, s, pe);
  if (a.E <= 64) return launch_rows<T, 64>(mode, tab, a, sc, s, pe);
  if (a.E <= 128) return launch_rows<T, 128>(mode, tab, a, sc, s, pe);
  return launch_rows<T, 256>(mode, tab, a, sc, s, pe);
}

// Launch-time choice of the unit schedule for large launches.  The cost of
// the signature stores under a given schedule differs between otherwise
// identical boards (it follows how the concurrent store streams fall on
// the HBM channels), while it repeats within one process.  So for each
// large launch shape the first launches try the candidates in turn with
// events around them; completed measurements are collected with
// hipEventQuery, which never waits, and once every candidate has kTuneTrials
// of them, the one with the fastest launch is used for all later launches of
// that shape (it must beat the first candidate by 2 %).  Measuring starts
// kTuneDelayMs after the first launch of a shape: launches right after an idle
// period run slower for some tens of milliseconds (7.3 ms falling to 5.6 ms
// over the first six launches of workload 4), which would hide a 12 %
// difference between the schedules.  Launches under stream capture and
// launches below kTuneMinUnits use the first candidate (or the one already
// chosen for the shape); a capture never touches the measurement events.
// When every slot of the table holds a shape, a decided one is recycled.
constexpr Sched kSchedCand[2] = {Sched{4, 3}, Sched{0, 0}};  // XCD partitions; contiguous ranges
constexpr int kNumCand = 2;
constexpr int64_t kTuneMinUnits = 1024;  // 512 Ki tokens
constexpr int kTuneTrials = 3;           // measured launches per candidate
constexpr double kTuneDelayMs = 100.0;   // no measurement before this long after a shape's first launch
constexpr int kTuneSlots = 16;

struct Tune {
  uint64_t key;
  int device;
  int calls;
  std::chrono::steady_clock::time_point first;  // host time of the shape's first launch
  int chosen;                 // index into kSchedCand, or -1 while measuring
  float best[kNumCand];       // fastest completed launch per candidate (ms), < 0 if none yet
  int trials[kNumCand];       // completed measurements per candidate
  bool pending[kNumCand];     // a measured launch is in flight
  hipEvent_t ev[kNumCand][2];
};
std::mutex g_tune_mu;
Tune g_tune[kTuneSlots];
int g_ntune = 0;
int g_tune_next = 0;  // next slot considered for recycling

uint64_t mix(uint64_t h, uint64_t v) {
  h ^= v + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
  return h;
}

void release_events(Tune& t) {
  for (int c = 0; c < kNumCand; ++c)
    for (int i = 0; i < 2; ++i)
      if (t.ev[c][i] != nullptr) {
        (void)hipEventDestroy(t.ev[c][i]);
        t.ev[c][i] = nullptr;
      }
}

void decide(Tune& t, int c) {
  t.chosen = c;
  release_events(t);  // no trial is pending once a candidate is chosen
}

// Picks the schedule of one launch and, when it is a measured trial, sets
// *ev_out to the candidate's start/stop events.
Sched tuned_schedule(do_dtype dt, const SegTable& tab, const PathArgs& a, RowMode mode, bool fast, hipStream_t s,
                     hipEvent_t* ev_out) {
  ev_out[0] = ev_out[1] = nullptr;
  const int64_t units = tab.tile_start[tab.nseg];
  if (units < kTuneMinUnits) return kSchedCand[0];
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return kSchedCand[0];
  uint64_t key = 0;
  key = mix(key, (uint64_t)dt);
  key = mix(key, (uint64_t)a.E);
  key = mix(key, (uint64_t)a.k);
  key = mix(key, (uint64_t)units);
  key = mix(key, (uint64_t)tab.nseg);
  key = mix(key, (uint64_t)tab.s[tab.nseg - 1].layer - (uint64_t)tab.s[0].layer);
  key = mix(key, (uint64_t)(a.bits != nullptr) | ((uint64_t)(a.cacc != nullptr) << 1) |
                     ((uint64_t)a.or_partial << 2) | ((uint64_t)fast << 3) | ((uint64_t)mode << 4));
  std::lock_guard<std::mutex> lock(g_tune_mu);
  Tune* t = nullptr;
  for (int i = 0; i < g_ntune; ++i)
    if (g_tune[i].key == key && g_tune[i].device == dev) t = &g_tune[i];
  if (t != nullptr && t->chosen >= 0) return kSchedCand[t->chosen];
  if (capturing) return kSchedCand[0];
  if (t == nullptr) {
    if (g_ntune < kTuneSlots) {
      t = &g_tune[g_ntune++];
    } else {
      for (int i = 0; i < kTuneSlots && t == nullptr; ++i) {
        Tune& c = g_tune[(g_tune_next + i) % kTuneSlots];
        if (c.chosen >= 0) {
          t = &c;
          g_tune_next = (g_tune_next + i + 1) % kTuneSlots;
        }
      }
      if (t == nullptr) return kSchedCand[0];  // every slot is still measuring
    }
    *t = Tune{};
    t->key = key;
    t->device = dev;
    t->chosen = -1;
    for (int c = 0; c < kNumCand; ++c) t->best[c] = -1.f;
  }
  // collect finished trials
  bool all = true;
  for (int c = 0; c < kNumCand; ++c) {
    if (t->pending[c]) {
      const hipError_t q = hipEventQuery(t->ev[c][1]);
      if (q == hipSuccess) {
        float ms = -1.f;
        if (hipEventElapsedTime(&ms, t->ev[c][0], t->ev[c][1]) == hipSuccess && ms > 0.f) {
          t->best[c] = t->best[c] < 0.f ? ms : std::min(t->best[c], ms);
          ++t->trials[c];
        }
        t->pending[c] = false;
      } else if (q != hipErrorNotReady) {
        t->pending[c] = false;
        decide(*t, 0);  // measurement failed: keep the first candidate
        return kSchedCand[0];
      }
    }
    all = all && t->trials[c] >= kTuneTrials;
  }
  if (all) {
    int bc = 0;
    for (int c = 1; c < kNumCand; ++c)
      if (t->best[c] < 0.98f * t->best[bc]) bc = c;  // switch only for a clear gain
    if (getenv("DOLOSS_TUNE_LOG") != nullptr)
      fprintf(stderr, "[doloss] unit schedule for %lld units: candidates %.4f / %.4f ms, chose %d\n",
              (long long)units, t->best[0], t->best[1], bc);
    decide(*t, bc);
    return kSchedCand[bc];
  }
  const auto now = std::chrono::steady_clock::now();
  if (t->calls++ == 0) t->first = now;
  if (std::chrono::duration<double, std::milli>(now - t->first).count() < kTuneDelayMs) return kSchedCand[0];
  // the candidate with the fewest measurements that has none in flight
  // (ties to the one measured least recently, so the candidates alternate)
  int pick = -1;
  for (int i = 0; i < kNumCand; ++i) {
    const int c = (t->calls + i) % kNumCand;
    if (t->pending[c] || t->trials[c] >= kTuneTrials) continue;
    if (pick < 0 || t->trials[c] < t->trials[pick]) pick = c;
  }
  if (pick < 0) return kSchedCand[0];  // every candidate still has a launch in flight
  if (t->ev[pick][0] == nullptr) {
    if (hipEventCreate(&t->ev[pick][0]) != hipSuccess || hipEventCreate(&t->ev[pick][1]) != hipSuccess) {
      decide(*t, 0);
      return kSchedCand[0];
    }
  }
  t->pending[pick] = true;
  ev_out[0] = t->ev[pick][0];
  ev_out[1] = t->ev[pick][1];
  return kSchedCand[pick];
}

// ---------------------------------------------------------------------------
// Gram of stored signatures of 97 to 256 experts (which of them:
// launch_gram_mfma) on the same fp4 MFMA tiles as k_topk.  Block b takes layer b / bpl and the part b % bpl of
// that layer's 8-word chunks, kGramGroup chunks per step.  A chunk's words of
// every expert are staged in LDS in the bit-tile layout of k_topk (word s of
// expert e at s * EP + (e ^ bt_swz(s))); the next step's words are loaded
// into registers while the current step is multiplied, so one barrier and one
// memory round trip cover kGramGroup chunks.  Each block adds its counts into
// cacc at the end; its chunk count stays below 2^24 / 512 (exact fp32 counts).
// ---------------------------------------------------------------------------
constexpr int64_t kGramMaxChunks = ((1 << 24) / 512) - 1;
constexpr int kGramGroup = 4;  // chunks per step

template <int EP>
__global__ __launch_bounds__(kFusedThreads) void k_gram_mfma(const u64* bits, int64_t W, int E, int L, int bpl,
                                                             uint32_t* cacc, bool pair64) {
  constexpr int kTileWords = EP * kFusedWaves;
  constexpr int kPer = kTileWords / kFusedThreads;  // words per thread and chunk: 2 or 4
  typedef GramShape<EP> GS;
  typedef typename Mfma<GS::TS>::Acc Acc;
  __shared__ __align__(16) u64 bt[2][kGramGroup][kTileWords];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = (int)blockIdx.x / bpl, part = (int)blockIdx.x % bpl;
  if (l >= L) return;
  const int64_t nch = (W + kFusedWaves - 1) / kFusedWaves;
  const int64_t c0 = part * nch / bpl, c1 = (part + 1) * nch / bpl;
  if (c0 >= c1) return;
  const u64* lb = bits + (int64_t)l * E * sig_words(W);
  const WaveTiles wt = wave_tiles(GS::T, wave);
  Acc acc[kGP];
#pragma unroll
  for (int p = 0; p < kGP; ++p)
#pragma unroll
    for (int r = 0; r < Mfma<GS::TS>::kRegs; ++r) acc[p][r] = 0.0f;
  // thread tid holds words (e, s) = (idx / 8, idx % 8) for idx = tid + q * 512
  // of each chunk: a chunk is one unit of the signature layout, E * 64
  // contiguous bytes; chunks at or past c1 read as zero
  u64 r[kGramGroup][kPer];
  auto load = [&](int64_t g0) {
#pragma unroll
    for (int g = 0; g < kGramGroup; ++g)
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int idx = tid + q * kFusedThreads, e = idx >> 3;
        const int64_t w = (g0 + g) * kFusedWaves + (idx & 7);
        r[g][q] = (g0 + g < c1 && e < E && w < W)
                      ? __builtin_nontemporal_load(lb + sig_off(w, e, E))
                      : 0ull;
      }
  };
  load(c0);
  int buf = 0;
  for (int64_t g0 = c0; g0 < c1; g0 += kGramGroup) {
#pragma unroll
    for (int g = 0; g < kGramGroup; ++g)
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int idx = tid + q * kFusedThreads, e = idx >> 3, sl = idx & 7;
        bt[buf][g][sl * EP + (e ^ bt_swz(sl))] = r[g][q];
      }
    // the tiles are complete; every wave is done with the tiles written two
    // steps ago (it multiplied those before reaching this barrier)
    __syncthreads();
    if (g0 + kGramGroup < c1) load(g0 + kGramGroup);
    const int ng = (int)min((int64_t)kGramGroup, c1 - g0);
    for (int g = 0; g < ng; ++g) mfma_slots<GS::TS>(acc, wt, bt[buf][g], EP, 0, kFusedWaves, lane);
    buf ^= 1;
  }
  mfma_flush<GS::TS>(acc, wt, cacc + (int64_t)l * E * E, E, lane, (int)(blockIdx.x % kGP), pair64);
}

// ---------------------------------------------------------------------------
// Gram of stored signatures up to 128 experts (NT tiles of 32).  Bound by the
// matrix cores.  Every wave multiplies whole units by itself: lane l loads 32
// bytes of expert l % 32 of each tile (its half l / 32 of the unit's words)
// straight into the operand layout, so nothing is staged in LDS, no barrier
// runs between units, and a word is expanded once for all NT (NT + 1) / 2
// tile pairs instead of once per wave that uses its tile (k_gram_mfma: four
// times at 128 experts).  The token order along k follows the lane halves and
// is the same in both operands.  Loads run two units ahead.
// do_pairwise_hamming of 48 layers x 262,144 tokens, k_gram_mfma -> this: 32
// experts 55 -> 25 us, 64: 69 -> 39, 96: 135 -> 59, 128: 139 -> 84 to 87; one
// layer of 1,048,576 tokens, 128 experts: 41 -> 36 us.
// The units of all layers are split evenly over the blocks; a block sums its
// four waves' counts in LDS and adds them at the end of a layer and at the
// latest after kGramMaxChunks units, so that every sum is exact in fp32.
// ---------------------------------------------------------------------------
constexpr int kGuWaves = 4;

template <int NT>
__global__ __launch_bounds__(kGuWaves * kWave, 1) void k_gram_units(const u64* bits, int64_t W, int E, int L,
                                                                    uint32_t* cacc, bool pair64) {
  constexpr int NP = NT * (NT + 1) / 2;
  typedef v4u v4u_any8 __attribute__((aligned(8)));
  __shared__ float sum[NP][16][kWave];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t last_on = (NT - 1) * 32 + (lane & 31) < E ? ~0u : 0u;  // the last tile's experts past E
  const int64_t U = (W + 7) >> 3, T = (int64_t)L * U;
  const int64_t t1 = (int64_t)((unsigned __int128)T * (blockIdx.x + 1) / gridDim.x);
  for (int64_t t = (int64_t)((unsigned __int128)T * blockIdx.x / gridDim.x); t < t1;) {
    const int64_t l = t / U, u0 = t - l * U;
    const int64_t n = min(min(t1 - t, U - u0), kGramMaxChunks);
    const u64* lb = bits + l * E * sig_words(W) + u0 * E * 8;
    v16f acc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[p][r] = 0.0f;
    // unit i of the segment (past its end: the last one again, not multiplied)
    auto load = [&](int64_t i, v4u (&r)[NT][2]) __attribute__((always_inline)) {
      const u64* ub = lb + min(i, n - 1) * E * 8 + half * 4;
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const v4u_any8* p = reinterpret_cast<const v4u_any8*>(ub + min(a * 32 + (lane & 31), E - 1) * 8);
        r[a][0] = __builtin_nontemporal_load(p);
        r[a][1] = __builtin_nontemporal_load(p + 1);
      }
    };
    auto mult = [&](int64_t i, v4u (&r)[NT][2]) __attribute__((always_inline)) {
      if (i >= n) return;
#pragma unroll
      for (int d = 0; d < 8; ++d) r[NT - 1][d >> 2][d & 3] &= last_on;
      if (8 * (u0 + i) + 8 > W) {  // words past W
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const uint32_t in = 8 * (u0 + i) + half * 4 + (d >> 1) < W ? ~0u : 0u;
#pragma unroll
          for (int a = 0; a < NT; ++a) r[a][d >> 2][d & 3] &= in;
        }
      }
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        v8i f[NT];
#pragma unroll
        for (int a = 0; a < NT; ++a) f[a] = expand32_fp4(r[a][d >> 2][d & 3]);
        int p = 0;
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = a; b < NT; ++b, ++p) acc[p] = Mfma<32>::mac(f[a], f[b], acc[p]);
      }
    };
    v4u ra[NT][2], rb[NT][2], rc[NT][2];
    load(wave, ra);
    load(wave + kGuWaves, rb);
    load(wave + 2 * kGuWaves, rc);
#pragma unroll 1
    for (int64_t i = wave; i < n; i += 3 * kGuWaves) {
      mult(i, ra);
      load(i + 3 * kGuWaves, ra);
      mult(i + kGuWaves, rb);
      load(i + 4 * kGuWaves, rb);
      mult(i + 2 * kGuWaves, rc);
      load(i + 5 * kGuWaves, rc);
    }
    // one wave after the other (LDS float atomics took twice the kernel's time);
    // unrolled, so that the first wave's stores read nothing
#pragma unroll
    for (int w = 0; w < kGuWaves; ++w) {
      if (w < n) {  // the waves that had a unit
        if (w == wave) {
#pragma unroll
          for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[p][r][lane] = w == 0 ? acc[p][r] : sum[p][r][lane] + acc[p][r];
        }
        __syncthreads();
      }
    }
    for (int p = wave; p < NP; p += kGuWaves) {
      int I = 0, J = p;
      while (J >= NT - I) {
        J -= NT - I;
        ++I;
      }
      v16f v;
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = sum[p][r][lane];
      flush_slot<32>(v, I, I + J, cacc + l * E * E, E, lane, pair64);
    }
    __syncthreads();  // the sums are read before the next segment's
    t += n;
  }
}

// ---------------------------------------------------------------------------
// Gram of stored signatures beyond 256 experts.  A block multiplies one pair
// (I, J), I <= J, of 128-expert groups over a range of a layer's units: wave w
// owns row tile w / 2 of I against column tiles 2 (w % 2) and 2 (w % 2) + 1 of
// J (32 x 32 experts each), so a word costs it three fragment expansions and
// two MFMAs.  kWideGroup units of both groups are staged in LDS in the bit-tile
// layout while the next ones are loaded into registers.  Every block adds 128
// x 128 counts at its end, which is why launch_gram_wide asks for about one
// block per CU only: the atomics of 512 experts on two blocks per CU cost more
// than the multiplication.  262,144 tokens of 512 experts: 41 us, against 200
// us for the popcount kernel.
// ---------------------------------------------------------------------------
constexpr int kGroup = 128;   // experts per group
constexpr int kWideGroup = 2; // units per step

__global__ __launch_bounds__(kFusedThreads) void k_gram_wide(const u64* bits, int64_t W, int64_t ld, int E, int pairs,
                                                             int slices, uint32_t* cacc, bool pair64) {
  constexpr int kTile = kGroup * kFusedWaves;  // words of one group and unit
  typedef v2u64 v2u64_any __attribute__((aligned(8)));
  __shared__ __align__(16) u64 bt[2][kWideGroup][2][kTile];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b = (int)blockIdx.x;
  const int pr = b % pairs;
  b /= pairs;
  const int part = b % slices, l = b / slices;
  const int ngr = (E + kGroup - 1) / kGroup;
  int I = 0, J = pr;
  while (J >= ngr - I) {
    J -= ngr - I;
    ++I;
  }
  J += I;
  const int64_t U = (W + 7) >> 3;
  const int64_t u0 = part * U / slices, u1 = (part + 1) * U / slices;
  if (u0 >= u1) return;
  const u64* lb = bits + (int64_t)l * E * ld;
  const int nside = I == J ? 1 : 2;
  // thread tid loads word pair tid % 4 of the group's expert tid / 4, 16 bytes
  const int te = tid >> 2, ts = 2 * (tid & 3);
  v2u64 r[kWideGroup][2];
  auto load = [&](int64_t g0) {
#pragma unroll
    for (int g = 0; g < kWideGroup; ++g)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int e = (x == 0 ? I : J) * kGroup + te;
        v2u64 v = {0ull, 0ull};
        if (x < nside && g0 + g < u1 && e < E)
          v = *reinterpret_cast<const v2u64_any*>(lb + ((g0 + g) * E + e) * 8 + ts);
        const int64_t w = (g0 + g) * 8 + ts;  // words at or past W are not part of the history
        r[g][x] = v2u64{w < W ? v[0] : 0ull, w + 1 < W ? v[1] : 0ull};
      }
  };
  const int rt = wave >> 1, ct = 2 * (wave & 1);
  const bool on[2] = {I != J || ct >= rt, I != J || ct + 1 >= rt};
  v16f acc[2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[p][i] = 0.0f;
  load(u0);
  int buf = 0;
  for (int64_t g0 = u0; g0 < u1; g0 += kWideGroup) {
#pragma unroll
    for (int g = 0; g < kWideGroup; ++g)
#pragma unroll
      for (int x = 0; x < 2; ++x)
        if (x < nside) {
          bt[buf][g][x][ts * kGroup + (te ^ bt_swz(ts))] = r[g][x][0];
          bt[buf][g][x][(ts + 1) * kGroup + (te ^ bt_swz(ts + 1))] = r[g][x][1];
        }
    __syncthreads();  // as in k_gram_mfma: one barrier per step, two buffers
    if (g0 + kWideGroup < u1) load(g0 + kWideGroup);
    if (on[0] || on[1]) {
#pragma unroll 1
      for (int g = 0; g < kWideGroup; ++g) {
        const uint32_t* ta = reinterpret_cast<const uint32_t*>(bt[buf][g][0]);
        const uint32_t* tb = reinterpret_cast<const uint32_t*>(bt[buf][g][nside - 1]);
#pragma unroll
        for (int s = 0; s < kFusedWaves; ++s) {
          const int h = lane >> 5, le = (lane & 31) ^ bt_swz(s);
          const v8i fa = expand32_fp4(ta[(s * kGroup + rt * 32 + le) * 2 + h]);
          const v8i f0 = expand32_fp4(tb[(s * kGroup + ct * 32 + le) * 2 + h]);
          const v8i f1 = expand32_fp4(tb[(s * kGroup + ct * 32 + 32 + le) * 2 + h]);
          acc[0] = Mfma<32>::mac(fa, f0, acc[0]);
          acc[1] = Mfma<32>::mac(fa, f1, acc[1]);
        }
      }
    }
    buf ^= 1;
  }
  uint32_t* c = cacc + (int64_t)l * E * E;
#pragma unroll
  for (int p = 0; p < 2; ++p)
    if (on[p]) flush_slot<32>(acc[p], I * 4 + rt, J * 4 + ct + p, c, E, lane, pair64);
}

}  // namespace

hipError_t launch_topk(do_dtype dt, SegTable& tab, int nseg, const PathArgs& a, bool vec_rows, hipStream_t s,
                       const ProfEv& pe) {
  tab.nseg = nseg;
  tab.tile_start[0] = 0;
  for (int i = 0; i < nseg; ++i) {
    const int64_t n = tab.s[i].n, off = tab.s[i].tok_off;
    const int64_t words = n > 0 ? ((off + n - 1) >> 6) - (off >> 6) + 1 : 0;
    tab.tile_start[i + 1] = tab.tile_start[i] + (words + kFusedWaves - 1) / kFusedWaves;  // 8-word units
  }
  if (tab.tile_start[nseg] == 0) {  // nothing to launch: the timing events still complete, back to back
    if (pe.start != nullptr) {
      const hipError_t e = hipEventRecord(pe.start, s);
      if (e != hipSuccess) return e;
    }
    return pe.stop != nullptr ? hipEventRecord(pe.stop, s) : hipSuccess;
  }
  if (a.E > kFastMaxE && a.k <= kWideMaxK) return launch_wide(dt, tab, a, s, pe);
  // the in-register ranking needs rows of at least one 16-byte piece
  const int rowB = a.E * (dt == DO_F32 ? 4 : 2);
  const bool fast = rowB >= 16 && a.k <= kFastMaxK && a.E <= kFastMaxE;
  // 16-byte aligned rows load straight into LDS at every length but one piece;
  // kRagged, which takes them too, was 0 to 46 % slower than kPieces (see RowMode).
  // It packs the 64 rows of one piece into a single load: 4 fp32 experts, 4 x
  // 262,144 tokens 25.6 us, kPieces 26.9, 100,003 tokens (do_fused) 21.5 and 23.2.
  const RowMode mode = !vec_rows || !fast || rowB == 16 ? kRagged
                       : rowB % 128 != 0                ? kPieces
                       : !aligned_segments(tab)         ? kDirect
                                                        : kAligned;
  hipEvent_t ev[2] = {nullptr, nullptr};
  const int forced = g_opt_sched.load(std::memory_order_relaxed);
  Sched sc = forced >= 0 ? kSchedCand[forced] : tuned_schedule(dt, tab, a, mode, fast, s, ev);
  // partitions of about one layer each: a block flushes its Gram counts once per
  // layer it works in.  do_fused of bf16 scores with 128 experts, us with 8 / 16 /
  // 32 partitions: 16 layers x 65,536 tokens 90 / 74 / 74, 32 x 65,536 164 / 134 /
  // 121, 48 x 16,384 76.5 / 74.7 / 73.9, 48 x 262,144 685 / 653 / 636.  Below 16
  // layers the choice is not clear: 8 layers x 262,144 take 150 / 125 / 129 in
  // bf16 and 193 / 198 / 202 in fp32.  Below four units per CU a block's share is
  // one range; small partitions that it does not divide move those ranges off the
  // layers' ends (36 layers x 3,762: 36.1 / 36.4 / 41.3, in fp32 41.5 / 41.5 /
  // 46.3), even ones gain a little (48 x 8,192: 49.3 / 48.5 / 48.4).
  const int layers = tab.s[nseg - 1].layer - tab.s[0].layer + 1;
  const int64_t units = tab.tile_start[nseg], cus = device_info().cu_count;
  if (sc.lp == 3 && a.cacc != nullptr && (units >= 4 * cus || units % cus == 0))
    sc.lp = layers >= 32 ? 5 : layers >= 16 ? 4 : 3;
  // a tuner trial binds its events to the dispatch (the kernel alone), unless
  // the caller's timing events already are; then they go around the launch
  ProfEv use = pe;
  const bool around = ev[0] != nullptr && (pe.start != nullptr || pe.stop != nullptr);
  if (ev[0] != nullptr && !around) use = ProfEv{ev[0], ev[1]};
  if (around) {
    const hipError_t e = hipEventRecord(ev[0], s);
    if (e != hipSuccess) return e;
  }
  const hipError_t e = mode == kRagged ? launch_ragged(dt, gram_mode(), tab, a, fast, sc, s, use)
                       : mode == kPieces ? launch_pieces(dt, gram_mode(), tab, a, sc, s, use)
                       : dt == DO_F32  ? launch_ep<float>(mode, tab, a, sc, s, use)
                                       : launch_ep<uint16_t>(mode, tab, a, sc, s, use);
  if (e != hipSuccess || !around) return e;
  return hipEventRecord(ev[1], s);
}

bool gram_mfma_enabled() { return gram_mode() == kGramMfma; }

bool set_option(int opt, int value) {
  if (opt == DO_OPT_SCHEDULE && value >= -1 && value < kNumCand) {
    g_opt_sched.store(value, std::memory_order_relaxed);
    return true;
  }
  if (opt == DO_OPT_GRAM && (value == 0 || value == 1)) {
    g_opt_gram.store(value, std::memory_order_relaxed);
    return true;
  }
  return false;
}

hipError_t launch_gram_mfma(const u64* bits, int64_t W, int64_t ld, int32_t E, int32_t L, uint32_t* cacc,
                            hipStream_t s) {
  if (W < 1) return hipErrorInvalidValue;
  const int64_t nch = (W + kFusedWaves - 1) / kFusedWaves;
  const DevInfo di = device_info();
  if (E > kFastMaxE) {
    const int64_t ngr = (E + kGroup - 1) / kGroup, pairs = ngr * (ngr + 1) / 2;
    int64_t slices = std::max<int64_t>(1, di.cu_count / (pairs * L));
    slices = std::max<int64_t>(slices, (nch + kGramMaxChunks - 1) / kGramMaxChunks);
    slices = std::min<int64_t>(slices, nch);
    if ((int64_t)L * pairs * slices > 0x7FFFFFFF) return hipErrorInvalidValue;
    const bool p64 = (E & 1) == 0 && (reinterpret_cast<uintptr_t>(cacc) & 7) == 0;
    hipLaunchKernelGGL(k_gram_wide, dim3((unsigned)(L * pairs * slices)), dim3(kFusedThreads), 0, s, bits, W, ld, E,
                       (int)pairs, (int)slices, cacc, p64);
    return hipGetLastError();
  }
  if (ld != sig_words(W)) return hipErrorInvalidValue;
  const bool pair64 = (E & 1) == 0 && (reinterpret_cast<uintptr_t>(cacc) & 7) == 0;
  if (E <= 96 || (E <= 128 && (int64_t)L * nch >= di.cu_count)) {
    // one wave per SIMD keeps the matrix cores busy with three or four tiles;
    // below that the loads of two are needed to keep the memory busy
    const int64_t per_cu = E <= 64 ? 2 : 1;
    const dim3 grid((unsigned)std::min<int64_t>(di.cu_count * per_cu, (int64_t)L * nch));
    const dim3 block(kGuWaves * kWave);
    switch ((E + 31) / 32) {
      case 1: hipLaunchKernelGGL(k_gram_units<1>, grid, block, 0, s, bits, W, E, L, cacc, pair64); break;
      case 2: hipLaunchKernelGGL(k_gram_units<2>, grid, block, 0, s, bits, W, E, L, cacc, pair64); break;
      case 3: hipLaunchKernelGGL(k_gram_units<3>, grid, block, 0, s, bits, W, E, L, cacc, pair64); break;
      default: hipLaunchKernelGGL(k_gram_units<4>, grid, block, 0, s, bits, W, E, L, cacc, pair64); break;
    }
    return hipGetLastError();
  }
  // fewer units than CUs of 97 to 128 experts (8 units: 18.3 us, k_gram_units 22.9
  // us), and more than 128 experts: one block per CU and layer share (the kernel
  // takes 208 VGPRs at 256), each below the exact-count limit; every block flushes
  // its counts with atomics at its end
  int64_t bpl = std::max<int64_t>(1, ((int64_t)di.cu_count + L - 1) / L);
  bpl = std::max<int64_t>(bpl, (nch + kGramMaxChunks - 1) / kGramMaxChunks);
  bpl = std::min<int64_t>(bpl, nch);
  if ((int64_t)L * bpl > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(L * bpl));
  if (E <= 128)
    hipLaunchKernelGGL(k_gram_mfma<128>, grid, dim3(kFusedThreads), 0, s, bits, W, E, L, (int)bpl, cacc, pair64);
  else
    hipLaunchKernelGGL(k_gram_mfma<256>, grid, dim3(kFusedThreads), 0, s, bits, W, E, L, (int)bpl, cacc, pair64);
  return hipGetLastError();
}

}  // namespace dol
