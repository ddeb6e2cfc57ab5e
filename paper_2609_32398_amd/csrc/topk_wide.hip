// Top-K and signature packing for more than 256 experts (up to 1,024) and
// k <= 16: the experts no longer fit the 8 index bits of k_topk's keys, and
// its two signature tiles and stage buffers no longer fit the LDS.
//
// A block of 4 wavefronts owns 4 consecutive signature words (half a unit) per
// step; lane l of wave w ranks token 64 * word + l.  A wave streams its 64
// rows in 128-byte column chunks: the next chunk is loaded into registers
// (16-byte loads at the rows' own alignment, 8 rows of 8 pieces per
// instruction) while the current one is ranked from the wave's 8 KiB stage
// buffer, so one chunk per wave is always in flight.  Keys are 32-bit
// composites as in k_topk, with more index bits: bf16 keys keep all 16 value
// bits above a 16-bit complemented index; fp32 keys keep 22 value bits above
// 10 index bits, and a token whose k-th and (k+1)-th keys share a bucket is
// settled by the whole wave from the full values.  Keys are inserted into a
// sorted list of KL = 8 or 16 with one v_med3 per entry.
//
// Bound by the VALU: about 19 instructions per score with the list of 16.  512
// bf16 experts, 262,144 tokens: k = 12 638 us with the exact per-lane selection
// (every lane reading its own row), 92 us here (268 MB of scores: 2.9 TB/s).
#include "topk_kernel.h"

namespace dol {
namespace {

constexpr int kWideWaves = 4;  // words per block step (half a unit)
constexpr int kWideThreads = kWideWaves * kWave;

template <typename T>
struct WideKey;
template <>
struct WideKey<float> {
  static constexpr int kIdxBits = 10;
  static constexpr int kPosMin = 0x400;                 // positive keys: the threshold must be >= this
  static constexpr int kZeroLo = -1024, kZeroHi = 1023;  // general keys of the -0 / +0 buckets
};
template <>
struct WideKey<uint16_t> {
  static constexpr int kIdxBits = 16;
  static constexpr int kPosMin = 0x10000;
  static constexpr int kZeroLo = -65536, kZeroHi = 65535;
};

// insert8 for a list of KL entries.
template <int KL, bool TRACK>
__device__ __forceinline__ void insert_key(int (&top)[KL], int x, int& rej) {
  if (TRACK) rej = med3(rej, top[KL - 1], x);
#pragma unroll
  for (int i = KL - 1; i > 0; --i) top[i] = med3(top[i], top[i - 1], x);
  top[0] = max(top[0], x);
}

__device__ __forceinline__ int bfi(uint32_t mask, uint32_t x, uint32_t sidx) {
  int r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(x), "s"(sidx));
  return r;
}

// Rank the first nv pieces of a staged chunk (piece q of row r at slot
// q ^ stage_swz(r, 3)).  e0: expert of the chunk's first element; tail_q / dup
// as in rank_staged.  hi: byte or bit mask of the value bits (a VGPR).
template <typename T, int KL, bool GEN>
__device__ __forceinline__ void rank_wide(const unsigned char* sbuf, int lane, int e0, int nv, int tail_q, int dup,
                                          int E, uint32_t vmask, uint32_t sel_lo, uint32_t sel_hi, int (&top)[KL],
                                          int& rej) {
  constexpr int kV = Traits<T>::kVec;
  const unsigned char* row = sbuf + lane * 128;
  const int sw = stage_swz(lane, 3) << 4;
  auto piece = [&](int q) { return *reinterpret_cast<const v4u*>(row + ((min(q, nv - 1) << 4) ^ sw)); };
  v4u xn = piece(0);
#pragma unroll 1
  for (int q = 0; q < nv; ++q) {
    v4u x = xn;
    xn = piece(q + 1);
    int e = e0 + q * kV;
    if (q == tail_q) {  // the row's last 16 bytes: the first dup bytes repeat the piece before it
      e = E - kV;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int b = dup - 4 * i;
        x[i] |= b >= 4 ? ~0u : b == 2 ? 0xFFFFu : 0u;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t u = x[i];
      if constexpr (kV == 4) {
        if (GEN) u ^= (uint32_t)((int32_t)u >> 31) & 0x7FFFFFFFu;
        insert_key<KL, true>(top, bfi(vmask, u, (uint32_t)(1023 - (e + i))), rej);
      } else {
        const v2s s = __builtin_bit_cast(v2s, u) >> (short)15;
        u ^= __builtin_bit_cast(uint32_t, s) & 0x7FFF7FFFu;
        const uint32_t i0 = (uint32_t)(1023 - (e + 2 * i));
        const uint32_t idx = i0 | ((i0 - 1) << 16);  // the indices of the two scores
        insert_key<KL, false>(top, (int)perm(u, idx, sel_lo), rej);
        insert_key<KL, false>(top, (int)perm(u, idx, sel_hi), rej);
      }
    }
  }
}

// resolve_ties for fp32 rows of up to 1,024 scores and 22-bit buckets: lane l
// takes the elements l + 64 j, marked with a 20-bit sub-key (low 10 value
// bits, then the complemented index).  Every lane must be active.
__device__ __attribute__((noinline)) void resolve_ties_wide(u64 tie_mask, int sk_v, int need_v, bool gen_keys,
                                                           u64* mybt, const unsigned char* row0, int E, int swz) {
  const int lane = (int)__lane_id();
  while (tie_mask != 0ull) {
    const int L = __builtin_ctzll(tie_mask);
    tie_mask &= tie_mask - 1;
    const int B = __builtin_amdgcn_readlane(sk_v, L) >> 10;
    const int need_l = __builtin_amdgcn_readlane(need_v, L);
    const uint32_t* row = reinterpret_cast<const uint32_t*>(row0 + (int64_t)L * E * 4);
    uint32_t x[kMaxE / kWave];
#pragma unroll
    for (int j = 0; j < kMaxE / kWave; ++j) x[j] = row[min(lane + kWave * j, E - 1)];
    int sub[kMaxE / kWave];
#pragma unroll
    for (int j = 0; j < kMaxE / kWave; ++j) {
      uint32_t u = x[j];
      if (gen_keys) u ^= (uint32_t)((int32_t)u >> 31) & 0x7FFFFFFFu;
      const int e = lane + kWave * j;
      sub[j] = (e < E && ((int32_t)u >> 10) == B) ? (int)(((u & 0x3FFu) << 10) | (uint32_t)(1023 - e)) : -1;
    }
    for (int r = 0; r < need_l; ++r) {
      int m = -1;
#pragma unroll
      for (int j = 0; j < kMaxE / kWave; ++j) m = max(m, sub[j]);
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) m = max(m, __shfl_xor(m, d));
      if (m < 0) break;
      if (lane == 0) atomicOr(&mybt[(1023 - (m & 1023)) ^ swz], 1ull << L);
#pragma unroll
      for (int j = 0; j < kMaxE / kWave; ++j) sub[j] = (sub[j] == m) ? -1 : sub[j];
    }
  }
}

template <typename T, int KL>
__global__ __launch_bounds__(kWideThreads) void k_topk_wide(const SegTable tab_arg, const PathArgs a) {
  (void)tab_arg;  // read in place, see load_seg
  const SegTablePtr tab = (SegTablePtr)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int E = a.E, k = a.k;
  const int EW = (E + 31) & ~31;  // words per tile row: the swizzle permutes groups of 32
  const int rowB = E * (int)sizeof(T);
  const int nch = (rowB + 127) >> 7;
  const int dup = (16 - (rowB & 15)) & 15;
  unsigned char* st = smem + wave * kChunkBytes;
  u64* bt = reinterpret_cast<u64*>(smem + kWideWaves * kChunkBytes);  // [kWideWaves][EW]
  u64* mybt = bt + wave * EW;
  const int swz = bt_swz(2 * wave);

  const uint32_t H = 2u * (uint32_t)tab->tile_start[tab->nseg];  // half units
  bool gen = Traits<T>::kExact;  // fp32: positive keys until a threshold is not positive
  uint32_t vmask = 0xFFFFFC00u, sel_lo = 0x05040100u, sel_hi = 0x07060302u;  // opaque: kept in VGPRs
  asm volatile("" : "+v"(vmask), "+v"(sel_lo), "+v"(sel_hi));

  auto row_bounds = [&](const Seg& sg, uint32_t wl, int& r_lo, int& r_hi) {
    r_lo = wl == 0 ? (int)sg.sh : 0;
    r_hi = (int)max((int64_t)0, min((int64_t)64, (int64_t)sg.sh + (int64_t)sg.n - ((int64_t)wl << 6)));
  };
  // chunk c_ of the 64 rows of a word: instruction j fills slots 64 j + lane
  v4u pre[8];
  auto fetch = [&](const Seg& sg, uint32_t wl, int c_) __attribute__((always_inline)) {
    const int nv = (min(128, rowB - 128 * c_) + 15) >> 4;
    const int row_in = lane >> 3;
    const int q0 = (lane & 7) ^ stage_swz(row_in, 3);
    const uint32_t p0 = (uint32_t)min(128 * c_ + 16 * min(q0, nv - 1), rowB - 16);
    const uint32_t p1 = (uint32_t)min(128 * c_ + 16 * min(q0 ^ 4, nv - 1), rowB - 16);
    const unsigned char* wbase = word_rows(sg, wl, rowB);
    int r_lo, r_hi;
    row_bounds(sg, wl, r_lo, r_hi);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // rows without a token re-read a valid one (never used)
      const int r = min(max(row_in + 8 * j, r_lo), r_hi - 1);
      pre[j] = __builtin_nontemporal_load(
          reinterpret_cast<const v4u_any*>(wbase + ((uint32_t)(r * rowB) + ((j & 1) ? p1 : p0))));
    }
  };

  int seg = 0;
  Seg sv{};
  // local word of slot 0 of half unit h (and its segment)
  auto locate = [&](uint32_t h, int& sg_i, Seg& sg) -> uint32_t {
    const uint32_t u = h >> 1;
    if (sg.words == 0u || u >= (uint32_t)tab->tile_start[sg_i + 1]) {
      sg_i = seg_of(tab, u, sg_i);
      sg = load_seg(tab, sg_i, rowB);
    }
    return 8 * (u - sg.u_begin) + 4 * (h & 1);
  };
  uint32_t h = blockIdx.x;
  uint32_t tl0 = 0;
  if (h < H) {
    tl0 = locate(h, seg, sv);
    if (tl0 + wave < sv.words) fetch(sv, tl0 + wave, 0);
  }
  for (; h < H; h += gridDim.x) {
    const uint32_t wl = tl0 + wave;
    const bool mine = wl < sv.words;
    const uint32_t hn = h + gridDim.x;
    int seg_n = seg;
    Seg svn = sv;
    const uint32_t tl0n = hn < H ? locate(hn, seg_n, svn) : 0u;
    const bool next_mine = hn < H && tl0n + wave < svn.words;
    for (int e = lane; e < EW; e += kWave) mybt[e] = 0;
    DOL_WAVE_FENCE();
    if (mine) {
      const uint32_t row = (wl << 6) + (uint32_t)lane;
      const bool valid = (wl >= sv.full_lo && wl < sv.full_hi) ||
                         (row >= sv.sh && (uint64_t)row < (uint64_t)sv.sh + (uint64_t)sv.n);
      int top[KL];
      int rej = INT_MIN;
#pragma unroll
      for (int i = 0; i < KL; ++i) top[i] = INT_MIN;
      int sk, sk1;
      // fp32: a row whose threshold is not positive is loaded and ranked once more
      // with general keys, which the wave then keeps (569 experts, 5 x 56 negative
      // tokens: 149 us with the exact per-lane selection after the first ranking,
      // 55 this way)
      for (;;) {
        for (int c = 0; c < nch; ++c) {
#pragma unroll
          for (int j = 0; j < 8; ++j) *reinterpret_cast<v4u*>(st + j * 1024 + lane * 16) = pre[j];
          DOL_WAVE_FENCE();
          if (c + 1 < nch)
            fetch(sv, wl, c + 1);
          else if (next_mine)
            fetch(svn, tl0n + wave, 0);
          const int nv = (min(128, rowB - 128 * c) + 15) >> 4;
          const int tail_q = dup != 0 && c + 1 == nch ? nv - 1 : -1;
          const int e0 = c * 8 * Traits<T>::kVec;
          if (gen)
            rank_wide<T, KL, true>(st, lane, e0, nv, tail_q, dup, E, vmask, sel_lo, sel_hi, top, rej);
          else
            rank_wide<T, KL, false>(st, lane, e0, nv, tail_q, dup, E, vmask, sel_lo, sel_hi, top, rej);
          DOL_WAVE_FENCE();
        }
        sk = top[0], sk1 = rej;
#pragma unroll
        for (int i = 0; i < KL; ++i) {
          sk = i == k - 1 ? top[i] : sk;
          sk1 = i == k ? top[i] : sk1;
        }
        if (Traits<T>::kExact || gen || __ballot(valid && sk < WideKey<T>::kPosMin) == 0ull) break;
        gen = true;
        rej = INT_MIN;
#pragma unroll
        for (int i = 0; i < KL; ++i) top[i] = INT_MIN;
        fetch(sv, wl, 0);
      }
      bool ok = top[0] < kCompPosInf;
      if (gen) ok = ok && sk > kCompNegInfMax && (sk < WideKey<T>::kZeroLo || sk > WideKey<T>::kZeroHi);
      const bool tie = !Traits<T>::kExact && valid && ok && ((sk1 >> 10) == (sk >> 10));
      // the k selected entries are top[0..k); a lane or a tied entry that
      // selects nothing ORs a zero (no divergent branches, as in k_topk)
      int need = 0;
      const u64 bit = valid && ok ? 1ull << lane : 0ull;
#pragma unroll
      for (int i = 0; i < KL; ++i) {
        if (i >= k) break;  // wave-uniform
        const bool tied = tie && (top[i] >> 10) == (sk >> 10);
        need += tied ? 1 : 0;
        atomicOr(&mybt[min(1023 - (top[i] & 1023), EW - 1) ^ swz], tied ? 0ull : bit);
      }
      if (!Traits<T>::kExact) {
        const u64 tm = __ballot(tie);
        if (tm != 0ull) resolve_ties_wide(tm, sk, need, gen, mybt, word_rows(sv, wl, rowB), E, swz);
      }
      const bool slow = valid && !ok;
      if (__ballot(slow) != 0ull) {
        const T* rp = reinterpret_cast<const T*>(word_rows(sv, wl, rowB) + (uint32_t)lane * (uint32_t)rowB);
        exact_select_lane<T>(slow, rp, E, k, mybt, swz, 1ull << lane);
      }
    } else if (next_mine) {
      fetch(svn, tl0n + wave, 0);  // idle at a segment's end, busy in the next step
    }
    __syncthreads();
    // The words of this half unit: 32 contiguous bytes per expert.  Words that
    // a stream append shares with a neighbouring micro-batch are OR-ed in;
    // without or_partial the words past the layer's last one are its padding
    // and are written as zeros (their tile rows are zero).
    u64* lb = a.bits + (int64_t)sv.layer * a.bits_layer_words;
    const uint32_t w0 = sv.w_first + tl0;
    const int cnt = (int)min((uint32_t)kWideWaves, sv.words > tl0 ? sv.words - tl0 : 0u);
    const bool shared_lo = a.or_partial && tl0 == 0 && sv.sh != 0;
    const int shared_hi =
        a.or_partial && tl0 + (uint32_t)kWideWaves >= sv.words && ((sv.sh + sv.n) & 63) != 0 ? cnt - 1 : -1;
    if ((w0 & 1) == 0 && !shared_lo && shared_hi < 0 && (cnt == kWideWaves || !a.or_partial)) {
      for (int i = tid; i < 2 * E; i += kWideThreads) {
        const int e = i >> 1, s = (i & 1) * 2;
        const v2u64 v = {bt[s * EW + (e ^ bt_swz(2 * s))], bt[(s + 1) * EW + (e ^ bt_swz(2 * s + 2))]};
        __builtin_nontemporal_store(v, reinterpret_cast<v2u64*>(lb + sig_off(w0 + s, e, E)));
      }
    } else {
      for (int i = tid; i < kWideWaves * E; i += kWideThreads) {
        const int e = i >> 2, s = i & 3;
        const u64 v = bt[s * EW + (e ^ bt_swz(2 * s))];
        if (s >= cnt) continue;
        u64* dst = lb + sig_off(w0 + s, e, E);
        if ((s == 0 && shared_lo) || s == shared_hi) {
          if (v) atomicOr(dst, v);
        } else {
          *dst = v;
        }
      }
    }
    __syncthreads();  // the tile is free
    seg = seg_n;
    sv = svn;
    tl0 = tl0n;
  }
}

template <typename T, int KL>
hipError_t launch_one_wide(const SegTable& tab, const PathArgs& a, hipStream_t s, const ProfEv& pe) {
  auto kern = k_topk_wide<T, KL>;
  const size_t lds = (size_t)kWideWaves * (kChunkBytes + ((a.E + 31) & ~31) * sizeof(u64));
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  int occ = 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, kWideThreads, lds) != hipSuccess || occ < 1) occ = 1;
  const int64_t half = 2 * tab.tile_start[tab.nseg];
  const int64_t blocks = std::min<int64_t>((int64_t)device_info().cu_count * occ, half);
  if (pe.start != nullptr || pe.stop != nullptr)
    hipExtLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kWideThreads), lds, s, pe.start, pe.stop, 0u, tab, a);
  else
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kWideThreads), lds, s, tab, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wide(do_dtype dt, const SegTable& tab, const PathArgs& a, hipStream_t s, const ProfEv& pe) {
  if (a.cacc != nullptr || a.bits == nullptr || a.k > kWideMaxK) return hipErrorInvalidValue;
  if (dt == DO_F32)
    return a.k <= 8 ? launch_one_wide<float, 8>(tab, a, s, pe) : launch_one_wide<float, 16>(tab, a, s, pe);
  return a.k <= 8 ? launch_one_wide<uint16_t, 8>(tab, a, s, pe) : launch_one_wide<uint16_t, 16>(tab, a, s, pe);
}

}  // namespace dol
