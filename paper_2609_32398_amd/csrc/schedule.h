// Unit schedule of the Top-K kernel: which 512-token units each block of the
// persistent grid walks, in which order.  Plain C++ (constexpr functions run
// on the host and the device alike), so that the launch and the kernel cannot
// disagree about it.
//
// The units [0, U) are cut into 2^lp partitions of consecutive units, one for
// the blocks b with b mod 2^lp equal to its number, and a partition into
// groups of gu consecutive units, which its Gs blocks take in turn: groups
// pos, pos + Gs, pos + 2 Gs, ...  One contiguous range per block is the case
// of one group per block.
//   lp = 0: one partition.
//   lp = 3: one per XCD (blocks are dispatched round-robin, so block b runs on
//      XCD b mod 8): the XCD's blocks work on adjacent groups, so their
//      signature stores land side by side while each block stays in few layers
//      (few Gram flushes, and those of different XCDs go to different layers).
//   lp = 4, 5: two or four partitions per XCD: fewer layers per block still.
#pragma once

#include <cstdint>

namespace dol {

struct Sched {
  int64_t gu;  // units per group, 0: one contiguous range per block
  int lp;      // log2 of the partitions
};

// The schedule of a launch of `blocks` blocks (at most `units` of them) nearest
// to `want`: at most its partitions, so many that the grid is a multiple of
// them (every partition then has the same number of blocks), and groups no
// longer than a block's even share of its partition.  A grid of one block per
// unit gives every block one unit.  (Groups sized for partitions that the kernel
// then dropped left half of such a grid without work: 40 layers x 2,560 bf16
// tokens with 128 experts 40.4 us, 30.3 this way; 17 x 512 38.3, 26.2; one layer
// of 100,352 31.3, 30.4.)
constexpr Sched plan_units(int64_t units, int64_t blocks, Sched want) {
  int lp = want.lp;
  while (blocks % (int64_t(1) << lp) != 0) --lp;
  const int64_t parts = int64_t(1) << lp;
  const int64_t per_part = (units + parts - 1) / parts, gs = blocks / parts;
  int64_t gu = want.gu;
  if (gu <= 0 || gu * gs > per_part) gu = (per_part + gs - 1) / gs;  // contiguous ranges
  return Sched{gu, lp};
}

// The units of one block, in order: from first() on, next(u) after each, until
// the result is U.  All unit counts are below 2^29 (64 segments of fewer than
// 2^32 tokens).
struct UnitWalk {
  uint32_t U, hi, gu, step, g_start, g_end;

  constexpr UnitWalk(uint32_t units, uint32_t blocks, uint32_t block, int lp, uint32_t group)
      : U(units), hi(0), gu(group), step(0), g_start(0), g_end(0) {
    const uint32_t part = block & ((1u << lp) - 1);
    const uint32_t lo = (uint32_t)(((uint64_t)part * units) >> lp);
    hi = (uint32_t)(((uint64_t)(part + 1) * units) >> lp);
    step = (blocks >> lp) * group;
    g_start = lo + (block >> lp) * group;
    g_end = g_start + group < hi ? g_start + group : hi;
  }
  constexpr uint32_t first() const { return g_start < hi ? g_start : U; }
  constexpr uint32_t next(uint32_t u) {
    if (u + 1 < g_end) return u + 1;
    g_start += step;
    if (g_start >= hi) return U;
    g_end = g_start + gu < hi ? g_start + gu : hi;
    return g_start;
  }
};

}  // namespace dol
