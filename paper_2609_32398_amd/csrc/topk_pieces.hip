// The Top-K kernel (topk_kernel.h) for the kPieces rows: 16-byte aligned rows of
// whole 16-byte pieces.
#include "topk_kernel.h"

namespace dol {
namespace {

template <typename T>
hipError_t launch_ep(int gm, const SegTable& tab, const PathArgs& a, Sched sc, hipStream_t s, const ProfEv& pe) {
  if (a.E <= 32) return launch_mode<T, 32, kPieces>(gm, tab, a, true, sc, s, pe);
  if (a.E <= 64) return launch_mode<T, 64, kPieces>(gm, tab, a, true, sc, s, pe);
  if (a.E <= 128) return launch_mode<T, 128, kPieces>(gm, tab, a, true, sc, s, pe);
  return launch_mode<T, 256, kPieces>(gm, tab, a, true, sc, s, pe);
}

}  // namespace

hipError_t launch_pieces(do_dtype dt, int gm, const SegTable& tab, const PathArgs& a, Sched sc, hipStream_t s,
                         const ProfEv& pe) {
  return dt == DO_F32 ? launch_ep<float>(gm, tab, a, sc, s, pe) : launch_ep<uint16_t>(gm, tab, a, sc, s, pe);
}

}  // namespace dol
