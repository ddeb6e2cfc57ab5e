// The Top-K kernel (topk_kernel.h) for the kRagged rows: any row length and
// alignment, and the shapes that only the exact per-lane selection takes (the
// kTiny rows among them).
#include "topk_kernel.h"

namespace dol {
namespace {

template <typename T>
hipError_t launch_ep(int gm, const SegTable& tab, const PathArgs& a, bool fast, Sched sc, hipStream_t s,
                     const ProfEv& pe) {
  if (a.E * (int)sizeof(T) < 16) return launch_mode<T, 32, kTiny>(gm, tab, a, false, sc, s, pe);
  if (a.E <= 32) return launch_mode<T, 32, kRagged>(gm, tab, a, fast, sc, s, pe);
  if (a.E <= 64) return launch_mode<T, 64, kRagged>(gm, tab, a, fast, sc, s, pe);
  if (a.E <= 128) return launch_mode<T, 128, kRagged>(gm, tab, a, fast, sc, s, pe);
  if (a.E <= 256) return launch_mode<T, 256, kRagged>(gm, tab, a, fast, sc, s, pe);
  // E in (256, 1024]: exact per-lane selection, signatures only
  if (a.cacc != nullptr) return hipErrorInvalidValue;
  if (a.E <= 512) return launch_one<T, 512, kGramNone, kRagged>(tab, a, false, sc, s, pe);
  return launch_one<T, 1024, kGramNone, kRagged>(tab, a, false, sc, s, pe);
}

}  // namespace

hipError_t launch_ragged(do_dtype dt, int gm, const SegTable& tab, const PathArgs& a, bool fast, Sched sc,
                         hipStream_t s, const ProfEv& pe) {
  return dt == DO_F32 ? launch_ep<float>(gm, tab, a, fast, sc, s, pe)
                      : launch_ep<uint16_t>(gm, tab, a, fast, sc, s, pe);
}

}  // namespace dol
