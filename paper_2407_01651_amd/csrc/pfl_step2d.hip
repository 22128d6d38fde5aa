// Fused 2D step: FP64 instantiations (the parity form, built without
// floating-point contraction) and the dispatch by storage type; the FP32
// and 16-bit instantiations live in pfl_step2d_lowp.hip.
#include "pfl_step2d_f64.h"

namespace pfl {

hipError_t launch_step2d(const DevParams& P, int fields, int store, const void* fin, void* fout,
                         void* hist, double* mout, int mode, hipStream_t s, bool& ok) {
  if (store >= 1 && store <= 3) return launch_step2d_lowp(P, fields, store, fin, fout, hist, mout, mode, s, ok);
  ok = store == 0;
  if (!ok) return hipSuccess;
  // without the bubble phase the lattice of phi makes no difference
#define PFL_CASE(F)                                                                              \
  case F:                                                                                        \
    if (((F) & F_PHI) && P.q_phi == 9)                                                           \
      return launch_step2d_f64<F, ((F) & F_PHI) ? 9 : 5>(P, fin, fout, hist, mout, mode, s);     \
    return launch_step2d_f64<F, 5>(P, fin, fout, hist, mout, mode, s);
  switch (fields) {
    PFL_CASE(F_NS | F_PHI | F_PSI | F_C | F_TH)
    PFL_CASE(F_PSI | F_C)
    PFL_CASE(F_PSI | F_C | F_TH)
    PFL_CASE(F_NS | F_PHI)
    PFL_CASE(F_PHI | F_PSI | F_C | F_TH)
    PFL_CASE(F_PSI)
    PFL_CASE(F_PHI)
    PFL_CASE(F_NS | F_PSI | F_TH)
    PFL_CASE(F_NS | F_PSI | F_C | F_TH)
    PFL_CASE(F_PSI | F_TH)
    default:
      ok = false;
      return hipSuccess;
  }
#undef PFL_CASE
}

bool step2d_supported(int fields) {
  switch (fields) {
    case F_NS | F_PHI | F_PSI | F_C | F_TH:
    case F_PSI | F_C:
    case F_PSI | F_C | F_TH:
    case F_NS | F_PHI:
    case F_PHI | F_PSI | F_C | F_TH:
    case F_PSI:
    case F_PHI:
    case F_NS | F_PSI | F_TH:
    case F_NS | F_PSI | F_C | F_TH:
    case F_PSI | F_TH:
      return true;
    default:
      return false;
  }
}

}  // namespace pfl
