// The register passes' kernels and their launches (passes.h).  The build
// compiles this file once per part (QEC_PART 0: plain passes, 1: speculative
// passes, 2: passes with a basis change) and precision (QEC_T), side by side;
// without these macros everything is compiled at once.
#include "passes.h"
#include "kernels_flip.hip"

namespace qec {

#if !defined(QEC_PART) || QEC_PART == 0
// One pass kernel launch; the instantiation with the dense Kraus code exists
// only for unit pairs with an X check, the one summing a Z chain amplitude by
// amplitude (bmode 0) only for a Z chain B.
template <typename T, int AK, int AP, int BK, int BP>
void launch_pass(bool dense, bool bm0, dim3 g, dim3 b, hipStream_t s, T* st, const UnitPass* pd,
                 const JobConst* jc, const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db,
                 double* part, int rev, SlotStrides ss, const BlockDense* dna, const BlockDense* dnb) {
#define QEC_K(DNV, BMV)                                                                                  \
  hipLaunchKernelGGL((k_upass<T, AK, AP, BK, BP, DNV, BMV, 0>), g, b, 0, s, st, pd, jc, rta, rtb, da, db, part, \
                     rev, ss, dna, dnb, SpecArgs{})
  if constexpr (BK == U_Z) {
    if (bm0) {
      if constexpr (AK == U_X) {
        if (dense) {
          QEC_K(true, true);
          return;
        }
      }
      QEC_K(false, true);
      return;
    }
  }
  if constexpr ((AK == U_X || BK == U_X) && AK != U_XP && BK != U_XP) {  // pairs are never dense
    if (dense) {
      QEC_K(true, false);
      return;
    }
  }
  QEC_K(false, false);
#undef QEC_K
}

// Launches the pass kernel instantiated for the descriptor's unit kinds.
template <typename T>
int launch_upass(const UnitPass& h, dim3 g, dim3 b, hipStream_t s, T* st, const UnitPass* pd,
                 const JobConst* jc, const BlockRT* rta, const BlockRT* rtb,
                 const Decision* da, Decision* db, double* part, int rev,
                 SlotStrides ss, const BlockDense* dna,
                 const BlockDense* dnb) {
#define QEC_UP(AK, AP, BK, BP)                                                                      \
  if (h.akind == AK && ap == AP && h.bkind == BK && bp == BP) {                                     \
    launch_pass<T, AK, AP, BK, BP>(h.adense || h.bdense, h.bkind == U_Z && h.bmode == 0, g, b, s, st, pd, jc, \
                                   rta, rtb, da, db, part, \
                                   rev, ss, dna, dnb);                                              \
    return 0;                                                                                   \
  }
#define QEC_UP_B(AK, AP) \
  QEC_UP(AK, AP, U_X, 2) QEC_UP(AK, AP, U_X, 4) QEC_UP(AK, AP, U_Z, 1) QEC_UP(AK, AP, U_Z, 2) \
  QEC_UP(AK, AP, U_Z, 3) QEC_UP(AK, AP, U_Z, 4) QEC_UP(AK, AP, U_Z, 5) QEC_UP(AK, AP, U_Z, 6)
  if ((h.adense && !dna) || (h.bdense && !dnb)) return kLaunchNoTable;
  if (h.tb <= 0) return kLaunchNoFit;
  const int ap = h.akind == U_X ? h.wa : (h.akind == U_Z ? h.la : 0);
  const int bp = h.bkind == U_X ? h.wb : (h.bkind == U_Z ? h.lb : 0);
  QEC_UP_B(U_INIT, 0)
  QEC_UP_B(U_X, 2) QEC_UP_B(U_X, 4) QEC_UP(U_X, 2, U_NONE, 0) QEC_UP(U_X, 4, U_NONE, 0)
  QEC_UP_B(U_Z, 1) QEC_UP_B(U_Z, 2) QEC_UP_B(U_Z, 3) QEC_UP_B(U_Z, 4) QEC_UP_B(U_Z, 5) QEC_UP_B(U_Z, 6)
  QEC_UP(U_Z, 1, U_NONE, 0) QEC_UP(U_Z, 2, U_NONE, 0) QEC_UP(U_Z, 3, U_NONE, 0) QEC_UP(U_Z, 4, U_NONE, 0)
  QEC_UP(U_Z, 5, U_NONE, 0) QEC_UP(U_Z, 6, U_NONE, 0)
  // X pairs (weights handled at run time)
  QEC_UP(U_INIT, 0, U_XP, 0) QEC_UP(U_X, 2, U_XP, 0) QEC_UP(U_X, 4, U_XP, 0)
  QEC_UP(U_Z, 1, U_XP, 0) QEC_UP(U_Z, 2, U_XP, 0) QEC_UP(U_Z, 3, U_XP, 0) QEC_UP(U_Z, 4, U_XP, 0)
  QEC_UP(U_Z, 5, U_XP, 0) QEC_UP(U_Z, 6, U_XP, 0)
  QEC_UP_B(U_XP, 0) QEC_UP(U_XP, 0, U_XP, 0) QEC_UP(U_XP, 0, U_NONE, 0)
  QEC_UP(U_INIT, 0, U_NONE, 0)  // logical |0> alone (speculative runs)
#undef QEC_UP_B
#undef QEC_UP
  return kLaunchNoKernel;
}
#endif

#if !defined(QEC_PART) || QEC_PART == 1
// A speculative unit's prediction pass (redo = false) or redo: reads st,
// writes sa.out; the unit is A (an X check or pair, B none) or B (a Z chain,
// A the pending renormalisation).
template <typename T>
int launch_spass(const UnitPass& h, bool redo, dim3 g, dim3 b, hipStream_t s, T* st, const UnitPass* pd,
                 const JobConst* jc, const BlockRT* rta, const BlockRT* rtb, const Decision* da,
                 Decision* db, double* part, int rev, SpecArgs sa, SlotStrides ss) {
#define QEC_SP(AK, AP, BK, BP)                                                                              \
  if (h.akind == AK && ap == AP && h.bkind == BK && bp == BP) {                                             \
    if (redo)                                                                                               \
      hipLaunchKernelGGL((k_uredo<T, AK, AP, BK, BP>), g, b, 0, s, st, pd, jc, rta, rtb, da, db, part, rev, \
                         ss, nullptr, nullptr, sa);                                                         \
    else                                                                                                    \
      hipLaunchKernelGGL((k_upass<T, AK, AP, BK, BP, false, false, 1>), g, b, 0, s, st, pd, jc, rta, rtb,   \
                         da, db, part, rev, ss, nullptr, nullptr, sa);                                      \
    return 0;                                                                                           \
  }
  if (h.tb <= 0) return kLaunchNoFit;
  if (h.adense || h.bdense || (h.bkind == U_Z && h.bmode == 0))
    return kLaunchNoKernel;
  const int ap = h.akind == U_X ? h.wa : 0;
  const int bp = h.bkind == U_Z ? h.lb : 0;
  QEC_SP(U_X, 2, U_NONE, 0) QEC_SP(U_X, 4, U_NONE, 0) QEC_SP(U_XP, 0, U_NONE, 0)
  QEC_SP(U_SC, 0, U_Z, 1) QEC_SP(U_SC, 0, U_Z, 2) QEC_SP(U_SC, 0, U_Z, 3) QEC_SP(U_SC, 0, U_Z, 4)
  QEC_SP(U_SC, 0, U_Z, 5) QEC_SP(U_SC, 0, U_Z, 6)
#undef QEC_SP
  return kLaunchNoKernel;
}
#endif

#if !defined(QEC_PART) || QEC_PART == 2
template <typename T>
int launch_flip(const FlipPass& h, int mode, bool keep, dim3 g, hipStream_t s, T* st, const FlipPass* pd,
                 const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db, double* part, int rev,
                 int n_cls_wg, bool per_tile, double* chunk_sums, SlotStrides ss) {
#define QEC_FL(LBV, MODEV, L5V)                                                                                   \
  if (h.lb == LBV && mode == MODEV && (h.lane5 != 0) == L5V) {                                                    \
    hipLaunchKernelGGL((k_flip<T, LBV, MODEV, L5V>), g, dim3(256), 0, s, st, pd, rta, rtb, da, db, part, rev, \
                       n_cls_wg, per_tile ? 1 : 0, chunk_sums, keep ? 1 : 0, ss);                                 \
    return 0;                                                                                                     \
  }
#define QEC_FL_B(LBV)                                                                                        \
  QEC_FL(LBV, kFlipPass, false) QEC_FL(LBV, kFlipPass, true) QEC_FL(LBV, kFlipSums, false)                   \
  QEC_FL(LBV, kFlipFirst, false) QEC_FL(LBV, kFlipFirst, true)
  QEC_FL(0, kFlipPass, false) QEC_FL_B(1) QEC_FL_B(2) QEC_FL_B(3) QEC_FL_B(4) QEC_FL_B(5) QEC_FL_B(6)
#undef QEC_FL_B
#undef QEC_FL
  return kLaunchNoKernel;
}
#endif

#if !defined(QEC_PART) || QEC_PART == 0
#define QEC_INSTANCE_0(QEC_TT) \
  template int launch_upass<QEC_TT>(const UnitPass& h, dim3 g, dim3 b, hipStream_t s, QEC_TT* st, const UnitPass* pd, const JobConst* jc, const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db, double* part, int rev, SlotStrides ss, const BlockDense* dna, const BlockDense* dnb);
#else
#define QEC_INSTANCE_0(QEC_TT)
#endif
#if !defined(QEC_PART) || QEC_PART == 1
#define QEC_INSTANCE_1(QEC_TT) \
  template int launch_spass<QEC_TT>(const UnitPass& h, bool redo, dim3 g, dim3 b, hipStream_t s, QEC_TT* st, const UnitPass* pd, const JobConst* jc, const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db, double* part, int rev, SpecArgs sa, SlotStrides ss);
#else
#define QEC_INSTANCE_1(QEC_TT)
#endif
#if !defined(QEC_PART) || QEC_PART == 2
#define QEC_INSTANCE_2(QEC_TT) \
  template int launch_flip<QEC_TT>(const FlipPass& h, int mode, bool keep, dim3 g, hipStream_t s, QEC_TT* st, const FlipPass* pd, const BlockRT* rta, const BlockRT* rtb, const Decision* da, Decision* db, double* part, int rev, int n_cls_wg, bool per_tile, double* chunk_sums, SlotStrides ss);
#else
#define QEC_INSTANCE_2(QEC_TT)
#endif
#define QEC_INSTANCES(QEC_TT) QEC_INSTANCE_0(QEC_TT) QEC_INSTANCE_1(QEC_TT) QEC_INSTANCE_2(QEC_TT)
#ifdef QEC_T
QEC_INSTANCES(QEC_T)
#else
QEC_INSTANCES(float)
QEC_INSTANCES(double)
#endif

}  // namespace qec
