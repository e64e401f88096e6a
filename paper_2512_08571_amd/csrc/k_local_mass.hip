// The consistent mass operator of affine cells on the plane kernels
// (k_local_planes.h), all precisions.  Bound by the gather and scatter of each
// colour phase; 11 x 13 x 12 cells degree 6 x 101 FP64 vectors: 953 us as the
// staged operator with zero derivative tables, 380 here (nine phases).
#include "k_local_planes.h"

namespace fehx {

namespace {
template <int NP> fe_status run_mass(const LocalBatch &B, hipStream_t s) {
  const LocalLaunch &L = B.Ls[0];
  if (L.prec == FE_F64) return run_planes<NP, NP, false, double, double, 1, true>(B, s);
  const bool f32 = L.prec == FE_F32 || L.store32;
  const bool pairs = B.kind == LOCAL_MASS_PAIRS && plane_pairs_pay(B, NP);
  if (f32) return pairs ? run_planes<NP, NP, false, float, float, 2, true>(B, s) : run_planes<NP, NP, false, float, float, 1, true>(B, s);
  return pairs ? run_planes<NP, NP, false, bf16s, float, 2, true>(B, s) : run_planes<NP, NP, false, bf16s, float, 1, true>(B, s);
}
}  // namespace

fe_status launch_local_mass(const LocalBatch &B, hipStream_t s) {
  switch (B.ms[0]->np) {
    case 3: return run_mass<3>(B, s);
    case 4: return run_mass<4>(B, s);
    case 5: return run_mass<5>(B, s);
    case 6: return run_mass<6>(B, s);
    case 7: return run_mass<7>(B, s);
    case 8: return run_mass<8>(B, s);
    case 9: return run_mass<9>(B, s);
    default: return set_error(FE_EUNSUPPORTED, "FE degree outside 2..8");
  }
}

}  // namespace fehx
