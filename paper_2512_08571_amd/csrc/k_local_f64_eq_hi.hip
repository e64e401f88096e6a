// Local-operator launcher instantiations for f64 (see k_local_impl.h), n_q = n_p >= 7.
#include "k_local_planes.h"

namespace fehx {

fe_status local_f64_eq_hi(const LocalBatch &B, hipStream_t s) {
  switch (B.ms[0]->np) {
    case 7: return pick_planes_f64<7, 7>(B, s);
    case 8: return pick_planes_f64<8, 8>(B, s);
    case 9: return pick_planes_f64<9, 9>(B, s);
    default: return set_error(FE_EUNSUPPORTED, "FE degree outside 2..8");
  }
}

}  // namespace fehx
