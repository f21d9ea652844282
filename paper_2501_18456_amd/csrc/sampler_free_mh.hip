// Single-site Metropolis of the gather form by free-running waves
// (adabmDCA 2.0, Sec. 2.1, the Metropolis option of the sampler).
#include "gather_free.hpp"

namespace bmdca {

hipError_t launch_free_metropolis(int q, const GatherShape& gs, const GatherArgs& a) {
  switch (q) {
#define BMDCA_GQ(n) \
  case n:           \
    return launch_free_shape<n, true>(gs, a);
    BMDCA_GQ(2) BMDCA_GQ(3) BMDCA_GQ(4) BMDCA_GQ(5) BMDCA_GQ(6) BMDCA_GQ(7) BMDCA_GQ(8)
    BMDCA_GQ(9) BMDCA_GQ(10) BMDCA_GQ(11) BMDCA_GQ(12) BMDCA_GQ(13) BMDCA_GQ(14) BMDCA_GQ(15)
    BMDCA_GQ(16) BMDCA_GQ(17) BMDCA_GQ(18) BMDCA_GQ(19) BMDCA_GQ(20) BMDCA_GQ(21) BMDCA_GQ(22)
    BMDCA_GQ(23) BMDCA_GQ(24) BMDCA_GQ(25) BMDCA_GQ(26) BMDCA_GQ(27) BMDCA_GQ(28) BMDCA_GQ(29)
    BMDCA_GQ(30) BMDCA_GQ(31) BMDCA_GQ(32)
#undef BMDCA_GQ
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace bmdca
