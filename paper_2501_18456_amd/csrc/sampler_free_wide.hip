// Heat-bath sweeps of the gather form by free-running waves (adabmDCA 2.0,
// Sec. 2.1), q > 16.
#include "gather_free.hpp"

namespace bmdca {

hipError_t launch_free_heat_wide(int q, const GatherShape& gs, const GatherArgs& a) {
  switch (q) {
#define BMDCA_GQ(n) \
  case n:           \
    return launch_free_shape<n, false>(gs, a);
    BMDCA_GQ(17) BMDCA_GQ(18) BMDCA_GQ(19) BMDCA_GQ(20) BMDCA_GQ(21) BMDCA_GQ(22) BMDCA_GQ(23)
    BMDCA_GQ(24) BMDCA_GQ(25) BMDCA_GQ(26) BMDCA_GQ(27) BMDCA_GQ(28) BMDCA_GQ(29) BMDCA_GQ(30)
    BMDCA_GQ(31) BMDCA_GQ(32)
#undef BMDCA_GQ
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace bmdca
