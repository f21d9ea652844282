// Heat-bath sweeps of the gather form by free-running waves (adabmDCA 2.0,
// Sec. 2.1), q <= 16.  The instantiations stand in three files so that they
// compile in parallel.
#include "gather_free.hpp"

namespace bmdca {

hipError_t launch_free_heat(int q, const GatherShape& gs, const GatherArgs& a) {
  switch (q) {
#define BMDCA_GQ(n) \
  case n:           \
    return launch_free_shape<n, false>(gs, a);
    BMDCA_GQ(2) BMDCA_GQ(3) BMDCA_GQ(4) BMDCA_GQ(5) BMDCA_GQ(6) BMDCA_GQ(7) BMDCA_GQ(8)
    BMDCA_GQ(9) BMDCA_GQ(10) BMDCA_GQ(11) BMDCA_GQ(12) BMDCA_GQ(13) BMDCA_GQ(14) BMDCA_GQ(15)
    BMDCA_GQ(16)
#undef BMDCA_GQ
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace bmdca
