// Instances of the register-resident COCG kernel with p and x in registers (rres_kernel.h).
#include "rres_kernel.h"

namespace rpa {
namespace rres {

// Ten registers per point of the column (v, w, p, x) and about fifty more: 256 per thread hold 20
// points; from 12 points down 168 are enough and leave a third wave per SIMD.
KernelFn full_variant(int nz) {
#define RPA_N(N) \
    case N: return full_wg<N, N <= 12 ? 3 : 2>;
    switch (nz) {
        RPA_N(12) RPA_N(13) RPA_N(14) RPA_N(15) RPA_N(16) RPA_N(17) RPA_N(18) RPA_N(19) RPA_N(20)
        default: return nullptr;
    }
#undef RPA_N
}

}  // namespace rres
}  // namespace rpa
