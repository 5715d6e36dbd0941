// Instances of the register-resident COCG kernel with p and x in registers (rres_kernel.h).
#include "rres_kernel.h"

namespace rpa {
namespace rres {

// Ten registers per point of the column (v, w, p, x) and about fifty more.  256 per thread hold 18
// points; 19 and 20 spill 6 and 18 vector registers to scratch.  At 12 points 168 registers leave a
// third wave per SIMD and spill 26.  Every instance parks 85 to 113 scalars in vector lanes.  Even so
// the class edges win: kernel times against the streaming kernel, 1024 and 8 systems: 12^3 0.73 and
// 0.32 ms against 1.61 and 0.80, 20 x 25 x 20 3.1 and 0.84 against 7.2 and 1.86.
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
