// Instances of the register-resident COCG kernel with p and x in memory (rres_kernel.h).
#include "rres_kernel.h"

namespace rpa {
namespace rres {

// Four registers per point of the column (v, w) and about fifty more for the sweep; the fold's two
// chunks want about as many, whatever the column.  With 12 waves (168 registers) every height from 12
// to 26 spills 36 to 68 vector registers to scratch (halves of eight), with 8 waves (256) only 31 and
// 32 points do, 2 to 10; 122 to 198 scalars are parked in vector lanes.
KernelFn ring_variant(int nz, bool xc, int half) {
    // short halves only for complex solutions of the columns whose real ones full_wg takes
    if (half == kRingHalfMin && (!xc || nz > 20)) return nullptr;
#define RPA_S(N)                                                               \
    case N: return half == kRingHalfMin ? ring_wg<N, 768, 3, kRingHalfMin, true> \
                 : xc ? ring_wg<N, 768, 3, kRing, true> : ring_wg<N, 768, 3, kRing, false>;
#define RPA_A(N) \
    case N: return xc ? ring_wg<N, 768, 3, kRing, true> : ring_wg<N, 768, 3, kRing, false>;
#define RPA_B(N) \
    case N: return xc ? ring_wg<N, 512, 2, kRing, true> : ring_wg<N, 512, 2, kRing, false>;
    switch (nz) {
        RPA_S(12) RPA_S(13) RPA_S(14) RPA_S(15) RPA_S(16) RPA_S(17) RPA_S(18) RPA_S(19) RPA_S(20)
        RPA_A(21) RPA_A(22) RPA_A(23) RPA_A(24) RPA_A(25) RPA_A(26)
        RPA_B(27) RPA_B(28) RPA_B(29) RPA_B(30) RPA_B(31) RPA_B(32)
        default: return nullptr;
    }
#undef RPA_S
#undef RPA_A
#undef RPA_B
}

}  // namespace rres
}  // namespace rpa
