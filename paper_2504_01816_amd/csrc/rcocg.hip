// Launch-shape selection for the real-form COCG kernels (design in rcocg_kernel.h and
// rres_kernel.h).
//
// Grids whose columns and plane fit the registers of one workgroup take a resident kernel
// (choose_resident).  Elsewhere the vectors stream, and a shape is (C rows per thread, Z planes per
// barrier step).  One row per thread up to 1024 columns: more rows share LDS reads, but the kernel
// waits on memory and wants waves (24^3, ring of 8: 26.5 ms with C = 1, 34 with 2, 47 with 3).  Two
// planes per step where n2 is even (26.5 against 28.8 ms).  Planes over 1024 points take the fewest
// rows that fit their threads (40^3: 37.2 ms with C = 2, 40.3 with 3), with one plane per step (two
// spill: 77 ms; with one, three rows in 768 threads spill 33 registers outside the plane loop).
// So a plane has a shape if n0 n1 <= 1024, n0 ceil(n1 / 2) <= 1024 or n0 ceil(n1 / 3) <= 768 (all of
// these fit LDS); others stay on the complex kernel: every plane over 2304 points, but also 36 x 64,
// 46 x 49 and 257 x 7.
// RPA_RCOCG_SHAPE="C,Z" forces a streaming shape; RPA_COCG_VERBOSE=1 prints the one launched.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "rres_kernel.h"

namespace rpa {

namespace {

using KernelFn = void (*)(rcocg::Args);
using CheckFn = void (*)(rcocg::CheckArgs);

struct Variant {
    int C, Z, bsmax;
    bool ragged;           // C does not divide n1
    KernelFn real, cplx;
    CheckFn check;
};

#define RPA_V(CC, ZZ, BM, RG)                                        \
    {CC, ZZ, BM, RG, rcocg::rcocg_wg<double, CC, ZZ, BM, RG>,        \
     rcocg::rcocg_wg<double2, CC, ZZ, BM, RG>, rcocg::check_wg<CC, BM, RG>}
const Variant kTable[] = {
    RPA_V(1, 1, 256, false), RPA_V(1, 1, 512, false),  RPA_V(1, 1, 768, false), RPA_V(1, 1, 1024, false),
    RPA_V(1, 2, 256, false), RPA_V(1, 2, 512, false),  RPA_V(1, 2, 768, false), RPA_V(1, 2, 1024, false),
    RPA_V(2, 1, 768, false), RPA_V(2, 1, 1024, false), RPA_V(3, 1, 768, false),
    RPA_V(2, 1, 768, true),  RPA_V(2, 1, 1024, true),  RPA_V(3, 1, 768, true)};
#undef RPA_V

struct Shape {
    const Variant* v = nullptr;
    int bs = 0, nbuf = 2, rs = 0;
    size_t lds = 0;
};

void stencil_weights(double h, double cw[7]) {
    double w[7];
    fd_weights(w);
    const double ih2 = 1.0 / (h * h);
    cw[0] = -0.5 * 3.0 * w[0] * ih2;
    for (int k = 1; k <= 6; ++k) cw[k] = -0.5 * w[k] * ih2;
}

constexpr size_t kLds = 160 * 1024;

size_t lds_bytes(const Grid& g, int C, int Z, int nbuf, int rs) {
    return 16 * 3 * sizeof(double) + rcocg::kRingLong * sizeof(rcocg::Coef) + 16 +
           size_t(nbuf) * Z * (g.n1 + 11 + C) * rs * sizeof(double);
}

Shape choose(const Grid& g) {
    int fC = 0, fZ = 0;
    if (const char* e = std::getenv("RPA_RCOCG_SHAPE"))
        if (std::sscanf(e, "%d,%d", &fC, &fZ) < 2) fC = fZ = 0;
    Shape best;
    double best_cost = 1e30;
    for (const Variant& v : kTable) {
        if (g.n2 % v.Z != 0 || (g.n1 % v.C != 0) != v.ragged) continue;
        if (fC && (v.C != fC || v.Z != fZ)) continue;
        const int cols = g.n0 * ((g.n1 + v.C - 1) / v.C);
        const int bs = (cols + 63) / 64 * 64;
        if (bs > v.bsmax || bs <= v.bsmax - (v.C == 3 ? 512 : 256)) continue;
        Shape s;
        s.v = &v;
        s.bs = bs;
        s.rs = (g.n0 + 12 + 7) / 8 * 8;
        const size_t delay = v.C > 1 ? size_t(rcocg::kDelay) * v.C * bs * sizeof(double) : 0;
        s.lds = lds_bytes(g, v.C, v.Z, 2, s.rs) + delay;
        if (s.lds > kLds) {
            s.nbuf = 1;
            s.lds = lds_bytes(g, v.C, v.Z, 1, s.rs) + delay;
        }
        if (s.lds > kLds) continue;
        const double cost = double(bs - cols) / bs + 0.1 * (2 - v.Z) + 0.05 * v.C;
        if (cost < best_cost) {
            best_cost = cost;
            best = s;
        }
    }
    return best;
}

// Workgroups per CU the pool is sized for.
int per_cu(int bs) { return bs > 512 ? 1 : bs > 320 ? 2 : bs > 192 ? 3 : 4; }

constexpr int kCUs = 256;

// The register-resident kernels where a column and the plane fit (see their instances): real
// solutions with p and x in registers, else with p and x in memory and up to four waves that fold.
// They are taken up to the last shape that fits, where one wave is left to fold and registers spill:
// streaming is slower there too.  Kernel ms for 1024 and 8 systems, resident, streaming (and the complex
// kernel): 26 x 27 x 26 10.9 and 2.19, 12.4 and 2.85 (34.1, 7.4); 26 x 27 x 14 4.6 and 1.10, 6.8 and
// 1.59; 25 x 28 x 24 8.5 and 1.82, 11.4 and 2.69; 22 x 27 x 25 7.8 and 1.54, 11.3 and 2.91;
// 20 x 22 x 32 6.3 and 1.47, 11.2 and 2.72; 21 x 21 x 32 6.4 and 1.47, 11.3 and 2.70.
struct Resident {
    KernelFn fn = nullptr;
    bool full = false;
    int bs = 0, per_cu = 1, half = 0;      // half: vectors of a ring half
    size_t lds = 0;
};

// vecs: vectors of pool per workgroup.
Resident choose_resident(const Grid& g, bool x_complex, int vecs) {
    Resident r;
    const char* e = std::getenv("RPA_RCOCG_SHAPE");
    if (e) return r;                                   // a streaming shape is forced
    r.lds = rres::lds_fixed() +
            size_t(2) * rres::kPairs * (g.n1 + 12) * (g.n0 + 16) * sizeof(double2);
    if (r.lds > 156 * 1024) return r;
    const int waves = (g.n0 * g.n1 + 63) / 64;
    if (!x_complex && waves <= 8) r.fn = rres::full_variant(g.n2);
    if (r.fn) {
        r.full = true;
        r.bs = 64 * waves;
        // workgroups of a CU: LDS, and 8 waves (12 with columns of 12 points)
        r.per_cu = std::max(1, std::min(int(160 * 1024 / r.lds), (g.n2 <= 12 ? 12 : 8) / waves));
        return r;
    }
    const int most = g.n2 <= 26 ? 12 : 8;
    for (int half : {rcocg::kRing, rres::kRingHalfMin})
        if (!r.fn && waves < most && vecs >= 2 * half + rcocg::kSlotExtra) {
            r.fn = rres::ring_variant(g.n2, x_complex, half);
            r.half = half;
        }
    r.bs = 64 * std::min(most, waves + 4);
    return r;
}

}  // namespace

bool rcocg_fits(const Grid& g) { return choose(g).v != nullptr; }

size_t rcocg_pool_bytes(const Grid& g, int nsys) {
    const Shape s = choose(g);
    if (!s.v) return 0;
    const size_t vec = size_t(g.nd()) * sizeof(double);
    // real and complex solutions may take different kernels
    const int all = 2 * rcocg::kRing + rcocg::kSlotExtra;
    const Resident re = choose_resident(g, false, all), cx = choose_resident(g, true, all);
    size_t need = 0;
    if (!re.fn || !cx.fn)
        // a ring of kRing; kRingLong is for launches that fill the chip, and these have the room
        need = size_t(std::min(nsys, kCUs * per_cu(s.bs))) * (rcocg::kRing + rcocg::kSlotExtra);
    if (cx.fn) need = std::max(need, size_t(std::min(nsys, kCUs)) * all);
    // where real solutions need no pool, complex ones make do with 48 B per point and system
    if (re.full) need = std::min(need, size_t(nsys) * 6);
    return need * vec;
}

namespace {

// A launch on nsys systems with a pool of pool_bytes.  kind: 0 no shape, 1 streaming, 2 resident with
// a ring, 3 resident with p and x in registers.
struct Plan {
    Shape s;
    KernelFn fn = nullptr;
    int kind = 0, bs = 0, grid = 0, ring = 0;
    size_t lds = 0;
};

Plan make_plan(const Grid& g, int nsys, bool x_complex, size_t pool_bytes) {
    Plan p;
    p.s = choose(g);
    if (!p.s.v) return p;
    const size_t vec = size_t(g.nd()) * sizeof(double);
    const Resident res =
        choose_resident(g, x_complex, int(pool_bytes / (size_t(std::min(nsys, kCUs)) * vec)));
    p.fn = res.fn ? res.fn : x_complex ? p.s.v->cplx : p.s.v->real;
    p.kind = res.full ? 3 : res.fn ? 2 : 1;
    p.grid = std::min(nsys, kCUs * (res.fn ? res.per_cu : per_cu(p.s.bs)));
    p.lds = res.fn ? res.lds : p.s.lds;
    p.bs = res.fn ? res.bs : p.s.bs;
    p.ring = res.fn ? 2 * res.half
                    : std::min(rcocg::kRingLong,
                               int(pool_bytes / (size_t(p.grid) * vec)) - rcocg::kSlotExtra);
    return p;
}

}  // namespace

hipError_t launch_rcocg(const RcocgLaunch& L, hipStream_t st) {
    if (L.nsys <= 0) return hipSuccess;
    const Plan p = make_plan(L.g, L.nsys, L.x_complex, L.pool_bytes);
    if (!p.fn) return hipErrorInvalidConfiguration;
    if (p.kind == 1 && p.ring < rcocg::kRingMin) return hipErrorInvalidValue;
    rcocg::Args a{};
    a.n0 = L.g.n0;
    a.n1 = L.g.n1;
    a.n2 = L.g.n2;
    a.P = L.g.n0 * L.g.n1;
    stencil_weights(L.g.h, a.cw);
    a.vloc = L.vloc;
    a.eps = L.eps;
    a.ns = L.ns;
    a.nsys = L.nsys;
    a.omega_v = L.omega_v;
    a.order = L.order;
    a.counter = L.counter;
    a.tol2 = L.tol * L.tol;
    a.max_iter = L.max_iter;
    a.tiny_status = L.tiny_status;
    a.nd = L.g.nd();
    a.rhs = L.rhs;
    a.x = L.x;
    a.pool = L.pool;
    a.xc = L.x_complex ? 1 : 0;
    a.iters = L.iters;
    a.status = L.status;
    a.refinements = L.refinements;
    a.nbuf = p.s.nbuf;
    a.rs = p.s.rs;
    a.periodic = L.g.periodic() ? 1 : 0;
    a.ring = p.ring;
    if (std::getenv("RPA_COCG_VERBOSE")) {
        const char* const kinds[] = {"", "streaming", "resident-ring", "resident"};
        std::fprintf(stderr, "rcocg shape %s C=%d Z=%d bs=%d grid=%d ring=%d lds=%zu\n",
                     kinds[p.kind], p.kind > 1 ? 1 : p.s.v->C, p.kind > 1 ? 2 * rres::kPairs : p.s.v->Z,
                     p.bs, p.grid, p.ring, p.lds);
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(p.fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(p.lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(p.fn, dim3(p.grid), dim3(p.bs), p.lds, st, a);
    return hipGetLastError();
}

namespace {

hipError_t launch_check(const RcocgLaunch& L, const int* order, double* r, double* b2,
                        hipStream_t st) {
    const Shape s = choose(L.g);
    if (!s.v) return hipErrorInvalidConfiguration;
    rcocg::CheckArgs a{};
    a.n0 = L.g.n0;
    a.n1 = L.g.n1;
    a.n2 = L.g.n2;
    a.P = L.g.n0 * L.g.n1;
    stencil_weights(L.g.h, a.cw);
    a.vloc = L.vloc;
    a.eps = L.eps;
    a.omega_v = L.omega_v;
    a.rhs = L.rhs;
    a.ns = L.ns;
    a.order = order;
    a.x = static_cast<const double2*>(L.x);
    a.rout = reinterpret_cast<double2*>(r);
    a.tol2 = L.tol * L.tol;
    a.nd = L.g.nd();
    a.status = L.status;
    a.refinements = L.refinements;
    a.b2 = b2;
    a.rs = s.rs;
    a.nbuf = 2;
    a.periodic = L.g.periodic() ? 1 : 0;
    size_t lds = lds_bytes(L.g, s.v->C, 1, 2, s.rs);
    if (lds > 150 * 1024) {
        a.nbuf = 1;
        lds = lds_bytes(L.g, s.v->C, 1, 1, s.rs);
    }
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(s.v->check),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(s.v->check, dim3(L.nsys), dim3(s.bs), lds, st, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_residual(const RcocgLaunch& L, double* r, hipStream_t s) {
    return launch_check(L, L.order, r, nullptr, s);
}

hipError_t launch_residual_check(const RcocgLaunch& L, double* b2, hipStream_t s) {
    return launch_check(L, nullptr, nullptr, b2, s);
}

}  // namespace rpa

// For bench.py and the tests: which kernel solves on a grid, and the ring it keeps, where the
// workspace is that of the size query.
extern "C" int rpa_internal_real_form(const int32_t* n, int32_t nsys, int32_t x_complex, int32_t* ring) {
    const rpa::Grid g{n[0], n[1], n[2], 1.0, 0};
    if (rpa::cocg_shape_forced()) return 0;
    const size_t state = size_t(nsys) * g.nd() * 40;
    const rpa::Plan p =
        rpa::make_plan(g, nsys, x_complex != 0, std::max(state, rpa::rcocg_pool_bytes(g, nsys)));
    *ring = p.ring;
    return p.kind;
}
