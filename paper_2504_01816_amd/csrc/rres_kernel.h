// Real-form COCG (rcocg_kernel.h) for grids whose Lanczos vectors fit the registers of one
// workgroup: thread = column of the x-y plane, the column's n2 = NZ points of v_k and of w / v_{k-1}
// in registers, every z neighbour a register of its own.
//
// What it removes: the streaming kernel moves 43 B per point-iteration, 32 of them w and v_k going
// to memory and back between iterations, and so runs at the memory rate.  With FULL p and x stay in
// registers as well and a solve touches memory only at its start and end (0.3 B per point-iteration
// counted at 20^3); else each v_k goes to the ring (8 B) and comes back once for the update of p and x
// (8 + 48 / m B; 24.7 counted at 24^3).
// That update is done by waves of its own while the others sweep: the ring has two halves of m
// vectors, one filled by the sweeps, one folded into p and x, a few elements per barrier step.
// What bounds it: waits on LDS (24 neighbours of x and y per point) and on the barriers, 60% of the
// waves' cycles at 24^3; LDS itself is busy in 39% of the CUs' cycles (40% at 20^3).  Two planes are
// staged side by side, so that one 16-byte read serves the points of both, with a row stride of
// n0 + 16 entries: bank conflicts are 0 (24^3) and 2.4% (20^3) of the LDS cycles.
//
// Measured, calls with the streaming kernel against this one: 24^3, 1024 systems, omega 0.02, tol
// 1e-10: 24.3 -> 16.7 ms (the fold by the sweeping waves themselves, between sweeps, took 3.2 more);
// the same isolated, omega 0.31: 12.1 -> 8.8 ms; 20^3, 2048 systems over eight frequencies, twice (p
// and x in registers): 39.2 -> 17.7 ms; 12^3, 16 systems: 1.25 -> 0.55 ms; 22 x 27 x 25, 143 systems:
// 8.7 -> 5.0 ms.
//
// n2 is a template parameter because a register array needs constant indices; the rule that picks
// this kernel (rcocg.hip) is the register budget of the column height and the workgroup.
#pragma once

#include "rcocg_kernel.h"

namespace rpa {
namespace rres {

using cocg::ld;
using cocg::lds_barrier;
using cocg::st;
using cocg::uniform;
using cocg::wg_reduce;
using rcocg::Args;
using rcocg::Coef;
using rcocg::global_barrier;
using rcocg::kRing;
using rcocg::kSlotExtra;
using rcocg::Recurrence;

constexpr int kPairs = 2;     // plane pairs staged between two barriers


// LDS: reductions, the coefficients of both ring halves, the system counter, then two buffers of
// kPairs staged pairs of (n1 + 12) rows of n0 + 16 entries.
__host__ __device__ constexpr size_t lds_fixed() {
    return 16 * 3 * sizeof(double) + 2 * kRing * sizeof(Coef) + 16;
}

// One column's state in the sweep.
struct Column {
    int n0, n1, P, rs, PL, corner, gx, gy;
    unsigned col;
    bool own, hx, hy, hx2, hy2, narrow;
    double cz[7];          // weights of the z neighbours across the periodic boundary
};

__device__ __forceinline__ Column make_column(const Args& a) {
    Column c;
    const bool per = a.periodic != 0;
    c.n0 = a.n0;
    c.n1 = a.n1;
    c.P = a.P;
    c.rs = a.n0 + 16;
    c.PL = (a.n1 + 12) * c.rs;
    c.own = int(threadIdx.x) < a.P;
    c.col = c.own ? threadIdx.x : 0;
    const int cx = int(c.col) % a.n0, cy = int(c.col) / a.n0;
    c.corner = cy * c.rs + cx;               // the entry of (cx - 6, cy - 6)
    // ghost images: at most one along each axis from 12 points on
    c.gx = cx < 6 ? a.n0 : -a.n0;
    c.gy = (cy < 6 ? a.n1 : -a.n1) * c.rs;
    c.hx = c.own && per && (cx < 6 || cx >= a.n0 - 6);
    c.hy = c.own && per && (cy < 6 || cy >= a.n1 - 6);
    c.hx2 = c.hx && cx < 6 && cx >= a.n0 - 6;
    c.hy2 = c.hy && cy < 6 && cy >= a.n1 - 6;
    c.narrow = a.n0 < 12 || a.n1 < 12;
#pragma unroll
    for (int k = 0; k < 7; ++k) c.cz[k] = per ? a.cw[k] : 0.0;
    return c;
}

// W = (A - sigma) V - cp W over the column (ds = diagonal without V_loc), its sums into acc; with
// STORE the column of V goes to vnew.
template <int NZ, bool STORE>
__device__ __forceinline__ void sweep(const Args& a, const Column& c, double2* planes, double ds,
                                      double cp, double* vnew, const double (&V)[NZ],
                                      double (&W)[NZ], bool first, double (&acc)[3]) {
    constexpr int kStep = 2 * kPairs;
    // STORE: V_loc of a step is read before the stores of the step in front of it, since the memory
    // counter is in order and a wait behind them would be a wait for the stores
    double vn[kStep];
#pragma unroll
    for (int zz = 0; zz < kStep; ++zz)
        if (STORE && zz < NZ) vn[zz] = ld(a.vloc + zz * c.P, c.col);
#pragma unroll
    for (int z0 = 0; z0 < NZ; z0 += kStep) {
        // opaque bases per step: otherwise the addresses of all planes are hoisted out of the solve
        // and take the registers of the vectors
        int o = ((z0 / kStep) & 1) * kPairs * c.PL + c.corner;
        unsigned col = c.col;
        asm volatile("" : "+v"(o), "+v"(col));
        double vl[kStep];
#pragma unroll
        for (int zz = 0; zz < kStep; ++zz) {
            if (z0 + zz >= NZ) continue;
            vl[zz] = STORE ? vn[zz] : ld(a.vloc + (z0 + zz) * c.P, col);
        }
#pragma unroll
        for (int q = 0; q < kPairs; ++q) {
            const int z = z0 + 2 * q;
            if (z >= NZ) continue;
            double2* L = planes + o + q * c.PL + 6 * c.rs + 6;
            const double2 v{V[z], V[z + 1 < NZ ? z + 1 : z]};
            if (c.own) L[0] = v;
            if (c.hx) L[c.gx] = v;
            if (c.hy) L[c.gy] = v;
            if (c.narrow) {
                if (c.hx2) L[-c.n0] = v;
                if (c.hy2) L[-c.n1 * c.rs] = v;
            }
        }
        lds_barrier();
#pragma unroll
        for (int zz = 0; zz < kStep; ++zz)
            if (STORE && z0 + kStep + zz < NZ) vn[zz] = ld(a.vloc + (z0 + kStep + zz) * c.P, col);
        if (STORE) asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < kPairs; ++q) {
            const int z = z0 + 2 * q;
            if (z >= NZ) continue;
            int oz = o + q * c.PL;
            asm volatile("" : "+v"(oz));
            const double2* Lx = planes + oz + 6 * c.rs;              // row of the point
            const double2* Ly = planes + oz + 6;                     // column of the point
            constexpr int kTwo = 2;
            double s[kTwo];
#pragma unroll
            for (int e = 0; e < kTwo; ++e) {
                const int ze = z + e < NZ ? z + e : z;
                s[e] = (ds + vl[2 * q + (z + e < NZ ? e : 0)]) * V[ze] - cp * W[ze];
            }
#pragma unroll
            for (int k = 1; k <= 6; ++k) {
                const double2 a1 = Lx[6 + k], a2 = Lx[6 - k];
                const double2 b1 = Ly[(6 + k) * c.rs], b2 = Ly[(6 - k) * c.rs];
#pragma unroll
                for (int e = 0; e < kTwo; ++e) {
                    const int ze = z + e;
                    if (ze >= NZ) continue;
                    const bool up = ze + k < NZ, dn = ze - k >= 0;
                    const double vu = V[up ? ze + k : ze + k - NZ], vd = V[dn ? ze - k : ze - k + NZ];
                    double t = e == 0 ? (a1.x + a2.x) + (b1.x + b2.x) : (a1.y + a2.y) + (b1.y + b2.y);
                    if (up) t += vu;
                    if (dn) t += vd;
                    s[e] += a.cw[k] * t;
                    if (!up) s[e] += c.cz[k] * vu;
                    if (!dn) s[e] += c.cz[k] * vd;
                }
                rcocg::hold<kTwo>(s);
            }
#pragma unroll
            for (int e = 0; e < kTwo; ++e) {
                if (z + e >= NZ) continue;
                W[z + e] = s[e];
                acc[0] += V[z + e] * s[e];
                acc[1] += s[e] * s[e];
                if (first) acc[2] += V[z + e] * V[z + e];
                if (STORE && c.own) st(vnew + (z + e) * c.P, col, V[z + e]);
            }
        }
    }
    if (!c.own) acc[0] = acc[1] = acc[2] = 0.0;
}

// v_k = (w - delta v_{k-1}) / beta; W becomes v_{k-1}.
template <int NZ>
__device__ __forceinline__ void advance(const Recurrence& rc, double (&V)[NZ], double (&W)[NZ]) {
    const double c1 = rc.sc * rc.ibeta, c2 = -rc.delta * rc.sc * rc.ibeta;
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        const double t = rcocg::vnext(c1, W[z], c2, V[z]);
        W[z] = V[z];
        V[z] = t;
    }
}

// Cancellation in |w|^2 - delta^2: w with sigma = alpha is w - delta v_k; its sums once more.
template <int NZ>
__device__ __forceinline__ void shift_w(double dl, bool own, const double (&V)[NZ], double (&W)[NZ],
                                        double (&acc)[3]) {
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
        W[z] -= dl * V[z];
        acc[0] += V[z] * W[z];
        acc[1] += W[z] * W[z];
    }
    if (!own) acc[0] = acc[1] = 0.0;
}

// The next system in dispatch order, or -1 (every wave of the workgroup gets the same).
__device__ __forceinline__ int next_system(const Args& a, int* next) {
    global_barrier();           // slot and LDS free for the next system
    if (threadIdx.x == 0) *next = atomicAdd(a.counter, 1);
    lds_barrier();
    const int pos = __builtin_amdgcn_readfirstlane(*next);
    return pos < a.nsys ? a.order[pos] : -1;
}

__device__ __forceinline__ void finish(const Args& a, int sys, const Recurrence& rc) {
    if (threadIdx.x == 0) {
        a.iters[sys] = rc.it;
        a.status[sys] = rc.stat;
        if (a.refinements) a.refinements[sys] = 0;
    }
}

// Nothing solved: x = 0 (not a number where b is not finite).
__device__ __forceinline__ void zero_x(const Args& a, int sys, const double* b) {
    for (unsigned i = threadIdx.x; i < unsigned(a.nd); i += blockDim.x) {
        const double v = 0.0 * ld(b, i);
        if (a.xc) st(reinterpret_cast<double2*>(a.x) + int64_t(sys) * a.nd, i, double2{v, 0.0});
        else st(reinterpret_cast<double*>(a.x) + int64_t(sys) * a.nd, i, v);
    }
}

// ---------------------------------------------------------------- p and x in registers
// Real solutions.  WPE: waves per SIMD that the registers have to allow.
template <int NZ, int WPE>
__global__ __attribute__((amdgpu_flat_work_group_size(64, 512), amdgpu_waves_per_eu(WPE, 8)))
void full_wg(Args a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* red = reinterpret_cast<double*>(smem_raw);                 // 16 waves x 3
    int* next = reinterpret_cast<int*>(smem_raw + lds_fixed() - 16);
    double2* planes = reinterpret_cast<double2*>(smem_raw + lds_fixed());
    const Column c = make_column(a);
    if (!a.periodic)        // ghost entries outside an isolated box read zero
        for (int e = threadIdx.x; e < 2 * kPairs * c.PL; e += blockDim.x) planes[e] = double2{0.0, 0.0};
    for (int sys; (sys = next_system(a, next)) >= 0;) {
        const double* b = a.rhs + int64_t(sys) * a.nd;
        const double diag = a.cw[0] - a.eps[sys % a.ns];
        Recurrence rc(a.omega_v[sys / a.ns], a);
        double V[NZ], W[NZ], PR[NZ], PI[NZ], X[NZ];
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
            V[z] = c.own ? ld(b + z * c.P, c.col) : 0.0;
            W[z] = PR[z] = PI[z] = X[z] = 0.0;
        }
        while (!rc.done) {
            const bool first = rc.it == 0;
            if (!first) advance<NZ>(rc, V, W);
            double acc[3] = {0.0, 0.0, 0.0};
            sweep<NZ, false>(a, c, planes, diag - rc.sigma, rc.cp(), nullptr, V, W, first, acc);
            wg_reduce<3>(acc, red);
            if (!rc.norms(acc)) break;                // zero or too small a right-hand side
            if (rc.cancels(acc)) {
                const double dl = rc.shift(acc);
                double ac2[3] = {0.0, 0.0, 0.0};
                shift_w<NZ>(dl, c.own, V, W, ac2);
                wg_reduce<3>(ac2, red);
                rc.reshifted(ac2, acc);
            }
            const Coef cf = rc.step(acc);
            // the operations of update_px, every step
            const double s1 = first ? rc.ibn : 1.0;
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                const double pr = s1 * V[z] - cf.lr * PR[z] + cf.li * PI[z];
                PI[z] = -cf.lr * PI[z] - cf.li * PR[z];
                PR[z] = pr;
                X[z] += cf.er * pr - cf.ei * PI[z];
            }
        }
        if (rc.it == 0) {
            zero_x(a, sys, b);
        } else if (c.own) {
            double* x = reinterpret_cast<double*>(a.x) + int64_t(sys) * a.nd;
#pragma unroll
            for (int z = 0; z < NZ; ++z) st(x + z * c.P, c.col, X[z]);
        }
        finish(a, sys, rc);
    }
}

// ---------------------------------------------------------------- p and x in memory
// Folds one ring half (M vectors) into p and x, kE elements per lane and chunk, with the loads of
// two chunks in flight: a chunk then waits a barrier step for its data and not for the memory.  That
// needs a wait on the older chunk alone, so nothing here branches: lanes past the end (and chunks
// with nothing to fold) read the last element and store to `spare`.
constexpr int kE = 2;

template <int M, bool XC>
struct Chunk {
    using X = typename std::conditional<XC, double2, double>::type;
    double v[kE][M];
    double2 pv[kE];
    X xv[kE];
    unsigned pos;          // element of lane 0
};

template <int M, bool XC>
struct Fold {
    using X = typename Chunk<M, XC>::X;
    const double* ring;    // the half's vectors
    const Coef* coef;
    double2* p;
    X* x;
    double* spare;
    int64_t nd;
    unsigned pos, n, lanes, lane;  // next element to load, elements, lanes that share the work
    bool first;
    double s1;

    __device__ __forceinline__ void load(Chunk<M, XC>& c) {
        c.pos = pos;
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const unsigned i = min(pos + e * lanes + lane, n - 1);
#pragma unroll
            for (int j = 0; j < M; ++j) c.v[e][j] = ld(ring + j * nd, i);
            c.pv[e] = ld(p, i);
            c.xv[e] = ld(x, i);
        }
        pos = min(pos + kE * lanes, n);
    }
    // the operations of update_px on the loaded elements, then the loads of another chunk
    __device__ __forceinline__ void run(Chunk<M, XC>& c) {
        const double sv = first ? s1 : 1.0;
        double xr[kE], xi[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            c.v[e][0] *= sv;
            // p and x start at zero: what memory holds before the first half is not used
            c.pv[e].x = first ? 0.0 : c.pv[e].x;
            c.pv[e].y = first ? 0.0 : c.pv[e].y;
            if constexpr (XC) {
                xr[e] = first ? 0.0 : c.xv[e].x;
                xi[e] = first ? 0.0 : c.xv[e].y;
            } else {
                xr[e] = first ? 0.0 : c.xv[e];
                xi[e] = 0.0;
            }
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const Coef q = coef[j];
#pragma unroll
            for (int e = 0; e < kE; ++e) {
                const double pr = c.v[e][j] - q.lr * c.pv[e].x + q.li * c.pv[e].y;
                c.pv[e].y = -q.lr * c.pv[e].y - q.li * c.pv[e].x;
                c.pv[e].x = pr;
                xr[e] += q.er * c.pv[e].x - q.ei * c.pv[e].y;
                if (XC) xi[e] += q.er * c.pv[e].y + q.ei * c.pv[e].x;
            }
            asm volatile("" ::: "memory");        // one step's coefficients at a time
        }
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const unsigned i = c.pos + e * lanes + lane;
            double2* sp = reinterpret_cast<double2*>(spare) + lane;
            X* tx = i < n ? x + i : reinterpret_cast<X*>(sp);
            double2* tp = i < n ? p + i : sp;
            if constexpr (XC) *tx = double2{xr[e], xi[e]};
            else *tx = xr[e];
            *tp = c.pv[e];
        }
        load(c);
    }
};

// Waves past the plane's columns fold, the others sweep; both run the same recurrence on the same
// sums and meet at the same barriers.
// M: vectors of a ring half, XC: complex solutions.
template <int NZ, int BSMAX, int WPE, int M, bool XC>
__global__ __attribute__((amdgpu_flat_work_group_size(64, BSMAX), amdgpu_waves_per_eu(WPE, 8)))
void ring_wg(Args a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* red = reinterpret_cast<double*>(smem_raw);                 // 16 waves x 3
    Coef* coef = reinterpret_cast<Coef*>(smem_raw + 16 * 3 * sizeof(double));
    int* next = reinterpret_cast<int*>(smem_raw + lds_fixed() - 16);
    double2* planes = reinterpret_cast<double2*>(smem_raw + lds_fixed());
    constexpr int kSteps = (NZ + 2 * kPairs - 1) / (2 * kPairs);
    const int cwaves = (a.P + 63) / 64;
    const bool folds = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6) >= cwaves;
    if (!a.periodic)        // ghost entries outside an isolated box read zero
        for (int e = threadIdx.x; e < 2 * kPairs * (a.n1 + 12) * (a.n0 + 16); e += blockDim.x)
            planes[e] = double2{0.0, 0.0};
    using X = typename Chunk<M, XC>::X;
    double* ring = a.pool + int64_t(blockIdx.x) * (2 * M + kSlotExtra) * a.nd;
    double2* p = reinterpret_cast<double2*>(ring + 2 * M * a.nd);      // then one spare vector
    for (int sys; (sys = next_system(a, next)) >= 0;) {
        const double* b = a.rhs + int64_t(sys) * a.nd;
        X* x = reinterpret_cast<X*>(a.x) + int64_t(sys) * a.nd;
        const double diag = a.cw[0] - a.eps[sys % a.ns];
        Recurrence rc(a.omega_v[sys / a.ns], a);
        int slot = 0, half = 0;                         // fill of the half in use
        bool none = true;                               // no half folded yet
        if (!folds) {
            const Column c = make_column(a);
            double V[NZ], W[NZ];
#pragma unroll
            for (int z = 0; z < NZ; ++z) {
                V[z] = c.own ? ld(b + z * c.P, c.col) : 0.0;
                W[z] = 0.0;
            }
            while (!rc.done) {
                const bool first = rc.it == 0;
                if (!first) advance<NZ>(rc, V, W);
                double acc[3] = {0.0, 0.0, 0.0};
                sweep<NZ, true>(a, c, planes, diag - rc.sigma, rc.cp(), ring + (half * M + slot) * a.nd,
                                V, W, first, acc);
                wg_reduce<3>(acc, red);
                if (!rc.norms(acc)) break;            // zero or too small a right-hand side
                if (rc.cancels(acc)) {
                    const double dl = rc.shift(acc);
                    double ac2[3] = {0.0, 0.0, 0.0};
                    shift_w<NZ>(dl, c.own, V, W, ac2);
                    wg_reduce<3>(ac2, red);
                    rc.reshifted(ac2, acc);
                }
                const Coef cf = rc.step(acc);
                if (threadIdx.x == 0) coef[half * kRing + slot] = cf;
                ++slot;
                if (!rc.done && slot == M) {
                    global_barrier();                  // the other half is folded, this one is full
                    slot = 0;
                    half ^= 1;
                    none = false;
                }
            }
        } else {
            Fold<M, XC> f;
            Chunk<M, XC> c0, c1;
            f.nd = a.nd;
            f.lane = threadIdx.x - 64 * cwaves;
            f.p = p;
            f.x = x;
            f.n = unsigned(a.nd);
            f.lanes = blockDim.x - 64 * cwaves;
            f.spare = reinterpret_cast<double*>(p + a.nd);
            f.ring = ring;
            f.coef = coef;
            f.first = true;
            f.s1 = 0.0;
            f.pos = f.n;                               // nothing to fold yet
            f.load(c0);
            f.load(c1);
            while (!rc.done) {
#pragma unroll 1
                for (int s = 0; s < kSteps / 2; ++s) {
                    f.run(c0);
                    lds_barrier();
                    f.run(c1);
                    lds_barrier();
                }
                if (kSteps % 2) lds_barrier();
                double acc[3] = {0.0, 0.0, 0.0};
                wg_reduce<3>(acc, red);
                if (!rc.norms(acc)) break;
                if (rc.cancels(acc)) {
                    rc.shift(acc);
                    double ac2[3] = {0.0, 0.0, 0.0};
                    wg_reduce<3>(ac2, red);
                    rc.reshifted(ac2, acc);
                }
                rc.step(acc);
                ++slot;
                if (rc.done || slot == M)
                    while (c0.pos < f.n || c1.pos < f.n) {       // what the steps did not reach
                        f.run(c0);
                        f.run(c1);
                    }
                if (!rc.done && slot == M) {
                    global_barrier();
                    f.ring = ring + half * M * a.nd;
                    f.coef = coef + half * kRing;
                    f.first = none;
                    f.s1 = rc.ibn;
                    f.pos = 0;
                    f.load(c0);
                    f.load(c1);
                    slot = 0;
                    half ^= 1;
                    none = false;
                }
            }
        }
        if (rc.it == 0) {
            zero_x(a, sys, b);
        } else {
            // the vectors since the last full half, by every wave
            global_barrier();
            rcocg::update_px<X, kRing>(a.nd, ring + half * M * a.nd, p, x, coef + half * kRing, slot,
                                       none, rc.ibn, true);
        }
        finish(a, sys, rc);
    }
}

using KernelFn = void (*)(Args);

// Instances for a column of nz points, or null: full_wg for nz 12 .. 20 (up to 512 columns),
// ring_wg for nz 12 .. 26 (up to 704 columns, 12 waves) and 27 .. 32 (up to 448, 8 waves) with
// half = kRing, or kRingHalfMin where full_wg takes the real solutions.
constexpr int kRingHalfMin = 1;
KernelFn full_variant(int nz);
KernelFn ring_variant(int nz, bool xc, int half);

}  // namespace rres
}  // namespace rpa
