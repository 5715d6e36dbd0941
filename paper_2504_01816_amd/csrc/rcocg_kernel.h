// Batched COCG on real right-hand sides (H - eps_n - i omega) x = b, b real, in FP64.
//
// H - eps_n is real symmetric and b is real, so every COCG residual is a complex multiple of
// a real vector: the Krylov basis is the real Lanczos basis of H - eps_n,
//   w = (A - sigma) v_k - beta_k v_{k-1},  delta = v_k^T w,  alpha_k = sigma + delta,
//   beta_{k+1}^2 = |w|^2 - delta^2,        v_{k+1} = (w - delta v_k) / beta_{k+1},
// and the COCG iterate is the Galerkin solution on it, updated through the L D L^T factors of
// the shifted tridiagonal matrix:
//   d_k = alpha_k - i omega - beta_k l_k,  l_k = beta_k / d_{k-1},  zeta_k = -l_k zeta_{k-1},
//   p_k = v_k - l_k p_{k-1},  x_k = x_{k-1} + (zeta_k / d_k) p_k,  |r_k| = beta_{k+1} |zeta_k / d_k|.
// In exact arithmetic these are the iterates and residual norms of COCG, one product with A per
// iteration; |Im d_k| >= omega, so the recurrence cannot break down.
//
// What bounds it: memory.  COCG on complex vectors moves r, p, x twice through two sweeps
// (120 B per point-iteration measured at 24^3, 161 B at 48^3).  Here one sweep per iteration
// reads w and v_k and writes v_{k+1} and w (32 B), and p and x are updated once per m <= kRingLong
// iterations from the last m basis vectors, which a ring keeps (8 + 48 / m B per
// point-iteration; m = 16 instead of 8: 43.7 -> 41.9 ms at 48^3, 83.4 -> 81.5 ms at 32^3, the
// launches below).
//
//  * sigma is the previous alpha, so |w|^2 - delta^2 does not cancel; where it does (first step,
//    b close to an eigenvector) the sweep is repeated with sigma = alpha.
//  * One workgroup owns a system for its whole solve and takes the next one from a counter, in
//    dispatch order; its vectors live in a slot of the state pool (ring vectors, w, p).
//  * A sweep marches along z.  A thread owns C consecutive rows of the x-y plane at one x and
//    keeps planes z-6 .. z+5+Z of v_{k+1} in registers; the current planes are staged in LDS with
//    ghost columns and rows.  The C rows share their y neighbours: 12 + 12 / C LDS reads per
//    point instead of 24.
//  * The queue is carried from sweep to sweep (periodic grids): it starts the next sweep with 12
//    planes of w instead of 12 planes of w and v.
//  * Reductions are fixed-order and the operations of a solve depend on the grid alone: results
//    are bitwise reproducible, whatever slot, ring or launch a system gets.
//
// Measured, chi0 block-applies, the two-sweep complex kernel against this one: 24^3, 1024
// systems, omega 0.02, tol 1e-10: 62.2 -> 24.3 ms; 48^3, 1024 systems, omega 8.8, tol 1e-8: 136 ->
// 42 ms; 32^3, 2 x 1024 systems with complex solutions: 217 -> 81 ms.  At 48^3, 16384 systems, omega
// 0.11 counters give 48.6 B per point-iteration (43 by design), at 5.6 TB/s.
#pragma once

#include <type_traits>

#include "cocg_kernel.h"

namespace rpa {
namespace rcocg {

using cocg::ld;
using cocg::lds_barrier;
using cocg::st;
using cocg::uniform;
using cocg::wg_reduce;

constexpr int kRing = 8;       // basis vectors of one half of a resident kernel's ring
constexpr int kRingLong = 16;  // most basis vectors kept between two updates of p and x here
constexpr int kRingMin = 2;    // the sweep reads v_k and writes v_{k+1}
constexpr int kDelay = 5;      // planes of v_k between lead and centre that LDS holds (C > 1)
constexpr int kSlotExtra = 3;  // vectors of a slot besides the ring: w, complex p

struct Args {
    int n0, n1, n2, P;
    double cw[7];          // cw[k] = -1/2 w_k / h^2 for k >= 1; cw[0] = -1/2 * 3 w_0 / h^2
    const double* vloc;
    const double* eps;
    int ns, nsys;
    const double* omega_v; // per trial vector j (system s = n + ns j)
    const int* order;      // the i-th system to start is order[i]
    int* counter;          // next position in order (0 before the launch)
    double tol2;
    int max_iter;
    int tiny_status;       // status of a right-hand side that is too small to solve for (x = 0)
    int64_t nd;
    const double* rhs;     // system-major, N_d real each
    void* x;               // system-major: N_d real (XS = double) or complex (double2)
    int xc;                // x is complex (kernels that do not know it by their type)
    double* pool;          // gridDim.x slots of (ring + kSlotExtra) * N_d doubles
    int ring;              // basis vectors kept, kRingMin .. kRingLong
    int* iters;
    int* status;
    int* refinements;      // written 0 per system if not null
    int nbuf;              // LDS plane buffers (2: one barrier per step, 1: two barriers)
    int rs;                // LDS row stride in entries, >= n0 + 12
    int periodic;
};

// Ragged, periodic sweeps: the reads of v past the top (plane z + 7 - n2 of v in step z, from
// z = n2 - 7 on) go to rows that other threads stored in step z + 7 - n2.  Whether step z starts
// with the barrier that orders them.  It stands in front of the step's own stores, so the one in
// step n2 - 7 covers planes 0 .. n2 - 8: all six from n2 = 13 on; n2 = 12 needs another one for
// plane 5, which step n2 - 2 reads.
__host__ __device__ constexpr bool wrap_barrier(int n2, int z) {
    return z == n2 - 7 || (n2 == 12 && z == n2 - 2);
}
// Every such read has a barrier after its store's step and no later than its own.
constexpr bool wrap_ordered(int n2) {
    for (int z = n2 - 7; z <= n2 - 2; ++z) {
        bool ok = false;
        for (int b = z + 7 - n2 + 1; b <= z; ++b) ok = ok || wrap_barrier(n2, b);
        if (!ok) return false;
    }
    return true;
}
static_assert(wrap_ordered(12) && wrap_ordered(13) && wrap_ordered(14) && wrap_ordered(48), "");

__device__ __forceinline__ void global_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The thread's place in the plane: x = cx, rows y0 .. y0 + C - 1.  Threads past the last row
// group own no row and read the first columns.  Where C does not divide n1 (ragged), the last
// group reads the rows past n1 - 1 from their periodic images (zero in a box), which other
// threads own and store: own(i) says what this thread stages, stores and sums.
template <int C>
struct Rows {
    int cx, y0;
    unsigned col[C];       // y n0 + x: the only per-thread part of an address
    bool on, own_[C];
    template <bool RAG>
    __device__ bool own(int i) const { return RAG ? own_[i] : on; }
};

template <int C, bool RAG>
__device__ __forceinline__ Rows<C> make_rows(int n0, int n1) {
    Rows<C> rw;
    const int tid = threadIdx.x;
    rw.on = tid < (n1 + C - 1) / C * n0;
    const int t = rw.on ? tid : 0;
    rw.cx = t % n0;
    rw.y0 = t / n0 * C;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const int y = rw.y0 + i;
        rw.own_[i] = rw.on && y < n1;
        rw.col[i] = unsigned((RAG && y >= n1 ? y - n1 : y) * n0 + rw.cx);
    }
    return rw;
}

// Ends a group of LDS reads: what was read is consumed here, which bounds the registers held by
// reads in flight.
template <int C>
__device__ __forceinline__ void hold(double (&s)[C]) {
#pragma unroll
    for (int i = 0; i < C; ++i) asm volatile("" : "+v"(s[i])::"memory");
}

// s[i] += the off-diagonal stencil of the thread's C rows: x and outer y neighbours from the LDS
// plane (Lc: the first row's entry), z neighbours and the thread's own rows from the queue.
template <int NQ, int C>
__device__ __forceinline__ void stencil(const double (&cw)[7], const double* Lc, int rs,
                                        const double (&Q)[NQ][C], int zc, double (&s)[C]) {
    // y: the rows above and below the thread's rows from LDS, its own from the queue
#pragma unroll
    for (int k = 1; k <= 6; ++k) {
        const double b1 = Lc[-k * rs], b2 = Lc[(C - 1 + k) * rs];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (k + i <= 6) s[i] += cw[k + i] * b1;
            if (k + C - 1 - i <= 6) s[i] += cw[k + C - 1 - i] * b2;
        }
        hold<C>(s);
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int j = 0; j < C; ++j)
            if (i != j) s[i] += cw[i > j ? i - j : j - i] * Q[zc][j];
#pragma unroll
    for (int k = 1; k <= 6; ++k) {
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const double a1 = Lc[i * rs + k], a2 = Lc[i * rs - k];
            s[i] += cw[k] * ((a1 + a2) + (Q[zc + k][i] + Q[zc - k][i]));
        }
        hold<C>(s);
    }
}

// v_{k+1} at a point, with one rounding order wherever it is formed.
__device__ __forceinline__ double vnext(double cw, double w, double cv, double v) {
    return __builtin_fma(cw, w, cv * v);
}

// One sweep: from the lead vectors lw, lv it forms v = cw lw + cv lv plane by plane, stores v to
// vout, and q = (A - sigma) v - cp lv to wout.  lw may be wout (in place: a plane is read
// at least 6 planes before it is written; the periodic images read past the top come
// from vout).  acc = (v.q, q.q, v.v).  With warm = true, Q[0..11] holds the swept vector of the
// previous sweep (that is lv) on planes -6 .. 5.
template <int C, int Z, bool RAG>
__device__ __forceinline__ void sweep(const Args& a, const Rows<C>& rw, double* planes,
                                      double diag0, const double* lw, const double* lv,
                                      double cw, double cv, double cp, double* vout, double* wout,
                                      double (&Q)[12 + Z][C], bool warm, double (&acc)[3],
                                      double* delay) {
    const int n2 = a.n2, P = a.P, rs = a.rs, n0 = a.n0, n1 = a.n1;
    // lv at the centre planes: with one row per thread a second queue holds it from the lead plane
    // on; with more there are no registers for it (48^3, C = 3: spilled, 163 ms against 48), and the
    // thread's own values wait in LDS, the newest plane in H (read again from memory: 48.3
    // ms instead of 43.7)
    constexpr bool UQ = C == 1;
    static_assert(UQ || Z == 1, "the delay line advances one plane per step");
    constexpr int NU = UQ ? 6 + Z : 1;
    double U[NU][C], H[C];
    const int BS = blockDim.x;
    double* dl = delay + threadIdx.x * C;    // [plane mod kDelay][BS][C]
    const int PL = (n1 + 11 + C) * rs;
    const bool per = a.periodic != 0;
    constexpr int kWarm = C == 1 ? 6 : 3;    // planes of w loaded together
    if (warm) {
#pragma unroll
        for (int s0 = 0; s0 < 12; s0 += kWarm) {
            double t[kWarm][C];
#pragma unroll
            for (int s = 0; s < kWarm; ++s) {
                int z = s0 + s - 6;
                z += (z < 0) ? n2 : 0;
#pragma unroll
                for (int i = 0; i < C; ++i) t[s][i] = ld(lw + z * P, rw.col[i]);
            }
#pragma unroll
            for (int s = 0; s < kWarm; ++s)
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    const double vo = Q[s0 + s][i];
                    if (UQ && s0 + s >= 6) U[(s0 + s + 6) % 12 % NU][i] = vo;
                    if (!UQ && s0 + s == 11) H[i] = vo;
                    if (!UQ && s0 + s >= 6 && s0 + s < 11) dl[(s0 + s - 6) * BS * C + i] = vo;
                    Q[s0 + s][i] = vnext(cw, t[s][i], cv, vo);
                }
        }
    } else {
#pragma unroll
        for (int s = 0; s < 12; ++s) {
            const int z = s - 6 + ((s < 6) ? n2 : 0);
            double w[C], v[C];
#pragma unroll
            for (int i = 0; i < C; ++i) w[i] = v[i] = 0.0;
            if (per || s >= 6) {                          // box: planes below 0 are zero
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    w[i] = ld(lw + z * P, rw.col[i]);
                    v[i] = ld(lv + z * P, rw.col[i]);
                    if (RAG && !per && !rw.own_[i]) w[i] = v[i] = 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < C; ++i) {
                Q[s][i] = vnext(cw, w[i], cv, v[i]);
                if (UQ && s >= 6) U[(s + 6) % 12 % NU][i] = v[i];
                if (!UQ && s == 11) H[i] = v[i];
                if (!UQ && s >= 6 && s < 11) dl[(s - 6) * BS * C + i] = v[i];
            }
            // one plane's loads at a time: a cold start is rare, its registers are not
            asm volatile("" ::: "memory");
        }
    }
    double LW[Z][C], LV[Z][C], PV[Z][C];
    // lead planes zo + 6 + zz of the step at zo, and V_loc of its centre planes
    auto fetch = [&](int zo) {
#pragma unroll
        for (int zz = 0; zz < Z; ++zz) {
            const int zu = zo + 6 + zz;
            if (zu < n2) {
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    LW[zz][i] = ld(lw + zu * P, rw.col[i]);
                    LV[zz][i] = ld(lv + zu * P, rw.col[i]);
                    if (RAG && !per && !rw.own_[i]) LW[zz][i] = LV[zz][i] = 0.0;
                }
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    LW[zz][i] = per ? ld(vout + (zu - n2) * P, rw.col[i]) : 0.0;
                    LV[zz][i] = 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < C; ++i) PV[zz][i] = ld(a.vloc + (zo + zz) * P, rw.col[i]);
        }
    };
    fetch(0);
    const int nsteps = n2 / Z;
    int du = 0;                              // zo mod kDelay
#pragma unroll 1
    for (int stp = 0; stp < nsteps; ++stp) {
        const int zo = stp * Z;
        double VV[Z][C];
#pragma unroll
        for (int zz = 0; zz < Z; ++zz) {
            const bool past = zo + 6 + zz >= n2;
            const double c1 = past ? 1.0 : cw;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                Q[12 + zz][i] = vnext(c1, LW[zz][i], cv, LV[zz][i]);
                if constexpr (UQ) {
                    U[6 + zz][i] = LV[zz][i];
                } else {
                    double* d = dl + du * BS * C + i;
                    U[0][i] = *d;
                    *d = H[i];
                    H[i] = LV[zz][i];
                }
                VV[zz][i] = PV[zz][i];
            }
        }
        du = du + 1 == kDelay ? 0 : du + 1;
        static_assert(!RAG || Z == 1, "wrap_barrier counts single planes");
        if (RAG && per && wrap_barrier(n2, zo)) global_barrier();
        if (stp + 1 < nsteps) fetch(zo + Z);
        double* L = planes + (a.nbuf == 2 ? (stp & 1) : 0) * Z * PL;
#pragma unroll
        for (int zz = 0; zz < Z; ++zz)
#pragma unroll
            for (int i = 0; i < C; ++i)
                if (rw.template own<RAG>(i))
                    cocg::stage_point(L + zz * PL, rs, n0, n1, rw.cx, rw.y0 + i, Q[6 + zz][i], per,
                                      true);
        lds_barrier();
#pragma unroll
        for (int zz = 0; zz < Z; ++zz) {
            const double* Lc = L + zz * PL + cocg::lds_center(rs, rw.cx, rw.y0);
            double s[C];
#pragma unroll
            for (int i = 0; i < C; ++i) s[i] = (diag0 + VV[zz][i]) * Q[6 + zz][i] - cp * U[zz][i];
            stencil<12 + Z, C>(a.cw, Lc, rs, Q, 6 + zz, s);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                if (!rw.template own<RAG>(i)) continue;
                const int off = (zo + zz) * P;
                const double c = Q[6 + zz][i];
                st(vout + off, rw.col[i], c);
                st(wout + off, rw.col[i], s[i]);
                acc[0] += c * s[i];
                acc[1] += s[i] * s[i];
                acc[2] += c * c;
            }
        }
        if (a.nbuf == 1) lds_barrier();      // single buffer: reads done before the next write
#pragma unroll
        for (int s = 0; s < 12; ++s)
#pragma unroll
            for (int i = 0; i < C; ++i) Q[s][i] = Q[s + Z][i];
        if constexpr (UQ) {
#pragma unroll
            for (int s = 0; s < 6; ++s)
#pragma unroll
                for (int i = 0; i < C; ++i) U[s][i] = U[s + Z][i];
        }
    }
}

// l_k and e_k = zeta_k / d_k of one step.
struct Coef {
    double lr, li, er, ei;
};

// A right-hand side so small that squares of residuals between |b| and the tolerance (or, for
// tighter tolerances, rounding) are no normal numbers, and no test of them means anything.
__device__ __forceinline__ bool too_small(double bb, double tol2) {
    return bb * fmax(tol2, 1e-32) < 2.2250738585072014e-308;
}

// The scalars of one solve: what the reductions of a sweep turn into.  Every value is uniform over
// the workgroup (wg_reduce), and every thread computes all of them.
struct Recurrence {
    double omega, tol2;
    int max_iter, tiny_status;
    double sigma = 0.0, delta = 0.0, beta = 0.0, ibeta = 1.0;
    double sc = 1.0, bn = 0.0, ibn = 0.0, tgt2 = 0.0;        // sc: 1 / |b| while v_1 stands for b
    double zr = 0.0, zi = 0.0, ir = 0.0, ii = 0.0, b2 = 0.0;  // zeta, 1 / d, beta^2
    int it = 0, stat = 0;
    bool done = false;

    __device__ __forceinline__ Recurrence(double w, const Args& a)
        : omega(w), tol2(a.tol2), max_iter(a.max_iter), tiny_status(a.tiny_status) {}
    __device__ __forceinline__ double cp() const { return it == 0 ? 0.0 : beta * sc; }
    // acc = (v.w, w.w, v.v) of the sweep.  The first one is on b itself: its sums are scaled to
    // v_1 = b / |b|.  False for a right-hand side that is zero or too small.
    __device__ __forceinline__ bool norms(double (&acc)[3]) {
        if (it == 0) {
            if (!(acc[2] > 0.0)) return false;
            if (too_small(acc[2], tol2)) {
                stat = tiny_status;
                return false;
            }
            tgt2 = uniform(tol2 * acc[2]);
            bn = uniform(sqrt(acc[2]));
            ibn = uniform(1.0 / bn);
            acc[0] = uniform(acc[0] / acc[2]);
            acc[1] = uniform(acc[1] / acc[2]);
        }
        b2 = uniform(acc[1] - acc[0] * acc[0]);
        return true;
    }
    __device__ __forceinline__ bool cancels(const double (&acc)[3]) const { return b2 < 1e-3 * acc[1]; }
    // sigma <- alpha; returns delta, which w - delta v removes
    __device__ __forceinline__ double shift(const double (&acc)[3]) {
        sigma = uniform(sigma + acc[0]);
        return acc[0];
    }
    __device__ __forceinline__ void reshifted(const double (&ac2)[3], double (&acc)[3]) {
        const double s1 = it == 0 ? acc[2] : 1.0;
        acc[0] = uniform(ac2[0] / s1);
        acc[1] = uniform(ac2[1] / s1);
        b2 = uniform(acc[1] - acc[0] * acc[0]);
    }
    // the factor step; sets done and stat, returns l and zeta / d
    __device__ __forceinline__ Coef step(const double (&acc)[3]) {
        sc = it == 0 ? ibn : 1.0;
        const double alpha = sigma + acc[0];
        delta = uniform(acc[0]);
        b2 = b2 > 0.0 ? b2 : (b2 <= 0.0 ? 0.0 : b2);          // NaN stays
        Coef c;
        c.lr = uniform(beta * ir);
        c.li = uniform(beta * ii);
        const double dr = alpha - beta * c.lr, di = -omega - beta * c.li;
        if (it == 0) {
            zr = bn;
            zi = 0.0;
        } else {
            const double t = -(c.lr * zr - c.li * zi);
            zi = uniform(-(c.lr * zi + c.li * zr));
            zr = uniform(t);
        }
        const double id2 = 1.0 / (dr * dr + di * di);
        ir = uniform(dr * id2);
        ii = uniform(-di * id2);
        c.er = uniform(zr * ir - zi * ii);
        c.ei = uniform(zr * ii + zi * ir);
        beta = uniform(sqrt(b2));
        ibeta = uniform(b2 > 0.0 ? 1.0 / sqrt(b2) : 0.0);
        sigma = uniform(alpha);
        const double res2 = b2 * (c.er * c.er + c.ei * c.ei);
        ++it;
        if (!(res2 >= 0.0) || !(res2 < INFINITY)) {
            stat = 2;                                          // not a number: a breakdown
            done = true;
        } else if (res2 <= tgt2) {
            done = true;
        } else if (it >= max_iter) {
            stat = 1;
            done = true;
        }
        return c;
    }
};

// p <- v_j - l_j p, x <- x + e_j p (e = zeta / d) over the m newest basis vectors, in order: the
// same operations on every point however many steps one update takes, so a solve's bits do not
// depend on the ring.  The first update starts from x = 0, p = 0, and scales v_1, which is stored
// as b, by s1 = 1 / |b|.  p is not stored at the end of a solve (done).  The coefficients are read
// from LDS at every point: in registers they spilled (48^3: 77 ms against 42, ring of 16).
template <typename XS, int M>
__device__ __forceinline__ void update_px(int64_t nd, const double* ring, double2* p, XS* x,
                                          const Coef* coef, int m, bool first, double s1,
                                          bool done) {
    constexpr bool CX = std::is_same<XS, double2>::value;
    const unsigned n = unsigned(nd);
    for (unsigned i = threadIdx.x; i < n; i += blockDim.x) {
        double v[M];
#pragma unroll
        for (int j = 0; j < M; ++j)
            if (j < m) v[j] = ld(ring + j * nd, i);
        double2 pv{0.0, 0.0};
        double xr = 0.0, xi = 0.0;
        if (first) {
            v[0] *= s1;
        } else {
            pv = ld(p, i);
            if constexpr (CX) {
                const double2 t = ld(x, i);
                xr = t.x;
                xi = t.y;
            } else {
                xr = ld(x, i);
            }
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            if (j < m) {
                asm volatile("" ::: "memory");
                const Coef c = coef[j];
                const double pr = v[j] - c.lr * pv.x + c.li * pv.y;
                pv.y = -c.lr * pv.y - c.li * pv.x;
                pv.x = pr;
                xr += c.er * pv.x - c.ei * pv.y;
                if constexpr (CX) xi += c.er * pv.y + c.ei * pv.x;
            }
        }
        if constexpr (CX) st(x, i, double2{xr, xi});
        else st(x, i, xr);
        if (!done) st(p, i, pv);
    }
}

// RAG: C does not divide n1.
template <typename XS, int C, int Z, int BSMAX, bool RAG>
__global__ __attribute__((amdgpu_flat_work_group_size(64, BSMAX)))
void rcocg_wg(Args a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* red = reinterpret_cast<double*>(smem_raw);                 // 16 waves x 3
    Coef* coef = reinterpret_cast<Coef*>(smem_raw + 16 * 3 * sizeof(double));
    int* next = reinterpret_cast<int*>(coef + kRingLong);
    double* planes = reinterpret_cast<double*>(coef + kRingLong) + 2;
    double* delay = planes + a.nbuf * Z * (a.n1 + 11 + C) * a.rs;
    const int tid = threadIdx.x, BS = blockDim.x;
    const Rows<C> rw = make_rows<C, RAG>(a.n0, a.n1);
    {   // ghost entries outside an isolated box read zero
        const int nent = a.nbuf * Z * (a.n1 + 11 + C) * a.rs;
        for (int e = tid; e < nent; e += BS) planes[e] = 0.0;
    }
    double* ring = a.pool + int64_t(blockIdx.x) * (a.ring + kSlotExtra) * a.nd;
    double* w = ring + a.ring * a.nd;
    double2* p = reinterpret_cast<double2*>(w + a.nd);
    double Q[12 + Z][C];
    for (;;) {
        global_barrier();           // slot and LDS free for the next system
        if (tid == 0) *next = atomicAdd(a.counter, 1);
        lds_barrier();
        const int pos = __builtin_amdgcn_readfirstlane(*next);
        if (pos >= a.nsys) break;
        const int sys = a.order[pos];
        const double omega = a.omega_v[sys / a.ns];
        const double diag = a.cw[0] - a.eps[sys % a.ns];
        const double* b = a.rhs + int64_t(sys) * a.nd;
        XS* x = reinterpret_cast<XS*>(a.x) + int64_t(sys) * a.nd;
        Recurrence rc(omega, a);
        int slot = 0;                                 // rc.it mod ring
        bool px_first = true, carry = false, redo = false;
        while (!rc.done) {
            const bool first = rc.it == 0;
            double* vnew = ring + slot * a.nd;
            const double* vold = first ? b : ring + ((slot ? slot : a.ring) - 1) * a.nd;
            // v_k = (w - delta v_{k-1}) / beta; v_1 stays unnormalised (rc.sc carries its norm): the
            // first sweep reads b itself.  A repeated sweep reads the stored v_k.
            const bool plain = first || redo;
            const double c1 = plain ? 1.0 : rc.sc * rc.ibeta;
            const double c2 = plain ? 0.0 : -rc.delta * rc.sc * rc.ibeta;
            double acc[3] = {0.0, 0.0, 0.0};
            sweep<C, Z, RAG>(a, rw, planes, diag - rc.sigma, redo ? vnew : (first ? b : w), vold, c1,
                             c2, rc.cp(), vnew, w, Q, carry, acc, delay);
            if (RAG) global_barrier();           // w of rows that other threads stored
            wg_reduce<3>(acc, red);
            if (!rc.norms(acc)) break;           // zero or too small a right-hand side
            if (rc.cancels(acc) && !redo) {
                // cancellation: once more with sigma = alpha
                rc.shift(acc);
                carry = false;
#pragma unroll
                for (int q = 0; q < 12 + Z; ++q)
#pragma unroll
                    for (int i = 0; i < C; ++i) Q[q][i] = 0.0;
                redo = true;
                continue;
            }
            redo = false;
            carry = a.periodic != 0;
            const Coef cf = rc.step(acc);
            if (tid == 0) coef[slot] = cf;
            const int m = ++slot;                     // basis vectors not yet in x
            if (slot == a.ring) slot = 0;
            if (rc.done || slot == 0) {
                global_barrier();
                update_px<XS, kRingLong>(a.nd, ring, p, x, coef, m, px_first, rc.ibn, rc.done);
                px_first = false;
                carry = false;              // the queue's registers are free for the update
#pragma unroll
                for (int q = 0; q < 12 + Z; ++q)
#pragma unroll
                    for (int i = 0; i < C; ++i) Q[q][i] = 0.0;
                global_barrier();
            }
        }
        if (rc.it == 0) {
            // nothing solved: x = 0 (not a number where b is not finite)
            for (unsigned i = tid; i < unsigned(a.nd); i += BS) {
                const double v = 0.0 * ld(b, i);
                if constexpr (std::is_same<XS, double>::value) st(x, i, v);
                else st(x, i, double2{v, 0.0});
            }
        }
        if (tid == 0) {
            a.iters[sys] = rc.it;
            a.status[sys] = rc.stat;
            if (a.refinements) a.refinements[sys] = 0;
        }
    }
}

// ---------------------------------------------------------------- exact residual
// r = b - (H - eps_n - i omega) x of a finished solve with complex solutions, in float64, one
// system per workgroup: the real and the imaginary part of x are marched one after the other on
// the solver's planes (the second finds x in the caches).  Norms mode (rout null): status 0
// becomes 1 where |r| > tol |b|, refinements is 1, b2 = |b|^2.  Else r is stored, interleaved.
// 48^3, 16384 systems: 23 ms beside 339 for the shortest solves (21 iterations); plain gathers of
// the 37 points took 60.
struct CheckArgs {
    int n0, n1, n2, P;
    double cw[7];
    const double *vloc, *eps, *omega_v, *rhs;
    int ns;
    const int* order;      // null: system = block
    const double2* x;
    double2* rout;
    double tol2;
    int64_t nd;
    int *status, *refinements;
    double* b2;
    int nbuf, rs, periodic;
};

template <int C, int BSMAX, bool RAG>
__global__ __attribute__((amdgpu_flat_work_group_size(64, BSMAX))) void check_wg(CheckArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* red = reinterpret_cast<double*>(smem_raw);                 // 16 waves x 3
    double* planes = red + 48;
    const int sys = a.order ? a.order[blockIdx.x] : int(blockIdx.x);
    const int n0 = a.n0, n1 = a.n1, n2 = a.n2, P = a.P, rs = a.rs;
    const int PL = (n1 + 11 + C) * rs;
    const bool per = a.periodic != 0;
    const double om = a.omega_v[sys / a.ns], diag = a.cw[0] - a.eps[sys % a.ns];
    const double* x = reinterpret_cast<const double*>(a.x + int64_t(sys) * a.nd);
    const double* b = a.rhs + int64_t(sys) * a.nd;
    double* rout = a.rout ? reinterpret_cast<double*>(a.rout + int64_t(sys) * a.nd) : nullptr;
    const Rows<C> rw = make_rows<C, RAG>(n0, n1);
    for (int e = threadIdx.x; e < a.nbuf * PL; e += blockDim.x) planes[e] = 0.0;
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int part = 0; part < 2; ++part) {
        lds_barrier();
        const double* xp = x + part;                 // the marched part, stride 2
        const double* xo = x + 1 - part;             // the other one
        const double so = part == 0 ? om : -om;
        double Q[13][C];
#pragma unroll
        for (int s = 0; s < 13; ++s) {
            const int zu = s - 6, z = zu < 0 ? zu + n2 : zu;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                Q[s][i] = 0.0;
                if (per || zu >= 0) Q[s][i] = ld(xp + 2 * z * P, 2 * rw.col[i]);
                if (RAG && !per && !rw.own_[i]) Q[s][i] = 0.0;
            }
        }
#pragma unroll 1
        for (int z = 0; z < n2; ++z) {
            double nx[C], V[C], xc[C], bv[C];
            const int zn = z + 7;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                nx[i] = 0.0;
                if (per || zn < n2) nx[i] = ld(xp + 2 * (zn < n2 ? zn : zn - n2) * P, 2 * rw.col[i]);
                if (RAG && !per && !rw.own_[i]) nx[i] = 0.0;
                V[i] = ld(a.vloc + z * P, rw.col[i]);
                xc[i] = ld(xo + 2 * z * P, 2 * rw.col[i]);
                bv[i] = part == 0 ? ld(b + z * P, rw.col[i]) : 0.0;
            }
            double* L = planes + (a.nbuf == 2 ? (z & 1) : 0) * PL;
#pragma unroll
            for (int i = 0; i < C; ++i)
                if (rw.template own<RAG>(i))
                    cocg::stage_point(L, rs, n0, n1, rw.cx, rw.y0 + i, Q[6][i], per, true);
            lds_barrier();
            double s[C];
#pragma unroll
            for (int i = 0; i < C; ++i) s[i] = (diag + V[i]) * Q[6][i] + so * xc[i];
            stencil<13, C>(a.cw, L + cocg::lds_center(rs, rw.cx, rw.y0), rs, Q, 6, s);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                if (!rw.template own<RAG>(i)) continue;
                const double r = bv[i] - s[i];
                acc[0] += r * r;
                acc[1] += bv[i] * bv[i];
                if (rout) st(rout + part + 2 * z * P, 2 * rw.col[i], r);
            }
            if (a.nbuf == 1) lds_barrier();
#pragma unroll
            for (int q = 0; q < 12; ++q)
#pragma unroll
                for (int i = 0; i < C; ++i) Q[q][i] = Q[q + 1][i];
#pragma unroll
            for (int i = 0; i < C; ++i) Q[12][i] = nx[i];
        }
    }
    if (rout) return;
    wg_reduce<3>(acc, red);
    if (threadIdx.x == 0) {
        if (a.status[sys] == 0 && !(acc[0] <= a.tol2 * acc[1]) && !too_small(acc[1], a.tol2))
            a.status[sys] = 1;
        if (a.refinements) a.refinements[sys] = 1;
        a.b2[sys] = acc[1];
    }
}

}  // namespace rcocg
}  // namespace rpa
