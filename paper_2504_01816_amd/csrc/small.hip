// Small dense FP64 kernels of the subspace step (Algorithm 1) and the pointwise epilogues.
//  * Cholesky of the N_r x N_r overlap M = R^T R and T = L^{-T}, so V = R T (orthonormalisation)
//  * E_{c,m} = W/(2 pi) sum_k g(mu_k) through sum_k g(mu_k) = ln det(I - C) + tr C, with
//    I - C symmetric positive definite because C <= 0 (Eq. 10)
//  * eigenvalues of C (Householder tridiagonal form and bisection) for the Ritz values, cyclic
//    Jacobi where the vectors are needed too
//  * Delta rho = 4 sum_n psi_n Re(x_n) (Eq. 8) and the gradient accumulation
// N_r is at most a few hundred, so these are latency-bound: what counts is the number of
// barriers and launches.
#include <algorithm>

#include "internal.h"

namespace rpa {
namespace {

constexpr int SB = 1024;

__device__ double block_sum(double v, double* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += red[w];
    __syncthreads();
    return s;
}

// ------------------------------------------------------------------ Cholesky
// One workgroup of 16 waves, right-looking in panels of 16 columns.  The diagonal block is
// factorised by one wave in registers (lane i holds row i, the pivot row comes by readlane: no
// barrier inside), the panel rows are solved one per thread against it, and the trailing matrix
// is updated in 4 x 4 register tiles from an LDS copy of the panel: three barriers per 16
// columns.  The column-by-column forms that this replaces (three barriers per column in LDS, a
// serial dot product per element in global memory) took 50 us at m = 64 and 3.67 ms at m = 256
// for I - C.
constexpr int NB = 16;

// Broadcast of a double from a lane known at compile time.
__device__ __forceinline__ double lane_of(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(int(b), l);
    const int hi = __builtin_amdgcn_readlane(int(b >> 32), l);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// Factor of the block A[k0 .. k0+nb) in place and into D (column-major, stride NB + 1, padded with
// the identity); inv[j] = 1 / D[j][j].  One wave.
__device__ __forceinline__ void chol_diag(int nb, double* A, int64_t ld, int k0, double* D,
                                          double* inv, int* sflag) {
    const int i = threadIdx.x & 63;
    double a[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
        a[j] = (i < nb && j < nb && i >= j) ? A[(k0 + i) + ld * (k0 + j)] : (i == j ? 1.0 : 0.0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const double d = lane_of(a[j], j);
        const bool ok = d > 0.0;
        if (!ok && i == 0 && *sflag == 0) *sflag = k0 + j + 1;
        // 1 / sqrt(d) by two Newton steps on the hardware estimate, s = sqrt(d) corrected once
        double r = __builtin_amdgcn_rsq(ok ? d : 1.0), s = (ok ? d : 1.0);
        r = fma(0.5 * r, fma(-s * r, r, 1.0), r);
        r = fma(0.5 * r, fma(-s * r, r, 1.0), r);
        const double t = s * r;
        s = fma(0.5 * r, fma(-t, t, s), t);
        a[j] = (i == j) ? s : a[j] * r;
        if (i == j) inv[j] = r;
#pragma unroll
        for (int k = j + 1; k < NB; ++k) a[k] -= a[j] * lane_of(a[j], k);
    }
    if (i < NB) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const double v = i >= j ? a[j] : 0.0;
            D[i + (NB + 1) * j] = v;
            if (i < nb && j < nb && i >= j) A[(k0 + i) + ld * (k0 + j)] = v;
        }
    }
}

// Lower Cholesky factor of A (m x m, leading dimension ld, LDS or global memory) in place; the
// upper triangle is not touched.  P: LDS, NB * m doubles for a copy of the panel;
// null: the panel is read from A.  DI (global, m x m, or null) receives the
// inverses of the diagonal blocks, transposed, at its own diagonal blocks.
__device__ __forceinline__ void chol_blocked(int m, double* A, int64_t ld, double* P, double* D, double* inv,
                             int* sflag, double* DI) {
    const int tid = threadIdx.x, bs = blockDim.x;
    for (int k0 = 0; k0 < m; k0 += NB) {
        const int nb = min(NB, m - k0), r0 = k0 + nb, n = m - r0;
        if (tid < 64) chol_diag(nb, A, ld, k0, D, inv, sflag);
        __syncthreads();
        if (DI && tid >= bs - 64 && tid < bs - 64 + NB) {
            // column c of the inverse of the diagonal block, by the last wave
            const int c = tid - (bs - 64);
            double x[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                double t = (i == c) ? 1.0 : 0.0;
#pragma unroll
                for (int k = 0; k < i; ++k) t -= D[i + (NB + 1) * k] * x[k];
                x[i] = t * inv[i];
                asm volatile("" : "+v"(x[i])::"memory");   // one row's LDS reads at a time
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (i < nb && c < nb) DI[(k0 + c) + int64_t(m) * (k0 + i)] = x[i];
        }
        for (int r = tid; r < n; r += bs) {
            double x[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) x[j] = (j < nb) ? A[(r0 + r) + ld * (k0 + j)] : 0.0;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int k = 0; k < j; ++k) x[j] -= x[k] * D[j + (NB + 1) * k];
                x[j] *= inv[j];
                asm volatile("" : "+v"(x[j])::"memory");   // one row's LDS reads at a time
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (j < nb) A[(r0 + r) + ld * (k0 + j)] = x[j];
                if (P) P[r + int64_t(m) * j] = x[j];
            }
        }
        __syncthreads();
        if (n > 0) {
            // 4 x 4 tiles of the trailing lower triangle
            const int nt = (n + 3) / 4;
            const double* Q = P ? P : A + r0 + ld * k0;
            const int64_t qs = P ? m : ld;
            for (int e = tid; e < nt * nt; e += bs) {
                const int ti = e % nt, tj = e / nt;
                if (ti < tj) continue;
                double c[4][4] = {};
                int ri[4], rj[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ri[q] = min(4 * ti + q, n - 1);
                    rj[q] = min(4 * tj + q, n - 1);
                }
                for (int k = 0; k < nb; ++k) {
                    double x[4], y[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        x[q] = Q[ri[q] + qs * k];
                        y[q] = Q[rj[q] + qs * k];
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p)
#pragma unroll
                        for (int q = 0; q < 4; ++q) c[p][q] += x[p] * y[q];
                }
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int i = 4 * ti + p, j = 4 * tj + q;
                        if (i < n && j < n && i >= j) A[(r0 + i) + ld * (r0 + j)] -= c[p][q];
                    }
            }
        }
        __syncthreads();
    }
}

// LDS of the Cholesky kernels: D, inv, and then the matrix (m <= kCholLds) or the panel.
constexpr int kCholLds = 120;       // 120 x 121 doubles: 116 KB
constexpr int kCholPanel = 1024;    // largest m whose panel is kept in LDS (128 KB)
constexpr int kCholFix = (NB * (NB + 1) + NB) * int(sizeof(double));

size_t chol_lds(int m) {
    if (m <= kCholLds) return kCholFix + size_t(m) * (m + 1) * sizeof(double);
    return kCholFix + (m <= kCholPanel ? size_t(m) * NB * sizeof(double) : 0);
}

// M -> L (lower, the rest zero) and the transposed inverses of L's diagonal blocks at the diagonal
// blocks of T.
// One matrix per workgroup: matrix at.f[blockIdx.x] of arrays of m x m matrices, with its info 8
// entries on.  One launch per matrix took 19.4 us each at m = 32, 8 frequencies one after another;
// all 8 in one launch take 22.
__global__ __launch_bounds__(SB) void chol_kernel(int m, const double* M, double* L, double* T,
                                                  int* info, MatrixList at) {
    extern __shared__ double sh[];
    {
        const int f = at.f[blockIdx.x];
        const int64_t o = int64_t(f) * m * m;
        M += o;
        L += o;
        T += o;
        info += 8 * f;
    }
    __shared__ int sflag;
    double* D = sh;
    double* inv = sh + NB * (NB + 1);
    double* W = inv + NB;
    const int tid = threadIdx.x, bs = blockDim.x;
    const bool in_lds = m <= kCholLds;
    double* A = in_lds ? W : L;
    const int64_t ld = in_lds ? m + 1 : m;
    for (int e = tid; e < m * m; e += bs) {
        const int r = e % m, c = e / m;
        A[r + ld * c] = (r >= c) ? M[e] : 0.0;
    }
    if (tid == 0) sflag = 0;
    __syncthreads();
    if (in_lds) chol_blocked(m, W, m + 1, nullptr, D, inv, &sflag, T);
    else chol_blocked(m, L, m, m > kCholPanel ? nullptr : W, D, inv, &sflag, T);
    if (in_lds)
        for (int e = tid; e < m * m; e += bs) L[e] = A[e % m + ld * (e / m)];
    if (tid == 0) *info = sflag;
}

// T = L^{-T}, NB rows of T (columns c0 .. of X = L^{-1}) per workgroup, block row by block row:
// X_i = D_i (I_i - sum_{k < i} L_ik X_k) with the diagonal inverses D_i that chol_kernel left
// (transposed) in T.  T[c + m i] = X[i][c].
__global__ __launch_bounds__(NB * NB) void tri_inv_kernel(int m, const double* L, double* T,
                                                          MatrixList at) {
    L += int64_t(at.f[blockIdx.y]) * m * m;
    T += int64_t(at.f[blockIdx.y]) * m * m;
    __shared__ double Rs[NB][NB + 1];
    const int c0 = blockIdx.x * NB, tid = threadIdx.x;
    const int c = tid & (NB - 1), i = tid / NB;          // one output of a block row per thread
    const bool cin = c0 + c < m;
    for (int r = tid; r < NB * c0; r += NB * NB) {            // rows above the block are zero
        const int cc = r % NB, ii = r / NB;
        if (c0 + cc < m) T[(c0 + cc) + int64_t(m) * ii] = 0.0;
    }
    for (int i0 = c0 + NB; i0 < m; i0 += NB) {
        const int gi = i0 + i;
        double s = 0.0;
        __syncthreads();                                 // the rows written so far are visible
        if (gi < m && cin)
            for (int k = c0; k < i0; ++k) s -= L[gi + int64_t(m) * k] * T[(c0 + c) + int64_t(m) * k];
        Rs[i][c] = s;
        __syncthreads();
        if (gi < m && cin) {
            double x = 0.0;
            for (int k = 0; k <= i; ++k) x += T[(i0 + k) + int64_t(m) * gi] * Rs[k][c];
            // the block row's own diagonal block is read above and never written here
            T[(c0 + c) + int64_t(m) * gi] = x;
        }
    }
}

// E = scale (ln det(I - C) + tr C) through the Cholesky factor of I - C, one matrix per workgroup (as
// chol_kernel; out is 8 entries apart).
__global__ __launch_bounds__(SB) void energy_kernel(int m, const double* C, double* work, double* out,
                                                    int* info, MatrixList at) {
    extern __shared__ double sh[];
    const double scale = at.scale[blockIdx.x];
    {
        const int f = at.f[blockIdx.x];
        C += int64_t(f) * m * m;
        out += 8 * f;
        info += 8 * f;
    }
    __shared__ int sflag;
    __shared__ double red[SB / 64];
    double* D = sh;
    double* inv = sh + NB * (NB + 1);
    double* W = inv + NB;
    const int tid = threadIdx.x, bs = blockDim.x;
    const bool in_lds = m <= kCholLds;
    double* A = in_lds ? W : work;
    const int64_t ld = in_lds ? m + 1 : m;
    for (int e = tid; e < m * m; e += bs) {
        const int r = e % m, c = e / m;
        A[r + ld * c] = (r >= c) ? ((r == c ? 1.0 : 0.0) - C[e]) : 0.0;
    }
    if (tid == 0) sflag = 0;
    __syncthreads();
    if (in_lds) chol_blocked(m, W, m + 1, nullptr, D, inv, &sflag, nullptr);
    else chol_blocked(m, work, m, m > kCholPanel ? nullptr : W, D, inv, &sflag, nullptr);
    double v = 0.0;
    for (int i = tid; i < m; i += bs) v += 2.0 * log(A[i + ld * i]) + C[i + int64_t(m) * i];
    const double sum = block_sum(v, red);
    if (tid == 0) {
        out[0] = scale * sum;
        *info = sflag;
    }
}

__global__ void symmetrize_kernel(int m, double* C) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m * m) return;
    const int r = i % m, c = i / m;
    if (r < c) {
        const double a = C[r + int64_t(m) * c], b = C[c + int64_t(m) * r];
        const double s = 0.5 * (a + b);
        C[r + int64_t(m) * c] = s;
        C[c + int64_t(m) * r] = s;
    }
}

// Cyclic Jacobi with the round-robin ordering: each step rotates m/2 disjoint pairs at once,
// A <- J^T A J in 2 x 2 blocks (pair of rows times pair of columns, one thread each) and
// Y <- Y J: two barriers per step.  A (overwritten by its eigenvalues' diagonal) and Y have
// leading dimension ld; cs: 2 np doubles and 2 np ints of LDS; red: SB / 64 doubles.
__device__ __forceinline__ void jacobi(int m, double* A, double* Y, int ld, double* cs,
                                       double* red) {
    const int tid = threadIdx.x, bs = blockDim.x;
    const int mm = m + (m & 1), np = mm / 2;
    int* pp = reinterpret_cast<int*>(cs + 2 * np);
    double fro = 0.0;
    for (int i = tid; i < m * m; i += bs) {
        const double t = A[i % m + ld * (i / m)];
        fro += t * t;
    }
    fro = block_sum(fro, red);
    for (int sweep = 0; sweep < 60; ++sweep) {
        double off = 0.0;
        for (int i = tid; i < m * m; i += bs)
            if (i % m != i / m) {
                const double t = A[i % m + ld * (i / m)];
                off += t * t;
            }
        off = block_sum(off, red);
        if (!(off > 1e-30 * fro) || fro == 0.0) break;
        for (int t = 0; t < mm - 1; ++t) {
            for (int k = tid; k < np; k += bs) {
                const int a0 = (k == 0) ? 0 : ((k - 1 + t) % (mm - 1)) + 1;
                const int k2 = mm - 1 - k;
                const int b0 = ((k2 - 1 + t) % (mm - 1)) + 1;
                const int p = min(a0, b0), q = max(a0, b0);
                double c = 1.0, s = 0.0;
                if (q < m) {
                    const double apq = A[p + ld * q];
                    if (apq != 0.0) {
                        const double app = A[p + ld * p], aqq = A[q + ld * q];
                        const double tau = (aqq - app) / (2.0 * apq);
                        const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        c = 1.0 / sqrt(1.0 + tt * tt);
                        s = tt * c;
                    }
                }
                cs[2 * k] = c;
                cs[2 * k + 1] = s;
                pp[2 * k] = p;
                pp[2 * k + 1] = q;               // m (odd sizes): the row without a partner
            }
            __syncthreads();
            for (int it = tid; it < np * np; it += bs) {
                const int k = it % np, l = it / np;
                const int p = pp[2 * k], q = pp[2 * k + 1], r = pp[2 * l], u = pp[2 * l + 1];
                const double c = cs[2 * k], s = cs[2 * k + 1], d = cs[2 * l], e = cs[2 * l + 1];
                const bool hq = q < m, hu = u < m;
                const double apr = A[p + ld * r], apu = hu ? A[p + ld * u] : 0.0;
                const double aqr = hq ? A[q + ld * r] : 0.0, aqu = hq && hu ? A[q + ld * u] : 0.0;
                const double xr = c * apr - s * aqr, xu = c * apu - s * aqu;
                const double yr = s * apr + c * aqr, yu = s * apu + c * aqu;
                A[p + ld * r] = d * xr - e * xu;
                if (hu) A[p + ld * u] = e * xr + d * xu;
                if (hq) A[q + ld * r] = d * yr - e * yu;
                if (hq && hu) A[q + ld * u] = e * yr + d * yu;
            }
            for (int it = tid; it < np * m; it += bs) {
                const int k = it / m, row = it % m;
                const int p = pp[2 * k], q = pp[2 * k + 1];
                if (q >= m) continue;
                const double c = cs[2 * k], s = cs[2 * k + 1];
                const double ap = Y[row + ld * p], aq = Y[row + ld * q];
                Y[row + ld * p] = c * ap - s * aq;
                Y[row + ld * q] = s * ap + c * aq;
            }
            __syncthreads();
        }
    }
}

// Largest m whose A and Y the Jacobi kernels keep in LDS, with an odd stride: 2 x 88 x 89 doubles.
constexpr int kJacobiLds = 88;

__global__ __launch_bounds__(SB) void syevj_kernel(int m, const double* Ain, double* work,
                                                   double* w, double* Yout) {
    extern __shared__ double sh[];
    __shared__ double red[SB / 64];
    const int tid = threadIdx.x, bs = blockDim.x, np = (m + 1) / 2;
    const bool in_lds = m <= kJacobiLds;
    const int ld = in_lds ? m | 1 : m;
    double* A = in_lds ? sh + 3 * np : work;
    double* Y = A + int64_t(ld) * m;
    for (int i = tid; i < m * m; i += bs) {
        const int r = i % m, c = i / m;
        A[r + ld * c] = 0.5 * (Ain[i] + Ain[c + int64_t(m) * r]);
        Y[r + ld * c] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
    if (in_lds) jacobi(m, sh + 3 * np, sh + 3 * np + ld * m, ld, sh, red);
    else jacobi(m, work, work + int64_t(m) * m, m, sh, red);
    // sort ascending (stable by index)
    for (int i = tid; i < m; i += bs) {
        const double di = A[i + int64_t(ld) * i];
        int rank = 0;
        for (int j = 0; j < m; ++j) {
            const double dj = A[j + int64_t(ld) * j];
            rank += (dj < di) || (dj == di && j < i);
        }
        w[rank] = di;
        for (int r = 0; r < m; ++r) Yout[r + int64_t(m) * rank] = Y[r + int64_t(ld) * i];
    }
}

// Eigenbases of -D2 on the three axes of an isolated box, one workgroup per axis and parity.
// The matrix (banded Toeplitz of the weights, reaches beyond the walls dropped) is symmetric
// about its centre too, so its eigenvectors are even or odd there: with n = 2 h (+ 1) the even
// ones solve a problem of size h (+ 1), the odd ones one of size h, and each half-size Jacobi
// takes half the steps.  U[t + n a], kappa[a]: the even modes first, each parity in Jacobi order.
// 48^3: three Jacobi kernels of n = 48 one after another took 4.5 ms.
constexpr int kBoxLds = 2 * kJacobiLds - 1;

struct BoxAxes {
    int n[3];
    double* U[3];
    double* kappa[3];
    double ih2;
    double w[7];
};

__global__ __launch_bounds__(SB) void box_basis_kernel(BoxAxes ax) {
    extern __shared__ double sh[];
    __shared__ double red[SB / 64];
    const int tid = threadIdx.x, axis = blockIdx.x >> 1;
    const bool odd = blockIdx.x & 1;
    const int n = ax.n[axis], h = n / 2, m = odd ? h : n - h, ld = m | 1;
    const int np = (m + 1) / 2, mid = n - h - 1;           // the centre point, if n is odd
    double* A = sh + 3 * np;
    double* Y = A + ld * m;
    auto t = [&](int i, int j) {
        const int d = i > j ? i - j : j - i;
        return d <= 6 ? -ax.w[d] * ax.ih2 : 0.0;
    };
    for (int e = tid; e < m * m; e += SB) {
        const int r = e % m, c = e / m;
        // points r and n - 1 - r combined: T(r, c) +- T(r, n - 1 - c), the centre scaled by sqrt 2
        const bool cr = 2 * r + 1 == n, cc = 2 * c + 1 == n;
        double v = cr && cc ? t(r, c) : cr || cc ? sqrt(2.0) * t(r, c)
                                                 : t(r, c) + (odd ? -1.0 : 1.0) * t(r, n - 1 - c);
        A[r + ld * c] = v;
        Y[r + ld * c] = r == c ? 1.0 : 0.0;
    }
    __syncthreads();
    jacobi(m, A, Y, ld, sh, red);
    const int a0 = odd ? n - h : 0;
    for (int a = tid; a < m; a += SB) ax.kappa[axis][a0 + a] = A[a + ld * a];
    for (int e = tid; e < m * n; e += SB) {
        const int i = e % n, a = e / n;
        const bool up = i > mid;                           // mirrored half
        const int r = up ? n - 1 - i : i;
        double v = 0.0;
        if (r < m) v = (2 * r + 1 == n ? 1.0 : sqrt(0.5)) * Y[r + ld * a];
        ax.U[axis][i + int64_t(n) * (a0 + a)] = (up && odd) ? -v : v;
    }
}

// ------------------------------------------------------------------ eigenvalues alone
// Householder tridiagonalisation and bisection with Sturm counts.  The Jacobi iteration above
// rotates a matrix of m = 256 in L2 from one workgroup for 260 ms (m = 64: 3.5 ms).  Up to
// kTriLds the matrix stays in the LDS of one workgroup (two barriers per column); beyond, one
// launch per column applies the previous reflector to the columns of each workgroup and
// multiplies the updated columns with the next one.
constexpr int kTriLds = 120;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Reflector of x (x0 = alpha, the rest with sum of squares sig): beta, tau and the factor of
// x_i in v_i (v_0 = 1).
__device__ __forceinline__ void reflector(double alpha, double sig, double* beta, double* tau,
                                          double* f) {
    if (sig == 0.0) {
        *beta = alpha;
        *tau = 0.0;
        *f = 0.0;
    } else {
        const double b = sqrt(alpha * alpha + sig);
        *beta = alpha <= 0.0 ? b : -b;
        *tau = (*beta - alpha) / *beta;
        *f = 1.0 / (alpha - *beta);
    }
}

// Eigenvalues [first + lane group] of the tridiagonal (d, e2 = e^2, LDS): eight lanes per
// eigenvalue count at eight inner points of its bracket at once (9 brackets per round).
// Every lane of the group returns the eigenvalue.
__device__ double bisect(int m, const double* d, const double* e2, int t, double lo, double hi,
                         double pivmin) {
    const int l = threadIdx.x & 7, g = threadIdx.x & 56;
    for (int round = 0; round < 20; ++round) {
        const double x = lo + (hi - lo) * (double(l + 1) / 9.0);
        int cnt = 0;
        double q = d[0] - x;
        for (int i = 0;;) {
            if (fabs(q) < pivmin) q = -pivmin;
            cnt += q < 0.0;
            if (++i == m) break;
            double r = __builtin_amdgcn_rcp(q);            // two Newton steps: full precision
            r = fma(fma(-q, r, 1.0), r, r);
            r = fma(fma(-q, r, 1.0), r, r);
            q = d[i] - x - e2[i - 1] * r;
        }
        const unsigned long long below = __ballot(cnt <= t);
        const int c = __popcll((below >> g) & 0xffull);
        const double nlo = __shfl(x, g + (c > 0 ? c - 1 : 0), 64);
        const double nhi = __shfl(x, g + (c < 8 ? c : 7), 64);
        if (c > 0) lo = nlo;
        if (c < 8) hi = nhi;
    }
    return 0.5 * (lo + hi);
}

// Gershgorin bracket of the tridiagonal, over the block; red: LDS, 48 doubles.
__device__ void bracket(int m, const double* d, const double* e, double* red, double* lo,
                        double* hi, double* pivmin) {
    double a = INFINITY, b = -INFINITY, c = 0.0;
    for (int i = threadIdx.x; i < m; i += blockDim.x) {
        const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i < m - 1 ? fabs(e[i]) : 0.0);
        a = fmin(a, d[i] - r);
        b = fmax(b, d[i] + r);
        c = fmax(c, i < m - 1 ? e[i] * e[i] : 0.0);
    }
    for (int o = 32; o > 0; o >>= 1) {
        a = fmin(a, __shfl_xor(a, o, 64));
        b = fmax(b, __shfl_xor(b, o, 64));
        c = fmax(c, __shfl_xor(c, o, 64));
    }
    const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[w] = a;
        red[16 + w] = b;
        red[32 + w] = c;
    }
    __syncthreads();
    for (int i = 0; i < nw; ++i) {
        a = fmin(a, red[i]);
        b = fmax(b, red[16 + i]);
        c = fmax(c, red[32 + i]);
    }
    const double n = fmax(fabs(a), fabs(b));
    *lo = a - 1e-15 * n;
    *hi = b + 1e-15 * n;
    *pivmin = fmax(2.3e-308, 2.3e-308 * c);
}

__global__ __launch_bounds__(SB) void syev_lds_kernel(int m, const double* Ain, double* w) {
    extern __shared__ double sh[];
    __shared__ double red[48];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ld = m + 1;
    double* A = sh;
    double* p = A + m * ld;
    double* d = p + m;
    double* e = d + m;
    for (int i = tid; i < m * m; i += SB) {
        const int r = i % m, c = i / m;
        A[r + ld * c] = 0.5 * (Ain[i] + Ain[c + int64_t(m) * r]);
    }
    __syncthreads();
    for (int k = 0; k < m; ++k) {
        const int n = m - k - 1;                    // rows below the diagonal, two per lane
        if (tid == 0) d[k] = A[k + ld * k];
        if (n == 0) break;
        const double* x = A + (k + 1) + ld * k;
        const double x0 = lane < n ? x[lane] : 0.0, x1 = lane + 64 < n ? x[lane + 64] : 0.0;
        const double sig = wave_sum((lane > 0 ? x0 * x0 : 0.0) + x1 * x1);
        double beta, tau, f;
        reflector(__shfl(x0, 0, 64), sig, &beta, &tau, &f);
        const double v0 = lane == 0 ? 1.0 : x0 * f, v1 = x1 * f;
        if (tid == 0) e[k] = beta;
        double* B = A + (k + 1) + ld * (k + 1);     // trailing matrix
        for (int j = wave; j < n; j += SB / 64) {
            const double* b = B + ld * j;
            const double s = wave_sum((lane < n ? b[lane] * v0 : 0.0)
                                      + (lane + 64 < n ? b[lane + 64] * v1 : 0.0));
            if (lane == 0) p[j] = tau * s;
        }
        __syncthreads();
        double w0 = lane < n ? p[lane] : 0.0, w1 = lane + 64 < n ? p[lane + 64] : 0.0;
        const double h = 0.5 * tau * wave_sum(w0 * v0 + w1 * v1);
        w0 -= h * v0;
        w1 -= h * v1;
        for (int j = wave; j < n; j += SB / 64) {
            double* b = B + ld * j;
            const double vj = __shfl(j < 64 ? v0 : v1, j & 63, 64);
            const double wj = __shfl(j < 64 ? w0 : w1, j & 63, 64);
            if (lane < n) b[lane] -= v0 * wj + w0 * vj;
            if (lane + 64 < n) b[lane + 64] -= v1 * wj + w1 * vj;
        }
        __syncthreads();
    }
    __syncthreads();
    double lo, hi, piv;
    bracket(m, d, e, red, &lo, &hi, &piv);
    __syncthreads();
    for (int i = tid; i < m - 1; i += SB) e[i] *= e[i];
    __syncthreads();
    const int t = tid >> 3;                          // m <= 120 <= SB / 8
    const double ev = bisect(m, d, e, t < m ? t : m - 1, lo, hi, piv);
    if (t < m && (tid & 7) == 0) w[t] = ev;
}

// One column of the tridiagonalisation (see above).  st: two halves of 2 m + 2 doubles, used in
// turn: v (zero up to the column), p = tau A v, tau.
__global__ __launch_bounds__(256) void tri_step_kernel(int m, int k, double* A, double* st,
                                                       double* d, double* e) {
    extern __shared__ double sh[];
    __shared__ double red[8];
    double *v = sh, *w = sh + m, *u = sh + 2 * m;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = 2 * m + 2;
    const double* old = st + (k & 1) * half;
    double* out = st + ((k + 1) & 1) * half;
    auto total = [&](double t) {
        t = wave_sum(t);
        __syncthreads();
        if (lane == 0) red[wave] = t;
        __syncthreads();
        return red[0] + red[1] + red[2] + red[3];
    };
    // previous reflector: w = p - (tau / 2) (p.v) v on rows k ..
    double pv = 0.0;
    if (k > 0)
        for (int i = k + tid; i < m; i += 256) {
            v[i] = old[i];
            w[i] = old[m + i];
            pv += v[i] * w[i];
        }
    pv = total(pv);
    const double h = k > 0 ? 0.5 * old[2 * m] * pv : 0.0;
    if (k > 0)
        for (int i = k + tid; i < m; i += 256) w[i] -= h * v[i];
    __syncthreads();
    // column k, updated; its reflector
    double sig = 0.0;
    for (int i = k + tid; i < m; i += 256) {
        double x = A[i + int64_t(m) * k];
        if (k > 0) x -= v[i] * w[k] + w[i] * v[k];
        u[i] = x;
        if (i > k + 1) sig += x * x;
    }
    sig = total(sig);
    if (blockIdx.x == 0 && tid == 0) d[k] = u[k];
    if (k == m - 1) return;
    double beta, tau, f;
    reflector(u[k + 1], sig, &beta, &tau, &f);
    __syncthreads();
    for (int i = k + 1 + tid; i < m; i += 256) {
        u[i] = i == k + 1 ? 1.0 : u[i] * f;
        if (blockIdx.x == 0) out[i] = u[i];
    }
    if (blockIdx.x == 0 && tid == 0) {
        out[2 * m] = tau;
        e[k] = beta;
    }
    __syncthreads();
    // own columns: update, store, multiply
    for (int j = k + 1 + blockIdx.x * 4 + wave; j < m; j += gridDim.x * 4) {
        double* a = A + int64_t(m) * j;
        const double vj = k > 0 ? v[j] : 0.0, wj = k > 0 ? w[j] : 0.0;
        double s = 0.0;
        for (int i = k + 1 + lane; i < m; i += 64) {
            double x = a[i];
            if (k > 0) {
                x -= v[i] * wj + w[i] * vj;
                a[i] = x;
            }
            s += x * u[i];
        }
        s = wave_sum(s);
        if (lane == 0) out[m + j] = tau * s;
    }
}

__global__ void sym_copy_kernel(int m, const double* Ain, double* A) {
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i < int64_t(m) * m) A[i] = 0.5 * (Ain[i] + Ain[(i / m) + int64_t(m) * (i % m)]);
}

__global__ __launch_bounds__(64) void bisect_kernel(int m, const double* d, const double* e,
                                                    double* w) {
    extern __shared__ double sh[];
    __shared__ double red[48];
    for (int i = threadIdx.x; i < m; i += 64) {
        sh[i] = d[i];
        if (i < m - 1) sh[m + i] = e[i];
    }
    __syncthreads();
    double lo, hi, piv;
    bracket(m, sh, sh + m, red, &lo, &hi, &piv);
    __syncthreads();
    for (int i = threadIdx.x; i < m - 1; i += 64) sh[m + i] *= sh[m + i];
    __syncthreads();
    const int t = blockIdx.x * 8 + (threadIdx.x >> 3);
    const double ev = bisect(m, sh, sh + m, t < m ? t : m - 1, lo, hi, piv);
    if (t < m && (threadIdx.x & 7) == 0) w[t] = ev;
}

template <int STRIDE>
__global__ void drho_kernel(int64_t nd, int ns, const double* psi, const double* x, double* out) {
    const int64_t r = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    const int j = blockIdx.y;
    if (r >= nd) return;
    double s = 0.0;
    for (int n = 0; n < ns; ++n)
        s += psi[r + nd * n] * x[STRIDE * ((int64_t(n) + int64_t(ns) * j) * nd + r)];
    out[r + nd * j] = 4.0 * s;
}

// d[l, s] = coeff[l, s] / (eps_l - eps_n - i omega), s = n + ns k
__global__ void grad_d_kernel(int ns, int S, const double* eps, double omega, const double* coeff,
                              double2* d) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns * S) return;
    const int l = i % ns, s = i / ns, n = s % ns;
    const double a = eps[l] - eps[n], b = -omega;   // denominator a + i b
    const double den = a * a + b * b;
    const double c = coeff[i];
    d[i] = double2{c * a / den, -c * b / den};
}

template <typename T2, int NSMAX>
__global__ void grad_kernel(int64_t nd, int ns, int nvec, const double* psi, const double2* d,
                            const double* coefk, const T2* x, double* grad) {
    const int64_t r = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (r >= nd) return;
    double pr[NSMAX];
#pragma unroll
    for (int l = 0; l < NSMAX; ++l) pr[l] = (l < ns) ? psi[r + nd * l] : 0.0;
    double acc = 0.0;
    for (int k = 0; k < nvec; ++k) {
        double ak = 0.0;
        for (int n = 0; n < ns; ++n) {
            const int s = n + ns * k;
            double ore = 0.0, oim = 0.0;
#pragma unroll
            for (int l = 0; l < NSMAX; ++l) {
                if (l < ns) {
                    const double2 dl = d[l + int64_t(ns) * s];
                    ore -= pr[l] * dl.x;
                    oim -= pr[l] * dl.y;
                }
            }
            const T2 xv = x[int64_t(s) * nd + r];
            const double xr = double(xv.x), xi = double(xv.y);
            // Re[(x + o) x]
            ak += (xr + ore) * xr - (xi + oim) * xi;
        }
        acc += coefk[k] * 4.0 * ak;
    }
    grad[r] += acc;
}

__global__ void scale_kernel(int64_t n, double a, double* x) {
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i < n) x[i] *= a;
}
__global__ void fill_kernel(int64_t n, double v, double* x) {
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i < n) x[i] = v;
}
__global__ void copy_kernel(int64_t n, const double* src, double* dst) {
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// ------------------------------------------------------------------ Gauss spectral quadrature
// E = scale * sum_r sum_t Q_r(1,t)^2 g(lambda_t): for each standard basis vector e_r, n_o
// Lanczos steps on C give the tridiagonal J_r, whose eigenvalues (nodes) and squared first
// eigenvector components (weights) form the Gauss rule for e_r^T g(C) e_r (Sec. 3,
// Algorithm 1, SQ method).  One workgroup per r; the m x m matrix C is read once per step
// (coalesced along columns); Lanczos stops early when beta <= 1e-14 max|C| (exhausted Krylov
// space).  The small tridiagonal eigenproblem is solved by cyclic Jacobi on one wave.

__global__ __launch_bounds__(256) void absmax_kernel(int64_t n, const double* a, double* out) {
    __shared__ double red[4];
    double v = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) v = fmax(v, fabs(a[i]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int w = 0; w < int(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
        out[0] = m;
    }
}

constexpr int SQ_MAX = 32;   // largest quadrature order

__device__ double block_sum256(double v, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < 4; ++w) s += red[w];
    return s;
}

__global__ __launch_bounds__(256) void sq_lanczos_kernel(int m, const double* C, int n_o,
                                                         const double* cmax, double* part) {
    extern __shared__ double sh[];
    double* q = sh;             // m
    double* qp = sh + m;        // m
    double* w = sh + 2 * m;     // m
    __shared__ double red[4];
    __shared__ double A[SQ_MAX * SQ_MAX], Vv[SQ_MAX * SQ_MAX];
    __shared__ int kdim;
    const int r = blockIdx.x, tid = threadIdx.x;
    for (int i = tid; i < m; i += 256) {
        q[i] = (i == r) ? 1.0 : 0.0;
        qp[i] = 0.0;
    }
    for (int i = tid; i < SQ_MAX * SQ_MAX; i += 256) A[i] = 0.0;
    if (tid == 0) kdim = n_o;
    __syncthreads();
    const double tiny = 1e-14 * fmax(cmax[0], 1e-300);
    double beta = 0.0;
    for (int k = 0; k < n_o; ++k) {
        // w = C q - beta q_prev
        for (int i = tid; i < m; i += 256) {
            double s = 0.0;
            for (int j = 0; j < m; ++j) s += C[i + int64_t(m) * j] * q[j];
            w[i] = s - beta * qp[i];
        }
        __syncthreads();
        double pa = 0.0;
        for (int i = tid; i < m; i += 256) pa += q[i] * w[i];
        const double alpha = block_sum256(pa, red);
        for (int i = tid; i < m; i += 256) w[i] -= alpha * q[i];
        if (tid == 0) A[k + SQ_MAX * k] = alpha;
        __syncthreads();
        if (k == n_o - 1) break;
        double pb = 0.0;
        for (int i = tid; i < m; i += 256) pb += w[i] * w[i];
        beta = sqrt(block_sum256(pb, red));
        if (!(beta > tiny)) {
            if (tid == 0) kdim = k + 1;
            __syncthreads();
            break;
        }
        for (int i = tid; i < m; i += 256) {
            qp[i] = q[i];
            q[i] = w[i] / beta;
        }
        if (tid == 0) {
            A[k + 1 + SQ_MAX * k] = beta;
            A[k + SQ_MAX * (k + 1)] = beta;
        }
        __syncthreads();
    }
    __syncthreads();
    // cyclic Jacobi on the kdim x kdim tridiagonal (one thread; kdim <= 32)
    if (tid == 0) {
        const int n = kdim;
        for (int i = 0; i < n; ++i)
            for (int j = 0; j < n; ++j) Vv[i + SQ_MAX * j] = (i == j) ? 1.0 : 0.0;
        for (int sweep = 0; sweep < 100; ++sweep) {
            double off = 0.0, dia = 0.0;
            for (int i = 0; i < n; ++i) {
                dia += A[i + SQ_MAX * i] * A[i + SQ_MAX * i];
                for (int j = i + 1; j < n; ++j) off += A[i + SQ_MAX * j] * A[i + SQ_MAX * j];
            }
            if (!(off > 1e-30 * dia)) break;
            for (int p = 0; p < n - 1; ++p)
                for (int qq = p + 1; qq < n; ++qq) {
                    const double apq = A[p + SQ_MAX * qq];
                    if (apq == 0.0) continue;
                    const double app = A[p + SQ_MAX * p], aqq = A[qq + SQ_MAX * qq];
                    const double theta = (aqq - app) / (2.0 * apq);
                    const double t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                    const double c = 1.0 / sqrt(t * t + 1.0), sn = t * c;
                    for (int k = 0; k < n; ++k) {   // A <- A G (columns p, q)
                        const double akp = A[k + SQ_MAX * p], akq = A[k + SQ_MAX * qq];
                        A[k + SQ_MAX * p] = c * akp - sn * akq;
                        A[k + SQ_MAX * qq] = sn * akp + c * akq;
                    }
                    for (int k = 0; k < n; ++k) {   // A <- G^T A (rows p, q)
                        const double apk = A[p + SQ_MAX * k], aqk = A[qq + SQ_MAX * k];
                        A[p + SQ_MAX * k] = c * apk - sn * aqk;
                        A[qq + SQ_MAX * k] = sn * apk + c * aqk;
                    }
                    for (int k = 0; k < n; ++k) {   // V <- V G
                        const double vkp = Vv[k + SQ_MAX * p], vkq = Vv[k + SQ_MAX * qq];
                        Vv[k + SQ_MAX * p] = c * vkp - sn * vkq;
                        Vv[k + SQ_MAX * qq] = sn * vkp + c * vkq;
                    }
                }
        }
        double e = 0.0;
        for (int t = 0; t < n; ++t) {
            const double lam = A[t + SQ_MAX * t], q0 = Vv[0 + SQ_MAX * t];
            e += q0 * q0 * (log1p(-lam) + lam);
        }
        part[r] = e;
    }
}

// out[0] = scale * sum_r part[r] in a fixed order (deterministic); info[0] = 0, or 1 if the
// sum is not finite
__global__ __launch_bounds__(256) void sq_sum_kernel(int m, const double* part, double scale,
                                                     double* out, int* info) {
    __shared__ double red[4];
    double v = 0.0;
    for (int i = threadIdx.x; i < m; i += 256) v += part[i];
    const double s = block_sum256(v, red);
    if (threadIdx.x == 0) {
        out[0] = scale * s;
        info[0] = isfinite(s) ? 0 : 1;
    }
}

}  // namespace

hipError_t launch_sq_energy(int m, const double* C, int n_o, double scale, double* work,
                            double* out, int* info, hipStream_t s) {
    if (n_o < 1 || n_o > SQ_MAX) return hipErrorInvalidValue;
    double* cmax = work;
    double* part = work + 1;
    hipLaunchKernelGGL(absmax_kernel, dim3(1), dim3(256), 0, s, int64_t(m) * m, C, cmax);
    const size_t sh = 3 * size_t(m) * sizeof(double);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(sq_lanczos_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(sh));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sq_lanczos_kernel, dim3(m), dim3(256), sh, s, m, C, n_o, cmax, part);
    hipLaunchKernelGGL(sq_sum_kernel, dim3(1), dim3(256), 0, s, m, part, scale, out, info);
    return hipGetLastError();
}


hipError_t launch_symmetrize(int m, double* C, hipStream_t s) {
    hipLaunchKernelGGL(symmetrize_kernel, dim3((m * m + 255) / 256), dim3(256), 0, s, m, C);
    return hipGetLastError();
}

hipError_t launch_chol_inv(int m, const double* M, double* L, double* T, int* info,
                           const MatrixList& at, hipStream_t s) {
    const size_t lds = chol_lds(m);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(chol_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(chol_kernel, dim3(at.n), dim3(SB), lds, s, m, M, L, T, info, at);
    hipLaunchKernelGGL(tri_inv_kernel, dim3((m + NB - 1) / NB, at.n), dim3(NB * NB), 0, s, m, L, T, at);
    return hipGetLastError();
}

hipError_t launch_energy_logdet(int m, const double* C, double* work, double* out, int* info,
                                const MatrixList& at, hipStream_t s) {
    const size_t lds = chol_lds(m);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(energy_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
    if (m <= kCholLds) {
        hipLaunchKernelGGL(energy_kernel, dim3(at.n), dim3(SB), lds, s, m, C, work, out, info, at);
        return hipGetLastError();
    }
    for (int i = 0; i < at.n; ++i)       // work holds one matrix
        hipLaunchKernelGGL(energy_kernel, dim3(1), dim3(SB), lds, s, m, C, work, out, info,
                           MatrixList(at.f[i], at.scale[i]));
    return hipGetLastError();
}

hipError_t launch_syevj(int m, const double* A, double* work, double* w, double* Y,
                        hipStream_t s) {
    if (!Y) {
        // eigenvalues alone; beyond kTriLds m^2 + 6 m + 4 doubles of work
        if (m <= kTriLds) {
            const size_t sh = (size_t(m) * (m + 1) + 3 * size_t(m)) * sizeof(double);
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(syev_lds_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(sh));
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(syev_lds_kernel, dim3(1), dim3(SB), sh, s, m, A, w);
            return hipGetLastError();
        }
        double* st = work + size_t(m) * m;
        double* d = st + 4 * m + 4;
        double* off = d + m;
        hipLaunchKernelGGL(sym_copy_kernel, dim3(unsigned((size_t(m) * m + 255) / 256)), dim3(256),
                           0, s, m, A, work);
        const size_t sh = 3 * size_t(m) * sizeof(double);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(tri_step_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(sh));
        if (e != hipSuccess) return e;
        for (int k = 0; k < m; ++k) {
            // two columns per wave, at most one workgroup per CU
            const int wg = std::min(256, std::max(1, (m - k + 7) / 8));
            hipLaunchKernelGGL(tri_step_kernel, dim3(wg), dim3(256), sh, s, m, k, work, st, d, off);
        }
        const size_t sb = 2 * size_t(m) * sizeof(double);
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(bisect_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, int(sb));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(bisect_kernel, dim3((m + 7) / 8), dim3(64), sb, s, m, d, off, w);
        return hipGetLastError();
    }
    const int np = (m + 1) / 2;
    size_t sh = size_t(3 * np) * sizeof(double);
    if (m <= kJacobiLds) sh += 2 * size_t(m | 1) * m * sizeof(double);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(syevj_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(sh));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(syevj_kernel, dim3(1), dim3(SB), sh, s, m, A, work, w, Y);
    return hipGetLastError();
}

hipError_t launch_box_basis(const int n[3], double h, double* const U[3], double* const kappa[3],
                            hipStream_t s, bool* done) {
    const int nm = std::max(n[0], std::max(n[1], n[2]));
    *done = nm <= kBoxLds;
    if (!*done) return hipSuccess;
    BoxAxes ax;
    for (int a = 0; a < 3; ++a) {
        ax.n[a] = n[a];
        ax.U[a] = U[a];
        ax.kappa[a] = kappa[a];
    }
    ax.ih2 = 1.0 / (h * h);
    fd_weights(ax.w);
    const int m = nm - nm / 2;
    const size_t sh = (3 * size_t((m + 1) / 2) + 2 * size_t(m | 1) * m) * sizeof(double);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(box_basis_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(sh));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(box_basis_kernel, dim3(6), dim3(SB), sh, s, ax);
    return hipGetLastError();
}

hipError_t launch_drho(int64_t nd, int ns, int nvec, const double* psi, const double* x,
                       int stride, double* out, hipStream_t s) {
    const dim3 grid(unsigned((nd + 255) / 256), nvec);
    if (stride == 2)
        hipLaunchKernelGGL(drho_kernel<2>, grid, dim3(256), 0, s, nd, ns, psi, x, out);
    else
        hipLaunchKernelGGL(drho_kernel<1>, grid, dim3(256), 0, s, nd, ns, psi, x, out);
    return hipGetLastError();
}

hipError_t launch_grad_accum_d(int64_t nd, int ns, int nvec, const double* psi,
                               const double* eps, double omega, const double* coeff,
                               double2* dbuf, const double* coefk, const void* x, bool x_fp32,
                               double* grad, hipStream_t s) {
    const int S = ns * nvec;
    hipLaunchKernelGGL(grad_d_kernel, dim3((ns * S + 255) / 256), dim3(256), 0, s, ns, S, eps,
                       omega, coeff, dbuf);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(unsigned((nd + 127) / 128)), block(128);
#define RPA_G(NSM)                                                                           \
    if (ns <= NSM) {                                                                         \
        if (x_fp32)                                                                          \
            hipLaunchKernelGGL((grad_kernel<float2, NSM>), grid, block, 0, s, nd, ns, nvec,  \
                               psi, dbuf, coefk, reinterpret_cast<const float2*>(x), grad);  \
        else                                                                                 \
            hipLaunchKernelGGL((grad_kernel<double2, NSM>), grid, block, 0, s, nd, ns, nvec, \
                               psi, dbuf, coefk, reinterpret_cast<const double2*>(x), grad); \
        return hipGetLastError();                                                            \
    }
    RPA_G(8) RPA_G(16) RPA_G(32) RPA_G(64) RPA_G(128)
#undef RPA_G
    return hipErrorInvalidValue;
}

hipError_t launch_scale(int64_t n, double a, double* x, hipStream_t s) {
    hipLaunchKernelGGL(scale_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, a, x);
    return hipGetLastError();
}

hipError_t launch_fill(int64_t n, double v, double* x, hipStream_t s) {
    hipLaunchKernelGGL(fill_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, v, x);
    return hipGetLastError();
}

__global__ void to_float_kernel(int64_t n, const double* __restrict__ src,
                                float* __restrict__ dst) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = float(src[i]);
}

hipError_t launch_to_float(int64_t n, const double* src, float* dst, hipStream_t s) {
    hipLaunchKernelGGL(to_float_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, src,
                       dst);
    return hipGetLastError();
}

__global__ void real_part_kernel(int64_t n, const double* __restrict__ src,
                                 double* __restrict__ dst) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[2 * i];
}

hipError_t launch_real_part(int64_t n, const double* src, double* dst, hipStream_t s) {
    hipLaunchKernelGGL(real_part_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, src,
                       dst);
    return hipGetLastError();
}

hipError_t launch_copy(int64_t n, const double* src, double* dst, hipStream_t s) {
    hipLaunchKernelGGL(copy_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s, n, src, dst);
    return hipGetLastError();
}

}  // namespace rpa
