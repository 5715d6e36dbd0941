// Kronecker transforms of whole vectors in three passes, for grids whose axes have at most
// kKronAxis points: x and y of a z-plane forward; z forward, the diagonal scale and z back on 64
// columns; x and y back.  They serve nu^{1/2} and nu (real vectors) and the shifted-Laplacian
// preconditioner (complex vectors as pairs of real ones).  A pass moves 16 B per point and does two
// products of 2 n flops per point, so memory bounds it (48^3, 256 vectors: 97 us at 4.67 TB/s, 75 us
// of FP64 MFMA at 72.5 TFLOP/s), if no latency shows.  Therefore a workgroup has one wave per
// 16 x 16 tile of its plane (or of its 64 columns): each wave keeps the two factors of its tile in
// registers for all planes it takes, only the data goes through LDS (two buffers, two barriers per
// plane), the next plane is loaded behind the products, and no branch lies between loads and stores.
// Measured, 48^3, 256 vectors, traced, the mean of four calls with the cold first: 149, 117 and
// 142 us; with four waves a workgroup and the factors in LDS, 270 us each (9 tiles over 4 waves, 2
// workgroups per CU); with branches around the stores, 164, 128 and 158 (the wait for the loads
// waits for the stores).  With 9 waves the registers allow two workgroups per CU, which is what
// keeps the x-y passes from 97 us.
#include <algorithm>
#include <type_traits>

#include "cocg_kernel.h"
#include "internal.h"

namespace rpa {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kKronAxis = 64;   // 16 waves of one tile each, and their factors in 128 registers
constexpr int kCols = 64;         // columns of a z tile
constexpr int kLdz = kCols + 16;  // its LDS stride: neighbouring rows in different bank halves

constexpr int tiles(int n) { return (n + 15) / 16; }

// One 16 x 16 tile over KS steps of 4, one operand in registers: f times the rows of m (4 KS x 16,
// stride ldb), or, TRANS, m (16 x 4 KS, stride ldb) times f.
template <int KS, bool TRANS>
__device__ __forceinline__ d4 product(const double (&f)[KS], const double* m, int ldb, int lane) {
    d4 acc{0, 0, 0, 0};
    const double* p = TRANS ? m + (lane & 15) * ldb + (lane >> 4) : m + (lane >> 4) * ldb + (lane & 15);
    const int step = TRANS ? 4 : 4 * ldb;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        const double v = p[k * step];
        acc = TRANS ? __builtin_amdgcn_mfma_f64_16x16x4f64(v, f[k], acc, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f64_16x16x4f64(f[k], v, acc, 0, 0, 0);
    }
    return acc;
}

// f[k] = M(row, 4 k + lane/16), zero outside n x n: M(r, t) = U[t + n r], or U[r + n t] (TR).
template <int KS>
__device__ __forceinline__ void factor(double (&f)[KS], const double* __restrict__ U, int n, int row,
                                       bool tr, int lane) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        const int t = 4 * k + (lane >> 4);
        const bool in = row < n && t < n;
        const double v = U[in ? (tr ? row + n * t : t + n * row) : 0];
        f[k] = in ? v : 0.0;
    }
}

// Stores without branches: an offset past the buffer is dropped.  A branch around them would make the
// wait for the next plane's loads a wait for the stores as well.
constexpr unsigned kDrop = 0x80000000u;
typedef unsigned u2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(double* p, int64_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, int(n * 8), 0x00027000);
}
__device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t b, unsigned off, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), b, off, 0, 0);
}

struct XyShape {
    int ldx, ldt, rows;   // LDS strides; rows of the second buffer
    int dump;             // where the values past the plane go
    size_t bytes;
};
__host__ __device__ inline XyShape xy_shape(int n0, int n1, int ks) {
    const int m0 = 16 * tiles(n0), m1 = 16 * tiles(n1);
    XyShape s;
    s.ldx = 4 * ks + 1;
    s.ldt = m0 | 16;
    s.rows = m1 > 4 * ks ? m1 : 4 * ks;
    s.dump = m1 * s.ldx + s.rows * s.ldt;
    s.bytes = sizeof(double) * size_t(s.dump + 1);
    return s;
}
__host__ __device__ inline int z_rows(int n2, int ks) {
    return 16 * tiles(n2) > 4 * ks ? 16 * tiles(n2) : 4 * ks;
}
inline size_t z_bytes(int n2, int ks) {
    return sizeof(double) * (size_t(kLdz) * size_t(4 * ks + z_rows(n2, ks)) + 1);
}

constexpr int xy_threads(int ks) { return 64 * tiles(4 * ks) * tiles(4 * ks); }
constexpr int z_threads(int ks) { return 64 * (kCols / 16) * tiles(4 * ks); }

// Planes of n1 rows of n0, 4 KS >= n0, n1: c = Uy^T f Ux forward, f = Uy c Ux^T back (U[t + n a]:
// mode a at point t).  in == out is allowed: a workgroup reads and writes its own planes.
template <int KS, bool INV>
__global__ __launch_bounds__(xy_threads(KS)) void kron_xy(int n0, int n1, int64_t nplanes,
                                                          const double* in, double* out,
                                                          const double* Ux, const double* Uy) {
    extern __shared__ double sh[];
    const XyShape sp = xy_shape(n0, n1, KS);
    const int m1 = 16 * tiles(n1), P = n0 * n1;
    double* X = sh;                 // the plane, m1 x ldx
    double* T = X + m1 * sp.ldx;    // after the x product, rows x ldt
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = wave % tiles(n0) * 16, r0 = wave / tiles(n0) * 16;
    double fx[KS], fy[KS];
    factor<KS>(fx, Ux, n0, c0 + (lane & 15), INV, lane);
    factor<KS>(fy, Uy, n1, r0 + (lane & 15), INV, lane);
    for (int e = tid; e < sp.dump; e += nthr) sh[e] = 0.0;
    // at most 4 points per thread: 16 x 16 per wave
    int src[4], dst[4];
    double nx[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = tid + nthr * q;
        src[q] = e < P ? e : P - 1;
        dst[q] = e < P ? e / n0 * sp.ldx + e % n0 : sp.dump;
    }
    unsigned off[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int x = c0 + (lane & 15), y = r0 + (lane >> 4) + 4 * v;
        off[v] = x < n0 && y < n1 ? 8u * unsigned(y * n0 + x) : kDrop;
    }
    int64_t pl = blockIdx.x;
#pragma unroll
    for (int q = 0; q < 4; ++q) nx[q] = in[pl * P + src[q]];
#pragma unroll
    for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(nx[q]));   // arrived before the loop
    cocg::lds_barrier();
    for (; pl < nplanes; pl += gridDim.x) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            X[dst[q]] = nx[q];
        cocg::lds_barrier();
        const double* next = in + (pl + gridDim.x < nplanes ? pl + gridDim.x : pl) * P;
#pragma unroll
        for (int q = 0; q < 4; ++q) nx[q] = next[src[q]];
        __builtin_amdgcn_sched_barrier(0);
        const d4 t = product<KS, true>(fx, X + r0 * sp.ldx, sp.ldx, lane);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            T[(r0 + (lane >> 4) + 4 * v) * sp.ldt + c0 + (lane & 15)] = t[v];
        cocg::lds_barrier();
        const d4 d = product<KS, false>(fy, T + c0, sp.ldt, lane);
        const auto b = buffer(out + pl * P, P);
#pragma unroll
        for (int v = 0; v < 4; ++v) store(b, off[v], d[v]);
    }
}

// z forward, scale, z back, in place, 4 KS >= n2.  A workgroup keeps its columns of the plane
// (blockIdx.x) and so its modes, and takes vectors blockIdx.y, + gridDim.y, ...
// PRE = false: 64 columns of one vector; scale (4 pi / K)^{power/2}, K = kx + ky + kz, 0 for the
// constant of a periodic grid (zero_mode).
// PRE = true: 32 columns of the real vector 2 v and the imaginary vector 2 v + 1, each tile of 16
// with 8 columns of either, so that a mode's parts meet in lanes l and l ^ 8; division by
// K / 2 + sigma_v - i omega_v, kshift[v] = (sigma_v, omega_v).
template <int KS, bool PRE>
__global__ __launch_bounds__(z_threads(KS)) void kron_z(int n0, int n1, int n2, int nvec, double* X,
                                                        const double* Uz, const double* kx,
                                                        const double* ky, const double* kz, int power,
                                                        int zero_mode, const double2* kshift) {
    extern __shared__ double sh[];
    const int P = n0 * n1, rows = z_rows(n2, KS);
    const int64_t nd = int64_t(P) * n2;
    double* B = sh;                     // 4 KS x kLdz
    double* S = B + 4 * KS * kLdz;      // rows x kLdz
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = wave % (kCols / 16) * 16, r0 = wave / (kCols / 16) * 16;
    double fw[KS], bw[KS];
    factor<KS>(fw, Uz, n2, r0 + (lane & 15), false, lane);
    factor<KS>(bw, Uz, n2, r0 + (lane & 15), true, lane);
    for (int e = tid; e < (4 * KS + rows) * kLdz; e += nthr) sh[e] = 0.0;
    // the column of an LDS column: q in the plane, part (PRE)
    const int q0 = blockIdx.x * (PRE ? kCols / 2 : kCols);
    const int cc = c0 + (lane & 15);
    const int q = q0 + (PRE ? cc / 16 * 8 + (cc & 7) : cc);
    const int64_t part = PRE && (cc & 8) ? nd : 0;
    double f[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int z = r0 + (lane >> 4) + 4 * v;
        const bool ok = q < P && z < n2;
        const double K = ok ? kx[q % n0] + ky[q / n0] + kz[z] : 1.0;
        if (PRE) f[v] = 0.5 * K;
        else if (!ok || (zero_mode && z == 0 && q == 0)) f[v] = 0.0;
        else f[v] = power == 2 ? 4.0 * M_PI / K : sqrt(4.0 * M_PI / K);
    }
    // loads: lanes along the columns (32 of either part where PRE), waves along z
    const int lq = q0 + (PRE ? lane & 31 : lane);
    const int64_t lpart = PRE && lane >= 32 ? nd : 0;
    const int lcol = PRE ? (lane & 31) / 8 * 16 + (lane >> 5) * 8 + (lane & 7) : lane;
    const int nw = nthr >> 6;
    int64_t src[4];
    int dst[4];
    unsigned off[4];
    double nx[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int z = wave + nw * k, zo = r0 + (lane >> 4) + 4 * k;
        dst[k] = z < n2 ? z * kLdz + lcol : (4 * KS + rows) * kLdz;
        off[k] = q < P && zo < n2 ? 8u * unsigned(part + int64_t(zo) * P + q) : kDrop;
        src[k] = lpart + int64_t(z < n2 ? z : n2 - 1) * P + (lq < P ? lq : P - 1);
    }
    const int64_t stride = PRE ? 2 * nd : nd;
    int v = blockIdx.y;
#pragma unroll
    for (int k = 0; k < 4; ++k) nx[k] = X[v * stride + src[k]];
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(nx[k]));   // arrived before the loop
    cocg::lds_barrier();
    for (; v < nvec; v += gridDim.y) {
#pragma unroll
        for (int k = 0; k < 4; ++k) B[dst[k]] = nx[k];
        cocg::lds_barrier();
        const double* next = X + (v + int(gridDim.y) < nvec ? v + int(gridDim.y) : v) * stride;
#pragma unroll
        for (int k = 0; k < 4; ++k) nx[k] = next[src[k]];
        __builtin_amdgcn_sched_barrier(0);
        const d4 t = product<KS, false>(fw, B + c0, kLdz, lane);
        double2 ks{0.0, 0.0};
        if (PRE) ks = kshift[v];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double s;
            if (PRE && r0 + (lane >> 4) + 4 * k >= n2) {
                s = 0.0;    // rows past the axis meet zero factors: they have to be finite
            } else if (PRE) {
                const double d = f[k] + ks.x, w = part ? ks.y : -ks.y;
                s = (t[k] * d + __shfl_xor(t[k], 8, 64) * w) / (d * d + w * w);
            } else {
                s = t[k] * f[k];
            }
            S[(r0 + (lane >> 4) + 4 * k) * kLdz + cc] = s;
        }
        cocg::lds_barrier();
        const d4 d = product<KS, false>(bw, S + c0, kLdz, lane);
        const auto b = buffer(X + v * stride, stride);
#pragma unroll
        for (int k = 0; k < 4; ++k) store(b, off[k], d[k]);
    }
}

template <typename F>
hipError_t lds_limit(F fn, size_t bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

// Workgroups that the chip holds at once (LDS; registers for 4 to 5 waves per SIMD).
int64_t resident(size_t lds, int threads) {
    return 256 * std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / int64_t(lds), 1280 / threads));
}

template <int KS, bool INV>
hipError_t run_xy(const Grid& g, int64_t nplanes, const double* in, double* out, const double* Ux,
                  const double* Uy, hipStream_t s) {
    const size_t lds = xy_shape(g.n0, g.n1, KS).bytes;
    const int threads = 64 * tiles(g.n0) * tiles(g.n1);
    const hipError_t e = lds_limit(kron_xy<KS, INV>, lds);
    if (e != hipSuccess) return e;
    // rounds of equal length
    const int64_t rounds = (nplanes + resident(lds, threads) - 1) / resident(lds, threads);
    const int64_t wgs = (nplanes + rounds - 1) / rounds;
    hipLaunchKernelGGL((kron_xy<KS, INV>), dim3(unsigned(wgs)), dim3(threads), lds, s, g.n0, g.n1,
                       nplanes, in, out, Ux, Uy);
    return hipGetLastError();
}

template <int KS, bool PRE>
hipError_t run_z(const Grid& g, int nvec, double* X, const double* Uz, const double* kx,
                 const double* ky, const double* kz, int power, const double2* kshift,
                 hipStream_t s) {
    const size_t lds = z_bytes(g.n2, KS);
    const int threads = 64 * (kCols / 16) * tiles(g.n2), cols = PRE ? kCols / 2 : kCols;
    const hipError_t e = lds_limit(kron_z<KS, PRE>, lds);
    if (e != hipSuccess) return e;
    const int per = (g.n0 * g.n1 + cols - 1) / cols;
    const int64_t split = std::max<int64_t>(1, std::min<int64_t>(65535, resident(lds, threads) / per));
    const int64_t rounds = (nvec + split - 1) / split;
    const int64_t wgs = (nvec + rounds - 1) / rounds;
    hipLaunchKernelGGL((kron_z<KS, PRE>), dim3(unsigned(per), unsigned(wgs)), dim3(threads), lds, s,
                       g.n0, g.n1, g.n2, nvec, X, Uz, kx, ky, kz, power, g.periodic() ? 1 : 0, kshift);
    return hipGetLastError();
}

// The compiled number of K steps (4 points each) for an axis of n points.
template <typename F>
hipError_t with_steps(int n, F f) {
    if (n <= 16) return f(std::integral_constant<int, 4>{});
    if (n <= 24) return f(std::integral_constant<int, 6>{});
    if (n <= 32) return f(std::integral_constant<int, 8>{});
    if (n <= 40) return f(std::integral_constant<int, 10>{});
    if (n <= 48) return f(std::integral_constant<int, 12>{});
    return f(std::integral_constant<int, 16>{});
}

// mid: where the transform lies between the passes; out, or a block apart from both.
template <bool PRE>
hipError_t run(const Grid& g, int nvec, const double* in, double* mid, double* out,
               const double* Ux, const double* Uy, const double* Uz, const double* kx,
               const double* ky, const double* kz, int power, const double2* kshift, hipStream_t s) {
    const int64_t planes = int64_t(g.n2) * nvec * (PRE ? 2 : 1);
    const int nxy = std::max(g.n0, g.n1);
    hipError_t e = with_steps(nxy, [&](auto K) {
        return run_xy<decltype(K)::value, false>(g, planes, in, mid, Ux, Uy, s);
    });
    if (e != hipSuccess) return e;
    e = with_steps(g.n2, [&](auto K) {
        return run_z<decltype(K)::value, PRE>(g, nvec, mid, Uz, kx, ky, kz, power, kshift, s);
    });
    if (e != hipSuccess) return e;
    return with_steps(nxy, [&](auto K) {
        return run_xy<decltype(K)::value, true>(g, planes, mid, out, Ux, Uy, s);
    });
}

}  // namespace

bool kron_fused_fits(const Grid& g) { return std::max(g.n0, std::max(g.n1, g.n2)) <= kKronAxis; }

// The first pass reads planes of `in` in any order while it writes others: blocks that overlap
// without being the same go through tmp, so that all of `in` is read before `out` is written.
hipError_t launch_kron_fused(const Grid& g, int power, int nvec, const double* in, double* out,
                             double* tmp, const double* Ux, const double* Uy, const double* Uz, const double* kx,
                             const double* ky, const double* kz, hipStream_t s) {
    if (nvec <= 0) return hipSuccess;
    const size_t bytes = size_t(g.nd()) * nvec * sizeof(double);
    const uintptr_t a = reinterpret_cast<uintptr_t>(in), b = reinterpret_cast<uintptr_t>(out);
    double* mid = a != b && a < b + bytes && b < a + bytes ? tmp : out;
    return run<false>(g, nvec, in, mid, out, Ux, Uy, Uz, kx, ky, kz, power, nullptr, s);
}

hipError_t launch_kron_fused_precond(const Grid& g, int nsys, const double* in, double* out,
                                     const double* Ux, const double* Uy, const double* Uz,
                                     const double* kx, const double* ky, const double* kz,
                                     const double2* kshift, hipStream_t s) {
    if (nsys <= 0) return hipSuccess;
    return run<true>(g, nsys, in, out, out, Ux, Uy, Uz, kx, ky, kz, 0, kshift, s);
}

}  // namespace rpa
