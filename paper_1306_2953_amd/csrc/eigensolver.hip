// One RMM-DIIS eigensolver step on gfx950 (Secs. 3, 6 and 9).
//
// The step, for N states in nblk blocks of B (all on the caller's stream, one
// host synchronisation at the end, and one after 2. where blocks can freeze):
//   1. H psi for all blocks; Rayleigh-Ritz (subspace matrix, Jacobi, rotate).
//   2. Per state: eps0 = <psi|H psi>/<psi|psi>, R0 = H psi - eps0 psi,
//      residual norm.  A block whose states are all below tol is frozen.
//   3. d1 = K R0 (filter), H d1; the trial step lambda minimises the Rayleigh
//      quotient of psi + lambda d1 (2x2 generalised problem per state); psi1 =
//      psi + lambda d1.  With a learned preconditioner its direction d_n =
//      K_n R0 joins the filter's: the Rayleigh quotient is minimised over
//      span{psi, d_f, d_n} (3x3 problem per state), giving K = a K_f + b K_n
//      for the state's step (lambda 1); a singular 3x3 problem leaves the
//      state on the filter (b = 0).
//   4. m - 1 DIIS iterations: residuals R_i = H psi_i - eps_i psi_i of the
//      history; minimise |sum c R| / |sum c psi| over the history written in
//      the basis {psi_L, psi_i - psi_L} (generalised eigenproblem per state,
//      lowest eigenvector, c_0 = 1); psi_bar, R_bar; d = K R_bar; psi_{j+1} =
//      psi_bar + lambda d.
//   5. Orthonormalise (Cholesky, eq. 8).
// The iterates are never formed: all of them are psi plus multiples of d1 and
// d2, and their residuals are R0 plus multiples of psi and of d_i and H d_i,
// so the DIIS matrices follow per state from the inner products of {psi, R0,
// d1, g1, d2, g2}, g = H d - eps0 d.  Residuals enter as R0 and g (small as
// the residuals themselves), not as H psi, so the products lose no digits to
// cancellation.  One pass over {psi, R0, d1, H d1} gives lambda and the first
// DIIS coefficients, one over those and {d2, H d2} the second, each followed
// by one pass that writes R_bar; the last psi_bar + lambda K R_bar is formed
// by the filter itself.  Storing the iterates and their H took 45 field reads
// and writes a step beside H psi and the dense stage, this takes 30.
// Per-state inner products are sums over points with FP64 accumulation and
// a fixed-order reduction over point chunks; the small per-state problems
// are solved in FP64, one thread per state.
#include <cmath>
#include <cstring>

#include "colreduce.hpp"
#include "dense.hpp"
#include "internal.hpp"
#include "rotation.hpp"

rs_status subspace_diag_capped(rs_ctx *c, void *psi, void *hpsi, double *eig, int nblk, int B, int dtype,
                               int prec, int max_sweeps, int nreal, hipStream_t st);
rs_status orthonormalize_impl(rs_ctx *c, void *psi, int nblk, int B, int dtype, int prec, double *S_out,
                              int32_t *info, int nreal, hipStream_t s);
rs_status orthonormalize_async(rs_ctx *c, void *psi, int nblk, int B, int dtype, int prec, double *S_out, int nreal,
                               hipStream_t s);
rs_status orthonormalize_status(int info);
const int *ctx_sweeps(const rs_ctx *c);
const int *ctx_info(const rs_ctx *c);

namespace rs {
rs_status hpsi_apply(const rs_grid *g, const rs_nl *nl, const void *vloc, const void *psi, void *hpsi,
                     int nblk, int B, int dtype, hipStream_t st, int of);
rs_status filter_apply(const rs_grid *g, double alpha, const void *r, void *out, int nblk, int B, int dtype,
                       hipStream_t st, const FilterUpdate *upd = nullptr);
rs_status kinetic_apply(const rs_grid *g, const void *psi, void *out, int nblk, int B, int dtype,
                        hipStream_t st);
rs_status cnn_precondition(rs_cnn *c, const rs_grid *g, const void *r, const double *sigma, void *out, int nblk,
                           int B, int dtype, hipStream_t st);
}

namespace {
using namespace rsred;

constexpr int kMaxIter = 3;   // largest m
constexpr int kMaxSweeps = 30;  // Jacobi sweeps that reach FP64 accuracy from any start

template <typename F> struct OpDots2 {   // <x|x>, <x|y>
    typedef F T;
    static constexpr int NF = 2;
    const T *x, *y;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = y[i];
    }
    __device__ void operator()(const T *w, int64_t, int, double *a) const {
        const double u = w[0], v = w[1];
        a[0] += u * u;
        a[1] += u * v;
    }
};
template <typename F> struct OpResid {   // R = h - eps x, <R|R>
    typedef F T;
    static constexpr int NF = 2;
    const T *x, *h;
    T *R;
    const double *eps;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = h[i];
    }
    __device__ void operator()(const T *w, int64_t i, int c, double *a) const {
        const T r = (T)((double)w[1] - eps[c] * (double)w[0]);
        R[i] = r;
        a[0] += (double)r * (double)r;
    }
};
// The trial subspace {x, d, e} (filter and network directions): <x|Hd>,
// <d|Hx>, <d|Hd>, <x|d>, <d|d>, the same five for e, then <d|He>, <e|Hd>,
// <d|e>.
template <typename F> struct OpLam3 {
    typedef F T;
    static constexpr int NF = 6;
    const T *x, *hx, *d, *hd, *e, *he;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = hx[i];
        v[2] = d[i];
        v[3] = hd[i];
        v[4] = e[i];
        v[5] = he[i];
    }
    __device__ void operator()(const T *f, int64_t, int, double *a) const {
        const double u = f[0], hu = f[1], v = f[2], hv = f[3], w = f[4], hw = f[5];
        a[0] += u * hv;
        a[1] += v * hu;
        a[2] += v * hv;
        a[3] += u * v;
        a[4] += v * v;
        a[5] += u * hw;
        a[6] += w * hu;
        a[7] += w * hw;
        a[8] += u * w;
        a[9] += w * w;
        a[10] += v * hw;
        a[11] += w * hv;
        a[12] += v * w;
    }
};
// Inner products of {x, R, d, g}, g = hd - eps0 d, without <x|x> and <R|R>:
// <x|R>, <x|d>, <x|g>, <R|d>, <R|g>, <d|d>, <d|g>, <g|g>.
template <typename F> struct OpGram1 {
    typedef F T;
    static constexpr int NF = 4;
    const T *x, *R, *d, *hd;
    const double *eps;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = R[i];
        v[2] = d[i];
        v[3] = hd[i];
    }
    __device__ void operator()(const T *f, int64_t, int c, double *a) const {
        const double u = f[0], r = f[1], v = f[2], g = (double)f[3] - eps[c] * v;
        a[0] += u * r;
        a[1] += u * v;
        a[2] += u * g;
        a[3] += r * v;
        a[4] += r * g;
        a[5] += v * v;
        a[6] += v * g;
        a[7] += g * g;
    }
};
// The products that {e, f}, f = he - eps0 e, add: e and f with x, R, d, g,
// then <e|e>, <e|f>, <f|f>.
template <typename F> struct OpGram2 {
    typedef F T;
    static constexpr int NF = 6;
    const T *x, *R, *d, *hd, *e, *he;
    const double *eps;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = R[i];
        v[2] = d[i];
        v[3] = hd[i];
        v[4] = e[i];
        v[5] = he[i];
    }
    __device__ void operator()(const T *z, int64_t, int c, double *a) const {
        const double w = z[4], f = (double)z[5] - eps[c] * w;
        const double u = z[0], r = z[1], v = z[2], g = (double)z[3] - eps[c] * v;
        a[0] += u * w;
        a[1] += u * f;
        a[2] += r * w;
        a[3] += r * f;
        a[4] += v * w;
        a[5] += v * f;
        a[6] += g * w;
        a[7] += g * f;
        a[8] += w * w;
        a[9] += w * f;
        a[10] += f * f;
    }
};

// --------------------------------------------------------- map kernels
// blockIdx.y: the block (or its entry in the block map); a thread takes
// kMapPts values of one state (256 and its multiples are multiples of B), so
// the state's factors are read once.
constexpr int kMapPts = 4;
template <typename F>
__device__ __forceinline__ void map_block(int64_t np, int B, const int *bmap, F f) {
    const int blk = bmap ? bmap[blockIdx.y] : (int)blockIdx.y;
    const int64_t n = np * B, i0 = (int64_t)blockIdx.x * (256 * kMapPts) + threadIdx.x;
    f(blk * B + (int)(i0 & (B - 1)), [&](auto g) {
#pragma unroll
        for (int k = 0; k < kMapPts; ++k)
            if (i0 + 256 * k < n) g(blk * n + i0 + 256 * k);
    });
}
dim3 map_grid(int64_t np, int B, int nblk) {
    return dim3((unsigned)((np * B + 256 * kMapPts - 1) / (256 * kMapPts)), nblk);
}

// rb = R + a0 x + a1 d + a2 hd (+ a3 e + a4 he when e is given): the mixed
// residual R_bar; lin [5][N] per state.
template <typename T>
__global__ void __launch_bounds__(256)
residual_mix_kernel(const T *__restrict__ x, const T *__restrict__ R, const T *__restrict__ d,
                    const T *__restrict__ hd, const T *__restrict__ e, const T *__restrict__ he,
                    const double *__restrict__ lin, T *__restrict__ rb, int64_t np, int B, int N,
                    const int *__restrict__ bmap) {
    map_block(np, B, bmap, [&](int c, auto each) {
        const double a0 = lin[c], a1 = lin[N + c], a2 = lin[2 * N + c];
        if (e) {
            const double a3 = lin[3 * N + c], a4 = lin[4 * N + c];
            each([&](int64_t i) {
                rb[i] = (T)((double)R[i] + a0 * (double)x[i] + a1 * (double)d[i] + a2 * (double)hd[i] +
                            a3 * (double)e[i] + a4 * (double)he[i]);
            });
        } else {
            each([&](int64_t i) {
                rb[i] = (T)((double)R[i] + a0 * (double)x[i] + a1 * (double)d[i] + a2 * (double)hd[i]);
            });
        }
    });
}

// x += a0 d1 + a1 d2 + a2 dl (d1, d2 where given): the newest iterate, where
// the filter does not form it itself; upd [3][N] per state.
template <typename T>
__global__ void __launch_bounds__(256)
update_kernel(T *__restrict__ x, const T *__restrict__ d1, const T *__restrict__ d2, const T *__restrict__ dl,
              const double *__restrict__ upd, int64_t np, int B, int N, const int *__restrict__ bmap) {
    map_block(np, B, bmap, [&](int c, auto each) {
        const double a0 = upd[c], a1 = upd[N + c], a2 = upd[2 * N + c];
        each([&](int64_t i) {
            double v = (double)x[i] + a2 * (double)dl[i];
            if (d1) v += a0 * (double)d1[i];
            if (d2) v += a1 * (double)d2[i];
            x[i] = (T)v;
        });
    });
}

// ----------------------------------------------------- per-state solvers
// Lowest eigenpair of the symmetric generalised problem A c = mu B c
// (n <= 4): scale by diag(B)^-1/2, Cholesky of B, Jacobi on L^-1 A L^-T.
// Returns false when B is not positive definite.  n is a template parameter
// and every loop over indices unrolls, so the matrices live in registers;
// with n at run time they lay in scratch memory and a call took 81-111 us,
// now 5-8 (a serial chain of FP64 divisions and square roots).
template <int n>
__device__ __forceinline__ bool lowest_geneig(const double (&A_in)[n * n], const double (&B_in)[n * n],
                                              double (&c)[n]) {
    double A[n * n], Bm[n * n], D[n], L[n * n], C[n * n], V[n * n];
#pragma unroll
    for (int i = 0; i < n; ++i) {
        if (!(B_in[i * n + i] > 0.0)) return false;
        D[i] = 1.0 / sqrt(B_in[i * n + i]);
    }
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
        for (int j = 0; j < n; ++j) {
            A[i * n + j] = A_in[i * n + j] * D[i] * D[j];
            Bm[i * n + j] = B_in[i * n + j] * D[i] * D[j];
        }
#pragma unroll
    for (int j = 0; j < n; ++j) {
        double d = Bm[j * n + j];
#pragma unroll
        for (int k = 0; k < j; ++k) d -= L[j * n + k] * L[j * n + k];
        if (!(d > 0.0)) return false;
        L[j * n + j] = sqrt(d);
#pragma unroll
        for (int i = j + 1; i < n; ++i) {
            double s = Bm[i * n + j];
#pragma unroll
            for (int k = 0; k < j; ++k) s -= L[i * n + k] * L[j * n + k];
            L[i * n + j] = s / L[j * n + j];
        }
    }
    // C = L^-1 A L^-T: solve L Y = A, then L C^T = Y^T
    double Y[n * n];
#pragma unroll
    for (int col = 0; col < n; ++col)
#pragma unroll
        for (int i = 0; i < n; ++i) {
            double s = A[i * n + col];
#pragma unroll
            for (int k = 0; k < i; ++k) s -= L[i * n + k] * Y[k * n + col];
            Y[i * n + col] = s / L[i * n + i];
        }
#pragma unroll
    for (int row = 0; row < n; ++row)
#pragma unroll
        for (int i = 0; i < n; ++i) {
            double s = Y[row * n + i];
#pragma unroll
            for (int k = 0; k < i; ++k) s -= L[i * n + k] * C[row * n + k];
            C[row * n + i] = s / L[i * n + i];
        }
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
        for (int j = 0; j < n; ++j) {
            V[i * n + j] = i == j ? 1.0 : 0.0;
            if (j > i) C[i * n + j] = C[j * n + i] = 0.5 * (C[i * n + j] + C[j * n + i]);
        }
#pragma unroll 1
    for (int sweep = 0; sweep < 50; ++sweep) {
        double off = 0.0, tot = 0.0;
#pragma unroll
        for (int i = 0; i < n; ++i)
#pragma unroll
            for (int j = 0; j < n; ++j) {
                tot += C[i * n + j] * C[i * n + j];
                if (i != j) off += C[i * n + j] * C[i * n + j];
            }
        if (!(off > 1e-32 * tot)) break;
#pragma unroll
        for (int p = 0; p < n; ++p)
#pragma unroll
            for (int q = p + 1; q < n; ++q) {
                const double2 r = rs::jacobi_rotation(C[p * n + p], C[p * n + q], C[q * n + q]);
                const double cs = r.x, sn = r.y;
#pragma unroll
                for (int k = 0; k < n; ++k) {
                    const double kp = C[k * n + p], kq = C[k * n + q];
                    C[k * n + p] = cs * kp - sn * kq;
                    C[k * n + q] = sn * kp + cs * kq;
                }
#pragma unroll
                for (int k = 0; k < n; ++k) {
                    const double pk = C[p * n + k], qk = C[q * n + k];
                    C[p * n + k] = cs * pk - sn * qk;
                    C[q * n + k] = sn * pk + cs * qk;
                }
#pragma unroll
                for (int k = 0; k < n; ++k) {
                    const double kp = V[k * n + p], kq = V[k * n + q];
                    V[k * n + p] = cs * kp - sn * kq;
                    V[k * n + q] = sn * kp + cs * kq;
                }
            }
    }
    // the lowest pair, taken by selects (an index would spill V)
    double mu = C[0], y[n];
#pragma unroll
    for (int i = 0; i < n; ++i) y[i] = V[i * n];
#pragma unroll
    for (int j = 1; j < n; ++j) {
        const bool lower = C[j * n + j] < mu;
        mu = lower ? C[j * n + j] : mu;
#pragma unroll
        for (int i = 0; i < n; ++i) y[i] = lower ? V[i * n + j] : y[i];
    }
    // c = D L^-T y
#pragma unroll
    for (int i = n - 1; i >= 0; --i) {
        double s = y[i];
#pragma unroll
        for (int k = i + 1; k < n; ++k) s -= L[k * n + i] * c[k];
        c[i] = s / L[i * n + i];
    }
    bool finite = true;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        c[i] *= D[i];
        finite = finite && isfinite(c[i]);
    }
    return finite;
}

// Rayleigh quotient of the Rayleigh-Ritz state from <x|x>, <x|Hx> (0 for zero
// padding states); the sums are kept.
struct Eps0 {
    double *d2, *eps;
    int N;
    __device__ void operator()(int c, const double *s) const {
        d2[c] = s[0];
        d2[N + c] = s[1];
        eps[c] = s[0] > 0.0 ? s[1] / s[0] : 0.0;
    }
};

// p^T G q for the symmetric G (n x n).
template <int n> __device__ __forceinline__ double quad(const double (&G)[n][n], const double (&p)[n], const double (&q)[n]) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        double u = 0.0;
#pragma unroll
        for (int j = 0; j < n; ++j) u += G[i][j] * q[j];
        t += p[i] * u;
    }
    return t;
}
// DIIS coefficients over n iterates from the residuals rho and the differences
// e as combinations of the k vectors of G (c_0 = 1; degenerate: e_0).
template <int n, int k>
__device__ __forceinline__ void diis(const double (&G)[k][k], const double (&rho)[n][k], const double (&e)[n][k],
                                     double (&c)[n]) {
    double A[n * n], Bm[n * n], v[n];
#pragma unroll
    for (int p = 0; p < n; ++p)
#pragma unroll
        for (int q = p; q < n; ++q) {
            A[p * n + q] = A[q * n + p] = quad<k>(G, rho[p], rho[q]);
            Bm[p * n + q] = Bm[q * n + p] = quad<k>(G, e[p], e[q]);
        }
    const bool ok = lowest_geneig<n>(A, Bm, v) && v[0] != 0.0;
#pragma unroll
    for (int i = 0; i < n; ++i) c[i] = ok ? v[i] / v[0] : (i == 0 ? 1.0 : 0.0);
}

// What the second stage needs of the first, [kStage][N]: lambda, mu, delta1,
// and the sums of OpGram1.
constexpr int kStage = 11;

// After OpGram1: the trial step (unless lam_in, with a network, holds it;
// frozen or zero direction: 0), iterate 1's Rayleigh quotient eps0 + delta1,
// and the DIIS coefficients of iterates 0 and 1.  R_bar's factors go to lin,
// the update's to upd: psi_bar = psi + mu d1.
struct Solve1 {
    const double *d2, *rr, *eps, *lam_in;
    const int *active;
    double *stage, *lin, *upd;
    int N, m;
    __device__ void operator()(int c, const double *s) const {
        const double xx = d2[c], RR = rr[c], e0 = eps[c];
        const double xR = s[0], xd = s[1], xg = s[2], Rd = s[3], Rg = s[4], dd = s[5], dg = s[6], gg = s[7];
        double lam = 0.0;
        if (lam_in) {
            lam = lam_in[c];
        } else if (active[c] && dd > 0.0) {
            // lowest pair of H - eps0 in {x, d / |d|}
            const double sc = 1.0 / sqrt(dd), a12 = 0.5 * (xg + Rd) * sc, b12 = xd * sc;
            const double A[4] = {xR, a12, a12, dg * sc * sc}, Bm[4] = {xx, b12, b12, 1.0};
            double v[2];
            if (lowest_geneig<2>(A, Bm, v) && v[0] != 0.0) lam = v[1] / v[0] * sc;
        }
        double mu = lam, delta = 0.0, f[3] = {0.0, 0.0, 0.0};
        if (lam != 0.0 && m > 1) {
            const double n1 = xx + lam * (2.0 * xd + lam * dd);
            delta = n1 > 0.0 ? (xR + lam * (xg + Rd) + lam * lam * dg) / n1 : 0.0;
            const double G[4][4] = {{xx, xR, xd, xg}, {xR, RR, Rd, Rg}, {xd, Rd, dd, dg}, {xg, Rg, dg, gg}};
            const double rho[2][4] = {{-delta, 1.0, -delta * lam, lam}, {delta, 0.0, delta * lam, -lam}};
            const double e[2][4] = {{1.0, 0.0, lam, 0.0}, {0.0, 0.0, -lam, 0.0}};
            double co[2];
            diis<2, 4>(G, rho, e, co);
            const double k1 = 1.0 - co[1];
            mu = lam * k1;
            f[0] = -k1 * delta;
            f[1] = -k1 * delta * lam - mu * e0;
            f[2] = mu;
        }
        stage[c] = lam;
        stage[N + c] = mu;
        stage[2 * N + c] = delta;
#pragma unroll
        for (int k = 0; k < 8; ++k) stage[(3 + k) * N + c] = s[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) lin[k * N + c] = f[k];
        upd[c] = mu;
        upd[N + c] = 0.0;
        upd[2 * N + c] = lam;
    }
};

// After OpGram2: iterate 2 = psi + mu d1 + lambda d2, its Rayleigh quotient
// eps0 + delta2, and the DIIS coefficients of iterates 0, 1 and 2.
struct Solve2 {
    const double *d2, *rr, *eps, *stage;
    double *lin, *upd;
    int N;
    __device__ void operator()(int c, const double *s) const {
        const double lam = stage[c], mu = stage[N + c], del1 = stage[2 * N + c], e0 = eps[c];
        double f[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, a1 = 0.0, a2 = 0.0;
        if (lam != 0.0) {
            double p[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k] = stage[(3 + k) * N + c];
            // order x, R, d1, g1, d2, g2
            const double G[6][6] = {{d2[c], p[0], p[1], p[2], s[0], s[1]}, {p[0], rr[c], p[3], p[4], s[2], s[3]},
                                    {p[1], p[3], p[5], p[6], s[4], s[5]},  {p[2], p[4], p[6], p[7], s[6], s[7]},
                                    {s[0], s[2], s[4], s[6], s[8], s[9]},  {s[1], s[3], s[5], s[7], s[9], s[10]}};
            const double x2[6] = {1.0, 0.0, mu, 0.0, lam, 0.0}, g2[6] = {0.0, 1.0, 0.0, mu, 0.0, lam};
            const double n2 = quad<6>(G, x2, x2);
            const double del2 = n2 > 0.0 ? quad<6>(G, x2, g2) / n2 : 0.0;
            const double r1[6] = {-del1, 1.0, -del1 * lam, lam, 0.0, 0.0};
            double rho[3][6], e[3][6];
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                rho[0][k] = g2[k] - del2 * x2[k];
                rho[1][k] = (k == 1 ? 1.0 : 0.0) - rho[0][k];
                rho[2][k] = r1[k] - rho[0][k];
                e[0][k] = x2[k];
                e[1][k] = (k == 0 ? 1.0 : 0.0) - x2[k];
                e[2][k] = (k == 0 ? 1.0 : k == 2 ? lam : 0.0) - x2[k];
            }
            double co[3], r[6];
            diis<3, 6>(G, rho, e, co);
#pragma unroll
            for (int k = 0; k < 6; ++k) r[k] = rho[0][k] + co[1] * rho[1][k] + co[2] * rho[2][k];
            const double k2 = 1.0 - co[1] - co[2];
            a1 = mu * k2 + lam * co[2];
            a2 = lam * k2;
            f[0] = r[0];
            f[1] = r[2] - e0 * r[3];
            f[2] = r[3];
            f[3] = r[4] - e0 * r[5];
            f[4] = r[5];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) lin[k * N + c] = f[k];
        upd[c] = a1;
        upd[N + c] = a2;
        upd[2 * N + c] = lam;
    }
};

// Filter and network coefficients of the trial step (state frozen: lambda
// 0).  d2: [<x|x>, <x|Hx>]; d13: the dots of OpLam3.  The Rayleigh quotient
// is minimised over {x, d/|d|, e/|e|}; the lowest generalised eigenvector,
// first component one, gives mix = (a, b) and lambda = 1.  When that 3x3
// problem is singular the 2x2 filter step is kept: lambda from it, mix =
// (lambda, 0).
__global__ void mix_kernel(const double *__restrict__ d2, const double *__restrict__ d13,
                           const int *__restrict__ active, int N, double *__restrict__ lam,
                           double *__restrict__ mix) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    double l = 0.0, ma = 0.0, mb = 0.0;
    const double bdd = d13[4 * N + c], bee = d13[9 * N + c];
    if (active[c] && bdd > 0.0) {
        const double s = 1.0 / sqrt(bdd);
        const double a11 = d2[1 * N + c], b11 = d2[0 * N + c];
        const double a12 = 0.5 * (d13[0 * N + c] + d13[1 * N + c]) * s;
        const double a22 = d13[2 * N + c] * s * s;
        const double b12 = d13[3 * N + c] * s;
        {
            const double A[4] = {a11, a12, a12, a22}, Bm[4] = {b11, b12, b12, 1.0};
            double v[2];
            if (lowest_geneig<2>(A, Bm, v) && v[0] != 0.0) l = v[1] / v[0] * s;
            ma = l;
        }
        if (bee > 0.0 && isfinite(bee)) {
            const double t = 1.0 / sqrt(bee);
            const double a13 = 0.5 * (d13[5 * N + c] + d13[6 * N + c]) * t;
            const double a33 = d13[7 * N + c] * t * t;
            const double b13 = d13[8 * N + c] * t;
            const double a23 = 0.5 * (d13[10 * N + c] + d13[11 * N + c]) * s * t;
            const double b23 = d13[12 * N + c] * s * t;
            const double A[9] = {a11, a12, a13, a12, a22, a23, a13, a23, a33};
            const double Bm[9] = {b11, b12, b13, b12, 1.0, b23, b13, b23, 1.0};
            double v[3];
            if (lowest_geneig<3>(A, Bm, v) && v[0] != 0.0) {
                ma = v[1] / v[0] * s;
                mb = v[2] / v[0] * t;
                l = 1.0;
            }
        }
    }
    lam[c] = l;
    mix[c] = ma;
    mix[N + c] = mb;
}

// d = a d + b e (and hd = a hd + b he when given) for the states whose
// network coefficient b is nonzero.
template <typename T>
__global__ void __launch_bounds__(256)
mixdir_kernel(T *__restrict__ d, const T *__restrict__ e, T *__restrict__ hd, const T *__restrict__ he,
              const double *__restrict__ mix, int64_t np, int B, int N, const int *__restrict__ bmap) {
    // blockIdx.y: the block (or its entry in the block map); B is a power of two
    const int blk = bmap ? bmap[blockIdx.y] : (int)blockIdx.y;
    const int64_t il = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (il >= np * B) return;
    const int64_t i = (int64_t)blk * np * B + il;
    const int c = blk * B + (int)(il & (B - 1));
    const double b = mix[N + c];
    if (b == 0.0) return;
    const double a = mix[c];
    d[i] = (T)(a * (double)d[i] + b * (double)e[i]);
    if (hd) hd[i] = (T)(a * (double)hd[i] + b * (double)he[i]);
}

// eps0 = <x|Hx>/<x|x>; after the residual pass: res = sqrt(<R|R>), and a
// block is active unless every state in it is below tol.
// sigma_k = -<psi_k|T psi_k> / <psi_k|psi_k>
__global__ void sigma_kernel(const double *__restrict__ d2, int N, double *__restrict__ sigma) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    const double nn = d2[0 * N + c];
    sigma[c] = nn > 0.0 ? -d2[1 * N + c] / nn : 0.0;
}

__global__ void active_kernel(const double *__restrict__ rr, int N, int B, double tol, int block_stop,
                              double *__restrict__ res, int *__restrict__ active, int *__restrict__ host_active) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    const double r = sqrt(rr[c]);
    res[c] = r;
    int act = 1;
    if (block_stop) {
        const int b0 = (c / B) * B;
        act = 0;
        for (int k = b0; k < b0 + B; ++k) act |= !(sqrt(rr[k]) < tol);
    }
    active[c] = act;
    host_active[c] = act;
}

// What a step reports, written by the device straight into pinned host memory
// and waited for once.  Five pageable copies and two waits in its place cost a
// small system 100 us a step: two FP64 steps of 8 states on 32768 points take 507
// against 711 us.  active is written by active_kernel; the rest here.
struct StepReport {
    double *eig, *res, *mix;
    int *active, *sweeps, *info;
};
__global__ void report_kernel(StepReport r, const double *__restrict__ eig, const double *__restrict__ res,
                              const double *__restrict__ mix, const int *__restrict__ sweeps,
                              const int *__restrict__ info, int N) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c == 0) {
        *r.sweeps = *sweeps;
        *r.info = *info;
    }
    if (c >= N) return;
    r.eig[c] = eig[c];
    r.res[c] = res[c];
    r.mix[c] = mix ? mix[c] : 0.0;
}

}  // namespace

struct rs_solver {
    const rs_grid *g = nullptr;
    const rs_nl *nl = nullptr;
    const void *vloc = nullptr;
    int N = 0, B = 0, nblk = 0, dtype = 0, prec = 0;
    int nreal = 0;                  // states asked for; N - nreal zero padding states
    rs_solver_opts opts{};
    rs_ctx *ctx = nullptr;
    size_t field_bytes = 0;
    rs::DevBuf h;                // H psi; from the first DIIS iteration on R_bar
    rs::DevBuf R;                // R0
    rs::DevBuf d[2], hd[2];      // the directions that H was applied to (the second one for m = 3)
    rs::DevBuf partial, d2, rr, res, eig, lam, eps, stage, lin, upd, active;
    rs::DevBuf sigma, R0;        // shifts, recorded residuals
    rs::DevBuf dn, hdn;          // network direction and H applied (with a network)
    rs::DevBuf d13, mix;         // trial-subspace dots; filter / network coefficients
    rs::DevBuf bmap;             // int [nblk]: blocks of the trial step and DIIS when some are frozen
    std::vector<int> host_map;
    void *pinned = nullptr;      // the step's report
    StepReport report{};
    rs_cnn *cnn = nullptr;
    int rr_sweeps = kMaxSweeps;
    int steps = 0;
    rs_solver_stats stats{};
};

extern "C" rs_status rs_eigensolve_create(const rs_grid *g, const rs_nl *nl, const void *vloc, int32_t nstates,
                                          int32_t B, int32_t dtype, const rs_solver_opts *opts, rs_solver **out) {
    using namespace rs;
    if (!g || !vloc || !out) return fail(RS_EINVAL, "rs_eigensolve_create: null argument");
    *out = nullptr;
    if (B < 1 || B > 64 || (B & (B - 1))) return fail(RS_EINVAL, "rs_eigensolve_create: bad B");
    if (nstates < 1 || nstates > 256) return fail(RS_EINVAL, "rs_eigensolve_create: nstates must be in [1, 256]");
    if (dtype != RS_F64 && dtype != RS_F32) return fail(RS_EINVAL, "rs_eigensolve_create: bad dtype");
    if (nl && nl->max_states < (nstates + B - 1) / B * B)
        return fail(RS_EINVAL, "rs_eigensolve_create: projector set too small (needs whole blocks)");
    auto s = new (std::nothrow) rs_solver();
    if (!s) return fail(RS_ENOMEM, "host allocation failed");
    s->g = g;
    s->nl = nl;
    s->vloc = vloc;
    s->nblk = (nstates + B - 1) / B;
    s->N = s->nblk * B;               // the last block is padded with zero states
    s->nreal = nstates;
    s->B = B;
    s->dtype = dtype;
    s->prec = dtype == RS_F64 ? RS_PREC_NATIVE : RS_PREC_BF16X3;
    rs_solver_opts o;
    o.m = 3;
    o.alpha = 0.52;
    o.tol = 1e-6;
    o.block_stop = 1;
    o.record = 0;
    o.rr_sweeps = 0;
    if (opts) o = *opts;
    if (o.m < 1 || o.m > kMaxIter) { delete s; return fail(RS_EINVAL, "rs_eigensolve_create: m must be 1..3"); }
    if (o.rr_sweeps < 0 || o.rr_sweeps > kMaxSweeps) {
        delete s;
        return fail(RS_EINVAL, "rs_eigensolve_create: rr_sweeps must be 0..30");
    }
    s->opts = o;
    s->rr_sweeps = o.rr_sweeps ? o.rr_sweeps : kMaxSweeps;
    rs_status st = rs_ctx_create(g, s->N, &s->ctx);
    if (st) { delete s; return st; }
    const size_t es = dtype == RS_F64 ? 8 : 4;
    s->field_bytes = (size_t)g->np * s->N * es;
    const int N = s->N;
    const int nchunks = rsred::chunk_count(g->np, B, s->nblk);
    st = s->h.alloc(s->field_bytes);
    if (!st) st = s->R.alloc(s->field_bytes);
    for (int i = 0; i < (o.m == 3 ? 2 : 1) && !st; ++i) {
        st = s->d[i].alloc(s->field_bytes);
        if (!st) st = s->hd[i].alloc(s->field_bytes);
    }
    if (!st) st = s->partial.alloc(sizeof(double) * 13 * (size_t)nchunks * N);
    if (!st) st = s->d2.alloc(sizeof(double) * 2 * N);
    if (!st) st = s->rr.alloc(sizeof(double) * N);
    if (!st) st = s->res.alloc(sizeof(double) * N);
    if (!st) st = s->eig.alloc(sizeof(double) * N);
    if (!st) st = s->lam.alloc(sizeof(double) * N);
    if (!st) st = s->eps.alloc(sizeof(double) * N);
    if (!st) st = s->stage.alloc(sizeof(double) * kStage * N);
    if (!st) st = s->lin.alloc(sizeof(double) * 5 * N);
    if (!st) st = s->upd.alloc(sizeof(double) * 3 * N);
    if (!st) st = s->active.alloc(sizeof(int) * N);
    if (!st) st = s->sigma.alloc(sizeof(double) * N);
    if (!st) st = s->d13.alloc(sizeof(double) * 13 * N);
    if (!st) st = s->mix.alloc(sizeof(double) * 2 * N);
    if (!st) st = s->bmap.alloc(sizeof(int) * s->nblk);
    // reductions over a subset of the blocks leave the other columns'
    // partial sums as they were: start them at zero
    if (!st && hipMemset(s->partial.p, 0, sizeof(double) * 13 * (size_t)nchunks * N) != hipSuccess)
        st = fail(RS_EHIP, "rs_eigensolve_create: clearing the reduction scratch failed");
    if (!st && o.record) st = s->R0.alloc(s->field_bytes);
    if (!st && hipHostMalloc(&s->pinned, sizeof(double) * 3 * N + sizeof(int) * (N + 2), hipHostMallocDefault) !=
                   hipSuccess) {
        s->pinned = nullptr;
        st = fail(RS_ENOMEM, "rs_eigensolve_create: pinned host allocation failed");
    }
    if (st) {
        rs_eigensolve_destroy(s);
        return st;
    }
    double *pd = static_cast<double *>(s->pinned);
    int *pi = reinterpret_cast<int *>(pd + 3 * N);
    s->report = StepReport{pd, pd + N, pd + 2 * N, pi, pi + N, pi + N + 1};
    *out = s;
    return RS_OK;
}

extern "C" void rs_eigensolve_destroy(rs_solver *s) {
    if (!s) return;
    rs_ctx_destroy(s->ctx);
    if (s->pinned) (void)hipHostFree(s->pinned);
    delete s;
}

namespace {

// d = K r for the DIIS iterations: the filter, or per state a K_f r + b K_n r
// with the trial step's coefficients (the network output goes to S->dn).
// The blocks a step's trial and DIIS passes run on: all of them, or, when
// the block stopping rule froze some, the others (map: their indices on the
// device, runs: contiguous ranges for the stencil and network calls, which
// take a first block and a count).
struct Blocks {
    const int *map = nullptr;
    int n = 0;
    std::vector<std::pair<int, int>> runs;
};

// d = K r on the listed blocks: the filter, and with a network its direction
// mixed in per state
template <typename T>
rs_status precond(rs_solver *S, const T *r, T *d, const Blocks &bs, hipStream_t st) {
    using namespace rs;
    const rs_grid *g = S->g;
    const int64_t bel = g->np * S->B;
    for (const auto &run : bs.runs) {
        const int64_t off = run.first * bel;
        rs_status e = filter_apply(g, S->opts.alpha, r + off, d + off, run.second, S->B, S->dtype, st);
        if (e) return e;
        if (S->cnn && (e = cnn_precondition(S->cnn, g, r + off, S->sigma.as<double>() + run.first * S->B,
                                            S->dn.as<T>() + off, run.second, S->B, S->dtype, st)))
            return e;
    }
    if (!S->cnn) return RS_OK;
    const dim3 gb((unsigned)((g->np * S->B + 255) / 256), bs.n);
    hipLaunchKernelGGL(mixdir_kernel<T>, gb, dim3(256), 0, st, d, S->dn.as<T>(), (T *)nullptr, (const T *)nullptr,
                       S->mix.as<double>(), g->np, S->B, S->N, bs.map);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// H applied to the listed blocks of x, with the kernel that all blocks would take
template <typename T>
rs_status hpsi_blocks(rs_solver *S, const T *x, T *hx, const Blocks &bs, hipStream_t st) {
    const int64_t bel = S->g->np * S->B;
    for (const auto &run : bs.runs) {
        const int64_t off = run.first * bel;
        rs_status e = rs::hpsi_apply(S->g, S->nl, S->vloc, x + off, hx + off, run.second, S->B, S->dtype, st,
                                      S->nblk);
        if (e) return e;
    }
    return RS_OK;
}

template <typename T>
rs_status step_impl(rs_solver *S, T *psi, hipStream_t st) {
    using namespace rs;
    const rs_grid *g = S->g;
    const int64_t np = g->np;
    const int B = S->B, nblk = S->nblk, N = S->N, m = S->opts.m;
    const double dv = g->h * g->h * g->h;
    const unsigned gs = (unsigned)((N + 63) / 64);
    T *h0 = S->h.as<T>(), *R = S->R.as<T>(), *d1 = S->d[0].as<T>(), *hd1 = S->hd[0].as<T>();
    double *partial = S->partial.as<double>();
    rs_status e;
    // 1. H psi, Rayleigh-Ritz
    if ((e = hpsi_apply(g, S->nl, S->vloc, psi, h0, nblk, B, S->dtype, st, nblk))) return e;
    if ((e = subspace_diag_capped(S->ctx, psi, h0, S->eig.as<double>(), nblk, B, S->dtype, S->prec, S->rr_sweeps,
                                  S->nreal, st)))
        return e;
    // shifts for the learned preconditioner: sigma = -<psi|T psi>
    if (S->cnn || S->opts.record) {
        if ((e = kinetic_apply(g, psi, d1, nblk, B, S->dtype, st))) return e;
        if ((e = colreduce<2>(OpDots2<T>{psi, d1}, np, B, nblk, dv, partial, S->d2.as<double>(), st)))
            return e;
        hipLaunchKernelGGL(sigma_kernel, dim3(gs), dim3(64), 0, st, S->d2.as<double>(), N, S->sigma.as<double>());
    }
    // 2. eps0, residual, activity
    double *eps = S->eps.as<double>(), *rr = S->rr.as<double>(), *d2 = S->d2.as<double>();
    if ((e = colreduce_then<2>(OpDots2<T>{psi, h0}, np, B, nblk, dv, partial, Eps0{d2, eps, N}, st))) return e;
    if ((e = colreduce<1>(OpResid<T>{psi, h0, R, eps}, np, B, nblk, dv, partial, rr, st))) return e;
    hipLaunchKernelGGL(active_kernel, dim3(gs), dim3(64), 0, st, S->rr.as<double>(), N, B, S->opts.tol,
                       S->opts.block_stop, S->res.as<double>(), S->active.as<int>(), S->report.active);
    RS_HIP(hipGetLastError());
    if (S->opts.record) RS_HIP(hipMemcpyAsync(S->R0.p, S->R.p, S->field_bytes, hipMemcpyDeviceToDevice, st));
    // Block stopping rule (Sec. 9): the trial step and the DIIS iterations
    // run only on blocks with a state above tolerance; frozen blocks keep
    // psi.  Reading the flags costs one wait on the stream per step, taken
    // only when a block can freeze (block_stop and tol > 0).
    Blocks bs;
    bs.n = nblk;
    bs.runs.assign(1, {0, nblk});
    if (S->opts.block_stop && S->opts.tol > 0.0) {
        RS_HIP(hipStreamSynchronize(st));
        S->host_map.clear();
        for (int b = 0; b < nblk; ++b)
            if (S->report.active[(size_t)b * B]) S->host_map.push_back(b);
        if (S->host_map.empty()) {
            // every block frozen: psi stays; no state mixed a network direction
            if (S->cnn) RS_HIP(hipMemsetAsync(S->mix.p, 0, sizeof(double) * 2 * N, st));
            return RS_OK;
        }
        if ((int)S->host_map.size() < nblk) {
            RS_HIP(hipMemcpyAsync(S->bmap.p, S->host_map.data(), sizeof(int) * S->host_map.size(),
                                  hipMemcpyHostToDevice, st));
            bs.map = S->bmap.as<int>();
            bs.n = (int)S->host_map.size();
            bs.runs.clear();
            for (int i = 0; i < bs.n; ++i) {
                if (i > 0 && S->host_map[i] == S->host_map[i - 1] + 1) ++bs.runs.back().second;
                else bs.runs.push_back({S->host_map[i], 1});
            }
        }
    }
    // 3. trial step
    for (const auto &run : bs.runs) {
        const int64_t off = run.first * np * B;
        if ((e = filter_apply(g, S->opts.alpha, R + off, d1 + off, run.second, B, S->dtype, st, nullptr))) return e;
    }
    if ((e = hpsi_blocks<T>(S, d1, hd1, bs, st))) return e;
    if (S->cnn) {
        // the network's direction and the 3x3 trial problem; the mixed
        // direction replaces d (and H d) for the states that use it
        for (const auto &run : bs.runs) {
            const int64_t off = run.first * np * B;
            if ((e = cnn_precondition(S->cnn, g, R + off, S->sigma.as<double>() + run.first * B,
                                      S->dn.as<T>() + off, run.second, B, S->dtype, st)))
                return e;
        }
        if ((e = hpsi_blocks<T>(S, S->dn.as<T>(), S->hdn.as<T>(), bs, st))) return e;
        if ((e = colreduce<13>(OpLam3<T>{psi, h0, d1, hd1, S->dn.as<T>(), S->hdn.as<T>()}, np, B, nblk, dv, partial,
                               S->d13.as<double>(), st, bs.map, bs.n)))
            return e;
        hipLaunchKernelGGL(mix_kernel, dim3(gs), dim3(64), 0, st, d2, S->d13.as<double>(), S->active.as<int>(), N,
                           S->lam.as<double>(), S->mix.as<double>());
        hipLaunchKernelGGL(mixdir_kernel<T>, dim3((unsigned)((np * B + 255) / 256), bs.n), dim3(256), 0, st, d1,
                           S->dn.as<T>(), hd1, S->hdn.as<T>(), S->mix.as<double>(), np, B, N, bs.map);
        RS_HIP(hipGetLastError());
    }
    double *stage = S->stage.as<double>(), *lin = S->lin.as<double>(), *upd = S->upd.as<double>();
    const dim3 ga = map_grid(np, B, bs.n);
    if ((e = colreduce_then<8>(OpGram1<T>{psi, R, d1, hd1, eps}, np, B, nblk, dv, partial,
                               Solve1{d2, rr, eps, S->cnn ? S->lam.as<double>() : nullptr, S->active.as<int>(), stage,
                                      lin, upd, N, m},
                               st, bs.map, bs.n)))
        return e;
    if (m == 1) {
        // the trial iterate is the newest: straight into psi
        hipLaunchKernelGGL(update_kernel<T>, ga, dim3(256), 0, st, psi, (const T *)nullptr, (const T *)nullptr, d1,
                           upd, np, B, N, bs.map);
        RS_HIP(hipGetLastError());
        return RS_OK;
    }
    // 4. DIIS: R_bar (over H psi, which nothing reads any more)
    T *rb = h0, *d2f = nullptr, *dl = hd1;
    hipLaunchKernelGGL(residual_mix_kernel<T>, ga, dim3(256), 0, st, psi, R, d1, hd1, (const T *)nullptr,
                       (const T *)nullptr, lin, rb, np, B, N, bs.map);
    RS_HIP(hipGetLastError());
    if (m == 3) {
        T *hd2 = S->hd[1].as<T>();
        d2f = S->d[1].as<T>();
        dl = hd2;
        if ((e = precond<T>(S, rb, d2f, bs, st))) return e;
        if ((e = hpsi_blocks<T>(S, d2f, hd2, bs, st))) return e;
        if ((e = colreduce_then<11>(OpGram2<T>{psi, R, d1, hd1, d2f, hd2, eps}, np, B, nblk, dv, partial,
                                    Solve2{d2, rr, eps, stage, lin, upd, N}, st, bs.map, bs.n)))
            return e;
        hipLaunchKernelGGL(residual_mix_kernel<T>, ga, dim3(256), 0, st, psi, R, d1, hd1, d2f, hd2, lin, rb, np, B, N,
                           bs.map);
        RS_HIP(hipGetLastError());
    }
    // the newest iterate, straight into psi: formed by the filter, or with a
    // network after its direction (which goes where H d is no longer read)
    if (S->cnn) {
        if ((e = precond<T>(S, rb, dl, bs, st))) return e;
        hipLaunchKernelGGL(update_kernel<T>, ga, dim3(256), 0, st, psi, d1, d2f, dl, upd, np, B, N, bs.map);
        RS_HIP(hipGetLastError());
        return RS_OK;
    }
    for (const auto &run : bs.runs) {
        const int64_t off = run.first * np * B;
        const FilterUpdate u{psi + off, d1 + off, d2f ? d2f + off : nullptr, upd + run.first * B, N};
        if ((e = filter_apply(g, S->opts.alpha, rb + off, psi + off, run.second, B, S->dtype, st, &u))) return e;
    }
    return RS_OK;
}

}  // namespace

extern "C" rs_status rs_eigensolve_step(rs_solver *s, void *psi, double *eig, double *resnorm, int32_t *nconv,
                                        void *stream) {
    using namespace rs;
    if (!s || !psi) return fail(RS_EINVAL, "rs_eigensolve_step: null argument");
    hipStream_t st = (hipStream_t)stream;
    rs_status e = s->dtype == RS_F64 ? step_impl<double>(s, (double *)psi, st) : step_impl<float>(s, (float *)psi, st);
    if (e) return e;
    if ((e = orthonormalize_async(s->ctx, psi, s->nblk, s->B, s->dtype, s->prec, nullptr, s->nreal, st))) return e;
    hipLaunchKernelGGL(report_kernel, dim3((unsigned)((s->N + 63) / 64)), dim3(64), 0, st, s->report,
                       s->eig.as<double>(), s->res.as<double>(), s->cnn ? s->mix.as<double>() + s->N : nullptr,
                       ctx_sweeps(s->ctx), ctx_info(s->ctx), s->N);
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(st));
    const int n = s->nreal;
    const double *ev = s->report.eig, *rn = s->report.res;
    e = orthonormalize_status(*s->report.info);
    s->stats.rr_sweeps = *s->report.sweeps;
    s->stats.frozen_blocks = 0;
    for (int b = 0; b < s->nblk; ++b) s->stats.frozen_blocks += s->report.active[(size_t)b * s->B] == 0;
    s->stats.net_states = 0;
    if (s->cnn)
        for (int k = 0; k < n; ++k) s->stats.net_states += s->report.mix[k] != 0.0;
    if (eig) std::memcpy(eig, ev, sizeof(double) * n);
    if (resnorm) std::memcpy(resnorm, rn, sizeof(double) * n);
    int c = 0;
    for (int k = 0; k < n; ++k) c += rn[k] < s->opts.tol;
    if (nconv) *nconv = c;
    for (int k = 0; k < n; ++k)
        if (!std::isfinite(ev[k]) || !std::isfinite(rn[k]))
            return fail(RS_ENONFINITE, "rs_eigensolve_step: non-finite eigenvalue or residual");
    s->steps++;
    s->stats.steps = s->steps;
    return e;
}

extern "C" rs_status rs_eigensolve_stats(const rs_solver *s, rs_solver_stats *out) {
    if (!s || !out) return rs::fail(RS_EINVAL, "rs_eigensolve_stats: null argument");
    *out = s->stats;
    return RS_OK;
}

extern "C" rs_status rs_eigensolve_set_precond(rs_solver *s, rs_cnn *c) {
    if (!s) return rs::fail(RS_EINVAL, "rs_eigensolve_set_precond: null solver");
    if (c && !s->dn.p) {
        rs_status st = s->dn.alloc(s->field_bytes);
        if (!st) st = s->hdn.alloc(s->field_bytes);
        if (st) return st;
    }
    s->cnn = c;
    return RS_OK;
}

extern "C" rs_status rs_eigensolve_residuals(rs_solver *s, void *R, double *sigma, void *stream) {
    if (!s || !R || !sigma) return rs::fail(RS_EINVAL, "rs_eigensolve_residuals: null argument");
    if (!s->opts.record) return rs::fail(RS_EINVAL, "rs_eigensolve_residuals: the solver was created without record");
    if (s->steps == 0) return rs::fail(RS_EINVAL, "rs_eigensolve_residuals: no step taken yet");
    hipStream_t st = (hipStream_t)stream;
    RS_HIP(hipMemcpyAsync(R, s->R0.p, s->field_bytes, hipMemcpyDeviceToDevice, st));
    RS_HIP(hipMemcpyAsync(sigma, s->sigma.p, sizeof(double) * s->N, hipMemcpyDeviceToDevice, st));
    return RS_OK;
}

extern "C" rs_status rs_eigensolve_orthonormalize(rs_solver *s, void *psi, void *stream) {
    if (!s || !psi) return rs::fail(RS_EINVAL, "rs_eigensolve_orthonormalize: null argument");
    int32_t info = 0;
    return orthonormalize_impl(s->ctx, psi, s->nblk, s->B, s->dtype, s->prec, nullptr, &info, s->nreal,
                               (hipStream_t)stream);
}
