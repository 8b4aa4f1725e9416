// Hartree potential by FFT on an enlarged cubic box (Sec. 7, eq. (5)).
//
// The density on the domain's points is placed in an N^3 box (zeros
// elsewhere), transformed by a 3-D complex FFT, multiplied by the Coulomb
// interaction cut off at R_c,
//     v(k) = 4 pi / k^2 (1 - cos(k R_c)),  v(0) = 2 pi R_c^2,
// transformed back and read out at the domain's points.  R_c bounds every
// pair distance in the domain and the box is longer than the domain's span
// plus R_c on every axis, so no periodic image of the density comes within
// R_c of a domain point: on the domain the result is the free-space
// potential int n(r') / |r - r'| d^3r'.
//
// The density is real and fills only ex x ey x ez of the N^3 points, and the
// potential is wanted only there, so the transforms skip everything else:
//   1. x, forward: ex real values of each of the ey ez lines (two lines as
//      one complex line) -> half spectra, kx <= N/2            [ez][ey][kx]
//   2. y, forward: ey values -> N                              [ez][N][kx]
//   3. z: ez values -> N, times v(k) / N^3, and back -> ez     [ez][N][kx]
//   4. y, inverse: N -> ey values                              [ez][ey][kx]
//   5. x, inverse: half spectra -> ex real values, to the points
// For the 904k-point sphere (121^3 points in a 256^3 box) the five passes
// read and write 0.38 GB, which the 256 MB last-level cache holds most of,
// instead of the 3.2 GB of six complex passes over the whole box (radix 2
// in LDS), two elementwise passes, the clearing and the scatter: 109 us a
// solve (x 13 + 14, y 18 + 19, z 40) instead of 832.
// A line is transformed by N / E threads holding E values each: passes of
// radix up to 16 in registers (Stockham order, so the output is in natural
// order), exchanged through LDS between passes; the first pass takes its
// input from global memory and the last one leaves value j + e N/E in
// register e, just where the next transform's first pass wants it.
#include <cmath>
#include <vector>

#include "internal.hpp"

namespace {

typedef double2 cplx;

constexpr int kPoissonMinN = 16, kPoissonMaxN = 512;

__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
    return cplx{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}

__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return cplx{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return cplx{a.x - b.x, a.y - b.y}; }

// Forward transforms of R values in registers, natural order.
template <int R> __device__ __forceinline__ void dft(cplx (&v)[R]);
template <> __device__ __forceinline__ void dft<2>(cplx (&v)[2]) {
    const cplx a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}
template <> __device__ __forceinline__ void dft<4>(cplx (&v)[4]) {
    const cplx a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = csub(v[1], v[3]);
    v[0] = cadd(a, c);
    v[1] = cplx{b.x + d.y, b.y - d.x};
    v[2] = csub(a, c);
    v[3] = cplx{b.x - d.y, b.y + d.x};
}
constexpr double kR2 = 0.70710678118654752440, kC16 = 0.92387953251128675613, kS16 = 0.38268343236508977173;
template <> __device__ __forceinline__ void dft<8>(cplx (&v)[8]) {
    cplx e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft<4>(e);
    dft<4>(o);
    o[1] = cplx{kR2 * (o[1].x + o[1].y), kR2 * (o[1].y - o[1].x)};
    o[2] = cplx{o[2].y, -o[2].x};
    o[3] = cplx{kR2 * (o[3].y - o[3].x), -kR2 * (o[3].x + o[3].y)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = cadd(e[k], o[k]);
        v[k + 4] = csub(e[k], o[k]);
    }
}
// n = n1 + 4 n2, k = k2 + 4 k1
template <> __device__ __forceinline__ void dft<16>(cplx (&v)[16]) {
    constexpr cplx w[10] = {{1, 0}, {kC16, -kS16}, {kR2, -kR2}, {kS16, -kC16}, {0, -1}, {0, 0}, {-kR2, -kR2},
                            {0, 0}, {0, 0}, {-kC16, kS16}};   // exp(-2 pi i k / 16)
    cplx t[4][4];
#pragma unroll
    for (int n1 = 0; n1 < 4; ++n1) {
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) t[n1][n2] = v[n1 + 4 * n2];
        dft<4>(t[n1]);
    }
#pragma unroll
    for (int n1 = 1; n1 < 4; ++n1)
#pragma unroll
        for (int k2 = 1; k2 < 4; ++k2) t[n1][k2] = cmul(w[n1 * k2], t[n1][k2]);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) {
        cplx u[4] = {t[0][k2], t[1][k2], t[2][k2], t[3][k2]};
        dft<4>(u);
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) v[k2 + 4 * k1] = u[k1];
    }
}

// The radices of a length: the first and the last are E, the values per
// thread, so that a transform's output registers are the next one's input;
// three passes have M in the middle (M = 1: two passes).
template <int N> struct Plan;
template <> struct Plan<16> { static constexpr int E = 4, M = 1; };
template <> struct Plan<32> { static constexpr int E = 4, M = 2; };
template <> struct Plan<64> { static constexpr int E = 8, M = 1; };
template <> struct Plan<128> { static constexpr int E = 8, M = 2; };
template <> struct Plan<256> { static constexpr int E = 16, M = 1; };
template <> struct Plan<512> { static constexpr int E = 8, M = 8; };

constexpr int kLines = 8;   // lines per work-group: 128 bytes of neighbouring kx

// One pass of radix R with NS points already transformed: butterfly q of the
// thread takes registers q + r E/R (values j + (q + r E/R) N/E), times
// exp(-2 pi i (b % NS) r / (NS R)), b = j + q N/E.
template <int N, int R, int NS>
__device__ __forceinline__ void radix_pass(cplx (&v)[Plan<N>::E], int j, const cplx *__restrict__ tw) {
    constexpr int E = Plan<N>::E, T = N / E, Q = E / R;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        cplx u[R];
        const int p = (j + q * T) % NS * (N / (NS * R));
#pragma unroll
        for (int r = 0; r < R; ++r) u[r] = NS > 1 && r > 0 ? cmul(tw[p * r], v[q + r * Q]) : v[q + r * Q];
        dft<R>(u);
#pragma unroll
        for (int r = 0; r < R; ++r) v[q + r * Q] = u[r];
    }
}

// LDS place of value pos of a line.  Lines fastest: 8 lanes cover 128
// contiguous bytes.  Values fastest: one value of padding per E, so that the
// first exchange's stride of E values spreads over the banks.
template <int N, bool LINES>
__device__ __forceinline__ int place(int line, int pos) {
    constexpr int E = Plan<N>::E;
    return LINES ? pos * kLines + line : line * (N + N / E) + pos + pos / E;
}
template <int N> constexpr int lds_values() { return kLines * (N + N / Plan<N>::E); }

template <int N, int R, int NS, bool LINES>
__device__ __forceinline__ void exchange(cplx (&v)[Plan<N>::E], int j, int line, cplx *buf) {
    constexpr int E = Plan<N>::E, T = N / E, Q = E / R;
    __syncthreads();   // earlier reads of the buffer are done
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = j + q * T;
#pragma unroll
        for (int r = 0; r < R; ++r) buf[place<N, LINES>(line, b / NS * (NS * R) + b % NS + r * NS)] = v[q + r * Q];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = buf[place<N, LINES>(line, j + e * T)];
}

// Forward transform of the line whose values j + e N/E this thread holds in
// v[e]; in place.  An inverse one is the same with real and imaginary parts
// swapped before and after.
template <int N, bool LINES>
__device__ __forceinline__ void fft(cplx (&v)[Plan<N>::E], int j, int line, cplx *buf, const cplx *__restrict__ tw) {
    constexpr int E = Plan<N>::E, M = Plan<N>::M;
    radix_pass<N, E, 1>(v, j, tw);
    exchange<N, E, 1, LINES>(v, j, line, buf);
    if constexpr (M > 1) {
        radix_pass<N, M, E>(v, j, tw);
        exchange<N, M, E, LINES>(v, j, line, buf);
    }
    radix_pass<N, E, N / E>(v, j, tw);
}
template <int E> __device__ __forceinline__ void swap_parts(cplx (&v)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = cplx{v[e].y, v[e].x};
}

// The domain's place in the box: ex x ey x ez points, half spectra of nk =
// N/2 + 1 values in rows of pitch values; map[z][y][x] is the point's number
// or -1 outside the domain.
struct Extent {
    int ex, ey, ez, nk, pitch;
};

// x, forward: 16 neighbouring lines of one z as 8 complex lines, Z = A + i B;
// A_k = (Z_k + conj Z_-k) / 2, B_k = (Z_k - conj Z_-k) / 2i.
template <int N>
__global__ void __launch_bounds__(kLines *N / Plan<N>::E)
x_forward_kernel(const double *__restrict__ rho, const int32_t *__restrict__ map, Extent d,
                 const cplx *__restrict__ tw, cplx *__restrict__ out) {
    constexpr int E = Plan<N>::E, T = N / E;
    __shared__ cplx buf[lds_values<N>()];
    const int j = threadIdx.x % T, line = threadIdx.x / T;
    const int y = 2 * (blockIdx.x * kLines + line);
    const int64_t row = (int64_t)blockIdx.y * d.ey + y;
    const bool ok0 = y < d.ey, ok1 = y + 1 < d.ey;
    cplx v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = j + e * T;
        const int a = ok0 && x < d.ex ? map[row * d.ex + x] : -1, b = ok1 && x < d.ex ? map[(row + 1) * d.ex + x] : -1;
        v[e] = cplx{a >= 0 ? rho[a] : 0.0, b >= 0 ? rho[b] : 0.0};
    }
    fft<N, false>(v, j, line, buf, tw);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) buf[place<N, false>(line, j + e * T)] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e <= E / 2; ++e) {
        const int k = j + e * T;
        if (k > N / 2) continue;
        const cplx z = v[e], c = buf[place<N, false>(line, (N - k) % N)];
        if (ok0) out[row * d.pitch + k] = cplx{0.5 * (z.x + c.x), 0.5 * (z.y - c.y)};
        if (ok1) out[(row + 1) * d.pitch + k] = cplx{0.5 * (z.y + c.y), 0.5 * (c.x - z.x)};
    }
}

// x, inverse: the same lines back, Z_k = A_k + i B_k with A_-k = conj A_k.
template <int N>
__global__ void __launch_bounds__(kLines *N / Plan<N>::E)
x_inverse_kernel(const cplx *__restrict__ in, const int32_t *__restrict__ map, Extent d, const cplx *__restrict__ tw,
                 double *__restrict__ vh) {
    constexpr int E = Plan<N>::E, T = N / E;
    __shared__ cplx buf[lds_values<N>()];
    const int j = threadIdx.x % T, line = threadIdx.x / T;
    const int y = 2 * (blockIdx.x * kLines + line);
    const int64_t row = (int64_t)blockIdx.y * d.ey + y;
    const bool ok0 = y < d.ey, ok1 = y + 1 < d.ey;
    cplx v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = j + e * T, kk = k > N / 2 ? N - k : k;
        cplx a{0.0, 0.0}, b{0.0, 0.0};
        if (ok0) a = in[row * d.pitch + kk];
        if (ok1) b = in[(row + 1) * d.pitch + kk];
        // A + i B (conjugated parts past N/2), real and imaginary swapped
        v[e] = k > N / 2 ? cplx{b.x - a.y, a.x + b.y} : cplx{a.y + b.x, a.x - b.y};
    }
    fft<N, false>(v, j, line, buf, tw);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = j + e * T;
        if (x >= d.ex) continue;
        const int a = ok0 ? map[row * d.ex + x] : -1, b = ok1 ? map[(row + 1) * d.ex + x] : -1;
        if (a >= 0) vh[a] = v[e].y;
        if (b >= 0) vh[b] = v[e].x;
    }
}

// y: 8 neighbouring kx of one z, between ey values (near) and N (far).
template <int N, bool INVERSE>
__global__ void __launch_bounds__(kLines *N / Plan<N>::E)
y_kernel(cplx *__restrict__ near, cplx *__restrict__ far, Extent d, const cplx *__restrict__ tw) {
    constexpr int E = Plan<N>::E, T = N / E;
    __shared__ cplx buf[kLines * N];
    const int line = threadIdx.x % kLines, j = threadIdx.x / kLines;
    const int k = blockIdx.x * kLines + line;
    const bool ok = k < d.nk;
    cplx *pn = near + (int64_t)blockIdx.y * d.ey * d.pitch + k, *pf = far + (int64_t)blockIdx.y * N * d.pitch + k;
    cplx v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int y = j + e * T;
        v[e] = cplx{0.0, 0.0};
        if (INVERSE ? ok : ok && y < d.ey) v[e] = INVERSE ? pf[(int64_t)y * d.pitch] : pn[(int64_t)y * d.pitch];
    }
    if constexpr (INVERSE) swap_parts(v);
    fft<N, true>(v, j, line, buf, tw);
    if constexpr (INVERSE) swap_parts(v);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int y = j + e * T;
        if constexpr (INVERSE) {
            if (ok && y < d.ey) pn[(int64_t)y * d.pitch] = v[e];
        } else {
            if (ok) pf[(int64_t)y * d.pitch] = v[e];
        }
    }
}

// z: 8 neighbouring kx of one ky; ez values to N, times the Coulomb kernel
// (kern [|kz|][|ky|][kx], with the 1/N^3), and back, in place.
template <int N>
__global__ void __launch_bounds__(kLines *N / Plan<N>::E)
z_kernel(cplx *__restrict__ data, Extent d, const double *__restrict__ kern, const cplx *__restrict__ tw) {
    constexpr int E = Plan<N>::E, T = N / E;
    __shared__ cplx buf[kLines * N];
    const int line = threadIdx.x % kLines, j = threadIdx.x / kLines;
    const int k = blockIdx.x * kLines + line, ky = blockIdx.y;
    const bool ok = k < d.nk;
    cplx *p = data + (int64_t)ky * d.pitch + k;
    const int64_t step = (int64_t)N * d.pitch;
    const double *kr = kern + (int64_t)min(ky, N - ky) * d.pitch + k;
    cplx v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int z = j + e * T;
        v[e] = cplx{0.0, 0.0};
        if (ok && z < d.ez) v[e] = p[z * step];
    }
    fft<N, true>(v, j, line, buf, tw);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int kz = j + e * T;
        const double f = ok ? kr[(int64_t)min(kz, N - kz) * (N / 2 + 1) * d.pitch] : 0.0;
        v[e] = cplx{v[e].y * f, v[e].x * f};
    }
    fft<N, true>(v, j, line, buf, tw);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int z = j + e * T;
        if (ok && z < d.ez) p[z * step] = cplx{v[e].y, v[e].x};
    }
}

// kern[z][y][x] = v(k) / N^3, k = 2 pi (x, y, z) / (N h), 0 <= x, y, z <= N/2
// (v is even in every component).
__global__ void __launch_bounds__(256)
coulomb_kernel(double *__restrict__ kern, int n, int pitch, double dk, double rc, double scale) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t h = n / 2 + 1;
    if (e >= h * h * pitch) return;
    const int x = (int)(e % pitch), y = (int)((e / pitch) % h), z = (int)(e / (pitch * h));
    const double kx = x * dk, ky = y * dk, kz = z * dk;
    const double k2 = (kx * kx + ky * ky) + kz * kz;
    double vk = 2.0 * M_PI * rc * rc;
    if (k2 > 0.0) {
        const double k = sqrt(k2);
        vk = 4.0 * M_PI / k2 * (1.0 - cos(k * rc));
    }
    kern[e] = vk * scale;
}

}  // namespace

struct rs_poisson {
    const rs_grid *g = nullptr;
    int n = 0;
    double rc = 0.0;
    Extent d{};
    rs::DevBuf near;   // complex double [ez][ey][pitch]
    rs::DevBuf far;    // complex double [ez][n][pitch]
    rs::DevBuf kern;   // double [n/2+1][n/2+1][pitch]: v(k) / n^3
    rs::DevBuf map;    // int32 [ez][ey][ex]: inner point or -1
    rs::DevBuf tw;     // complex double [n]: exp(-2 pi i k / n)
};

namespace {

template <int N>
rs_status solve(const rs_poisson *p, const double *rho, double *vh, hipStream_t st) {
    const Extent &d = p->d;
    const dim3 wg(kLines * N / Plan<N>::E);
    const dim3 gx((d.ey + 2 * kLines - 1) / (2 * kLines), d.ez), gy((d.nk + kLines - 1) / kLines, d.ez),
        gz((d.nk + kLines - 1) / kLines, N);
    cplx *near = p->near.as<cplx>(), *far = p->far.as<cplx>();
    const cplx *tw = p->tw.as<cplx>();
    const int32_t *map = p->map.as<int32_t>();
    hipLaunchKernelGGL((x_forward_kernel<N>), gx, wg, 0, st, rho, map, d, tw, near);
    RS_HIP(hipGetLastError());
    hipLaunchKernelGGL((y_kernel<N, false>), gy, wg, 0, st, near, far, d, tw);
    RS_HIP(hipGetLastError());
    hipLaunchKernelGGL((z_kernel<N>), gz, wg, 0, st, far, d, p->kern.as<double>(), tw);
    RS_HIP(hipGetLastError());
    hipLaunchKernelGGL((y_kernel<N, true>), gy, wg, 0, st, near, far, d, tw);
    RS_HIP(hipGetLastError());
    hipLaunchKernelGGL((x_inverse_kernel<N>), gx, wg, 0, st, near, map, d, tw, vh);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

}  // namespace

extern "C" rs_status rs_poisson_create(const rs_grid *g, rs_poisson **out) {
    using rs::fail;
    if (!g || !out) return fail(RS_EINVAL, "rs_poisson_create: null argument");
    *out = nullptr;
    if (g->host_only) return fail(RS_EINVAL, "rs_poisson_create: host-only grid");
    if (g->kind == RS_GRID_PERIODIC) return fail(RS_EINVAL, "rs_poisson_create: the free-boundary solve is for finite systems");
    if (g->np < 1) return fail(RS_EINVAL, "rs_poisson_create: empty grid");
    int32_t lo[3], hi[3];
    for (int a = 0; a < 3; ++a) { lo[a] = g->inner[a]; hi[a] = g->inner[a]; }
    for (int64_t p = 1; p < g->np; ++p)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], g->inner[3 * p + a]);
            hi[a] = std::max(hi[a], g->inner[3 * p + a]);
        }
    // R_c: twice the largest distance from the bounding box's centre
    double m = 0.0;
    for (int64_t p = 0; p < g->np; ++p) {
        double s = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double d = (double)g->inner[3 * p + a] - 0.5 * ((double)lo[a] + (double)hi[a]);
            s += d * d;
        }
        m = std::max(m, s);
    }
    const double rc = (2.0 * g->h) * std::sqrt(m);
    int ext = 0;
    for (int a = 0; a < 3; ++a) ext = std::max(ext, hi[a] - lo[a] + 1);
    int n = 2;
    while (!((double)n > (double)(ext - 1) + rc / g->h)) n *= 2;
    if (n < kPoissonMinN) n = kPoissonMinN;
    if (n > kPoissonMaxN) return fail(RS_ENOTSUP, "rs_poisson_create: the domain needs an FFT box above 512^3");
    auto p = new (std::nothrow) rs_poisson();
    if (!p) return fail(RS_ENOMEM, "host allocation failed");
    p->g = g;
    p->n = n;
    p->rc = rc;
    Extent &d = p->d;
    d.ex = hi[0] - lo[0] + 1;
    d.ey = hi[1] - lo[1] + 1;
    d.ez = hi[2] - lo[2] + 1;
    d.nk = n / 2 + 1;
    d.pitch = (d.nk + kLines - 1) / kLines * kLines;
    std::vector<int32_t> map((size_t)d.ex * d.ey * d.ez, -1);
    for (int64_t q = 0; q < g->np; ++q) {
        const int64_t x = g->inner[3 * q] - lo[0], y = g->inner[3 * q + 1] - lo[1], z = g->inner[3 * q + 2] - lo[2];
        map[(z * d.ey + y) * d.ex + x] = (int32_t)q;
    }
    std::vector<cplx> tw(n);
    for (int k = 0; k < n; ++k) {
        const double a = -2.0 * M_PI * (double)k / (double)n;
        tw[k] = cplx{std::cos(a), std::sin(a)};
    }
    const int64_t nkern = (int64_t)d.nk * d.nk * d.pitch;
    rs_status s = p->near.alloc((size_t)d.ez * d.ey * d.pitch * sizeof(cplx));
    if (!s) s = p->far.alloc((size_t)d.ez * n * d.pitch * sizeof(cplx));
    if (!s) s = p->kern.alloc((size_t)nkern * sizeof(double));
    if (!s) s = p->map.upload(map);
    if (!s) s = p->tw.upload(tw);
    if (s) { delete p; return s; }
    const double dk = 2.0 * M_PI * (1.0 / ((double)n * g->h));
    hipLaunchKernelGGL(coulomb_kernel, dim3((unsigned)((nkern + 255) / 256)), dim3(256), 0, (hipStream_t)0,
                       p->kern.as<double>(), n, d.pitch, dk, rc, 1.0 / ((double)n * n * n));
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)0);   // before a call on any other stream
    if (e != hipSuccess) { delete p; return rs::hip_fail(e, "rs_poisson_create: kernel table"); }
    *out = p;
    return RS_OK;
}

extern "C" void rs_poisson_destroy(rs_poisson *p) { delete p; }

extern "C" rs_status rs_poisson_info(const rs_poisson *p, int32_t *nbox, double *rc) {
    if (!p) return rs::fail(RS_EINVAL, "rs_poisson_info: null handle");
    if (nbox) *nbox = p->n;
    if (rc) *rc = p->rc;
    return RS_OK;
}

extern "C" rs_status rs_poisson_solve(rs_poisson *p, const double *rho, double *vh, void *stream) {
    using namespace rs;
    if (!p || !rho || !vh) return fail(RS_EINVAL, "rs_poisson_solve: null argument");
    hipStream_t st = (hipStream_t)stream;
    switch (p->n) {
        case 16: return solve<16>(p, rho, vh, st);
        case 32: return solve<32>(p, rho, vh, st);
        case 64: return solve<64>(p, rho, vh, st);
        case 128: return solve<128>(p, rho, vh, st);
        case 256: return solve<256>(p, rho, vh, st);
        case 512: return solve<512>(p, rho, vh, st);
    }
    return fail(RS_ENOTSUP, "poisson: FFT box edge must be a power of two in [16, 512]");
}
