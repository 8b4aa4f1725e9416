// Learned preconditioner for the RMM-DIIS step, and the shifted-kinetic
// solves that produce its training targets.
//
// The paper leaves the eigensolver's preconditioner open (Sec. 3 uses a
// filter); this is the project's learned replacement.  Network f: three
// 3x3x3 cross-correlation layers without bias, channels 1 -> 8 -> 8 -> 1,
// tanh after the first two, every layer's output zeroed off the domain.
// Preconditioner: K(r) = s g(sigma) f(r / s), s the rms of r over the grid
// points, g = softplus(a + b log(-sigma h^2)).  Targets: x = (T - sigma)^-1 r
// by conjugate gradients with the 25-point kinetic stencil (Sec. 5.1).
//
// Network fields are dense boxes, channels last: [n][Z][Y][X][C], FP32.  On
// a grid the box is the smallest axis-aligned box holding every point, zero
// outside the domain (periodic grids wrap).  Parameters are one FP32 vector:
// w1 [8][1][27], w2 [8][8][27], w3 [1][8][27] (tap t = 9 dz + 3 dy + dx,
// input offset (dx-1, dy-1, dz-1)), then a, b.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "colreduce.hpp"
#include "internal.hpp"

namespace rs {
rs_status kinetic_apply(const rs_grid *g, const void *psi, void *out, int nblk, int B, int dtype,
                        hipStream_t st);
}

namespace {
using namespace rsred;

constexpr int kW1 = 0, kW2 = 216, kW3 = 1944, kNW = 2160, kNP = 2162;
constexpr int kWgPts = 2048;   // points per work-group in the weight gradients, about

__device__ __forceinline__ int wrap_or_flag(int v, int n, bool wrap, bool &ok) {
    if (wrap) return v < 0 ? v + n : (v >= n ? v - n : v);
    ok = ok && v >= 0 && v < n;
    return v;
}

// ------------------------------------------------------------ convolution
// Taps outside the box are zero (or wrap); W is [CO][CI][27].
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

// x = hi + lo in bfloat16, each rounded to nearest even.
__device__ __forceinline__ void split(f4 x, bf4 &hi, bf4 &lo) {
    hi = __builtin_convertvector(x, bf4);
    lo = __builtin_convertvector(x - __builtin_convertvector(hi, f4), bf4);
}

// tanh without a branch: an odd polynomial (weighted least squares, 1e-9 of
// x) below 0.95 and 1 - 2 / (e^2x + 1) with the hardware's exponential and
// reciprocal above.  Against FP64 over -20 .. 20 and down to 2^-20 it errs by
// 1.38 units in the last place at most and 0.265 rms; the library's tanhf, whose two
// branches both run in nearly every wave here, by 1.40 and 0.267.
__device__ __forceinline__ float tanh_f(float x) {
    const float a = fabsf(x), s = x * x;
    float p = fmaf(s, -0x1.ac83ccp-12f, 0x1.41d0d2p-9f);
    p = fmaf(s, p, -0x1.0a65b2p-7f);
    p = fmaf(s, p, 0x1.61cbd4p-6f);
    p = fmaf(s, p, -0x1.b9a448p-5f);
    p = fmaf(s, p, 0x1.110e1ap-3f);
    p = fmaf(s, p, -0x1.555548p-2f);
    const float lo = fmaf(a * s, p, a);
    const float e = __builtin_amdgcn_exp2f(a * 2.88539008f);   // 2 log2(e)
    const float hi = fmaf(-2.f, __builtin_amdgcn_rcpf(e + 1.f), 1.f);
    return copysignf(a < 0.95f ? lo : hi, x);
}

// The layers with 8 output channels, on the matrix cores.
// MODE 0: out = mask * tanh(conv(in));  MODE 2: out = mask * conv(in) *
// (1 - act^2) (backward through tanh).  A pair of rows of 16 outputs, y and
// y + 1, is one implicit GEMM D[(row j, co)][point] = sum over k = (dz, dy',
// dx, ci) of A[(j, co)][k] B[k][point], where the rows share the four input
// rows dy' = dy + j: 36 taps (27 of them with weights per row) fill all 16
// rows of D, where one output row at a time would fill 8 at 28.  Lane l
// supplies A row and B column l % 16 and receives D rows 4 (l / 16) + r, r <
// 4, of column l % 16: four channels of one point, stored in one access, a
// pair of rows in whole lines.
//   SPLIT (8 input channels, layer 2 forward): inputs and weights are hi + lo
//     bfloat16 and the four products lo.lo + hi.lo + lo.hi + hi.hi are summed
//     in FP32 on mfma_f32_16x16x32_bf16, an instruction per (dz, dx) and
//     product with dy' = l / 16, the 8 channels in the lane.
//   otherwise FP32 products on mfma_f32_16x16x4_f32: per (dz, dx) with dy' =
//     l / 16 (one input channel), or per tap and channel parity with channels
//     2 (l / 16) + {0, 1} (eight).
// A work-group owns a column of 16 x 16 x cz points and runs down z: four
// planes with their border in LDS, channels last, three in use while the
// fourth is filled from registers, one barrier a plane; its four waves take two
// row pairs each, one where only 8 rows or fewer are left (15625 boxes of 4^3, all
// layers: 570 us with that, 779 without).  The weights stay in registers.
// Consecutive work-groups of an XCD take neighbouring columns, whose borders its
// L2 then holds.
//   No single unit bounds it: for 32 boxes of 96^3 (28 M points) layer 2
// takes 750 us, of which the matrix instructions are 250, the vector units (half
// of it tanh) 330, and the 0.9 GB written 190 on top of both; blocks of 16 x 8 x
// 4 with one output row per D tile took 1270.  Layer 1 takes 360 (418 with
// fused multiply-adds on the vector units), for 32 boxes of 16^3 the adjoint of
// layer 2 14 (34) and that of layer 3 6 (9).
constexpr int kCX = 16, kCY = 16;          // a column's footprint
constexpr int kPX = kCX + 2, kPY = kCY + 2, kPP = kPX * kPY;   // and its planes with their border

// The pieces of a plane (half a point of 8 channels, or a point of one) that
// thread tid of NT stages: off[k] is the point of piece tid + NT k in the
// plane (any point where the piece is zero), bit k of the result says that
// it is not zero.  Positions more than one point past the box feed only
// outputs that are not computed.
template <int CI, int NT, int NL>
__device__ __forceinline__ unsigned plane_offsets(int tid, int x0, int y0, int Y, int X, int wrap, int off[NL]) {
    unsigned valid = 0;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const int e = tid + NT * k, p = e / (CI == 8 ? 2 : 1);
        const int gx = x0 + p % kPX - 1, gy = y0 + p / kPX - 1;
        bool ok = gx <= X && gy <= Y && p < kPP;
        const int xx = wrap_or_flag(gx, X, wrap, ok), yy = wrap_or_flag(gy, Y, wrap, ok);
        ok = ok && xx >= 0 && xx < X && yy >= 0 && yy < Y;
        off[k] = ok ? yy * X + xx : 0;
        valid |= (unsigned)ok << k;
    }
    return valid;
}
// Loads them, without a branch; plane_piece selects afterwards.
template <int CI, int NL>
__device__ __forceinline__ void load_plane(const float *__restrict__ base, int gz, int Z, int plane, int wrap,
                                           const int off[NL], f4 v[NL]) {
    const int zz = gz < 0 ? (wrap ? gz + Z : 0) : gz >= Z ? (wrap ? gz - Z : 0) : gz;
    const float *src = base + (int64_t)zz * plane * CI + (CI == 8 ? 4 * (threadIdx.x & 1) : 0);
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        if constexpr (CI == 8) v[k] = *(const f4 *)(src + (int64_t)off[k] * 8);
        else v[k][0] = src[off[k]];
    }
}
__device__ __forceinline__ f4 plane_piece(f4 v, unsigned valid, int k, int gz, int Z, int wrap) {
    const bool ok = (valid >> k & 1) && (wrap || (gz >= 0 && gz < Z));
    return ok ? v : f4{0.f, 0.f, 0.f, 0.f};
}

// Column of work-group bid of 8 per: a contiguous range of the n columns for
// each of the 8 XCDs, or -1.
__device__ __forceinline__ int xcd_column(int bid, int n) {
    const int per = (n + 7) / 8, c = bid % 8 * per + bid / 8;
    return c < n ? c : -1;
}

// A operands of lane row px = l % 16: channel px % 8 of output row px / 8.
template <int CI, bool SPLIT> struct Weights {
    bf8 ah[9], al[9];
    f2 aw[SPLIT ? 1 : CI == 8 ? 36 : 9];
    __device__ __forceinline__ void load(const float *__restrict__ W, int px, int g) {
        const int co = px % 8, j = px / 8;
        if constexpr (SPLIT) {
            const int dy = g - j;
#pragma unroll
            for (int c = 0; c < 9; ++c) {
#pragma unroll
                for (int ci = 0; ci < 8; ci += 4) {
                    f4 w;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        w[k] = dy >= 0 && dy < 3 ? W[(co * 8 + ci + k) * 27 + 9 * (c / 3) + 3 * dy + c % 3] : 0.f;
                    bf4 h, l;
                    split(w, h, l);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        ah[c][ci + k] = h[k];
                        al[c][ci + k] = l[k];
                    }
                }
            }
        } else if constexpr (CI == 8) {
#pragma unroll
            for (int t = 0; t < 36; ++t) {
                const int dy = (t / 3) % 4 - j;
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    aw[t][k] = dy >= 0 && dy < 3 ? W[(co * 8 + 2 * g + k) * 27 + 9 * (t / 12) + 3 * dy + t % 3] : 0.f;
            }
        } else {
            const int dy = g - j;
#pragma unroll
            for (int c = 0; c < 9; ++c)
                aw[c][0] = dy >= 0 && dy < 3 ? W[co * 27 + 9 * (c / 3) + 3 * dy + c % 3] : 0.f;
        }
    }
};

// NH: row pairs a wave takes (1: a column of 16 x 8, for the rows left at the
// end of a box); img: the box's first point.  LOAD: the weights are loaded here,
// behind the first planes.
template <int CI, int MODE, bool SPLIT, int NH, bool LOAD>
__device__ __forceinline__ void
conv8_column(const float *__restrict__ base, float *__restrict__ out, const float *__restrict__ W,
             const float *__restrict__ act, const int32_t *__restrict__ boxpt, float (&ring)[4][kPP * CI], int64_t img,
             int x0, int y0, int z0, int z1, int Z, int Y, int X, int wrap, Weights<CI, SPLIT> &w) {
    constexpr int PIECES = kPX * (8 * NH + 2) * (CI == 8 ? 2 : 1), NL = (PIECES + 255) / 256;
    const int tid = threadIdx.x, lane = tid & 63, g = lane / 16, px = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int off[NL];
    const unsigned valid = plane_offsets<CI, 256, NL>(tid, x0, y0, Y, X, wrap, off);
    auto store = [&](int z, const f4 *loaded) {
        float *dst = ring[z & 3];
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = tid + 256 * k;
            if (e >= PIECES) break;
            const f4 v = plane_piece(loaded[k], valid, k, z, Z, wrap);
            if constexpr (SPLIT) {
                bf4 h, l;
                split(v, h, l);
                *(bf4 *)((__bf16 *)dst + 4 * e) = h;
                *(bf4 *)((__bf16 *)dst + kPP * 8 + 4 * e) = l;
            } else if constexpr (CI == 8) {
                *(f4 *)(dst + 4 * e) = v;
            } else {
                dst[e] = v[0];
            }
        }
    };
    f4 v[NL], v1[NL], v2[NL];
    load_plane<CI, NL>(base, z0 - 1, Z, Y * X, wrap, off, v);
    load_plane<CI, NL>(base, z0, Z, Y * X, wrap, off, v1);
    load_plane<CI, NL>(base, z0 + 1, Z, Y * X, wrap, off, v2);
    if constexpr (LOAD) w.load(W, px, g);
    // this lane's point of the wave's row pairs: in the box or not, and where its
    // mask and activations are in a plane
    bool ok[NH];
    int64_t qp[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const int x = x0 + px, y = y0 + 2 * (wave + 4 * h) + g / 2;
        ok[h] = x < X && y < Y;
        qp[h] = (int64_t)min(y, Y - 1) * X + min(x, X - 1);
    }
    int m[NH] = {};
    f4 ac[NH];
    auto load_marks = [&](int z) {
        const int64_t zp = (int64_t)z * Y * X;
        if (boxpt != nullptr)
#pragma unroll
            for (int h = 0; h < NH; ++h) m[h] = boxpt[zp + qp[h]];
        if (MODE == 2)
#pragma unroll
            for (int h = 0; h < NH; ++h) ac[h] = *(const f4 *)(act + (img + zp + qp[h]) * 8 + 4 * (g & 1));
    };
    auto activate = [](f4 d, f4 a, bool inside) {
        f4 r;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float o = MODE == 0 ? tanh_f(d[k]) : d[k] * (1.f - a[k] * a[k]);
            r[k] = inside ? o : 0.f;
        }
        return r;
    };
    load_marks(z0);
    store(z0 - 1, v);
    store(z0, v1);
    store(z0 + 1, v2);
    __syncthreads();
    for (int z = z0; z < z1; ++z) {
        // loads of the next plane, its mask and activations: nothing below
        // waits for them before the plane is stored to LDS
        const bool more = z + 1 < z1;
        bool in[NH];
        f4 acn[NH], res[NH];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            in[h] = ok[h] && m[h] >= 0;
            acn[h] = ac[h];
        }
        if (more) {
            load_plane<CI, NL>(base, z + 2, Z, Y * X, wrap, off, v);
            load_marks(z + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        const float *pl[3] = {ring[(z - 1) & 3], ring[z & 3], ring[(z + 1) & 3]};
        // both row pairs of the wave in one block of code: the second's matrix
        // instructions run beside the first's tanh
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int rb = 2 * (wave + 4 * h) * kPX + px;
            f4 d;
            if constexpr (SPLIT) {
                f4 acc[4];   // one chain per product
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 9; ++c) {
                    const __bf16 *p = (const __bf16 *)pl[c / 3] + (rb + g * kPX + c % 3) * 8;
                    const bf8 bh = *(const bf8 *)p, bl = *(const bf8 *)(p + kPP * 8);
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.al[c], bl, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.al[c], bh, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.ah[c], bl, acc[2], 0, 0, 0);
                    acc[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.ah[c], bh, acc[3], 0, 0, 0);
                }
                d = ((acc[0] + acc[1]) + acc[2]) + acc[3];   // the small products first
            } else if constexpr (CI == 8) {
                f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int t = 0; t < 36; ++t) {
                    const f2 b = *(const f2 *)(pl[t / 12] + (rb + (t / 3) % 4 * kPX + t % 3) * 8 + 2 * g);
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.aw[t][0], b[0], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.aw[t][1], b[1], acc[1], 0, 0, 0);
                }
                d = acc[0] + acc[1];
            } else {
                f4 acc[3];   // one chain per plane
#pragma unroll
                for (int k = 0; k < 3; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < 9; ++c)
                    acc[c / 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.aw[c][0], pl[c / 3][rb + g * kPX + c % 3],
                                                                      acc[c / 3], 0, 0, 0);
                d = (acc[0] + acc[1]) + acc[2];
            }
            res[h] = activate(d, acn[h], in[h]);
        }
        // the pair's other row brings 0 x Inf or 0 x NaN into a sum that does not
        // have that input: a lane with a NaN forms its sums again, own taps only
        f4 sum = res[0];
        if constexpr (NH == 2) sum += res[1];
        if (__builtin_isnan((sum[0] + sum[1]) + (sum[2] + sum[3]))) {
#pragma unroll 1
            for (int h = 0; h < NH; ++h) {
                const int e0 = (2 * (wave + 4 * h) + g / 2) * kPX + px;
                f4 d = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (int t = 0; t < 27; ++t) {
                    const float *p = ring[(z - 1 + t / 9) & 3];
                    const int e = e0 + t / 3 % 3 * kPX + t % 3;
#pragma unroll 1
                    for (int ci = 0; ci < CI; ++ci) {
                        float x;
                        if constexpr (SPLIT) {
                            const __bf16 *q = (const __bf16 *)p + e * 8 + ci;
                            x = (float)q[0] + (float)q[kPP * 8];
                        } else {
                            x = p[e * CI + ci];
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k) d[k] = fmaf(W[((4 * (g & 1) + k) * CI + ci) * 27 + t], x, d[k]);
                    }
                }
#pragma unroll
                for (int i = 0; i < NH; ++i)
                    if (h == i) res[i] = activate(d, acn[i], in[i]);
            }
        }
        // to LDS first: waiting for the loads then does not wait for the results' stores
        if (more) store(z + 2, v);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < NH; ++h)
            if (ok[h])
                __builtin_nontemporal_store(res[h], (f4 *)(out + (img + (int64_t)z * Y * X + qp[h]) * 8 + 4 * (g & 1)));
        __syncthreads();
    }
}

// LOOP: the work-group takes further columns where there are more than
// work-groups, with the weights kept: they take as long to load and split as
// four planes.  It has to keep to 168 registers (the two column forms' weights
// came to 171): three waves per SIMD.
template <int CI, int MODE, bool SPLIT, bool LOOP>
__global__ void __launch_bounds__(256, LOOP ? 3 : 1)
conv8_kernel(const float *__restrict__ in, float *__restrict__ out, const float *__restrict__ W,
             const float *__restrict__ act, const int32_t *__restrict__ boxpt, int ncol, int Z, int Y, int X,
             int wrap, int ntx, int nty, int ntz, int cz) {
    __shared__ __attribute__((aligned(16))) float ring[4][kPP * CI];   // SPLIT: kPP * 8 hi, then kPP * 8 lo
    Weights<CI, SPLIT> w;
    if constexpr (LOOP) w.load(W, threadIdx.x % 16, (threadIdx.x & 63) / 16);
    for (int bid = blockIdx.x; bid < (ncol + 7) / 8 * 8; bid += gridDim.x) {
        const int col = xcd_column(bid, ncol);
        if (col < 0) return;
        const int tx = col % ntx, ty = (col / ntx) % nty, tz = (col / (ntx * nty)) % ntz;
        const int64_t img = (int64_t)(col / (ntx * nty * ntz)) * Z * Y * X;
        const int x0 = tx * kCX, y0 = ty * kCY, z0 = tz * cz, z1 = min(z0 + cz, Z);
        const float *base = in + img * CI;
        // half of a column's rows are left out where they lie outside the box
        if (y0 + 8 < Y)
            conv8_column<CI, MODE, SPLIT, 2, !LOOP>(base, out, W, act, boxpt, ring, img, x0, y0, z0, z1, Z, Y, X, wrap, w);
        else
            conv8_column<CI, MODE, SPLIT, 1, !LOOP>(base, out, W, act, boxpt, ring, img, x0, y0, z0, z1, Z, Y, X, wrap, w);
        if (!LOOP) return;
    }
}

// Columns of nbox boxes of Z x Y x X points: counts and depth cz.  32 planes a
// column cost a sixteenth more border; 16 or 8 where that would leave fewer than
// 2048 work-groups, about two rounds of what is resident (32 boxes of 52^3: 363
// us against 404); below that the border weighs more, and 1024 must do (16 boxes
// of 36^3: 123 against 142), 512 for columns of 4 (740 boxes of 3^3: all layers 33
// us against 41, 128 of 16^3 47 against 50).  At least 2: single planes read three
// for one and gain nothing (layer 2 for 32 boxes of 16^3: 14 us either way).
struct Columns {
    int ntx, nty, ntz, cz, n;
    Columns(int nbox, int Z, int Y, int X) : ntx((X + kCX - 1) / kCX), nty((Y + kCY - 1) / kCY), cz(32) {
        auto count = [&] { return (int64_t)ntx * nty * ((Z + cz - 1) / cz) * nbox; };
        while (cz > 8 && count() < 2048) cz /= 2;
        while (cz > 4 && count() < 1024) cz /= 2;
        while (cz > 2 && count() < 512) cz /= 2;
        ntz = (Z + cz - 1) / cz;
        n = ntx * nty * ntz * nbox;
    }
    dim3 grid() const { return dim3((unsigned)((n + 7) / 8 * 8)); }
};

constexpr unsigned kLoopGroups = 768;   // three a compute unit

// Launches conv8_kernel over n boxes of Z x Y x X points.
template <int CI, int MODE, bool SPLIT>
void conv8(const float *in, float *out, const float *W, const float *act, const int32_t *boxpt, int n, int Z, int Y,
           int X, int wrap, hipStream_t st) {
    const Columns c(n, Z, Y, X);
    dim3 grid = c.grid();
    if constexpr (SPLIT) {
        // shallow columns: as many work-groups as are resident (15625 boxes of
        // 4^3, all layers: 402 us, one column a work-group 546; 390 of 8^3 46, 50)
        if (std::min(c.cz, Z) < 8 && grid.x > kLoopGroups) {
            hipLaunchKernelGGL((conv8_kernel<CI, MODE, SPLIT, true>), dim3(kLoopGroups), dim3(256), 0, st, in, out, W,
                               act, boxpt, c.n, Z, Y, X, wrap, c.ntx, c.nty, c.ntz, c.cz);
            return;
        }
    }
    hipLaunchKernelGGL((conv8_kernel<CI, MODE, SPLIT, false>), grid, dim3(256), 0, st, in, out, W, act, boxpt, c.n, Z,
                       Y, X, wrap, c.ntx, c.nty, c.ntz, c.cz);
}

// Layer 3, 8 -> 1 channels: out = mask * conv(in).  The vector units' 216
// fused multiply-adds a point bound it if the inputs are not read from LDS
// once per output: a thread runs down z over two y-neighbouring columns, a
// plane's 12 points feeding six sums (two columns, three outputs in z), 12
// 32-byte reads for two outputs.  The planes of a 16 x 16 block and its
// border are staged in two buffers, four channels in each half of a plane,
// so that 16 lanes read 256 contiguous bytes.  Per output the sum runs over
// taps 9 dz + 3 dy + dx, then channels, one fused multiply-add each.  wt:
// [27][8].  28 M points take 375 us, 190 of them the multiply-adds; two outputs
// a thread that read their taps from blocks of 16 x 8 x 4 took 560.
__global__ void __launch_bounds__(128)
conv1_kernel(const float *__restrict__ in, float *__restrict__ out, const float *__restrict__ wt,
             const int32_t *__restrict__ boxpt, int ncol, int Z, int Y, int X, int wrap, int ntx, int nty, int ntz,
             int cz) {
    constexpr int NL = (2 * kPP + 127) / 128;
    __shared__ __attribute__((aligned(16))) f4 buf[2][2 * kPP];
    const int col = xcd_column(blockIdx.x, ncol);
    if (col < 0) return;
    const int tx = col % ntx, ty = (col / ntx) % nty, tz = (col / (ntx * nty)) % ntz;
    const int64_t vol = (int64_t)Z * Y * X, img = col / (ntx * nty * ntz);
    const int x0 = tx * kCX, y0 = ty * kCY, z0 = tz * cz, z1 = min(z0 + cz, Z);
    const float *base = in + img * vol * 8;
    const int tid = threadIdx.x;
    int off[NL];
    const unsigned valid = plane_offsets<8, 128, NL>(tid, x0, y0, Y, X, wrap, off);
    f4 v[NL];
    auto store = [&](int b, int z) {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = tid + 128 * k;
            if (e < 2 * kPP) buf[b][(e & 1) * kPP + e / 2] = plane_piece(v[k], valid, k, z, Z, wrap);
        }
    };
    const int lx = tid % kCX, ly = 2 * (tid / kCX);
    bool ok[2];
    int64_t qp[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int x = x0 + lx, y = y0 + ly + j;
        ok[j] = x < X && y < Y;
        qp[j] = (int64_t)min(y, Y - 1) * X + min(x, X - 1);
    }
    // a wave without rows in the box only stages
    const bool live = y0 + 8 * __builtin_amdgcn_readfirstlane(tid >> 6) < Y;
    // sums of the outputs one plane back, of this plane and one ahead
    float a0[2] = {0.f, 0.f}, a1[2] = {0.f, 0.f}, a2[2] = {0.f, 0.f};
    load_plane<8, NL>(base, z0 - 1, Z, Y * X, wrap, off, v);
    store(0, z0 - 1);
    __syncthreads();
    for (int z = z0 - 1, b = 0; z <= z1; ++z, b ^= 1) {
        int m[2] = {0, 0};
        if (boxpt != nullptr && z > z0)
#pragma unroll
            for (int j = 0; j < 2; ++j) m[j] = boxpt[(int64_t)(z - 1) * Y * X + qp[j]];
        if (z < z1) load_plane<8, NL>(base, z + 1, Z, Y * X, wrap, off, v);
        __builtin_amdgcn_sched_barrier(0);
        if (live) {
            const f4 *row = buf[b] + ly * kPX + lx;
            f4 r[2][6];
#pragma unroll
            for (int k = 0; k < 6; ++k) r[0][k] = row[(k & 1) * kPP + k / 2];
#pragma unroll
            for (int dyp = 0; dyp < 4; ++dyp) {
                if (dyp < 3)
#pragma unroll
                    for (int k = 0; k < 6; ++k) r[(dyp + 1) & 1][k] = row[(k & 1) * kPP + (dyp + 1) * kPX + k / 2];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int dy = dyp - j;
                    if (dy < 0 || dy > 2) continue;
                    // the weights are loaded here, 72 at a time: all 216, kept
                    // over the planes, would not fit the scalar registers
                    int wo = 3 * dy * 8;
                    asm volatile("" : "+s"(wo));
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                        for (int c = 0; c < 8; ++c) {
                            const float u = r[dyp & 1][2 * dx + c / 4][c % 4];
                            const float *w = wt + wo + dx * 8 + c;
                            a0[j] = fmaf(w[2 * 72], u, a0[j]);
                            a1[j] = fmaf(w[72], u, a1[j]);
                            a2[j] = fmaf(w[0], u, a2[j]);
                        }
                    asm volatile("" : "+v"(a0[j]), "+v"(a1[j]), "+v"(a2[j]));
                }
            }
        }
        // to LDS first: waiting for the loads then does not wait for the results' stores
        if (z < z1) store(b ^ 1, z + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (z > z0 && ok[j]) out[img * vol + (int64_t)(z - 1) * Y * X + qp[j]] = m[j] >= 0 ? a0[j] : 0.f;
            a0[j] = a1[j];
            a1[j] = a2[j];
            a2[j] = 0.f;
        }
        __syncthreads();
    }
}

// The same sums for problems too small for deep columns: blocks of 16 x 8 x 4
// outputs, staged with their border at once, two x-neighbouring outputs a
// thread, which share the loads of their taps.
constexpr int kSX = 16, kSY = 8, kSZ = 4;
__global__ void __launch_bounds__(256)
conv1_block_kernel(const float *__restrict__ in, float *__restrict__ out, const float *__restrict__ wt,
                   const int32_t *__restrict__ boxpt, int Z, int Y, int X, int wrap, int ntx, int nty, int ntz) {
    constexpr int HX = kSX + 2, HY = kSY + 2, HZ = kSZ + 2;
    __shared__ __attribute__((aligned(16))) float tile[HZ * HY * HX * 8];
    const int bid = blockIdx.x;
    const int tx = bid % ntx, ty = (bid / ntx) % nty, tz = (bid / (ntx * nty)) % ntz;
    const int img = bid / (ntx * nty * ntz);
    const int x0 = tx * kSX, y0 = ty * kSY, z0 = tz * kSZ;
    const int vol = Z * Y * X;
    const float *base = in + (int64_t)img * vol * 8;
    for (int e = threadIdx.x; e < HZ * HY * HX; e += 256) {
        const int hx = e % HX, hy = (e / HX) % HY, hz = e / (HX * HY);
        const int gx = x0 + hx - 1, gy = y0 + hy - 1, gz = z0 + hz - 1;
        bool ok = gx <= X && gy <= Y && gz <= Z;
        const int xx = wrap_or_flag(gx, X, wrap, ok);
        const int yy = wrap_or_flag(gy, Y, wrap, ok);
        const int zz = wrap_or_flag(gz, Z, wrap, ok);
        ok = ok && xx >= 0 && xx < X && yy >= 0 && yy < Y && zz >= 0 && zz < Z;
        f4 lo = f4{0.f, 0.f, 0.f, 0.f}, hi = lo;
        if (ok) {
            const float *src = base + ((int64_t)(zz * Y + yy) * X + xx) * 8;
            lo = *(const f4 *)src;
            hi = *(const f4 *)(src + 4);
        }
        *(f4 *)(tile + e * 8) = lo;
        *(f4 *)(tile + e * 8 + 4) = hi;
    }
    __syncthreads();
    const int t = threadIdx.x;
    const int lx = 2 * (t % (kSX / 2)), ly = (t / (kSX / 2)) % kSY, lz = t / (kSX / 2 * kSY);
    float acc[2] = {0.f, 0.f};
    // (dz, dy) stays a loop: unrolled, the loads of all nine rows would be
    // hoisted and the work-group would run at one wave per SIMD
#pragma unroll 1
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll 1
        for (int dy = 0; dy < 3; ++dy) {
            const float *row = tile + (((lz + dz) * HY + (ly + dy)) * HX + lx) * 8;
            f4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = *(const f4 *)(row + 4 * k);
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float w = wt[(9 * dz + 3 * dy + dx) * 8 + c];
#pragma unroll
                    for (int k = 0; k < 2; ++k) acc[k] = fmaf(w, v[2 * (dx + k) + c / 4][c % 4], acc[k]);
                }
        }
    const int y = y0 + ly, z = z0 + lz;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int x = x0 + lx + k;
        if (x >= X || y >= Y || z >= Z) continue;
        const int q = (z * Y + y) * X + x;
        out[(int64_t)img * vol + q] = boxpt == nullptr || boxpt[q] >= 0 ? acc[k] : 0.f;
    }
}

// Layer 3 over n boxes of Z x Y x X points.  Columns of a few planes stage most
// of them twice, or two planes more than they write, and run few waves: 32 boxes
// of 16^3 in columns of 2 take 12.6 us, in blocks 7.6; 15625 of 4^3 214 and 141;
// 32 boxes of 96^3 in columns of 32 375, in blocks 560.
void conv1(const float *in, float *out, const float *wt, const int32_t *boxpt, int n, int Z, int Y, int X, int wrap,
           hipStream_t st) {
    const Columns c(n, Z, Y, X);
    if (std::min(c.cz, Z) >= 8) {
        hipLaunchKernelGGL(conv1_kernel, c.grid(), dim3(128), 0, st, in, out, wt, boxpt, c.n, Z, Y, X, wrap, c.ntx,
                           c.nty, c.ntz, c.cz);
        return;
    }
    const int ntx = (X + kSX - 1) / kSX, nty = (Y + kSY - 1) / kSY, ntz = (Z + kSZ - 1) / kSZ;
    hipLaunchKernelGGL(conv1_block_kernel, dim3((unsigned)((int64_t)ntx * nty * ntz * n)), dim3(256), 0, st, in, out, wt,
                       boxpt, Z, Y, X, wrap, ntx, nty, ntz);
}

// Weights of the input adjoint, Wt[ci][co][26 - t] = W[co][ci][t] of layers 2
// and 3, and the two layers with one output channel in conv1_kernel's order
// [27][8]: layer 3, and layer 1's adjoint in place of its Wt.
constexpr int kW3T = kNW, kNWT = kNW + 216;
__device__ __forceinline__ void place_weight(int i, float w, float *__restrict__ wt) {
    if (i < kW2) {
        wt[kW1 + (26 - i % 27) * 8 + i / 27] = w;
    } else if (i < kW3) {
        const int j = i - kW2, t = j % 27, ci = (j / 27) % 8, co = j / (27 * 8);
        wt[kW2 + (ci * 8 + co) * 27 + (26 - t)] = w;
    } else {
        const int j = i - kW3, t = j % 27, ci = j / 27;
        wt[kW3 + ci * 27 + (26 - t)] = w;
        wt[kW3T + t * 8 + ci] = w;
    }
}
__global__ void place_kernel(const float *__restrict__ params, float *__restrict__ wt) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kNW) place_weight(i, params[i], wt);
}

// Weight gradient partials on the FP32 matrix cores.  With q = p + (dx - 1)
//   dW[co][ci][dz][dy][dx] = sum_q x[q + (dz - 1, dy - 1)][ci] d[q - (dx - 1)][co],
// a contraction over the points q of a (9 CI) x (3 CO) matrix: rows (dz, dy,
// ci), columns (dx, co), so the nine (dz, dy) shifts come from one LDS copy
// of x and the three dx shifts from one of d, and 8 -> 8 channels fill 72 x 24
// of five by two 16 x 16 tiles.  A work-group stages a TZ x TY x TX block of
// q (x with its border in z and y, d with its border in x; zero outside the
// box), each wave takes every fourth row of 16 points, four points per
// mfma_f32_16x16x4_f32 (FP32 products and sums, as fused multiply-adds), and
// the waves' tiles are added in LDS in wave order.  Bound by the matrix
// cores' 32 cycles per instruction.  A work-group takes further blocks in
// turn where there are more than kWgMax of them, so that the partials stay
// small, and no more than about kWgPts points, so that the FP32 sums stay
// short; wgrad_final_kernel adds the work-groups in FP64.  One thread per (tap, ci) that
// gathered its taps from global memory took 792-843 us a layer for 32 crops of 16^3;
// this takes 8 (1 -> 8), 15 (8 -> 8) and 17 us (8 -> 1).
constexpr int kTX = 16, kTY = 8, kTZ = 4;   // points of a block
constexpr int kWgMax = 1024;
template <int CI, int CO>
__global__ void __launch_bounds__(256)
wgrad_kernel(const float *__restrict__ xin, const float *__restrict__ d, int n, int Z, int Y, int X, int ntx, int nty,
             int ntz, float *__restrict__ partial) {
    constexpr int HY = kTY + 2, HZ = kTZ + 2, HX = kTX + 2;
    constexpr int MT = (9 * CI + 15) / 16, NT = (3 * CO + 15) / 16;
    constexpr int NXS = HZ * HY * kTX * CI, NDS = kTZ * kTY * HX * CO, NRED = 3 * MT * NT * 256;
    __shared__ __attribute__((aligned(16))) float buf[NXS + NDS > NRED ? NXS + NDS : NRED];
    float *xs = buf, *ds = buf + NXS;
    const int tid = threadIdx.x, lane = tid & 63, k4 = lane / 16;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: it guards matrix instructions
    const int vol = Z * Y * X;
    // operand offsets of this lane's rows and columns; those past the matrix
    // read a valid word and are dropped at the end
    int aoff[MT], boff[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int m = 16 * i + lane % 16, s = m / CI;
        aoff[i] = m < 9 * CI ? ((s / 3) * HY + s % 3) * kTX * CI + m % CI : 0;
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int c = 16 * j + lane % 16;
        boff[j] = c < 3 * CO ? (2 - c / CO) * CO + c % CO : 0;
    }
    f4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    const int ntile = ntx * nty * ntz * n;
    for (int bid = blockIdx.x; bid < ntile; bid += gridDim.x) {
        const int x0 = (bid % ntx) * kTX, y0 = (bid / ntx) % nty * kTY, z0 = (bid / (ntx * nty)) % ntz * kTZ;
        const int64_t base = (int64_t)(bid / (ntx * nty * ntz)) * vol;
        __syncthreads();   // the previous block's reads are done
        for (int e = tid; e < NXS / CI; e += 256) {
            const int x = x0 + e % kTX, y = y0 + (e / kTX) % HY - 1, z = z0 + e / (kTX * HY) - 1;
            const bool ok = x < X && y >= 0 && y < Y && z >= 0 && z < Z;
            const float *src = xin + (base + (int64_t)(z * Y + y) * X + x) * CI;
            if constexpr (CI == 8) {
                const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
                *(float4 *)(xs + e * 8) = ok ? *(const float4 *)src : zero;
                *(float4 *)(xs + e * 8 + 4) = ok ? *(const float4 *)(src + 4) : zero;
            } else {
#pragma unroll
                for (int c = 0; c < CI; ++c) xs[e * CI + c] = ok ? src[c] : 0.f;
            }
        }
        for (int e = tid; e < NDS / CO; e += 256) {
            const int x = x0 + e % HX - 1, y = y0 + (e / HX) % kTY, z = z0 + e / (HX * kTY);
            const bool ok = x >= 0 && x < X && y < Y && z < Z;
            const float *src = d + (base + (int64_t)(z * Y + y) * X + x) * CO;
            if constexpr (CO == 8) {
                const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
                *(float4 *)(ds + e * 8) = ok ? *(const float4 *)src : zero;
                *(float4 *)(ds + e * 8 + 4) = ok ? *(const float4 *)(src + 4) : zero;
            } else {
#pragma unroll
                for (int c = 0; c < CO; ++c) ds[e * CO + c] = ok ? src[c] : 0.f;
            }
        }
        __syncthreads();
        const int nk = (min(kTX, X - x0) + 3) / 4;
        for (int row = wave; row < kTZ * kTY; row += 4) {
            const int lz = row / kTY, ly = row % kTY;
            if (z0 + lz >= Z || y0 + ly >= Y) continue;
            const float *xr = xs + ((lz * HY + ly) * kTX + k4) * CI, *dr = ds + (row * HX + k4) * CO;
#pragma unroll
            for (int k = 0; k < kTX / 4; ++k) {
                if (k >= nk) break;
                float a[MT], b[NT];
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = xr[4 * k * CI + aoff[i]];
#pragma unroll
                for (int j = 0; j < NT; ++j) b[j] = dr[4 * k * CO + boff[j]];
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    }
    __syncthreads();
    if (wave > 0)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) *(f4 *)(buf + (((wave - 1) * MT * NT + i * NT + j) * 64 + lane) * 4) = acc[i][j];
    __syncthreads();
    if (wave > 0) return;
    float *out = partial + (int64_t)blockIdx.x * (CO * CI * 27);
    bool nan = false;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            f4 v = acc[i][j];
#pragma unroll
            for (int w = 0; w < 3; ++w) v += *(const f4 *)(buf + ((w * MT * NT + i * NT + j) * 64 + lane) * 4);
            const int c = 16 * j + lane % 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 16 * i + 4 * k4 + r;
                if (m < 9 * CI && c < 3 * CO) {
                    out[((c % CO) * CI + m % CI) * 27 + m / CI * 3 + c / CO] = v[r];
                    nan = nan || __builtin_isnan(v[r]);
                }
            }
        }
    // the zeros around a block times Inf or NaN are no part of a gradient: with a
    // NaN among them the sums are formed again over the taps in the box, a lane
    // per (tap, ci)
    if (!__any(nan)) return;
    for (int e = lane; e < 27 * CI; e += 64) {
        const int t = e / CI, ci = e % CI;
        float sum[CO];
#pragma unroll
        for (int c = 0; c < CO; ++c) sum[c] = 0.f;
        for (int bid = blockIdx.x; bid < ntile; bid += gridDim.x) {
            const int x0 = (bid % ntx) * kTX, y0 = (bid / ntx) % nty * kTY, z0 = (bid / (ntx * nty)) % ntz * kTZ;
            const int64_t base = (int64_t)(bid / (ntx * nty * ntz)) * vol;
#pragma unroll 1
            for (int p = 0; p < kTZ * kTY * kTX; ++p) {
                // x at (zx, yx, x), d at (z, y, xd): the pairs the matrix form has
                const int x = x0 + p % kTX, y = y0 + p / kTX % kTY, z = z0 + p / (kTX * kTY);
                const int xd = x + 1 - t % 3, yx = y + t / 3 % 3 - 1, zx = z + t / 9 - 1;
                if (x >= X || y >= Y || z >= Z || xd < 0 || xd >= X || yx < 0 || yx >= Y || zx < 0 || zx >= Z) continue;
                const float xv = xin[(base + (int64_t)(zx * Y + yx) * X + x) * CI + ci];
                const float *dv = d + (base + (int64_t)(z * Y + y) * X + xd) * CO;
#pragma unroll
                for (int c = 0; c < CO; ++c) sum[c] = fmaf(xv, dv[c], sum[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < CO; ++c) out[(c * CI + ci) * 27 + t] = sum[c];
    }
}

// Work-groups of the weight gradients for n boxes of Z x Y x X points.
int wgrad_groups(int64_t tot, int64_t ntile) {
    return (int)std::min<int64_t>(ntile, std::max<int64_t>(kWgMax, (tot + kWgPts - 1) / kWgPts));
}

// grad[j] = sum over work-groups of the layers' partials (FP64, fixed
// order), all three layers in one launch; 64 entries x 16 shares of the
// work-groups per block.
__global__ void __launch_bounds__(1024)
wgrad_final_kernel(const float *__restrict__ partial, int nwg, float *__restrict__ grad) {
    __shared__ double red[16][64];
    const int e = threadIdx.x & 63, part = threadIdx.x >> 6, j = blockIdx.x * 64 + e;
    if (j < kNW) {
        const int off = j < kW2 ? kW1 : j < kW3 ? kW2 : kW3, nw = j < kW2 || j >= kW3 ? 216 : 1728;
        const float *p = partial + (int64_t)off * nwg + (j - off);
        double s = 0.0;
#pragma unroll 4
        for (int w = part; w < nwg; w += 16) s += p[(int64_t)w * nw];
        red[part][e] = s;
    }
    __syncthreads();
    if (part == 0 && j < kNW) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s += red[w][e];
        grad[j] = (float)s;
    }
}

__device__ double softplus_d(double z) { return z > 0 ? z + log1p(exp(-z)) : log1p(exp(z)); }
__device__ double sigmoid_d(double z) { return 0.5 * (1.0 + tanh(0.5 * z)); }

// g_i = softplus(a + b l_i), l_i = log(-sigma_i h^2); gz = [g, z, l] per sample.
__global__ void gain_kernel(const float *__restrict__ params, const double *__restrict__ sigma, double h, int n,
                            double *__restrict__ gz) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double l = log(-sigma[i] * h * h);
    const double z = (double)params[kNW] + (double)params[kNW + 1] * l;
    gz[3 * i] = softplus_d(z);
    gz[3 * i + 1] = z;
    gz[3 * i + 2] = l;
}

__device__ __forceinline__ bool interior(int q, int Z, int Y, int X, int margin) {
    const int x = q % X, y = (q / X) % Y, z = q / (X * Y);
    return !(x < margin || y < margin || z < margin || x >= X - margin || y >= Y - margin || z >= Z - margin);
}

// em = M (g f - t), tm = M t (M: points at least `margin` from the faces).
__global__ void err_kernel(const float *__restrict__ f, const float *__restrict__ t, const double *__restrict__ gz,
                           int Z, int Y, int X, int margin, int n, float *__restrict__ em, float *__restrict__ tm) {
    const int vol = Z * Y * X;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    if (gid >= vol * n) return;
    const int i = gid / vol, q = gid - i * vol;
    const bool in = interior(q, Z, Y, X, margin);
    em[gid] = in ? (float)(gz[3 * i] * (double)f[gid] - (double)t[gid]) : 0.f;
    tm[gid] = in ? t[gid] : 0.f;
}

// out = (T - sigma_i) x on each box, zero outside: the 25-point star of
// Sec. 5.1 in first-difference form.
__global__ void kin_kernel(const float *__restrict__ x, float *__restrict__ out, const double *__restrict__ sigma,
                           double h, int Z, int Y, int X, int n) {
    const int vol = Z * Y * X;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    if (gid >= vol * n) return;
    const int i = gid / vol, q = gid - i * vol;
    const int cx = q % X, cy = (q / X) % Y, cz = q / (X * Y);
    const float *b = x + (int64_t)i * vol;
    const float c[5] = {0.f, 8.f / 5.f, -1.f / 5.f, 8.f / 315.f, -1.f / 560.f};
    const float v = b[q];
    float acc = 0.f;
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
        const float xm = cx - m >= 0 ? b[q - m] : 0.f, xp = cx + m < X ? b[q + m] : 0.f;
        const float ym = cy - m >= 0 ? b[q - m * X] : 0.f, yp = cy + m < Y ? b[q + m * X] : 0.f;
        const float zm = cz - m >= 0 ? b[q - m * X * Y] : 0.f, zp = cz + m < Z ? b[q + m * X * Y] : 0.f;
        acc += c[m] * (((xm - v) + (xp - v)) + ((ym - v) + (yp - v)) + ((zm - v) + (zp - v)));
    }
    out[gid] = (float)(-0.5 / (h * h) * (double)acc - sigma[i] * (double)v);
}

// Per (chunk, sample) sums: <em|A em>, <tm|A tm>, <M f|A em>.
__global__ void __launch_bounds__(256)
loss_partial_kernel(const float *__restrict__ em, const float *__restrict__ ae, const float *__restrict__ tm,
                    const float *__restrict__ at, const float *__restrict__ f, int Z, int Y, int X, int margin,
                    int nch, double *__restrict__ partial) {
    __shared__ double red[3][256];
    const int i = blockIdx.y, tid = threadIdx.x;
    const int vol = Z * Y * X, per = (vol + nch - 1) / nch;
    const int q0 = blockIdx.x * per, q1 = min(vol, q0 + per);
    double a0 = 0, a1 = 0, a2 = 0;
    for (int q = q0 + tid; q < q1; q += 256) {
        const int64_t k = (int64_t)i * vol + q;
        const double aev = ae[k];
        a0 += (double)em[k] * aev;
        a1 += (double)tm[k] * (double)at[k];
        if (interior(q, Z, Y, X, margin)) a2 += (double)f[k] * aev;
    }
    red[0][tid] = a0;
    red[1][tid] = a1;
    red[2][tid] = a2;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s)
            for (int k = 0; k < 3; ++k) red[k][tid] += red[k][tid + s];
        __syncthreads();
    }
    if (tid < 3) partial[((int64_t)i * nch + blockIdx.x) * 3 + tid] = red[tid][0];
}

// loss = sum_i <e|Ae>_i / sum_i <t|At>_i; coef = 2 / sum_i <t|At>_i (so
// dL/dpred = coef M A e); gain-parameter gradient into grad[kNW], grad[kNW + 1].
// One work-group, a thread per sample (samples i, i + 256, ... where there are
// more), then sums over the threads in a fixed order; one thread doing it all
// took 19 us for 32 samples, this 5.
__device__ __forceinline__ double sum256(double v, double *red) {
    const int t = threadIdx.x;
    __syncthreads();
    red[t] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    return red[0];
}
__global__ void __launch_bounds__(256)
loss_final_kernel(const double *__restrict__ partial, int n, int nch, const double *__restrict__ gz,
                  double *__restrict__ coef, double *__restrict__ loss, float *__restrict__ grad) {
    __shared__ double red[256];
    double e2 = 0, t2 = 0, ga = 0, gb = 0;
    for (int i = threadIdx.x; i < n; i += 256) {
        double ef = 0;
        for (int c = 0; c < nch; ++c) {
            const double *p = partial + ((int64_t)i * nch + c) * 3;
            e2 += p[0];
            t2 += p[1];
            ef += p[2];
        }
        const double d = ef * sigmoid_d(gz[3 * i + 1]);
        ga += d;
        gb += d * gz[3 * i + 2];
    }
    const double E2 = sum256(e2, red), T2 = sum256(t2, red), GA = sum256(ga, red), GB = sum256(gb, red);
    const double cf = T2 > 0 ? 2.0 / T2 : 0.0;
    for (int i = threadIdx.x; i < n; i += 256) coef[i] = cf;
    if (threadIdx.x) return;
    *loss = T2 > 0 ? E2 / T2 : 0.0;
    grad[kNW] = (float)(cf * GA);
    grad[kNW + 1] = (float)(cf * GB);
}

__global__ void df_kernel(const float *__restrict__ ae, const double *__restrict__ gz,
                          const double *__restrict__ coef, int Z, int Y, int X, int margin, int n,
                          float *__restrict__ df) {
    const int vol = Z * Y * X;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    if (gid >= vol * n) return;
    const int i = gid / vol, q = gid - i * vol;
    df[gid] = interior(q, Z, Y, X, margin) ? (float)(gz[3 * i] * coef[i] * (double)ae[gid]) : 0.f;
}

// Adam (Kingma and Ba, 2015): c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ void adam_kernel(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, float *__restrict__ wt, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kNP) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    if (i < kNW) place_weight(i, pi, wt);
}

// ------------------------------------------------- grid <-> dense boxes
// Transposing copies through LDS: a work-group moves 64 consecutive box
// points (or grid points) of the B states of one block.
template <typename T>
__global__ void __launch_bounds__(256)
scatter_kernel(const T *__restrict__ r, const int32_t *__restrict__ boxpt, const double *__restrict__ scale,
               int k0, int B, int64_t np, int vol, float *__restrict__ u) {
    __shared__ float tile[64][65];
    const int blk = blockIdx.y, tid = threadIdx.x;
    const int q0 = blockIdx.x * 64;
    const int kb = k0 + blk * B;               // first state of the block
    // loads in flight before their uses: the box point, then its field entry
    for (int e0 = tid; e0 < 64 * B; e0 += 256 * 8) {
        int pt[8];
        T v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = e0 + 256 * k, q = q0 + e / B;
            pt[k] = e < 64 * B && q < vol ? boxpt[q] : -1;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            v[k] = T(0);
            if (pt[k] >= 0) v[k] = r[((int64_t)(kb / B) * np + pt[k]) * B + (e0 + 256 * k) % B];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int e = e0 + 256 * k, s = e % B;
            if (e < 64 * B) tile[s][e / B] = pt[k] >= 0 ? (float)((double)v[k] * scale[kb + s]) : 0.f;
        }
    }
    __syncthreads();
    for (int e = tid; e < 64 * B; e += 256) {
        const int s = e / 64, qi = e % 64, q = q0 + qi;
        if (q < vol) u[(int64_t)(blk * B + s) * vol + q] = tile[s][qi];
    }
}

template <typename T>
__global__ void __launch_bounds__(256)
gather_kernel(const float *__restrict__ f, const int32_t *__restrict__ boxidx, const double *__restrict__ scale,
              int k0, int B, int64_t np, int vol, T *__restrict__ out) {
    __shared__ float tile[64][65];
    // bricks along x share lines of f: consecutive ones go to one XCD's L2
    const int blk = blockIdx.y, tid = threadIdx.x, chunk = xcd_column(blockIdx.x, (int)((np + 63) / 64));
    if (chunk < 0) return;
    const int64_t p0 = (int64_t)chunk * 64;
    const int kb = k0 + blk * B;
    const int pi = tid % 64;
    const bool in = p0 + pi < np;
    const float *src = f + (int64_t)blk * B * vol + (in ? boxidx[p0 + pi] : 0);
    for (int s0 = tid / 64; s0 < B; s0 += 4 * 8) {   // eight loads in flight
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = in && s0 + 4 * k < B ? src[(int64_t)(s0 + 4 * k) * vol] : 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (s0 + 4 * k < B) tile[s0 + 4 * k][pi] = v[k];
    }
    __syncthreads();
    for (int e = tid; e < 64 * B; e += 256) {
        const int pi = e / B, s = e % B;
        const int64_t p = p0 + pi;
        if (p < np) out[((int64_t)(kb / B) * np + p) * B + s] = (T)((double)tile[s][pi] * scale[kb + s]);
    }
}

// Crops: u[c][z][y][x] = r(point at box origin + (x, y, z)) * inv_s[state],
// t likewise from x; zero off the domain (or beyond the box unless periodic).
template <typename T>
__global__ void __launch_bounds__(256)
crop_kernel(const T *__restrict__ r, const T *__restrict__ xs, const int32_t *__restrict__ boxpt,
            const int32_t *__restrict__ desc, const double *__restrict__ inv_s, int B, int64_t np, int BZ, int BY,
            int BX, int wrap, int CZ, int CY, int CX, int ncrops, float *__restrict__ u, float *__restrict__ t) {
    const int cvol = CZ * CY * CX;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    if (gid >= cvol * ncrops) return;
    const int c = gid / cvol, q = gid - c * cvol;
    const int k = desc[4 * c];
    bool ok = true;
    const int x = wrap_or_flag(desc[4 * c + 1] + q % CX, BX, wrap, ok);
    const int y = wrap_or_flag(desc[4 * c + 2] + (q / CX) % CY, BY, wrap, ok);
    const int z = wrap_or_flag(desc[4 * c + 3] + q / (CX * CY), BZ, wrap, ok);
    float uv = 0.f, tv = 0.f;
    if (ok) {
        const int pt = boxpt[(z * BY + y) * BX + x];
        if (pt >= 0) {
            const int64_t i = ((int64_t)(k / B) * np + pt) * B + k % B;
            uv = (float)((double)r[i] * inv_s[k]);
            tv = (float)((double)xs[i] * inv_s[k]);
        }
    }
    u[gid] = uv;
    t[gid] = tv;
}

template <typename F> struct OpSumSq {
    typedef F T;
    static constexpr int NF = 1;
    const T *x;
    __device__ void load(int64_t i, T *v) const { v[0] = x[i]; }
    __device__ void operator()(const T *f, int64_t, int, double *a) const {
        const double v = f[0];
        a[0] += v * v;
    }
};

// scale: [inv_s | s * g] per state from the sums of squares and shifts.
__global__ void prescale_kernel(const double *__restrict__ ss, const double *__restrict__ sigma,
                                const float *__restrict__ params, double h, int64_t np, int N,
                                double *__restrict__ inv_s, double *__restrict__ outs) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= N) return;
    const double s = sqrt(ss[k] / (double)np);
    const double z = (double)params[kNW] + (double)params[kNW + 1] * log(-sigma[k] * h * h);
    inv_s[k] = s > 0 ? 1.0 / s : 0.0;
    outs[k] = s > 0 ? s * softplus_d(z) : 0.0;
}

__global__ void invs_kernel(const double *__restrict__ ss, int64_t np, int N, double *__restrict__ inv_s) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= N) return;
    const double s = sqrt(ss[k] / (double)np);
    inv_s[k] = s > 0 ? 1.0 / s : 0.0;
}

// ------------------------------------------------- conjugate gradients
template <typename F> struct OpPAp {      // <p|(T - sigma) p> with q = T p
    typedef F T;
    static constexpr int NF = 2;
    const T *p, *q;
    const double *sig;
    __device__ void load(int64_t i, T *v) const {
        v[0] = p[i];
        v[1] = q[i];
    }
    __device__ void operator()(const T *f, int64_t, int c, double *a) const {
        const double pv = f[0];
        a[0] += pv * ((double)f[1] - sig[c] * pv);
    }
};
template <typename F> struct OpCgUpdate { // x += al p, r -= al (q - sigma p), <r|r>
    typedef F T;
    static constexpr int NF = 4;
    T *x, *r;
    const T *p, *q;
    const double *sig, *al;
    __device__ void load(int64_t i, T *v) const {
        v[0] = x[i];
        v[1] = r[i];
        v[2] = p[i];
        v[3] = q[i];
    }
    __device__ void operator()(const T *f, int64_t i, int c, double *a) const {
        const double pv = f[2], l = al[c];
        x[i] = (T)((double)f[0] + l * pv);
        const double rv = (double)f[1] - l * ((double)f[3] - sig[c] * pv);
        r[i] = (T)rv;
        a[0] += rv * rv;
    }
};

__global__ void cg_alpha_kernel(const double *__restrict__ rr, const double *__restrict__ pap,
                                const int *__restrict__ done, int N, double *__restrict__ al) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= N) return;
    al[k] = (done[k] || !(pap[k] > 0)) ? 0.0 : rr[k] / pap[k];
}

__global__ void cg_beta_kernel(const double *__restrict__ rrn, double *__restrict__ rr,
                               const double *__restrict__ rr0, double tol2, int *__restrict__ done, int N,
                               double *__restrict__ be, int *__restrict__ ndone) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= N) return;
    if (!done[k]) {
        be[k] = rr[k] > 0 ? rrn[k] / rr[k] : 0.0;
        rr[k] = rrn[k];
        if (!(rrn[k] > tol2 * rr0[k])) done[k] = 1;
    } else {
        be[k] = 0.0;
    }
    if (done[k]) atomicAdd(ndone, 1);
}

__global__ void cg_init_kernel(const double *__restrict__ rr, int N, double *__restrict__ rr0,
                               int *__restrict__ done, int *__restrict__ ndone) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k == 0) *ndone = 0;
    if (k >= N) return;
    rr0[k] = rr[k];
    done[k] = rr[k] > 0 ? 0 : 1;
}

__global__ void zero_int_kernel(int *p) { *p = 0; }

template <typename T>
__global__ void __launch_bounds__(256)
cg_p_kernel(T *__restrict__ p, const T *__restrict__ r, const double *__restrict__ be, int64_t np, int B,
            int64_t total) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int c = (int)(i / (np * B)) * B + (int)(i % B);
    p[i] = (T)((double)r[i] + be[c] * (double)p[i]);
}

template <typename T>
__global__ void __launch_bounds__(256)
fill_kernel(T *__restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = T(0);
}

}  // namespace

// ================================================================ handle
struct rs_cnn {
    int max_batch = 0;
    int64_t max_box = 0;
    int64_t adam_t = 0;
    rs::DevBuf params, wt, grad, m, v;
    rs::DevBuf a1, a2, f, u;       // forward activations (max_batch * max_box points)
    rs::DevBuf d1, d2, df, t;      // backward deltas (allocated on first training call)
    rs::DevBuf wpart, lpart, gz, coef, loss;
    rs::DevBuf ss, inv_s, outs, partial;   // preconditioner scratch
    // dense box of the last grid used (its id; 0: none)
    uint64_t box_grid = 0;
    int bdims[3] = {0, 0, 0};      // Z, Y, X
    rs::DevBuf boxpt, boxidx;
};

namespace {

rs_status set_box(rs_cnn *c, const rs_grid *g) {
    if (c->box_grid == g->id) return RS_OK;
    int32_t lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
    for (int64_t p = 0; p < g->np; ++p)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], g->inner[3 * p + a]);
            hi[a] = std::max(hi[a], g->inner[3 * p + a]);
        }
    const int X = hi[0] - lo[0] + 1, Y = hi[1] - lo[1] + 1, Z = hi[2] - lo[2] + 1;
    const int64_t vol = (int64_t)X * Y * Z;
    if (vol > c->max_box) return rs::fail(RS_EINVAL, "cnn: the grid's box exceeds max_box of the network handle");
    std::vector<int32_t> pt(vol, -1), idx(g->np);
    for (int64_t p = 0; p < g->np; ++p) {
        const int64_t q = ((int64_t)(g->inner[3 * p + 2] - lo[2]) * Y + (g->inner[3 * p + 1] - lo[1])) * X +
                          (g->inner[3 * p] - lo[0]);
        pt[q] = (int32_t)p;
        idx[p] = (int32_t)q;
    }
    c->box_grid = 0;   // until both tables are this grid's
    rs_status s = c->boxpt.upload(pt);
    if (!s) s = c->boxidx.upload(idx);
    if (s) return s;
    c->bdims[0] = Z;
    c->bdims[1] = Y;
    c->bdims[2] = X;
    c->box_grid = g->id;
    return RS_OK;
}

// Parameters from the host, in every layout the kernels read.
rs_status upload_params(rs_cnn *c, const float *params) {
    RS_HIP(hipMemcpy(c->params.p, params, kNP * sizeof(float), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(place_kernel, dim3((kNW + 255) / 256), dim3(256), 0, nullptr, c->params.as<float>(),
                       c->wt.as<float>());
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(nullptr));
    return RS_OK;
}

rs_status ensure(rs::DevBuf &b, size_t bytes) { return b.bytes >= bytes ? RS_OK : b.alloc(bytes); }

// f = network(u) for n boxes; activations kept in a1, a2.
rs_status forward(rs_cnn *c, const float *u, float *f, int n, int Z, int Y, int X, int wrap,
                  const int32_t *boxpt, hipStream_t st) {
    const float *P = c->params.as<float>();
    conv8<1, 0, false>(u, c->a1.as<float>(), P + kW1, nullptr, boxpt, n, Z, Y, X, wrap, st);
    conv8<8, 0, true>(c->a1.as<float>(), c->a2.as<float>(), P + kW2, nullptr, boxpt, n, Z, Y, X, wrap, st);
    conv1(c->a2.as<float>(), f, c->wt.as<float>() + kW3T, boxpt, n, Z, Y, X, wrap, st);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

rs_status check_batch(rs_cnn *c, int n, const int32_t *dims, const char *who) {
    if (!c || !dims) return rs::fail(RS_EINVAL, std::string(who) + ": null argument");
    if (n < 1 || dims[0] < 1 || dims[1] < 1 || dims[2] < 1) return rs::fail(RS_EINVAL, std::string(who) + ": empty batch");
    const int64_t vol = (int64_t)dims[0] * dims[1] * dims[2];
    if (n > c->max_batch || vol > c->max_box)
        return rs::fail(RS_EINVAL, std::string(who) + ": batch exceeds the handle's max_batch / max_box");
    return RS_OK;
}

}  // namespace

extern "C" rs_status rs_cnn_create(int32_t max_batch, int64_t max_box, rs_cnn **out) {
    using namespace rs;
    if (!out) return fail(RS_EINVAL, "rs_cnn_create: null out");
    *out = nullptr;
    if (max_batch < 1 || max_box < 1 || (int64_t)max_batch * max_box > (int64_t)1 << 28)
        return fail(RS_EINVAL, "rs_cnn_create: need 1 <= max_batch, max_box and max_batch*max_box <= 2^28");
    auto c = new (std::nothrow) rs_cnn();
    if (!c) return fail(RS_ENOMEM, "host allocation failed");
    c->max_batch = max_batch;
    c->max_box = max_box;
    const size_t pts = (size_t)max_batch * max_box;
    rs_status s = c->params.alloc(kNP * sizeof(float));
    if (!s) s = c->wt.alloc(kNWT * sizeof(float));
    if (!s) s = c->grad.alloc(kNP * sizeof(float));
    if (!s) s = c->m.alloc(kNP * sizeof(float));
    if (!s) s = c->v.alloc(kNP * sizeof(float));
    if (!s) s = c->a1.alloc(pts * 8 * sizeof(float));
    if (!s) s = c->a2.alloc(pts * 8 * sizeof(float));
    if (!s) s = c->f.alloc(pts * sizeof(float));
    if (!s) s = c->u.alloc(pts * sizeof(float));
    if (!s) s = c->gz.alloc((size_t)std::max(max_batch, 256) * 3 * sizeof(double));
    if (!s) s = c->coef.alloc((size_t)std::max(max_batch, 256) * sizeof(double));
    if (!s) s = c->loss.alloc(sizeof(double));
    if (s) { delete c; return s; }
    std::vector<float> zero(kNP, 0.f);
    if (upload_params(c, zero.data()) ||
        hipMemcpy(c->m.p, zero.data(), kNP * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->v.p, zero.data(), kNP * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->grad.p, zero.data(), kNP * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
        delete c;
        return fail(RS_EHIP, "rs_cnn_create: initial copy failed");
    }
    *out = c;
    return RS_OK;
}

extern "C" void rs_cnn_destroy(rs_cnn *c) { delete c; }

extern "C" rs_status rs_cnn_set_params(rs_cnn *c, const float *params) {
    if (!c || !params) return rs::fail(RS_EINVAL, "rs_cnn_set_params: null argument");
    if (const rs_status s = upload_params(c, params)) return s;
    std::vector<float> zero(kNP, 0.f);
    RS_HIP(hipMemcpy(c->m.p, zero.data(), kNP * sizeof(float), hipMemcpyHostToDevice));
    RS_HIP(hipMemcpy(c->v.p, zero.data(), kNP * sizeof(float), hipMemcpyHostToDevice));
    c->adam_t = 0;
    return RS_OK;
}

extern "C" rs_status rs_cnn_get_params(const rs_cnn *c, float *params) {
    if (!c || !params) return rs::fail(RS_EINVAL, "rs_cnn_get_params: null argument");
    RS_HIP(hipMemcpy(params, c->params.p, kNP * sizeof(float), hipMemcpyDeviceToHost));
    return RS_OK;
}

// Checkpoint file: 8-byte tag, int64 parameter count, int64 Adam step count,
// then the parameters and the two Adam moments (float each), little endian.
namespace {
constexpr char kCnnTag[8] = {'R', 'S', 'C', 'N', 'N', '0', '0', '1'};
}

extern "C" rs_status rs_cnn_save(const rs_cnn *c, const char *path) {
    using rs::fail;
    if (!c || !path) return fail(RS_EINVAL, "rs_cnn_save: null argument");
    std::vector<float> buf(3 * (size_t)kNP);
    RS_HIP(hipMemcpy(buf.data(), c->params.p, kNP * sizeof(float), hipMemcpyDeviceToHost));
    RS_HIP(hipMemcpy(buf.data() + kNP, c->m.p, kNP * sizeof(float), hipMemcpyDeviceToHost));
    RS_HIP(hipMemcpy(buf.data() + 2 * kNP, c->v.p, kNP * sizeof(float), hipMemcpyDeviceToHost));
    FILE *f = std::fopen(path, "wb");
    if (!f) return fail(RS_EINVAL, std::string("rs_cnn_save: cannot open ") + path);
    const int64_t hdr[2] = {(int64_t)kNP, c->adam_t};
    bool ok = std::fwrite(kCnnTag, 1, 8, f) == 8 && std::fwrite(hdr, sizeof(int64_t), 2, f) == 2 &&
              std::fwrite(buf.data(), sizeof(float), buf.size(), f) == buf.size();
    ok = (std::fclose(f) == 0) && ok;
    if (!ok) return fail(RS_EINVAL, std::string("rs_cnn_save: write failed: ") + path);
    return RS_OK;
}

extern "C" rs_status rs_cnn_load(rs_cnn *c, const char *path) {
    using rs::fail;
    if (!c || !path) return fail(RS_EINVAL, "rs_cnn_load: null argument");
    FILE *f = std::fopen(path, "rb");
    if (!f) return fail(RS_EINVAL, std::string("rs_cnn_load: cannot open ") + path);
    char tag[8];
    int64_t hdr[2];
    std::vector<float> buf(3 * (size_t)kNP);
    const bool ok = std::fread(tag, 1, 8, f) == 8 && std::memcmp(tag, kCnnTag, 8) == 0 &&
                    std::fread(hdr, sizeof(int64_t), 2, f) == 2 && hdr[0] == kNP && hdr[1] >= 0 &&
                    std::fread(buf.data(), sizeof(float), buf.size(), f) == buf.size();
    std::fclose(f);
    if (!ok) return fail(RS_EINVAL, std::string("rs_cnn_load: not a network checkpoint of this layout: ") + path);
    if (const rs_status s = upload_params(c, buf.data())) return s;
    RS_HIP(hipMemcpy(c->m.p, buf.data() + kNP, kNP * sizeof(float), hipMemcpyHostToDevice));
    RS_HIP(hipMemcpy(c->v.p, buf.data() + 2 * kNP, kNP * sizeof(float), hipMemcpyHostToDevice));
    c->adam_t = hdr[1];
    return RS_OK;
}

extern "C" rs_status rs_cnn_forward(rs_cnn *c, const float *u, float *f, int32_t n, const int32_t dims[3],
                                    int32_t periodic, void *stream) {
    rs_status s = check_batch(c, n, dims, "rs_cnn_forward");
    if (s) return s;
    if (!u || !f) return rs::fail(RS_EINVAL, "rs_cnn_forward: null field");
    return forward(c, u, f, n, dims[0], dims[1], dims[2], periodic ? 1 : 0, nullptr, (hipStream_t)stream);
}

extern "C" rs_status rs_cnn_loss_grad(rs_cnn *c, const float *u, const float *t, const double *sigma, int32_t n,
                                      const int32_t dims[3], double h, int32_t margin, double *loss, float *grad,
                                      float *du, void *stream) {
    using namespace rs;
    rs_status s = check_batch(c, n, dims, "rs_cnn_loss_grad");
    if (s) return s;
    if (!u || !t || !sigma) return fail(RS_EINVAL, "rs_cnn_loss_grad: null field");
    if (!(h > 0) || margin < 0) return fail(RS_EINVAL, "rs_cnn_loss_grad: bad h or margin");
    hipStream_t st = (hipStream_t)stream;
    const int Z = dims[0], Y = dims[1], X = dims[2];
    const int vol = Z * Y * X;
    const int64_t tot = (int64_t)n * vol;
    const unsigned gsz = (unsigned)((tot + 255) / 256);
    const size_t pts = (size_t)c->max_batch * c->max_box;
    const int ntx = (X + kTX - 1) / kTX, nty = (Y + kTY - 1) / kTY, ntz = (Z + kTZ - 1) / kTZ;
    const int nwg = wgrad_groups(tot, (int64_t)ntx * nty * ntz * n);
    const int nch = std::max(1, std::min(64, vol / 4096));
    if ((s = ensure(c->d1, pts * 8 * sizeof(float)))) return s;
    if ((s = ensure(c->d2, pts * 8 * sizeof(float)))) return s;
    if ((s = ensure(c->df, pts * sizeof(float)))) return s;
    if ((s = ensure(c->wpart, std::max<size_t>(kWgMax, (pts + kWgPts - 1) / kWgPts) * kNW * sizeof(float)))) return s;
    if ((s = ensure(c->lpart, (size_t)c->max_batch * 64 * 3 * sizeof(double)))) return s;
    const float *P = c->params.as<float>();
    float *G = c->grad.as<float>(), *WT = c->wt.as<float>();
    float *f = c->f.as<float>(), *df = c->df.as<float>();
    float *a1 = c->a1.as<float>(), *a2 = c->a2.as<float>(), *d1 = c->d1.as<float>(), *d2 = c->d2.as<float>();
    if ((s = forward(c, u, f, n, Z, Y, X, 0, nullptr, st))) return s;
    hipLaunchKernelGGL(gain_kernel, dim3((n + 255) / 256), dim3(256), 0, st, P, sigma, h, n, c->gz.as<double>());
    // energy-norm error terms in the (not yet used) delta buffer d1
    float *em = d1, *tm = d1 + tot, *ae = d1 + 2 * tot, *at = d1 + 3 * tot;
    hipLaunchKernelGGL(err_kernel, dim3(gsz), dim3(256), 0, st, f, t, c->gz.as<double>(), Z, Y, X, margin, n, em, tm);
    hipLaunchKernelGGL(kin_kernel, dim3(gsz), dim3(256), 0, st, em, ae, sigma, h, Z, Y, X, n);
    hipLaunchKernelGGL(kin_kernel, dim3(gsz), dim3(256), 0, st, tm, at, sigma, h, Z, Y, X, n);
    hipLaunchKernelGGL(loss_partial_kernel, dim3(nch, n), dim3(256), 0, st, em, ae, tm, at, f, Z, Y, X, margin, nch,
                       c->lpart.as<double>());
    hipLaunchKernelGGL(loss_final_kernel, dim3(1), dim3(256), 0, st, c->lpart.as<double>(), n, nch,
                       c->gz.as<double>(), c->coef.as<double>(), c->loss.as<double>(), G);
    hipLaunchKernelGGL(df_kernel, dim3(gsz), dim3(256), 0, st, ae, c->gz.as<double>(), c->coef.as<double>(), Z, Y, X,
                       margin, n, df);
    RS_HIP(hipGetLastError());
    // layer 3: weights, then delta of layer 2 (through tanh)
    float *wp = c->wpart.as<float>();
    const dim3 gw((unsigned)nwg);
    hipLaunchKernelGGL((wgrad_kernel<8, 1>), gw, dim3(256), 0, st, a2, df, n, Z, Y, X, ntx, nty, ntz,
                       wp + (int64_t)kW3 * nwg);
    conv8<1, 2, false>(df, d2, WT + kW3, a2, nullptr, n, Z, Y, X, 0, st);
    // layer 2
    hipLaunchKernelGGL((wgrad_kernel<8, 8>), gw, dim3(256), 0, st, a1, d2, n, Z, Y, X, ntx, nty, ntz,
                       wp + (int64_t)kW2 * nwg);
    conv8<8, 2, false>(d2, d1, WT + kW2, a1, nullptr, n, Z, Y, X, 0, st);
    // layer 1
    hipLaunchKernelGGL((wgrad_kernel<1, 8>), gw, dim3(256), 0, st, u, d1, n, Z, Y, X, ntx, nty, ntz,
                       wp + (int64_t)kW1 * nwg);
    hipLaunchKernelGGL(wgrad_final_kernel, dim3((kNW + 63) / 64), dim3(1024), 0, st, wp, nwg, G);
    if (du) conv1(d1, du, WT + kW1, nullptr, n, Z, Y, X, 0, st);
    RS_HIP(hipGetLastError());
    if (loss) RS_HIP(hipMemcpyAsync(loss, c->loss.p, sizeof(double), hipMemcpyDeviceToHost, st));
    if (grad) RS_HIP(hipMemcpyAsync(grad, G, kNP * sizeof(float), hipMemcpyDeviceToHost, st));
    if (loss || grad) RS_HIP(hipStreamSynchronize(st));
    return RS_OK;
}

extern "C" rs_status rs_cnn_adam_step(rs_cnn *c, float lr, float beta1, float beta2, float eps, void *stream) {
    if (!c) return rs::fail(RS_EINVAL, "rs_cnn_adam_step: null handle");
    if (!(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
        return rs::fail(RS_EINVAL, "rs_cnn_adam_step: bad hyper-parameters");
    c->adam_t++;
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)c->adam_t));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)c->adam_t));
    hipLaunchKernelGGL(adam_kernel, dim3((kNP + 255) / 256), dim3(256), 0, (hipStream_t)stream, c->params.as<float>(),
                       c->grad.as<float>(), c->m.as<float>(), c->v.as<float>(), c->wt.as<float>(), lr, beta1, beta2, eps, c1, c2);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

namespace rs {

// out = K(r) for nblk blocks of B states; sigma DEVICE double [nblk*B].
rs_status cnn_precondition(rs_cnn *c, const rs_grid *g, const void *r, const double *sigma, void *out, int nblk,
                           int B, int dtype, hipStream_t st) {
    rs_status s = set_box(c, g);
    if (s) return s;
    const int Z = c->bdims[0], Y = c->bdims[1], X = c->bdims[2];
    const int vol = Z * Y * X;
    const int N = nblk * B;
    const int cb = c->max_batch / B;          // blocks per chunk
    if (cb < 1) return fail(RS_EINVAL, "cnn precondition: max_batch of the network handle is below B");
    const int64_t np = g->np;
    // one chunk size for any number of blocks: a solver that leaves out frozen
    // blocks calls with parts of them, which then neither round differently nor
    // need more scratch than the whole
    const int nchunks = chunk_count(np, B, 1);
    if ((s = ensure(c->ss, (size_t)N * sizeof(double)))) return s;
    if ((s = ensure(c->inv_s, (size_t)N * sizeof(double)))) return s;
    if ((s = ensure(c->outs, (size_t)N * sizeof(double)))) return s;
    if ((s = ensure(c->partial, (size_t)nchunks * N * sizeof(double)))) return s;
    if (dtype == RS_F64)
        s = colreduce<1>(OpSumSq<double>{(const double *)r}, np, B, nblk, 1.0, c->partial.as<double>(),
                         c->ss.as<double>(), st, nullptr, 0, 1);
    else
        s = colreduce<1>(OpSumSq<float>{(const float *)r}, np, B, nblk, 1.0, c->partial.as<double>(),
                         c->ss.as<double>(), st, nullptr, 0, 1);
    if (s) return s;
    hipLaunchKernelGGL(prescale_kernel, dim3((N + 255) / 256), dim3(256), 0, st, c->ss.as<double>(), sigma,
                       c->params.as<float>(), g->h, np, N, c->inv_s.as<double>(), c->outs.as<double>());
    const int wrap = g->kind == RS_GRID_PERIODIC ? 1 : 0;
    for (int b0 = 0; b0 < nblk; b0 += cb) {
        const int nb = std::min(cb, nblk - b0);
        const int k0 = b0 * B;
        if (dtype == RS_F64)
            hipLaunchKernelGGL(scatter_kernel<double>, dim3((vol + 63) / 64, nb), dim3(256), 0, st, (const double *)r,
                               c->boxpt.as<int32_t>(), c->inv_s.as<double>(), k0, B, np, vol, c->u.as<float>());
        else
            hipLaunchKernelGGL(scatter_kernel<float>, dim3((vol + 63) / 64, nb), dim3(256), 0, st, (const float *)r,
                               c->boxpt.as<int32_t>(), c->inv_s.as<double>(), k0, B, np, vol, c->u.as<float>());
        RS_HIP(hipGetLastError());
        if ((s = forward(c, c->u.as<float>(), c->f.as<float>(), nb * B, Z, Y, X, wrap, c->boxpt.as<int32_t>(), st)))
            return s;
        if (dtype == RS_F64)
            hipLaunchKernelGGL(gather_kernel<double>, dim3((unsigned)((np + 511) / 512 * 8), nb), dim3(256), 0, st,
                               c->f.as<float>(), c->boxidx.as<int32_t>(), c->outs.as<double>(), k0, B, np, vol,
                               (double *)out);
        else
            hipLaunchKernelGGL(gather_kernel<float>, dim3((unsigned)((np + 511) / 512 * 8), nb), dim3(256), 0, st,
                               c->f.as<float>(), c->boxidx.as<int32_t>(), c->outs.as<double>(), k0, B, np, vol,
                               (float *)out);
        RS_HIP(hipGetLastError());
    }
    return RS_OK;
}

rs_status check_fields_cnn(const rs_grid *g, int nblk, int B, int dtype, const char *who) {
    if (!g) return fail(RS_EINVAL, std::string(who) + ": null grid");
    if (g->host_only) return fail(RS_EINVAL, std::string(who) + ": grid was built host-only");
    if (!g->kernels_ok) return fail(RS_ENOTSUP, std::string(who) + ": kernels need 4x4x4 bricks");
    if (B < 1 || B > 64 || (B & (B - 1))) return fail(RS_EINVAL, std::string(who) + ": B must be a power of two <= 64");
    if (nblk < 1 || nblk > 65535) return fail(RS_EINVAL, std::string(who) + ": bad nblk");
    if (dtype != RS_F64 && dtype != RS_F32) return fail(RS_EINVAL, std::string(who) + ": bad dtype");
    return RS_OK;
}

}  // namespace rs

extern "C" rs_status rs_cnn_precondition(rs_cnn *c, const rs_grid *g, const void *r, const double *sigma, void *out,
                                         int32_t nblk, int32_t B, int32_t dtype, void *stream) {
    using namespace rs;
    if (!c || !r || !sigma || !out) return fail(RS_EINVAL, "rs_cnn_precondition: null argument");
    rs_status s = check_fields_cnn(g, nblk, B, dtype, "rs_cnn_precondition");
    if (s) return s;
    if (r == out) return fail(RS_EINVAL, "rs_cnn_precondition: r and out must differ");
    return cnn_precondition(c, g, r, sigma, out, nblk, B, dtype, (hipStream_t)stream);
}

extern "C" rs_status rs_cnn_crops(rs_cnn *c, const rs_grid *g, const void *r, const void *x, int32_t nblk, int32_t B,
                                  int32_t dtype, int32_t ncrops, const int32_t *desc, const int32_t cdims[3],
                                  float *u_out, float *t_out, void *stream) {
    using namespace rs;
    if (!c || !r || !x || !desc || !cdims || !u_out || !t_out) return fail(RS_EINVAL, "rs_cnn_crops: null argument");
    rs_status s = check_fields_cnn(g, nblk, B, dtype, "rs_cnn_crops");
    if (s) return s;
    if (ncrops < 1 || cdims[0] < 1 || cdims[1] < 1 || cdims[2] < 1)
        return fail(RS_EINVAL, "rs_cnn_crops: empty crop set");
    if ((int64_t)ncrops * cdims[0] * cdims[1] * cdims[2] > ((int64_t)1 << 31) - 1)
        return fail(RS_EINVAL, "rs_cnn_crops: too many crop points");
    if ((s = set_box(c, g))) return s;
    const int N = nblk * B;
    const int BZ = c->bdims[0], BY = c->bdims[1], BX = c->bdims[2];
    for (int i = 0; i < ncrops; ++i) {
        const int32_t *d = desc + 4 * i;
        if (d[0] < 0 || d[0] >= N || d[1] < 0 || d[1] >= BX || d[2] < 0 || d[2] >= BY || d[3] < 0 || d[3] >= BZ)
            return fail(RS_EINVAL, "rs_cnn_crops: crop state or origin out of range");
    }
    hipStream_t st = (hipStream_t)stream;
    const int64_t np = g->np;
    const int nchunks = chunk_count(np, B, 1);   // as cnn_precondition
    if ((s = ensure(c->ss, (size_t)N * sizeof(double)))) return s;
    if ((s = ensure(c->inv_s, (size_t)N * sizeof(double)))) return s;
    if ((s = ensure(c->partial, (size_t)nchunks * N * sizeof(double)))) return s;
    rs::DevBuf ddesc;
    if ((s = ddesc.upload(std::vector<int32_t>(desc, desc + 4 * (size_t)ncrops)))) return s;
    if (dtype == RS_F64)
        s = colreduce<1>(OpSumSq<double>{(const double *)r}, np, B, nblk, 1.0, c->partial.as<double>(),
                         c->ss.as<double>(), st, nullptr, 0, 1);
    else
        s = colreduce<1>(OpSumSq<float>{(const float *)r}, np, B, nblk, 1.0, c->partial.as<double>(),
                         c->ss.as<double>(), st, nullptr, 0, 1);
    if (s) return s;
    hipLaunchKernelGGL(invs_kernel, dim3((N + 255) / 256), dim3(256), 0, st, c->ss.as<double>(), np, N,
                       c->inv_s.as<double>());
    const int wrap = g->kind == RS_GRID_PERIODIC ? 1 : 0;
    const int64_t tot = (int64_t)ncrops * cdims[0] * cdims[1] * cdims[2];
    const unsigned gsz = (unsigned)((tot + 255) / 256);
    if (dtype == RS_F64)
        hipLaunchKernelGGL(crop_kernel<double>, dim3(gsz), dim3(256), 0, st, (const double *)r, (const double *)x,
                           c->boxpt.as<int32_t>(), ddesc.as<int32_t>(), c->inv_s.as<double>(), B, np, BZ, BY, BX, wrap,
                           cdims[0], cdims[1], cdims[2], ncrops, u_out, t_out);
    else
        hipLaunchKernelGGL(crop_kernel<float>, dim3(gsz), dim3(256), 0, st, (const float *)r, (const float *)x,
                           c->boxpt.as<int32_t>(), ddesc.as<int32_t>(), c->inv_s.as<double>(), B, np, BZ, BY, BX, wrap,
                           cdims[0], cdims[1], cdims[2], ncrops, u_out, t_out);
    RS_HIP(hipGetLastError());
    RS_HIP(hipStreamSynchronize(st));   // the descriptor buffer is freed on return
    return RS_OK;
}

extern "C" rs_status rs_cnn_box(rs_cnn *c, const rs_grid *g, int32_t dims[3]) {
    if (!c || !g || !dims) return rs::fail(RS_EINVAL, "rs_cnn_box: null argument");
    rs_status s = set_box(c, g);
    if (s) return s;
    for (int a = 0; a < 3; ++a) dims[a] = c->bdims[a];
    return RS_OK;
}

// ------------------------------------------------------ shifted solves
namespace {

template <typename T>
rs_status shifted_cg(const rs_grid *g, const T *b, const double *sigma, T *x, int nblk, int B, double tol, int maxit,
                     int *iters, hipStream_t st) {
    using namespace rs;
    const int N = nblk * B;
    const int64_t np = g->np, total = np * N;
    const size_t bytes = (size_t)total * sizeof(T);
    const int nchunks = chunk_count(np, B, nblk);
    rs::DevBuf r, p, q, partial, small, flags;
    rs_status s = r.alloc(bytes);
    if (!s) s = p.alloc(bytes);
    if (!s) s = q.alloc(bytes);
    if (!s) s = partial.alloc((size_t)nchunks * N * sizeof(double));
    if (!s) s = small.alloc((size_t)6 * N * sizeof(double));
    if (!s) s = flags.alloc((size_t)(N + 1) * sizeof(int));
    if (s) return s;
    double *rr = small.as<double>(), *rr0 = rr + N, *pap = rr + 2 * N, *rrn = rr + 3 * N, *al = rr + 4 * N,
           *be = rr + 5 * N;
    int *done = flags.as<int>(), *ndone = done + N;
    const unsigned gm = (unsigned)((total + 255) / 256), gs = (unsigned)((N + 255) / 256);
    hipLaunchKernelGGL(fill_kernel<T>, dim3(gm), dim3(256), 0, st, x, total);
    RS_HIP(hipMemcpyAsync(r.p, b, bytes, hipMemcpyDeviceToDevice, st));
    RS_HIP(hipMemcpyAsync(p.p, b, bytes, hipMemcpyDeviceToDevice, st));
    if ((s = colreduce<1>(OpSumSq<T>{b}, np, B, nblk, 1.0, partial.as<double>(), rr, st))) return s;
    hipLaunchKernelGGL(cg_init_kernel, dim3(gs), dim3(256), 0, st, rr, N, rr0, done, ndone);
    RS_HIP(hipGetLastError());
    const double tol2 = tol * tol;
    int it = 0;
    int nd = 0;
    while (it < maxit) {
        if ((s = kinetic_apply(g, p.p, q.p, nblk, B, sizeof(T) == 8 ? RS_F64 : RS_F32, st))) return s;
        if ((s = colreduce<1>(OpPAp<T>{p.as<T>(), q.as<T>(), sigma}, np, B, nblk, 1.0, partial.as<double>(), pap, st)))
            return s;
        hipLaunchKernelGGL(cg_alpha_kernel, dim3(gs), dim3(256), 0, st, rr, pap, done, N, al);
        if ((s = colreduce<1>(OpCgUpdate<T>{x, r.as<T>(), p.as<T>(), q.as<T>(), sigma, al}, np, B, nblk, 1.0,
                              partial.as<double>(), rrn, st)))
            return s;
        hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, st, ndone);
        hipLaunchKernelGGL(cg_beta_kernel, dim3(gs), dim3(256), 0, st, rrn, rr, rr0, tol2, done, N, be, ndone);
        hipLaunchKernelGGL(cg_p_kernel<T>, dim3(gm), dim3(256), 0, st, p.as<T>(), r.as<T>(), be, np, B, total);
        RS_HIP(hipGetLastError());
        ++it;
        if (it % 10 == 0 || it == maxit) {
            RS_HIP(hipMemcpyAsync(&nd, ndone, sizeof(int), hipMemcpyDeviceToHost, st));
            RS_HIP(hipStreamSynchronize(st));
            if (nd == N) break;
        }
    }
    RS_HIP(hipStreamSynchronize(st));   // scratch is freed on return
    if (iters) *iters = it;
    return nd == N ? RS_OK : fail(RS_ENOTCONV, "rs_shifted_solve: not converged within maxit");
}

}  // namespace

extern "C" rs_status rs_shifted_solve(const rs_grid *g, const void *r, const double *sigma, void *x, int32_t nblk,
                                      int32_t B, int32_t dtype, double tol, int32_t maxit, int32_t *iters,
                                      void *stream) {
    using namespace rs;
    rs_status s = check_fields_cnn(g, nblk, B, dtype, "rs_shifted_solve");
    if (s) return s;
    if (!r || !sigma || !x || r == x) return fail(RS_EINVAL, "rs_shifted_solve: null or aliased argument");
    if (!(tol > 0) || maxit < 1) return fail(RS_EINVAL, "rs_shifted_solve: bad tol or maxit");
    hipStream_t st = (hipStream_t)stream;
    if (dtype == RS_F64)
        return shifted_cg<double>(g, (const double *)r, sigma, (double *)x, nblk, B, tol, maxit, iters, st);
    return shifted_cg<float>(g, (const float *)r, sigma, (float *)x, nblk, B, tol, maxit, iters, st);
}
