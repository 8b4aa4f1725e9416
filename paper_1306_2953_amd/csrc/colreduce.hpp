// Per-state reductions over grid points for fields in the block layout
// [nblk][np][B]: sums with FP64 accumulation, per chunk of points, then a
// fixed-order sum over the chunks (deterministic, independent of timing).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"

namespace rsred {
namespace {

// Points per reduction chunk: as many as leave about 2048 work-groups (8 per
// CU, enough loads in flight to stream), at least 8 per thread (the tree over
// a work-group's rows and the final sum then stay small) and at most 2048.
// With 2048 points everywhere a grid of 26k points ran on 13 work-groups:
// reductions of 32 states took 40-195 us each, now 5-12; 262k points and 128
// FP32 states, 512 work-groups: 156-398 us, now 143-190.
constexpr int kMaxChunk = 2048;
inline int chunk_points(int64_t np, int B, int nblk) {
    const int64_t lo = 8 * (256 / B), want = (np * nblk + 2047) / 2048;
    return (int)std::min<int64_t>(kMaxChunk, std::max<int64_t>(lo, (want + 63) / 64 * 64));
}
inline int chunk_count(int64_t np, int B, int nblk) {
    const int c = chunk_points(np, B, nblk);
    return (int)((np + c - 1) / c);
}

// partial[k][chunk][col], col = blk * B + s.  One work-group per (chunk,
// block); lanes: state s, rows r striding over the chunk's points.  With a
// block map, grid row y covers block bmap[y] (the other blocks' partial
// sums are left as they are).  An Op names the type T of its NF fields,
// loads them at element i (load) and adds their products (operator()): the
// loads of several points are issued before any is used.  Left to itself the
// compiler kept one load in flight where there are many sums (6 fields, 11
// sums, 262k points and 128 FP32 states: 352 us, now 142).
template <int K, typename Op>
__global__ void __launch_bounds__(256)
colreduce_kernel(Op op, int64_t np, int B, int chunk, int nchunks, int N, double *__restrict__ partial,
                 const int *__restrict__ bmap) {
    __shared__ double red[K][256];
    const int blk = bmap ? bmap[blockIdx.y] : (int)blockIdx.y, tid = threadIdx.x;
    const int s = tid % B, r = tid / B, R = 256 / B;
    const int64_t p0 = (int64_t)blockIdx.x * chunk, p1 = min<int64_t>(np, p0 + chunk);
    const int col = blk * B + s;
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    constexpr int NF = Op::NF, U = NF <= 2 ? 8 : 4;
    for (int64_t p = p0 + r; p < p1; p += U * R) {
        typename Op::T v[U][NF];
#pragma unroll
        for (int u = 0; u < U; ++u)
            op.load((int64_t)blk * np * B + min<int64_t>(p + u * R, p1 - 1) * B + s, v[u]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (p + u * R < p1) op(v[u], (int64_t)blk * np * B + (p + u * R) * B + s, col, acc);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) red[k][tid] = acc[k];
    __syncthreads();
    for (int st = R / 2; st > 0; st >>= 1) {
        if (r < st)
#pragma unroll
            for (int k = 0; k < K; ++k) red[k][tid] += red[k][tid + st * B];
        __syncthreads();
    }
    if (r == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) partial[((int64_t)k * nchunks + blockIdx.x) * N + col] = red[k][s];
}

// One wave per output: lanes sum strided chunks, then a fixed butterfly.
__global__ void __launch_bounds__(256)
colreduce_final(const double *__restrict__ partial, int K, int nchunks, int N, double dv, double *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int idx = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (idx >= K * N) return;
    const int k = idx / N, c = idx % N;
    double s = 0.0;
    for (int ch = lane; ch < nchunks; ch += 64) s += partial[((int64_t)k * nchunks + ch) * N + c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) out[idx] = dv * s;
}

// The sums of every column, handed to f(column, sums): 8 columns x 32 shares
// of the chunks per work-group, added in a fixed order; one thread per column
// then runs f, so a per-state solve needs no launch of its own.
template <int K, typename F>
__global__ void __launch_bounds__(256)
colreduce_apply(const double *__restrict__ partial, int nchunks, int N, double dv, F f) {
    __shared__ double red[K][32][8];
    const int s = threadIdx.x % 8, r = threadIdx.x / 8, c = blockIdx.x * 8 + s;
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    if (c < N)
#pragma unroll 2
        for (int ch = r; ch < nchunks; ch += 32)
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] += partial[((int64_t)k * nchunks + ch) * N + c];
#pragma unroll
    for (int k = 0; k < K; ++k) red[k][r][s] = acc[k];
    __syncthreads();
    if (r < K) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < 32; ++i) t += red[r][i][s];
        red[r][0][s] = dv * t;
    }
    __syncthreads();
    if (r == 0 && c < N) {
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] = red[k][0][s];
        f(c, acc);
    }
}

// Partial sums of all columns, or with bmap (device, nmap entries) of the
// listed blocks.  The chunks, and with them a sum's rounding, are those of `of`
// blocks.
template <int K, typename Op>
rs_status colreduce_partial(const Op &op, int64_t np, int B, int nblk, double *partial, hipStream_t st,
                            const int *bmap, int nmap, int of) {
    const int N = nblk * B, nchunks = chunk_count(np, B, of);
    hipLaunchKernelGGL((colreduce_kernel<K, Op>), dim3(nchunks, bmap ? nmap : nblk), dim3(256), 0, st, op, np, B,
                       chunk_points(np, B, of), nchunks, N, partial, bmap);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// Sums for all nblk * B columns; with bmap (device, nmap entries) only the
// listed blocks are reduced this time and the other columns' outputs repeat
// whatever their partial sums last held.  A caller that works through parts of
// a problem gives one `of` for all of them (0: nblk): a column's sum is then the
// same in any part, and nblk * B * chunk_count(np, B, of) partial sums grow with
// nblk.
template <int K, typename Op>
rs_status colreduce(const Op &op, int64_t np, int B, int nblk, double dv, double *partial, double *out,
                    hipStream_t st, const int *bmap = nullptr, int nmap = 0, int of = 0) {
    if (of == 0) of = nblk;
    const int N = nblk * B, nchunks = chunk_count(np, B, of);
    rs_status e = colreduce_partial<K>(op, np, B, nblk, partial, st, bmap, nmap, of);
    if (e) return e;
    hipLaunchKernelGGL(colreduce_final, dim3((K * N + 3) / 4), dim3(256), 0, st, partial, K, nchunks, N, dv,
                       out);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// The same sums handed to f (colreduce_apply).
template <int K, typename Op, typename F>
rs_status colreduce_then(const Op &op, int64_t np, int B, int nblk, double dv, double *partial, const F &f,
                         hipStream_t st, const int *bmap = nullptr, int nmap = 0) {
    static_assert(K <= 32, "one row of threads per sum");
    const int N = nblk * B, nchunks = chunk_count(np, B, nblk);
    rs_status e = colreduce_partial<K>(op, np, B, nblk, partial, st, bmap, nmap, nblk);
    if (e) return e;
    hipLaunchKernelGGL((colreduce_apply<K, F>), dim3((N + 7) / 8), dim3(256), 0, st, partial, nchunks, N, dv, f);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

}  // namespace
}  // namespace rsred
