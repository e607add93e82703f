// Fixed-order sums of per-workgroup partials.  They lie as [RHS][sum][workgroup],
// so that a reduction reads whole lines: with the workgroup outermost each of
// 4096 workgroups' three sums for 8 RHS lay in a line of its own (7.9 us per
// reduction against 5).  Only the many-lattice batch keeps the workgroup
// outermost: its workgroups write a row of hundreds of systems, which
// scattered cost more (13 us per stencil) than its reductions gain (4 us).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace grg {

// Threads of a reduction workgroup for n rows: enough that a thread's rows are
// one round of loads or two.
inline int reduce_threads(int n) { return n > 1024 ? 1024 : 256; }

// acc[k] = sum over i < n of partials[(r K + k) n + i] (or, with nrows > 0, of
// partials[i nrows K + r K + k]), by the whole workgroup
// (at most 1024 threads; thread 0 gets the result): each thread its rows
// in order, four loads issued before any is added (the partials come from
// another kernel: each load is a round trip to L2 or memory), then the
// wavefronts, then the workgroup, always in the same order.
template <int K>
__device__ __forceinline__ void block_rows_sum(const double *__restrict__ partials, int n, int r,
                                               double (&acc)[3], int nrows = 0)
{
    __shared__ double sm[16][3];
    const int T = blockDim.x;
    const size_t di = nrows ? (size_t)nrows * K : 1, dk = nrows ? 1 : n, r0 = nrows ? (size_t)r * K : (size_t)r * K * n;
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * T < n; i += 4 * T) {
        double v[4][K];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) v[u][k] = partials[r0 + k * dk + (size_t)(i + u * T) * di];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] += v[u][k];
    }
    for (; i < n; i += T)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += partials[r0 + k * dk + (size_t)i * di];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
        if (lane == 0) sm[wave][k] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < T >> 6; ++w)
            for (int k = 0; k < K; ++k) acc[k] += sm[w][k];
}

// The same sums by one wavefront (every lane gets them), in an order of its own
// that is the same in every wavefront: for the vector kernels that take their
// scalars straight from the partials (a few hundred rows).
template <int K>
__device__ __forceinline__ void wave_rows_sum(const double *__restrict__ partials, int n, int r, double (&acc)[K])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    int i = lane;
    for (; i + 3 * 64 < n; i += 4 * 64) {
        double v[4][K];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) v[u][k] = partials[(size_t)(r * K + k) * n + i + u * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] += v[u][k];
    }
    for (; i < n; i += 64)
#pragma unroll
        for (int k = 0; k < K; ++k) acc[k] += partials[(size_t)(r * K + k) * n + i];
#pragma unroll
    for (int k = 0; k < K; ++k)
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
}

// alpha = <q, r> / |q|^2 from the sums (re, im, |q|^2)
__device__ __forceinline__ double2 mr_alpha(const double (&s)[3], bool on)
{
    return on && s[2] > 0 ? make_double2(s[0] / s[2], s[1] / s[2]) : make_double2(0.0, 0.0);
}
// BiCGstab: alpha = rho / <r0, v> from the sums of conj(v) r0
__device__ __forceinline__ double2 bicg_alpha(double2 rho, const double (&s)[3], bool on)
{
    // <r0, v> = conj(sum conj(v) r0)
    const double sr = s[0], si = -s[1];
    const double den = sr * sr + si * si;
    return on && den > 0 ? make_double2((rho.x * sr + rho.y * si) / den, (rho.y * sr - rho.x * si) / den)
                         : make_double2(0.0, 0.0);
}
// beta = (rho' / rho) (alpha / omega)
__device__ __forceinline__ double2 bicg_beta(double2 rn, double2 rho, double2 al, double2 om, bool on)
{
    const double d1 = rho.x * rho.x + rho.y * rho.y, d2 = om.x * om.x + om.y * om.y;
    if (!on || !(d1 > 0) || !(d2 > 0)) return make_double2(0.0, 0.0);
    const double2 q1 = make_double2((rn.x * rho.x + rn.y * rho.y) / d1, (rn.y * rho.x - rn.x * rho.y) / d1);
    const double2 q2 = make_double2((al.x * om.x + al.y * om.y) / d2, (al.y * om.x - al.x * om.y) / d2);
    return make_double2(q1.x * q2.x - q1.y * q2.y, q1.x * q2.y + q1.y * q2.x);
}

}  // namespace grg
