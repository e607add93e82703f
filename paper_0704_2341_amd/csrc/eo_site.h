// Sites of the compact parity halves, and where the defect correction's
// element lies: shared by the stencils' forms.
#pragma once

#include "common.h"
#include "engine.h"
#include "stencil.h"

namespace grg {

// site of half index h with parity p, and its coordinates
__device__ __forceinline__ int eo_site(int h, int p, const Geom &g, SiteGeo &q)
{
    const int s0 = 2 * h;
    q = site_geo(s0, g);
    const int b = (p ^ q.c[1] ^ q.c[2] ^ q.c[3]) & 1;  // parity of s0 is y + z + t (x0 even)
    q.c[0] += b;
    return s0 + b;
}

// The compact parity halves and their links.  In FP32 two components share 16
// bytes of a lane: the L1 answers a wavefront's 8-byte loads at half the rate
// of its 16-byte ones (16 cache accesses for 512 bytes and for 1024), and the
// half-steps read 21 complex numbers per hop.  BF16 (4 bytes: 4 accesses for
// 256 bytes) and FP64 keep a component per lane and line.
template <class S>
__device__ __forceinline__ size_t hidx(int H, int r, int c, int nrhs)
{
    if constexpr (sizeof(S) == 8)
        return ((size_t)(H >> 6) * nrhs + r) * 768 + (c >> 1) * 128 + (H & 63) * 2 + (c & 1);
    else
        return fidx(H, r, c, nrhs);
}

template <class S>
__device__ __forceinline__ size_t hlidx(int H, int mu, int e)
{
    if constexpr (sizeof(S) == 8)
        return (size_t)(H >> 6) * 2304 + mu * 576 + (e < 8 ? (e >> 1) * 128 + (H & 63) * 2 + (e & 1) : 512 + (H & 63));
    else
        return lidx(H, mu, e);
}

// a site's spinor and a link in the operand form of the hops
template <class S, class R, class T>
__device__ __forceinline__ void load_half(T (&p)[12], const S *__restrict__ f, int H, int r, int nrhs)
{
    if constexpr (sizeof(S) == 8) {
        const float4 *q = (const float4 *)(f + hidx<S>(H, r, 0, nrhs));
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const float4 v = q[i * 64];
            p[2 * i] = {v.x, v.y};
            p[2 * i + 1] = {v.z, v.w};
        }
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = Operand<S, R>::load(f, hidx<S>(H, r, c, nrhs));
    }
}

template <class S, class R, class T>
__device__ __forceinline__ void load_half_link(T (&u)[9], const S *__restrict__ U, int H, int mu)
{
    if constexpr (sizeof(S) == 8) {
        const float4 *q = (const float4 *)(U + hlidx<S>(H, mu, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 v = q[i * 64];
            u[2 * i] = {v.x, v.y};
            u[2 * i + 1] = {v.z, v.w};
        }
        const float2 v = U[hlidx<S>(H, mu, 8)];
        u[8] = {v.x, v.y};
    } else {
#pragma unroll
        for (int e = 0; e < 9; ++e) u[e] = Operand<S, R>::load(U, hlidx<S>(H, mu, e));
    }
}

// its values
template <class S, class R>
__device__ __forceinline__ void load_half_vals(cpx<R> (&p)[12], const S *__restrict__ f, int H, int r, int nrhs)
{
    if constexpr (sizeof(S) == 8) {
        load_half<S, R>(p, f, H, r, nrhs);
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = ldc(f, hidx<S>(H, r, c, nrhs));
    }
}

template <class S, class R>
__device__ __forceinline__ void store_half(S *__restrict__ f, const cpx<R> (&p)[12], int H, int r, int nrhs)
{
    if constexpr (sizeof(S) == 8) {
        float4 *q = (float4 *)(f + hidx<S>(H, r, 0, nrhs));
#pragma unroll
        for (int i = 0; i < 6; ++i) q[i * 64] = make_float4(p[2 * i].re, p[2 * i].im, p[2 * i + 1].re, p[2 * i + 1].im);
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) stc(f, hidx<S>(H, r, c, nrhs), p[c]);
    }
}

// The defect correction's residual element i, stored in FP64 or (late steps,
// DcArgs::r_in32 / r_out32) in FP32 at the same element index.
__device__ __forceinline__ double2 dc_load_r(const DcArgs &a, const double2 *r, size_t i)
{
    if (a.r_in32) {
        const float2 v = ((const float2 *)r)[i];
        return make_double2((double)v.x, (double)v.y);
    }
    return r[i];
}
__device__ __forceinline__ void dc_store_r(const DcArgs &a, double2 *r, size_t i, double2 v)
{
    if (a.r_out32) ((float2 *)r)[i] = make_float2((float)v.x, (float)v.y);
    else r[i] = v;
}

// Where r_next's element (r, c) of site s goes: the full layout (i), or the
// compact half of the site's parity at its compact index s / 2.
struct DcNext {
    size_t base = 0;
    int hs;
    bool compact;
    __device__ DcNext(const DcArgs &a, int s) : hs(s), compact(a.next_half != 0)
    {
        if (compact) {
            const SiteGeo q = site_geo(s, a.g);
            base = ((q.c[0] ^ q.c[1] ^ q.c[2] ^ q.c[3]) & 1) == a.next_par ? 0 : a.next_half;
            hs = s >> 1;
        }
    }
    template <class S>
    __device__ size_t at(const S *, size_t i, int r, int c, int nrhs) const
    {
        return compact ? base + hidx<S>(hs, r, c, nrhs) : i;
    }
};

}  // namespace grg
