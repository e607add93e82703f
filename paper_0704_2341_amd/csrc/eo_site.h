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
    __device__ size_t at(size_t i, int r, int c, int nrhs) const
    {
        return compact ? base + fidx(hs, r, c, nrhs) : i;
    }
};

}  // namespace grg
