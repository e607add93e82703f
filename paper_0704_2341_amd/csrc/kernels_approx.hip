// The Schur complement approximations of section 3, on the sites that matter.
//
// With d = 4 + m0, d~ the row sums of D_rr and u = x_b on the coarse sites,
//     S~_bb x = [D w]_b,  w = u - ((y - z) / d + t),  y = D_rb x, t = y / d~, z = D_rr t
// (and S0_bb x the same with w = u - y / d).  y and t vanish except on the
// rest sites next to a coarse site (the boundary), and [D w]_b reads w on the
// coarse sites and the boundary only, so y, t, z and w are formed on the
// boundary alone, in compact fields over its sites: with the all-even coarse
// set 4 of the 15 rest sites in 16.  At 32^4 with 12 RHS the six passes over the
// whole lattice took 7.7 ms (9.4 with the former stencil launch).
//
// A rest site off the boundary has y = 0, so t = 0 there, unless its row sum
// is zero or not finite: then 0 / d~ is not a number and spreads to its
// neighbours, here as in the formula (kBadRow marks such sites).
#include <algorithm>

#include "common.h"
#include "engine.h"
#include "split.h"

namespace grg {

constexpr int kBadRow = -2;

// ------------------------------------------------------------------ the boundary
// flag of site s: a rest site with a coarse neighbour
__device__ __forceinline__ bool on_boundary(int s, const Geom &g, const int32_t *__restrict__ bidx)
{
    if (s >= g.V || bidx[s] >= 0) return false;
    const SiteGeo q = site_geo(s, g);
    bool b = false;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        int sp, sm;
        nbr(s, mu, q, g, sp, sm);
        b = b || bidx[sp] >= 0 || bidx[sm] >= 0;
    }
    return b;
}

// A first call makes the tables in two launches and, with rows, a third; nothing is
// read back: the kernels after them take the number of boundary sites from info[0],
// and the last one of the call leaves what later calls want in pinned words.  (List,
// map and counts allocated by themselves and three waits for the host: first
// S~_bb on 8^4, 1 RHS, 97 us against 78 over the whole lattice.)
constexpr int kBoundaryBlock = 1024;

// per block of sites, the boundary sites' number
__global__ void __launch_bounds__(kBoundaryBlock) boundary_count_kernel(Geom g, const int32_t *__restrict__ bidx,
                                                                        int *count, int *info)
{
    __shared__ int n[16];
    const int s = blockIdx.x * kBoundaryBlock + threadIdx.x;
    const unsigned long long m = __ballot(on_boundary(s, g, bidx));
    if ((threadIdx.x & 63) == 0) n[threadIdx.x >> 6] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < 16; ++w) t += n[w];
        count[blockIdx.x] = t;
        if (blockIdx.x == 0) info[1] = 0;
    }
}

// site[j] = the j-th boundary site in lattice order, map[s] = its j, or -1;
// info[0] the sites' number.  Each block adds the counts before it itself.
__global__ void __launch_bounds__(kBoundaryBlock) boundary_fill_kernel(Geom g, const int32_t *__restrict__ bidx,
                                                                       const int *__restrict__ count, int32_t *site,
                                                                       int32_t *map, int *info)
{
    __shared__ int n[16], before[16];
    const int s = blockIdx.x * kBoundaryBlock + threadIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int sum = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kBoundaryBlock) sum += count[i];
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const bool b = on_boundary(s, g, bidx);
    const unsigned long long m = __ballot(b);
    if (lane == 0) {
        n[wave] = __popcll(m);
        before[wave] = sum;
    }
    __syncthreads();
    int j = __popcll(m & ((1ull << lane) - 1));
    for (int w = 0; w < 16; ++w) j += before[w] + (w < wave ? n[w] : 0);
    if (b) site[j] = s;
    if (s < g.V) map[s] = b ? j : -1;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kBoundaryBlock - 1) info[0] = j + (b ? 1 : 0);
}

// The row sums d~ = D_rr 1 of the rest sites (the sums of the stencil on a field
// that is 1 there); rest sites off the boundary: kBadRow where a row sum's 0 / d~
// is not zero; info[1] = stamp if a boundary site has a neighbour with t != 0 (one
// on the boundary, or a kBadRow site).
__global__ void __launch_bounds__(256) boundary_rows_kernel(Geom g, const int32_t *__restrict__ bidx,
                                                            const double2 *__restrict__ U, double diag,
                                                            double2 *__restrict__ rows, int32_t *map, int *info,
                                                            int stamp)
{
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V || bidx[s] >= 0) return;
    const SiteGeo q = site_geo(s, g);
    cpx<double> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = {diag, 0.0};
    bool near = false;  // a neighbour is on the boundary
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
        int sp, sm;
        nbr(s, mu, q, g, sp, sm);
        cpx<double> uf[9], ub[9], pf[12], pb[12];
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const double2 f = U[lidx(s, mu, e)], w = U[lidx(sm, mu, e)];
            uf[e] = {f.x, f.y};
            ub[e] = {w.x, w.y};
        }
        const double vf = bidx[sp] < 0 ? 1.0 : 0.0, vb = bidx[sm] < 0 ? 1.0 : 0.0;
        // (a neighbour's entry may be changing between its negative values)
        near = near || map[sp] >= 0 || map[sm] >= 0;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            pf[c] = {vf, 0.0};
            pb[c] = {vb, 0.0};
        }
        switch (mu) {
        case 0: hop_math<0, true>(acc, pf, uf); hop_math<0, false>(acc, pb, ub); break;
        case 1: hop_math<1, true>(acc, pf, uf); hop_math<1, false>(acc, pb, ub); break;
        case 2: hop_math<2, true>(acc, pf, uf); hop_math<2, false>(acc, pb, ub); break;
        default: hop_math<3, true>(acc, pf, uf); hop_math<3, false>(acc, pb, ub); break;
        }
    }
    bool t_set = map[s] >= 0;
#pragma unroll
    for (int c = 0; c < 12; ++c) rows[fidx(s, 0, c, 1)] = make_double2(acc[c].re, acc[c].im);
    if (!t_set) {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const double den = acc[c].re * acc[c].re + acc[c].im * acc[c].im;
            t_set = t_set || !(den > 0.0 && isfinite(den));
        }
        map[s] = t_set ? kBadRow : -1;
    }
    if (t_set && near) info[1] = stamp;
}

// t = a / b as the formula divides
__device__ __forceinline__ cpx<double> row_divide(double2 a, double2 b)
{
    const double den = b.x * b.x + b.y * b.y;
    return {(a.x * b.x + a.y * b.y) / den, (a.y * b.x - a.x * b.y) / den};
}

// -w = (y - z) / d + t, in the formula's order: where z is close to y (row sums
// close to d), y / d + t - z / d has up to three times its rounding error
__device__ __forceinline__ double minus_w(double y, double z, double t, double inv_d)
{
    return (y - z) * inv_d + t;
}

// c v, rounded (not fused into what it is subtracted from): the bits of a z that is
// formed in a pass of its own
__device__ __forceinline__ cpx<double> scaled(double c, cpx<double> v)
{
#pragma clang fp contract(off)
    return {c * v.re, c * v.im};
}

// ------------------------------------------------------------------ the fields
// Boundary site j, RHS r: y = (D x)_j from its coarse neighbours, then p = -w
// or what it is formed from:
//   kNoRows   p = y / d                                  (S0_bb)
//   kTwoPass  p = y, and t, from which boundary_apply_kernel forms z and -w
//   kOnePass  p = (y - z) / d + t with z = d t: no neighbour carries a t (the
//             all-even coarse set, where this saves writing t and three more
//             passes over the boundary: S~_bb at 32^4 with 12 RHS 1.18 ms in
//             two passes)
// FIRST: the number of sites, and which of the last two forms, from info (a variant
// of its own: looking there costs every call 0.3 us).
// Work items (256 boundary sites, RHS), RHS fastest: the RHS share the links
// in L2.
enum { kNoRows = 0, kTwoPass = 1, kOnePass = 2 };
template <int MODE, bool FIRST>
__global__ void __launch_bounds__(256) boundary_source_kernel(Geom g, const double2 *__restrict__ xb,
                                                              const int32_t *__restrict__ bidx, int nb,
                                                              const double2 *__restrict__ U,
                                                              const double2 *__restrict__ rows,
                                                              const int32_t *__restrict__ site, int most,
                                                              const int *__restrict__ info, int stamp, double diag,
                                                              double inv_d, double2 *__restrict__ t,
                                                              double2 *__restrict__ p, int nrhs)
{
    __shared__ double2 lds[4][64 * kSpinorRow];
    const int nbnd = FIRST ? info[0] : most;
    const bool two = MODE == kTwoPass && (!FIRST || info[1] == stamp);
    const int nsb = (nbnd + 255) >> 8;
    const ItemRange it = xcd_items(nsb * nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int sb = w / nrhs, r = w - sb * nrhs;
        const int j = sb * 256 + (int)threadIdx.x;
        const bool in = j < nbnd;
        const int s = in ? site[j] : 0;
        const SiteGeo q = site_geo(s, g);
        const double2 *x = xb + (size_t)r * nb * 12;
        cpx<double> acc[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = {0, 0};
        coarse_hops(acc, x, bidx, U, s, in, q, g, lds[threadIdx.x >> 6]);
        if (!in) continue;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const size_t i = fidx(j, r, c, nrhs);
            cpx<double> pv = acc[c];
            if constexpr (MODE == kNoRows) {
                pv = {acc[c].re * inv_d, acc[c].im * inv_d};
            } else {
                const cpx<double> tv = row_divide(make_double2(acc[c].re, acc[c].im), rows[fidx(s, 0, c, 1)]);
                if (two) {
                    t[i] = make_double2(tv.re, tv.im);
                } else {
                    const cpx<double> z = scaled(diag, tv);
                    pv = {minus_w(acc[c].re, z.re, tv.re, inv_d), minus_w(acc[c].im, z.im, tv.im, inv_d)};
                }
            }
            p[i] = make_double2(pv.re, pv.im);
        }
    }
}

// p (y) <- -w on the boundary, z = D_rr t from the neighbours on it
// (t = 0 off it, but for the kBadRow sites)
template <bool FIRST>
__global__ void __launch_bounds__(256) boundary_apply_kernel(Geom g, const double2 *__restrict__ U,
                                                             const double2 *__restrict__ rows,
                                                             const int32_t *__restrict__ site,
                                                             const int32_t *__restrict__ map, int most,
                                                             const int *__restrict__ info, int stamp, double diag,
                                                             double inv_d,
                                                             const double2 *__restrict__ t, double2 *p, int nrhs)
{
    // this site's t, wanted again at the end (read twice, 762 -> 808 us for the whole
    // S~_bb on the inverse Type II ordering at 32^4, 12 RHS; it does not fit the
    // registers), and its neighbours, asked for all together
    __shared__ double2 own[12][256];
    __shared__ int nbj[8][256];
    if (FIRST && info[1] != stamp) return;  // p is -w already
    const int nbnd = FIRST ? info[0] : most;
    const int nsb = (nbnd + 255) >> 8;
    const ItemRange it = xcd_items(nsb * nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int sb = w / nrhs, r = w - sb * nrhs;
        const int j = sb * 256 + (int)threadIdx.x;
        if (j >= nbnd) continue;
        const int s = site[j];
        const SiteGeo q = site_geo(s, g);
        cpx<double> acc[12];
        int jk[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            int sp, sm;
            nbr(s, k >> 1, q, g, sp, sm);
            jk[k] = map[(k & 1) ? sm : sp];
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const double2 v = t[fidx(j, r, c, nrhs)];
            acc[c] = {diag * v.x, diag * v.y};
            own[c][threadIdx.x] = v;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) nbj[k][threadIdx.x] = jk[k];
        asm volatile("" ::: "memory");
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
            const int mu = k >> 1;
            const int jn = nbj[k][threadIdx.x];
            if (jn == -1) continue;  // coarse, or t = 0
            int sp, sm;
            nbr(s, mu, q, g, sp, sm);
            const int n = (k & 1) ? sm : sp;
            cpx<double> v[12], u[9];
            if (jn >= 0) {
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const double2 x = t[fidx(jn, r, c, nrhs)];
                    v[c] = {x.x, x.y};
                }
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) v[c] = row_divide(make_double2(0.0, 0.0), rows[fidx(n, 0, c, 1)]);
            }
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 l = U[lidx((k & 1) ? sm : s, mu, e)];
                u[e] = {l.x, l.y};
            }
            switch (k) {
            case 0: hop_math<0, true>(acc, v, u); break;
            case 1: hop_math<0, false>(acc, v, u); break;
            case 2: hop_math<1, true>(acc, v, u); break;
            case 3: hop_math<1, false>(acc, v, u); break;
            case 4: hop_math<2, true>(acc, v, u); break;
            case 5: hop_math<2, false>(acc, v, u); break;
            case 6: hop_math<3, true>(acc, v, u); break;
            default: hop_math<3, false>(acc, v, u); break;
            }
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const size_t i = fidx(j, r, c, nrhs);
            const double2 y = p[i], tv = own[c][threadIdx.x];
            p[i] = make_double2(minus_w(y.x, acc[c].re, tv.x, inv_d), minus_w(y.y, acc[c].im, tv.y, inv_d));
        }
    }
}

// y_b = [D w]_b, w = x_b on the coarse sites and -p on the boundary: every
// neighbour of a coarse site is one or the other.  64 coarse sites and one RHS
// per workgroup, a hop per wavefront (split.h), RHS fastest.  FIRST: the values of
// info also go to the pinned words `host` (see ApproxArgs).
template <bool FIRST>
__global__ void __launch_bounds__(kSplitThreads) boundary_coarse_kernel(Geom g, const double2 *__restrict__ xb,
                                                                        const int32_t *__restrict__ qsites,
                                                                        const int32_t *__restrict__ bidx, int nb,
                                                                        const int32_t *__restrict__ map,
                                                                        const double2 *__restrict__ U, double diag,
                                                                        const double2 *__restrict__ p,
                                                                        double2 *__restrict__ yb, int nrhs,
                                                                        const int *__restrict__ info, int *host,
                                                                        int stamp)
{
    __shared__ HopSums<double> sums;
    if (FIRST && blockIdx.x == 0 && threadIdx.x == 0) {
        __hip_atomic_store(host, info[0] + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (stamp)
            __hip_atomic_store(host + 1, info[1] == stamp ? stamp : -stamp, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    }
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nkb = (nb + 63) >> 6;
    const ItemRange it = xcd_items(nkb * nrhs);
    for (int wi = it.begin; wi < it.end; wi += it.step) {
        const int kb = wi / nrhs, r = wi - kb * nrhs;
        const int kc = kb * 64 + lane;
        if (kc < nb) {
            const int s = qsites[kc];
            const SiteGeo q = site_geo(s, g);
            const int mu = k >> 1;
            int sp, sm;
            nbr(s, mu, q, g, sp, sm);
            const int n = (k & 1) ? sm : sp;
            const int kn = bidx[n];
            cpx<double> v[12], u[9], w[6];
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 l = U[lidx((k & 1) ? sm : s, mu, e)];
                u[e] = {l.x, l.y};
            }
            if (kn >= 0) {
                const double2 *x = xb + ((size_t)r * nb + kn) * 12;
#pragma unroll
                for (int c = 0; c < 12; ++c) v[c] = {x[c].x, x[c].y};
            } else {
                const int jn = map[n];
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const double2 x = p[fidx(jn, r, c, nrhs)];
                    v[c] = {-x.x, -x.y};
                }
            }
            hop_w_k(k, w, v, u);
            sums.put(k, lane, w);
        }
        __syncthreads();
        if (k < 6 && kc < nb) {
            const int row = k % 3, spin = k < 3 ? 0 : 2;
            const size_t i = ((size_t)r * nb + kc) * 12 + 3 * spin + row;
            const double2 x0 = xb[i], x1 = xb[i + 3];
            cpx<double> a0 = {diag * x0.x, diag * x0.y}, a1 = {diag * x1.x, diag * x1.y};
            if (spin == 0) sums.add<false>(row, lane, a0, a1);
            else sums.add<true>(row, lane, a0, a1);
            yb[i] = make_double2(a0.re, a0.im);
            yb[i + 3] = make_double2(a1.re, a1.im);
        }
        __syncthreads();  // the sums are read before the next item's overwrite them
    }
}

// ------------------------------------------------------------------ launchers
static inline int round8_grid(long n)
{
    n = std::min<long>(n, kMaxGridValue);
    return (int)std::max<long>(8, (n + 7) / 8 * 8);
}

int boundary_blocks(const Geom &g) { return (g.V + kBoundaryBlock - 1) / kBoundaryBlock; }

hipError_t launch_boundary_build(const Geom &g, const int32_t *bidx, int *count, int32_t *site, int32_t *map,
                                 int *info, hipStream_t st)
{
    const int n = boundary_blocks(g);
    hipLaunchKernelGGL(boundary_count_kernel, dim3(n), dim3(kBoundaryBlock), 0, st, g, bidx, count, info);
    hipLaunchKernelGGL(boundary_fill_kernel, dim3(n), dim3(kBoundaryBlock), 0, st, g, bidx, (const int *)count, site,
                       map, info);
    return hipGetLastError();
}

hipError_t launch_boundary_rows(const Geom &g, const int32_t *bidx, const void *U, double diag, void *rows,
                                int32_t *map, int *info, int stamp, hipStream_t st)
{
    hipLaunchKernelGGL(boundary_rows_kernel, dim3((g.V + 255) / 256), dim3(256), 0, st, g, bidx, (const double2 *)U,
                       diag, (double2 *)rows, map, info, stamp);
    return hipGetLastError();
}

hipError_t launch_boundary_source(const ApproxArgs &a, hipStream_t st)
{
    if (a.nrhs < 1 || a.nrhs > kMaxRhs || a.nb < 1 || a.nbnd < 0) return hipErrorInvalidValue;
    if (a.nbnd == 0) return hipSuccess;
    const dim3 grd(round8_grid((long)((a.nbnd + 255) / 256) * a.nrhs)), blk(256);
#define SRC(M, F)                                                                                              \
    hipLaunchKernelGGL((boundary_source_kernel<M, F>), grd, blk, 0, st, a.g, (const double2 *)a.xb, a.bidx, a.nb, \
                       (const double2 *)a.U, (const double2 *)a.rows, a.site, a.nbnd, a.info, a.stamp, a.diag, \
                       1.0 / a.diag, (double2 *)a.t, (double2 *)a.p, a.nrhs)
    if (!a.rows && a.info) SRC(kNoRows, true);
    else if (!a.rows) SRC(kNoRows, false);
    else if (a.info) SRC(kTwoPass, true);
    else if (a.linked) SRC(kTwoPass, false);
    else SRC(kOnePass, false);
#undef SRC
    return hipGetLastError();
}

hipError_t launch_boundary_apply(const ApproxArgs &a, hipStream_t st)
{
    if (a.nrhs < 1 || a.nrhs > kMaxRhs || a.nbnd < 0 || !a.rows) return hipErrorInvalidValue;
    if (a.nbnd == 0 || !a.linked) return hipSuccess;
    const dim3 grd(round8_grid((long)((a.nbnd + 255) / 256) * a.nrhs)), blk(256);
#define APP(F)                                                                                              \
    hipLaunchKernelGGL(boundary_apply_kernel<F>, grd, blk, 0, st, a.g, (const double2 *)a.U, (const double2 *)a.rows, \
                       a.site, a.map, a.nbnd, a.info, a.stamp, a.diag, 1.0 / a.diag, (const double2 *)a.t,     \
                       (double2 *)a.p, a.nrhs)
    if (a.info) APP(true);
    else APP(false);
#undef APP
    return hipGetLastError();
}

hipError_t launch_boundary_coarse(const ApproxArgs &a, hipStream_t st)
{
    if (a.nrhs < 1 || a.nrhs > kMaxRhs || a.nb < 1) return hipErrorInvalidValue;
    const dim3 grd(round8_grid((long)((a.nb + 63) / 64) * a.nrhs)), blk(kSplitThreads);
#define COARSE(F)                                                                                           \
    hipLaunchKernelGGL(boundary_coarse_kernel<F>, grd, blk, 0, st, a.g, (const double2 *)a.xb, a.q, a.bidx, a.nb, \
                       a.map, (const double2 *)a.U, a.diag, (const double2 *)a.p, (double2 *)a.yb, a.nrhs, a.info, \
                       a.host, a.stamp)
    if (a.info) COARSE(true);
    else COARSE(false);
#undef COARSE
    return hipGetLastError();
}

}  // namespace grg
