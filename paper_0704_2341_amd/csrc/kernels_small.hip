// BiCGstab on a lattice of at most kSmallSites sites, a whole solve in one
// launch: a workgroup per right-hand side.
//
// The V-cycle's lower levels have 16 to 256 sites.  Launched step by step, such
// a solve is all latency: seven launches and three to five waits of the host per
// iteration (4 RHS: 500 us for the four iterations of a solve on 16 sites, 310 for
// the two of a D_rr solve on 256; here 37 and 86).  One workgroup holds
// everything: the operator's input field lies in LDS, the hops of 64 sites run
// on eight wavefronts (split.h), and the BiCGstab vectors stay in the registers
// of the six wavefronts that sum the hops, where lane and wavefront own a site's
// colour row in one spin pair (of four tiles, v lies in LDS).  Sums go through
// the wavefronts' shuffles and LDS; every thread forms the step lengths itself.
// What bounds it then is the chain of an iteration: two applications (per 64
// sites 3 us: the hops' FP64 arithmetic on one CU, their LDS image and two
// barriers) and three reductions.
#include "common.h"
#include "engine.h"
#include "split.h"
#include "stencil.h"

namespace grg {

static_assert(kSmallSites % 64 == 0, "whole tiles");

template <int T>  // tiles of 64 sites
struct SmallLattice {
    static constexpr bool kVLds = T > 2;  // v = A p here instead of in registers
    cpx<double> fld[12][64 * T];
    cpx<double> v[12][kVLds ? 64 * T : 1];
    HopSums<double> hops;
    double red[2][6][3];
};

namespace {

struct Vec {  // a lane's two components of a tile: colour row `row` of two spins
    cpx<double> a, b;
};

__device__ __forceinline__ cpx<double> cmul(cpx<double> a, cpx<double> b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cpx<double> cdiv(cpx<double> a, cpx<double> b)
{
    const double d = b.re * b.re + b.im * b.im;
    if (!(d > 0)) return {0, 0};
    return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
__device__ __forceinline__ void axpy(Vec &y, cpx<double> c, const Vec &x)  // y += c x
{
    cmac(y.a, c, x.a);
    cmac(y.b, c, x.b);
}
// conj(x) y and |y|^2
__device__ __forceinline__ void dot(double (&d)[3], const Vec &x, const Vec &y)
{
    auto one = [&](cpx<double> u, cpx<double> v) {
        d[0] += u.re * v.re + u.im * v.im;
        d[1] += u.re * v.im - u.im * v.re;
        d[2] += v.re * v.re + v.im * v.im;
    };
    one(x.a, y.a);
    one(x.b, y.b);
}

}  // namespace

template <int T>
__global__ void __launch_bounds__(kSplitThreads, 2) small_bicgstab_kernel(SmallArgs a)
{
    __shared__ SmallLattice<T> L;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int V = a.g.V, row = k % 3, spin = k < 3 ? 0 : 2;
    const int c0 = 3 * spin + row, c1 = c0 + 3;
    const double2 *__restrict__ U = (const double2 *)a.U;
    const double2 *f = (const double2 *)a.f + (size_t)blockIdx.x * V * 12;
    double2 *x = (double2 *)a.x + (size_t)blockIdx.x * V * 12;
    // this lane's site per tile, hop k's neighbour and link, and whether its
    // row takes part
    bool on[T], own[T];
    int nb[T], lk[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int s = 64 * i + lane;
        on[i] = s < V && (a.mask == nullptr || a.mask[s] == 0);
        own[i] = k < 6 && s < V;
        const int sc = s < V ? s : 0;
        const SiteGeo q = site_geo(sc, a.g);
        int sp, sm;
        nbr(sc, k >> 1, q, a.g, sp, sm);
        nb[i] = (k & 1) ? sm : sp;
        lk[i] = (k & 1) ? sm : sc;
    }
    // the links of hop k, a tile ahead: the next tile's are requested as soon as
    // this one's hop is done, the first one's for the next application
    cpx<double> u[9];
    auto load_u = [&](int i) {
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const double2 l = U[lidx(lk[i], k >> 1, e)];
            u[e] = {l.x, l.y};
        }
    };
    load_u(0);
    // out(i, c D in of tile i) (masked)
    auto apply = [&](const Vec (&in)[T], auto &&out) {
        if (k < 6) {
#pragma unroll
            for (int i = 0; i < T; ++i) {
                L.fld[c0][64 * i + lane] = in[i].a;
                L.fld[c1][64 * i + lane] = in[i].b;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if (on[i]) {
                cpx<double> p[12], w[6];
#pragma unroll
                for (int c = 0; c < 12; ++c) p[c] = L.fld[c][nb[i]];
                hop_w_k(k, w, p, u);
                L.hops.put(k, lane, w);
            }
            if (T > 1) load_u((i + 1) % T);
            __syncthreads();
            Vec o = {{0, 0}, {0, 0}};
            if (k < 6 && on[i]) {
                cpx<double> s0 = {a.diag * in[i].a.re, a.diag * in[i].a.im};
                cpx<double> s1 = {a.diag * in[i].b.re, a.diag * in[i].b.im};
                if (spin == 0) L.hops.template add<false>(row, lane, s0, s1);
                else L.hops.template add<true>(row, lane, s0, s1);
                o = {{a.c * s0.re, a.c * s0.im}, {a.c * s1.re, a.c * s1.im}};
            }
            out(i, o);
            __syncthreads();  // the hops (and the last tile's field) are read
        }
    };
    int flip = 0;
    // the workgroup's sums of d, the same in every thread
    auto sum = [&](double (&d)[3]) {
        double(*red)[3] = L.red[flip];
        flip ^= 1;
        if (k < 6) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double t = wave_sum(d[j]);
                if (lane == 0) red[k][j] = t;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double t = 0;
            for (int w = 0; w < 6; ++w) t += red[w][j];
            d[j] = t;
        }
    };
    auto load_f = [&](int i) -> Vec {
        if (!own[i] || !on[i]) return {{0, 0}, {0, 0}};
        const double2 u = f[(size_t)(64 * i + lane) * 12 + c0], v = f[(size_t)(64 * i + lane) * 12 + c1];
        return {{u.x, u.y}, {v.x, v.y}};
    };
    auto load_x = [&](int i) -> Vec {
        if (!own[i]) return {{0, 0}, {0, 0}};
        const double2 u = x[(size_t)(64 * i + lane) * 12 + c0], v = x[(size_t)(64 * i + lane) * 12 + c1];
        return {{u.x, u.y}, {v.x, v.y}};
    };
    auto store_x = [&](int i, const Vec &v) {
        if (!own[i]) return;
        x[(size_t)(64 * i + lane) * 12 + c0] = make_double2(v.a.re, v.a.im);
        x[(size_t)(64 * i + lane) * 12 + c1] = make_double2(v.b.re, v.b.im);
    };
    constexpr bool kVLds = SmallLattice<T>::kVLds;
    Vec r[T], p[T], t[T], vr[kVLds ? 1 : T];
    auto put_v = [&](int i, const Vec &o) {
        if constexpr (!kVLds) vr[i] = o;
        else if (k < 6) {
            L.v[c0][64 * i + lane] = o.a;
            L.v[c1][64 * i + lane] = o.b;
        }
    };
    auto get_v = [&](int i) -> Vec {
        if constexpr (!kVLds) return vr[i];
        else return k < 6 ? Vec{L.v[c0][64 * i + lane], L.v[c1][64 * i + lane]} : Vec{{0, 0}, {0, 0}};
    };
    double b2;
    {
        double d[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < T; ++i) {
            r[i] = load_f(i);
            store_x(i, Vec{{0, 0}, {0, 0}});
            dot(d, r[i], r[i]);
        }
        sum(d);
        b2 = d[2];
    }
    double r2 = b2;
    const double thr = a.tol * a.tol * b2;
    int it = 0, outer = 0;
    bool done = !(b2 > 0) && b2 == b2;
    // (again from the recomputed residual, should it miss the tolerance that the
    // recursion's has reached)
    while (!done) {
        cpx<double> rho;
        {
            double d[3] = {0, 0, 0};
#pragma unroll
            for (int i = 0; i < T; ++i) {
                p[i] = r[i];
                dot(d, load_f(i), r[i]);
            }
            sum(d);
            rho = {d[0], d[1]};
            r2 = d[2];
        }
        while (r2 > thr && r2 < HUGE_VAL && it < a.max_iter) {  // (a NaN ends it too)
            apply(p, put_v);
            double d[3] = {0, 0, 0};
#pragma unroll
            for (int i = 0; i < T; ++i) dot(d, load_f(i), get_v(i));
            sum(d);
            const cpx<double> alpha = cdiv(rho, {d[0], d[1]}), ma = {-alpha.re, -alpha.im};
#pragma unroll
            for (int i = 0; i < T; ++i) axpy(r[i], ma, get_v(i));  // s
            apply(r, [&](int i, const Vec &o) { t[i] = o; });
            d[0] = d[1] = d[2] = 0;
#pragma unroll
            for (int i = 0; i < T; ++i) dot(d, r[i], t[i]);
            sum(d);
            const cpx<double> om = d[2] > 0 ? cpx<double>{d[0] / d[2], -d[1] / d[2]} : cpx<double>{0, 0};
            const cpx<double> mo = {-om.re, -om.im};
            d[0] = d[1] = d[2] = 0;
#pragma unroll
            for (int i = 0; i < T; ++i) {
                Vec xv = load_x(i);
                axpy(xv, alpha, p[i]);
                axpy(xv, om, r[i]);
                store_x(i, xv);
                axpy(r[i], mo, t[i]);
                dot(d, load_f(i), r[i]);
            }
            sum(d);
            const cpx<double> rho2 = {d[0], d[1]};
            r2 = d[2];
            cpx<double> beta = {0, 0};
            if ((rho.re != 0 || rho.im != 0) && (om.re != 0 || om.im != 0))
                beta = cmul(cdiv(rho2, rho), cdiv(alpha, om));
            rho = rho2;
#pragma unroll
            for (int i = 0; i < T; ++i) {  // p = r + beta (p - omega v)
                Vec q = p[i];
                axpy(q, mo, get_v(i));
                p[i] = r[i];
                axpy(p[i], beta, q);
            }
            ++it;
        }
        if (!a.check || !(r2 <= thr || it >= a.max_iter)) break;
        // the residual recomputed from x
#pragma unroll
        for (int i = 0; i < T; ++i) p[i] = load_x(i);
        apply(p, put_v);
        double d[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < T; ++i) {
            r[i] = load_f(i);
            axpy(r[i], {-1, 0}, get_v(i));
            dot(d, r[i], r[i]);
        }
        sum(d);
        r2 = d[2];
        done = r2 <= thr || it >= a.max_iter || !(r2 == r2) || ++outer >= a.check;
        if (done && r2 > b2) {  // no better than x = 0
#pragma unroll
            for (int i = 0; i < T; ++i) store_x(i, Vec{{0, 0}, {0, 0}});
        }
    }
    if (threadIdx.x == 0) {
        if (!isfinite(r2)) a.flags[1] = 1;
        else if (r2 > thr) a.flags[0] = 1;
    }
}

hipError_t launch_small_bicgstab(const SmallArgs &a, int nrhs, hipStream_t st)
{
    if (a.g.V < 1 || a.g.V > kSmallSites || nrhs < 1 || nrhs > kMaxRhs || a.max_iter > kSmallIters)
        return hipErrorInvalidValue;
#define SB(T)                                                                                                   \
    hipLaunchKernelGGL(small_bicgstab_kernel<T>, dim3(nrhs), dim3(kSplitThreads), 0, st, a)
    switch ((a.g.V + 63) / 64) {
    case 1: SB(1); break;
    case 2: SB(2); break;
    case 3: SB(3); break;
    default: SB(4); break;
    }
#undef SB
    return hipGetLastError();
}

}  // namespace grg
