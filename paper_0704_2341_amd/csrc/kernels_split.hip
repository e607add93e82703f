// The stencils in the hop-per-wavefront form (split.h), for fields too small
// to fill the chip with one lane per site: the full stencil, the half-lattice
// stencil of the even-odd reduction and the FP64 defect-correction step.  Work
// items are 64 sites with one RHS, RHS fastest.  Each writes what the other
// forms of the same operation write, bit for bit (the hops are summed in the
// same order; sums over sites differ in rounding).
#include <algorithm>

#include "common.h"
#include "engine.h"
#include "eo_site.h"
#include "split.h"

namespace grg {

// per-wavefront sums of K values per RHS, written as one partial row per
// workgroup (wavefronts 0..5, which hold the sites' outputs)
template <int K>
struct SplitSums {
    double red[6][kMaxRhs][K];
    __device__ void clear(int nrhs)
    {
        for (int i = threadIdx.x; i < 6 * nrhs * K; i += blockDim.x)
            red[i / (nrhs * K)][(i / K) % nrhs][i % K] = 0.0;
        __syncthreads();
    }
    __device__ void add(int wave, int lane, int r, const double (&v)[K])
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double t = wave_sum(v[k]);
            if (lane == 0) red[wave][r][k] += t;
        }
    }
    __device__ void flush(double *partials, int nrhs)
    {
        __syncthreads();
        for (int i = threadIdx.x; i < nrhs * K; i += blockDim.x) {
            double t = 0;
            for (int w = 0; w < 6; ++w) t += red[w][i / K][i % K];
            partials[(size_t)i * gridDim.x + blockIdx.x] = t;
        }
    }
};

// Field element (site s, RHS r, component c) as the stencil holds it, from the
// internal tiles or (CANON) from a canonical complex128 field, converted to the
// precision as pack_spinor_kernel does.
template <int P, bool CANON>
struct SplitIn {
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    typedef Operand<S, R> OP;
    typedef typename OP::T PT;
    __device__ static void load(PT (&p)[12], const void *in, int s, int r, int nrhs, int V)
    {
        if constexpr (CANON) {
            const double2 *v = (const double2 *)in + ((size_t)r * V + s) * 12;
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                const double2 x = v[c];
                if constexpr (P == GRG_BF16) p[c] = pack_bf16((float)x.x, (float)x.y);
                else p[c] = {(R)x.x, (R)x.y};
            }
        } else {
#pragma unroll
            for (int c = 0; c < 12; ++c) p[c] = OP::load((const S *)in, fidx(s, r, c, nrhs));
        }
    }
};

// out = D in on the selected rows (zero elsewhere), with the fused sums, as
// dslash_kernel.  CANON: canonical complex128 in and out (the result rounded
// to the precision and widened), in one launch.
template <int P, bool CANON>
__global__ void __launch_bounds__(kSplitThreads) dslash_split_kernel(DslashArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    typedef SplitIn<P, CANON> IN;
    typedef typename IN::OP OP;
    typedef typename OP::T PT;
    __shared__ HopSums<R> hs;
    __shared__ SplitSums<3> sums;
    const S *__restrict__ U = (const S *)a.U;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool dots = a.partials != nullptr;
    if (dots) sums.clear(a.nrhs);
    const int nt = (a.g.V + 63) >> 6;
    const ItemRange it = xcd_items(nt * a.nrhs);
    for (int wi = it.begin; wi < it.end; wi += it.step) {
        const int tile = wi / a.nrhs, r = wi - tile * a.nrhs;
        const int s = tile * 64 + lane;
        const bool valid = s < a.g.V;
        const bool on = valid && (a.mask == nullptr || a.mask[s] == a.sel);
        if (on) {
            const SiteGeo q = site_geo(s, a.g);
            int sp, sm;
            nbr(s, k >> 1, q, a.g, sp, sm);
            PT p[12], u[9];
            cpx<R> w[6];
#pragma unroll
            for (int e = 0; e < 9; ++e) u[e] = OP::load(U, lidx((k & 1) ? sm : s, k >> 1, e));
            const int n = (k & 1) ? sm : sp;
            if (!CANON || a.in_mask == nullptr || a.in_mask[n] == a.in_sel) {
                IN::load(p, a.in, n, r, a.nrhs, a.g.V);
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) p[c] = PT{};
            }
            hop_w_k(k, w, p, u);
            hs.put(k, lane, w);
        }
        __syncthreads();
        if (k < 6) {
            const int row = k % 3, spin = k < 3 ? 0 : 2;
            double d[3] = {0, 0, 0};
            if (valid) {
                const int c0 = 3 * spin + row, c1 = c0 + 3;
                cpx<R> a0 = {0, 0}, a1 = {0, 0}, v0 = {0, 0}, v1 = {0, 0};
                const size_t ci = ((size_t)r * a.g.V + s) * 12;
                if (on) {
                    if constexpr (CANON) {
                        const bool in_on = a.in_mask == nullptr || a.in_mask[s] == a.in_sel;
                        const double2 *x = (const double2 *)a.in + ci;
                        const double2 x0 = in_on ? x[c0] : make_double2(0.0, 0.0);
                        const double2 x1 = in_on ? x[c1] : make_double2(0.0, 0.0);
                        if constexpr (P == GRG_BF16) {
                            v0 = as_cpx(pack_bf16((float)x0.x, (float)x0.y));
                            v1 = as_cpx(pack_bf16((float)x1.x, (float)x1.y));
                        } else {
                            v0 = {(R)x0.x, (R)x0.y};
                            v1 = {(R)x1.x, (R)x1.y};
                        }
                    } else {
                        v0 = ldr<R>((const S *)a.in, fidx(s, r, c0, a.nrhs));
                        v1 = ldr<R>((const S *)a.in, fidx(s, r, c1, a.nrhs));
                    }
                    const R diag = (R)a.diag;
                    a0 = {diag * v0.re, diag * v0.im};
                    a1 = {diag * v1.re, diag * v1.im};
                    if (spin == 0) hs.template add<false>(row, lane, a0, a1);
                    else hs.template add<true>(row, lane, a0, a1);
                }
                if constexpr (CANON) {
                    double2 *o = (double2 *)a.out + ci;
                    if constexpr (P == GRG_BF16) {
                        a0 = as_cpx(pack_bf16(a0.re, a0.im));
                        a1 = as_cpx(pack_bf16(a1.re, a1.im));
                    }
                    o[c0] = make_double2((double)a0.re, (double)a0.im);
                    o[c1] = make_double2((double)a1.re, (double)a1.im);
                } else {
                    stc((S *)a.out, fidx(s, r, c0, a.nrhs), a0);
                    stc((S *)a.out, fidx(s, r, c1, a.nrhs), a1);
                }
                if (dots && on) {
                    if (a.dot_with) {
                        v0 = ldr<R>((const S *)a.dot_with, fidx(s, r, c0, a.nrhs));
                        v1 = ldr<R>((const S *)a.dot_with, fidx(s, r, c1, a.nrhs));
                    }
                    R sre = 0, sim = 0, sqq = 0;
                    auto one = [&](cpx<R> o, cpx<R> v) {
                        sre = fma(o.re, v.re, fma(o.im, v.im, sre));
                        sim = fma(o.re, v.im, fma(-o.im, v.re, sim));
                        sqq = fma(o.re, o.re, fma(o.im, o.im, sqq));
                    };
                    one(a0, v0);
                    one(a1, v1);
                    d[0] = (double)sre;
                    d[1] = (double)sim;
                    d[2] = (double)sqq;
                }
            }
            if (dots) sums.add(k, lane, r, d);
        }
        __syncthreads();  // the hops are read before the next item's overwrite them
    }
    if (dots) sums.flush(a.partials, a.nrhs);
}

// out = alpha in2 + beta H in on one parity, as eo_hop_kernel (IO: its
// full-layout modes, here decided at run time: the field is small).
template <int P>
__global__ void __launch_bounds__(kSplitThreads) eo_split_kernel(EoArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    typedef Operand<S, R> OP;
    typedef typename OP::T PT;
    __shared__ HopSums<R> hs;
    __shared__ SplitSums<3> sums;
    const S *__restrict__ in = (const S *)a.in;
    const S *__restrict__ in2 = (const S *)a.in2;
    S *__restrict__ out = (S *)a.out;
    const S *__restrict__ Uo = (const S *)a.U + (size_t)a.po * 36 * a.Vhs;
    const S *__restrict__ Ui = (const S *)a.U + (size_t)(1 - a.po) * 36 * a.Vhs;
    const uint8_t *__restrict__ mk = a.mask + (size_t)a.po * a.Vhs;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool dots = a.partials != nullptr;
    if (dots) sums.clear(a.nrhs);
    const R al = (R)a.alpha, be = (R)a.beta;
    const int nt = (a.Vh + 63) >> 6;
    const ItemRange it = xcd_items(nt * a.nrhs);
    for (int wi = it.begin; wi < it.end; wi += it.step) {
        const int tile = wi / a.nrhs, r = wi - tile * a.nrhs;
        const int h = tile * 64 + lane;
        const bool valid = h < a.Vh;
        const bool on = valid && mk[h] == 0;
        const bool act = a.active == nullptr || a.active[r] != 0;
        SiteGeo q;
        int s = 0;
        if (valid) s = eo_site(h, a.po, a.g, q);
        if (on) {
            int sp, sm;
            nbr(s, k >> 1, q, a.g, sp, sm);
            const int n = (k & 1) ? sm : sp, hn = n >> 1;
            PT p[12], u[9];
            cpx<R> w[6];
            if (a.in_full) {
#pragma unroll
                for (int c = 0; c < 12; ++c) p[c] = OP::load(in, fidx(n, r, c, a.nrhs));
            } else {
                load_half<S, R>(p, in, hn, r, a.nrhs);
            }
            load_half_link<S, R>(u, (k & 1) ? Ui : Uo, (k & 1) ? hn : h, k >> 1);
            hop_w_k(k, w, p, u);
            hs.put(k, lane, w);
        }
        __syncthreads();
        if (k < 6) {
            const int row = k % 3, spin = k < 3 ? 0 : 2;
            double d[3] = {0, 0, 0};
            if (valid) {
                const int c0 = 3 * spin + row;
                cpx<R> acc[2] = {{0, 0}, {0, 0}};
                if (on) {
                    if (spin == 0) hs.template add<false>(row, lane, acc[0], acc[1]);
                    else hs.template add<true>(row, lane, acc[0], acc[1]);
                }
                R sre = 0, sim = 0, sqq = 0;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int c = c0 + 3 * j;
                    const size_t i = hidx<S>(h, r, c, a.nrhs);
                    cpx<R> o = {0, 0};
                    if (on && act) {
                        o = {be * acc[j].re, be * acc[j].im};
                        if (in2) {
                            const cpx<R> v = ldr<R>(in2, a.in2_full ? fidx(s, r, c, a.nrhs) : i);
                            o.re = fma(al, v.re, o.re);
                            o.im = fma(al, v.im, o.im);
                        }
                    }
                    if (a.out_full) {
                        // this site, and the other parity's site of the same index
                        stc(out, fidx(s, r, c, a.nrhs), o);
                        out[fidx(s ^ 1, r, c, a.nrhs)] = ((const S *)a.partner)[i];
                    } else {
                        stc(out, i, o);
                    }
                    if (dots && on) {
                        const cpx<R> v = a.dot_with ? ldr<R>((const S *)a.dot_with, i) : cpx<R>{0, 0};
                        sre = fma(o.re, v.re, fma(o.im, v.im, sre));
                        sim = fma(o.re, v.im, fma(-o.im, v.re, sim));
                        sqq = fma(o.re, o.re, fma(o.im, o.im, sqq));
                    }
                }
                d[0] = (double)sre;
                d[1] = (double)sim;
                d[2] = (double)sqq;
            }
            if (dots) sums.add(k, lane, r, d);
        }
        __syncthreads();
    }
    if (dots) sums.flush(a.partials, a.nrhs);
}

// One FP64 defect-correction step, as dc_update_kernel.
template <int P>
__global__ void __launch_bounds__(kSplitThreads) dc_split_kernel(DcArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R RN;
    typedef Operand<S, double> OP;
    typedef typename OP::T PT;
    __shared__ HopSums<double> hs;
    __shared__ SplitSums<1> sums;
    const S *__restrict__ e = (const S *)a.e;
    const double2 *__restrict__ U = (const double2 *)a.U;
    const double2 *r_in = (const double2 *)a.r_in, *x_in = (const double2 *)a.x_in;
    double2 *r_out = (double2 *)a.r_out, *x_out = (double2 *)a.x_out;
    S *r_next = (S *)a.r_next;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    sums.clear(a.nrhs);
    const int nt = (a.g.V + 63) >> 6;
    const ItemRange it = xcd_items(nt * a.nrhs);
    for (int wi = it.begin; wi < it.end; wi += it.step) {
        const int tile = wi / a.nrhs, r = wi - tile * a.nrhs;
        const int s = tile * 64 + lane;
        const bool valid = s < a.g.V;
        const bool on = valid && a.mask[s] == 0;
        if (on) {
            const SiteGeo q = site_geo(s, a.g);
            int sp, sm;
            nbr(s, k >> 1, q, a.g, sp, sm);
            const int n = (k & 1) ? sm : sp;
            PT p[12];
            cpx<double> u[9], w[6];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const double2 l = U[lidx((k & 1) ? sm : s, k >> 1, i)];
                u[i] = {l.x, l.y};
            }
#pragma unroll
            for (int c = 0; c < 12; ++c) p[c] = OP::load(e, fidx(n, r, c, a.nrhs));
            hop_w_k(k, w, p, u);
            hs.put(k, lane, w);
        }
        __syncthreads();
        if (k < 6) {
            const int row = k % 3, spin = k < 3 ? 0 : 2;
            double nrm[1] = {0};
            if (valid) {
                const DcNext nx(a, s);
                const double f = a.f[r], sn = r_next ? a.s_next[r] : 0.0;
                cpx<double> acc[2], ev[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    ev[j] = on ? ldr<double>(e, fidx(s, r, 3 * spin + row + 3 * j, a.nrhs)) : cpx<double>{0, 0};
                    acc[j] = {a.diag * ev[j].re, a.diag * ev[j].im};
                }
                if (on) {
                    if (spin == 0) hs.template add<false>(row, lane, acc[0], acc[1]);
                    else hs.template add<true>(row, lane, acc[0], acc[1]);
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int c = 3 * spin + row + 3 * j;
                    const size_t i = fidx(s, r, c, a.nrhs);
                    double2 d = make_double2(0.0, 0.0);
                    if (on) {
                        const double2 rv = dc_load_r(a, r_in, i);
                        d = make_double2(rv.x - f * acc[j].re, rv.y - f * acc[j].im);
                        nrm[0] += d.x * d.x + d.y * d.y;
                    }
                    dc_store_r(a, r_out, i, d);
                    if (r_next) stc(r_next, nx.at(r_next, i, r, c, a.nrhs), cpx<RN>{(RN)(sn * d.x), (RN)(sn * d.y)});
                    if (x_out) {
                        const double2 xv = on && x_in ? x_in[i] : make_double2(0.0, 0.0);
                        x_out[i] = on ? make_double2(xv.x + f * ev[j].re, xv.y + f * ev[j].im)
                                      : make_double2(0.0, 0.0);
                    }
                }
            }
            sums.add(k, lane, r, nrm);
        }
        __syncthreads();
    }
    sums.flush(a.partials, a.nrhs);
}

// ------------------------------------------------------------------ launchers
hipError_t launch_dslash_split(int prec, const DslashArgs &a, bool canonical, int grid, hipStream_t st)
{
    if (a.nrhs < 1 || a.nrhs > kMaxRhs || grid < 8 || grid % 8) return hipErrorInvalidValue;
    if (canonical ? a.partials != nullptr : (a.out_canon || a.in_mask)) return hipErrorInvalidValue;
    const dim3 g(grid), b(kSplitThreads);
#define DSP(PP)                                                                     \
    if (canonical) hipLaunchKernelGGL((dslash_split_kernel<PP, true>), g, b, 0, st, a); \
    else hipLaunchKernelGGL((dslash_split_kernel<PP, false>), g, b, 0, st, a);
    switch (prec) {
    case GRG_FP64: DSP(GRG_FP64) break;
    case GRG_FP32: DSP(GRG_FP32) break;
    case GRG_BF16: DSP(GRG_BF16) break;
    default: return hipErrorInvalidValue;
    }
#undef DSP
    return hipGetLastError();
}

hipError_t launch_eo_split(int prec, const EoArgs &a, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kSplitThreads);
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(eo_split_kernel<GRG_FP64>, g, b, 0, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(eo_split_kernel<GRG_FP32>, g, b, 0, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(eo_split_kernel<GRG_BF16>, g, b, 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_dc_split(int prec, const DcArgs &a, int grid, hipStream_t st)
{
    const dim3 g(grid), b(kSplitThreads);
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(dc_split_kernel<GRG_FP64>, g, b, 0, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(dc_split_kernel<GRG_FP32>, g, b, 0, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(dc_split_kernel<GRG_BF16>, g, b, 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace grg
