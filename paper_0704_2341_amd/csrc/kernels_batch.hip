// Many-lattice batch: every kernel covers all lattices of the batch in one
// launch.  The lattices are concatenated in the site index (each starts on a
// 256-site boundary, so no workgroup straddles two of them); a per-tile table
// names the lattice of every 64-site tile, and per-lattice tables hold the
// extents, the first site and the diagonal 4 + m0.  A "system" is one
// (lattice, right-hand side) pair, sys = lattice * nrhs + rhs; step lengths,
// norms and convergence flags are per system.
#include <algorithm>

#include "batch.h"
#include "common.h"
#include "engine.h"
#include "eo_site.h"
#include "reduce.h"
#include "vec16.h"
#include "split.h"
#include "stencil.h"

namespace grg {

struct BSite {
    int l;      // lattice
    Geom g;     // its geometry (V = its volume)
    int local;  // site index inside it
};

__device__ __forceinline__ BSite bsite(const BatchTable &bt, int s)
{
    BSite b;
    b.l = bt.tile_lat[s >> 6];
    const int4 d = bt.dims[b.l];
    b.g.L[0] = d.x;
    b.g.L[1] = d.y;
    b.g.L[2] = d.z;
    b.g.L[3] = d.w;
    b.g.V = d.x * d.y * d.z * d.w;
    b.g.Vs = b.g.V;
    b.local = s - bt.off[b.l];
    return b;
}

// per-wave LDS accumulators over the systems, written as one partial per
// workgroup and system at the end
template <int K>
struct SysPartial {
    double *red;  // [4 waves][nsys][K]
    int nsys;
    __device__ void init(double *smem, int n)
    {
        red = smem;
        nsys = n;
        for (int i = threadIdx.x; i < 4 * n * K; i += blockDim.x) red[i] = 0.0;
        __syncthreads();
    }
    __device__ void add(int sys, const double (&v)[K])
    {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double t = wave_sum(v[k]);
            if (lane == 0) red[(wave * nsys + sys) * K + k] += t;
        }
    }
    __device__ void flush(double *partials)
    {
        __syncthreads();
        const int nw = blockDim.x >> 6;
        for (int i = threadIdx.x; i < nsys * K; i += blockDim.x) {
            double t = 0;
            for (int w = 0; w < nw; ++w) t += red[w * nsys * K + i];
            partials[(size_t)blockIdx.x * nsys * K + i] = t;
        }
    }
};

// Whether any of the n flags is set: the same answer in every thread of the
// workgroup (a gate read at the start of a launch, before any barrier of the
// kernel, so a launch with nothing to do returns as a whole).
__device__ bool any_set(const int *flags, int n)
{
    __shared__ int s_any;
    if (threadIdx.x == 0) s_any = 0;
    __syncthreads();
    int mine = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) mine |= flags[i];
    if (mine) s_any = 1;
    __syncthreads();
    return s_any != 0;
}

// A stencil's work item per wavefront: 64 sites with one RHS, RHS fastest, so
// that the wavefronts of a workgroup read the same links (nrhs 4: one link
// fetch from L2 for the four).
__device__ __forceinline__ void tile_item(int w, int nrhs, int &tile, int &r)
{
    const int i = __builtin_amdgcn_readfirstlane(w * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6));
    tile = i / nrhs;
    r = i - tile * nrhs;
}

// out = mask_sel D in over all lattices; fused dots per system when partials.
template <int P>
__global__ void __launch_bounds__(256) dslash_batch_kernel(BatchDslashArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    extern __shared__ double smem[];
    const S *__restrict__ in = (const S *)a.in;
    S *__restrict__ out = (S *)a.out;
    const S *__restrict__ U = (const S *)a.U;
    const int nsys = a.bt.nlat * a.nrhs;
    if (a.act && !any_set(a.act, nsys)) return;
    const bool dots = a.partials != nullptr;
    SysPartial<3> part;
    if (dots) part.init(smem, nsys);
    const int ngroups = (a.nrhs + a.RG - 1) / a.RG;
    const int nsb = a.Vtot / blockDim.x;  // every lattice is a whole number of blocks
    const ItemRange it = xcd_items(nsb * ngroups);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int sb = w / ngroups, grp = w - sb * ngroups;
        const int s = sb * blockDim.x + (int)threadIdx.x;
        const BSite b = bsite(a.bt, s);
        const bool on = a.mask[s] == a.sel;
        const SiteGeo q = site_geo(b.local, b.g);
        const R diag = (R)a.bt.diag[b.l];
        const int r0 = grp * a.RG, r1 = min(r0 + a.RG, a.nrhs);
        for (int r = r0; r < r1; ++r) {
            // (a workgroup lies inside one lattice: the skip is uniform)
            if (a.act && !a.act[b.l * a.nrhs + r]) continue;
            cpx<R> acc[12];
            if (on) {
                dslash_site<S, R, true>(acc, in, U, s, q, b.g, r, a.nrhs, diag);
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) acc[c] = {0, 0};
            }
#pragma unroll
            for (int c = 0; c < 12; ++c) stc(out, fidx(s, r, c, a.nrhs), acc[c]);
            if (dots) {
                R sre = 0, sim = 0, sqq = 0;
                if (on) {
#pragma unroll
                    for (int c = 0; c < 12; ++c) {
                        const cpx<R> v = ldc(in, fidx(s, r, c, a.nrhs));
                        sre = fma(acc[c].re, v.re, fma(acc[c].im, v.im, sre));
                        sim = fma(acc[c].re, v.im, fma(-acc[c].im, v.re, sim));
                        sqq = fma(acc[c].re, acc[c].re, fma(acc[c].im, acc[c].im, sqq));
                    }
                }
                const double d[3] = {(double)sre, (double)sim, (double)sqq};
                part.add(b.l * a.nrhs + r, d);
            }
        }
    }
    if (dots) part.flush(a.partials);
}

// x += alpha r ; r -= alpha q ; partial |r|^2  (per system).  XM: x as that
// says (kMrXAdd), left to the next step (kMrXLater), or given the step before
// and this one together (kMrXPair); the two terms are rounded one after the
// other as two steps would.  A system that converged in between still gets the
// first term: pend holds the systems that the first step took, written also by
// one that had none.
//
// The streams are the cost; a wavefront takes a unit of kUnitVecs 16-byte
// vectors per lane of one (tile, RHS), as mr_update_kernel does.  With a site
// per lane, 8 bytes of each component and the RHS one after the other it ran at
// 4.3 TB/s of the copy's 6.2 (48 lattices, 4 RHS, FP32, a single step: 0.277 ->
// 0.236 ms; the whole apply 21.3 -> 21.1 ms), and with the streams read past L2
// 0.193 ms, 6.1 TB/s, and 20.5 ms.
template <int P, int XM>
__global__ void __launch_bounds__(256) batch_mr_update_kernel(BatchBlasArgs a, void *x_, void *r_,
                                                              const void *q_)
{
    typedef VecIO<P> IO;
    typedef typename IO::R R;
    constexpr int N = IO::N, PARTS = 12 / N / kUnitVecs, UV = kUnitVecs * 64;
    constexpr bool LATER = XM == kMrXLater, PAIR = XM == kMrXPair;
    extern __shared__ double smem[];
    const int nsys = a.bt.nlat * a.nrhs;
    if (LATER && blockIdx.x == 0)
        for (int i = threadIdx.x; i < nsys; i += blockDim.x) a.pend[i] = a.act[i];
    const bool any = a.act == nullptr || any_set(a.act, nsys);
    if (!any && !(PAIR && any_set(a.pend, nsys))) return;
    if (any && a.ctr && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(a.ctr, 1);
    SysPartial<1> part;
    part.init(smem, nsys);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint4 *x = (uint4 *)x_, *r = (uint4 *)r_, *r_out = LATER ? (uint4 *)a.r_later : PAIR ? (uint4 *)a.r_prev : r;
    const uint4 *q = (const uint4 *)q_, *r_prev = (const uint4 *)a.r_prev;
    const int nunits = a.Vtot / 64 * a.nrhs * PARTS;
    const ItemRange it = xcd_items((nunits + 3) >> 2);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int u = w * 4 + wave;
        if (u >= nunits) continue;  // the whole wavefront
        const int tr = u / PARTS, tile = tr / a.nrhs, k = tr - tile * a.nrhs;
        const int sys = a.bt.tile_lat[tile] * a.nrhs + k;
        const bool on = !a.act || a.act[sys];
        if (PAIR ? !a.pend[sys] : !on) continue;  // converged: x and r stay
        cpx<R> ap = {0, 0};
        if constexpr (PAIR) ap = {(R)a.alpha_prev[sys].x, (R)a.alpha_prev[sys].y};
        const size_t base = (size_t)u * UV + lane;
        if (PAIR && !on) {  // converged by the step before
#pragma unroll
            for (int v = 0; v < kUnitVecs; ++v) {
                cpx<R> xc[N], pc[N];
                IO::get(x[base + v * 64], xc);
                IO::get(r_prev[base + v * 64], pc);
#pragma unroll
                for (int e = 0; e < N; ++e) cmac(xc[e], ap, pc[e]);
                x[base + v * 64] = IO::put(xc);
            }
            continue;
        }
        const double2 a2 = a.alpha[sys];
        const cpx<R> al = {(R)a2.x, (R)a2.y}, na = {(R)-a2.x, (R)-a2.y};
        R rr = 0;
#pragma unroll
        for (int v = 0; v < kUnitVecs; ++v) {
            const size_t i = base + v * 64;
            const uint4 rv = stream_load(r + i), qv = stream_load(q + i);
            cpx<R> xc[N], rc[N], qc[N];
            IO::get(rv, rc);
            IO::get(qv, qc);
            if constexpr (!LATER) {
                IO::get(stream_load(x + i), xc);
                if constexpr (PAIR) {
                    cpx<R> pc[N];
                    IO::get(stream_load(r_prev + i), pc);
#pragma unroll
                    for (int e = 0; e < N; ++e) cmac(xc[e], ap, pc[e]);
                    IO::get(IO::put(xc), xc);  // as the step before would have stored it
                }
#pragma unroll
                for (int e = 0; e < N; ++e) cmac(xc[e], al, rc[e]);
                stream_store(x + i, IO::put(xc));
            }
#pragma unroll
            for (int e = 0; e < N; ++e) cmac(rc[e], na, qc[e]);
            const uint4 ro = IO::put(rc);
            r_out[i] = ro;
            IO::get(ro, rc);  // the norm of the values as stored
#pragma unroll
            for (int e = 0; e < N; ++e) rr = fma(rc[e].re, rc[e].re, fma(rc[e].im, rc[e].im, rr));
        }
        const double t[1] = {(double)rr};
        part.add(sys, t);
    }
    part.flush(a.partials);
}

// r_out = r_in - f (D_rr e), x_out = x_in + f e in FP64, f = sqrt(fr2[sys]).
// 48 lattices, 1.2 million sites, 4 RHS: 1.6 ms, its bytes 0.9 of it; the rest
// is the wait for operands with four wavefronts per SIMD (112 VGPRs).
template <int P>
__global__ void __launch_bounds__(128) batch_dc_update_kernel(BatchDcArgs a)
{
    typedef typename Store<P>::S S;
    extern __shared__ double smem[];
    SysPartial<1> part;
    part.init(smem, a.bt.nlat * a.nrhs);
    const S *__restrict__ e = (const S *)a.e;
    const double2 *__restrict__ U = (const double2 *)a.U;
    const double2 *r_in = (const double2 *)a.r_in;
    const double2 *x_in = (const double2 *)a.x_in;
    double2 *r_out = (double2 *)a.r_out;
    double2 *x_out = (double2 *)a.x_out;
    const int nsys = a.bt.nlat * a.nrhs;
    const bool in_place = a.r_in == a.r_out && a.x_in == a.x_out;
    if (a.act) {
        const bool any = any_set(a.act, nsys);
        if (any && a.ctr && blockIdx.x == 0 && threadIdx.x == 0) atomicAdd(a.ctr, 1);
        if (a.gate && !any) return;
    }
    const ItemRange it = xcd_items(a.Vtot / blockDim.x * a.nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        int tile, r;
        tile_item(w, a.nrhs, tile, r);
        const int s = tile * 64 + (int)(threadIdx.x & 63);
        const BSite b = bsite(a.bt, s);
        const bool on = a.mask[s] == 0;
        const SiteGeo q = site_geo(b.local, b.g);
        {
            const int sys = b.l * a.nrhs + r;
            const bool sys_on = a.act == nullptr || a.act[sys] != 0;
            if (in_place && !sys_on) continue;  // converged: r and x stay
            double nrm = 0;
            if (on && !sys_on) {
                // converged before this step: r and x copied, e not read
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const size_t i = fidx(s, r, c, a.nrhs);
                    const double2 rv = r_in[i];
                    r_out[i] = rv;
                    nrm += rv.x * rv.x + rv.y * rv.y;
                    x_out[i] = x_in ? x_in[i] : make_double2(0.0, 0.0);
                }
            } else if (on) {
                cpx<double> acc[12];
                dslash_site<S, double, true, double2>(acc, e, U, s, q, b.g, r, a.nrhs, a.bt.diag[b.l]);
                const double f = sqrt(a.fr2[sys]);
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const size_t i = fidx(s, r, c, a.nrhs);
                    const double2 rv = r_in[i];
                    const double2 d = make_double2(rv.x - f * acc[c].re, rv.y - f * acc[c].im);
                    r_out[i] = d;
                    nrm += d.x * d.x + d.y * d.y;
                    const cpx<double> ev = ldr<double>(e, i);
                    const double2 xv = x_in ? x_in[i] : make_double2(0.0, 0.0);
                    x_out[i] = make_double2(xv.x + f * ev.re, xv.y + f * ev.im);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const size_t i = fidx(s, r, c, a.nrhs);
                    r_out[i] = make_double2(0.0, 0.0);
                    x_out[i] = make_double2(0.0, 0.0);
                }
            }
            const double v[1] = {nrm};
            part.add(sys, v);
        }
    }
    part.flush(a.partials);
}

// in_r = r_src / sqrt(fr2) in the inner precision, in_x = 0, partial |in_r|^2
// (of the stored values); systems whose flag is 0 get zeros
template <int PO>
__global__ void __launch_bounds__(256) batch_inner_init_kernel(BatchBlasArgs a, const double2 *r_src,
                                                               const double *fr2, void *in_r_, void *in_x_)
{
    typedef typename Store<PO>::S S;
    typedef typename Store<PO>::R R;
    extern __shared__ double smem[];
    const int nsys = a.bt.nlat * a.nrhs;
    if (a.act && !any_set(a.act, nsys)) return;
    SysPartial<1> part;
    part.init(smem, nsys);
    S *in_r = (S *)in_r_, *in_x = (S *)in_x_;
    const ItemRange it = xcd_items(a.Vtot / 256);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int s = w * 256 + threadIdx.x;
        const int l = a.bt.tile_lat[s >> 6];
        for (int k = 0; k < a.nrhs; ++k) {
            const int sys = l * a.nrhs + k;
            const bool on = a.act == nullptr || a.act[sys] != 0;
            const double f2 = fr2[sys];
            const double f = on && f2 > 0 ? 1.0 / sqrt(f2) : 0.0;
            double t = 0;
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                const size_t i = fidx(s, k, c, a.nrhs);
                const double2 v = on ? r_src[i] : make_double2(0.0, 0.0);
                stc(in_r, i, cpx<R>{(R)(f * v.x), (R)(f * v.y)});
                stc(in_x, i, cpx<R>{(R)0, (R)0});
                const cpx<R> st = ldc(in_r, i);
                t += (double)st.re * st.re + (double)st.im * st.im;
            }
            const double vv[1] = {t};
            part.add(sys, vv);
        }
    }
    part.flush(a.partials);
}

// one workgroup per system: the fixed-order sum of its partials (as the
// single-lattice reduction), gated by act_in
__global__ void __launch_bounds__(256) batch_reduce_kernel(int mode, const double *partials, int nparts,
                                                           int nsys, double2 *alpha, double *out2,
                                                           const double *thr2, const int *act_in,
                                                           int *act_out)
{
    if (act_in && !any_set(act_in, nsys)) return;
    const int r = blockIdx.x;
    if (act_in && !act_in[r]) {
        if (threadIdx.x == 0) {
            if (mode == kAlpha) alpha[r] = make_double2(0.0, 0.0);
            if (act_out && act_out != act_in) act_out[r] = 0;
        }
        return;
    }
    double sums[3] = {0, 0, 0};
    if (mode == kNorm) block_rows_sum<1>(partials, nparts, r, sums, nsys);
    else block_rows_sum<3>(partials, nparts, r, sums, nsys);
    if (threadIdx.x != 0) return;
    if (mode == kAlpha) {
        alpha[r] = mr_alpha(sums, true);
    } else {
        const double n2 = sums[mode == kNorm3 ? 2 : 0];
        if (out2) out2[r] = n2;
        if (act_out) act_out[r] = n2 > thr2[r] ? 1 : 0;
    }
}

// the outer control of the defect correction, one thread per system: the
// relative FP64 residual against tol, the next inner threshold (the inner
// solve reduces the scaled residual by max(inner_tol, need / 2), or by need
// itself in FP64, need = tol |b| / |r|) and the scale |r|^2
__global__ void __launch_bounds__(256) batch_ctl_kernel(BatchCtlArgs c)
{
    if (c.init && blockIdx.x == 0 && threadIdx.x < 2) c.ctr[threadIdx.x] = 0;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < c.nsys; k += gridDim.x * blockDim.x) {
        const double b2 = c.bn2[k];
        if (c.init) c.rn2[k] = b2;
        const double r2 = c.rn2[k];
        const double rel = b2 > 0 ? sqrt(r2 / b2) : 0.0;
        const bool on = b2 > 0 && rel > c.tol;  // a NaN residual is left to the host's check
        const double need = b2 > 0 && r2 > 0 ? c.tol * sqrt(b2 / r2) : 1.0;
        const double relt = c.fp64_inner ? need : fmax(c.inner_tol, 0.5 * need);
        c.thr2[k] = on ? relt * relt : 2.0;
        c.fr2[k] = r2;
        c.oact[k] = on ? 1 : 0;
    }
}

// The site of side po (0: the lattice's reduced parity, 1: the other) at
// half-site h: 2h and 2h + 1 differ in parity (Lx even), 2h having the
// parity of y + z + t.
__device__ __forceinline__ int half_site(int h, int4 d, int parity)
{
    const int t1 = (2 * h) / d.x;
    const int y = t1 % d.y, t2 = t1 / d.y;
    const int z = t2 % d.z, t = t2 / d.z;
    return 2 * h + ((parity ^ (y + z + t)) & 1);
}

// b = D_rb x_b over the batch (FP64, zero on the coarse sites), from the
// coarse neighbours alone, with the per-system |b|^2: as rb_apply_kernel.
// (48 lattices, 1.2 million sites, 4 RHS: 0.46 ms, the write of b 0.2 of it;
// a scatter of x_b, D over the whole field and a norm pass took 1.4.)
__global__ void __launch_bounds__(256) batch_rb_kernel(BatchCoarseArgs a, double2 *__restrict__ b, double *partials)
{
    extern __shared__ double smem[];
    SysPartial<1> part;
    part.init(smem, a.bt.nlat * a.nrhs);
    const double2 *__restrict__ xb = (const double2 *)a.xb, *__restrict__ U = (const double2 *)a.U;
    const ItemRange it = xcd_items(a.Vtot / 256 * a.nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        int tile, r;
        tile_item(w, a.nrhs, tile, r);
        const int s = tile * 64 + (int)(threadIdx.x & 63);
        const BSite bs = bsite(a.bt, s);
        cpx<double> acc[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = {0, 0};
        if (a.bidx[s] < 0) {
            const SiteGeo q = site_geo(bs.local, bs.g);
            const int fo = a.bt.off[bs.l];
            const double2 *x = xb + a.coff[bs.l] + (size_t)r * a.nb[bs.l] * 12;
#pragma unroll 1
            for (int k = 0; k < 8; ++k) {
                int sp, sm;
                nbr(bs.local, k >> 1, q, bs.g, sp, sm);
                const int kb = a.bidx[fo + ((k & 1) ? sm : sp)];
                if (kb < 0) continue;
                cpx<double> p[12], u[9];
#pragma unroll
                for (int c = 0; c < 12; ++c) p[c] = {x[(size_t)kb * 12 + c].x, x[(size_t)kb * 12 + c].y};
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    const double2 l = U[lidx(fo + ((k & 1) ? sm : bs.local), k >> 1, e)];
                    u[e] = {l.x, l.y};
                }
                switch (k) {
                case 0: hop_math<0, true>(acc, p, u); break;
                case 1: hop_math<0, false>(acc, p, u); break;
                case 2: hop_math<1, true>(acc, p, u); break;
                case 3: hop_math<1, false>(acc, p, u); break;
                case 4: hop_math<2, true>(acc, p, u); break;
                case 5: hop_math<2, false>(acc, p, u); break;
                case 6: hop_math<3, true>(acc, p, u); break;
                default: hop_math<3, false>(acc, p, u); break;
                }
            }
        }
        double n2 = 0;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            b[fidx(s, r, c, a.nrhs)] = make_double2(acc[c].re, acc[c].im);
            n2 += acc[c].re * acc[c].re + acc[c].im * acc[c].im;
        }
        const double v[1] = {n2};
        part.add(bs.l * a.nrhs + r, v);
    }
    part.flush(partials);
}

// r = b - D_rr x on the rest sites, zero on the coarse ones, with the
// per-system |r|^2 (the same batch: 1.26 ms; D, then the difference with its
// norm took 1.0 + 0.53)
__global__ void __launch_bounds__(256) batch_residual_kernel(BatchResidualArgs a)
{
    extern __shared__ double smem[];
    SysPartial<1> part;
    part.init(smem, a.bt.nlat * a.nrhs);
    const double2 *__restrict__ x = (const double2 *)a.x, *__restrict__ U = (const double2 *)a.U;
    const double2 *__restrict__ b = (const double2 *)a.b;
    double2 *__restrict__ ro = (double2 *)a.r;
    const ItemRange it = xcd_items(a.Vtot / 256 * a.nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        int tile, r;
        tile_item(w, a.nrhs, tile, r);
        const int s = tile * 64 + (int)(threadIdx.x & 63);
        const BSite bs = bsite(a.bt, s);
        double n2 = 0;
        if (a.mask[s] == 0) {
            const SiteGeo q = site_geo(bs.local, bs.g);
            cpx<double> acc[12];
            dslash_site<double2, double, true>(acc, x, U, s, q, bs.g, r, a.nrhs, a.bt.diag[bs.l]);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                const size_t i = fidx(s, r, c, a.nrhs);
                const double2 d = make_double2(b[i].x - acc[c].re, b[i].y - acc[c].im);
                ro[i] = d;
                n2 += d.x * d.x + d.y * d.y;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 12; ++c) ro[fidx(s, r, c, a.nrhs)] = make_double2(0.0, 0.0);
        }
        const double v[1] = {n2};
        part.add(bs.l * a.nrhs + r, v);
    }
    part.flush(a.partials);
}

// y_b = [D (u - z)]_b, u = x_b on the coarse sites: the neighbours of a coarse
// site are read as x_b or -z.  64 coarse sites and one RHS per workgroup, a
// hop per wavefront (split.h); a workgroup may span lattices.  (The same batch:
// 0.18 ms; u - z over the whole field and a lane per coarse site took 0.53 + 0.2.)
__global__ void __launch_bounds__(kSplitThreads) batch_coarse_kernel(BatchCoarseArgs a, const double2 *__restrict__ z,
                                                                     double2 *__restrict__ yb)
{
    __shared__ HopSums<double> sums;
    const double2 *__restrict__ xb = (const double2 *)a.xb, *__restrict__ U = (const double2 *)a.U;
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nkb = (a.nbtot + 63) >> 6;
    const ItemRange it = xcd_items(nkb * a.nrhs);
    for (int wi = it.begin; wi < it.end; wi += it.step) {
        const int kb = wi / a.nrhs, r = wi - kb * a.nrhs;
        const int kg = kb * 64 + lane;
        size_t x0 = 0;
        int l = 0;
        if (kg < a.nbtot) {
            const int s = a.qg[kg];
            const BSite bs = bsite(a.bt, s);
            l = bs.l;
            x0 = a.coff[l] + (size_t)r * a.nb[l] * 12;
            const int fo = a.bt.off[l];
            const SiteGeo q = site_geo(bs.local, bs.g);
            int sp, sm;
            nbr(bs.local, k >> 1, q, bs.g, sp, sm);
            const int n = fo + ((k & 1) ? sm : sp), kn = a.bidx[n];
            cpx<double> p[12], u[9], w[6];
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const double2 v = U[lidx(fo + ((k & 1) ? sm : bs.local), k >> 1, e)];
                u[e] = {v.x, v.y};
            }
            if (kn >= 0) {
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const double2 v = xb[x0 + (size_t)kn * 12 + c];
                    p[c] = {v.x, v.y};
                }
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const double2 v = z[fidx(n, r, c, a.nrhs)];
                    p[c] = {0.0 - v.x, 0.0 - v.y};
                }
            }
            hop_w_k(k, w, p, u);
            sums.put(k, lane, w);
        }
        __syncthreads();
        if (k < 6 && kg < a.nbtot) {
            const int row = k % 3, spin = k < 3 ? 0 : 2;
            const size_t i = x0 + (size_t)(kg - a.nboff[l]) * 12 + 3 * spin + row;
            const double2 v0 = xb[i], v1 = xb[i + 3];
            const double diag = a.bt.diag[l];
            cpx<double> a0 = {diag * v0.x, diag * v0.y}, a1 = {diag * v1.x, diag * v1.y};
            if (spin == 0) sums.add<false>(row, lane, a0, a1);
            else sums.add<true>(row, lane, a0, a1);
            yb[i] = make_double2(a0.re, a0.im);
            yb[i + 3] = make_double2(a1.re, a1.im);
        }
        __syncthreads();  // the sums are read before the next item's overwrite them
    }
}

// The links once more by side (0: the reduced parity's sites, 1: the others),
// compact like the half fields: a half-step over the full layout's links used
// half of every line it read, forward and backward (48 lattices, 1.2 million
// sites, FP32, 4 RHS: 313 us per half-step, 290 with these).
template <class S>
__global__ void __launch_bounds__(256) batch_half_links_kernel(BatchTable bt, BatchHalf hf, const S *__restrict__ U,
                                                               S *__restrict__ Uh)
{
    const int H = blockIdx.x * 256 + threadIdx.x;
    if (H >= hf.Vtot) return;
    const int l = hf.tile_lat[H >> 6];
    const int4 d = bt.dims[l];
    const int h = H - hf.off[l];
    const bool valid = 2 * h < d.x * d.y * d.z * d.w;
    const int sp = valid ? half_site(h, d, hf.par[l]) : 0;
    for (int side = 0; side < 2; ++side) {
        const int s = bt.off[l] + (side ? sp ^ 1 : sp);
        for (int mu = 0; mu < 4; ++mu)
#pragma unroll
            for (int e = 0; e < 9; ++e)
                Uh[(size_t)side * 36 * hf.Vtot + hlidx<S>(H, mu, e)] = valid ? U[lidx(s, mu, e)] : S{};
    }
}

// The scaled residual r / sqrt(fr2) in the inner precision straight into the
// two compact halves of the reduced solve's right-hand side (the padding of
// the halves stays zero); systems whose flag is 0 get zeros.  Bound by its bytes
// (48 lattices, 4 RHS: 0.28 ms at 4.9 TB/s; through the full layout 0.75).
template <int PO>
__global__ void __launch_bounds__(256) batch_inner_split_kernel(BatchBlasArgs a, BatchHalf hf,
                                                                const double2 *__restrict__ r_src,
                                                                const double *__restrict__ fr2, void *bp_, void *bq_)
{
    typedef typename Store<PO>::S S;
    typedef typename Store<PO>::R R;
    if (a.act && !any_set(a.act, a.bt.nlat * a.nrhs)) return;
    S *bp = (S *)bp_, *bq = (S *)bq_;
    const ItemRange it = xcd_items(a.Vtot / 256 * a.nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        const int sb = w / a.nrhs, r = w - sb * a.nrhs;
        const int s = sb * 256 + (int)threadIdx.x;
        const BSite bs = bsite(a.bt, s);
        const int sys = bs.l * a.nrhs + r;
        const bool on = a.act == nullptr || a.act[sys] != 0;
        const double f2 = fr2[sys];
        const double f = on && f2 > 0 ? 1.0 / sqrt(f2) : 0.0;
        const SiteGeo q = site_geo(bs.local, bs.g);
        const bool p_side = ((q.c[0] ^ q.c[1] ^ q.c[2] ^ q.c[3]) & 1) == hf.par[bs.l];
        S *o = p_side ? bp : bq;
        const int H = hf.off[bs.l] + (bs.local >> 1);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const double2 v = on ? r_src[fidx(s, r, c, a.nrhs)] : make_double2(0.0, 0.0);
            stc(o, hidx<S>(H, r, c, a.nrhs), cpx<R>{(R)(f * v.x), (R)(f * v.y)});
        }
    }
}

// ------------------------------------------------------------------ launchers
static size_t lds_sys(int nsys, int K) { return (size_t)4 * nsys * K * sizeof(double); }

// ------------------------------------------------------------------ even-odd reduced form
template <int P>
__global__ void __launch_bounds__(256) batch_eo_kernel(BatchEoArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    typedef Operand<S, R> OP;
    typedef typename OP::T PT;
    extern __shared__ double smem[];
    const S *__restrict__ in = (const S *)a.in;
    const S *__restrict__ in2 = (const S *)a.in2;
    S *__restrict__ out = (S *)a.out;
    // the links of the output's side and of the input's
    const S *__restrict__ Uo = (const S *)a.U + (size_t)a.po * 36 * a.hf.Vtot;
    const S *__restrict__ Ui = (const S *)a.U + (size_t)(1 - a.po) * 36 * a.hf.Vtot;
    const int nsys = a.bt.nlat * a.nrhs;
    if (a.act && !any_set(a.act, nsys)) return;
    const bool dots = a.partials != nullptr;
    SysPartial<3> part;
    if (dots) part.init(smem, nsys);
    const uint8_t *mk = a.hf.mask + (size_t)a.po * a.hf.Vtot;
    const ItemRange it = xcd_items(a.hf.Vtot / 256 * a.nrhs);
    for (int w = it.begin; w < it.end; w += it.step) {
        int tile, r;
        tile_item(w, a.nrhs, tile, r);
        const int H = tile * 64 + (int)(threadIdx.x & 63);
        const int l = a.hf.tile_lat[tile];
        const int4 d = a.bt.dims[l];
        Geom g;
        g.L[0] = d.x;
        g.L[1] = d.y;
        g.L[2] = d.z;
        g.L[3] = d.w;
        g.V = g.Vs = d.x * d.y * d.z * d.w;
        const bool on = mk[H] == 0;  // rest site (coarse sites and padding are masked)
        const int par = a.po ? 1 - a.hf.par[l] : a.hf.par[l];
        const int s = half_site(on ? H - a.hf.off[l] : 0, d, par);  // local full site
        const SiteGeo q = site_geo(s, g);
        const int co = a.hf.off[l];
        const R ca = (R)a.ca[l], cb = (R)a.cb[l];
        {
            if (a.act && !a.act[l * a.nrhs + r]) continue;  // uniform in the wavefront
            cpx<R> acc[12], v2[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) acc[c] = v2[c] = {0, 0};
            if (on) {
#pragma unroll 1
                for (int hp = 0; hp < 8; ++hp) {
                    const int mu = hp >> 1;
                    int sp, sm;
                    nbr(s, mu, q, g, sp, sm);
                    // the neighbour (other side) at its half-site index
                    const int n = co + (((hp & 1) ? sm : sp) >> 1);
                    PT p[12], u[9];
                    load_half<S, R>(p, in, n, r, a.nrhs);
                    load_half_link<S, R>(u, (hp & 1) ? Ui : Uo, (hp & 1) ? n : H, mu);
                    switch (hp) {
                    case 0: hop<0, true>(acc, p, u); break;
                    case 1: hop<0, false>(acc, p, u); break;
                    case 2: hop<1, true>(acc, p, u); break;
                    case 3: hop<1, false>(acc, p, u); break;
                    case 4: hop<2, true>(acc, p, u); break;
                    case 5: hop<2, false>(acc, p, u); break;
                    case 6: hop<3, true>(acc, p, u); break;
                    default: hop<3, false>(acc, p, u); break;
                    }
                }
                if (in2) load_half_vals<S, R>(v2, in2, H, r, a.nrhs);
#pragma unroll
                for (int c = 0; c < 12; ++c)
                    acc[c] = {ca * v2[c].re + cb * acc[c].re, ca * v2[c].im + cb * acc[c].im};
            }
            store_half<S, R>(out, acc, H, r, a.nrhs);
            if (dots) {
                R sre = 0, sim = 0, sqq = 0;
                if (on) {
#pragma unroll
                    for (int c = 0; c < 12; ++c) {
                        const cpx<R> v = v2[c];
                        sre = fma(acc[c].re, v.re, fma(acc[c].im, v.im, sre));
                        sim = fma(acc[c].re, v.im, fma(-acc[c].im, v.re, sim));
                        sqq = fma(acc[c].re, acc[c].re, fma(acc[c].im, acc[c].im, sqq));
                    }
                }
                const double dd[3] = {(double)sre, (double)sim, (double)sqq};
                part.add(l * a.nrhs + r, dd);
            }
        }
    }
    if (dots) part.flush(a.partials);
}

template <int P>
__global__ void __launch_bounds__(256) batch_eo_join_kernel(BatchTable bt, BatchHalf hf, int nrhs, void *x_,
                                                            const void *xp_, const void *xq_)
{
    typedef typename Store<P>::S S;
    S *x = (S *)x_;
    const S *xp = (const S *)xp_, *xq = (const S *)xq_;
    const size_t n = (size_t)hf.Vtot * nrhs * 12;
    for (size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (size_t)gridDim.x * blockDim.x) {
        // j = (compact tile, RHS, component, lane)
        const size_t rest = j >> 6;
        const int tile = (int)(rest / ((size_t)nrhs * 12)), rc = (int)(rest - (size_t)tile * nrhs * 12);
        const int r = rc / 12, c = rc - r * 12;
        const int H = tile * 64 + (int)(j & 63);
        const int l = hf.tile_lat[tile];
        const int4 d = bt.dims[l];
        const int h = H - hf.off[l];
        const bool valid = 2 * h < d.x * d.y * d.z * d.w;
        const int sp = half_site(valid ? h : 0, d, hf.par[l]);
        const int sq = sp ^ 1;  // the other site of the pair
        const size_t gp = fidx(bt.off[l] + sp, r, c, nrhs), gq = fidx(bt.off[l] + sq, r, c, nrhs);
        if (valid) {
            const size_t i = hidx<S>(H, r, c, nrhs);
            x[gp] = xp[i];
            x[gq] = xq[i];
        }
    }
}

hipError_t launch_batch_eo(int prec, const BatchEoArgs &a, int grid, hipStream_t st)
{
    const size_t lds = a.partials ? lds_sys(a.bt.nlat * a.nrhs, 3) : 0;
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(batch_eo_kernel<GRG_FP64>, dim3(grid), dim3(256), lds, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(batch_eo_kernel<GRG_FP32>, dim3(grid), dim3(256), lds, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(batch_eo_kernel<GRG_BF16>, dim3(grid), dim3(256), lds, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_eo_join(int prec, const BatchTable &bt, const BatchHalf &hf, int nrhs, void *x,
                                const void *xp, const void *xq, int grid, hipStream_t st)
{
    switch (prec) {
    case GRG_FP64:
        hipLaunchKernelGGL(batch_eo_join_kernel<GRG_FP64>, dim3(grid), dim3(256), 0, st, bt, hf, nrhs, x, xp, xq);
        break;
    case GRG_FP32:
        hipLaunchKernelGGL(batch_eo_join_kernel<GRG_FP32>, dim3(grid), dim3(256), 0, st, bt, hf, nrhs, x, xp, xq);
        break;
    case GRG_BF16:
        hipLaunchKernelGGL(batch_eo_join_kernel<GRG_BF16>, dim3(grid), dim3(256), 0, st, bt, hf, nrhs, x, xp, xq);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_dslash_batch(int prec, const BatchDslashArgs &a, int grid, int SB, hipStream_t st)
{
    if (SB != 64 && SB != 128 && SB != 256) return hipErrorInvalidValue;
    const size_t lds = a.partials ? lds_sys(a.bt.nlat * a.nrhs, 3) : 0;
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(dslash_batch_kernel<GRG_FP64>, dim3(grid), dim3(SB), lds, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(dslash_batch_kernel<GRG_FP32>, dim3(grid), dim3(SB), lds, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(dslash_batch_kernel<GRG_BF16>, dim3(grid), dim3(SB), lds, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define BDISP(prec, KERNEL, lds, ...)                                                                  \
    switch (prec) {                                                                                    \
    case GRG_FP64: hipLaunchKernelGGL(KERNEL<GRG_FP64>, dim3(a.grid), dim3(256), lds, st, __VA_ARGS__); break; \
    case GRG_FP32: hipLaunchKernelGGL(KERNEL<GRG_FP32>, dim3(a.grid), dim3(256), lds, st, __VA_ARGS__); break; \
    case GRG_BF16: hipLaunchKernelGGL(KERNEL<GRG_BF16>, dim3(a.grid), dim3(256), lds, st, __VA_ARGS__); break; \
    default: return hipErrorInvalidValue;                                                             \
    }

hipError_t launch_batch_mr_update(int prec, const BatchBlasArgs &a, void *x, void *r, const void *q,
                                  hipStream_t st)
{
    const size_t lds = lds_sys(a.bt.nlat * a.nrhs, 1);
    const bool later = a.r_later != nullptr, pair = a.r_prev != nullptr;
    if ((later || pair) && (later == pair || !a.act || !a.pend || (pair && !a.alpha_prev)))
        return hipErrorInvalidValue;
    switch (prec) {
#define BMR(PP, XM) \
    hipLaunchKernelGGL((batch_mr_update_kernel<PP, XM>), dim3(a.grid), dim3(256), lds, st, a, x, r, q)
#define BMU(PP)                          \
    if (later) BMR(PP, kMrXLater);       \
    else if (pair) BMR(PP, kMrXPair);    \
    else BMR(PP, kMrXAdd);               \
    break;
    case GRG_FP64: BMU(GRG_FP64)
    case GRG_FP32: BMU(GRG_FP32)
    case GRG_BF16: BMU(GRG_BF16)
#undef BMU
#undef BMR
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_dc_update(int prec, const BatchDcArgs &a, int grid, hipStream_t st)
{
    const size_t lds = lds_sys(a.bt.nlat * a.nrhs, 1);
    dim3 g(grid), b(128);
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(batch_dc_update_kernel<GRG_FP64>, g, b, lds, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(batch_dc_update_kernel<GRG_FP32>, g, b, lds, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(batch_dc_update_kernel<GRG_BF16>, g, b, lds, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_inner_init(int prec, const BatchBlasArgs &a, const void *r_src, const double *fr2,
                                   void *in_r, void *in_x, hipStream_t st)
{
    BDISP(prec, batch_inner_init_kernel, lds_sys(a.bt.nlat * a.nrhs, 1), a, (const double2 *)r_src, fr2, in_r,
          in_x);
    return hipGetLastError();
}

hipError_t launch_batch_reduce(int mode, const double *partials, int nparts, int nsys, double2 *alpha,
                               double *out2, const double *thr2, const int *act_in, int *act_out,
                               hipStream_t st)
{
    if (nsys < 1 || nparts < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_reduce_kernel, dim3(nsys), dim3(256), 0, st, mode, partials, nparts, nsys, alpha,
                       out2, thr2, act_in, act_out);
    return hipGetLastError();
}

hipError_t launch_batch_ctl(const BatchCtlArgs &c, hipStream_t st)
{
    if (c.nsys < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_ctl_kernel, dim3((c.nsys + 255) / 256), dim3(256), 0, st, c);
    return hipGetLastError();
}

hipError_t launch_batch_rb(const BatchCoarseArgs &c, double2 *b, double *partials, int grid, hipStream_t st)
{
    hipLaunchKernelGGL(batch_rb_kernel, dim3(grid), dim3(256), lds_sys(c.bt.nlat * c.nrhs, 1), st, c, b, partials);
    return hipGetLastError();
}

hipError_t launch_batch_residual(const BatchResidualArgs &a, int grid, hipStream_t st)
{
    hipLaunchKernelGGL(batch_residual_kernel, dim3(grid), dim3(256), lds_sys(a.bt.nlat * a.nrhs, 1), st, a);
    return hipGetLastError();
}

hipError_t launch_batch_coarse(const BatchCoarseArgs &c, const void *z, double *yb, hipStream_t st)
{
    const long items = (long)((c.nbtot + 63) / 64) * c.nrhs;
    const int grid = (int)std::max<long>(8, (std::min<long>(items, 2048) + 7) / 8 * 8);
    hipLaunchKernelGGL(batch_coarse_kernel, dim3(grid), dim3(kSplitThreads), 0, st, c, (const double2 *)z,
                       (double2 *)yb);
    return hipGetLastError();
}

hipError_t launch_batch_half_links(int prec, const BatchTable &bt, const BatchHalf &hf, const void *U, void *Uh,
                                   hipStream_t st)
{
    const dim3 g((hf.Vtot + 255) / 256), b(256);
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(batch_half_links_kernel<double2>, g, b, 0, st, bt, hf, (const double2 *)U, (double2 *)Uh); break;
    case GRG_FP32: hipLaunchKernelGGL(batch_half_links_kernel<float2>, g, b, 0, st, bt, hf, (const float2 *)U, (float2 *)Uh); break;
    case GRG_BF16: hipLaunchKernelGGL(batch_half_links_kernel<bf16x2>, g, b, 0, st, bt, hf, (const bf16x2 *)U, (bf16x2 *)Uh); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_inner_split(int prec, const BatchBlasArgs &a, const BatchHalf &hf, const void *r_src,
                                    const double *fr2, void *bp, void *bq, hipStream_t st)
{
    const dim3 g((unsigned)std::max<long>(8, std::min<long>((long)a.Vtot / 256 * a.nrhs, 2048) / 8 * 8)), b(256);
#define BIS(PP) hipLaunchKernelGGL(batch_inner_split_kernel<PP>, g, b, 0, st, a, hf, (const double2 *)r_src, fr2, bp, bq)
    switch (prec) {
    case GRG_FP64: BIS(GRG_FP64); break;
    case GRG_FP32: BIS(GRG_FP32); break;
    case GRG_BF16: BIS(GRG_BF16); break;
    default: return hipErrorInvalidValue;
    }
#undef BIS
    return hipGetLastError();
}

}  // namespace grg
