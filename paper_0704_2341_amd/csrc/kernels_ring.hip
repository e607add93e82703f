// D on large canonical complex128 fields in one launch: a t-march whose
// wavefronts keep their column in LDS.
//
// A workgroup is one wavefront: 64 consecutive sites of a 3-d slice for one
// right-hand side, walking t.  Its LDS holds three images of 64 spinors: slices t - 1 and t of the column, and
// a stage through which every other neighbour passes.  A chunk of 64 spinors is
// read with four lanes on each 64 bytes, so that a load touches 16 lines instead of
// the 64 of a lane per spinor, and a lane then takes its spinor from LDS; the
// result goes out the same way.  The chunk of the next hop and the links of the
// next direction are in flight while a hop is summed.  The stage ends a slice
// holding slice t + 1, and the three images change roles.
//
// Why: packing the field into tiles first costs its read and write again, and
// the site-parallel stencil then reads nine spinors and eight links per site and
// RHS from L2, which bounds it (32^4, 12 RHS, FP64: 1.18 + 2.70 ms, 33 GB from L2 in
// the second).  Here a spinor is read five times (the x neighbours come from the
// slice's image where x-rows tile the 64 lanes, the t neighbours always): 2.07 ms,
// its bytes 1.1 of it, in FP32 3.41 -> 1.83, in BF16 2.61 -> 1.63; 16^4, 12 RHS: 246 ->
// 130, 193 -> 100, 149 -> 104 us.  What is left is latency: a wavefront per SIMD in
// FP64 (its registers, 40 KB of LDS each), two in the others.  Four wavefronts per
// workgroup gained nothing over one (2.13 ms), and streaming stores leave the caches
// to the input (16^4, FP64: 130 us, 147 without).
//
// The hops of a site are summed in the order of dslash_site, to the same bits.
#include "common.h"
#include "engine.h"
#include "stencil.h"

namespace grg {

namespace {

// an LDS element: a component as the hops take it, 16-byte aligned in FP64
template <int P>
struct RingEl;
template <>
struct RingEl<GRG_FP64> {
    typedef double2 T;
    __device__ static T in(double2 v) { return v; }
    __device__ static cpx<double> op(T v) { return {v.x, v.y}; }
    __device__ static T out(cpx<double> v) { return make_double2(v.re, v.im); }
    __device__ static double2 wide(T v) { return v; }
};
template <>
struct RingEl<GRG_FP32> {
    typedef float2 T;
    __device__ static T in(double2 v) { return make_float2((float)v.x, (float)v.y); }
    __device__ static cpx<float> op(T v) { return {v.x, v.y}; }
    __device__ static T out(cpx<float> v) { return make_float2(v.re, v.im); }
    __device__ static double2 wide(T v) { return make_double2((double)v.x, (double)v.y); }
};
template <>
struct RingEl<GRG_BF16> {
    typedef uint32_t T;
    __device__ static T in(double2 v) { return pack_bf16((float)v.x, (float)v.y); }
    __device__ static uint32_t op(T v) { return v; }
    __device__ static T out(cpx<float> v) { return pack_bf16(v.re, v.im); }
    __device__ static double2 wide(T v)
    {
        const cpx<float> c = as_cpx(v);
        return make_double2((double)c.re, (double)c.im);
    }
};

typedef double ring_v2 __attribute__((ext_vector_type(2)));
constexpr int kRingRow = 13;  // elements per spinor in LDS: lanes' reads meet no bank twice

}  // namespace

template <int P>
__global__ void __launch_bounds__(64, P == GRG_FP64 ? 1 : 2) canon_march_kernel(DslashArgs a)
{
    typedef typename Store<P>::S S;
    typedef typename Store<P>::R R;
    typedef Operand<S, R> OP;
    typedef typename OP::T PT;
    typedef RingEl<P> EL;
    typedef typename EL::T LT;
    __shared__ LT lds[3][64 * kRingRow];
    const double2 *__restrict__ in = (const double2 *)a.in;
    double2 *__restrict__ out = (double2 *)a.out;
    const S *__restrict__ U = (const S *)a.U;
    const int lane = threadIdx.x;
    const int q4 = lane & 3, l4 = lane >> 2;  // this lane's piece of the chunks' 64 bytes
    const int Lx = a.g.L[0], Lt = a.g.L[3], V = a.g.V;
    const int V3 = Lx * a.g.L[1] * a.g.L[2];
    const int nb3 = (V3 + 63) >> 6, T = a.march;
    const int ntc = (Lt + T - 1) / T;
    const int nitems = nb3 * ntc * a.nrhs;
    const R diag = (R)a.diag;
    // x neighbours in the slice's own image, by lane
    const bool xrow = 64 % Lx == 0 && (V3 & 63) == 0;
    const int xh = lane % Lx, rs = lane - xh;
    const int lp = rs + (xh + 1 == Lx ? 0 : xh + 1), lm = rs + (xh == 0 ? Lx - 1 : xh - 1);
    const int C = a.chunk > 0 ? a.chunk : (nitems + 7) / 8;
    for (int j = blockIdx.x >> 3;; j += gridDim.x >> 3) {
        const int w = xcd_chunk_item(j, C, nitems);
        if (w < 0) break;
        const int rest = w / a.nrhs, r = w - rest * a.nrhs;
        const int tc = rest / nb3, b3 = rest - tc * nb3;
        const int s3 = min(b3 * 64 + lane, V3 - 1);  // (lanes past the slice repeat its last site)
        const int t0 = tc * T, t1 = min(t0 + T, Lt);
        const double2 *__restrict__ inr = in + (size_t)r * V * 12;
        SiteGeo g3 = site_geo(s3, a.g);
        // the 64 spinors at the lanes' sites n, four lanes to 64 bytes
        double2 G[12];
        auto gather = [&](int n) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double2 *v = inr + (size_t)__shfl(n, l4 + 16 * i) * 12 + q4;
#pragma unroll
                for (int k = 0; k < 3; ++k) G[3 * i + k] = v[4 * k];
            }
        };
        // into an image (same-wavefront LDS accesses keep their order)
        auto put = [&](LT *dst) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < 3; ++k) dst[(l4 + 16 * i) * kRingRow + q4 + 4 * k] = EL::in(G[3 * i + k]);
            asm volatile("" ::: "memory");
        };
        auto get = [&](PT (&p)[12], const LT *src, int l) {
#pragma unroll
            for (int c = 0; c < 12; ++c) p[c] = EL::op(src[l * kRingRow + c]);
            asm volatile("" ::: "memory");
        };
        auto load_u = [&](PT (&u)[9], int site, int mu) {
#pragma unroll
            for (int e = 0; e < 9; ++e) u[e] = OP::load(U, lidx(site, mu, e));
        };
        LT *prev = lds[0], *cur = lds[1], *stage = lds[2];
        gather(s3 + V3 * (t0 == 0 ? Lt - 1 : t0 - 1));
        put(prev);
        gather(s3 + V3 * t0);
        put(cur);
        int sp, sm;
        nbr(s3, 0, g3, a.g, sp, sm);
        const int dxp = sp - s3, dxm = sm - s3;
        nbr(s3, 1, g3, a.g, sp, sm);
        const int d0 = xrow ? sp - s3 : dxp;  // the first staged hop's
        gather(s3 + V3 * t0 + d0);
        PT uf[9], ub[9];  // the direction's forward and backward link
        load_u(uf, s3 + V3 * t0, 0);
        load_u(ub, s3 + V3 * t0 + dxm, 0);
#pragma unroll 1
        for (int t = t0; t < t1; ++t) {
            const int s = s3 + V3 * t;
            g3.c[3] = t;
            const int sf = s3 + V3 * (t + 1 == Lt ? 0 : t + 1);
            cpx<R> acc[12];
            {
                PT p[12];
                get(p, cur, lane);
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const cpx<R> v = as_cpx(p[c]);
                    acc[c] = {diag * v.re, diag * v.im};
                }
            }
#pragma unroll 1
            for (int mu = 0; mu < 4; ++mu) {
                const bool own = mu == 0 && xrow;
                PT p[12];
                // forward; the chunk and link after it (after the last slice they are
                // not used, but in range)
                if (!own) put(stage);
                get(p, own ? cur : stage, own ? lp : lane);
                nbr(s, mu, g3, a.g, sp, sm);
                if (!own) gather(mu == 3 ? sf + d0 : sm);
                switch (mu) {
                case 0: hop<0, true>(acc, p, uf); break;
                case 1: hop<1, true>(acc, p, uf); break;
                case 2: hop<2, true>(acc, p, uf); break;
                default: hop<3, true>(acc, p, uf); break;
                }
                load_u(uf, mu == 3 ? sf : s, (mu + 1) & 3);
                // backward
                if (!own && mu < 3) put(stage);
                get(p, own ? cur : mu == 3 ? prev : stage, own ? lm : lane);
                nbr(s, (mu + 1) & 3, g3, a.g, sp, sm);
                if (!own && mu < 3) gather(sp);
                switch (mu) {
                case 0: hop<0, false>(acc, p, ub); break;
                case 1: hop<1, false>(acc, p, ub); break;
                case 2: hop<2, false>(acc, p, ub); break;
                default: hop<3, false>(acc, p, ub); break;
                }
                load_u(ub, mu == 3 ? sf + dxm : sm, (mu + 1) & 3);
            }
            // the result through the image of t - 1
#pragma unroll
            for (int c = 0; c < 12; ++c) prev[lane * kRingRow + c] = EL::out(acc[c]);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int l = l4 + 16 * i;
                if (b3 * 64 + l < V3) {
                    double2 *o = out + ((size_t)r * V + V3 * t + b3 * 64 + l) * 12 + q4;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double2 v = EL::wide(prev[l * kRingRow + q4 + 4 * k]);
                        __builtin_nontemporal_store(ring_v2{v.x, v.y}, (ring_v2 *)(o + 4 * k));
                    }
                }
            }
            asm volatile("" ::: "memory");
            LT *free = prev;
            prev = cur;
            cur = stage;
            stage = free;
        }
    }
}

hipError_t launch_canon_march(int prec, const DslashArgs &a, int grid, hipStream_t st)
{
    if (a.march < 1 || grid < 8 || grid % 8) return hipErrorInvalidValue;
    switch (prec) {
    case GRG_FP64: hipLaunchKernelGGL(canon_march_kernel<GRG_FP64>, dim3(grid), dim3(64), 0, st, a); break;
    case GRG_FP32: hipLaunchKernelGGL(canon_march_kernel<GRG_FP32>, dim3(grid), dim3(64), 0, st, a); break;
    case GRG_BF16: hipLaunchKernelGGL(canon_march_kernel<GRG_BF16>, dim3(grid), dim3(64), 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace grg
