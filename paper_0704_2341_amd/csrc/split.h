// A site's eight hops on eight wavefronts.
//
// A workgroup of 512 threads takes 64 sites for one right-hand side; wavefront
// k computes hop k (0..7 = +x, -x, ..., -t) of every site, up to the link
// product: the two colour vectors w0, w1 (six complex) that the hop's four spins
// are made of.  They meet in LDS, where six wavefronts (colour row, upper or
// lower spin pair) sum them in hop order, with the operations and the order of
// dslash_site, so that every output has the same bits.
//
// Why: a lane that walks the eight hops one after the other needs as many
// dependent round trips to memory.  On a small lattice there are too few lanes
// to cover them (4^4 to 12^4: 8.5 us per stencil however small the field), and a
// gather from scattered sites waits on each.  Here every hop's operands are in
// flight at once.
#pragma once

#include "common.h"
#include "engine.h"
#include "stencil.h"

namespace grg {

constexpr int kSplitThreads = 8 * kSplitSites;

// w = U h or U^+ h for both spins of h
template <bool FWD, class R>
__device__ __forceinline__ void link_mult(cpx<R> (&w)[6], const cpx<R> (&h0)[3], const cpx<R> (&h1)[3],
                                          const cpx<R> (&u)[9])
{
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        cpx<R> w0 = {0, 0}, w1 = {0, 0};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (FWD) {
                cmac(w0, u[3 * r + c], h0[c]);
                cmac(w1, u[3 * r + c], h1[c]);
            } else {
                cmacc(w0, u[3 * c + r], h0[c]);
                cmacc(w1, u[3 * c + r], h1[c]);
            }
        }
        w[r] = w0;
        w[3 + r] = w1;
    }
}

template <int MU, bool FWD, class R>
__device__ __forceinline__ void hop_w(cpx<R> (&w)[6], const cpx<R> (&p)[12], const cpx<R> (&u)[9])
{
    cpx<R> h0[3], h1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) project1<MU, FWD>(h0[a], h1[a], p[a], p[3 + a], p[6 + a], p[9 + a]);
    link_mult<FWD>(w, h0, h1, u);
}

// packed BF16 spinors with FP64 links (the defect correction of a BF16 inner
// solution) and with BF16 links
template <int MU, bool FWD>
__device__ __forceinline__ void hop_w(cpx<double> (&w)[6], const uint32_t (&p)[12], const cpx<double> (&u)[9])
{
    cpx<double> h0[3], h1[3];
    auto wd = [](uint32_t x) -> cpx<double> {
        return {(double)__uint_as_float(x << 16), (double)__uint_as_float(x & 0xffff0000u)};
    };
#pragma unroll
    for (int a = 0; a < 3; ++a)
        project1<MU, FWD>(h0[a], h1[a], wd(p[a]), wd(p[3 + a]), wd(p[6 + a]), wd(p[9 + a]));
    link_mult<FWD>(w, h0, h1, u);
}
template <int MU, bool FWD>
__device__ __forceinline__ void hop_w(cpx<float> (&w)[6], const uint32_t (&p)[12], const uint32_t (&u)[9])
{
    cpx<float> w0[3], w1[3];
    hop_bf16_w<MU, FWD>(w0, w1, p, u);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        w[r] = w0[r];
        w[3 + r] = w1[r];
    }
}

// hop k (the same in a wavefront)
template <class R, class PT, class UT>
__device__ __forceinline__ void hop_w_k(int k, cpx<R> (&w)[6], const PT (&p)[12], const UT (&u)[9])
{
    switch (k) {
    case 0: hop_w<0, true>(w, p, u); break;
    case 1: hop_w<0, false>(w, p, u); break;
    case 2: hop_w<1, true>(w, p, u); break;
    case 3: hop_w<1, false>(w, p, u); break;
    case 4: hop_w<2, true>(w, p, u); break;
    case 5: hop_w<2, false>(w, p, u); break;
    case 6: hop_w<3, true>(w, p, u); break;
    default: hop_w<3, false>(w, p, u); break;
    }
}

// The LDS image of a workgroup's hops.
template <class R>
struct HopSums {
    cpx<R> w[8][6][64];

    __device__ void put(int k, int lane, const cpx<R> (&v)[6])
    {
#pragma unroll
        for (int i = 0; i < 6; ++i) w[k][i][lane] = v[i];
    }
    // a0, a1 += the hops' contributions to colour `row` of spins 0, 1 (LOWER:
    // 2, 3) of site `lane`, hop 0 first
    template <bool LOWER>
    __device__ void add(int row, int lane, cpx<R> &a0, cpx<R> &a1) const
    {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int mu = k >> 1;
            const bool fwd = (k & 1) == 0;
            const cpx<R> w0 = w[k][row][lane], w1 = w[k][3 + row][lane];
            cpx<R> d0 = w0, d1 = w1;
            R f = R(-0.5);
            if (LOWER) {  // +/- 1/2 B^+ w, as hop_mult
                f = fwd ? R(0.5) : R(-0.5);
                if (mu == 0) {
                    d0 = {w1.im, -w1.re};
                    d1 = {w0.im, -w0.re};
                } else if (mu == 1) {
                    d0 = w1;
                    d1 = {-w0.re, -w0.im};
                } else if (mu == 2) {
                    d0 = {w0.im, -w0.re};
                    d1 = {-w1.im, w1.re};
                }
            }
            a0.re = fma(f, d0.re, a0.re);
            a0.im = fma(f, d0.im, a0.im);
            a1.re = fma(f, d1.re, a1.re);
            a1.im = fma(f, d1.im, a1.im);
        }
    }
};

}  // namespace grg
