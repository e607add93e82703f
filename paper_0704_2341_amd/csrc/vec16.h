// Fields as streams of 16-byte vectors, for kernels that treat every element
// alike (the minimal-residual updates).
#pragma once

#include "common.h"

namespace grg {

// 16-byte vectors of a field: 4 complex in BF16, 2 in FP32, 1 in FP64.
template <int P>
struct VecIO;
template <>
struct VecIO<GRG_BF16> {
    static constexpr int N = 4;
    typedef float R;
    __device__ static void get(const uint4 &v, cpx<float> (&c)[N])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < N; ++e) c[e] = {__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xffff0000u)};
    }
    __device__ static uint4 put(const cpx<float> (&c)[N])
    {
        return make_uint4(pack_bf16(c[0].re, c[0].im), pack_bf16(c[1].re, c[1].im),
                          pack_bf16(c[2].re, c[2].im), pack_bf16(c[3].re, c[3].im));
    }
};
template <>
struct VecIO<GRG_FP32> {
    static constexpr int N = 2;
    typedef float R;
    __device__ static void get(const uint4 &v, cpx<float> (&c)[N])
    {
        c[0] = {__uint_as_float(v.x), __uint_as_float(v.y)};
        c[1] = {__uint_as_float(v.z), __uint_as_float(v.w)};
    }
    __device__ static uint4 put(const cpx<float> (&c)[N])
    {
        return make_uint4(__float_as_uint(c[0].re), __float_as_uint(c[0].im), __float_as_uint(c[1].re),
                          __float_as_uint(c[1].im));
    }
};
template <>
struct VecIO<GRG_FP64> {
    static constexpr int N = 1;
    typedef double R;
    __device__ static void get(const uint4 &v, cpx<double> (&c)[N])
    {
        c[0] = {__hiloint2double((int)v.y, (int)v.x), __hiloint2double((int)v.w, (int)v.z)};
    }
    __device__ static uint4 put(const cpx<double> (&c)[N])
    {
        const long long a = __double_as_longlong(c[0].re), b = __double_as_longlong(c[0].im);
        return make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
    }
};

// Loads and stores past L2, for a stream that nothing near reads again.
typedef uint32_t vec16_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load(const uint4 *p)
{
    const vec16_u4 v = __builtin_nontemporal_load((const vec16_u4 *)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stream_store(uint4 *p, uint4 v)
{
    __builtin_nontemporal_store((vec16_u4){v.x, v.y, v.z, v.w}, (vec16_u4 *)p);
}

// Vectors per lane and stream of a wavefront's unit of one (64-site tile, RHS):
// all of it in BF16, a half in FP32, a quarter in FP64.
constexpr int kUnitVecs = 3;

}  // namespace grg
