// fp32 values as bf16 pieces and their products on the matrix cores: what the shape-agnostic kernels share (k_generic.hip,
// k_generic_chain.hip).
#pragma once
#include "aif_dev.h"

namespace aif {

// what the launch rules of these kernels go by
inline int compute_units()
{
    static const int n = [] {
        int dev = 0;
        hipDeviceProp_t prop;
        return hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0
                   ? prop.multiProcessorCount : 256;
    }();
    return n;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct stored;
template <> struct stored<float> { static constexpr int P = 3; };       // pieces of a tensor of this storage type
template <> struct stored<uint16_t> { static constexpr int P = 1; };

template <int P> struct Pieces { bf16x8 p[P]; };

// x = p[0] + p[1] + p[2], each piece the rest so far rounded to bf16: exact for three pieces.  A value that is not
// finite (or rounds to infinity) makes NaN pieces: whoever multiplies them sees a NaN and takes the plain route.
// Two values at a time: the conversion takes a pair, and their rests come off the two halves of its word (value by value it is
// two conversions a pair and piece).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int P> __device__ __forceinline__ void split2(float a, float b, uint32_t (&w)[P])
{
#pragma unroll
    for (int q = 0; q < P; ++q) {
        w[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
        if (q + 1 < P) {
            a -= __uint_as_float(w[q] << 16);
            b -= __uint_as_float(w[q] & 0xFFFF0000u);
        }
    }
}
template <int P> __device__ __forceinline__ Pieces<P> split8(const float *v)
{
    uint32_t w[P][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t x[P];
        split2<P>(v[2 * j], v[2 * j + 1], x);
#pragma unroll
        for (int q = 0; q < P; ++q) w[q][j] = x[q];
    }
    Pieces<P> o;
#pragma unroll
    for (int q = 0; q < P; ++q) o.p[q] = __builtin_bit_cast(bf16x8, make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]));
    return o;
}

// 2 max(x, 0) in one instruction, NaN for a NaN and for minus infinity (a sum of pieces may overflow where the plain one does not): whatever
// is not finite comes up again in the pieces and in all that follows from them.  The weights that meet it are packed halved.
__device__ __forceinline__ float relu_twice(float x) { return x + __builtin_fabsf(x); }

// acc += a * b over the k-step's 32 terms.  The product of the leading pieces goes to `big`, the others, at most 2^-8 of
// it, to `small`: they are added to each other first, so `big` is rounded once per k-step.
template <int PA, int PB>
__device__ __forceinline__ void mfma_pieces(const Pieces<PA> &a, const Pieces<PB> &b, f32x4 &big, f32x4 &small)
{
#pragma unroll
    for (int i = PA - 1; i >= 0; --i)
#pragma unroll
        for (int j = PB - 1; j >= 0; --j)
            if (i + j > 0 && i + j <= 2) small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[i], b.p[j], small, 0, 0, 0);
    big = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[0], b.p[0], big, 0, 0, 0);
}

// eight consecutive elements (16-byte aligned for fp32 in halves of four) as fp32; elements at and past `n` are zero
template <typename T> __device__ __forceinline__ void load8(const T *p, int n, float *v);
template <> __device__ __forceinline__ void load8<float>(const float *p, int n, float *v)
{
    float4 a = make_float4(0, 0, 0, 0), b = a;
    if (n > 0) a = *(const float4 *)p;
    if (n > 4) b = *(const float4 *)(p + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
}
template <> __device__ __forceinline__ void load8<uint16_t>(const uint16_t *p, int n, float *v)
{
    uint4 a = make_uint4(0, 0, 0, 0);
    if (n > 0) a = *(const uint4 *)p;
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[2 * j] = __uint_as_float(w[j] << 16);
        v[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
    }
}
// the same as pieces: a bf16 element is one
__device__ __forceinline__ Pieces<3> load_pieces(const float *p, int n)
{
    float v[8];
    load8<float>(p, n, v);
    return split8<3>(v);
}
__device__ __forceinline__ Pieces<1> load_pieces(const uint16_t *p, int n)
{
    return {{__builtin_bit_cast(bf16x8, n > 0 ? *(const uint4 *)p : make_uint4(0, 0, 0, 0))}};
}

}  // namespace aif
