// Device-side helpers shared by the kernels of libeclip (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace eclip {

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>).  Unlike `#pragma unroll`
// it cannot be declined by the unroller's size threshold, which matters where a loop index selects an
// accumulator register: a loop left rolled there sends the whole accumulator array to scratch memory.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// n / d for n < 2^31: (2 n * mul >> 32) >> shift with mul = floor(2^(31 + shift) / d) + 1, shift = ceil(log2 d)
struct Magic {
    unsigned d, mul, shift;
};
inline Magic magic_of(unsigned d)
{
    Magic m{d, 0, 0};
    while ((1ull << m.shift) < d) ++m.shift;
    m.mul = (unsigned)((1ull << (31 + m.shift)) / d + 1);
    return m;
}
__device__ __forceinline__ unsigned div_by(unsigned n, const Magic &m) { return __umulhi(n + n, m.mul) >> m.shift; }

enum { ACT_NONE = 0, ACT_RELU = 1, ACT_RELU6 = 2, ACT_GELU = 3 };

// 16-bit storage types are carried as raw bit patterns; the tag types select the conversions.
struct bf16_t { uint16_t bits; };
struct f16_t { uint16_t bits; };

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
// float -> bfloat16, round to nearest even: gfx950 has the conversion in hardware (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
}
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// two floats -> two 16-bit values in one word (a in the low half)
__device__ __forceinline__ uint32_t f32x2_to_bf16x2_bits(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
__device__ __forceinline__ uint32_t f32x2_to_f16x2_bits(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, f16x2));
}
__device__ __forceinline__ float f16_bits_to_f32(uint32_t b)
{
    return (float)__builtin_bit_cast(_Float16, (uint16_t)b);
}
__device__ __forceinline__ uint32_t f32_to_f16_bits(float f)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)f);
}

template <typename T> struct Cvt;
template <> struct Cvt<float> {
    static constexpr int VEC = 4;                                 // elements per 16-byte access
    __device__ static __forceinline__ float load(const float *p) { return *p; }
    __device__ static __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct Cvt<bf16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ float load(const bf16_t *p) { return bf16_bits_to_f32(p->bits); }
    __device__ static __forceinline__ void store(bf16_t *p, float v) { p->bits = (uint16_t)f32_to_bf16_bits(v); }
    __device__ static __forceinline__ float from_bits(uint32_t b) { return bf16_bits_to_f32(b); }
    __device__ static __forceinline__ uint32_t to_bits(float v) { return f32_to_bf16_bits(v); }
    __device__ static __forceinline__ uint32_t pack2(float a, float b) { return f32x2_to_bf16x2_bits(a, b); }
};
template <> struct Cvt<f16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ float load(const f16_t *p) { return f16_bits_to_f32(p->bits); }
    __device__ static __forceinline__ void store(f16_t *p, float v) { p->bits = (uint16_t)f32_to_f16_bits(v); }
    __device__ static __forceinline__ float from_bits(uint32_t b) { return f16_bits_to_f32(b); }
    __device__ static __forceinline__ uint32_t to_bits(float v) { return f32_to_f16_bits(v); }
    __device__ static __forceinline__ uint32_t pack2(float a, float b) { return f32x2_to_f16x2_bits(a, b); }
};

// V consecutive elements <-> V floats.  V == Cvt<T>::VEC uses one 16-byte access, V == 4 of a 16-bit type an 8-byte
// one, V == 1 a scalar one.
template <typename T, int V> struct Pack {
    __device__ static __forceinline__ void load(const T *p, float (&v)[V])
    {
        if constexpr (V == 1) {
            v[0] = Cvt<T>::load(p);
        } else if constexpr (sizeof(T) == 4) {
            const float4 q = *reinterpret_cast<const float4 *>(p);
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else if constexpr (V == 4) {               // four 16-bit elements: one 8-byte access
            const uint2 q = *reinterpret_cast<const uint2 *>(p);
            v[0] = Cvt<T>::from_bits(q.x & 0xffffu); v[1] = Cvt<T>::from_bits(q.x >> 16);
            v[2] = Cvt<T>::from_bits(q.y & 0xffffu); v[3] = Cvt<T>::from_bits(q.y >> 16);
        } else {
            const uint4 q = *reinterpret_cast<const uint4 *>(p);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = Cvt<T>::from_bits(w[i] & 0xffffu);
                v[2 * i + 1] = Cvt<T>::from_bits(w[i] >> 16);
            }
        }
    }
    __device__ static __forceinline__ void store(T *p, const float (&v)[V])
    {
        if constexpr (V == 1) {
            Cvt<T>::store(p, v[0]);
        } else if constexpr (sizeof(T) == 4) {
            *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
        } else if constexpr (V == 4) {
            *reinterpret_cast<uint2 *>(p) = make_uint2(Cvt<T>::pack2(v[0], v[1]), Cvt<T>::pack2(v[2], v[3]));
        } else {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = Cvt<T>::pack2(v[2 * i], v[2 * i + 1]);
            *reinterpret_cast<uint4 *>(p) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
};

// GELU with the exact-erf definition, v Phi(v) = v / 2 (1 + erf(v / sqrt 2)).  The two signs share one expression,
//     v Phi(v) = max(v, 0) - a Q(a),  a = |v|,  Q(a) = Phi(-a),
// which needs no sign transfer and has no 1 - erf cancellation in the negative tail.  log2 Q is close to a parabola, so
// Q(a) = exp2(P(a)) with P of degree 8: a minimax fit over [0, 8], its weight the relative error of a Q(a) that the rational
// form of Abramowitz & Stegun 7.1.26 leaves at that a, so that the largest error grows in no part of the range.  In float32 the
// largest relative error of the negative branch is 5e-7 below 1, 3e-6 below 2, 3e-5 below 3 and 1.4e-3 below 6 (rational
// form: 7e-7, 3e-6, 5e-5, 3.6e-3), the largest absolute error 1.5e-7 (2.1e-7).  The root mean square error over N(0, 1) inputs is
// 5.1e-8 (5.3e-8); between 0.01 and 0.1 alone it is 6.9e-9 (5.5e-9), between 0.5 and 1 3.9e-8 (3.6e-8), elsewhere smaller.  Past 8 the
// result is under 5e-15 and its relative accuracy goes: P falls faster than log2 Q (at 10 the result is 0.4 of the true one, at 12 4e-5)
// until exp2 underflows at 12.5; the leading coefficient is negative, so nothing beyond comes back.
// 11 instructions, one of them quarter-rate, instead of 13 with two (the reciprocal went): 56 cycles instead of 76 for a
// wavefront's 64 values.  In a GEMM epilogue nothing else runs on the CU while the vector ALU works through the tile: BERT-large
// at batch 4 on 96 CUs (24 layers of 1536 x 1024 x 4096) 3112 -> 3059 us a request.
__device__ __forceinline__ float gelu_erf(float v)
{
    const float a = fabsf(v);
    float p = fmaf(-4.156125427e-7f, a, 7.803465712e-6f);
    p = fmaf(p, a, -2.437867252e-5f);
    p = fmaf(p, a, -5.528675629e-4f);
    p = fmaf(p, a, 7.633461454e-3f);
    p = fmaf(p, a, -5.290499573e-2f);
    p = fmaf(p, a, -4.590687787e-1f);
    p = fmaf(p, a, -1.151122950f);
    p = fmaf(p, a, -9.999996258e-1f);
    return fmaf(-__builtin_amdgcn_exp2f(p), a, fmaxf(v, 0.0f));
}

__device__ __forceinline__ float apply_act(int act, float v)
{
    switch (act) {
    case ACT_RELU:  return fmaxf(v, 0.0f);
    case ACT_RELU6: return fminf(fmaxf(v, 0.0f), 6.0f);
    case ACT_GELU:  return gelu_erf(v);
    default:        return v;
    }
}

// The same for the values of a thread's outputs, with one branch for all of them: each(f) replaces every value v by f(v).
template <typename F> __device__ __forceinline__ void activate(int act, F each)
{
    if (act == ACT_GELU) {
        each([](float v) { return gelu_erf(v); });
    } else if (act != ACT_NONE) {
        const float top = act == ACT_RELU6 ? 6.0f : __builtin_inff();
        each([=](float v) { return fminf(fmaxf(v, 0.0f), top); });
    }
}

// The same with the activation fixed at compile time.  A kernel's epilogue is unrolled over its accumulator blocks, and
// with a run-time switch every copy carries the code of all activations: the code that runs then hops over the code
// that does not, which defeats the sequential instruction prefetch (measured: a 256 x 256 tile kernel of 146 KB, 52 KB
// without the switches, lost 5.6 us per launch to instruction-cache misses at its start).  Kernels therefore branch on
// the activation once, with ECLIP_ACT_SWITCH, into epilogues that each hold one activation.
template <int ACT>
__device__ __forceinline__ float apply_act_c(float v)
{
    if constexpr (ACT == ACT_RELU) return fmaxf(v, 0.0f);
    else if constexpr (ACT == ACT_RELU6) return fminf(fmaxf(v, 0.0f), 6.0f);
    else if constexpr (ACT == ACT_GELU) return gelu_erf(v);
    else return v;
}
#define ECLIP_ACT_SWITCH(act, CALL)          \
    switch (act) {                           \
    case ACT_RELU:  CALL(ACT_RELU); break;   \
    case ACT_RELU6: CALL(ACT_RELU6); break;  \
    case ACT_GELU:  CALL(ACT_GELU); break;   \
    default:        CALL(ACT_NONE); break;   \
    }

// Sum / max over aligned groups of W lanes (W = 16, 32 or 64) of a wavefront; every lane receives the result of its own group, and every
// lane has to take part.  Within a row of 16 lanes the operands move inside the vector instruction (DPP), across rows they are
// traded by v_permlane16_swap / v_permlane32_swap: six exchanges of a few cycles each, where __shfl_xor sends each through
// the LDS crossbar (about 100 cycles, one after the other).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int W, typename F>
__device__ __forceinline__ float group_reduce(float v, F f)
{
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    v = f(v, dpp_move<0xb1>(v));             // lane ^ 1 (quad_perm 1,0,3,2)
    v = f(v, dpp_move<0x4e>(v));             // lane ^ 2 (quad_perm 2,3,0,1)
    v = f(v, dpp_move<0x141>(v));            // lane i of 8 <-> 7 - i
    v = f(v, dpp_move<0x140>(v));            // lane i of 16 <-> 15 - i
    if constexpr (W >= 32) {
        const u32x2_t s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = f(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
    if constexpr (W == 64) {
        const u32x2_t s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = f(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
    return v;
}
// The same over the four lanes that share lane & 15.
template <typename F>
__device__ __forceinline__ float rows_reduce(float v, F f)
{
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(s[0]), __uint_as_float(s[1]));
    const u32x2_t t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
__device__ __forceinline__ float rows_sum(float v) { return rows_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float rows_max(float v) { return rows_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
template <int W>
__device__ __forceinline__ float group_sum(float v)
{
    return group_reduce<W>(v, [](float a, float b) { return a + b; });
}
template <int W>
__device__ __forceinline__ float group_max(float v)
{
    return group_reduce<W>(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace eclip
