// Types and small device helpers shared by the attention kernels (gfx950).
#pragma once
#include "kv_layout.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x4 mk4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return u32x4{a, b, c, d}; }
__device__ __forceinline__ u32x2 mk2(uint32_t a, uint32_t b) { return u32x2{a, b}; }

// Wave-uniform reads of data this kernel never writes (block tables, context
// lengths, the work plan, e4m3 scales): going through the constant address space
// makes them scalar loads, which are counted apart from the vector loads of K and V
// and so never force the KV pipeline to drain.
#define PKV_CONST(T_, p_) ((const T_ __attribute__((address_space(4))) *)(p_))

__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    f32x2 v = {lo, hi};
    bf16x2 b = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<uint32_t *>(&b);
}

// 4 e4m3 codes in one word -> 4 bf16 in two words (exact): gfx950's packed conversion with a
// scale of one, two codes per instruction (checked against the fp32 route on all 2^16 code pairs)
__device__ __forceinline__ u32x2 fp8x4_to_bf16x4(uint32_t w) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
    bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
    return mk2(*reinterpret_cast<uint32_t *>(&a), *reinterpret_cast<uint32_t *>(&b));
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return *reinterpret_cast<bf16x8 *>(&v); }

// max over the four 16-lane rows of a wave (lanes l, l^16, l^32, l^48), in every lane.
// v_permlane32_swap exchanges the upper half of its first operand with the lower half of
// its second, v_permlane16_swap the odd rows of the first with the even rows of the
// second; fed the same value twice, the two results hold both partners of every lane.
// No LDS traffic, so the step does not wait on the scalar-load / LDS counter.
__device__ __forceinline__ float rows_max(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// max over the two 32-lane halves of a wave (lanes l and l ^ 32), in every lane: v_permlane32_swap exchanges
// the upper half of its first operand with the lower half of its second; fed the same value twice, the two
// results hold both partners of every lane.
__device__ __forceinline__ float halves_max(float x) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// How far (in powers of two) a column's maximum may run ahead of the reference point of its
// exponentials before a softmax step moves that point and rescales the column's sums.  The reference
// point need not be the true maximum, only near it: results are the same up to rounding (probabilities
// up to 2^kRescaleSlack instead of 1, numerator and denominator alike), and the 32 multiplications of a
// rescale become rare.
constexpr float kRescaleSlack = 8.f;

}  // namespace
