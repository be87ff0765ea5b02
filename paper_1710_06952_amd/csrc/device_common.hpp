// Device helpers shared by the HIP kernels: 128-bit vector types, the
// counter-based generator, the synthetic normal gradient, bf16 rounding and
// wavefront reductions (64 lanes on CDNA).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"

namespace adpsgd_impl {

typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint16_t v4h __attribute__((ext_vector_type(4)));

// A pointer out of a table, known to the compiler to point to global memory.  Else it takes loads that may be from LDS as well
// (flat_load): these pass through LDS too, hold up its other accesses, and every wait after one is for all requests.
template <typename T>
using Global = const __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ Global<T> in_global(const void* p) {
    return (Global<T>)p;
}

template <bool STREAM>
__device__ __forceinline__ v4f load4(const float* p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    return *reinterpret_cast<const v4f*>(p);
}
template <bool STREAM>
__device__ __forceinline__ v4f load4(Global<float> p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<Global<v4f>>(p));
    return *reinterpret_cast<Global<v4f>>(p);
}
template <bool STREAM>
__device__ __forceinline__ void store4(float* p, v4f v) {
    if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(p));
    else *reinterpret_cast<v4f*>(p) = v;
}

// What binds the kernels that draw gradients in registers is the issue of vector instructions: a quad of variates with its
// generator (Philox, Box-Muller) takes a SIMD 326 cycles per wavefront.  Measured, time per
// instruction and SIMD with eight wavefronts: 1.05 ns for additions, products and FMAs in fp32, for 32-bit integer additions,
// AND / OR / XOR, three-input bit operations and right shifts; 1.83 ns for the same with an operand in a scalar register, for
// left shifts, bit fields, conversions, comparisons, selects and 32-bit products; 3.45 ns for logarithm and root.  So what
// every lane shares (keys, constants) is held in vector registers, and selects are bit operations.
__device__ __forceinline__ uint32_t in_vector(uint32_t s) {
    uint32_t v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(s));
    return v;
}
__device__ __forceinline__ float in_vector(float s) { return __uint_as_float(in_vector(__float_as_uint(s))); }
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }
// bits of a where mask is set, of b elsewhere
__device__ __forceinline__ float pick(uint32_t mask, float a, float b) {
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(mask, __float_as_uint(a), __float_as_uint(b), 0xCA));
}
// a with its sign flipped where the top bit of by is set
__device__ __forceinline__ float flip(float a, uint32_t by, uint32_t top) {
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(a), by, top, 0x78));
}

// The keys of kRounds rounds of Philox4x32 starting with (k0, k1): uniform over a workgroup, in vector registers where a
// wavefront draws often (kVector), else in scalar ones.
template <int kRounds>
struct PhiloxKeys {
    uint32_t k[2 * kRounds];
};
template <int kRounds, bool kVector = false>
__device__ __forceinline__ PhiloxKeys<kRounds> philox_keys(uint32_t k0, uint32_t k1) {
    PhiloxKeys<kRounds> keys;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        keys.k[2 * r] = kVector ? in_vector(k0 + r * kPhiloxW0) : k0 + r * kPhiloxW0;
        keys.k[2 * r + 1] = kVector ? in_vector(k1 + r * kPhiloxW1) : k1 + r * kPhiloxW1;
    }
    return keys;
}
// Philox4x32 (Salmon et al., SC'11), kRounds rounds.
template <int kRounds>
__device__ __forceinline__ v4u philox4x32_rounds(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, const PhiloxKeys<kRounds>& keys) {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t pa = static_cast<uint64_t>(kPhiloxM0) * c0;
        const uint64_t pb = static_cast<uint64_t>(kPhiloxM1) * c2;
        const uint32_t n0 = xor3(static_cast<uint32_t>(pb >> 32), c1, keys.k[2 * r]);
        const uint32_t n2 = xor3(static_cast<uint32_t>(pa >> 32), c3, keys.k[2 * r + 1]);
        c1 = static_cast<uint32_t>(pb);
        c3 = static_cast<uint32_t>(pa);
        c0 = n0;
        c2 = n2;
    }
    v4u out = {c0, c1, c2, c3};
    return out;
}

// What Box-Muller takes beside the words, the same for all lanes.
struct NormalConstants {
    SynthScale scale;
    uint32_t one, fraction, top; // bits of 1.0f, bits 22..1 of a fraction, the sign bit
};
template <bool kVector = false>
__device__ __forceinline__ NormalConstants normal_constants(SynthScale s) {
    const uint32_t one = 0x3F800000u, fraction = 0x007FFFFEu, top = 0x80000000u;
    if (!kVector) return NormalConstants{s, one, fraction, top};
    return NormalConstants{{in_vector(s.hi), in_vector(s.lo), s.refine}, in_vector(one), in_vector(fraction), in_vector(top)};
}

// Box-Muller on two 32-bit words: u1 = ((wa >> 9) + 1/2) 2^-23 in (0,1) and u2 = (wb >> 8) 2^-24 in [0,1) are exact
// in fp32; gives std r cos(2 pi u2), std r sin(2 pi u2) with r = sqrt(-2 ln u1).
// The kernels that draw gradients in registers are bound by these instructions, so nothing is computed that the
// ranges above rule out (no subnormals, infinities or large arguments):
//   u1      the 23 bits as the fraction of a number in [1, 2), less 1 - 2^-24 (exact);
//   r       std r = sqrt(-log2(u1)) std sqrt(2 ln 2), v_log_f32 and v_sqrt_f32 (which rounds all but correctly), the constant
//           in two parts (SynthScale).  Where std is a power of two (refine) the root keeps its remainder, by a Newton step on
//           v_rsq_f32, so that r is rounded once: a product by such a std is exact, and this form has the error of one;
//   angle   quarter turns: n = round(4 u2) and f = 4 u2 - n in [-1/2, 1/2), whose 22 bits become the fraction of 1.5 + f, are
//           read off the word; then polynomials in f^2 for sin(pi/2 f) / f (four terms) and cos(pi/2 f) (four terms beside the
//           1), least maximum relative error over [0, 1/4] by Remez's exchange: 3.2e-9, the leading coefficient in two parts,
//           and 6.4e-11, 7.7e-11 with the coefficients as written; swapped and signed by n.
// Against 64-bit arithmetic over 6.7e7 variates, rms error relative, most and mean:  std = 1 (any power of two) 4.77e-8, 2.1e-7 and
// 1.4e-8;  std = 0.0316 5.27e-8, 0.637 ulp, 2.4e-7 and 5e-10.  With the Newton step and a product by std 4.82e-8, 2.1e-7, 1.5e-8 and
// 5.44e-8, 2.6e-7, 1.5e-8 (other std 5.37e-8 ... 5.57e-8, now 5.27e-8);  with the plain root for all std 5.27e-8.  The step costs
// powers of two 6 % (n = 128, d = 25.6 M, 2000 events: 32.0 and 34.1 ms), other std nothing.
// Written out in single operations, so that every kernel that draws a gradient gets the same bits.
__device__ __forceinline__ float minus_log2(uint32_t wa) {
#pragma clang fp contract(off)
    return -__builtin_amdgcn_logf(__uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, wa, 9)) - 0x1.fffffep-1f);
}
__device__ __forceinline__ float radius(float t, const SynthScale& k) {
#pragma clang fp contract(off)
    const float root = __builtin_amdgcn_sqrtf(t);
    return __builtin_fmaf(root, k.hi, root * k.lo);
}
__device__ __forceinline__ float refined_radius(float t, const SynthScale& k) {
#pragma clang fp contract(off)
    const float y = __builtin_amdgcn_rsqf(t), root = t * y;
    const float rest = __builtin_fmaf(-root, root, t);             // of t; the root's is rest y / 2
    return __builtin_fmaf(root, k.hi, __builtin_fmaf(rest, y * (0.5f * k.hi), root * k.lo));
}
// r cos(2 pi u2), r sin(2 pi u2)
__device__ __forceinline__ void box_muller(float r, uint32_t wb, const NormalConstants& k, float& zc, float& zs) {
#pragma clang fp contract(off)
    const uint32_t turn = wb + 0x20000000u;             // bits 31..30: n mod 4
    const float f = __uint_as_float(__builtin_amdgcn_bitop3_b32(turn >> 7, k.fraction, k.one, 0xEA)) - 1.5f;
    const float y = f * f;
    constexpr float kS0 = 1.5707963217077767f, kS0Rest = static_cast<float>(1.5707963217077767 - static_cast<double>(kS0));
    float p = __builtin_fmaf(y, -0.004601657568828705f, 0.07968003262819402f);
    p = __builtin_fmaf(p, y, -0.6459634602154649f);
    p = __builtin_fmaf(p, y, kS0Rest);
    const float s = __builtin_fmaf(f, kS0, f * p);
    float q = __builtin_fmaf(y, 0.0009040605687702003f, -0.020860308502213997f);
    q = __builtin_fmaf(q, y, 0.25366924722875356f);
    q = __builtin_fmaf(q, y, -1.2337005435078803f);
    const float c = __builtin_fmaf(q, y, 1.0f);

    const uint32_t odd = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int32_t>(turn), 30, 1));
    zc = flip(r * pick(odd, s, c), turn + 0x40000000u, k.top);
    zs = flip(r * pick(odd, c, s), turn, k.top);
}

// The four normals of one generator output, times std.
__device__ __forceinline__ v4f synth_normals_of(v4u w, const NormalConstants& k) {
    const float t0 = minus_log2(w.x), t1 = minus_log2(w.z);
    float r0, r1;
    if (k.scale.refine) {              // uniform: the same for the launch
        r0 = refined_radius(t0, k.scale);
        r1 = refined_radius(t1, k.scale);
    } else {
        r0 = radius(t0, k.scale);
        r1 = radius(t1, k.scale);
    }
    v4f z;
    float a, b;
    box_muller(r0, w.y, k, a, b);
    z.x = a; z.y = b;
    box_muller(r1, w.w, k, a, b);
    z.z = a; z.w = b;
    return z;
}

// Elements 4q .. 4q+3 of the synthetic gradient of event k: std times a standard normal each.
__device__ __forceinline__ v4f synth_normals4(uint32_t q_lo, uint32_t q_hi, uint32_t k_lo, uint32_t k_hi,
                                              uint32_t key0, uint32_t key1, SynthScale scale) {
    return synth_normals_of(philox4x32_rounds<10>(q_lo, q_hi, k_lo, (k_hi & 0x00FFFFFFu) | kStreamGrad, philox_keys<10>(key0, key1)),
                            normal_constants(scale));
}

__device__ __forceinline__ uint16_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f), rounded = u + 0x7FFFu + ((u >> 16) & 1u);
    const bool nan = (u & 0x7FFFFFFFu) > 0x7F800000u;
    return static_cast<uint16_t>((nan ? u | 0x00400000u : rounded) >> 16);      // a select: no branch around three operations
}
__device__ __forceinline__ float bf16_to_float(uint16_t h) {
    return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// The three fp32 operations of the update keep their separate roundings: the
// product gamma*g and the subtraction must not be contracted into an FMA.
__device__ __forceinline__ void average_then_apply(float a, float b, float g, float gamma, float& new_i, float& new_j) {
#pragma clang fp contract(off)
    const float avg = (a + b) * 0.5f;
    const float step = g * gamma;
    new_j = avg;
    new_i = avg - step;
}

// The event with the experiments' optimizer (Sec. 5.2): per-worker momentum buffer v, weight decay on
// the averaged model;  u = g + wd * avg;  v <- mu * v + u;  x^i <- avg - gamma * v.  One rounding per
// operation, in this order.
__device__ __forceinline__ void average_then_apply_momentum(float a, float b, float g, float v_old, float gamma, float mu,
                                                            float wd, float& new_i, float& new_j, float& v_new) {
#pragma clang fp contract(off)
    const float avg = (a + b) * 0.5f;
    const float decay = wd * avg;
    const float u = g + decay;
    const float carried = mu * v_old;
    v_new = carried + u;
    const float step = gamma * v_new;
    new_j = avg;
    new_i = avg - step;
}

// all lanes of a wavefront have finished their LDS accesses before any of them goes on (LDS operations of one
// wavefront execute in order; this only keeps the compiler from moving accesses across)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace adpsgd_impl
