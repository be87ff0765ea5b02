// Device side of the kernels that execute chains of updates (chain_rounds): the updates of a round that share rows follow each
// other in one block, which reads the rows of its columns once, keeps them in registers from update to update and writes
// them once.
#pragma once

#include "device_common.hpp"

namespace adpsgd_impl {
namespace {

typedef __amdgpu_buffer_rsrc_t Buffer;
// `bytes` bytes from p on: what lies beyond reads as zero and touches no memory
__device__ __forceinline__ Buffer buffer_of(const float* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, bytes, 0x00027000);
}
template <bool kStream>
__device__ __forceinline__ v4f buffer_load4(Buffer b, int offset) {
    const v4u w = __builtin_amdgcn_raw_buffer_load_b128(b, offset, 0, kStream ? 2 : 0);
    return v4f{__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w)};
}
// four dwords `pitch` bytes apart
template <bool kStream>
__device__ __forceinline__ v4f buffer_gather4(Buffer b, int offset, int pitch) {
    v4f v;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, offset + u * pitch, 0, kStream ? 2 : 0));
    return v;
}
template <bool kStream>
__device__ __forceinline__ void buffer_scatter4(Buffer b, int offset, int pitch, v4f v) {
#pragma unroll
    for (int u = 0; u < 4; ++u) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[u]), b, offset + u * pitch, 0, kStream ? 2 : 0);
}

// A chain, all of it by scalar loads at once: no later load waits for a part of it.
__device__ __forceinline__ UpdateChain chain_at(const UpdateChain* p) {
    typedef uint32_t v8u __attribute__((ext_vector_type(8)));
    typedef const v8u __attribute__((address_space(4))) * Constant;
    struct Words {
        v8u w[sizeof(UpdateChain) / sizeof(v8u)];
    } words;
    static_assert(sizeof(Words) == sizeof(UpdateChain), "a chain is whole vectors");
    const Constant q = (Constant) reinterpret_cast<uintptr_t>(p);
#pragma unroll
    for (size_t i = 0; i < sizeof(UpdateChain) / sizeof(v8u); ++i) words.w[i] = q[i];
    return __builtin_bit_cast(UpdateChain, words);
}

// The entries a thread holds of a chain's rows (and of their momentum buffers): kN pieces of four of kPlaces rows.
template <bool MOM, int kPlaces, int kN>
struct ChainRows {
    v4f x[kPlaces][kN], v[MOM ? kPlaces : 1][kN];

    // masks of a place, the same for the whole block, in vector registers
    struct Place {
        uint32_t is[kPlaces];
        __device__ __forceinline__ explicit Place(int place) {
#pragma unroll
            for (int q = 0; q < kPlaces; ++q) is[q] = in_vector(place == q ? 0xFFFFFFFFu : 0u);
        }
    };
    // bit operations and no selects: of these the compiler makes a select of addresses, and with it the rows leave the registers
    static __device__ __forceinline__ v4f pick4(uint32_t mask, v4f a, v4f b) { return v4f{pick(mask, a.x, b.x), pick(mask, a.y, b.y), pick(mask, a.z, b.z), pick(mask, a.w, b.w)}; }
    static __device__ __forceinline__ v4f at(const v4f (&a)[kPlaces][kN], const Place& place, int r) {
        v4f w = a[0][r];
#pragma unroll
        for (int q = 1; q < kPlaces; ++q) w = pick4(place.is[q], a[q][r], w);
        return w;
    }
    static __device__ __forceinline__ void put(v4f (&a)[kPlaces][kN], const Place& place, int r, v4f w) {
#pragma unroll
        for (int q = 0; q < kPlaces; ++q) a[q][r] = pick4(place.is[q], w, a[q][r]);
    }

    __device__ __forceinline__ void update(const UpdateOp& op, float momentum, float weight_decay, const v4f (&gr)[kN]) {
        const Place pi(op.places & 15), pj(op.places >> 4);
        const uint32_t step = in_vector(op.event >= 0 ? 0xFFFFFFFFu : 0u);
#pragma unroll
        for (int r = 0; r < kN; ++r) {
            const v4f a = at(x, pi, r), b = at(x, pj, r), g = gr[r];
            const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w}, gv[4] = {g.x, g.y, g.z, g.w};
            float ni[4], nj[4];
            if constexpr (MOM) {
                const v4f o = at(v, pi, r);
                const float vo[4] = {o.x, o.y, o.z, o.w};
                float vn[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) average_then_apply_momentum(av[c], bv[c], gv[c], vo[c], op.gamma, momentum, weight_decay, ni[c], nj[c], vn[c]);
                put(v, pi, r, pick4(step, v4f{vn[0], vn[1], vn[2], vn[3]}, o));
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) average_then_apply(av[c], bv[c], gv[c], op.gamma, ni[c], nj[c]);
            }
            const v4f to_j = {nj[0], nj[1], nj[2], nj[3]};
            put(x, pj, r, to_j);              // before x^i: without a partner (i == j) the step stands
            put(x, pi, r, pick4(step, v4f{ni[0], ni[1], ni[2], ni[3]}, to_j));
        }
    }
};

}  // namespace
}  // namespace adpsgd_impl
