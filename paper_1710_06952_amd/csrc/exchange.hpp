// Device side of a persistent kernel whose blocks own columns (kernels_strips.hip): how the
// blocks of a launch find their places, and the words they exchange.
//
// A word is 8 bytes, the value and the sequence number of its gradient, written and read with one relaxed atomic access:
// a reader that finds the number has the value, so no fence and no second access is needed, and a word is never cleared.
// A block publishes a gradient only after it has consumed all but the last few before it, which the other blocks publish
// after they have consumed theirs: the ring is never overwritten early.  A word takes 0.36 us from block to block on one
// XCD and 0.64 us across the chip (0.9 and 1.2 us for all of 16 or 256 blocks to have the words of all).  So the blocks
// of an XCD (hardware register XCC_ID) form a group, and up to 32 strips are given to the blocks of a single XCD, of eight
// blocks launched for each.  Partial sums are added in a fixed order of the groups and blocks.
// Every block waits for all others.  A cooperative launch makes sure that the grid fits the device, not that the device is
// free: work of other streams or processes may hold compute units while the first blocks are there.  So the blocks agree
// once, before any of them touches the state (assemble): all have arrived, or the first one that has waited longer than the
// caller's limit goes alone and executes the whole call by itself while all others leave.  Once all have arrived they are
// resident and every further wait ends; it is bounded by a number of polls all the same, after which the block reports the
// launch as lost.
#pragma once

#include "device_common.hpp"
#include "strips.hpp"

namespace adpsgd_impl {
namespace {

constexpr uint32_t kSpinLimit = 1u << 21;

__device__ __forceinline__ void put_word(unsigned long long* base, uint32_t at, float v, uint32_t seq) {
    __hip_atomic_store(base + at, static_cast<unsigned long long>(seq) << 32 | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The values of N words at[0 .. N), of gradients seq[0 .. N) (0: no word, the value is 0).  All N are read again in every
// pass: a load of its own for each missing word would wait for them one after the other.
template <int N>
__device__ __forceinline__ void wait_words(const unsigned long long* base, const uint32_t (&at)[N], const uint32_t (&seq)[N], float (&v)[N],
                                           bool& given_up) {
    unsigned long long w[N];
    bool complete = given_up;
#pragma unroll
    for (int u = 0; u < N; ++u) w[u] = 0;
    for (uint32_t spins = 0; !complete && spins < kSpinLimit; ++spins) {
#pragma unroll
        for (int u = 0; u < N; ++u) w[u] = __hip_atomic_load(base + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        complete = true;
#pragma unroll
        for (int u = 0; u < N; ++u) complete &= seq[u] == 0 || static_cast<uint32_t>(w[u] >> 32) == seq[u];
    }
    given_up |= !complete;
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = seq[u] == 0 ? 0.0f : __uint_as_float(static_cast<uint32_t>(w[u]));
}
// Lanes that share a sum of n words, as a power of two.
__device__ __forceinline__ int sum_width(int n) { return n > 16 ? 5 : n > 8 ? 4 : n > 4 ? 3 : 2; }

template <int kControl>
__device__ __forceinline__ float lanes_of(float v) {       // data-parallel primitive of the vector ALUs: no trip through LDS
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kControl, 0xF, 0xF, true));
}
constexpr int kSwapOne = 0xB1, kSwapTwo = 0x4E, kMirrorEight = 0x141, kMirrorSixteen = 0x140, kRotate = 0x120;
// lower half of the pairs of rows (16 lanes) or of the wavefront: a's two halves added; upper half: b's
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over groups of 2^log_width lanes, 4 to 32, in all of them.
__device__ __forceinline__ float group_sum(float v, int log_width) {
    v += lanes_of<kSwapOne>(v);
    v += lanes_of<kSwapTwo>(v);
    if (log_width > 2) v += lanes_of<kMirrorEight>(v);
    if (log_width > 3) v += lanes_of<kMirrorSixteen>(v);
    if (log_width > 4) v = fold16(v, v);
    return v;
}
__device__ __forceinline__ float row_sum(float v) {
    v += lanes_of<kRotate + 8>(v);
    v += lanes_of<kRotate + 4>(v);
    v += lanes_of<kRotate + 2>(v);
    v += lanes_of<kRotate + 1>(v);
    return v;
}
__device__ __forceinline__ float all_sum(float v) {
    v = row_sum(v);
    v = fold16(v, v);
    return fold32(v, v);
}
// Sums of 4 or 8 values over the 64 lanes at once: lane l ends with the sum of value l / 16 or l / 8.
__device__ __forceinline__ float wave_sums(const float (&v)[4], int) {
    return row_sum(fold16(fold32(v[0], v[2]), fold32(v[1], v[3])));
}
__device__ __forceinline__ float wave_sums(const float (&v)[8], int lane) {
    const float a = fold16(fold32(v[0], v[4]), fold32(v[2], v[6])), b = fold16(fold32(v[1], v[5]), fold32(v[3], v[7]));
    const bool up = (lane & 8) != 0;
    return group_sum((up ? b : a) + lanes_of<kRotate + 8>(up ? a : b), 3);
}

// What a block learns about the others: its group and rank in it.
struct Assembly {
    int32_t strip, group, rank, group_blocks, groups;     // strip < 0: no strip, the block leaves
    bool alone;                                           // ... or executes the call by itself
};
constexpr unsigned int kAlone = 0x80000000u;
// The blocks count themselves, per XCD and in counters[8], until all are there or kAlone is set beside the count: both in
// one word, so only one of them can come first.  wait_ticks: how long they wait at most, in ticks of the constant clock, 0:
// one goes alone in any case.  Which columns form a group depends on the number of strips alone (so the order of the sums
// does); if the XCDs do not have the blocks for it, the groups are formed in the order of arrival.
__device__ __forceinline__ Assembly assemble(unsigned int* counters, int blocks, int group_size, uint64_t wait_ticks) {
    const uint64_t start = wall_clock64();
    const int xcd = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 7;        // HW_REG_XCC_ID, bits 3..0
    const int rank = static_cast<int>(__hip_atomic_fetch_add(counters + xcd, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const unsigned int before = __hip_atomic_fetch_add(counters + 8, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    const int arrival = static_cast<int>(before & ~kAlone);
    Assembly as;
    as.alone = false;
    unsigned int seen = before + 1;
    while ((seen & kAlone) == 0 && (seen != gridDim.x || wait_ticks == 0)) {
        if (wall_clock64() - start >= wait_ticks &&
            __hip_atomic_compare_exchange_strong(counters + 8, &seen, seen | kAlone, __ATOMIC_ACQ_REL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            as.alone = true;
            break;
        }
        seen = __hip_atomic_load(counters + 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (as.alone || (seen & kAlone) != 0) {
        as.strip = -1;
        return as;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");       // the counts of all blocks
    const int groups = (blocks + group_size - 1) / group_size;
    int count[kStripGroups], chosen = -1;
    bool enough = true;
#pragma unroll
    for (int x = 0; x < kStripGroups; ++x) {
        count[x] = static_cast<int>(__hip_atomic_load(counters + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (chosen < 0 && count[x] >= blocks) chosen = x;
        if (x < groups) enough &= count[x] >= min(group_size, blocks - x * group_size);
    }
    as.groups = groups;
    const bool placed = groups == 1 ? chosen >= 0 : enough;
    const int place = !placed ? arrival : groups > 1 ? (rank < group_size ? xcd * group_size + rank : blocks) : xcd == chosen ? rank : blocks;
    as.strip = place < blocks ? place : -1;
    as.group = place / group_size;
    as.rank = place % group_size;
    as.group_blocks = min(group_size, blocks - as.group * group_size);
    return as;
}

}  // namespace
}  // namespace adpsgd_impl
