// Minibatch gradients of the linear models with one pass over the minibatch rows.
//
// g = sum_m c_m a_m needs the dot products a_m . x^ of whole rows before any coefficient is known.  The three launches of
// kernels_grad_linear.hip read the rows twice for that.  Here a gradient is held by a group of blocks, one per compute unit,
// each with a strip of the columns of all its rows in registers; the blocks exchange the partial dot products and, when the
// coefficients are known, combine the rows that are still there.  A row that is done makes room for one of the block's next
// gradient of the round, and several groups work side by side.
//
// What binds is the memory while rows arrive and the exchange in between.  Three kernels, by the size of a gradient's rows
// (onepass_shape):
//   onepass_gradient_kernel   below 8 MB: a gradient at a time, nothing covers the exchange.
//   onepass_pipeline_kernel   as long as two gradients fit the registers (17 to 33 MB, onepass_pipeline_chunks), and the rows of a third
//                             are on their way to LDS meanwhile; with 6 rows a wavefront from 16 MB on.  n = 32,
//                             M = 8, d = 1 M, all 32 gradients of a synchronous iteration: 8.2 us a gradient with the kernel above (of
//                             the 16 us of two groups side by side 9.6 were the rows of both at the rate of the memory, the rest dot
//                             products, two steps of the exchange and combination), 6.7 now, of which 6.4 are its 42 MB (rows, x^, g)
//                             at 6.5 TB/s; 10 iterations 3.42 and 2.92 ms.  n = 64, M = 128, d = 65 536, logistic, 500 events: 4.40
//                             and 3.64 ms.
//   onepass_staged_kernel     to 100 MB: one gradient in registers, up to half of the next one's rows on their way to LDS.  n = 40,
//                             M = 128, d = 131 073, 200 events 4.02 and 3.42 ms; n = 12, M = 64, d = 327 681 4.95 and 4.40.
// Not taken: every block adds all sums by itself (M = 8: 372 us an iteration where two steps took 340, 656 words polled by every
// block); groups that start after each other or wait for each other's rows (340 ... 400 us: what the exchanges gain, the slower
// loads of half the compute units lose); two blocks with half the rows on a compute unit (376 us: polls stand behind the other
// block's rows); in the pipeline rows requested in two halves instead of four quarters (a wavefront waits where it requests more than
// the compute unit has room for: the logistic call 4.01 ms), sums or coefficients asked for half a phase earlier, later or twice (4.28,
// 3.79, 4.00 ms: an answer that is not there costs the time of the rows requested meanwhile).
//
// The exchange has two steps, both in words of exchange.hpp (value and sequence number in one relaxed 8-byte access, never
// cleared: a number is used once): every block publishes its partial sums, one block (sample mod strips) adds those of a
// sample, in the order of the strips, and publishes its coefficient.  A block writes the words of its next gradient only after
// it has the words of all samples of this one, which need all sums of this one, so nothing is overwritten early.  Among the
// samples is the point itself where losses are wanted (|x^|^2 of logistic regression): its word is awaited for that reason alone.
//
// The launch is not cooperative: nothing makes sure that all blocks of a group are resident, while other work of the device
// (another handle's call in one launch, say) holds compute units.  A block that waits longer than a limit leaves the exchange and
// the group's gradients are executed in shares that need no more blocks than there are (take_tickets): the blocks that are there
// claim the dot products of a strip, the coefficients, the combination of a strip one after the other, in an order in which a
// share waits for earlier ones only, and these belong to blocks that run.  The sums are formed in the same order, so a gradient
// has the same bits whichever way it goes.  A block that comes later finds out by waiting itself: to ask at the start whether the
// others have left holds up the first rows (n = 23, d = 67 471, M = 10, 392 events 911 us, 895 without), to ask while it waits
// lengthens the loop that waits (902; n = 32, M = 8, d = 1 M, synchronous, 10 iterations 3373, 3353 without).
#include <algorithm>
#include <iterator>
#include <utility>

#include "chains.hpp"
#include "device_common.hpp"
#include "exchange.hpp"
#include "onepass.hpp"

namespace adpsgd_impl {
namespace {

struct OnePassParams {
    OnePassArgs a;
    int64_t n_vec;
    int32_t samples;             // onepass_samples
    int32_t pitch;               // words of a group (GroupWords)
    int32_t log_groups;          // of row_groups, a power of two
};

// Buffers (chains.hpp) check every word, also of a 128-bit load: what lies beyond d in a padded row and rows beyond M need no masks.
__device__ __forceinline__ float dot4(v4f a, v4f b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
template <typename T>
__device__ __forceinline__ v4f zero_beyond(v4f v, T e, T d, T step = 1) {
    if (e >= d) v.x = 0.0f;
    if (e + step >= d) v.y = 0.0f;
    if (e + 2 * step >= d) v.z = 0.0f;
    if (e + 3 * step >= d) v.w = 0.0f;
    return v;
}
// The words at[u] (none where at[u] < 0) are asked for and, when they are needed, looked at: until all that the wavefront wants are
// of gradient seq, or the time is up (false).
template <int N>
__device__ __forceinline__ void ask_words(const unsigned long long* base, const int (&at)[N], unsigned long long (&w)[N]) {
#pragma unroll
    for (int u = 0; u < N; ++u) w[u] = at[u] >= 0 ? __hip_atomic_load(base + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
}
template <int N>
__device__ __forceinline__ bool answer_words(const unsigned long long* base, const int (&at)[N], uint32_t seq, uint64_t ticks, unsigned long long (&w)[N], float (&v)[N]) {
    auto missing = [&]() {
        bool complete = true;
#pragma unroll
        for (int u = 0; u < N; ++u) complete &= at[u] < 0 || static_cast<uint32_t>(w[u] >> 32) == seq;
        return !__all(complete);
    };
    if (missing()) {                // apart from the loop, in which the wait is for all that the wavefront has requested
        const uint64_t until = wall_clock64() + ticks;
        do {
            if (wall_clock64() >= until) return false;
            ask_words(base, at, w);
        } while (missing());
    }
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = __uint_as_float(static_cast<uint32_t>(w[u]));
    return true;
}
// ... asked for and awaited at once
template <int N>
__device__ __forceinline__ bool take_words(const unsigned long long* base, const int (&at)[N], uint32_t seq, uint64_t until, float (&v)[N]) {
    unsigned long long w[N];
    for (;;) {
        ask_words(base, at, w);
        bool complete = true;
#pragma unroll
        for (int u = 0; u < N; ++u) complete &= at[u] < 0 || static_cast<uint32_t>(w[u] >> 32) == seq;
        if (__all(complete)) break;
        if (wall_clock64() >= until) return false;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = __uint_as_float(static_cast<uint32_t>(w[u]));
    return true;
}

// A number that the compiler takes for a new one: what follows from it is not kept from turn to turn, for which the kernels that
// stage rows have no registers.  The one for small gradients has them, and keeps it: with the thread as a new number in every use and
// strips of any width its calls of 2 to 3 MB a gradient took 1 to 2.5 % longer (n = 16, d = 8000, M = 88, 200 events 557 us, 546 with it).
__device__ __forceinline__ int anew(int v) {
    asm volatile("" : "+s"(v));
    return v;
}
template <bool kAnew = true>
__device__ __forceinline__ int my_thread() {
    int v = threadIdx.x;
    if (kAnew) asm volatile("" : "+v"(v));
    return v;
}
// Coefficient (times gscale) and loss of a sample from its dot product with the point.
__device__ __forceinline__ v2f coefficient(const OnePassArgs& a, float dot, float target) {
    float coef, loss = 0.0f;
    if (a.model == ADPSGD_MODEL_LSQ) {
        const float r = dot - target;               // a.x - b
        loss = 0.5f * r * r;
        coef = r;
    } else {
        const float s = -target * dot;              // F = log(1 + e^s) + reg
        if (a.loss) loss = s > 0.0f ? s + log1pf(expf(-s)) : log1pf(expf(s));
        coef = -target / (1.0f + expf(-s));         // -y sigmoid(s)
    }
    return v2f{coef * a.gscale, loss};
}

constexpr uint64_t kShareTicks = 10ull * 1000 * 1000 * 100;      // of the constant clock: how long a share waits for one that is running

template <int kRows, int kChunks, bool kStage>
struct OnePassShared {
    // chunks whose partial gradients are in LDS at a time
    static constexpr int kReduce = !kStage ? (kChunks < 4 ? kChunks : 4) : kChunks == 4 ? 2 : kChunks < 3 ? kChunks : 3;
    static constexpr int kStaged = !kStage ? 0 : kRows * kChunks <= 16 ? kRows : 16 / kChunks;       // last rows of a wavefront's
    __attribute__((aligned(16))) v4f stage[kStage ? kOnePassWaves : 1][kStage ? kStaged : 1][kStage ? kChunks : 1][kStage ? 64 : 1];       // of the next gradient
    __attribute__((aligned(16))) v4f red[kOnePassWaves][kReduce][64];
    float part[kOnePassWaves][kOnePassMaxM + 1];            // [column group][sample]
    // by row group and row: entry place_of(m) is sample m's; beyond M: coefficient 0, row 0 (of which nothing is read)
    __attribute__((aligned(16))) float coef[kOnePassMaxM];
    int32_t idx[3][kOnePassMaxM];
    float loss[kOnePassMaxM + 1];
    uint32_t ticket;
    int late[2];                            // the wait of a wavefront was in vain; the pipeline has one a turn (late_seen), the others the first
    int lost;
};

// Columns of a wavefront: whole vectors where rows are not staged.
template <int kChunks, bool kStage>
__device__ __forceinline__ int wave_columns(const OnePassParams& p) { return kStage ? p.a.shape.wave_cols : 256 * kChunks; }
// What a thread has of a strip: the same in every block that works on it.
struct StripPlace {
    int64_t col0;                                // of its wavefront
    int bytes, offset, row_group, col_group;     // in bounds from col0 on; of its lane
    int rows;                                    // of its row group
    __device__ __forceinline__ StripPlace(const OnePassParams& p, int strip, int columns) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
        row_group = wave & (p.a.shape.row_groups - 1);
        col_group = wave >> p.log_groups;
        rows = (p.a.M - row_group + p.a.shape.row_groups - 1) >> p.log_groups;
        col0 = (static_cast<int64_t>(strip) * (kOnePassWaves >> p.log_groups) + col_group) * columns;
        const int64_t left = 4 * (p.a.d - col0);
        bytes = left <= 0 ? 0 : left < 4 * columns ? static_cast<int>(left) : 4 * columns;
        offset = 16 * lane;
    }
};
template <int kChunks>
__device__ __forceinline__ void request_point(const OnePassArgs& a, const GradOp& op, const StripPlace& at, int bytes, v4f (&x)[kChunks]) {
    const Buffer b = buffer_of(a.X + static_cast<int64_t>(op.worker) * a.ld + at.col0, bytes);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) x[c] = buffer_load4<false>(b, at.offset + 1024 * c);
}
// wait-free variant: x^ = row - gamma_k' g_k'
template <int kChunks>
__device__ __forceinline__ void compensate_point(const OnePassArgs& a, const GradOp& op, const StripPlace& at, v4f (&x)[kChunks]) {
#pragma clang fp contract(off)
    const Buffer b = buffer_of(a.slots + static_cast<int64_t>(op.comp_slot) * a.ld + at.col0, at.bytes);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
        const v4f step = buffer_load4<false>(b, at.offset + 1024 * c) * op.comp_gamma;
        x[c] = x[c] - step;
    }
}
// The partial sums go through LDS by instructions that the compiler does not know: before any access to LDS that it knows, it
// waits for all rows that are on their way there.  put_part: done when the wavefront has waited for lds_done().
__device__ __forceinline__ uint32_t lds_address(const float* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const float*)p));
}
template <bool kAside>
__device__ __forceinline__ void put_part(float* to, float v) {
    if (!kAside) *to = v;
    else asm volatile("ds_write_b32 %0, %1" : : "v"(lds_address(to)), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }
// A barrier after which accesses to LDS are in order, without a wait for what is on its way there.
__device__ __forceinline__ void block_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }
template <int N>
__device__ __forceinline__ void all_but() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }        // the last N requests have arrived
__device__ __forceinline__ void get_parts(const float* from, float (&v)[kOnePassWaves]) {
    static_assert(kOnePassWaves == 8 && kOnePassMaxM == 128, "the offsets below are those of part[0 .. 7][m]");
    asm volatile(
        "ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:516\n\tds_read_b32 %2, %8 offset:1032\n\tds_read_b32 %3, %8 offset:1548\n\t"
        "ds_read_b32 %4, %8 offset:2064\n\tds_read_b32 %5, %8 offset:2580\n\tds_read_b32 %6, %8 offset:3096\n\tds_read_b32 %7, %8 offset:3612\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
        : "v"(lds_address(from))
        : "memory");
}
// An operation by scalar loads: a vector load would stand behind the rows.
__device__ __forceinline__ GradOp op_at(const GradOp* p) {
    typedef uint32_t v2u __attribute__((ext_vector_type(2)));
    typedef const v2u __attribute__((address_space(4))) * Constant;
    struct Words {
        v2u w[sizeof(GradOp) / sizeof(v2u)];
    } words;
    static_assert(sizeof(Words) == sizeof(GradOp), "an operation is whole pairs of words");
    const Constant q = (Constant) reinterpret_cast<uintptr_t>(p);
#pragma unroll
    for (size_t i = 0; i < sizeof(GradOp) / sizeof(v2u); ++i) words.w[i] = q[i];
    return __builtin_bit_cast(GradOp, words);
}
// Both of the lines that an operation may lie in, to the scalar cache; its event.  held: keeps the load where it was written.
struct Touched {
    int32_t event, ld;
    __device__ __forceinline__ explicit Touched(const GradOp* p) {
        const GradOp op = op_at(p);
        event = op.event;
        ld = static_cast<int32_t>(op.ld);
    }
    __device__ __forceinline__ void held() { asm volatile("" : "+s"(event), "+s"(ld)); }
};
__device__ __forceinline__ float target_at(const GradOp& op, int32_t row) { return in_global<float>(op.targets)[row]; }
// Where coefficient and index of sample m are; beyond the last row of the groups none is.
template <int kRows>
__device__ __forceinline__ int place_of(const OnePassParams& p, int m) { return (m & (p.a.shape.row_groups - 1)) * kRows + (m >> p.log_groups); }
template <int kRows>
__device__ __forceinline__ void put_index(const OnePassParams& p, int32_t* to, int32_t index) {
    const int m = my_thread();
    if (m < kRows << p.log_groups) to[place_of<kRows>(p, m)] = index;
}
__device__ __forceinline__ int32_t index_of(const OnePassArgs& a, const GradOp& op) {
    const int m = my_thread();
    return m < a.M ? a.batch_idx[static_cast<int64_t>(op.event) * a.M + m] : 0;
}
// The indices of a wavefront's rows, row r's in lane r.
template <int kRows>
__device__ __forceinline__ int32_t row_indices(const StripPlace& at, const int32_t* idx) {
    return idx[at.row_group * kRows + min(static_cast<int>(my_thread() & 63), kRows - 1)];
}
// Where the wavefront's rows begin, row r's in lane r; indices: row_indices.
__device__ __forceinline__ uint64_t row_places(const GradOp& op, const StripPlace& at, int32_t indices) {
    return reinterpret_cast<uintptr_t>(op.features) + 4 * (static_cast<int64_t>(indices) * op.ld + at.col0);
}
// Row r of the row group; rows: of the group, at.rows.
__device__ __forceinline__ Buffer row_buffer(uint64_t places, int r, int rows, int bytes) {
    const uint64_t from = static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(places >> 32), r))) << 32 |
                          static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<uint32_t>(places), r));
    return buffer_of(reinterpret_cast<const float*>(from), r < rows ? bytes : 0);
}
template <int kChunks>
__device__ __forceinline__ void request_sample(const OnePassArgs& a, const GradOp& op, const StripPlace& at, const int32_t* index, int r, int bytes, v4f (&row)[kChunks]) {
    const int m = at.row_group + a.shape.row_groups * r;
    const int64_t from = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(index[m])) * op.ld + at.col0;
    const Buffer b = buffer_of(static_cast<const float*>(op.features) + from, m < a.M ? bytes : 0);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) row[c] = buffer_load4<true>(b, at.offset + 1024 * c);
}
template <int kChunks>
__device__ __forceinline__ void request_row(Buffer b, const StripPlace& at, v4f (&row)[kChunks]) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c) row[c] = buffer_load4<true>(b, at.offset + 1024 * c);
}
// ... to LDS, past the registers
template <int kChunks>
__device__ __forceinline__ void stage_row(Buffer b, const StripPlace& at, v4f (*to)[64]) {
#pragma unroll
    for (int c = 0; c < kChunks; ++c)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)&to[c][0], 16, at.offset + 1024 * c, 0, 0, 2);
}
// What requests to LDS do not write (columns and rows that the wavefront does not have) is zero from the start.
template <int kRows, int kChunks, int kStaged>
__device__ __forceinline__ void clear_stage(const StripPlace& at, v4f (*stage)[kChunks][64]) {
    if (at.bytes == 1024 * kChunks && at.rows >= kRows) return;            // the same for the wavefront
    const int lane = my_thread() & 63;
#pragma unroll
    for (int r = 0; r < kStaged; ++r)
#pragma unroll
        for (int c = 0; c < kChunks; ++c) stage[r][c][lane] = v4f{0, 0, 0, 0};
    lds_done();
}
// ... from there; the last vector may be beyond d in part.
template <int kChunks>
__device__ __forceinline__ void take_row(const StripPlace& at, int bytes, const v4f (*from)[64], v4f (&row)[kChunks]) {
    const int lane = my_thread() & 63;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) row[c] = from[c][lane];
    if ((bytes & 15) == 0) return;                     // the same for the wavefront
#pragma unroll
    for (int c = 0; c < kChunks; ++c) row[c] = zero_beyond(row[c], at.offset + 1024 * c, bytes, 4);
}
template <int kChunks>
__device__ __forceinline__ float row_dot(const v4f (&row)[kChunks], const v4f (&x)[kChunks]) {
    float v = 0.0f;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) v += dot4(row[c], x[c]);
    return v;
}
// Partial dot products of rows r0, r0 + 1, ... of the wavefront's, summed over its lanes, to part[column group][sample].
template <int kRows, bool kAside, int kBatch>
__device__ __forceinline__ void put_parts(const OnePassArgs& a, const StripPlace& at, int r0, const float (&v)[kBatch], float (*part)[kOnePassMaxM + 1]) {
    const int lane = my_thread<kAside>() & 63;
    const float z = wave_sums(v, lane);
    const int r = r0 + lane / (64 / kBatch), m = at.row_group + a.shape.row_groups * r;
    if (lane % (64 / kBatch) == 0 && r < kRows && m < a.M) put_part<kAside>(&part[at.col_group][m], z);
}
template <bool kAside, int kChunks>
__device__ __forceinline__ void put_square(const OnePassParams& p, const StripPlace& at, const v4f (&x)[kChunks], float (*part)[kOnePassMaxM + 1]) {
    if (p.samples <= p.a.M || at.row_group != 0) return;
    const float z = all_sum(row_dot(x, x));
    if ((my_thread<kAside>() & 63) == 0) put_part<kAside>(&part[at.col_group][p.a.M], z);
}
// A sample's sum over the column groups of a strip.
template <bool kAside>
__device__ __forceinline__ float strip_sum(const OnePassParams& p, const float (*part)[kOnePassMaxM + 1], int m) {
    if (!kAside) {
        float z = part[0][m];
        for (int g = 1; g < kOnePassWaves >> p.log_groups; ++g) z += part[g][m];
        return z;
    }
    float v[kOnePassWaves];
    get_parts(&part[0][m], v);
    float z = v[0];
#pragma unroll
    for (int g = 1; g < kOnePassWaves; ++g)
        if (g < kOnePassWaves / p.a.shape.row_groups) z += v[g];
    return z;
}
// Sums over the strips of samples m, m + step, ... below samples, kN at most, by a wavefront; false when the time is up.
constexpr int kLines = kOnePassMaxStrips / 64;
template <bool kAnew, int kN>
__device__ __forceinline__ void sums_at(int m, int step, int samples, int S, int (&at)[kN * kLines]) {
    const int lane = my_thread<kAnew>() & 63;
#pragma unroll
    for (int i = 0; i < kN; ++i)
#pragma unroll
        for (int u = 0; u < kLines; ++u) at[i * kLines + u] = m + i * step < samples && lane + 64 * u < S ? (m + i * step) * S + lane + 64 * u : -1;
}
template <int kN>
__device__ __forceinline__ void add_sums(const float (&v)[kN * kLines], float (&dot)[kN]) {
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        dot[i] = 0.0f;
#pragma unroll
        for (int u = 0; u < kLines; ++u) dot[i] += v[i * kLines + u];
        dot[i] = all_sum(dot[i]);
    }
}
template <bool kAnew, int kN>
__device__ __forceinline__ bool take_sums(const unsigned long long* sums, int m, int step, int samples, int S, uint32_t seq, uint64_t until, float (&dot)[kN]) {
    int at[kN * kLines];
    float v[kN * kLines];
    sums_at<kAnew, kN>(m, step, samples, S, at);
    const bool there = take_words(sums, at, seq, until, v);
    add_sums<kN>(v, dot);
    return there;
}
// The same for one sample in two steps.  Lanes without a word look at the one of the last lane.
__device__ __forceinline__ void ask_sums(const unsigned long long* sums, int m, int S, unsigned long long (&w)[kLines]) {
    const int lane = my_thread() & 63;
#pragma unroll
    for (int u = 0; u < kLines; ++u) w[u] = __hip_atomic_load(sums + m * S + min(lane + 64 * u, S - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool answer_sums(const unsigned long long* sums, int m, int S, uint32_t seq, uint64_t ticks, unsigned long long (&w)[kLines], float& dot) {
    auto missing = [&]() {
        bool complete = true;
#pragma unroll
        for (int u = 0; u < kLines; ++u) complete &= static_cast<uint32_t>(w[u] >> 32) == seq;
        return !__all(complete);
    };
    if (missing()) {
        const uint64_t until = wall_clock64() + ticks;
        do {
            if (wall_clock64() >= until) return false;
            ask_sums(sums, m, S, w);
        } while (missing());
    }
    const int lane = my_thread() & 63;
    float v[kLines];
#pragma unroll
    for (int u = 0; u < kLines; ++u) v[u] = lane + 64 * u < S ? __uint_as_float(static_cast<uint32_t>(w[u])) : 0.0f;
    static_assert(kLines == 4, "");
    dot = all_sum(((v[0] + v[1]) + v[2]) + v[3]);
    return true;
}
__device__ __forceinline__ v2f finish_sample(const OnePassArgs& a, int m, float dot, float target) {
    return m < a.M ? coefficient(a, dot, target) : v2f{0.0f, 0.5f * a.lambda * static_cast<float>(a.M) * dot};
}
// The minibatch loss from those of its samples, by a wavefront.
template <bool kAnew>
__device__ __forceinline__ void put_loss(const OnePassParams& p, const GradOp& op, const float* loss) {
    const int lane = my_thread<kAnew>() & 63;
    float sum = 0.0f;
    for (int m = lane; m < p.samples; m += 64) sum += loss[m];
    sum = all_sum(sum);
    if (lane == 0) p.a.loss[op.event] = sum * p.a.gscale;
}
__device__ __forceinline__ float point_weight(const OnePassArgs& a, const StripPlace& at) {
    return a.model == ADPSGD_MODEL_LOGREG && at.row_group == 0 ? a.lambda * a.gscale * static_cast<float>(a.M) : 0.0f;
}
// The gradient of a strip from what the row groups have of it.  Ends with a barrier before the next use of `red` only if the
// caller has one.
template <int kRows, int kChunks, bool kStage>
__device__ __forceinline__ void put_gradient(const OnePassParams& p, const GradOp& op, const StripPlace& at, int strip, const v4f (&acc)[kChunks], OnePassShared<kRows, kChunks, kStage>& s) {
    constexpr int kReduce = OnePassShared<kRows, kChunks, kStage>::kReduce;
    const int tid = my_thread<kStage>(), lane = tid & 63, wave = tid >> 6, row_groups = p.a.shape.row_groups, col_groups = kOnePassWaves / row_groups;
    float* const g = p.a.slots + static_cast<int64_t>(op.slot) * p.a.ld;
    if (row_groups == 1) {
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t e = at.col0 + 256 * c + 4 * lane;
            if (!kStage) {                               // whole vectors: the strip ends where its last one does
                if (e < 4 * p.n_vec) *reinterpret_cast<v4f*>(g + e) = zero_beyond(acc[c], e, p.a.d);
            } else if (16 * lane + 1024 * c + 16 <= at.bytes) *reinterpret_cast<v4f*>(g + e) = acc[c];
            else if (16 * lane + 1024 * c < at.bytes) *reinterpret_cast<v4f*>(g + e) = zero_beyond(acc[c], e, p.a.d);
        }
        return;
    }
    const int columns = wave_columns<kChunks, kStage>(p);
    const int64_t tile0 = static_cast<int64_t>(strip) * (col_groups * columns);       // the sums of the row groups through LDS
#pragma unroll
    for (int c0 = 0; c0 < kChunks; c0 += kReduce) {
        if (c0 > 0) {
            if (kStage) block_barrier();
            else __syncthreads();
        }
#pragma unroll
        for (int c = 0; c < kReduce; ++c)
            if (c0 + c < kChunks) s.red[wave][c][lane] = acc[c0 + c < kChunks ? c0 + c : 0];
        if (kStage) block_barrier();
        else __syncthreads();
        for (int u = tid; u < col_groups * kReduce * 64; u += kOnePassThreads) {
            const int l = u & 63, c = (u >> 6) % kReduce, cg = (u >> 6) / kReduce;
            const int within = (c0 + c) * 256 + 4 * l;
            const int64_t e = tile0 + cg * columns + within;
            if (c0 + c >= kChunks || within >= columns || e >= 4 * p.n_vec) continue;
            v4f sum = s.red[cg * row_groups][c][l];
            for (int w = 1; w < row_groups; ++w) sum += s.red[cg * row_groups + w][c][l];
            *reinterpret_cast<v4f*>(g + e) = zero_beyond(sum, e, p.a.d);
        }
    }
}

// Words of a group: of the exchange, of `ring` gradients, [samples][strips] sums, [samples] coefficients, [samples] losses; of the
// shares, apart from these, [samples][strips] sums, [samples] coefficients and two counts (number of the launch, count).
struct GroupWords {
    unsigned long long *sums, *coefs, *losses, *share_sums, *share_coefs, *tickets, *taken;
    __device__ __forceinline__ GroupWords(const OnePassParams& p, int group) {
        const int S = p.a.shape.strips, ring = p.a.shape.ring();
        sums = p.a.words + static_cast<int64_t>(group) * p.pitch;
        coefs = sums + ring * p.samples * S;
        losses = coefs + ring * p.samples;
        share_sums = losses + ring * p.samples;
        share_coefs = share_sums + p.samples * S;
        tickets = share_coefs + p.samples;
        taken = tickets + 1;
    }
};
// Counts of a launch begin at 0: every block sets them up before it counts (with one exchange; a loop of exchanges for every
// count took 128 blocks 0.1 ms).
__device__ __forceinline__ void begin_count(unsigned long long* word, uint32_t launch) {
    unsigned long long seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (static_cast<uint32_t>(seen >> 32) != launch &&
           !__hip_atomic_compare_exchange_strong(word, &seen, static_cast<unsigned long long>(launch) << 32, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    }
}
__device__ __forceinline__ uint32_t count_up(unsigned long long* word) {       // the count before
    return static_cast<uint32_t>(__hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// The gradients of a group by the blocks of it that are there, all from the first one on: shares, claimed in this order:
//   gradient after gradient: the dot products of every strip; the coefficients; the combination of every strip.
// A share waits for shares before it only, which are done or belong to blocks that run: dot products, before they replace the
// sums of the gradient before, for its coefficients;  coefficients, before they replace those of the gradient before, until all
// its combinations have taken them;  combinations for the coefficients.  The rows are read twice.  Blocks of the group that
// have stayed in the exchange write the same bits to the same places.  A wait is bounded all the same: the launch is then lost.
// Logistic regression, n = 32, d = 65 536, M = 128, 100 events (0.95 ms by itself) beside another handle's call in one launch
// that holds 16 (157) compute units for 5 ms: done in 4.2 (4.5) ms;  when a block that had waited in vain computed the dot
// products of whole rows by itself, for the rest of the launch, 88 (97);  three launches a round, which need no block to be
// there, 2.2 (2.5), of which the other call then took more.  All in shares from the start (limit 0) and without other work: 3.1 ms.
// A function of its own with its arguments in memory, since the kernel has no registers to spare for it.
template <int kRows, int kChunks, bool kStage>
__device__ __attribute__((noinline)) void take_tickets(const OnePassParams* params, int group, OnePassShared<kRows, kChunks, kStage>* shared) {
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4, kInFlight = kChunks == 1 ? kBatch : kChunks <= 4 ? 4 : 2;       // rows
    const OnePassParams& p = *params;
    const OnePassArgs& a = p.a;
    OnePassShared<kRows, kChunks, kStage>& s = *shared;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups, word_waves = (p.samples + 63) / 64;
    const GroupWords words(p, group);
    const uint32_t launch = a.seq0, per = 2 * S + 1, shares = static_cast<uint32_t>((a.n_ops - group + groups - 1) / groups) * per;
    if (tid < kOnePassMaxM) s.coef[tid] = 0.0f;
    if (tid == 0) {
        s.lost = 0;
        begin_count(words.taken, launch);
        begin_count(words.tickets, launch);
        __hip_atomic_fetch_add(a.late, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (;;) {
        __syncthreads();
        if (tid == 0) s.ticket = count_up(words.tickets);
        __syncthreads();
        const uint32_t ticket = __builtin_amdgcn_readfirstlane(s.ticket);
        if (ticket >= shares) return;
        const int i = static_cast<int>(ticket / per), share = static_cast<int>(ticket % per), q = group + groups * i;
        const int strip = share < S ? share : share - S - 1;
        const uint32_t seq = a.seq0 + static_cast<uint32_t>(q);
        const uint64_t until = wall_clock64() + kShareTicks;
        const GradOp op = op_at(a.ops + q);
        put_index<kRows>(p, s.idx[0], index_of(a, op));
        __syncthreads();
        bool there = true;
        const int word_at[1] = {tid < p.samples ? tid : -1};
        float word[1];
        if (share < S) {
            const StripPlace at(p, strip, wave_columns<kChunks, kStage>(p));
            v4f x[kChunks];
            request_point(a, op, at, at.bytes, x);
            if (op.comp_slot >= 0) compensate_point(a, op, at, x);
            const uint64_t places = row_places(op, at, row_indices<kRows>(at, s.idx[0]));
#pragma unroll 1
            for (int r0 = 0; r0 < kRows; r0 += kBatch) {
                float v[kBatch];
#pragma unroll
                for (int from = 0; from < kBatch; from += kInFlight) {
                    v4f row[kInFlight][kChunks];
#pragma unroll
                    for (int r = 0; r < kInFlight; ++r)
                        if (r0 + from + r < kRows) request_row(row_buffer(places, r0 + from + r, at.rows, at.bytes), at, row[r]);
#pragma unroll
                    for (int r = 0; r < kInFlight; ++r) v[from + r] = r0 + from + r < kRows ? row_dot(row[r], x) : 0.0f;
                    __builtin_amdgcn_sched_barrier(0);
                }
                put_parts<kRows, false>(a, at, r0, v, s.part);
            }
            put_square<false>(p, at, x, s.part);
            if (i > 0 && wave < word_waves) there = take_words(words.share_coefs, word_at, seq - groups, until, word);
            if (!there && lane == 0) s.lost = 1;
            __syncthreads();
            if (s.lost != 0) break;
            if (tid < p.samples) put_word(words.share_sums, tid * S + strip, strip_sum<false>(p, s.part, tid), seq);
        } else if (share == S) {
            if (i > 0 && tid == 0)
                for (;;) {
                    const unsigned long long seen = __hip_atomic_load(words.taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (static_cast<uint32_t>(seen >> 32) == launch && static_cast<uint32_t>(seen) >= static_cast<uint32_t>(S * i)) break;
                    if (wall_clock64() >= until) {
                        s.lost = 1;
                        break;
                    }
                }
            __syncthreads();
            if (s.lost != 0) break;
            constexpr int kAtOnce = 5;          // samples: all of a wavefront's for M = 32, the most in four turns
            for (int m0 = wave; there && m0 < p.samples; m0 += kAtOnce * kOnePassWaves) {
                float target[kAtOnce], dot[kAtOnce];
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const int m = m0 + u * kOnePassWaves;
                    target[u] = m < M ? target_at(op, s.idx[0][place_of<kRows>(p, m)]) : 0.0f;
                }
                there = take_sums<true>(words.share_sums, m0, kOnePassWaves, p.samples, S, seq, until, dot);
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const int m = m0 + u * kOnePassWaves;
                    const v2f r = finish_sample(a, m, dot[u], target[u]);
                    if (there && lane == 0 && m < p.samples) {
                        put_word(words.share_coefs, m, r.x, seq);
                        s.loss[m] = r.y;
                    }
                }
            }
            if (!there && lane == 0) s.lost = 1;
            __syncthreads();
            if (s.lost != 0) break;
            if (a.loss && wave == 0) put_loss<true>(p, op, s.loss);
        } else {
            const StripPlace at(p, strip, wave_columns<kChunks, kStage>(p));
            if (wave < word_waves) {
                there = take_words(words.share_coefs, word_at, seq, until, word);
                if (tid < M) s.coef[place_of<kRows>(p, tid)] = word[0];
            }
            if (!there && lane == 0) s.lost = 1;
            __syncthreads();
            if (s.lost != 0) break;
            if (tid == 0) count_up(words.taken);
            v4f acc[kChunks];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) acc[c] = v4f{0, 0, 0, 0};
            if (a.model == ADPSGD_MODEL_LOGREG && at.row_group == 0) {
                v4f x[kChunks];
                request_point(a, op, at, at.bytes, x);
                if (op.comp_slot >= 0) compensate_point(a, op, at, x);
#pragma unroll
                for (int c = 0; c < kChunks; ++c) acc[c] = x[c] * point_weight(a, at);
            }
            const uint64_t places = row_places(op, at, row_indices<kRows>(at, s.idx[0]));
#pragma unroll
            for (int r0 = 0; r0 < kRows; r0 += kInFlight) {
                v4f row[kInFlight][kChunks];
#pragma unroll
                for (int r = 0; r < kInFlight; ++r)
                    if (r0 + r < kRows) request_row(row_buffer(places, r0 + r, at.rows, at.bytes), at, row[r]);
#pragma unroll
                for (int r = 0; r < kInFlight; ++r) {
                    if (r0 + r >= kRows) continue;
                    const float coef = s.coef[at.row_group * kRows + r0 + r];
#pragma unroll
                    for (int c = 0; c < kChunks; ++c) acc[c] += row[r][c] * coef;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            put_gradient(p, op, at, strip, acc, s);
        }
    }
    if (tid == 0) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// grid: groups x strips blocks, block b strip b / groups of group b % groups (with eight groups or a multiple of them the
// blocks of a group share an XCD)
template <int kRows, int kChunks>
__global__ __launch_bounds__(kOnePassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void onepass_gradient_kernel(const OnePassParams p) {
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4;                       // dot products reduced at a time
    __shared__ OnePassShared<kRows, kChunks, false> s;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups, row_groups = a.shape.row_groups;
    const int group = blockIdx.x % groups, strip = blockIdx.x / groups;
    const bool logistic = a.model == ADPSGD_MODEL_LOGREG;
    const GroupWords words(p, group);
    const StripPlace at(p, strip, wave_columns<kChunks, false>(p));

    v4f row[kRows][kChunks], x[kChunks];
    int q = group, turn = 0;
    if (q >= a.n_ops) return;
    GradOp op = a.ops[q];
    if (tid == 0) s.late[0] = 0;
    if (tid < kOnePassMaxM) {
        s.coef[tid] = 0.0f;
        s.idx[0][tid] = tid < M ? a.batch_idx[static_cast<int64_t>(op.event) * M + tid] : 0;
    }
    __syncthreads();
    request_point(a, op, at, at.bytes, x);
#pragma unroll
    for (int r = 0; r < kRows; ++r) request_sample(a, op, at, s.idx[0], r, at.bytes, row[r]);
    for (;;) {
        const uint32_t seq = a.seq0 + static_cast<uint32_t>(q);
        const bool more = q + groups < a.n_ops;
        const GradOp next = a.ops[more ? q + groups : q];
        int32_t next_index = 0;
        if (tid < M) next_index = a.batch_idx[static_cast<int64_t>(next.event) * M + tid];
        if (op.comp_slot >= 0) compensate_point(a, op, at, x);
        // ---- partial dot products
#pragma unroll
        for (int r0 = 0; r0 < kRows; r0 += kBatch) {
            float v[kBatch];
#pragma unroll
            for (int r = 0; r < kBatch; ++r) v[r] = r0 + r < kRows ? row_dot(row[r0 + r < kRows ? r0 + r : 0], x) : 0.0f;
            put_parts<kRows, false>(a, at, r0, v, s.part);
        }
        put_square<false>(p, at, x, s.part);
        if (tid < kOnePassMaxM) s.idx[turn ^ 1][tid] = next_index;
        __syncthreads();

        // ---- the exchange
        if (tid < p.samples) put_word(words.sums, tid * S + strip, strip_sum<false>(p, s.part, tid), seq);
        const uint64_t until = wall_clock64() + a.wait_ticks;
        bool there = a.wait_ticks > 0;
        for (int m = strip + S * wave; there && m < p.samples; m += S * kOnePassWaves) {
            const float target = m < M ? target_at(op, s.idx[turn][m]) : 0.0f;
            float dot[1];
            there = take_sums<false>(words.sums, m, 0, p.samples, S, seq, until, dot);
            if (there && lane == 0) {
                const v2f r = finish_sample(a, m, dot[0], target);
                put_word(words.coefs, m, r.x, seq);
                if (a.loss) put_word(words.losses, m, r.y, seq);
            }
        }
        const int awaited = onepass_awaited(p.samples);
        if (there && wave < (awaited + 63) / 64) {
            const int word_at[1] = {tid < awaited ? tid : -1};
            float v[1];
            there = take_words(words.coefs, word_at, seq, until, v);
            if (tid < M) s.coef[tid] = v[0];
        }
        if (there && a.loss && strip == 0 && wave >= 4 && wave - 4 < (p.samples + 63) / 64) {
            const int m = tid - 256;
            const int word_at[1] = {m < p.samples ? m : -1};
            float v[1];
            there = take_words(words.losses, word_at, seq, until, v);
            if (m < p.samples) s.loss[m] = v[0];
        }
        if (!there && lane == 0) s.late[0] = 1;
        __syncthreads();
        if (s.late[0] != 0) {                         // uniform over the block
            take_tickets<kRows, kChunks, false>(static_cast<const OnePassParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()), group, &s);
            return;
        }

        // ---- g = sum_m c_m a_m (+ lambda x^); a row that is done makes room for one of the next gradient
        const int next_bytes = more ? at.bytes : 0;         // none: the requests touch no memory
        v4f acc[kChunks];
        const float regularise = point_weight(a, at);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) acc[c] = logistic && at.row_group == 0 ? x[c] * regularise : v4f{0, 0, 0, 0};
        request_point(a, next, at, next_bytes, x);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float coef = s.coef[at.row_group + row_groups * r];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                acc[c] += row[r][c] * coef;
                asm volatile("" : "+v"(acc[c]));      // here and not behind the request, which needs the row's registers
            }
            __builtin_amdgcn_sched_barrier(0);
            request_sample(a, next, at, s.idx[turn ^ 1], r, next_bytes, row[r]);
            __builtin_amdgcn_sched_barrier(0);
        }
        put_gradient(p, op, at, strip, acc, s);
        if (a.loss && strip == 0 && wave == 7) put_loss<false>(p, op, s.loss);
        if (!more) break;
        q += groups;
        op = next;
        turn ^= 1;
        __syncthreads();
    }
}

// The same for gradients that fill the registers (more than 16 vectors of four columns to a thread), of which the last rows of the
// next gradient are on their way to LDS while the blocks wait for each other, and go to the registers when this one is combined.
template <int kRows, int kChunks>
__global__ __launch_bounds__(kOnePassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void onepass_staged_kernel(const OnePassParams p) {
    constexpr bool kPointLast = kRows * kChunks > 40;                    // no registers for two points while rows are combined
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4;                       // dot products reduced at a time
    constexpr int kDirect = kRows - OnePassShared<kRows, kChunks, true>::kStaged;
    __shared__ OnePassShared<kRows, kChunks, true> s;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups;
    const int group = blockIdx.x % groups, strip = blockIdx.x / groups;
    const bool logistic = a.model == ADPSGD_MODEL_LOGREG;
    const GroupWords words(p, group);
    const StripPlace at(p, strip, wave_columns<kChunks, true>(p));

    v4f row[kRows][kChunks], x[kChunks];
    v4f(*const stage)[kChunks][64] = s.stage[wave];
    int q = group, turn = 0, turn1 = 1, turn2 = 2;                   // places of the indices: of this gradient and the two that follow
    if (q >= a.n_ops) return;
    if (tid == 0) s.late[0] = 0;
    if (tid < kOnePassMaxM) s.coef[tid] = 0.0f;
    GradOp op = op_at(a.ops + q);
    {
        Touched touched(a.ops + min(q + groups * (wave + 1), a.n_ops - 1));       // the operations of the turns to come
        const int32_t index = index_of(a, op), next_index = index_of(a, op_at(a.ops + (q + groups < a.n_ops ? q + groups : q)));
        put_index<kRows>(p, s.idx[0], index);
        put_index<kRows>(p, s.idx[1], next_index);
        __syncthreads();
        request_point(a, op, at, at.bytes, x);
        const uint64_t places = row_places(op, at, row_indices<kRows>(at, s.idx[0]));
#pragma unroll
        for (int i = 0; i < kRows; ++i) {                  // in the order of the dot products
            const int r = (i + kDirect) % kRows;
            request_row(row_buffer(places, r, at.rows, at.bytes), at, row[r]);
        }
        touched.held();
        if (q + groups < a.n_ops) clear_stage<kRows, kChunks, OnePassShared<kRows, kChunks, true>::kStaged>(at, stage);
    }
    for (;;) {
        const uint32_t seq = a.seq0 + static_cast<uint32_t>(q);
        const bool more = q + groups < a.n_ops;
        const GradOp next = op_at(a.ops + (more ? q + groups : q));
        const int32_t after_index = index_of(a, op_at(a.ops + (q + 2 * groups < a.n_ops ? q + 2 * groups : q)));
        if (op.comp_slot >= 0) compensate_point(a, op, at, x);
        const int next_bytes = more ? at.bytes : 0;         // none: the requests touch no memory
        {                                                   // (under a condition, all rows would be awaited behind it)
            const uint64_t places = row_places(next, at, row_indices<kRows>(at, s.idx[turn1]));
            const int rows = anew(at.rows);
#pragma unroll
            for (int r = kDirect; r < kRows; ++r) stage_row<kChunks>(row_buffer(places, r, rows, next_bytes), at, stage[r - kDirect]);
        }
        // ---- partial dot products, the rows that were in LDS first
#pragma unroll
        for (int i = 0; i < kRows; i += kBatch) {
            const int r0 = (kRows - 1) / kBatch * kBatch - i;
            float v[kBatch];
#pragma unroll
            for (int r = 0; r < kBatch; ++r) v[r] = r0 + r < kRows ? row_dot(row[r0 + r < kRows ? r0 + r : 0], x) : 0.0f;
            put_parts<kRows, true>(a, at, r0, v, s.part);
        }
        put_square<true>(p, at, x, s.part);
        block_barrier();

        // ---- the exchange
        if (tid < p.samples) put_word(words.sums, tid * S + strip, strip_sum<true>(p, s.part, tid), seq);
        const uint64_t until = wall_clock64() + a.wait_ticks;
        bool there = a.wait_ticks > 0;
        for (int m = strip + S * wave; there && m < p.samples; m += S * kOnePassWaves) {
            const float target = m < M ? target_at(op, s.idx[turn][place_of<kRows>(p, m)]) : 0.0f;
            float dot[1];
            there = take_sums<true>(words.sums, m, 0, p.samples, S, seq, until, dot);
            if (there && lane == 0) {
                const v2f r = finish_sample(a, m, dot[0], target);
                put_word(words.coefs, m, r.x, seq);
                if (a.loss) put_word(words.losses, m, r.y, seq);
            }
        }
        const int awaited = onepass_awaited(p.samples);
        if (there && wave < (awaited + 63) / 64) {
            const int word_at[1] = {tid < awaited ? tid : -1};
            float v[1];
            there = take_words(words.coefs, word_at, seq, until, v);
            if (tid < M) s.coef[place_of<kRows>(p, tid)] = v[0];
        }
        if (there && a.loss && strip == 0 && wave >= 4 && wave - 4 < (p.samples + 63) / 64) {
            const int m = tid - 256;
            const int word_at[1] = {m < p.samples ? m : -1};
            float v[1];
            there = take_words(words.losses, word_at, seq, until, v);
            if (m < p.samples) s.loss[m] = v[0];
        }
        if (!there && lane == 0) s.late[0] = 1;
        put_index<kRows>(p, s.idx[turn2], after_index);
        __syncthreads();
        if (s.late[0] != 0) {                         // uniform over the block
            __builtin_amdgcn_s_waitcnt(0);         // for rows on their way to LDS
            take_tickets<kRows, kChunks, true>(static_cast<const OnePassParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()), group, &s);
            return;
        }

        // ---- g = sum_m c_m a_m (+ lambda x^); a row that is done makes room for one of the next gradient
        const uint64_t places = row_places(next, at, row_indices<kRows>(at, s.idx[turn1]));
        const int rows = anew(at.rows);
        v4f acc[kChunks];
        const float regularise = point_weight(a, at);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) acc[c] = logistic && at.row_group == 0 ? x[c] * regularise : v4f{0, 0, 0, 0};
        if (!kPointLast) request_point(a, next, at, next_bytes, x);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float coef = s.coef[at.row_group * kRows + r];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                acc[c] += row[r][c] * coef;
                asm volatile("" : "+v"(acc[c]));      // here and not behind the request, which needs the row's registers
            }
            __builtin_amdgcn_sched_barrier(0);
            if (r < kDirect) request_row(row_buffer(places, r, rows, next_bytes), at, row[r]);
            else take_row(at, r < rows ? next_bytes : 0, stage[r < kDirect ? 0 : r - kDirect], row[r]);
            __builtin_amdgcn_sched_barrier(0);
        }
        put_gradient(p, op, at, strip, acc, s);
        if (kPointLast) request_point(a, next, at, next_bytes, x);
        if (a.loss && strip == 0 && wave == 7) put_loss<true>(p, op, s.loss);
        if (!more) {
            __builtin_amdgcn_s_waitcnt(0);             // nothing is on its way to LDS when the block ends
            break;
        }
        q += groups;
        op = next;
        const int done = turn;
        turn = turn1;
        turn1 = turn2;
        turn2 = done;
        lds_done();                                    // the staged rows are in registers
        __syncthreads();
    }
}

// The same for gradients that take a quarter of the registers: two of a group are on the chip at a time, and the rows of a third are
// on their way to LDS, so that the memory is kept busy while the blocks wait for each other.
//
// Turn t of a block, of its gradients 0, 1, ..., with the rows of t - 1 (whose coefficients are due) and t (whose sums are due) in
// registers and those of t + 1 on their way to LDS:
//   1  the coefficients of t - 1, asked for at the end of the turn before;
//   2  the first half of the rows of t - 1 is combined and makes room for those of t + 1;  the sums of t are asked for;  x^ and the
//      first quarter of the rows of t + 2 are requested;
//   3  the second half likewise;  the coefficients of t, where this block adds up samples, from the sums of t;  second quarter;
//   4  the gradient t - 1 is written;  third quarter;
//   5  the dot products of t + 1, published;
//   6  the coefficients of t are asked for;  last quarter.
// A compute unit returns loads in order: an answer stands behind the rows requested before the question and not behind those
// requested after it, so rows are on their way whatever a wavefront waits for.  And it takes in requests only as fast as rows arrive
// beyond some 64 KB: hence the quarters.
// Two gradients are in the exchange at a time, in words of their own (ring = 2): a block publishes sums of t + 1 when it has the
// coefficients of t - 1, which need all sums of t - 1, and coefficients of t when it has the sums of t of all blocks, which these
// publish when they have the coefficients of t - 2.
template <int kRows, int kChunks>
__global__ __launch_bounds__(kOnePassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void onepass_pipeline_kernel(const OnePassParams p) {
    constexpr int kQuarter = kRows / 4, kHalf = kRows / 2, kRest = kRows - (kRows + 3) / 4, kBatch = kRows % 8 == 0 ? 8 : 4;
    static_assert(OnePassShared<kRows, kChunks, true>::kStaged == kRows, "all rows go through LDS");
    __shared__ OnePassShared<kRows, kChunks, true> s;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups;
    const int group = blockIdx.x % groups, strip = blockIdx.x / groups;
    const int count = (a.n_ops - group + groups - 1) / groups;           // gradients of the group
    const bool logistic = a.model == ADPSGD_MODEL_LOGREG;
    const GroupWords words(p, group);
    const StripPlace at(p, strip, wave_columns<kChunks, true>(p));
    v4f(*const stage)[kChunks][64] = s.stage[wave];
    if (count <= 0) return;

    auto op_of = [&](int t) { return op_at(a.ops + group + groups * max(0, min(t, count - 1))); };
    auto index_at = [&](int t, int m) { return a.batch_idx[static_cast<int64_t>(op_of(t).event) * M + min(m, M - 1)]; };
    const int my_row = at.row_group + (min(lane, kRows - 1) << p.log_groups);
    const int adds = strip + S * ((wave + 5) & 7);       // sample that the wavefront adds up; the first on wavefront 3
    int word_at[1] = {-1};                               // coefficients on the first wavefronts, losses from the fifth on
    if (tid < 256) word_at[0] = tid < p.samples ? tid : -1;
    else if (a.loss && strip == 0) word_at[0] = tid - 256 < p.samples ? tid - 256 : -1;
    unsigned long long word[1] = {0};
    int32_t indices;                                     // of the rows of t + 2

    v4f rows_a[kRows][kChunks], rows_b[kRows][kChunks], x_a[kChunks], x_b[kChunks], x_in[kChunks];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int c = 0; c < kChunks; ++c) rows_a[r][c] = rows_b[r][c] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < kChunks; ++c) x_a[c] = x_b[c] = v4f{0, 0, 0, 0};
    clear_stage<kRows, kChunks, kRows>(at, stage);
    if (tid < 2) s.late[tid] = 0;
    if (tid < kOnePassMaxM) s.coef[tid] = 0.0f;
    auto stage_rows = [&](int t, int from, int to, uint64_t places) {
        const int bytes = t < count ? at.bytes : 0, rows = anew(at.rows);      // none: the requests touch no memory
#pragma unroll
        for (int r = 0; r < kRows; ++r)
            if (r >= from && r < to) stage_row<kChunks>(row_buffer(places, r, rows, bytes), at, stage[r]);
    };
    indices = index_at(0, my_row);
    int32_t target_row = index_at(0, adds);              // of the sample that it adds up
    request_point(a, op_of(0), at, at.bytes, x_in);
    {
        const uint64_t places = row_places(op_of(0), at, indices);
        stage_rows(0, 0, kRows, places);
    }
    indices = index_at(1, my_row);
    for (int t = 2 + wave; t < min(count, 66); t += kOnePassWaves) {        // the operations of the turns to come
        Touched touched(a.ops + group + groups * t);
        touched.held();
    }

    // turn t with the registers of t - 1 and t + 1; false: the block leaves the exchange
    auto turn = [&](int t, v4f(&row)[kRows][kChunks], v4f(&x)[kChunks]) -> bool {
        // ---- 1
        if (t >= 1) {
            bool there = a.wait_ticks > 0;
            float v[1];
            if (there) there = answer_words((tid < 256 ? words.coefs : words.losses) + ((t - 1) & 1) * p.samples, word_at, a.seq0 + static_cast<uint32_t>(group + groups * (t - 1)),
                                            a.wait_ticks, word, v);
            if (there && tid < M) s.coef[place_of<kRows>(p, tid)] = v[0];
            if (there && tid >= 256 && word_at[0] >= 0) s.loss[tid - 256] = v[0];
            if (!there && lane == 0) s.late[late_of_coefficients(t)] = 1;
        }
        block_barrier();
        if (s.late[late_seen(t)] != 0) return false;     // uniform over the block

        // ---- 2
        v4f acc[kChunks];
        const float regularise = point_weight(a, at);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            acc[c] = logistic && at.row_group == 0 ? x[c] * regularise : v4f{0, 0, 0, 0};
            x[c] = x_in[c];
        }
        const int bytes = t + 1 < count ? at.bytes : 0;
        auto combine_rows = [&](int from, int to) {
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                if (r >= from && r < to) {
                    const float coef = s.coef[at.row_group * kRows + r];
#pragma unroll
                    for (int c = 0; c < kChunks; ++c) acc[c] += row[r][c] * coef;
                }
#pragma unroll
            for (int c = 0; c < kChunks; ++c) asm volatile("" : "+v"(acc[c]));      // here and not behind the next rows, which need the registers
        };
        auto take_rows = [&](int from, int to) {
            const int rows = anew(at.rows);
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                if (r >= from && r < to) take_row(at, r < rows ? bytes : 0, stage[r], row[r]);
            lds_done();
        };
        combine_rows(0, kHalf);
        all_but<(kRows - kHalf) * kChunks>();            // the first half of t + 1 has arrived
        take_rows(0, kHalf);
        const bool sums_due = t >= 0 && t < count;
        const unsigned long long* const sums = words.sums + (t & 1) * p.samples * S;
        const uint64_t places = row_places(op_of(t + 2), at, indices);
        indices = index_at(t + 3, my_row);
        unsigned long long sum_word[kLines];
        const float target = target_at(op_of(t), target_row);
        target_row = index_at(t + 1, adds);
        const bool adding = sums_due && adds < p.samples;
        if (adding) ask_sums(sums, adds, S, sum_word);
        request_point(a, op_of(t + 2), at, t + 2 < count ? at.bytes : 0, x_in);
        stage_rows(t + 2, 0, kQuarter, places);

        // ---- 3
        combine_rows(kHalf, kRows);
        all_but<(kQuarter + 1) * kChunks>();             // the second half too
        take_rows(kHalf, kRows);
        if (adding) {
            const uint32_t seq = a.seq0 + static_cast<uint32_t>(group + groups * t);
            float dot;
            if (a.wait_ticks > 0 && answer_sums(sums, adds, S, seq, a.wait_ticks, sum_word, dot)) {
                const v2f r = finish_sample(a, adds, dot, target);
                if (lane == 0) {
                    put_word(words.coefs + (t & 1) * p.samples, adds, r.x, seq);
                    if (a.loss) put_word(words.losses + (t & 1) * p.samples, adds, r.y, seq);
                }
            } else if (lane == 0) s.late[late_of_sums(t)] = 1;
        }

        stage_rows(t + 2, kQuarter, kHalf, places);

        // ---- 4
        if (t >= 1) {
            const GradOp op = op_of(t - 1);
            put_gradient(p, op, at, strip, acc, s);
            if (a.loss && strip == 0 && wave == 7) put_loss<true>(p, op, s.loss);
        }

        stage_rows(t + 2, kHalf, kRest, places);

        // ---- 5
        if (t + 1 < count) {
            const GradOp op = op_of(t + 1);
            if (op.comp_slot >= 0) compensate_point(a, op, at, x);
#pragma unroll
            for (int r0 = 0; r0 < kRows; r0 += kBatch) {
                float v[kBatch];
#pragma unroll
                for (int r = 0; r < kBatch; ++r) v[r] = r0 + r < kRows ? row_dot(row[r0 + r < kRows ? r0 + r : 0], x) : 0.0f;
                put_parts<kRows, true>(a, at, r0, v, s.part);
            }
            put_square<true>(p, at, x, s.part);
        }
        block_barrier();
        if (t + 1 < count && tid < p.samples)
            put_word(words.sums + ((t + 1) & 1) * p.samples * S, tid * S + strip, strip_sum<true>(p, s.part, tid), a.seq0 + static_cast<uint32_t>(group + groups * (t + 1)));

        // ---- 6
        if (sums_due) ask_words((tid < 256 ? words.coefs : words.losses) + (t & 1) * p.samples, word_at, word);
        stage_rows(t + 2, kRest, kRows, places);
        return true;
    };
    bool there;
    for (int t = -1;; t += 2) {
        there = turn(t, rows_a, x_a);
        if (!there || t == count) break;
        there = turn(t + 1, rows_b, x_b);
        if (!there || t + 1 == count) break;
    }
    __builtin_amdgcn_s_waitcnt(0);             // nothing is on its way to LDS any more
    if (!there) take_tickets<kRows, kChunks, true>(static_cast<const OnePassParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()), group, &s);
}

}  // namespace

namespace {
template <int kRows, int kChunks>
hipError_t launch_shape(const OnePassParams& p, hipStream_t st) {
    const int32_t groups = p.a.shape.groups < p.a.n_ops ? p.a.shape.groups : p.a.n_ops;
    OnePassParams q = p;
    q.a.shape.groups = groups;
    const dim3 grid(groups * p.a.shape.strips), block(kOnePassThreads);
    if (q.a.shape.kernel == OnePassKernel::kPipeline) {
        if (kOnePassWaves * q.a.shape.strips < q.samples) return hipErrorInvalidValue;         // a wavefront adds up one sample
        if constexpr (onepass_built(OnePassKernel::kPipeline, kRows, kChunks)) hipLaunchKernelGGL((onepass_pipeline_kernel<kRows, kChunks>), grid, block, 0, st, q);
        else return hipErrorInvalidValue;
    } else if (q.a.shape.kernel == OnePassKernel::kStaged) {
        if constexpr (onepass_built(OnePassKernel::kStaged, kRows, kChunks)) hipLaunchKernelGGL((onepass_staged_kernel<kRows, kChunks>), grid, block, 0, st, q);
        else return hipErrorInvalidValue;
    } else {
        if constexpr (onepass_built(OnePassKernel::kPlain, kRows, kChunks)) hipLaunchKernelGGL((onepass_gradient_kernel<kRows, kChunks>), grid, block, 0, st, q);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <size_t... kAt>
hipError_t launch_held(const OnePassParams& p, hipStream_t st, std::index_sequence<kAt...>) {
    hipError_t e = hipErrorInvalidValue;
    (void)((p.a.shape.rows == kOnePassHeld[kAt].rows && p.a.shape.chunks == kOnePassHeld[kAt].chunks &&
            (e = launch_shape<kOnePassHeld[kAt].rows, kOnePassHeld[kAt].chunks>(p, st), true)) || ...);
    return e;
}
}  // namespace

hipError_t launch_onepass_gradient(const OnePassArgs& a, hipStream_t st) {
    if (a.n_ops <= 0) return hipSuccess;
    OnePassParams p;
    p.a = a;
    p.n_vec = (a.d + 3) / 4;
    p.samples = onepass_samples(a.model, a.M, a.loss != nullptr);
    p.pitch = static_cast<int32_t>(onepass_group_words(a.shape, p.samples));
    p.log_groups = __builtin_ctz(a.shape.row_groups);
    return launch_held(p, st, std::make_index_sequence<std::size(kOnePassHeld)>{});
}

}  // namespace adpsgd_impl
