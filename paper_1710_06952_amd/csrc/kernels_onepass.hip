// Minibatch gradients of the linear models with one pass over the minibatch rows.
//
// g = sum_m c_m a_m needs the dot products a_m . x^ of whole rows before any coefficient is known.  The three launches of
// kernels_grad_linear.hip read the rows twice for that.  Here a gradient is held by a group of blocks, one per compute unit,
// each with a strip of the columns of all its rows in registers; the blocks exchange the partial dot products and, when the
// coefficients are known, combine the rows that are still there.  A row that is done makes room for one of the block's next
// gradient of the round, and several groups work side by side.
//
// What binds is the memory while rows arrive and the exchange in between, which nothing covers: n = 32, M = 8, d = 1 M, all 32
// gradients of a synchronous iteration, 8.2 us each: of the 16 us of two groups side by side 9.6 are the rows of both at the
// rate of the memory, the rest dot products (1.2), two steps of the exchange (2.4 and 1.9) and combination (0.9; two wavefronts
// to a SIMD issue only half of what it could).  Measured, all of a call against three launches a round: that iteration 340 against 435 us; n = 64, M = 128, d = 65 536, logistic, 500 events 4.65
// against 5.93 ms.  Not taken: every block adds all sums by itself (M = 8: 372 us, 656 words polled by every block); groups that
// start after each other or wait for each other's rows (340 ... 400 us: what the exchanges gain, the slower loads of half the
// compute units lose); two blocks with half the rows on a compute unit (376 us: polls stand behind the other block's rows).
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

#include "chains.hpp"
#include "device_common.hpp"
#include "exchange.hpp"
#include "onepass.hpp"

namespace adpsgd_impl {
namespace {

struct OnePassParams {
    OnePassArgs a;
    int64_t n_vec;
    int32_t tile_cols;           // columns of a strip
    int32_t samples;             // onepass_samples
    int32_t pitch;               // words of a group (GroupWords)
};

// Buffers (chains.hpp) check every word, also of a 128-bit load: what lies beyond d in a padded row and rows beyond M need no masks.
__device__ __forceinline__ float dot4(v4f a, v4f b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
__device__ __forceinline__ v4f zero_beyond(v4f v, int64_t e, int64_t d) {
    if (e >= d) v.x = 0.0f;
    if (e + 1 >= d) v.y = 0.0f;
    if (e + 2 >= d) v.z = 0.0f;
    if (e + 3 >= d) v.w = 0.0f;
    return v;
}
// The word at[u] of gradient seq, for the lanes that want one; false when the time is up.
template <int N>
__device__ __forceinline__ bool take_words(const unsigned long long* base, const int (&at)[N], uint32_t seq, uint64_t until, float (&v)[N]) {
    unsigned long long w[N];
    for (;;) {
        bool complete = true;
#pragma unroll
        for (int u = 0; u < N; ++u) w[u] = at[u] >= 0 ? __hip_atomic_load(base + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
#pragma unroll
        for (int u = 0; u < N; ++u) complete &= at[u] < 0 || static_cast<uint32_t>(w[u] >> 32) == seq;
        if (__all(complete)) break;
        if (wall_clock64() >= until) return false;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = __uint_as_float(static_cast<uint32_t>(w[u]));
    return true;
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

template <int kChunks>
struct OnePassShared {
    static constexpr int kReduce = kChunks < 4 ? kChunks : 4;                          // chunks whose partial gradients are in LDS at a time
    __attribute__((aligned(16))) v4f red[kOnePassWaves][kReduce][64];
    float part[kOnePassWaves][kOnePassMaxM + 1];            // [column group][sample]
    float coef[kOnePassMaxM], loss[kOnePassMaxM + 1];       // beyond M: coefficient 0
    int32_t idx[2][kOnePassMaxM];                           // beyond M: row 0 (of which nothing is read)
    uint32_t ticket;
    int late, lost;
};

// What a thread has of a strip: the same in every block that works on it.
struct StripPlace {
    int64_t col0;                                // of its wavefront
    int bytes, offset, row_group, col_group;     // in bounds from col0 on; of its lane
    __device__ __forceinline__ StripPlace(const OnePassParams& p, int strip, int chunks) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
        row_group = wave % p.a.shape.row_groups;
        col_group = wave / p.a.shape.row_groups;
        col0 = static_cast<int64_t>(strip) * p.tile_cols + col_group * (256 * chunks);
        const int64_t left = 4 * (p.a.d - col0);
        bytes = left <= 0 ? 0 : left < 1024 * chunks ? static_cast<int>(left) : 1024 * chunks;
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
// row r of the thread's row group
template <int kChunks>
__device__ __forceinline__ void request_row(const OnePassArgs& a, const GradOp& op, const StripPlace& at, const int32_t* index, int r, int bytes, v4f (&row)[kChunks]) {
    const int m = at.row_group + a.shape.row_groups * r;
    const int64_t from = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(index[m])) * op.ld + at.col0;
    const Buffer b = buffer_of(static_cast<const float*>(op.features) + from, m < a.M ? bytes : 0);
#pragma unroll
    for (int c = 0; c < kChunks; ++c) row[c] = buffer_load4<true>(b, at.offset + 1024 * c);
}
template <int kChunks>
__device__ __forceinline__ float row_dot(const v4f (&row)[kChunks], const v4f (&x)[kChunks]) {
    float v = 0.0f;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) v += dot4(row[c], x[c]);
    return v;
}
// Partial dot products of rows r0, r0 + 1, ... of the wavefront's, summed over its lanes, to part[column group][sample].
template <int kRows, int kBatch>
__device__ __forceinline__ void put_parts(const OnePassArgs& a, const StripPlace& at, int r0, const float (&v)[kBatch], float (*part)[kOnePassMaxM + 1]) {
    const int lane = threadIdx.x & 63;
    const float z = wave_sums(v, lane);
    const int r = r0 + lane / (64 / kBatch), m = at.row_group + a.shape.row_groups * r;
    if (lane % (64 / kBatch) == 0 && r < kRows && m < a.M) part[at.col_group][m] = z;
}
template <int kChunks>
__device__ __forceinline__ void put_square(const OnePassParams& p, const StripPlace& at, const v4f (&x)[kChunks], float (*part)[kOnePassMaxM + 1]) {
    if (p.samples <= p.a.M || at.row_group != 0) return;
    const float z = all_sum(row_dot(x, x));
    if ((threadIdx.x & 63) == 0) part[at.col_group][p.a.M] = z;
}
// A sample's sum over the column groups of a strip.
__device__ __forceinline__ float strip_sum(const OnePassParams& p, const float (*part)[kOnePassMaxM + 1], int m) {
    float z = part[0][m];
    for (int g = 1; g < kOnePassWaves / p.a.shape.row_groups; ++g) z += part[g][m];
    return z;
}
// Sums over the strips of samples m, m + step, ... below samples, kN at most, by a wavefront; false when the time is up.
template <int kN>
__device__ __forceinline__ bool take_sums(const unsigned long long* sums, int m, int step, int samples, int S, uint32_t seq, uint64_t until, float (&dot)[kN]) {
    constexpr int kLines = kOnePassMaxStrips / 64;
    const int lane = threadIdx.x & 63;
    int at[kN * kLines];
    float v[kN * kLines];
#pragma unroll
    for (int i = 0; i < kN; ++i)
#pragma unroll
        for (int u = 0; u < kLines; ++u) at[i * kLines + u] = m + i * step < samples && lane + 64 * u < S ? (m + i * step) * S + lane + 64 * u : -1;
    const bool there = take_words(sums, at, seq, until, v);
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        dot[i] = 0.0f;
#pragma unroll
        for (int u = 0; u < kLines; ++u) dot[i] += v[i * kLines + u];
        dot[i] = all_sum(dot[i]);
    }
    return there;
}
__device__ __forceinline__ v2f finish_sample(const OnePassArgs& a, int m, float dot, float target) {
    return m < a.M ? coefficient(a, dot, target) : v2f{0.0f, 0.5f * a.lambda * static_cast<float>(a.M) * dot};
}
// The minibatch loss from those of its samples, by a wavefront.
__device__ __forceinline__ void put_loss(const OnePassParams& p, const GradOp& op, const float* loss) {
    const int lane = threadIdx.x & 63;
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
template <int kChunks>
__device__ __forceinline__ void put_gradient(const OnePassParams& p, const GradOp& op, const StripPlace& at, int strip, const v4f (&acc)[kChunks], OnePassShared<kChunks>& s) {
    constexpr int kReduce = OnePassShared<kChunks>::kReduce;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row_groups = p.a.shape.row_groups, col_groups = kOnePassWaves / row_groups;
    float* const g = p.a.slots + static_cast<int64_t>(op.slot) * p.a.ld;
    if (row_groups == 1) {
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t e = at.col0 + 256 * c + 4 * lane;
            if (e < 4 * p.n_vec) *reinterpret_cast<v4f*>(g + e) = zero_beyond(acc[c], e, p.a.d);
        }
        return;
    }
    const int64_t tile0 = static_cast<int64_t>(strip) * p.tile_cols;       // the sums of the row groups through LDS
#pragma unroll
    for (int c0 = 0; c0 < kChunks; c0 += kReduce) {
        if (c0 > 0) __syncthreads();
#pragma unroll
        for (int c = 0; c < kReduce; ++c)
            if (c0 + c < kChunks) s.red[wave][c][lane] = acc[c0 + c < kChunks ? c0 + c : 0];
        __syncthreads();
        for (int u = tid; u < col_groups * kReduce * 64; u += kOnePassThreads) {
            const int l = u & 63, c = (u >> 6) % kReduce, cg = (u >> 6) / kReduce;
            const int64_t e = tile0 + (cg * kChunks + c0 + c) * 256 + 4 * l;
            if (c0 + c >= kChunks || e >= 4 * p.n_vec) continue;
            v4f sum = s.red[cg * row_groups][c][l];
            for (int w = 1; w < row_groups; ++w) sum += s.red[cg * row_groups + w][c][l];
            *reinterpret_cast<v4f*>(g + e) = zero_beyond(sum, e, p.a.d);
        }
    }
}

// Words of a group: of the exchange [samples][strips] sums, [samples] coefficients, [samples] losses; of the shares, apart from
// these, [samples][strips] sums, [samples] coefficients and two counts (number of the launch, count).
struct GroupWords {
    unsigned long long *sums, *coefs, *losses, *share_sums, *share_coefs, *tickets, *taken;
    __device__ __forceinline__ GroupWords(const OnePassParams& p, int group) {
        sums = p.a.words + static_cast<int64_t>(group) * p.pitch;
        coefs = sums + p.samples * p.a.shape.strips;
        losses = coefs + p.samples;
        share_sums = losses + p.samples;
        share_coefs = share_sums + p.samples * p.a.shape.strips;
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
template <int kRows, int kChunks>
__device__ __attribute__((noinline)) void take_tickets(const OnePassParams* params, int group, OnePassShared<kChunks>* shared) {
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4, kInFlight = kChunks == 1 ? kBatch : kChunks <= 4 ? 4 : 2;       // rows
    const OnePassParams& p = *params;
    const OnePassArgs& a = p.a;
    OnePassShared<kChunks>& s = *shared;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups, word_waves = (p.samples + 63) / 64;
    const GroupWords words(p, group);
    const uint32_t launch = a.seq0, per = 2 * S + 1, shares = static_cast<uint32_t>((a.n_ops - group + groups - 1) / groups) * per;
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
        const GradOp op = a.ops[q];
        if (tid < kOnePassMaxM) s.idx[0][tid] = tid < M ? a.batch_idx[static_cast<int64_t>(op.event) * M + tid] : 0;
        __syncthreads();
        bool there = true;
        const int word_at[1] = {tid < p.samples ? tid : -1};
        float word[1];
        if (share < S) {
            const StripPlace at(p, strip, kChunks);
            v4f x[kChunks];
            request_point(a, op, at, at.bytes, x);
            if (op.comp_slot >= 0) compensate_point(a, op, at, x);
#pragma unroll 1
            for (int r0 = 0; r0 < kRows; r0 += kBatch) {
                float v[kBatch];
#pragma unroll
                for (int from = 0; from < kBatch; from += kInFlight) {
                    v4f row[kInFlight][kChunks];
#pragma unroll
                    for (int r = 0; r < kInFlight; ++r)
                        if (r0 + from + r < kRows) request_row(a, op, at, s.idx[0], r0 + from + r, at.bytes, row[r]);
#pragma unroll
                    for (int r = 0; r < kInFlight; ++r) v[from + r] = r0 + from + r < kRows ? row_dot(row[r], x) : 0.0f;
                    __builtin_amdgcn_sched_barrier(0);
                }
                put_parts<kRows>(a, at, r0, v, s.part);
            }
            put_square(p, at, x, s.part);
            if (i > 0 && wave < word_waves) there = take_words(words.share_coefs, word_at, seq - groups, until, word);
            if (!there && lane == 0) s.lost = 1;
            __syncthreads();
            if (s.lost != 0) break;
            if (tid < p.samples) put_word(words.share_sums, tid * S + strip, strip_sum(p, s.part, tid), seq);
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
                    target[u] = m < M ? static_cast<const float*>(op.targets)[s.idx[0][m]] : 0.0f;
                }
                there = take_sums(words.share_sums, m0, kOnePassWaves, p.samples, S, seq, until, dot);
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
            if (a.loss && wave == 0) put_loss(p, op, s.loss);
        } else {
            const StripPlace at(p, strip, kChunks);
            if (wave < word_waves) {
                there = take_words(words.share_coefs, word_at, seq, until, word);
                if (tid < M) s.coef[tid] = word[0];
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
#pragma unroll
            for (int r0 = 0; r0 < kRows; r0 += kInFlight) {
                v4f row[kInFlight][kChunks];
#pragma unroll
                for (int r = 0; r < kInFlight; ++r)
                    if (r0 + r < kRows) request_row(a, op, at, s.idx[0], r0 + r, at.bytes, row[r]);
#pragma unroll
                for (int r = 0; r < kInFlight; ++r) {
                    if (r0 + r >= kRows) continue;
                    const float coef = s.coef[at.row_group + a.shape.row_groups * (r0 + r)];
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
    constexpr bool kPointLast = kRows * kChunks > 40;                    // no registers for two points while rows are combined
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4;                       // dot products reduced at a time
    __shared__ OnePassShared<kChunks> s;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups, row_groups = a.shape.row_groups;
    const int group = blockIdx.x % groups, strip = blockIdx.x / groups;
    const bool logistic = a.model == ADPSGD_MODEL_LOGREG;
    const GroupWords words(p, group);
    const StripPlace at(p, strip, kChunks);

    v4f row[kRows][kChunks], x[kChunks];
    int q = group, turn = 0;
    if (q >= a.n_ops) return;
    GradOp op = a.ops[q];
    if (tid == 0) s.late = 0;
    if (tid < kOnePassMaxM) {
        s.coef[tid] = 0.0f;
        s.idx[0][tid] = tid < M ? a.batch_idx[static_cast<int64_t>(op.event) * M + tid] : 0;
    }
    __syncthreads();
    request_point(a, op, at, at.bytes, x);
#pragma unroll
    for (int r = 0; r < kRows; ++r) request_row(a, op, at, s.idx[0], r, at.bytes, row[r]);
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
            put_parts<kRows>(a, at, r0, v, s.part);
        }
        put_square(p, at, x, s.part);
        if (tid < kOnePassMaxM) s.idx[turn ^ 1][tid] = next_index;
        __syncthreads();

        // ---- the exchange
        if (tid < p.samples) put_word(words.sums, tid * S + strip, strip_sum(p, s.part, tid), seq);
        const uint64_t until = wall_clock64() + a.wait_ticks;
        bool there = a.wait_ticks > 0;
        for (int m = strip + S * wave; there && m < p.samples; m += S * kOnePassWaves) {
            const float target = m < M ? static_cast<const float*>(op.targets)[s.idx[turn][m]] : 0.0f;
            float dot[1];
            there = take_sums(words.sums, m, 0, p.samples, S, seq, until, dot);
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
        if (!there && lane == 0) s.late = 1;
        __syncthreads();
        if (s.late != 0) {                         // uniform over the block
            take_tickets<kRows, kChunks>(static_cast<const OnePassParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()), group, &s);
            return;
        }

        // ---- g = sum_m c_m a_m (+ lambda x^); a row that is done makes room for one of the next gradient
        const int next_bytes = more ? at.bytes : 0;         // none: the requests touch no memory
        v4f acc[kChunks];
        const float regularise = point_weight(a, at);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) acc[c] = logistic && at.row_group == 0 ? x[c] * regularise : v4f{0, 0, 0, 0};
        if (!kPointLast) request_point(a, next, at, next_bytes, x);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float coef = s.coef[at.row_group + row_groups * r];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                acc[c] += row[r][c] * coef;
                asm volatile("" : "+v"(acc[c]));      // here and not behind the request, which needs the row's registers
            }
            __builtin_amdgcn_sched_barrier(0);
            request_row(a, next, at, s.idx[turn ^ 1], r, next_bytes, row[r]);
            __builtin_amdgcn_sched_barrier(0);
        }
        put_gradient(p, op, at, strip, acc, s);
        if (kPointLast) request_point(a, next, at, next_bytes, x);
        if (a.loss && strip == 0 && wave == 7) put_loss(p, op, s.loss);
        if (!more) break;
        q += groups;
        op = next;
        turn ^= 1;
        __syncthreads();
    }
}

}  // namespace

// A thread holds up to 32 vectors of four columns, 256 KB a block: with 40 and 48, which gradients beyond 67 MB need, registers
// spill.  Below 20 strips the blocks hold less, so that a gradient spreads over more compute units (n = 16, M = 8, d = 131 000
// on the 4-regular graph: 786 us for 40 events in three launches a round, 708 with 16 strips, 609 with 32).
// Measured against the three launches, 450 set-ups of 16 and 40 workers, M = 1 ... 128, 0.25 to 100 MB a gradient:
//   logistic   1.02 ... 2.1 times as fast;
//   least squares, events   these leave the gradient as its M coefficients there, here it is written out and read again:
//              0.75 ... 1.1 times for M <= 5, 1.1 ... 1.3 for M = 6 (0.92 with 48 vectors), 1.04 ... 1.9 from M = 7 on;
//   least squares, synchronous or wait-free (dense in both)   0.94 ... 1.3 for M <= 3, 0.97 ... 1.8 from M = 5 on.
// What does not fit the chip (beyond 100 MB) and short models (d <= 2048: one block a gradient) stay with them.
OnePassShape onepass_shape(int model, int64_t d, int32_t M, int32_t compute_units) {
    OnePassShape s;
    if ((model != ADPSGD_MODEL_LSQ && model != ADPSGD_MODEL_LOGREG) || M < (model == ADPSGD_MODEL_LSQ ? 4 : 1) || M > kOnePassMaxM) return s;
    if (d <= 2048 || static_cast<double>(M) * static_cast<double>(d) < 50000.0) return s;
    s.row_groups = M <= 8 ? 1 : M <= 16 ? 2 : M <= 32 ? 4 : 8;
    const int rows = (M + s.row_groups - 1) / s.row_groups, most = std::min(compute_units, kOnePassMaxStrips);
    s.rows = rows <= 2 ? 2 : rows <= 4 ? 4 : rows <= 6 ? 6 : rows <= 8 ? 8 : rows <= 12 ? 12 : 16;
    int64_t strips = 0;
    auto hold = [&](int held) {
        s.chunks = std::max(1, held / s.rows);
        const int64_t tile = 256ll * s.chunks * (kOnePassWaves / s.row_groups);
        strips = (d + tile - 1) / tile;
    };
    hold(s.rows == 2 ? 16 : 32);
    if (strips > most && s.rows >= 6) hold(40);
    if (strips > most && s.rows >= 6) hold(48);
    if (strips < 20) hold(16);
    if (strips < 20) hold(8);
    if (strips > most) return s;
    s.strips = static_cast<int32_t>(strips);
    s.groups = static_cast<int32_t>(most / strips);
    return s;
}

bool onepass_for_events(const OnePassShape& s, int model, int32_t M, bool wait_free) {
    return model == ADPSGD_MODEL_LOGREG || wait_free || M >= (s.rows * s.chunks <= 40 ? 6 : 7);
}

size_t onepass_exchange_bytes(const OnePassShape& s, int32_t M) {
    return static_cast<size_t>(s.groups) * ((M + 1) * (2 * s.strips + 3) + 2) * sizeof(unsigned long long);
}

namespace {
template <int kRows, int kChunks>
hipError_t launch_shape(const OnePassParams& p, hipStream_t st) {
    const int32_t groups = p.a.shape.groups < p.a.n_ops ? p.a.shape.groups : p.a.n_ops;
    OnePassParams q = p;
    q.a.shape.groups = groups;
    hipLaunchKernelGGL((onepass_gradient_kernel<kRows, kChunks>), dim3(groups * p.a.shape.strips), dim3(kOnePassThreads), 0, st, q);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_onepass_gradient(const OnePassArgs& a, hipStream_t st) {
    if (a.n_ops <= 0) return hipSuccess;
    OnePassParams p;
    p.a = a;
    p.n_vec = (a.d + 3) / 4;
    p.tile_cols = 256 * a.shape.chunks * (kOnePassWaves / a.shape.row_groups);
    p.samples = onepass_samples(a.model, a.M, a.loss != nullptr);
    p.pitch = p.samples * (2 * a.shape.strips + 3) + 2;
    switch (a.shape.rows * 100 + a.shape.chunks) {
        case 204: return launch_shape<2, 4>(p, st);
        case 208: return launch_shape<2, 8>(p, st);
        case 402: return launch_shape<4, 2>(p, st);
        case 404: return launch_shape<4, 4>(p, st);
        case 408: return launch_shape<4, 8>(p, st);
        case 601: return launch_shape<6, 1>(p, st);
        case 602: return launch_shape<6, 2>(p, st);
        case 605: return launch_shape<6, 5>(p, st);
        case 606: return launch_shape<6, 6>(p, st);
        case 608: return launch_shape<6, 8>(p, st);
        case 801: return launch_shape<8, 1>(p, st);
        case 802: return launch_shape<8, 2>(p, st);
        case 804: return launch_shape<8, 4>(p, st);
        case 805: return launch_shape<8, 5>(p, st);
        case 806: return launch_shape<8, 6>(p, st);
        case 1201: return launch_shape<12, 1>(p, st);
        case 1202: return launch_shape<12, 2>(p, st);
        case 1203: return launch_shape<12, 3>(p, st);
        case 1204: return launch_shape<12, 4>(p, st);
        case 1601: return launch_shape<16, 1>(p, st);
        case 1602: return launch_shape<16, 2>(p, st);
        case 1603: return launch_shape<16, 3>(p, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace adpsgd_impl
