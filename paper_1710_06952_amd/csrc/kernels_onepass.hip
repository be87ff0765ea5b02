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
// The launch is not cooperative: nothing makes sure that all blocks of a group are resident.  A block that waits longer than
// a limit goes on by itself, for the rest of the launch: it computes the dot products of whole rows, combines its own strip
// and publishes nothing any more, so that blocks that wait for it come to the same end.  Every wait is bounded, only the
// pending slots and losses are written, and each by the block that owns it.
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
    int32_t pitch;               // words of a group: [samples][strips] sums, [samples] coefficients, [samples] losses
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

// The gradients from q on by a block that has waited too long: the dot products of whole rows, then the columns of its strip.
// Slow (one compute unit reads all rows) but complete, and it needs no other block.  A function of its own with its
// arguments in memory, since the kernel has no registers to spare for it.
__device__ __attribute__((noinline)) void run_alone(const OnePassParams* params, int q, int group, int strip, float* dot_s, float* coef_s, float* loss_s) {
    const OnePassParams& p = *params;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M = a.M;
    for (; q < a.n_ops; q += a.shape.groups) {
        const GradOp op = a.ops[q];
        const float* const features = static_cast<const float*>(op.features);
        const int32_t* const index = a.batch_idx + static_cast<int64_t>(op.event) * M;
        const float* const xr = a.X + static_cast<int64_t>(op.worker) * a.ld;
        const float* const gr = a.slots + static_cast<int64_t>(op.comp_slot < 0 ? 0 : op.comp_slot) * a.ld;
        auto point = [&](int64_t c) {
#pragma clang fp contract(off)
            if (op.comp_slot < 0) return xr[c];
            const float step = gr[c] * op.comp_gamma;
            return xr[c] - step;
        };
        for (int m = wave; m < p.samples; m += kOnePassWaves) {
            const float* const row = features + static_cast<int64_t>(index[m < M ? m : 0]) * op.ld;
            double z = 0.0;
            for (int64_t c = lane; c < a.d; c += 64) {
                const double x = point(c);
                z += x * (m < M ? static_cast<double>(row[c]) : x);
            }
            z = wave_sum(z);
            if (lane == 0) dot_s[m] = static_cast<float>(z);
        }
        __syncthreads();
        if (tid < M) {
            const v2f r = coefficient(a, dot_s[tid], static_cast<const float*>(op.targets)[index[tid]]);
            coef_s[tid] = r.x;
            loss_s[tid] = r.y;
        } else if (tid < p.samples) {
            loss_s[tid] = 0.5f * a.lambda * static_cast<float>(M) * dot_s[tid];
        }
        __syncthreads();
        const float regularise = a.model == ADPSGD_MODEL_LOGREG ? a.lambda * a.gscale * static_cast<float>(M) : 0.0f;
        float* const g = a.slots + static_cast<int64_t>(op.slot) * a.ld;
        const int64_t from = static_cast<int64_t>(strip) * p.tile_cols;
        for (int64_t c = from + tid; c < from + p.tile_cols && c < 4 * p.n_vec; c += kOnePassThreads) {
            double sum = 0.0;
            for (int m = 0; m < M && c < a.d; ++m) sum += static_cast<double>(coef_s[m]) * static_cast<double>(features[static_cast<int64_t>(index[m]) * op.ld + c]);
            float v = static_cast<float>(sum);
            if (a.model == ADPSGD_MODEL_LOGREG && c < a.d) v += point(c) * regularise;
            g[c] = v;
        }
        if (a.loss && strip == 0 && tid == 0) {
            float sum = 0.0f;
            for (int m = 0; m < p.samples; ++m) sum += loss_s[m];
            a.loss[op.event] = sum * a.gscale;
        }
        __syncthreads();
    }
}

// grid: groups x strips blocks, block b strip b / groups of group b % groups (with eight groups or a multiple of them the
// blocks of a group share an XCD)
template <int kRows, int kChunks>
__global__ __launch_bounds__(kOnePassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void onepass_gradient_kernel(const OnePassParams p) {
    constexpr int kReduce = kChunks < 4 ? kChunks : 4;                   // chunks whose partial gradients are in LDS at a time
    constexpr bool kPointLast = kRows * kChunks > 40;                    // no registers for two points while rows are combined
    constexpr int kBatch = kRows % 8 == 0 ? 8 : 4;                       // dot products reduced at a time
    __shared__ __attribute__((aligned(16))) v4f red_s[kOnePassWaves][kReduce][64];
    __shared__ float part_s[kOnePassWaves][kOnePassMaxM + 1];            // [column group][sample]
    __shared__ float coef_s[kOnePassMaxM], loss_s[kOnePassMaxM + 1];
    __shared__ int32_t idx_s[2][kOnePassMaxM];
    __shared__ int late_s;
    const OnePassArgs& a = p.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = a.shape.strips, groups = a.shape.groups, row_groups = a.shape.row_groups;
    const int group = blockIdx.x % groups, strip = blockIdx.x / groups;
    const int row_group = wave % row_groups, col_group = wave / row_groups, col_groups = kOnePassWaves / row_groups;
    const bool logistic = a.model == ADPSGD_MODEL_LOGREG;
    unsigned long long* const sums = a.words + static_cast<int64_t>(group) * p.pitch;     // [sample][strip]
    unsigned long long* const coefs = sums + p.samples * S;                               // [sample]
    unsigned long long* const losses = coefs + p.samples;                                 // [sample]
    const int offset = 16 * lane;

    v4f row[kRows][kChunks], x[kChunks];
    const int64_t col0 = static_cast<int64_t>(strip) * p.tile_cols + col_group * (256 * kChunks), left = 4 * (a.d - col0);
    const int bytes = left <= 0 ? 0 : left < 1024 * kChunks ? static_cast<int>(left) : 1024 * kChunks;
    auto request_point = [&](const GradOp& op, int bytes) {
        const Buffer b = buffer_of(a.X + static_cast<int64_t>(op.worker) * a.ld + col0, bytes);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) x[c] = buffer_load4<false>(b, offset + 1024 * c);
    };
    auto request_row = [&](const GradOp& op, const int32_t* index, int r, int bytes) {
        const int m = row_group + row_groups * r;
        const int64_t at = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(index[m])) * op.ld + col0;
        const Buffer b = buffer_of(static_cast<const float*>(op.features) + at, m < M ? bytes : 0);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) row[r][c] = buffer_load4<true>(b, offset + 1024 * c);
    };
    int q = group, turn = 0;
    if (q >= a.n_ops) return;
    GradOp op = a.ops[q];
    if (tid == 0) late_s = 0;
    if (tid < kOnePassMaxM) {             // beyond M: coefficient 0, row 0 (of which nothing is read)
        coef_s[tid] = 0.0f;
        idx_s[0][tid] = tid < M ? a.batch_idx[static_cast<int64_t>(op.event) * M + tid] : 0;
    }
    __syncthreads();
    request_point(op, bytes);
#pragma unroll
    for (int r = 0; r < kRows; ++r) request_row(op, idx_s[0], r, bytes);
    for (;;) {
        const uint32_t seq = a.seq0 + static_cast<uint32_t>(q);
        const bool more = q + groups < a.n_ops;
        const GradOp next = a.ops[more ? q + groups : q];
        int32_t next_index = 0;
        if (tid < M) next_index = a.batch_idx[static_cast<int64_t>(next.event) * M + tid];
        if (op.comp_slot >= 0) {          // wait-free variant: x^ = row - gamma_k' g_k'
#pragma clang fp contract(off)
            const Buffer b = buffer_of(a.slots + static_cast<int64_t>(op.comp_slot) * a.ld + col0, bytes);
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                const v4f step = buffer_load4<false>(b, offset + 1024 * c) * op.comp_gamma;
                x[c] = x[c] - step;
            }
        }
        // ---- partial dot products
#pragma unroll
        for (int r0 = 0; r0 < kRows; r0 += kBatch) {
            float v[kBatch];
#pragma unroll
            for (int r = 0; r < kBatch; ++r) {
                v[r] = 0.0f;
                if (r0 + r < kRows)
#pragma unroll
                    for (int c = 0; c < kChunks; ++c) v[r] += dot4(row[r0 + r < kRows ? r0 + r : 0][c], x[c]);
            }
            const float z = wave_sums(v, lane);
            const int r = r0 + lane / (64 / kBatch), m = row_group + row_groups * r;
            if (lane % (64 / kBatch) == 0 && r < kRows && m < M) part_s[col_group][m] = z;
        }
        if (p.samples > M && row_group == 0) {
            float z = 0.0f;
#pragma unroll
            for (int c = 0; c < kChunks; ++c) z += dot4(x[c], x[c]);
            z = all_sum(z);
            if (lane == 0) part_s[col_group][M] = z;
        }
        if (tid < kOnePassMaxM) idx_s[turn ^ 1][tid] = next_index;
        __syncthreads();

        // ---- the exchange
        if (tid < p.samples) {
            float z = part_s[0][tid];
            for (int g = 1; g < col_groups; ++g) z += part_s[g][tid];
            put_word(sums, tid * S + strip, z, seq);
        }
        const uint64_t until = wall_clock64() + a.wait_ticks;
        bool there = a.wait_ticks > 0;
        for (int m = strip + S * wave; there && m < p.samples; m += S * kOnePassWaves) {
            const float target = m < M ? static_cast<const float*>(op.targets)[idx_s[turn][m]] : 0.0f;
            int at[kOnePassMaxStrips / 64];
            float v[kOnePassMaxStrips / 64];
#pragma unroll
            for (int u = 0; u < kOnePassMaxStrips / 64; ++u) at[u] = lane + 64 * u < S ? m * S + lane + 64 * u : -1;
            there = take_words(sums, at, seq, until, v);
            float dot = 0.0f;
#pragma unroll
            for (int u = 0; u < kOnePassMaxStrips / 64; ++u) dot += v[u];
            dot = all_sum(dot);
            if (there && lane == 0) {
                const v2f r = m < M ? coefficient(a, dot, target) : v2f{0.0f, 0.5f * a.lambda * static_cast<float>(M) * dot};
                put_word(coefs, m, r.x, seq);
                if (a.loss) put_word(losses, m, r.y, seq);
            }
        }
        const int awaited = onepass_awaited(p.samples);
        if (there && wave < (awaited + 63) / 64) {
            const int at[1] = {tid < awaited ? tid : -1};
            float v[1];
            there = take_words(coefs, at, seq, until, v);
            if (tid < M) coef_s[tid] = v[0];
        }
        if (there && a.loss && strip == 0 && wave >= 4 && wave - 4 < (p.samples + 63) / 64) {
            const int m = tid - 256;
            const int at[1] = {m < p.samples ? m : -1};
            float v[1];
            there = take_words(losses, at, seq, until, v);
            if (m < p.samples) loss_s[m] = v[0];
        }
        if (!there && lane == 0) late_s = 1;
        __syncthreads();
        if (late_s != 0) {                         // on its own from here, uniform over the block
            if (tid == 0) __hip_atomic_fetch_add(a.late, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            run_alone(static_cast<const OnePassParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr()), q, group, strip, &part_s[0][0], coef_s, loss_s);
            return;
        }

        // ---- g = sum_m c_m a_m (+ lambda x^); a row that is done makes room for one of the next gradient
        const int next_bytes = more ? bytes : 0;         // none: the requests touch no memory
        v4f acc[kChunks];
        const float regularise = logistic && row_group == 0 ? a.lambda * a.gscale * static_cast<float>(M) : 0.0f;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) acc[c] = logistic && row_group == 0 ? x[c] * regularise : v4f{0, 0, 0, 0};
        if (!kPointLast) request_point(next, next_bytes);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float coef = coef_s[row_group + row_groups * r];
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                acc[c] += row[r][c] * coef;
                asm volatile("" : "+v"(acc[c]));      // here and not behind the request, which needs the row's registers
            }
            __builtin_amdgcn_sched_barrier(0);
            request_row(next, idx_s[turn ^ 1], r, next_bytes);
            __builtin_amdgcn_sched_barrier(0);
        }
        float* const g = a.slots + static_cast<int64_t>(op.slot) * a.ld;
        if (row_groups == 1) {
#pragma unroll
            for (int c = 0; c < kChunks; ++c) {
                const int64_t e = col0 + 256 * c + 4 * lane;
                if (e < 4 * p.n_vec) *reinterpret_cast<v4f*>(g + e) = zero_beyond(acc[c], e, a.d);
            }
        } else {                                   // the sums of the row groups through LDS
            const int64_t tile0 = static_cast<int64_t>(strip) * p.tile_cols;
#pragma unroll
            for (int c0 = 0; c0 < kChunks; c0 += kReduce) {
                if (c0 > 0) __syncthreads();
#pragma unroll
                for (int c = 0; c < kReduce; ++c)
                    if (c0 + c < kChunks) red_s[wave][c][lane] = acc[c0 + c < kChunks ? c0 + c : 0];
                __syncthreads();
                for (int u = tid; u < col_groups * kReduce * 64; u += kOnePassThreads) {
                    const int l = u & 63, c = (u >> 6) % kReduce, cg = (u >> 6) / kReduce;
                    const int64_t e = tile0 + (cg * kChunks + c0 + c) * 256 + 4 * l;
                    if (c0 + c >= kChunks || e >= 4 * p.n_vec) continue;
                    v4f s = red_s[cg * row_groups][c][l];
                    for (int w = 1; w < row_groups; ++w) s += red_s[cg * row_groups + w][c][l];
                    *reinterpret_cast<v4f*>(g + e) = zero_beyond(s, e, a.d);
                }
            }
        }
        if (kPointLast) request_point(next, next_bytes);
        if (a.loss && strip == 0 && wave == 7) {
            float sum_l = 0.0f;
            for (int m = lane; m < p.samples; m += 64) sum_l += loss_s[m];
            sum_l = all_sum(sum_l);
            if (lane == 0) a.loss[op.event] = sum_l * a.gscale;
        }
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
    return static_cast<size_t>(s.groups) * (M + 1) * (s.strips + 2) * sizeof(unsigned long long);
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
    p.pitch = p.samples * (a.shape.strips + 2);
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
