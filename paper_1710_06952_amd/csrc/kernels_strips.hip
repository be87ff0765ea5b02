// All events of a call of a linear model in one persistent launch.
//
// The rounds of short and medium models are chains of small kernels: launches, round trips to memory and the gather of
// minibatch rows that miss every cache bind them, not bytes (n = 16, d = 4096, M = 8: 22 us per round of four events,
// of which 14 us in the kernel of the dot products).  Here block c owns the columns [256 c, 256 c + 256) of all models
// for the whole call.  Averaging and updates couple rows, never columns, so the only thing the blocks exchange are the
// M dot products a_m . x^ of every gradient; models, momentum buffers and pending gradients of a strip stay in LDS,
// minibatch rows are read once, into registers, ahead of the events that need them (the schedule names them), and are
// still there when the coefficients arrive.
// Measured, a call against the same call in rounds of three launches:  n = 8, d = 1024, M = 32, 200 events 0.24 against
// 0.78 ms;  n = 16, d = 4096, M = 8, 1280 events 0.70 against 7.2 ms;  n = 16, d = 20 001, M = 50, wait-free with momentum, 400
// events 1.14 against 4.1 ms.  What binds is the chain of an iteration (updates and x^, dot products, exchange and coefficients,
// combination, barriers) times their number: 142, 4.6 us each with 9 gradients, for the second of these; with many rows per
// gradient (the third, 103 of 11 us) also their address translation, about 40 cycles per row and compute unit.
// An iteration evaluates a gradient per team.  With half of them, so that all rows are requested an iteration ahead, the three
// took 72, 217 and 203 iterations and 0.28, 1.07 and 1.70 ms: most calls run out of teams before they run out of events that
// could go on.  Where the events do not fill the teams an iteration takes 2 ... 9 % longer than it did then (n = 8, d = 40 000,
// M = 8, 400 events 550 -> 565 us;  n = 5, d = 20 001, M = 16, T_max = 0, 400 events 965 -> 1040).  That is not the wider records (with
// half as many evaluations and the present code 1034) but the polls of two sizes, whose code takes scalar registers
// from the helpers' chain: with one size of four words 970 there, and 829 for 800 us in the second of the above.  Two sets
// of rows per wavefront for M <= 8 were slower (0.88 ms for the second: a wavefront that works on one set waits for the rows of
// the other).
//
// A block has 12 main wavefronts in `teams` teams, each team with the rows of one gradient in its registers, and 4
// helper wavefronts (one thread per column, and one per minibatch sample).  An iteration has three phases:
//   A  helpers: finish the gradients of the last iteration, apply updates, write x^ of the next gradients to LDS (teams of one
//      wavefront take it from the state in LDS themselves: a third of the helpers' phase, 0.82 -> 0.71 ms for the second of the above);
//      main: idle teams request the rows of their next gradient (which may be one of this iteration)
//   B  main: dot products of a team's rows with x^, published;  helpers: wait for the sums, make the coefficients
//   C  main: sum_m c_m a_m of the team's rows to LDS
// A compute unit returns vector loads in order, so a wait of phase B stands behind the rows requested before it: they go
// out at the start of phase A (in phase B they cost 0.5 us per iteration), and the helpers load nothing else before a wait.
// Where several groups exchange, the helpers do not poll before the block's own words are out (kGate).
// Rows beyond M are requested again in vain (no branch around a load), up to 31 of 96 (M = 65): hence kernels for several numbers of
// rows of a wavefront (launch_strips).
//
// The sums go through the words of exchange.hpp: up to 32 strips exchange them directly; more sum within their XCD first
// (the blocks of a group share out the samples), and only these sums cross the chip, at most 8 per sample.
#include <type_traits>

#include "device_common.hpp"
#include "exchange.hpp"
#include "strips.hpp"

namespace adpsgd_impl {
namespace {

constexpr int kMainThreads = 64 * kStripMainWaves;
constexpr int kStripThreads = kMainThreads + kStripHelpers;

struct StripParams {
    StripArgs a;
    int32_t samples;             // words per block and gradient: M, and |x^|^2 of the logistic loss
    int32_t blocks, group_size;  // strips, and how many form a group
    unsigned long long* sums;    // the groups' sums, [ring][group][samples, whole lines]: a line is written on one XCD only
    int32_t sum_pitch;           // words of a group's sums
};

__device__ __forceinline__ float dot4(v4f a, v4f b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }

// Coefficient (times gscale) and loss of a sample from its dot product with the point (square: |x^|^2, for the loss).
__device__ __forceinline__ v2f strip_coefficient(const StripArgs& a, float dot, float target, float square) {
    float coef, loss;
    if (a.model == ADPSGD_MODEL_LSQ) {
        const float r = dot - target;               // a.x - b
        loss = 0.5f * r * r;
        coef = r;
    } else {
        const float s = -target * dot;              // F = log(1 + e^s) + reg
        loss = a.loss ? (s > 0.0f ? s + log1pf(expf(-s)) : log1pf(expf(s))) + 0.5f * a.lambda * square : 0.0f;
        coef = -target / (1.0f + expf(-s));         // -y sigmoid(s)
    }
    return v2f{coef * a.gscale, loss};
}

// LDS offsets fit 32 bits, places in global memory need 64
template <bool kLds> struct Pitch { typedef uint32_t type; };
template <> struct Pitch<false> { typedef int64_t type; };

// The whole call by one block, with the state in its global places: what a launch does whose blocks could not all become
// resident in time.  Slow (one compute unit reads all minibatch rows, twice) but complete, and it needs no other block.
// Columns belong to threads throughout; only the points of evaluation, which lie in the gradients' slots until these
// replace them, are read across threads.  A function of its own with its arguments in device memory: inlined, it cost the
// kernel's rows registers (M = 50: 1.72 -> 2.01 ms).
template <bool kMom>
__device__ __attribute__((noinline)) void run_alone(const StripArgs* args, int samples, v4u (*rows_of)[2], float* dots, float* coef_s, float* loss_s) {
    const StripArgs& a = *args;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M = a.M, half = a.teams;
    float* const slots = a.lds_state ? a.alone_slots : a.slots;
    for (int i = 0; i < a.n_in; ++i)
        for (int64_t c = tid; c < a.d; c += kStripThreads) slots[a.carry[2 * i] * a.ld + c] = a.slots[a.carry[2 * i + 1] * a.ld + c];
    for (int it = 0; it < a.iterations; ++it) {
        const v4u* rec = reinterpret_cast<const v4u*>(a.recs) + static_cast<int64_t>(it) * a.rec_len;
        const v4u head = rec[0];
        for (int64_t c = tid; c < a.d; c += kStripThreads)
            for (uint32_t u = 0; u < head.x; ++u) {
                const v4u op = rec[1 + 4 * half + u];
                if ((op.w & kStripEmpty) != 0) continue;
                float* const xi = a.X + static_cast<int64_t>(op.x & 0xFFFFu) * a.ld + c;
                float* const xj = a.X + static_cast<int64_t>(op.x >> 16) * a.ld + c;
                const bool average_only = (op.w & kStripAverage) != 0;
                const float g = average_only ? 0.0f : slots[op.y * a.ld + c];
                float ni, nj;
                if (kMom) {
                    float* const v = a.V + static_cast<int64_t>(op.x & 0xFFFFu) * a.ld + c;
                    float vn;
                    average_then_apply_momentum(*xi, *xj, g, *v, __uint_as_float(op.z), a.momentum, a.weight_decay, ni, nj, vn);
                    if (!average_only) *v = vn;
                } else {
                    average_then_apply(*xi, *xj, g, __uint_as_float(op.z), ni, nj);
                }
                *xj = nj;
                *xi = average_only ? nj : ni;
            }
        if (tid < a.teams && (head.y >> tid & 1) != 0) {
            const v4u* e = rec + 1 + 2 * half + 2 * __popc(head.y & ((1u << tid) - 1));
            rows_of[tid][0] = e[0];
            rows_of[tid][1] = e[1];
        }
        __syncthreads();
        const int evals = __popc(head.z);
        for (int i = 0; i < evals; ++i) {
            const v4u ev = rec[1 + 2 * i], ev2 = rec[2 + 2 * i];
            float* const point = slots + ev.w * a.ld;
            for (int64_t c = tid; c < a.d; c += kStripThreads) {
#pragma clang fp contract(off)
                float x = a.X[ev.z * a.ld + c];
                if (ev2.x != 0xFFFFFFFFu) {
                    const float step = slots[ev2.x * a.ld + c] * __uint_as_float(ev2.y);
                    x = x - step;
                }
                point[c] = x;
            }
            __syncthreads();
            const v4u f = rows_of[ev.x][0], g = rows_of[ev.x][1];
            const Global<float> features = in_global<float>(reinterpret_cast<const void*>(static_cast<uint64_t>(f.w) << 32 | f.z));
            const Global<float> targets = in_global<float>(reinterpret_cast<const void*>(static_cast<uint64_t>(g.y) << 32 | g.x));
            const int32_t* const index = a.idx + static_cast<int64_t>(ev.y - a.seq0) * M;
            for (int m = wave; m < samples; m += kStripThreads / 64) {
                const Global<float> row = m < M ? features + static_cast<int64_t>(index[m]) * f.y : in_global<float>(point);      // the last: |x^|^2
                double z = 0.0;
                for (int64_t c = lane; c < a.d; c += 64) z += static_cast<double>(row[c]) * static_cast<double>(point[c]);
                z = wave_sum(z);
                if (lane == 0) dots[m] = static_cast<float>(z);
            }
            __syncthreads();
            if (tid < M) {
                const v2f r = strip_coefficient(a, dots[tid], targets[index[tid]], samples > M ? dots[M] : 0.0f);
                coef_s[tid] = r.x;
                loss_s[tid] = r.y;
            }
            __syncthreads();
            if (a.loss && tid == 0) {
                float sum = 0.0f;
                for (int m = 0; m < M; ++m) sum += loss_s[m];
                a.loss[ev2.z] = sum * a.gscale;
            }
            const float regularise = a.model == ADPSGD_MODEL_LOGREG ? a.lambda * a.gscale * static_cast<float>(M) : 0.0f;
            for (int64_t c = tid; c < a.d; c += kStripThreads) {
                double sum = 0.0;
                for (int m = 0; m < M; ++m) sum += static_cast<double>(coef_s[m]) * static_cast<double>(features[static_cast<int64_t>(index[m]) * f.y + c]);
                point[c] = static_cast<float>(sum) + (a.model == ADPSGD_MODEL_LOGREG ? point[c] * regularise : 0.0f);
            }
            __syncthreads();
        }
    }
    for (int i = a.n_in; i < a.n_in + a.n_out; ++i)
        for (int64_t c = tid; c < a.d; c += kStripThreads) a.slots[a.carry[2 * i + 1] * a.ld + c] = slots[a.carry[2 * i] * a.ld + c];
}

// kTeams teams of 12 / kTeams wavefronts, kRows rows per wavefront; kLds: the strip's models, momentum buffers and
// slots in LDS, otherwise in their global places (every entry is touched by one thread only, its column's).
template <int kTeams, int kRows, bool kLds, bool kMom, bool kFar>
__global__ __launch_bounds__(kStripThreads) void strip_events_kernel(const StripParams p) {
    constexpr int kTeamWaves = kStripMainWaves / kTeams;
    constexpr int kTeamHelpers = kTeams == 12 ? kRows : kTeams == 6 ? 32 : kTeams == 4 ? 64 : 128;      // threads, one per sample
    constexpr int kWordsInFlight = kTeams == 12 && kLds ? 6 : 4;        // per lane of a helper
    // In a launch of several groups with many rows to a wavefront the rows are requested by flat loads, which go out more slowly, while the
    // helpers poll (what a compiler that finds out that these are global would cost):  two teams, n = 5, d = 12 000, M = 128 1.39 ms, 1.44
    // without;  four teams with 18 or 22 rows, 25 calls of M = 49 ... 64, d = 9001 ... 60 000 1.02 times as fast in the mean (0.99 ... 1.05), with
    // 16 rows (M = 36, 44) 0.955 ... 1.00 times.
    constexpr bool kSlowRows = kFar && (kTeams == 2 || (kTeams == 4 && kRows > 16));
    using Row = std::conditional_t<kSlowRows, const float*, Global<float>>;
    using Vector = std::conditional_t<kSlowRows, const v4f*, Global<v4f>>;
    static_assert(kTeams * kTeamHelpers <= kStripHelpers, "a helper per sample of every team");
    // teams of one wavefront have the whole gradient and put it into its slot themselves
    constexpr bool kDirect = kLds && kTeamWaves == 1;
    constexpr int kChunk = kRows > 16 ? 4 : kRows < 8 ? kRows : 8;      // rows whose sums or addresses are in registers at a time
    // In a launch of several groups the polls wait until the block's own words are out, so that they do not stand behind rows and
    // are not in vain: n = 6, d = 20 000, M = 64, 300 events 1.17 -> 1.03 ms, n = 8, d = 40 000, M = 8 0.63 -> 0.60.  Not with two teams
    // (n = 5, d = 12 000, M = 128 1.39 -> 1.43) nor in one group, where words are a short way off (n = 16, d = 4096, M = 8 0.71 -> 0.75).
    constexpr bool kGate = kFar && kTeams > 2;
    const StripArgs& a = p.a;
    extern __shared__ __attribute__((aligned(16))) float state_s[];      // [rows of X][rows of V][slots] x 256
    __shared__ __attribute__((aligned(16))) v4f red_s[kStripMainWaves][64];      // partial gradients, in the same order
    __shared__ __attribute__((aligned(16))) float xh_s[kTeams][kStripCols];            // points, in the order of a record's evaluations
    __shared__ v4u rec_s[4][kStripMaxRec];
    __shared__ const float* rowp_s[2][kStripHelpers];                    // [iteration][team][sample]: the sample's row ...
    __shared__ int32_t index_s[2][kStripHelpers];                        // ... its number ...
    __shared__ float target_s[kStripHelpers];                            // ... and its target
    __shared__ float coef_s[kStripHelpers];
    __shared__ float loss_s[kStripHelpers];
    __shared__ Assembly assembly_s;
    __shared__ int lost_s;
    __shared__ uint32_t published_s[2];                                  // by iteration: wavefronts whose words are out (kGate)

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = a.M, S = p.samples;
    if (tid == 0) lost_s = 0;
    if (kGate && tid < 2) published_s[tid] = 0;
    if (tid == 0) assembly_s = assemble(a.counters, p.blocks, p.group_size, a.wait_ticks);
    __syncthreads();
    const Assembly as = assembly_s;
    if (as.alone) {
        run_alone<kMom>(a.self, S, reinterpret_cast<v4u(*)[2]>(&rec_s[0][0]), target_s, coef_s, loss_s);
        return;
    }
    const int block = __builtin_amdgcn_readfirstlane(as.strip);
    if (block < 0) return;
    const int64_t col0 = static_cast<int64_t>(block) * kStripCols;
    const int group = __builtin_amdgcn_readfirstlane(as.group), rank = __builtin_amdgcn_readfirstlane(as.rank);
    const int group_blocks = __builtin_amdgcn_readfirstlane(as.group_blocks), groups = __builtin_amdgcn_readfirstlane(as.groups);

    const int slots_at = a.n * (kMom ? 2 : 1) * kStripCols;
    const float regularise = a.lambda * a.gscale * static_cast<float>(M);
    if (wave < kStripMainWaves) {
        // ---- main wavefronts ------------------------------------------------------------------------------------
        const int team = wave / kTeamWaves, first = wave % kTeamWaves;       // rows first, first + kTeamWaves, ...
        const bool ragged = col0 + kStripCols > a.d;
        float target = 0.0f;
        v4f row[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) row[r] = v4f{0, 0, 0, 0};
        __syncthreads();       // the first records
        __syncthreads();       // their addresses
        for (int it = 0; it < a.iterations; ++it) {
            const v4u* rec = rec_s[it & 3];
            // what depends on the lane is computed anew in every iteration: kept, it would cost the rows registers
            int l = lane;
            asm volatile("" : "+v"(l));
            const int64_t at = col0 + 4 * l;
            const int from = at < a.d ? 4 * l : 0;       // lanes beyond d read (and drop) the strip's first columns
            const int mine = first + kTeamWaves * l;     // the sample whose target this lane brings
            const uint32_t evaluate = __builtin_amdgcn_readfirstlane(rec[0].z), load = __builtin_amdgcn_readfirstlane(rec[0].y);
            if ((load >> team & 1) != 0) {      // early: the polls of phase B stand behind these loads
                // no branch around a load: the wavefront would wait for one row before it requests the next
#pragma unroll
                for (int r0 = 0; r0 < kRows; r0 += kChunk) {
                    Row src[kChunk];
#pragma unroll
                    for (int r = 0; r < kChunk; ++r) src[r] = (Row)rowp_s[it & 1][team * kTeamHelpers + min(first + kTeamWaves * (r0 + r), M - 1)];
#pragma unroll
                    for (int r = 0; r < kChunk; ++r)
                        if (r0 + r < kRows) row[r0 + r < kRows ? r0 + r : 0] = *reinterpret_cast<Vector>(src[r] + from);
                }
                const v4u e = rec[2 + 2 * kTeams + 2 * __popc(load & ((1u << team) - 1))];
                const uint32_t low = __builtin_amdgcn_readfirstlane(e.x), high = __builtin_amdgcn_readfirstlane(e.y);      // not signed
                const Global<float> targets = in_global<float>(reinterpret_cast<const void*>(static_cast<uint64_t>(high) << 32 | low));
                target = targets[index_s[it & 1][team * kTeamHelpers + min(mine, M - 1)]];
            }
            __syncthreads();   // phase A done
            const bool evaluates = (evaluate >> team & 1) != 0;
            const int number = __builtin_amdgcn_readfirstlane(__popc(evaluate & ((1u << team) - 1)));
            const v4u* eval = rec + 1 + 2 * number;
            if (evaluates) {
                const uint32_t seq = __builtin_amdgcn_readfirstlane(eval[0].y);
                const uint32_t words = ((seq % kStripRing) * groups + group) * S * kStripGroupBlocks + rank;
                v4f x;
                if (kDirect) {         // the point of evaluation, from the state
#pragma clang fp contract(off)
                    const v4u e2 = eval[1];
                    x = *reinterpret_cast<const v4f*>(state_s + static_cast<int>(__builtin_amdgcn_readfirstlane(eval[0].z)) * kStripCols + 4 * l);
                    const uint32_t comp = __builtin_amdgcn_readfirstlane(e2.x);
                    if (comp != 0xFFFFFFFFu) {
                        const v4f step = *reinterpret_cast<const v4f*>(state_s + slots_at + static_cast<int>(comp) * kStripCols + 4 * l) *
                                         __uint_as_float(__builtin_amdgcn_readfirstlane(e2.y));
                        x = x - step;
                    }
                    if (ragged) {      // zero beyond d, whatever infinite coefficients have left there
                        if (at >= a.d) x.x = 0.0f;
                        if (at + 1 >= a.d) x.y = 0.0f;
                        if (at + 2 >= a.d) x.z = 0.0f;
                        if (at + 3 >= a.d) x.w = 0.0f;
                    }
                    if (a.model == ADPSGD_MODEL_LOGREG && first == 0) *reinterpret_cast<v4f*>(&xh_s[number][4 * l]) = x;      // for lambda x^
                } else {
                    x = *reinterpret_cast<const v4f*>(&xh_s[number][4 * l]);
                }
                if (ragged && at + 4 > a.d) {       // what lies beyond d in a padded row is arbitrary
#pragma unroll
                    for (int r = 0; r < kRows; ++r) {
                        if (at >= a.d) row[r].x = 0.0f;
                        if (at + 1 >= a.d) row[r].y = 0.0f;
                        if (at + 2 >= a.d) row[r].z = 0.0f;
                        if (at + 3 >= a.d) row[r].w = 0.0f;
                    }
                }
                // the target of a sample is in LDS before any block can have the sample's sum
                if (mine < M && l < kRows) target_s[team * kTeamHelpers + mine] = target;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
#pragma unroll
                for (int r0 = 0; r0 < kRows; r0 += kChunk) {
                    float v[kChunk];
#pragma unroll
                    for (int r = 0; r < kChunk; ++r) v[r] = r0 + r < kRows ? dot4(row[r0 + r < kRows ? r0 + r : 0], x) : 0.0f;
                    const float z = wave_sums(v, lane);
                    const int r = r0 + lane / (64 / kChunk), m = first + kTeamWaves * r;
                    if (lane % (64 / kChunk) == 0 && r < kRows && m < M) put_word(a.words, words + m * kStripGroupBlocks, z, seq);
                }
                if (S > M && first == kTeamWaves - 1) {
                    const float z = all_sum(dot4(x, x));
                    if (lane == 0) put_word(a.words, words + M * kStripGroupBlocks, z, seq);
                }
                if (kGate && lane == 0) __hip_atomic_fetch_add(&published_s[it & 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();   // the coefficients are there
            if (evaluates) {
                v4f acc = {0, 0, 0, 0};      // sums of four rows at a time: shorter chains, smaller error
#pragma unroll
                for (int r0 = 0; r0 < kRows; r0 += kChunk) {
                    float coef[kChunk];
#pragma unroll
                    for (int r = 0; r < kChunk; ++r) coef[r] = coef_s[team * kTeamHelpers + min(first + kTeamWaves * (r0 + r), kTeamHelpers - 1)];
#pragma unroll
                    for (int r1 = 0; r1 < kChunk; r1 += 4) {
                        v4f part = {0, 0, 0, 0};
#pragma unroll
                        for (int r = r1; r < r1 + 4 && r < kChunk; ++r)
                            if (r0 + r < kRows && first + kTeamWaves * (r0 + r) < M) part += row[r0 + r < kRows ? r0 + r : 0] * coef[r];
                        acc += part;
                    }
                }
                if (a.loss && first == 0 && __builtin_amdgcn_readfirstlane(eval[1].w) == static_cast<uint32_t>(block)) {
                    float sum = lane < M ? loss_s[team * kTeamHelpers + lane] : 0.0f;
                    if (lane + 64 < M) sum += loss_s[team * kTeamHelpers + lane + 64];
                    sum = all_sum(sum);
                    if (lane == 0) a.loss[__builtin_amdgcn_readfirstlane(eval[1].z)] = sum * a.gscale;
                }
                if (kDirect) {
                    if (a.model == ADPSGD_MODEL_LOGREG) acc += *reinterpret_cast<const v4f*>(&xh_s[number][4 * l]) * regularise;
                    *reinterpret_cast<v4f*>(state_s + slots_at + static_cast<int>(__builtin_amdgcn_readfirstlane(eval[0].w)) * kStripCols + 4 * lane) = acc;
                } else {
                    red_s[number * kTeamWaves + first][l] = acc;
                }
            }
            __syncthreads();   // phase C done
        }
        return;
    }

    // ---- helper wavefronts: column t, and sample t % kTeamHelpers of team t / kTeamHelpers ---------------------------
    const int t = tid - kMainThreads, hw = t >> 6;
    const int team = min(t / kTeamHelpers, kTeams - 1), m = t / kTeamHelpers < kTeams ? t % kTeamHelpers : kStripHelpers;
    const int64_t col = col0 + t;
    const bool inside = col < a.d;
    const uint32_t inside_bits = inside ? 0xFFFFFFFFu : 0u;      // a point is zero beyond d, whatever infinite coefficients have left there
    float* const xs = kLds ? state_s + t : a.X + col;
    float* const vs = kLds ? xs + static_cast<int64_t>(a.n) * kStripCols : a.V + col;
    float* const gs = kLds ? state_s + t + slots_at : a.slots + col;
    const typename Pitch<kLds>::type ld = kLds ? kStripCols : static_cast<typename Pitch<kLds>::type>(a.ld);
    if (kLds) {
        for (int r = 0; r < a.n; ++r) {
            xs[r * ld] = inside ? a.X[r * a.ld + col] : 0.0f;
            if (kMom) vs[r * ld] = inside ? a.V[r * a.ld + col] : 0.0f;
        }
        for (int i = 0; i < a.n_in; ++i)
            gs[a.carry[2 * i] * ld] = inside ? a.slots[a.carry[2 * i + 1] * a.ld + col] : 0.0f;
    }
    const v4u* recs = reinterpret_cast<const v4u*>(a.recs) + lane;
    const bool copies = hw == 3 && lane < a.rec_len, copies_more = hw == 3 && lane + 64 < a.rec_len;
    v4u ahead = {0, 0, 0, 0}, ahead_more = {0, 0, 0, 0};       // wavefront 3: the record after the next one
    int32_t index = 0;                    // row of this thread's sample in the worker's data
    const uint32_t below = (1u << team) - 1;
    auto load_entry = [&](const v4u* rec, uint32_t load) { return rec + 1 + 2 * kTeams + 2 * __popc(load & below); };
    auto fetch_index = [&](const v4u* rec) {
        const uint32_t load = rec[0].y;
        if ((load >> team & 1) != 0 && m < M) index = a.idx[static_cast<int64_t>(load_entry(rec, load)[0].x) * M + m];
    };
    auto put_addresses = [&](const v4u* rec, int parity) {
        const uint32_t load = rec[0].y;
        if ((load >> team & 1) != 0 && m < M) {
            const v4u f = load_entry(rec, load)[0];
            rowp_s[parity][t] = reinterpret_cast<const float*>(static_cast<uint64_t>(f.w) << 32 | f.z) + static_cast<int64_t>(index) * f.y + col0;
            index_s[parity][t] = index;
        }
    };
    // What phase A and the waits of phase B take from a record, and the rows of the first updates: read while the
    // exchange before is under way.
    constexpr int kUps = kStripBatch, kEvals = kTeams < 3 ? kTeams : 3;
    uint32_t evaluate = 0;
    int n_updates = 0, n_evals = 0;
    v4u up[kUps], ev[kEvals], ev2[kEvals];
    float xi[kUps], xj[kUps], vi[kUps];
    auto read_rows = [&] {
#pragma unroll
        for (int u = 0; u < kUps; ++u) {
            xi[u] = kLds || inside ? xs[(up[u].x & 0xFFFFu) * ld] : 0.0f;
            xj[u] = kLds || inside ? xs[(up[u].x >> 16) * ld] : 0.0f;
            vi[u] = kMom && (kLds || inside) ? vs[(up[u].x & 0xFFFFu) * ld] : 0.0f;
        }
    };
    auto read_updates = [&](const v4u* rec, int from, int count) {
#pragma unroll
        for (int u = 0; u < kUps; ++u) up[u] = rec[1 + 4 * kTeams + min(from + u, max(count, 1) - 1)];      // none: row 0, unused
        read_rows();
    };
    // Known to the compiler but for two teams in several groups, whose code is the better when it is not: 1 ... 2.5 % of 20 calls of M = 66 ... 128;
    // in one group, where it is, M = 66 ... 104 gain 1 ... 4 %.
    const bool several = kFar && kTeams == 2 ? groups > 1 : kFar;
    const int log_width = sum_width(several ? groups : group_blocks), sub = t & ((1 << log_width) - 1);
    const int words = several ? groups : group_blocks;               // of a sum
    // word of sample q and partial sum `sub`: by groups of whole lines, or by samples
    const uint32_t q_pitch = several ? 1 : kStripGroupBlocks, sub_pitch = several ? p.sum_pitch : 1;
    const uint32_t ring_pitch = several ? groups * p.sum_pitch : S * kStripGroupBlocks;
    const int log_group = sum_width(group_blocks), part = t & ((1 << log_group) - 1), slots = kStripHelpers >> log_group;
    const int mine = rank < S ? (S - rank + group_blocks - 1) / group_blocks : 0;      // samples of a gradient that this block sums
    const uint32_t per_eval = (0xFFFFu + max(mine, 1)) / max(mine, 1);                  // d / mine = d per_eval >> 16 for d mine < 2^16
    const int pair0 = t >> log_width, pair_step = kStripHelpers >> log_width;
    const unsigned long long* const base = several ? p.sums : a.words;
    bool given_up = a.lose;
    // Coefficients of up to kWords (gradient, sample) pairs per group of lanes that share a sum, from pair `from` on; samples are
    // padded to kTeamHelpers.
    auto finish_pairs = [&](const v4u* rec, int from, int count, auto words_in_flight) {
        constexpr int kWords = decltype(words_in_flight)::value;
        uint32_t at[kWords], seq[kWords], place[kWords];
        float z[kWords], reg[kWords];
#pragma unroll
        for (int u = 0; u < kWords; ++u) {
            const int pair = from + u * pair_step + pair0, i = pair / kTeamHelpers, q = pair % kTeamHelpers;
            const bool live = i < count && q < M;
            const v4u e = rec[1 + 2 * min(i, count - 1)];
            place[u] = live ? e.x * kTeamHelpers + q : kStripHelpers;
            seq[u] = live && sub < words ? e.y : 0;
            at[u] = !live ? 0 : (e.y % kStripRing) * ring_pitch + min(q, M - 1) * q_pitch + min(sub, words - 1) * sub_pitch;      // idle: near others
            reg[u] = 0.0f;
        }
        wait_words<kWords>(base, at, seq, z, given_up);
        if (S > M) {
#pragma unroll
            for (int u = 0; u < kWords; ++u) at[u] += place[u] == kStripHelpers ? 0 : (M - place[u] % kTeamHelpers) * q_pitch;
            wait_words<kWords>(base, at, seq, reg, given_up);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
        for (int u = 0; u < kWords; ++u) {
            z[u] = group_sum(z[u], log_width);
            if (S > M) reg[u] = group_sum(reg[u], log_width);
        }
        // every lane of a group has the sums of its pairs: the u-th lane finishes the u-th pair
        const int lanes = kWords <= 4 ? kWords : min(1 << log_width, kWords);         // a group has four lanes at least
        for (int u0 = 0; u0 < kWords; u0 += lanes) {
            float dot = z[0], square = reg[0];
            uint32_t to = kStripHelpers;
#pragma unroll
            for (int u = 0; u < kWords; ++u)
                if (u0 + sub == u) {
                    dot = z[u];
                    square = reg[u];
                    to = place[u];
                }
            if (sub < lanes && to != kStripHelpers) {
                const v2f r = strip_coefficient(a, dot, target_s[to], square);
                coef_s[to] = r.x;
                loss_s[to] = r.y;
            }
        }
    };
    if (copies) {
        rec_s[0][lane] = recs[0];
        rec_s[1][lane] = recs[a.rec_len];
        ahead = recs[2 * a.rec_len];
    }
    if (copies_more) {
        rec_s[0][lane + 64] = recs[64];
        rec_s[1][lane + 64] = recs[a.rec_len + 64];
        ahead_more = recs[2 * a.rec_len + 64];
    }
    __syncthreads();
    fetch_index(rec_s[0]);
    put_addresses(rec_s[0], 0);
    __syncthreads();
    fetch_index(rec_s[1]);
    n_updates = __builtin_amdgcn_readfirstlane(rec_s[0][0].x);
    evaluate = __builtin_amdgcn_readfirstlane(rec_s[0][0].z);           // record 0 evaluates nothing
    read_updates(rec_s[0], 0, n_updates);
#pragma unroll
    for (int i = 0; i < kEvals; ++i) {
        ev[i] = rec_s[0][1 + 2 * i];
        ev2[i] = rec_s[0][2 + 2 * i];
    }

    for (int it = 0; it < a.iterations; ++it) {
        const v4u* rec = rec_s[it & 3];
        // ---- A1: the gradients of the last iteration
        if (!kDirect && it > 0) {
            const v4u* last = rec_s[(it - 1) & 3];
            const int n_last = __popc(__builtin_amdgcn_readfirstlane(last[0].z));
            for (int i0 = 0; i0 < n_last; i0 += kEvals) {
                v4u e[kEvals];
                float g[kEvals];
#pragma unroll
                for (int i = 0; i < kEvals; ++i) e[i] = last[1 + 2 * min(i0 + i, n_last - 1)];
#pragma unroll
                for (int i = 0; i < kEvals; ++i) {
                    const float* part = reinterpret_cast<const float*>(&red_s[min(i0 + i, n_last - 1) * kTeamWaves][0]) + t;
                    g[i] = part[0];
#pragma unroll
                    for (int w = 1; w < kTeamWaves; ++w) g[i] += part[w * kStripCols];
                    if (a.model == ADPSGD_MODEL_LOGREG) g[i] += xh_s[min(i0 + i, n_last - 1)][t] * regularise;
                }
#pragma unroll
                for (int i = 0; i < kEvals; ++i)
                    if (i0 + i < n_last && (kLds || inside)) gs[e[i].w * ld] = g[i];
            }
        }
        // ---- A2: updates; within a batch their rows are pairwise different
        for (int u0 = 0; u0 < n_updates; u0 += kUps) {
            if (u0 > 0) read_updates(rec, u0, n_updates);
            if (kLds || inside) {
                float g[kUps];
#pragma unroll
                for (int u = 0; u < kUps; ++u) g[u] = gs[up[u].y * ld];          // slot 0 where the pair is only averaged
#pragma unroll
                for (int u = 0; u < kUps; ++u) {
                    if (u0 + u < n_updates && (up[u].w & kStripEmpty) == 0) {
                        const float gamma = __uint_as_float(up[u].z);
                        const bool average_only = (up[u].w & kStripAverage) != 0;
                        float ni, nj;
                        if (kMom) {
                            float vn;
                            average_then_apply_momentum(xi[u], xj[u], g[u], vi[u], gamma, a.momentum, a.weight_decay, ni, nj, vn);
                            vs[(up[u].x & 0xFFFFu) * ld] = average_only ? vi[u] : vn;
                        } else {
                            average_then_apply(xi[u], xj[u], g[u], gamma, ni, nj);
                        }
                        xs[(up[u].x >> 16) * ld] = nj;       // before x^i: without a partner (i == j) the step stands
                        xs[(up[u].x & 0xFFFFu) * ld] = average_only ? nj : ni;
                    }
                }
            }
        }
        // ---- A3: points of evaluation
        n_evals = __popc(evaluate);
        for (int i0 = 0; !kDirect && i0 < n_evals; i0 += kEvals) {
            float x[kEvals];
            if (i0 > 0) {
#pragma unroll
                for (int i = 0; i < kEvals; ++i) {
                    ev[i] = rec[1 + 2 * min(i0 + i, n_evals - 1)];
                    ev2[i] = rec[2 + 2 * min(i0 + i, n_evals - 1)];
                }
            }
#pragma unroll
            for (int i = 0; i < kEvals; ++i) x[i] = kLds || inside ? xs[ev[i].z * ld] : 0.0f;      // none: row 0, unused
#pragma unroll
            for (int i = 0; i < kEvals; ++i) {
                if (i0 + i < n_evals) {
                    if (__builtin_amdgcn_readfirstlane(ev2[i].x) != 0xFFFFFFFFu && (kLds || inside)) {
#pragma clang fp contract(off)
                        const float step = gs[ev2[i].x * ld] * __uint_as_float(ev2[i].y);
                        x[i] = x[i] - step;
                    }
                    xh_s[i0 + i][t] = __uint_as_float(__float_as_uint(x[i]) & inside_bits);
                }
            }
        }
        if (copies) rec_s[(it + 2) & 3][lane] = ahead;
        if (copies_more) rec_s[(it + 2) & 3][lane + 64] = ahead_more;
        __syncthreads();

        // ---- B: sums of the dot products, coefficients; first what the next phase A needs
        const v4u* next = rec_s[(it + 1) & 3];
        n_updates = __builtin_amdgcn_readfirstlane(next[0].x);
        evaluate = __builtin_amdgcn_readfirstlane(next[0].z);
        read_updates(next, 0, n_updates);
#pragma unroll
        for (int i = 0; i < kEvals; ++i) {
            ev[i] = next[1 + 2 * i];
            ev2[i] = next[2 + 2 * i];
        }
        put_addresses(next, (it + 1) & 1);
        if (kGate) {
            const uint32_t all = static_cast<uint32_t>(n_evals * kTeamWaves);
            while (__hip_atomic_load(&published_s[it & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < all) __builtin_amdgcn_s_sleep(1);
        }
        if (several) {          // the group's sums: sample q is summed by the block of rank q mod group_blocks
            for (int d0 = 0; d0 < n_evals * mine; d0 += slots) {
                int d = d0 + (t >> log_group);
                const bool live = part < group_blocks && d < n_evals * mine;
                const int i = min(static_cast<int>(static_cast<uint32_t>(d) * per_eval >> 16), n_evals - 1);
                d -= i * mine;
                const uint32_t of = rec[1 + 2 * i].y;
                const uint32_t where[1] = {live ? (((of % kStripRing) * groups + group) * S + rank + d * group_blocks) * kStripGroupBlocks + part : 0};
                const uint32_t number[1] = {live ? of : 0};
                float v[1];
                wait_words<1>(a.words, where, number, v, given_up);
                const float sum = group_sum(v[0], log_group);
                if (part == 0 && live) put_word(p.sums, ((of % kStripRing) * groups + group) * p.sum_pitch + rank + d * group_blocks, sum, of);
            }
        }
        // few pairs take few words: what is polled in vain makes a poll longer (all lanes without a word poll the same one)
        const int pairs = n_evals * kTeamHelpers;
        if (n_evals > 0 && pairs <= 2 * pair_step) {
            finish_pairs(rec, 0, n_evals, std::integral_constant<int, 2>{});
        } else {
            for (int from = 0; from < pairs; from += kWordsInFlight * pair_step) finish_pairs(rec, from, n_evals, std::integral_constant<int, kWordsInFlight>{});
        }
        if (given_up) lost_s = 1;
        __syncthreads();

        if (kGate && t == 0) published_s[it & 1] = 0;
        // ---- C: indices and record of the iterations after the next (what a helper loads here has arrived when the next
        // waits of phase B begin)
        fetch_index(rec_s[(it + 2) & 3]);
        if (copies) ahead = recs[static_cast<int64_t>(it + 3) * a.rec_len];
        if (copies_more) ahead_more = recs[static_cast<int64_t>(it + 3) * a.rec_len + 64];
        __syncthreads();
    }
    if (given_up) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (!kLds) return;
    if (inside && lost_s == 0) {      // a lost launch writes nothing back
        for (int r = 0; r < a.n; ++r) {
            a.X[r * a.ld + col] = xs[r * ld];
            if (kMom) a.V[r * a.ld + col] = vs[r * ld];
        }
        for (int i = a.n_in; i < a.n_in + a.n_out; ++i) a.slots[a.carry[2 * i + 1] * a.ld + col] = gs[a.carry[2 * i] * ld];
    }
}

template <int kTeams, int kRows, bool kLds, bool kMom>
void* strip_kernel(bool far) {
    return far ? reinterpret_cast<void*>(&strip_events_kernel<kTeams, kRows, kLds, kMom, true>)
               : reinterpret_cast<void*>(&strip_events_kernel<kTeams, kRows, kLds, kMom, false>);
}
template <int kTeams, int kRows>
hipError_t launch_rows(StripParams& p, hipStream_t st) {
    const StripArgs& a = p.a;
    const size_t lds = a.lds_state ? static_cast<size_t>(a.n * (a.V ? 2 : 1) + a.n_lds_slots) * kStripCols * 4 : 0;
    const bool far = p.blocks > p.group_size;          // several groups
    void* fn = a.lds_state ? (a.V ? strip_kernel<kTeams, kRows, true, true>(far) : strip_kernel<kTeams, kRows, true, false>(far))
                           : (a.V ? strip_kernel<kTeams, kRows, false, true>(far) : strip_kernel<kTeams, kRows, false, false>(far));
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
    void* args[] = {&p};
    return hipLaunchCooperativeKernel(fn, dim3(static_cast<uint32_t>(a.grid)), dim3(kStripThreads), args, lds, st);
}

int strip_samples(int model, int32_t M) { return M + (model == ADPSGD_MODEL_LOGREG ? 1 : 0); }

}  // namespace

int32_t strip_blocks(int64_t d) { return static_cast<int32_t>((d + kStripCols - 1) / kStripCols); }

// Up to 32 strips form one group; more are spread evenly over 8.
int32_t strip_group_size(int64_t d) {
    const int32_t blocks = strip_blocks(d);
    return blocks <= kStripGroupBlocks ? blocks : (blocks + kStripGroups - 1) / kStripGroups;
}

size_t strip_exchange_bytes(int model, int32_t M) {
    return static_cast<size_t>(kStripRing) * (strip_samples(model, M) * kStripGroupBlocks + ((strip_samples(model, M) + 15) & ~15)) * kStripGroups * sizeof(unsigned long long);
}

// LDS of a block: the kernel's fixed arrays and the state of the strip
size_t strip_lds_bytes(int32_t M, int32_t n, bool momentum, int32_t n_slots, bool lds_state) {
    const size_t fixed = (kStripMainWaves + strip_teams(M)) * 1024 + 4 * kStripMaxRec * sizeof(StripEntry) + kStripHelpers * 40 + 1024;
    return fixed + (lds_state ? (static_cast<size_t>(n) * (momentum ? 2 : 1) + n_slots) * kStripCols * 4 : 0);
}

hipError_t launch_strips(const StripArgs& a, hipStream_t st) {
    const int32_t blocks = strip_blocks(a.d);
    if (a.d > kStripMaxD || a.M < 1 || a.M > kStripMaxM || a.rec_len > kStripMaxRec || a.teams != strip_teams(a.M) || a.grid < blocks)
        return hipErrorInvalidValue;
    StripParams p;
    p.a = a;
    p.samples = a.loss ? strip_samples(a.model, a.M) : a.M;
    p.blocks = blocks;
    p.group_size = strip_group_size(a.d);
    p.sum_pitch = (p.samples + 15) & ~15;
    p.sums = a.words + static_cast<int64_t>(kStripRing) * strip_samples(a.model, a.M) * kStripGroups * kStripGroupBlocks;
    // Rows of a wavefront: the next of 4, 8, 12, 16 with teams of one or two wavefronts (M = 3: 231 us with 4 rows, 285 with 8), of 16, 18, 22
    // with teams of three or six.  18 where 22 would request 18 to 27 % in vain, for all M = 49 ... 54 and 97 ... 108, 200 events:
    // n = 8, d = 1500  M = 49, 54, 97, 108: 400, 449, 692, 719 us, with 22 rows 428, 465, 756, 770;  n = 12, d = 20 001  M = 49, 50, 54: 608,
    // 603, 615 and 627, 624, 633.  With two teams up to 160 strips: d = 20 001, 30 000, 40 001 1.04 ... 1.07, 1.01 ... 1.03, 1.01 ... 1.03 times as
    // fast as with 22 rows, 45 001 0.99 ... 1.0, 52 001 and 60 000 0.955 ... 1.0.
    switch (a.teams) {
        case 12: return a.M <= 4 ? launch_rows<12, 4>(p, st) : a.M <= 8 ? launch_rows<12, 8>(p, st) : a.M <= 12 ? launch_rows<12, 12>(p, st) : launch_rows<12, 16>(p, st);
        case 6: return a.M <= 24 ? launch_rows<6, 12>(p, st) : launch_rows<6, 16>(p, st);
        case 4: return a.M <= 48 ? launch_rows<4, 16>(p, st) : a.M <= 54 ? launch_rows<4, 18>(p, st) : launch_rows<4, 22>(p, st);
        default: return a.M <= 96 ? launch_rows<2, 16>(p, st) : a.M <= 108 && p.blocks <= 160 ? launch_rows<2, 18>(p, st) : launch_rows<2, 22>(p, st);
    }
}

}  // namespace adpsgd_impl
