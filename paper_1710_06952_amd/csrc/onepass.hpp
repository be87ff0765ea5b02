// Interface of the linear gradients in one pass over the minibatch rows (kernels_onepass.hip).
#pragma once

#include "internal.hpp"

namespace adpsgd_impl {

constexpr int kOnePassThreads = 512;
constexpr int kOnePassWaves = kOnePassThreads / 64;
constexpr int kOnePassMaxM = 128;
constexpr int kOnePassMaxStrips = 256;
// How long a block waits for the others before it leaves the exchange.  Where the others come late because other work holds
// compute units, a longer wait is lost, once by the blocks that are there and once by each that comes later (1000, 300 and 100 us:
// 4.2, 4.2, 4.0 and 4.6, 4.5, 4.1 ms at take_tickets).  The first launch of a process may need it, though: with data that the
// device has not touched yet (M = 4, d = 327 679, five workers) some blocks of a group come more than 100 us after the others.
constexpr int64_t kOnePassWaitUs = 300;
// Bytes of a gradient's rows from which on the kernels for large ones take it, twice as many with 6 rows a wavefront (measured at onepass_shape).
constexpr double kOnePassLargeBytes = 8e6;
enum class OnePassKernel : int32_t { kPlain, kPipeline, kStaged };

// How a gradient lies on the chip: its columns in `strips` strips of one block each, the rows of a strip over
// `row_groups` groups of wavefronts with `rows` rows each, the strip's columns over 8 / row_groups wavefronts of `chunks` times
// 256 columns, of which the first `wave_cols` are in use; `groups` gradients at a time.
struct OnePassShape {
    int32_t rows = 0, chunks = 0, row_groups = 0, strips = 0, groups = 0, wave_cols = 0;
    OnePassKernel kernel = OnePassKernel::kPlain;
    bool ok() const { return strips > 0; }
    constexpr __host__ __device__ int32_t ring() const { return kernel == OnePassKernel::kPipeline ? 2 : 1; }     // gradients in the exchange
};
constexpr int64_t onepass_group_words(const OnePassShape& s, int32_t samples) {
    return static_cast<int64_t>(samples) * (s.ring() * (s.strips + 2) + s.strips + 1) + 2;
}
// Rows and chunks of the kernels that are built, and which of the three for them.
struct OnePassHeld {
    int rows, chunks;
};
constexpr OnePassHeld kOnePassHeld[] = {{2, 4}, {2, 8}, {4, 2}, {4, 4}, {4, 8}, {6, 1}, {6, 2}, {6, 5}, {6, 6}, {6, 8}, {8, 1},
                                        {8, 2}, {8, 4}, {8, 5}, {8, 6}, {12, 1}, {12, 2}, {12, 3}, {12, 4}, {16, 1}, {16, 2}, {16, 3}};
constexpr int onepass_pipeline_chunks(int rows) { return rows <= 4 ? 8 / rows : rows <= 8 ? 2 : 1; }      // two gradients of them fit
constexpr bool onepass_built(OnePassKernel kernel, int rows, int chunks) {
    return kernel == OnePassKernel::kPipeline ? chunks == onepass_pipeline_chunks(rows)
           : kernel == OnePassKernel::kStaged ? rows * chunks > (rows == 2 ? 8 : rows == 12 ? 32 : 16)
                                              : rows * chunks <= 32;
}
// The shape for a handle, by its sizes alone (so that a gradient has the same bits in every call and however its blocks are
// scheduled), or one that is not ok():
// three launches per round (kernels_grad_linear.hip) are the better route, or the only one.
// at_once: gradients of every launch, where that is known (the synchronous schedule), else 0.
OnePassShape onepass_shape(int model, int64_t d, int32_t M, int32_t compute_units, int32_t at_once = 0);
// Whether run_events takes it too (the synchronous schedule does wherever there is a shape).
bool onepass_for_events(const OnePassShape& s, int model, int32_t M, bool wait_free);
size_t onepass_exchange_bytes(const OnePassShape& s, int32_t M);

// Sums of a gradient that the blocks exchange: one per sample, and |x^|^2 for the logistic loss.
constexpr int32_t onepass_samples(int model, int32_t M, bool loss) { return M + (model == ADPSGD_MODEL_LOGREG && loss ? 1 : 0); }
// Of these, how many have to be finished before a block may publish sums of its next gradient in the same words: all.  One
// that is not awaited could be overwritten under the block that adds it up.
constexpr __host__ __device__ int32_t onepass_awaited(int32_t samples) { return samples; }

// The pipeline's flags for a wait that ended in vain, by turn.  A turn looks at its flag behind the barrier of step 1, and no barrier
// stands between that look and its wait for the sums: what this wait raises is the next turn's flag, or a wavefront that has
// not looked yet would leave a turn before the others.
constexpr __host__ __device__ int late_seen(int turn) { return turn & 1; }
constexpr __host__ __device__ int late_of_coefficients(int turn) { return late_seen(turn); }
constexpr __host__ __device__ int late_of_sums(int turn) { return late_seen(turn + 1); }

struct OnePassArgs {
    OnePassShape shape;
    int model;
    const float* X;
    int64_t ld, d;
    const GradOp* ops;          // device
    int32_t n_ops, M;
    const int32_t* batch_idx;   // device, by event
    float* slots;
    float gscale, lambda;
    float* loss;                // device, by event, or nullptr
    unsigned long long* words;  // onepass_exchange_bytes, zero before the first launch
    unsigned long long* late;   // counts the blocks that leave the exchange
    int* status;                // set when the launch is lost
    uint32_t seq0;              // sequence number of the first gradient; n_ops of them are used
    uint64_t wait_ticks;        // of the constant clock
};
hipError_t launch_onepass_gradient(const OnePassArgs& a, hipStream_t st);

}  // namespace adpsgd_impl
