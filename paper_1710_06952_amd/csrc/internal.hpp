// Internal declarations shared by the host-side translation units of libadpsgd.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>
#include <vector>

#include "adpsgd.h"

namespace adpsgd_impl {

// One update event as the fused gossip-average + apply kernel sees it.
struct alignas(32) PairOp {
    int32_t i;        // worker i_k (takes the gradient step)
    int32_t j;        // neighbour j_k (i == j: no partner, plain SGD step)
    uint32_t k_lo;    // global event number (addresses the synthetic-gradient generator)
    uint32_t k_hi;
    float gamma;
    int32_t slot;     // pending-gradient slot holding g_k (data models)
    int32_t flags;    // bit 0: average only (an extra pair of a general W_k): no gradient, no step
    int32_t pad;
};

// Updates of a round that share rows, executed one after the other (chain_rounds).
constexpr int kChain = 4;               // operations of a chain, at most; they touch one row more
// ... of the perceptron: with momentum buffers the rows of a longer chain do not fit the registers, and the larger the model, the more
// the kernel for four costs where chains of four save no round (T_max = 0, many workers).  Four against three: 36 set-ups up to 2^18
// parameters 0.97 ... 1.06 times as fast;  24 from there to 684 000  0.995 ... 1.08 with stale gradients, 0.965 ... 1.04 without;  728 650
// 0.998 and 1.045, 814 090 0.975 and 1.017 (M = 64 and 32).
constexpr int mlp_chain(bool momentum, int64_t d) { return momentum || d > (1 << 18) ? 3 : kChain; }
struct UpdateOp {
    const void* features;               // worker i's inputs (average only: those of a worker that has some, read and dropped), or nullptr
    int64_t feat_ld;
    int32_t slot;
    float gamma;
    int32_t places;                     // of rows i and j (bits 4 and up) in the chain's rows
    int32_t event;                      // index into the call's arrays; -1: an extra pair of a general W_k, no gradient, no step
};
struct alignas(32) UpdateChain {
    int32_t first, n_ops;               // position of the first operation in the order of the chains
    int32_t rows[kChain + 1];           // -1: none
    int32_t steps;                      // places whose row takes a gradient step (bits): their momentum is read and written
    UpdateOp ops[kChain];               // beyond n_ops: the last one again (its operands may be requested, and dropped)
};

// One stale read / gradient evaluation as the gradient kernels see it.
struct GradOp {
    int32_t worker;   // row read, and owner of the local data
    int32_t slot;     // where g_k goes
    int32_t event;    // index into the call's batch_idx / loss arrays
    int32_t comp_slot;   // wait-free variant: slot of the worker's own pending gradient g_k', or -1
    float comp_gamma;    // its step size: the read is x^ = row - comp_gamma * g_k'
    int32_t count;    // loss evaluation only: samples of the operation that count (the rest is padding)
    const void* features;   // the worker's local data (device), copied here so that a kernel reaches
    const void* targets;    //   it with one load instead of a second table look-up
    int64_t ld;             // leading dimension of features, in elements
    const void* xrow_bf16;  // perceptron, wait-free variant: bf16 row the gradient reads instead of the worker's
                            //   shadow (the compensated copy x - gamma_k' g_k'), or nullptr
};

// constants of the counter-based generator (Philox4x32): multipliers, key increments, stream of the gradients
constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;
constexpr uint32_t kStreamGrad = 2u << 24;

// std sqrt(2 ln 2) in two parts, the standard deviation of the synthetic gradients as the kernels take it; refine: std is a power
// of two, up to its sign (box_muller).
struct SynthScale {
    float hi, lo;
    bool refine;
};
inline SynthScale synth_scale(float std) {
    const double exact = static_cast<double>(std) * 1.1774100225154747;
    const float hi = static_cast<float>(exact);
    int exponent = 0;
    return SynthScale{hi, std::isfinite(hi) ? static_cast<float>(exact - static_cast<double>(hi)) : 0.0f, std::fabs(std::frexp(std, &exponent)) == 0.5f};
}

// One operation of the column kernel (kernels_columns.hip): an event of the synthetic model or an extra pair.
constexpr uint32_t kColumnEvent = 1, kColumnAverage = 2;
struct alignas(32) ColumnOp {
    uint32_t rows;      // places of rows i and j (upper half) in a strip, in bytes
    uint32_t flags;     // 0: empty, kColumnEvent, kColumnAverage
    float gamma;
    uint32_t a, b, c, d;   // what the first two Philox rounds take from the event number (see column_words)
    uint32_t pad;
};

struct WorkerData {
    const void* features = nullptr;
    const void* targets = nullptr;
    int64_t rows = 0;
    int64_t ld = 0;
};

struct Plan {
    std::vector<int32_t> r_round, u_round, slot;
    std::vector<int64_t> prev;   // wait-free variant: event whose pending gradient compensates the read, or -1
    int32_t n_rounds = 0;
};

// Grow-only device buffer owned by the library (small tables only).
struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
    hipError_t reserve(size_t bytes);
    void release();
};

// ---- host logic ------------------------------------------------------------
void philox4x32_10_host(const uint32_t ctr[4], const uint32_t key[2], uint32_t out[4]);
int plan_rounds(int32_t n, int64_t K, const int32_t* worker, const int32_t* neighbour,
                const int32_t* tau, int32_t n_slots, bool with_gradients, Plan& plan,
                std::string& err, const int64_t* extra_ptr = nullptr, const int32_t* extra_a = nullptr,
                const int32_t* extra_b = nullptr, bool local_compensation = false,
                int64_t n_apply = -1, const int32_t* carried_slot = nullptr, int32_t chain = 1);
bool verify_plan(int32_t n, int64_t K, const int32_t* worker, const int32_t* neighbour, const int32_t* tau,
                 int32_t n_slots, bool with_gradients, const Plan& plan, std::string& err,
                 const int64_t* extra_ptr = nullptr, const int32_t* extra_a = nullptr, const int32_t* extra_b = nullptr,
                 int64_t n_apply = -1, const int32_t* carried_slot = nullptr, bool chained = false);
bool graph_ok(const adpsgd_graph_t* g, std::string& err);

// ---- kernel launchers (each returns the hipError_t of the launch) ------------
struct FusedArgs {
    float* X;
    int64_t ld;
    int64_t d;
    const PairOp* ops;   // device
    int32_t n_ops;
    const float* slots;  // device, slot s at slots + s * ld (data models)
    float synth_std;
    uint64_t synth_seed;
    bool synth;
    bool streaming;      // rows do not fit the caches: bypass them
    bool has_solo;       // some event of the round has i == j (worker without a neighbour)
    float* V;            // device momentum buffers (n x ld) or nullptr: plain event
    float momentum;
    float weight_decay;
};
hipError_t launch_fused_gossip_apply(const FusedArgs& a, hipStream_t st);

// The updates of a round with dense gradients, in chains.
struct ChainArgs {
    float* X;
    int64_t ld, d;
    const UpdateChain* chains;      // device
    int32_t n_chains;
    const float* slots;
    bool streaming;         // X does not fit the caches
    float* V;               // momentum buffers or nullptr
    float momentum, weight_decay;
};
hipError_t launch_gossip_chains(const ChainArgs& a, hipStream_t st);

struct ColumnArgs {
    float* X;
    float* V;               // momentum buffers or nullptr
    int64_t ld, d;
    const ColumnOp* ops;    // device, [batches + 2][64 / quads]
    const int32_t* rows;    // device, the rows of X that the operations name
    int32_t n_rows, batches;
    int32_t quads;          // float4 columns per wavefront: 4, 8, 16, 32 or 64
    uint64_t synth_seed;
    float synth_std;
    float momentum, weight_decay;
    bool averages;          // some operations average only (extra pairs of a general W_k)
};
hipError_t launch_column_events(const ColumnArgs& a, hipStream_t st);

// Averaging and update operations of a call in the order of its events, for the column kernel.
struct ColumnPair {
    int32_t i, j;           // local row numbers
    int64_t event;          // index of the event in the call, or -1: averaging only
};
// The operations of every round (pairs[offset[r] .. offset[r + 1]), in event order) by chains: those connected by their rows.
struct ChainLayout {
    std::vector<int64_t> order;     // operations, chain after chain
    std::vector<int64_t> first;     // per chain: where it begins in `order` (and the end)
    std::vector<int64_t> round;     // per round: its first chain (and the end)
};
void chain_rounds(const std::vector<ColumnPair>& pairs, const std::vector<int64_t>& offset, int32_t n_rows, ChainLayout& out);
// Whether a layout keeps the order of every row and has at most `most` operations in a chain (ADPSGD_FLAG_VERIFY_PLAN).
bool verify_chains(const std::vector<ColumnPair>& pairs, const std::vector<int64_t>& offset, int32_t n_rows, int32_t most, const ChainLayout& c);
// The updates of a call, for the two functions below.
struct ChainCall {
    int32_t n;
    int64_t A;                      // events applied
    const int32_t *worker, *neighbour;
    const int64_t* extra_ptr;       // or nullptr
    const int32_t *extra_a, *extra_b;
    const float* gamma;             // per event, or nullptr: gamma_default
    float gamma_default;
    const Plan* plan;
    const WorkerData* data;         // by worker; the workers of the events have some, or none has
    const std::vector<int64_t>* offset;     // first update operation of every round (and the end)
};
// Its operations in the order of the rounds, as chain_rounds takes them.
void chain_pairs(const ChainCall& c, std::vector<ColumnPair>& pairs);
// The chains as the update kernels take them, and the event of every operation in their order (-1: averaging only).
// false: a chain has more than `most` operations.
bool fill_chains(const ChainCall& c, const std::vector<ColumnPair>& pairs, const ChainLayout& layout, int32_t most,
                 std::vector<UpdateChain>& chains, std::vector<int64_t>& events);
// Packs the operations into batches of `capacity` with pairwise disjoint rows such that the operations of every row
// keep their order from batch to batch: every operation goes into the first batch with room behind those of its rows.
// place[t] = batch * capacity + position; returns the number of batches.
int64_t pack_columns(const std::vector<ColumnPair>& pairs, int32_t n_rows, int32_t capacity, std::vector<int64_t>& place);
// Whether such a packing keeps the semantics (ADPSGD_FLAG_VERIFY_PLAN): places of their own, the rows of a batch pairwise
// different, the operations of every row in order from batch to batch.
bool verify_columns(const std::vector<ColumnPair>& pairs, int32_t n_rows, int32_t capacity, const std::vector<int64_t>& place, int64_t batches);
// Words a..d of an event's ColumnOp: with the counter (quad, 0, k_lo, k_hi) the first Philox round gives
//   (hi(M1 k_lo) ^ key0, lo(M1 k_lo), hi(M0 quad) ^ a, lo(M0 quad))
// and the second   (hi(p) ^ b, lo(p), lo(M0 quad) ^ c, d)   with p = M1 (hi(M0 quad) ^ a).
void column_words(uint64_t event, uint64_t seed, ColumnOp& op);

struct LinearGradArgs {
    int model;              // LSQ or LOGREG
    const float* X;
    int64_t ld;
    int64_t d;
    const GradOp* ops;      // device, this group's ops
    int32_t n_ops;
    int32_t M;
    const int32_t* batch_idx;  // device, K x M
    float* slots;
    float gscale;           // 1/M or 1
    float lambda;
    float* partial;         // device scratch: n_ops x (M + 1) x n_chunks
    float* coef;            // device scratch: n_ops x M
    float* loss;            // device, indexed by event, or nullptr
    bool factored;          // least squares: leave g as its M coefficients (start of the slot), no combine launch
};
int64_t linear_grad_chunks(int64_t d);
bool linear_can_factor(int model, int64_t d, int32_t M, int64_t ld);

// The updates of a round with the least-squares gradients still in factored form (see the kernel).
struct LinearApplyArgs {
    float* X;
    int64_t ld;
    int64_t d;
    const UpdateChain* chains;      // device; features / feat_ld / event / slot name the factors
    int32_t n_chains;
    const float* slots;
    const int32_t* batch_idx;
    int32_t M;
    bool streaming;         // X does not fit the caches
    float* V;               // momentum buffers or nullptr
    float momentum, weight_decay;
};
hipError_t launch_linear_apply_chains(const LinearApplyArgs& a, hipStream_t st);
hipError_t launch_linear_gradient(const LinearGradArgs& a, hipStream_t st, int* n_launches);

struct MlpGradArgs {
    const float* X;         // device fp32 master, n x ld (read by the wait-free variant only)
    const uint16_t* Xbf16;  // device bf16 shadow, n x ld
    int64_t ld;
    int32_t in, hid, out;
    const GradOp* ops;
    int32_t n_ops;
    int32_t M;
    const int32_t* batch_by_op;   // device, n_ops x M: row t holds the minibatch indices of ops[t] (a kernel finds them
                                  //   from its block index, without waiting for the operation's descriptor)
    float* slots;
    float gscale;
    float* loss;
    void* scratch;          // device scratch, mlp_scratch_bytes(n_ops, ...)
    bool factored;          // leave dW1 as its factors: dH goes to the start of the slot, no dW1 launch
    bool compensate;        // wait-free variant: first build the compensated bf16 rows the operations name
};
size_t mlp_scratch_bytes(int32_t n_ops, int32_t M, int32_t in, int32_t hid, int32_t out);
// forward pass and cross-entropy only: loss_sum[op] = sum over the first `count` samples of the operation (fp64);
// count_errors: the number of those samples whose largest logit (lowest class on ties) is not their label instead
hipError_t launch_mlp_loss(const MlpGradArgs& a, double* loss_sum, bool count_errors, hipStream_t st);
bool mlp_can_factor(int32_t in, int32_t hid, int32_t M);

// The perceptron's model update, with the first-layer gradient still in factored form where that is possible
// (dW1 = Xb^T dH, rank <= M): the product is formed tile by tile on the matrix cores inside
// the update kernel instead of being written to and read back from the pending slot.
struct MlpApplyArgs {
    float* X;
    int64_t ld;
    int64_t d;
    int32_t in, hid, M;
    const UpdateChain* chains; // device
    int32_t n_chains;
    const float* slots;
    uint16_t* Xbf16;
    const int32_t* batch_by_op; // device, rows of M: the minibatch indices of the chains' operations (factored)
    bool factored;              // dW1 as its factors, else the whole gradient is in the slot
    float* V;                   // momentum buffers or nullptr
    float momentum, weight_decay;
};
hipError_t launch_mlp_apply_chains(const MlpApplyArgs& a, hipStream_t st);
hipError_t launch_mlp_gradient(const MlpGradArgs& a, hipStream_t st, int* n_launches);

struct SyncArgs {
    float* X;
    int64_t ld;
    int64_t d;
    int32_t n;
    const int32_t* rowptr;   // device
    const int32_t* col;      // device
    const float* w_self;     // device
    const float* w_edge;     // device
    const float* slots;      // gradient of worker i in slot i, or nullptr with synth
    uint16_t* Xbf16;         // bf16 shadow to refresh, or nullptr
    float gamma;
    float synth_std;
    uint64_t synth_seed;
    uint64_t event0;         // synthetic gradients: worker i draws event event0 + i
    bool synth;
    float* V;                // momentum buffers or nullptr
    float momentum, weight_decay;
    bool ring;               // the graph is a ring with neighbour lists (i - 1, i + 1) mod n, n >= 3: no LDS staging needed
    float* Xdst = nullptr;   // write the new models to this matrix (same ld, not X) instead of in place
};
int32_t sync_tile_cols(int32_t n);   // 0: n too large for the in-place mixing kernel
bool sync_out_of_place_ok(int32_t n, int64_t d);   // the launch geometry of the out-of-place kernels exists
hipError_t launch_sync_mix_apply(const SyncArgs& a, hipStream_t st);

hipError_t launch_broadcast_rows(float* X, int64_t ld, int64_t d, int32_t n, const float* x0, hipStream_t st);
hipError_t launch_refresh_bf16(const float* X, uint16_t* Xb, int64_t ld, int32_t n, hipStream_t st);
hipError_t launch_mean_model(const float* X, int64_t ld, int64_t d, int32_t n, float* out, hipStream_t st);
int32_t consensus_blocks(int64_t d);
// adpsgd_consensus_distance_static: capacity of the library's fixed device array (block partials, worker
// probabilities) and its address on the current GPU (resolved on the first call per device)
constexpr int kStaticPartials = 2048;
constexpr int kStaticWeights = 4096;
hipError_t static_scratch(double** out);
// p: device, n doubles (the workers' update probabilities, psum their sum), or nullptr for the uniform weights 1 / n
hipError_t launch_consensus(const float* X, int64_t ld, int64_t d, int32_t n, double* partial,
                            double* result, const double* p, double psum, hipStream_t st);
hipError_t launch_count_nonfinite(const float* X, int64_t ld, int64_t d, int32_t n, unsigned long long* partial,
                                  int32_t blocks, hipStream_t st);
// one worker's local data as the objective kernel sees it
struct ObjectiveWorker {
    const void* features;
    const void* targets;
    int64_t rows;
    int64_t ld;
};
int64_t objective_row_groups(int64_t max_rows);
hipError_t launch_objective(int model, const float* x, int64_t d, int32_t n, const ObjectiveWorker* workers, int64_t max_rows,
                            float lambda, double* partial, double* result, bool count_errors, const double* weights,
                            hipStream_t st);   // weights: device, n probabilities, or nullptr for 1 / n
// out[t] (ld floats each) = X[ops[t].worker] - comp_gamma * slot[comp_slot] for the compensated operations of a group
hipError_t launch_compensated_rows(const float* X, int64_t ld, const GradOp* ops, int32_t n_ops, const float* slots, float* out,
                                   hipStream_t st);
hipError_t launch_synth_gradient(uint64_t seed, uint64_t k, float std, int64_t d, float* out, hipStream_t st);

}  // namespace adpsgd_impl
