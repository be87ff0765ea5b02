// Interface between the host code that lays a call of a linear model out as one persistent launch
// (strips.cpp) and the kernel that executes it (kernels_strips.hip).
#pragma once

#include <algorithm>
#include <string>

#include "internal.hpp"

namespace adpsgd_impl {

constexpr int kStripCols = 256;          // columns of the models a block owns
constexpr int kStripMainWaves = 12;      // wavefronts that hold minibatch rows, split evenly over the teams
constexpr int kStripHelpers = 256;       // further threads, one per column: models, slots, exchange
constexpr int kStripRing = 32;           // exchanges whose words are kept (more than twice the teams)
constexpr int kStripGroups = 8;          // groups of blocks that sum among themselves first (one per XCD) ...
constexpr int kStripGroupBlocks = 32;    // ... and blocks in a group, at most
constexpr int kStripCounters = 16;       // words that the blocks count themselves with, zero before the launch
constexpr int kStripMaxRec = 80;         // entries of a record (up to 128: two per lane of the wavefront that copies them)
constexpr int64_t kStripMaxD = kStripGroups * kStripGroupBlocks * kStripCols;    // at most one block per compute unit
constexpr int32_t kStripMaxM = 128;
constexpr int kStripLdsBytes = 160 * 1024;
constexpr uint64_t kClockTicksPerUs = 100;      // the constant clock of the device, 100 MHz on gfx950

// A record is one iteration of the kernel: a header, two entries for each of up to teams / 2 evaluations, two for each of
// as many loads (both in the order of their holders), then the updates.  A holder is a set of registers for the rows of one
// gradient.  An iteration requests rows before it evaluates, so a holder may do both in one record: teams / 2 holders are
// enough (with as many as `teams` all rows would be requested an iteration ahead).  All fields are 32-bit words.
//   header            updates, holders that load (bit mask), holders that evaluate (bit mask), -
//   evaluation        holder, sequence number of the gradient, worker read, slot the gradient goes to;
//                     slot of the pending gradient that compensates the read (or -1), its step size, the event, the
//                     strip that writes its loss
//   load              position in the index table, row pitch of the features, features (64 bits);  targets (64 bits), -, -
//   update            row i | row j << 16, slot, step size, flags; within a batch of kStripBatch all rows are different
constexpr int kStripBatch = 4;
constexpr uint32_t kStripAverage = 1, kStripEmpty = 2;      // flags of an update: averaging only; no update
struct alignas(16) StripEntry {
    uint32_t x, y, z, w;
};
// The iterations of a call, laid out by build_strips.
struct StripProgram {
    int32_t teams = 0, holders = 0, rec_len = 0;       // teams: twice the evaluations of a record
    int64_t iterations = 0;
    std::vector<StripEntry> recs;        // (iterations + 3) x rec_len, the last three empty
    std::vector<int64_t> order;          // events in the order their gradients are evaluated (rows of the index table)
    std::vector<int32_t> slot;           // per event: slot inside the call (-1: none)
    int32_t n_slots = 0;                 // slots used inside the call
};

struct StripCall {
    int32_t n, n_slots;    // workers, slots of the workspace
    int32_t window;        // strip_window
    int64_t K, A;          // events in the arrays, events applied
    const int32_t *worker, *neighbour, *tau;
    const float* gamma;                  // per event or nullptr
    float gamma_default;
    const int64_t* extra_ptr;
    const int32_t *extra_a, *extra_b;
    const Plan* plan;
    const int32_t* carried_slot;         // per event or nullptr
    const WorkerData* data;
    bool renumber;                       // slots of the call numbered from 0 by lifetime (they live in LDS)
    uint32_t seq0;                       // sequence number of the first gradient
    int32_t strips;                      // blocks with a strip
};
// Teams of wavefronts (gradients whose rows are held) for a minibatch of M samples: as many as their rows leave
// registers for (at most 22 rows of a wavefront).  A record evaluates as many gradients.
inline int32_t strip_teams(int32_t M) { return M <= 16 ? 12 : M <= 32 ? 6 : M <= 64 ? 4 : 2; }
// Gradients run at most this many events ahead of the first event not applied: as many as there are slots for, 64 at most
// and T_max + 1 at least.  In LDS slots_fit slots fit (lds_state: more than T_max); in the workspace there are n_slots, which
// may be fewer than T_max + 1 (the library uses 4096 at most): more than the largest tau of the call all the same, or there is
// no plan, and that is all the order needs.
inline int32_t strip_window(int64_t T_max, bool lds_state, int64_t slots_fit, int32_t n_slots) {
    return static_cast<int32_t>(lds_state ? std::max<int64_t>(T_max + 1, std::min<int64_t>(64, slots_fit))
                                          : std::min<int64_t>(n_slots, std::max<int64_t>(T_max + 1, 64)));
}
// false: the events do not come in any order (the plan is not one of this schedule), or there is no slot for a gradient
// teams: twice the evaluations of a record; holders: as many, or at least half (0: as many)
bool build_strips(const StripCall& c, int32_t teams, StripProgram& out, int32_t holders = 0);
// Executes the records on paper and compares with the serial semantics (ADPSGD_FLAG_VERIFY_PLAN): every read sees exactly
// the updates before its logical time and the pending gradient it is compensated with, every update finds its gradient and
// keeps the order of its rows, a batch of updates names a row once, minibatch rows are requested before they are used, for a
// holder that is idle, and no slot is given away early.
bool verify_strips(const StripCall& c, const StripProgram& p, std::string& err);

struct StripArgs {
    float* X;
    float* V;                // momentum buffers or nullptr
    int64_t ld, d;
    int32_t n;
    int model;               // LSQ or LOGREG
    int32_t M, teams;        // teams of wavefronts (strip_teams): the evaluations of a record, half the program's teams
    const StripEntry* recs;  // device
    int32_t rec_len, iterations;
    const int32_t* idx;      // device, minibatch indices in the order of evaluation
    const int32_t* carry;    // device: n_in + n_out pairs (slot of the call, slot of the workspace)
    int32_t n_in, n_out;
    float* slots;            // the workspace
    float* alone_slots;      // lds_state: place of the call's slots, n_lds_slots x ld, for a block that executes the call alone
    uint32_t seq0;           // sequence number of the first gradient
    int32_t n_lds_slots;
    bool lds_state;          // models, momentum buffers and slots of the strip live in LDS
    unsigned long long* words;    // exchange memory: strip_exchange_bytes
    unsigned int* counters;  // device, kStripCounters zeros
    int32_t grid;            // blocks to launch, at least one per strip
    float gscale, lambda, momentum, weight_decay;
    float* loss;             // device, indexed by event, or nullptr
    int* status;             // pinned host word, set when an exchange never completes
    const StripArgs* self;   // device: these arguments, for a block that executes the call alone
    uint64_t wait_ticks;     // how long the blocks wait until all are resident (constant clock); then one goes alone
    bool lose;               // wait for no word of the exchange: the launch ends as lost
};
int32_t strip_blocks(int64_t d);
int32_t strip_group_size(int64_t d);
size_t strip_exchange_bytes(int model, int32_t M);
size_t strip_lds_bytes(int32_t M, int32_t n, bool momentum, int32_t n_slots, bool lds_state);
hipError_t launch_strips(const StripArgs& a, hipStream_t st);

}  // namespace adpsgd_impl
