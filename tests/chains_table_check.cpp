// The table of chains that the update kernels read (fill_chains), checked on the CPU: the kernels may request the inputs of
// every operation, so none may be missing while the workers of the events have data, also where an extra pair names a worker
// that has none; and an operation that steps has the inputs, slot, step size and rows of its event.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "internal.hpp"

using namespace adpsgd_impl;

namespace {

std::mt19937 rng(7);
int below(int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); }

[[noreturn]] void die(int trial, const char* what) {
    std::printf("trial %d: %s\n", trial, what);
    std::exit(1);
}

}  // namespace

int main() {
    long bare = 0, operations = 0;
    for (int trial = 0; trial < 3000; ++trial) {
        const int32_t n = 4 + below(12), T = below(6), n_slots = T + 1 + below(16), steppers = 1 + below(n - 2), chain = 1 + below(kChain);
        const int64_t K = 1 + below(60), A = K - below(static_cast<int>(std::min<int64_t>(K, T + 1)));
        std::vector<WorkerData> data(n);       // only the first `steppers` workers step, and have data
        for (int i = 0; i < steppers; ++i)
            data[i] = WorkerData{reinterpret_cast<const void*>(static_cast<uintptr_t>(0x1000 * (i + 1))), reinterpret_cast<const void*>(static_cast<uintptr_t>(8)), 3, 8 + i};
        std::vector<int32_t> worker, neighbour, tau, extra_a, extra_b;
        std::vector<int64_t> extra_ptr(1, 0);
        std::vector<float> gamma;
        for (int64_t k = 0; k < K; ++k) {
            worker.push_back(below(steppers));
            neighbour.push_back(below(n));
            tau.push_back(below(static_cast<int>(std::min<int64_t>(k, T)) + 1));
            gamma.push_back(static_cast<float>(k + 1));
            if (below(2)) {
                int32_t a, b;
                do {
                    a = below(n);
                    b = below(n);
                } while (a == b || a == worker[k] || b == worker[k] || a == neighbour[k] || b == neighbour[k]);
                extra_a.push_back(a);
                extra_b.push_back(b);
            }
            extra_ptr.push_back(static_cast<int64_t>(extra_a.size()));
        }
        Plan plan;
        std::string err;
        if (plan_rounds(n, K, worker.data(), neighbour.data(), tau.data(), n_slots, true, plan, err, extra_ptr.data(), extra_a.data(), extra_b.data(),
                        false, A, nullptr, chain) != 0)
            continue;
        std::vector<int64_t> offset(plan.n_rounds + 1, 0);
        for (int64_t k = 0; k < A; ++k) offset[plan.u_round[k] + 1] += 1 + extra_ptr[k + 1] - extra_ptr[k];
        for (int32_t r = 0; r < plan.n_rounds; ++r) offset[r + 1] += offset[r];
        const bool per_event = below(2) != 0;
        const ChainCall call{n, A, worker.data(), neighbour.data(), extra_ptr.data(), extra_a.data(), extra_b.data(), per_event ? gamma.data() : nullptr, 0.5f,
                             &plan, data.data(), &offset};
        std::vector<ColumnPair> pairs;
        ChainLayout layout;
        std::vector<UpdateChain> chains;
        std::vector<int64_t> events;
        chain_pairs(call, pairs);
        chain_rounds(pairs, offset, n, layout);
        if (!verify_chains(pairs, offset, n, chain, layout) || !fill_chains(call, pairs, layout, chain, chains, events)) die(trial, "no table");
        for (const UpdateChain& ch : chains) {
            for (int u = 0; u < kChain; ++u)
                if (!ch.ops[u].features || ch.ops[u].feat_ld < 8) die(trial, "an operation without inputs");
            for (int u = 0; u < ch.n_ops; ++u) {
                const UpdateOp& op = ch.ops[u];
                const ColumnPair& pair = pairs[layout.order[ch.first + u]];
                ++operations;
                bare += !data[pair.i].features;
                if (op.event != pair.event || events[ch.first + u] != pair.event) die(trial, "an operation of the wrong event");
                if (ch.rows[op.places & 15] != pair.i || ch.rows[op.places >> 4] != pair.j) die(trial, "an operation on the wrong rows");
                if (op.event < 0) continue;
                if (op.features != data[pair.i].features || op.feat_ld != data[pair.i].ld) die(trial, "the wrong inputs");
                if (op.slot != plan.slot[op.event] || op.gamma != (per_event ? gamma[op.event] : 0.5f)) die(trial, "the wrong gradient or step size");
                if ((ch.steps >> (op.places & 15) & 1) == 0) die(trial, "a step without its momentum");
            }
        }
    }
    if (bare == 0) die(0, "no extra pair of a worker without data");
    std::printf("ok, operations %ld, of workers without data %ld\n", operations, bare);
}
