// Layouts of the strip kernel whose holders request and use rows in one record (fewer holders than `teams`), checked on the
// CPU: random schedules through plan_rounds, build_strips and verify_strips; then a request is moved behind the evaluation that
// needs it, and verify_strips has to find it.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "strips.hpp"

using namespace adpsgd_impl;

int main() {
    std::mt19937 rng(5);
    auto below = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    long iterations = 0, ahead = 0, at_once = 0, planted = 0;
    for (int trial = 0; trial < 3000; ++trial) {
        const int n = 2 + below(20), K = 1 + below(200), T = below(20), n_slots = T + 1 + below(64);
        const bool compensate = below(3) == 0, renumber = below(2) == 0;
        std::vector<int32_t> worker, neighbour, tau;
        for (int k = 0; k < K; ++k) {
            worker.push_back(below(n));
            neighbour.push_back(below(n));
            tau.push_back(below(std::min(k, T) + 1));
        }
        std::vector<WorkerData> data(n);
        for (int i = 0; i < n; ++i) data[i] = WorkerData{reinterpret_cast<const void*>(static_cast<uintptr_t>(0x1000 + i)), reinterpret_cast<const void*>(static_cast<uintptr_t>(0x2000 + i)), 3, 5};
        Plan plan;
        std::string err;
        if (plan_rounds(n, K, worker.data(), neighbour.data(), tau.data(), n_slots, true, plan, err, nullptr, nullptr, nullptr, compensate) != 0) continue;
        const StripCall call{n, n_slots, strip_window(T, renumber, 64, n_slots), K, K, worker.data(), neighbour.data(), tau.data(), nullptr, 0.5f, nullptr, nullptr, nullptr,
                             &plan, nullptr, data.data(), renumber, 7u, 3};
        const int evals[4] = {12, 6, 4, 2}, teams = 2 * evals[trial % 4];
        StripProgram p, twice;
        if (!build_strips(call, teams, p, teams / 2) || !build_strips(call, teams, twice, teams)) {
            std::printf("trial %d: no order\n", trial);
            return 1;
        }
        if (!verify_strips(call, p, err) || !verify_strips(call, twice, err) || p.iterations != twice.iterations) {
            std::printf("trial %d: %s, %ld and %ld iterations\n", trial, err.c_str(), static_cast<long>(p.iterations), static_cast<long>(twice.iterations));
            return 1;
        }
        iterations += p.iterations;
        for (int64_t it = 0; it < p.iterations; ++it) {
            at_once += __builtin_popcount(p.recs[it * p.rec_len].y & p.recs[it * p.rec_len].z);
            ahead += __builtin_popcount(twice.recs[it * p.rec_len].y & twice.recs[it * p.rec_len].z);
        }
        for (int64_t it = 0; it + 1 < p.iterations; ++it) {
            StripEntry *rec = &p.recs[it * p.rec_len], *next = rec + p.rec_len;
            const uint32_t both = rec[0].y & rec[0].z;
            if (__builtin_popcount(rec[0].y) != 1 || both == 0 || next[0].y != 0) continue;
            std::swap(rec[0].y, next[0].y);              // requested in the record after
            for (int e = 0; e < 2; ++e) std::swap(rec[1 + teams + e], next[1 + teams + e]);
            if (verify_strips(call, p, err)) {
                std::printf("trial %d: a late request not found\n", trial);
                return 1;
            }
            ++planted;
            break;
        }
    }
    if (ahead != 0 || at_once == 0 || planted == 0) {
        std::printf("requests at once %ld and %ld, planted %ld\n", at_once, ahead, planted);
        return 1;
    }
    std::printf("ok, iterations %ld, requests at once %ld, planted %ld\n", iterations, at_once, planted);
}
