// The layouts of calls that go in one launch, checked on the CPU.
//   strips    random schedules (stale reads, carried and looked-ahead events, extra pairs, the wait-free variant, few slots,
//             a T_max beyond the slots, all numbers of teams) through plan_rounds, build_strips and verify_strips; then one
//             mistake is planted into every layout, and verify_strips has to find it
//   columns   random operations through pack_columns and verify_columns, and planted mistakes
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

#include "strips.hpp"

using namespace adpsgd_impl;

namespace {

std::mt19937 rng(1);
int below(int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); }

[[noreturn]] void die(int trial, const std::string& what) {
    std::printf("trial %d: %s\n", trial, what.c_str());
    std::exit(1);
}

struct Schedule {
    int32_t n, T, n_slots, window;
    int64_t K, A;
    bool compensate, renumber;
    std::vector<int32_t> worker, neighbour, tau, carried, extra_a, extra_b;
    std::vector<int64_t> extra_ptr;
    std::vector<WorkerData> data;
    Plan plan;

    const int64_t* extras() const { return extra_a.empty() ? nullptr : extra_ptr.data(); }
    const int32_t* carried_or_null() const {
        return std::any_of(carried.begin(), carried.end(), [](int32_t s) { return s >= 0; }) ? carried.data() : nullptr;
    }
    StripCall call() const {
        return StripCall{n, n_slots, window, K, A, worker.data(), neighbour.data(), tau.data(), nullptr, 0.5f, extras(), extra_a.data(),
                         extra_b.data(), &plan, carried_or_null(), data.data(), renumber, 7u, 3};
    }
};

// false: no plan (the drawn taus do not fit the slots)
bool draw(Schedule& s) {
    s.n = 2 + below(20);
    s.K = 1 + below(150);
    s.T = below(12);
    s.A = s.K - (below(2) ? std::min<int64_t>(s.K, below(s.T + 3)) : 0);
    s.compensate = below(3) == 0;
    s.renumber = below(2) == 0;
    s.n_slots = s.T + 1 + below(20);
    s.window = std::min(s.n_slots, s.T + 1 + below(10));
    if (below(4) == 0) {          // T_max beyond the slots and the taus of this call
        s.window = strip_window(100 + below(50), false, 0, s.n_slots);
        s.renumber = false;
    }
    const bool extra = s.n >= 6 && below(3) == 0;
    const int pending = below(2) ? below(static_cast<int>(std::min<int64_t>(s.K, s.T)) + 1) : 0;      // leading events that may be carried
    std::vector<int32_t> slots(s.n_slots);
    for (int i = 0; i < s.n_slots; ++i) slots[i] = i;
    std::shuffle(slots.begin(), slots.end(), rng);
    size_t used = 0;
    s.carried.assign(s.K, -1);
    s.extra_ptr.assign(1, 0);
    for (int k = 0; k < s.K; ++k) {
        const int32_t w = below(s.n);
        int32_t j;
        do j = below(s.n);
        while (j == w && below(8));
        s.worker.push_back(w);
        s.neighbour.push_back(j);
        s.tau.push_back(below(std::min(k, s.T) + 1));
        if (k < pending && k < s.T && below(2)) {
            s.tau[k] = k + 1 + below(s.T - k);
            s.carried[k] = slots[used++];
        }
        if (extra && below(3) == 0) {
            int32_t a, b;
            do {
                a = below(s.n);
                b = below(s.n);
            } while (a == b || a == w || b == w || a == j || b == j);
            s.extra_a.push_back(a);
            s.extra_b.push_back(b);
        }
        s.extra_ptr.push_back(static_cast<int64_t>(s.extra_a.size()));
    }
    s.data.resize(s.n);
    for (int i = 0; i < s.n; ++i) {
        s.data[i].features = reinterpret_cast<const void*>(static_cast<uintptr_t>(0x1000 + i));
        s.data[i].targets = reinterpret_cast<const void*>(static_cast<uintptr_t>(0x2000 + i));
        s.data[i].ld = 5;
        s.data[i].rows = 3;
    }
    std::string err;
    return plan_rounds(s.n, s.K, s.worker.data(), s.neighbour.data(), s.tau.data(), s.n_slots, true, s.plan, err, s.extras(), s.extra_a.data(),
                       s.extra_b.data(), s.compensate, s.A, s.carried_or_null()) == 0;
}

// Changes one entry of a layout so that it no longer executes the schedule; false: nothing of that kind in it.
bool plant(StripProgram& p, int kind) {
    const int half = p.teams / 2;
    const int64_t start = below(static_cast<int>(p.iterations));
    for (int64_t i = 0; i < p.iterations; ++i) {
        StripEntry* rec = &p.recs[(start + i) % p.iterations * p.rec_len];
        const int updates = static_cast<int>(rec[0].x), evals = __builtin_popcount(rec[0].z), loads = __builtin_popcount(rec[0].y);
        StripEntry* up = rec + 1 + 4 * half;
        if (kind < 4) {
            for (int u = 0; u < updates; ++u) {
                if (up[u].w & kStripEmpty) continue;
                if (kind == 0) up[u].w |= kStripEmpty;                                      // an update left out
                if (kind == 1) up[u].x = (up[u].x & 0xFFFFu) | ((up[u].x >> 16) + 1) << 16;  // another partner
                if (kind == 2) {                                                            // another gradient
                    if (up[u].w & kStripAverage) continue;
                    up[u].y += 1;
                }
                if (kind == 3) up[u].w ^= kStripAverage;                                    // a step that is not taken, or one too many
                return true;
            }
        } else if (kind < 8 && evals > 0) {
            StripEntry* e = rec + 1 + 2 * below(evals);
            if (kind == 4) e[0].z ^= 1u;                                                    // the gradient of another worker
            if (kind == 5) e[0].y += 1;                                                     // a sequence number used twice
            if (kind == 6) e[1].x = e[1].x == 0xFFFFFFFFu ? 0u : 0xFFFFFFFFu;                // a read compensated, or not
            if (kind == 7) e[0].w += 1000;                                                  // a slot that does not exist
            return true;
        } else if (kind == 8 && loads > 0) {
            rec[1 + 2 * half].x ^= 1u;                                                      // the rows of another gradient
            return true;
        } else if (kind == 9 && loads > 0 && evals + loads < p.teams) {
            rec[0].y &= rec[0].y - 1;                                                       // rows that are not requested
            return true;
        }
    }
    return false;
}

}  // namespace

int main() {
    long iterations = 0, rounds = 0, planted = 0;
    for (int trial = 0; trial < 4000; ++trial) {
        Schedule s;
        if (!draw(s)) continue;
        const int teams_of[4] = {12, 6, 4, 2};
        const StripCall call = s.call();
        StripProgram p;
        std::string err;
        if (!build_strips(call, teams_of[below(4)], p)) die(trial, "no order");
        if (!verify_strips(call, p, err)) die(trial, err);
        iterations += p.iterations;
        rounds += s.plan.n_rounds;
        const int kind = trial % 10;
        if (plant(p, kind)) {
            ++planted;
            if (verify_strips(call, p, err)) die(trial, "planted mistake " + std::to_string(kind) + " not found");
        }
    }
    long batches = 0;
    for (int trial = 0; trial < 1000; ++trial) {
        const int n = 2 + below(40), count = 1 + below(300), capacity = 1 << below(5);
        std::vector<ColumnPair> pairs;
        for (int t = 0; t < count; ++t) pairs.push_back(ColumnPair{below(n), below(n), t});
        std::vector<int64_t> place;
        const int64_t b = pack_columns(pairs, n, capacity, place);
        batches += b;
        if (!verify_columns(pairs, n, capacity, place, b)) die(trial, "columns out of order");
        const int t = below(count);
        std::vector<int64_t> bad = place;
        bad[t] = bad[(t + 1) % count];                  // two operations in one place
        if (count > 1 && verify_columns(pairs, n, capacity, bad, b)) die(trial, "two operations in one place not found");
        bad = place;
        bad[t] += b * capacity;                         // a place behind the table
        if (verify_columns(pairs, n, capacity, bad, b)) die(trial, "a place behind the table not found");
        for (int u = 0; u < count; ++u)                 // an operation swapped with a later one of its row
            if (u > t && (pairs[u].i == pairs[t].i || pairs[u].j == pairs[t].i)) {
                bad = place;
                std::swap(bad[t], bad[u]);
                if (verify_columns(pairs, n, capacity, bad, b)) die(trial, "operations of a row out of order not found");
                break;
            }
    }
    std::printf("ok, iterations %ld rounds %ld, planted %ld, column batches %ld\n", iterations, rounds, planted, batches);
}
