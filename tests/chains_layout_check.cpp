// Rounds whose updates come in chains (plan_rounds with chain > 1, chain_rounds), checked on the CPU: random schedules (stale
// reads, carried and looked-ahead events, extra pairs, few slots, chains of 1 to 5) through verify_plan and verify_chains and
// executed on paper against the serial order; then one mistake is planted into every layout, and verify_chains has to find it.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "internal.hpp"

using namespace adpsgd_impl;

namespace {

std::mt19937 rng(3);
int below(int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); }

[[noreturn]] void die(int trial, const char* what) {
    std::printf("trial %d: %s\n", trial, what);
    std::exit(1);
}

struct Schedule {
    int32_t n, T, n_slots, chain;
    int64_t K, A;
    std::vector<int32_t> worker, neighbour, tau, carried, extra_a, extra_b;
    std::vector<int64_t> extra_ptr;
};

Schedule draw() {
    Schedule s;
    s.n = 2 + below(16);
    s.K = 1 + below(120);
    s.T = below(10);
    s.A = s.K - (below(2) ? std::min<int64_t>(s.K, below(s.T + 3)) : 0);
    s.n_slots = s.T + 1 + below(20);
    s.chain = 1 + below(5);
    const bool extra = s.n >= 6 && below(3) == 0;
    const int pending = below(2) ? below(static_cast<int>(std::min<int64_t>(s.K, s.T)) + 1) : 0;
    int32_t used = 0;
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
            s.carried[k] = used++;
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
    return s;
}

}  // namespace

int main() {
    long rounds = 0, single = 0, planted = 0;
    for (int trial = 0; trial < 6000; ++trial) {
        const Schedule s = draw();
        const int64_t* extra = s.extra_a.empty() ? nullptr : s.extra_ptr.data();
        const int32_t* carried = std::any_of(s.carried.begin(), s.carried.end(), [](int32_t c) { return c >= 0; }) ? s.carried.data() : nullptr;
        Plan plan, plain;
        std::string err;
        auto make = [&](int32_t chain, Plan& p) {
            return plan_rounds(s.n, s.K, s.worker.data(), s.neighbour.data(), s.tau.data(), s.n_slots, true, p, err, extra, s.extra_a.data(), s.extra_b.data(),
                               false, s.A, carried, chain);
        };
        if (make(s.chain, plan) != 0) continue;
        if (make(1, plain) != 0) die(trial, "a plan only with chains");
        if (!verify_plan(s.n, s.K, s.worker.data(), s.neighbour.data(), s.tau.data(), s.n_slots, true, plan, err, extra, s.extra_a.data(), s.extra_b.data(),
                         s.A, carried, s.chain > 1))
            die(trial, err.c_str());
        rounds += plan.n_rounds;
        single += plain.n_rounds;

        std::vector<int64_t> offset(plan.n_rounds + 1, 0);
        auto pairs_of = [&](int64_t k) { return 1 + (extra ? extra[k + 1] - extra[k] : 0); };
        for (int64_t k = 0; k < s.A; ++k) offset[plan.u_round[k] + 1] += pairs_of(k);
        for (int32_t r = 0; r < plan.n_rounds; ++r) offset[r + 1] += offset[r];
        std::vector<ColumnPair> pairs(offset.back());
        std::vector<int64_t> fill(offset.begin(), offset.end() - 1);
        for (int64_t k = 0; k < s.A; ++k) {
            pairs[fill[plan.u_round[k]]++] = ColumnPair{s.worker[k], s.neighbour[k], k};
            for (int64_t q = 0; q + 1 < pairs_of(k); ++q) pairs[fill[plan.u_round[k]]++] = ColumnPair{s.extra_a[extra[k] + q], s.extra_b[extra[k] + q], -1};
        }
        ChainLayout c;
        chain_rounds(pairs, offset, s.n, c);
        if (!verify_chains(pairs, offset, s.n, s.chain, c)) die(trial, "chains out of order");

        // on paper: every row's updates in the order of the events, every read before and after the right ones
        std::vector<std::vector<int64_t>> serial(s.n), done(s.n);
        for (int64_t k = 0; k < s.A; ++k) {
            serial[s.worker[k]].push_back(k);
            if (s.neighbour[k] != s.worker[k]) serial[s.neighbour[k]].push_back(k);
            for (int64_t q = 0; q + 1 < pairs_of(k); ++q) {
                serial[s.extra_a[extra[k] + q]].push_back(-1);
                serial[s.extra_b[extra[k] + q]].push_back(-1);
            }
        }
        std::vector<int64_t> slot(s.n_slots, -1);
        for (int64_t k = 0; k < s.K; ++k)
            if (s.carried[k] >= 0 && carried) slot[s.carried[k]] = k;
        for (int32_t r = 0; r < plan.n_rounds; ++r) {
            for (int64_t k = 0; k < s.K; ++k) {
                if (plan.r_round[k] != r) continue;
                int64_t before = 0;
                for (int64_t m = 0; m < std::min(s.A, k - s.tau[k]); ++m) {
                    bool names = s.worker[m] == s.worker[k] || s.neighbour[m] == s.worker[k];
                    for (int64_t q = 0; q + 1 < pairs_of(m); ++q) names |= s.extra_a[extra[m] + q] == s.worker[k] || s.extra_b[extra[m] + q] == s.worker[k];
                    before += names;
                }
                if (static_cast<int64_t>(done[s.worker[k]].size()) != before) die(trial, "a read of the wrong version");
                if (slot[plan.slot[k]] != -1) die(trial, "a slot in use");
                slot[plan.slot[k]] = k;
            }
            for (int64_t ch = c.round[r]; ch < c.round[r + 1]; ++ch)
                for (int64_t q = c.first[ch]; q < c.first[ch + 1]; ++q) {
                    const ColumnPair& p = pairs[c.order[q]];
                    done[p.i].push_back(p.event);
                    if (p.j != p.i) done[p.j].push_back(p.event);
                    if (p.event < 0) continue;
                    if (slot[plan.slot[p.event]] != p.event) die(trial, "an update without its gradient");
                    slot[plan.slot[p.event]] = -1;
                }
        }
        for (int32_t r = 0; r < s.n; ++r)
            if (done[r] != serial[r]) die(trial, "updates of a row out of order");

        // planted mistakes: two operations of a chain exchanged, a chain cut in two, two chains made one that is too long
        for (size_t ch = 0; ch + 1 < c.first.size(); ++ch) {
            if (c.first[ch + 1] - c.first[ch] < 2) continue;
            ChainLayout bad = c;
            std::swap(bad.order[c.first[ch]], bad.order[c.first[ch] + 1]);
            if (verify_chains(pairs, offset, s.n, s.chain, bad)) die(trial, "exchanged operations not found");
            bad = c;
            bad.first.insert(bad.first.begin() + ch + 1, c.first[ch] + 1);
            for (auto& at : bad.round)
                if (at > static_cast<int64_t>(ch)) ++at;
            if (verify_chains(pairs, offset, s.n, s.chain, bad)) die(trial, "a chain in two parts not found");
            if (verify_chains(pairs, offset, s.n, static_cast<int32_t>(c.first[ch + 1] - c.first[ch]) - 1, c)) die(trial, "a chain too long not found");
            ++planted;
            break;
        }
    }
    std::printf("ok, rounds %ld without chains %ld, planted %ld\n", rounds, single, planted);
}
