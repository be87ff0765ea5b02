// The exchange of the linear gradients in one pass, executed on paper in random orders of its steps: blocks with one strip each
// publish a sum per sample, the block of a sample (sample mod strips) adds up its row of words and publishes a word, and a block
// goes on to its next gradient when it has the words it awaits (onepass_awaited).  No word may be overwritten before the block
// that adds it up has read it: that block would wait for a number that never comes back.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "onepass.hpp"

using namespace adpsgd_impl;

// Gradients of a group in shares (take_tickets of kernels_onepass.hip), on paper: any number of blocks, also fewer than strips,
// claim the shares in order.  Some block can always go on, no word is replaced before all that need it have read it, and every
// strip of every gradient is combined once, with the coefficients of that gradient.
int shares_check(std::mt19937& rng) {
    auto below = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    long combined = 0;
    for (int trial = 0; trial < 2000; ++trial) {
        const int S = 1 + below(7), samples = 1 + below(9), gradients = 1 + below(4), resident = 1 + below(S + 2);
        const int per = 2 * S + 1, shares = gradients * per;
        std::vector<int> sums(static_cast<size_t>(samples) * S, -1), coefs(samples, -1), times(static_cast<size_t>(gradients) * S, 0);
        std::vector<int> sums_read(gradients, 0), coefs_taken(gradients, 0);
        int tickets = 0, taken = 0;
        struct Block {
            int ticket = -1, sample = 0;
        };
        std::vector<Block> blocks(resident);
        int left = resident;
        // one step of a block, if it can take one
        auto step = [&](Block& b) -> int {
            if (b.ticket == -1) {
                b.ticket = tickets++;
                b.sample = 0;
                if (b.ticket >= shares) --left;
                return 1;
            }
            const int i = b.ticket / per, share = b.ticket % per;
            if (share < S) {
                for (int m = 0; i > 0 && m < samples; ++m)
                    if (coefs[m] != i - 1) return 0;
                if (i > 0 && sums_read[i - 1] != samples) return -1;         // replaced before it was read
                for (int m = 0; m < samples; ++m) sums[m * S + share] = i;
            } else if (share == S) {
                if (i > 0 && taken < S * i) return 0;
                for (int s = 0; s < S; ++s)
                    if (sums[b.sample * S + s] != i) return 0;
                if (i > 0 && coefs_taken[i - 1] != S) return -1;
                ++sums_read[i];
                coefs[b.sample] = i;
                if (++b.sample < samples) return 1;
            } else {
                for (int m = 0; m < samples; ++m)
                    if (coefs[m] != i) return 0;
                ++coefs_taken[i];
                ++taken;
                ++times[i * S + share - S - 1];
                ++combined;
            }
            b.ticket = -1;
            return 1;
        };
        while (left > 0) {
            bool any = false;
            const int first = below(resident), turns = 1 + below(resident);
            for (int t = 0; t < resident; ++t) {
                Block& b = blocks[(first + t) % resident];
                if (b.ticket >= shares) continue;
                const int r = step(b);
                if (r < 0) {
                    std::printf("shares, trial %d: S %d, %d blocks: a word replaced early\n", trial, S, resident);
                    return 1;
                }
                any |= r > 0;
                if (any && t >= turns) break;
            }
            if (!any) {
                std::printf("shares, trial %d: S %d, %d blocks: no block can go on\n", trial, S, resident);
                return 1;
            }
        }
        for (int t : times)
            if (t != 1) {
                std::printf("shares, trial %d: a strip combined %d times\n", trial, t);
                return 1;
            }
    }
    std::printf("shares ok, combined %ld\n", combined);
    return 0;
}

int main() {
    std::mt19937 rng(11);
    auto below = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    long steps = 0, ahead = 0;
    for (int trial = 0; trial < 2000; ++trial) {
        const int S = 1 + below(8), M = 1 + below(12), gradients = 2 + below(4);
        const bool loss = below(2) != 0;
        const int samples = onepass_samples(loss ? ADPSGD_MODEL_LOGREG : ADPSGD_MODEL_LSQ, M, loss), awaited = onepass_awaited(samples);
        std::vector<uint32_t> sums(static_cast<size_t>(samples) * S, 0), words(samples, 0);      // numbers only
        struct Block {
            uint32_t gradient = 1;
            bool published = false;
            std::vector<std::vector<char>> read;      // per sample of this block: the sums taken so far
            std::vector<char> done;
        };
        std::vector<Block> blocks(S);
        auto begin = [&](int b) {
            blocks[b].published = false;
            blocks[b].read.assign(samples, std::vector<char>(S, 0));
            blocks[b].done.assign(samples, 0);
        };
        for (int b = 0; b < S; ++b) begin(b);
        int running = S;
        for (long idle = 0; running > 0; ++idle) {
            if (idle > 200000) {
                std::printf("trial %d: S %d, samples %d: the blocks wait for each other\n", trial, S, samples);
                return 1;
            }
            ++steps;
            const int b = below(S);
            Block& me = blocks[b];
            if (me.gradient > static_cast<uint32_t>(gradients)) continue;
            if (!me.published) {
                for (int m = 0; m < samples; ++m) {
                    const uint32_t before = sums[m * S + b];
                    if (before != 0 && blocks[m % S].gradient == before && !blocks[m % S].done[m] && !blocks[m % S].read[m][b]) {
                        std::printf("trial %d: S %d, samples %d: sum %d of strip %d overwritten before it was read\n", trial, S, samples, m, b);
                        return 1;
                    }
                    sums[m * S + b] = me.gradient;
                }
                me.published = true;
                continue;
            }
            bool progress = false;
            for (int m = b; m < samples && !progress; m += S) {       // the wavefronts of the block that add up samples
                if (me.done[m]) continue;
                bool all = true;
                for (int s = 0; s < S; ++s) {
                    if (!me.read[m][s] && sums[m * S + s] == me.gradient && below(2)) me.read[m][s] = 1, progress = true;
                    all &= me.read[m][s] != 0;
                }
                if (all) words[m] = me.gradient, me.done[m] = 1, progress = true;
            }
            if (progress) {
                idle = 0;
                continue;
            }
            bool go = true;
            for (int m = b; m < samples; m += S) go &= me.done[m] != 0;       // its own wavefronts meet at a barrier
            for (int m = 0; m < awaited; ++m) go &= words[m] == me.gradient;
            if (!go) continue;
            for (int o = 0; o < S; ++o) ahead += blocks[o].gradient < me.gradient;
            ++me.gradient;
            idle = 0;
            if (me.gradient > static_cast<uint32_t>(gradients)) --running;
            else begin(b);
        }
    }
    if (shares_check(rng) != 0) return 1;
    std::printf("ok, steps %ld, blocks left behind %ld\n", steps, ahead);
}
