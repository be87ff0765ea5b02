// The exchange of two gradients at a time (onepass_pipeline_kernel), executed on paper in random orders of its steps, with the ring, the
// number of sums and the flags of csrc/onepass.hpp.  A block is a few wavefronts that meet at barriers: in turn t each takes the
// coefficients (and losses) of t - 1, looks behind a barrier whether a wait of the block was in vain, adds up its samples of t when the
// sums of all strips are there and publishes their coefficients, and behind another barrier publishes sums of t + 1.  No word may be
// replaced before all that need it have read it, some block can always go on, and all wavefronts of a block leave in the same turn,
// whichever of their waits end in vain.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "onepass.hpp"

using namespace adpsgd_impl;

namespace {

struct Flags {
    int (*seen)(int), (*coefficients)(int), (*sums)(int);
};
enum class End { kDone, kReplaced, kStuck, kParted };

// vain: of 1000 waits that could go on or not, how many end without an answer (0: none, and every gradient is finished)
End exchange(std::mt19937& rng, const Flags& flags, int vain, long& turns) {
    auto below = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    OnePassShape shape;
    shape.kernel = OnePassKernel::kPipeline;
    const int ring = shape.ring(), S = 1 + below(6), W = 1 + below(4), M = 1 + below(8), count = 1 + below(6);
    const bool loss = below(2) != 0;
    const int samples = onepass_samples(ADPSGD_MODEL_LOGREG, M, loss);
    std::vector<int> sums(ring * samples * S, -1), coefs(ring * samples, -1), losses(ring * samples, -1);
    std::vector<int> sums_read(count * samples, 0), coefs_read(count, 0), losses_read(count, 0);
    enum Step { kTake, kLook, kAdd, kPublish };
    struct Wave {
        int t = -1, sample = 0;
        Step step = kTake;
        bool waits = false, gone = false;
    };
    struct Block {
        std::vector<Wave> waves;
        int late[2] = {0, 0}, at_barrier = 0;
    };
    std::vector<Block> blocks(S);
    for (Block& b : blocks) b.waves.resize(W);
    int left = S * W;
    End end = End::kDone;
    auto barrier = [&](Block& b, Wave& w) {
        w.waits = true;
        if (++b.at_barrier < W) return;
        b.at_barrier = 0;
        for (Wave& o : b.waves) o.waits = false;
    };
    // one step of a wavefront; false: it waits
    auto step = [&](int strip, int wave) {
        Block& b = blocks[strip];
        Wave& w = b.waves[wave];
        const int t = w.t, now = (t % ring + ring) % ring, before = (now + ring - 1) % ring;
        if (w.step == kTake) {                    // coefficients of t - 1 (the first wavefront), losses (the last, strip 0)
            const bool takes = t >= 1 && wave == 0, takes_loss = t >= 1 && loss && strip == 0 && wave == W - 1;
            bool there = true;
            for (int m = 0; m < samples; ++m) there &= (!takes || coefs[before * samples + m] == t - 1) && (!takes_loss || losses[before * samples + m] == t - 1);
            if (!there) {
                if (below(1000) >= vain) return false;
                b.late[flags.coefficients(t)] = 1;
            } else {
                if (takes) ++coefs_read[t - 1];
                if (takes_loss) ++losses_read[t - 1];
            }
            w.step = kLook;
            barrier(b, w);
        } else if (w.step == kLook) {
            if (b.late[flags.seen(t)] != 0) {
                w.gone = true;
                --left;
                return true;
            }
            w.sample = strip + S * wave;
            w.step = kAdd;
        } else if (w.step == kAdd) {
            if (t < 0 || t >= count || w.sample >= samples) {
                w.step = kPublish;
                barrier(b, w);
                return true;
            }
            const int m = w.sample;
            bool there = true;
            for (int s = 0; s < S; ++s) there &= sums[(now * samples + m) * S + s] == t;
            if (!there) {
                if (below(1000) >= vain) return false;
                b.late[flags.sums(t)] = 1;
                w.sample = samples;
                return true;
            }
            ++sums_read[t * samples + m];
            if (t >= ring && vain == 0 && (coefs_read[t - ring] != S || (loss && losses_read[t - ring] != 1))) end = End::kReplaced;
            coefs[now * samples + m] = losses[now * samples + m] = t;
            w.sample += S * W;
        } else {
            if (wave == 0 && t + 1 < count) {
                const int next = (now + 1) % ring;
                for (int m = 0; m < samples; ++m) {
                    if (t + 1 >= ring && sums_read[(t + 1 - ring) * samples + m] == 0) end = End::kReplaced;
                    sums[(next * samples + m) * S + strip] = t + 1;
                }
            }
            w.step = kTake;
            ++turns;
            if (++w.t > count) {
                w.gone = true;
                --left;
            }
        }
        return true;
    };
    while (left > 0 && end == End::kDone) {
        bool any = false;
        const int all = S * W, first = below(all), tries = 1 + below(all);
        for (int i = 0; i < all && !(any && i >= tries); ++i) {
            const int at = (first + i) % all;
            Wave& w = blocks[at / W].waves[at % W];
            if (!w.gone && !w.waits) any |= step(at / W, at % W);
        }
        if (any) continue;
        for (Block& b : blocks)                   // some wavefronts at a barrier that others will not come to
            for (Wave& w : b.waves)
                for (Wave& o : b.waves)
                    if (w.waits && o.gone) end = End::kParted;
        if (end == End::kDone && vain == 0) end = End::kStuck;
    }
    for (Block& b : blocks)
        for (Wave& w : b.waves)
            if (end == End::kDone && w.t != b.waves[0].t) end = End::kParted;
    return end;
}

}  // namespace

int main() {
    std::mt19937 rng(5);
    const Flags ours = {late_seen, late_of_coefficients, late_of_sums};
    // what this has to find: one flag for all turns, raised after some wavefronts have looked
    const Flags single = {[](int) { return 0; }, [](int) { return 0; }, [](int) { return 0; }};
    long turns = 0, parted = 0;
    for (int trial = 0; trial < 6000; ++trial) {
        const int vain = trial % 3 == 0 ? 0 : trial % 3 == 1 ? 20 : 1000;
        const End end = exchange(rng, ours, vain, turns);
        if (end != End::kDone) {
            std::printf("trial %d: %s\n", trial, end == End::kReplaced ? "a word replaced early" : end == End::kStuck ? "no block can go on" : "the wavefronts of a block part");
            return 1;
        }
        long ignored = 0;
        parted += exchange(rng, single, vain, ignored) == End::kParted;
    }
    if (parted == 0) return std::printf("a flag for all turns was not found out\n"), 1;
    std::printf("ok, turns %ld, parted with one flag %ld\n", turns, parted);
    return 0;
}
