// The exchange of two gradients at a time (onepass_pipeline_kernel), executed on paper in random orders of its steps: a block takes
// the coefficients of t - 1, adds up its samples of t when the sums of all strips are there and publishes their coefficients, then
// publishes its sums of t + 1.  Words of gradient t lie at t mod 2.  None may be replaced before all that need it have read it, and
// some block can always go on.
#include <cstdio>
#include <random>
#include <vector>

int main() {
    std::mt19937 rng(5);
    auto below = [&](int n) { return static_cast<int>(rng() % static_cast<unsigned>(n)); };
    long turns = 0;
    for (int trial = 0; trial < 3000; ++trial) {
        const int S = 1 + below(7), samples = 1 + below(9), count = 1 + below(6);
        std::vector<int> sums(2 * samples * S, -1), coefs(2 * samples, -1), sums_read(count * samples, 0), coefs_read(count, 0);
        struct Block {
            int t = -1, step = 0, sample;
        };
        std::vector<Block> blocks(S);
        int left = S;
        auto step = [&](int b) -> int {               // 1: went on, 0: waits, -1: a word was replaced early
            Block& me = blocks[b];
            const int t = me.t;
            if (me.step == 0) {                       // coefficients of t - 1
                for (int m = 0; t >= 1 && m < samples; ++m)
                    if (coefs[((t - 1) & 1) * samples + m] != t - 1) return 0;
                if (t >= 1) ++coefs_read[t - 1];
                me.sample = b;
                me.step = 1;
            } else if (me.step == 1) {                // sums of t, the block's next sample
                if (t < 0 || t >= count || me.sample >= samples) {
                    me.step = 2;
                    return 1;
                }
                for (int s = 0; s < S; ++s)
                    if (sums[((t & 1) * samples + me.sample) * S + s] != t) return 0;
                ++sums_read[t * samples + me.sample];
                if (t >= 2 && coefs_read[t - 2] != S) return -1;
                coefs[(t & 1) * samples + me.sample] = t;
                me.sample += S;
            } else {                                  // sums of t + 1
                for (int m = 0; t + 1 < count && m < samples; ++m) {
                    if (t >= 1 && sums_read[(t - 1) * samples + m] == 0) return -1;
                    sums[(((t + 1) & 1) * samples + m) * S + b] = t + 1;
                }
                me.step = 0;
                ++turns;
                if (++me.t > count) --left;
            }
            return 1;
        };
        while (left > 0) {
            bool any = false;
            const int first = below(S), tries = 1 + below(S);
            for (int i = 0; i < S && !(any && i >= tries); ++i) {
                const int b = (first + i) % S;
                if (blocks[b].t > count) continue;
                const int r = step(b);
                if (r < 0) return std::printf("trial %d: S %d, samples %d: a word replaced early\n", trial, S, samples), 1;
                any |= r > 0;
            }
            if (!any) return std::printf("trial %d: S %d, samples %d: no block can go on\n", trial, S, samples), 1;
        }
    }
    std::printf("ok, turns %ld\n", turns);
    return 0;
}
