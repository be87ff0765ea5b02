// How the linear gradients in one pass over the minibatch rows lie on the chip (kernels_onepass.hip).
#include "onepass.hpp"

#include <algorithm>

namespace adpsgd_impl {

// A thread holds up to 32 vectors of four columns, 256 KB a block: with 40 and 48, which gradients beyond 67 MB need, registers
// spill.  Two gradients fit up to 16 vectors, 33 MB on all 256 compute units, with 8 or 16 rows a wavefront;  12 and 25 MB with 6 or 12
// rows, 8 and 17 MB with 2 or 4 (few rows, and with them many columns of x^).  The line to the pipeline, 64 and 61 set-ups below and
// above 4 MB a gradient, against one gradient at a time: below 1 MB 0.80 ... 1.25 times as fast, 3 to 8 MB 0.90 ... 1.17, from 8 MB on
// 0.98 ... 1.29 (but see below); with 6 rows, of 16 vectors only 12 in use, 0.92 ... 1.1 at 9.6 MB.
// A place is the compute units of a gradient, of two in the pipeline.  A gradient a little beyond a half or a third of the device leaves the
// pipeline one place where the kernel for one at a time has three, or two where it has five, and most of the device idle.  460 set-ups of
// 8 to 33 MB, rounds of 6 and 14 gradients and synchronous iterations of 24, by places of the pipeline and of the other:
//   1 and 2, 2 and 4, 3 and 5, 3 and 6, 4 and 8   0.96 ... 1.32 times as fast (below 1 only rounds of 6 of 8 to 9.5 MB with M > 64);
//   1 and 3, 2 and 5   M > 64 0.84 ... 1.02, M = 52 and 64 0.95 ... 1.05 (the least with 1 and 3), M = 26 and 32 0.97 ... 1.12, M <= 8 1.0 ... 1.11;
//                      M = 45, six rows 1.02 ... 1.07;
//   1 and 6            M = 4 0.90 ... 1.04; with 1 and 5 0.99 ... 1.03.
// And to fill and drain the pipeline counts where a launch is short: synchronous iterations of 3 to 16 workers, 49 sizes, by the turns of a
// place of the pipeline against the steps of the other:  2 and more against 1  0.84 ... 1.01 times as fast, 1 against 1 0.98 ... 1.19;  4 against
// 2  M > 32 0.92 ... 1.03, else 0.985 ... 1.10;  6 against 2 0.91 ... 1.0;  3 against 2 1.03 ... 1.2;  6 against 3 0.97 ... 1.10;  others 0.97 ... 1.25.
// Staged rows against none where two gradients do not fit and one does (17 or 33 to 67 MB), 241 set-ups: M <= 32, 42, 45 and 97 ... 128 0.97 ... 1.14
// times as fast, 1.04 in the mean; M = 49 ... 96 0.94 ... 1.07, 0.98 in the mean.
// Strips of large gradients are of equal width, as many as the compute units of their group (with widths in whole vectors of a wavefront M = 128,
// d = 131 073 had 171 strips on 256 compute units).  Below 20 strips the blocks hold less, so that a gradient spreads over more compute units (n = 16, M = 8, d = 131 000
// on the 4-regular graph: 786 us for 40 events in three launches a round, 708 with 16 strips, 609 with 32).
// Measured against the three launches, 450 set-ups of 16 and 40 workers, M = 1 ... 128, 0.25 to 100 MB a gradient:
//   logistic   1.02 ... 2.1 times as fast;
//   least squares, events   these leave the gradient as its M coefficients there, here it is written out and read again:
//              0.75 ... 1.1 times for M <= 5, 1.1 ... 1.3 for M = 6 (0.92 with 48 vectors), 1.04 ... 1.9 from M = 7 on;
//   least squares, synchronous or wait-free (dense in both)   0.94 ... 1.3 for M <= 3, 0.97 ... 1.8 from M = 5 on.
// On devices (or partitions of one) with fewer compute units a smaller gradient may need more than 32 vectors a thread, for which
// there is the staged kernel alone: with 64 M = 9, d = 443 604, with 32 M = 80, d = 16 860.
// What does not fit the chip (beyond 100 MB) and short models (d <= 2048: one block a gradient) stay with them.
OnePassShape onepass_shape(int model, int64_t d, int32_t M, int32_t compute_units, int32_t at_once) {
    OnePassShape s;
    if ((model != ADPSGD_MODEL_LSQ && model != ADPSGD_MODEL_LOGREG) || M < (model == ADPSGD_MODEL_LSQ ? 4 : 1) || M > kOnePassMaxM) return s;
    if (d <= 2048 || static_cast<double>(M) * static_cast<double>(d) < 50000.0) return s;
    s.row_groups = M <= 8 ? 1 : M <= 16 ? 2 : M <= 32 ? 4 : 8;
    const int rows = (M + s.row_groups - 1) / s.row_groups, most = std::min(compute_units, kOnePassMaxStrips);
    s.rows = rows <= 2 ? 2 : rows <= 4 ? 4 : rows <= 6 ? 6 : rows <= 8 ? 8 : rows <= 12 ? 12 : 16;
    int64_t strips = 0;
    auto cut = [&](int chunks) {
        s.chunks = chunks;
        const int64_t tile = 256ll * s.chunks * (kOnePassWaves / s.row_groups);
        strips = (d + tile - 1) / tile;
    };
    auto hold = [&](int held) { cut(std::max(1, held / s.rows)); };
    auto at_a_time = [&] { return strips <= most ? most / strips : 0; };
    const int held = s.rows == 2 ? 16 : 32;
    if (4.0 * M * static_cast<double>(d) >= (s.rows == 6 ? 2.0 : 1.0) * kOnePassLargeBytes) {
        hold(held);
        const int64_t plain = at_a_time();
        cut(onepass_pipeline_chunks(s.rows));
        const int64_t pipeline = at_a_time();
        bool places = pipeline > 0 && plain <= (s.row_groups == 8 && s.rows >= 8 ? 2 : 5) * pipeline;
        if (places && at_once > 0) {
            const int64_t steps = (at_once + plain - 1) / plain, turns = (at_once + pipeline - 1) / pipeline;
            places = steps > 2 || turns < (steps == 1 || s.row_groups == 8 ? 2 : 3) * steps;
        }
        const bool staged = pipeline == 0 && (s.row_groups < 8 || s.rows == 6 || s.rows == 16);
        s.kernel = staged ? OnePassKernel::kStaged : places ? OnePassKernel::kPipeline : OnePassKernel::kPlain;
    }
    if (s.kernel != OnePassKernel::kPipeline) {
        hold(held);
        if (strips > most && s.rows >= 6) hold(40);
        if (strips > most && s.rows >= 6) hold(48);
        if (strips < 20) hold(16);
        if (strips < 20) hold(8);
        if (s.rows * s.chunks > 32) s.kernel = OnePassKernel::kStaged;
    }
    if (strips > most) return s;
    s.groups = static_cast<int32_t>(most / strips);
    // large: as many strips as the compute units of a group, of equal width
    const int64_t waves = kOnePassWaves / s.row_groups, parts = most / s.groups * waves;
    s.wave_cols = s.kernel != OnePassKernel::kPlain ? static_cast<int32_t>(((d + parts - 1) / parts + 31) / 32 * 32) : 256 * s.chunks;
    s.strips = static_cast<int32_t>((d + waves * s.wave_cols - 1) / (waves * s.wave_cols));
    return s;
}

bool onepass_for_events(const OnePassShape& s, int model, int32_t M, bool wait_free) {
    return model == ADPSGD_MODEL_LOGREG || wait_free || M >= (s.rows * s.chunks <= 40 ? 6 : 7);
}

size_t onepass_exchange_bytes(const OnePassShape& s, int32_t M) {
    return static_cast<size_t>(s.groups) * onepass_group_words(s, M + 1) * sizeof(unsigned long long);
}

}  // namespace adpsgd_impl
