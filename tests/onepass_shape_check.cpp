// The shapes of the linear gradients in one pass (csrc/onepass.cpp), over minibatches, lengths and numbers of compute units from a
// partition of the device to more than one has: whatever is accepted is built, covers the gradient and fits the chip, and
// whatever is built is chosen.
#include <cmath>
#include <cstdio>
#include <random>

#include "onepass.hpp"

using namespace adpsgd_impl;

int main() {
    std::mt19937 rng(3);
    long ok = 0, by_kernel[3] = {0, 0, 0}, chosen[3][17][9] = {};
    auto fail = [](const char* what, int model, long long d, int M, int cus, const OnePassShape& s) {
        std::printf("%s: model %d, d %lld, M %d, %d compute units: %d rows, %d chunks, %d row groups, %d strips, %d groups, %d columns, kernel %d\n", what, model, d, M,
                    cus, s.rows, s.chunks, s.row_groups, s.strips, s.groups, s.wave_cols, static_cast<int>(s.kernel));
        return 1;
    };
    for (int cus : {16, 20, 32, 38, 64, 80, 104, 128, 228, 256, 304})
        for (int M = 1; M <= 128; ++M)
            for (int i = 0; i < 500; ++i) {
                const int model = i & 1 ? ADPSGD_MODEL_LSQ : ADPSGD_MODEL_LOGREG;
                const auto d = static_cast<int64_t>(std::exp(std::uniform_real_distribution<double>(std::log(2000.0), std::log(4e7))(rng)));
                const int at_once = i % 3 == 0 ? 1 + static_cast<int>(rng() % 40) : 0;
                const OnePassShape s = onepass_shape(model, d, M, cus, at_once);
                if (s.ok() != onepass_shape(model, d, M, cus).ok()) return fail("accepted by the number of gradients", model, d, M, cus, s);
                if (!s.ok()) continue;
                ++ok;
                ++by_kernel[static_cast<int>(s.kernel)];
                bool held = false;
                for (const OnePassHeld& h : kOnePassHeld) held |= h.rows == s.rows && h.chunks == s.chunks;
                ++chosen[static_cast<int>(s.kernel)][s.rows][s.chunks];
                if (!held || !onepass_built(s.kernel, s.rows, s.chunks)) return fail("not built", model, d, M, cus, s);
                const int64_t columns = static_cast<int64_t>(kOnePassWaves / s.row_groups) * s.wave_cols;
                if (s.rows * s.row_groups < M || s.rows * s.row_groups > kOnePassMaxM) return fail("rows", model, d, M, cus, s);
                if (s.wave_cols > 256 * s.chunks || s.wave_cols % 32 != 0 || (s.kernel == OnePassKernel::kPlain && s.wave_cols != 256 * s.chunks)) return fail("columns", model, d, M, cus, s);
                if (columns * s.strips < d || columns * (s.strips - 1) >= d) return fail("strips", model, d, M, cus, s);
                if (s.kernel == OnePassKernel::kPipeline && kOnePassWaves * s.strips < onepass_samples(model, M, true)) return fail("a wavefront would add up two samples", model, d, M, cus, s);
                if (s.groups < 1 || s.strips * s.groups > cus || s.strips > kOnePassMaxStrips) return fail("compute units", model, d, M, cus, s);
            }
    for (const OnePassHeld& h : kOnePassHeld)
        for (OnePassKernel kernel : {OnePassKernel::kPlain, OnePassKernel::kPipeline, OnePassKernel::kStaged})
            if (onepass_built(kernel, h.rows, h.chunks) && chosen[static_cast<int>(kernel)][h.rows][h.chunks] == 0)
                return std::printf("kernel %d of %d rows, %d chunks is built and never chosen\n", static_cast<int>(kernel), h.rows, h.chunks), 1;
    // next to the sizes from which the pipeline has too few places on 256 compute units, and where places do not count (M <= 32)
    struct Size {
        int M;
        int64_t d;
        OnePassKernel kernel;
    };
    for (const Size& z : {Size{96, 32767, OnePassKernel::kPipeline}, Size{96, 32769, OnePassKernel::kPlain}, Size{128, 16384, OnePassKernel::kPipeline},
                          Size{128, 16385, OnePassKernel::kPlain}, Size{128, 32768, OnePassKernel::kPipeline}, Size{128, 32769, OnePassKernel::kPlain},
                          Size{128, 43521, OnePassKernel::kPipeline}, Size{64, 65537, OnePassKernel::kPlain}, Size{32, 131073, OnePassKernel::kPipeline},
                          Size{8, 524289, OnePassKernel::kPipeline}, Size{45, 98305, OnePassKernel::kPipeline}, Size{4, 688128, OnePassKernel::kPlain},
                          Size{4, 688129, OnePassKernel::kPipeline}, Size{128, 65537, OnePassKernel::kStaged}, Size{64, 131073, OnePassKernel::kPlain},
                          Size{96, 65537, OnePassKernel::kPlain}, Size{96, 131073, OnePassKernel::kStaged}, Size{32, 262145, OnePassKernel::kStaged}})
        if (onepass_shape(ADPSGD_MODEL_LOGREG, z.d, z.M, 256).kernel != z.kernel) return fail("another kernel", ADPSGD_MODEL_LOGREG, z.d, z.M, 256, onepass_shape(ADPSGD_MODEL_LOGREG, z.d, z.M, 256));
    // ... and by the gradients of a launch: 4 and 8 places, 3 and 6, 1 and 3
    struct Launch {
        int M;
        int64_t d;
        int at_once;
        OnePassKernel kernel;
    };
    for (const Launch& z : {Launch{64, 32768, 4, OnePassKernel::kPipeline}, Launch{64, 32768, 5, OnePassKernel::kPlain}, Launch{64, 32768, 8, OnePassKernel::kPlain},
                            Launch{64, 32768, 9, OnePassKernel::kPipeline}, Launch{128, 21504, 3, OnePassKernel::kPipeline}, Launch{128, 21504, 6, OnePassKernel::kPlain},
                            Launch{128, 21504, 9, OnePassKernel::kPipeline}, Launch{128, 21504, 12, OnePassKernel::kPlain}, Launch{128, 21504, 13, OnePassKernel::kPipeline},
                            Launch{32, 131073, 3, OnePassKernel::kPlain}, Launch{32, 131073, 4, OnePassKernel::kPipeline}, Launch{32, 131073, 6, OnePassKernel::kPlain},
                            Launch{32, 131073, 7, OnePassKernel::kPipeline}})
        if (onepass_shape(ADPSGD_MODEL_LOGREG, z.d, z.M, 256, z.at_once).kernel != z.kernel)
            return std::printf("%d gradients: ", z.at_once), fail("another kernel", ADPSGD_MODEL_LOGREG, z.d, z.M, 256, onepass_shape(ADPSGD_MODEL_LOGREG, z.d, z.M, 256, z.at_once));
    if (by_kernel[0] == 0 || by_kernel[1] == 0 || by_kernel[2] == 0) return std::printf("a kernel without shapes\n"), 1;
    std::printf("ok, %ld shapes, %ld + %ld + %ld\n", ok, by_kernel[0], by_kernel[1], by_kernel[2]);
    return 0;
}
