// All events of a call in one launch, for the model whose gradients ignore the models (ADPSGD_MODEL_SYNTH).
//
// With g_k independent of X every column of X evolves on its own: averaging couples rows, never columns.  So a
// wavefront owns a strip of kQuads float4 columns of every row that the call touches, keeps it in LDS, executes all
// events on it and writes it back: X (and V) cross HBM once per call instead of 16 (24) bytes per parameter and event.
//
// Events that touch different rows commute, so the host packs them into batches of P = 64 / kQuads operations with
// pairwise disjoint rows, keeping the order of the events on every row (pack_columns); lane l of a wavefront takes
// operation l / kQuads of a batch and quad l % kQuads of the strip.  LDS operations of one wavefront execute in order
// and no wavefront reads another one's strip: the kernel needs no barrier.  Each element goes through the same
// operations in the same order as in the streaming kernel (kernels_fused.hip), so the results are the same bits.
//
// What binds is the arithmetic of the generator.  Its counter is (quad, 0, event, ...): the first Philox round and one
// of the two products of the second depend either on the quad alone or on the event alone.  The quad's part is
// computed once per wavefront, the event's part once on the host (ColumnOp); the rest is in vector registers, since an
// operand in a scalar one nearly doubles the time of an instruction (see device_common.hpp).  Measured at n = 128, d = 25.6 M
// on the ring, 2000 events per call: 32.1 ms (39.7 with keys in scalar registers, one batch per turn of the loop and a Newton
// step on the root), 128.8 ms in rounds of the streaming kernel; an operation takes a SIMD 168 ns per 64 quads, of which the
// instructions issue for about 145.  n = 32, d = 3.0 M with momentum, 500 events: 1.34 ms (1.62 before), 6.18 in rounds.
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace adpsgd_impl {
namespace {

struct ColumnParams {
    float* X;
    float* V;                  // momentum buffers (MOM), else nullptr
    int64_t ld, d, n_vec;
    const ColumnOp* ops;       // [batches + 2][P], empty operations have flags 0
    const int32_t* rows;       // the rows of X behind the local row numbers of the operations
    int32_t n_rows, batches;
    uint32_t key0, key1;
    SynthScale synth;
    float momentum, weight_decay;
};

// Philox4x32-10 from the second round on: hq, lq the two words of M0 * quad, the operation's words a..d from the host
__device__ __forceinline__ v4u philox_rest(uint32_t hq, uint32_t lq, const ColumnOp& op, const PhiloxKeys<8>& keys) {
    const uint64_t pb = static_cast<uint64_t>(kPhiloxM1) * (hq ^ op.a);
    return philox4x32_rounds<8>(static_cast<uint32_t>(pb >> 32) ^ op.b, static_cast<uint32_t>(pb), lq ^ op.c, op.d, keys);
}

// grid: one wavefront per kQuads float4 columns; AVERAGES: some operations average only; REFINE: SynthScale's, a kernel of its own
// since a branch in the middle of the generator keeps its two halves from overlapping (n = 13, d = 9109, 845 events 119.5 us with
// the branch, 114.5 without; n = 128, d = 25.6 M, 2000 events 33.7 and 32.1 ms)
template <int kQuads, bool MOM, bool AVERAGES, bool REFINE>
__global__ __launch_bounds__(256) void column_events_kernel(const ColumnParams p) {
    constexpr int P = 64 / kQuads;
    extern __shared__ __attribute__((aligned(16))) v4f strips[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int sub = lane / kQuads, ql = lane % kQuads;
    const int64_t q = (static_cast<int64_t>(blockIdx.x) * waves + wave) * kQuads + ql;
    const bool live = q < p.n_vec;
    const bool tail = __any(4 * q + 4 > p.d);              // the strip reaches beyond d: entries there stay zero
    v4f* xs = strips + static_cast<int64_t>(wave) * p.n_rows * kQuads * (MOM ? 2 : 1) + ql;
    v4f* vs = xs + (MOM ? p.n_rows * kQuads : 0);

    constexpr int kBatch = 8;      // rows of a lane whose loads are in flight together
    for (int r0 = sub; r0 < p.n_rows; r0 += kBatch * P) {
        v4f x[kBatch], v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int r = r0 + u * P;
            x[u] = v[u] = v4f{0, 0, 0, 0};
            if (r < p.n_rows && live) {
                const int64_t at = static_cast<int64_t>(p.rows[r]) * p.ld + 4 * q;
                x[u] = *reinterpret_cast<const v4f*>(p.X + at);
                if (MOM) v[u] = *reinterpret_cast<const v4f*>(p.V + at);
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int r = r0 + u * P;
            if (r < p.n_rows) {
                xs[r * kQuads] = x[u];
                if (MOM) vs[r * kQuads] = v[u];
            }
        }
    }
    wave_lds_sync();

    const uint64_t mq = static_cast<uint64_t>(kPhiloxM0) * static_cast<uint32_t>(q);       // d <= 2^34: the quad fits a word
    const uint32_t hq = static_cast<uint32_t>(mq >> 32), lq = static_cast<uint32_t>(mq);
    const PhiloxKeys<8> keys = philox_keys<8, true>(p.key0 + 2u * kPhiloxW0, p.key1 + 2u * kPhiloxW1);
    const NormalConstants normal = normal_constants<true>(SynthScale{p.synth.hi, p.synth.lo, REFINE});
    const float mu = MOM ? in_vector(p.momentum) : 0.0f, wd = MOM ? in_vector(p.weight_decay) : 0.0f;
    const int v_at = p.n_rows * kQuads;                    // from a row of the strip to its momentum buffer
    auto execute = [&](const ColumnOp& op) {
        if (op.flags != 0) {
            v4f* xi = reinterpret_cast<v4f*>(reinterpret_cast<char*>(xs) + (op.rows & 0xFFFFu));
            v4f* xj = reinterpret_cast<v4f*>(reinterpret_cast<char*>(xs) + (op.rows >> 16));
            const v4f av = *xi, bv = *xj;
            const float a[4] = {av.x, av.y, av.z, av.w}, c[4] = {bv.x, bv.y, bv.z, bv.w};
            float ni[4], nj[4];
            if (AVERAGES && op.flags == kColumnAverage) {      // an extra pair of a general W_k: no gradient, no step
#pragma unroll
                for (int t = 0; t < 4; ++t) ni[t] = nj[t] = (a[t] + c[t]) * 0.5f;
            } else {
                v4f g = synth_normals_of(philox_rest(hq, lq, op, keys), normal);
                if (tail) {
                    if (4 * q + 0 >= p.d) g.x = 0.0f;
                    if (4 * q + 1 >= p.d) g.y = 0.0f;
                    if (4 * q + 2 >= p.d) g.z = 0.0f;
                    if (4 * q + 3 >= p.d) g.w = 0.0f;
                }
                const float gv[4] = {g.x, g.y, g.z, g.w};
                if (MOM) {
                    v4f* vi = xi + v_at;
                    const v4f vo = *vi;
                    const float vold[4] = {vo.x, vo.y, vo.z, vo.w};
                    float vn[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        average_then_apply_momentum(a[t], c[t], gv[t], vold[t], op.gamma, mu, wd, ni[t], nj[t], vn[t]);
                    *vi = v4f{vn[0], vn[1], vn[2], vn[3]};
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) average_then_apply(a[t], c[t], gv[t], op.gamma, ni[t], nj[t]);
                }
            }
            *xj = v4f{nj[0], nj[1], nj[2], nj[3]};      // before x^i: without a partner (i == j) the step stands
            *xi = v4f{ni[0], ni[1], ni[2], ni[3]};
        }
        wave_lds_sync();
    };
    // two batches per turn, each requested one batch ahead; the table ends with two batches of empty operations
    ColumnOp even = p.ops[sub];
    for (int b = 0; b < p.batches; b += 2) {
        const ColumnOp* __restrict__ next = p.ops + static_cast<int64_t>(b) * P;
        const ColumnOp odd = next[P + sub];
        execute(even);
        even = next[2 * P + sub];
        execute(odd);
    }

    if (!live) return;
#pragma unroll 4
    for (int r = sub; r < p.n_rows; r += P) {
        const int64_t to = static_cast<int64_t>(p.rows[r]) * p.ld + 4 * q;
        *reinterpret_cast<v4f*>(p.X + to) = xs[r * kQuads];
        if (MOM) *reinterpret_cast<v4f*>(p.V + to) = vs[r * kQuads];
    }
}

template <int kQuads, bool MOM, bool AVERAGES>
void launch_columns(const ColumnParams& p, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (p.synth.refine) hipLaunchKernelGGL((column_events_kernel<kQuads, MOM, AVERAGES, true>), grid, block, lds, st, p);
    else hipLaunchKernelGGL((column_events_kernel<kQuads, MOM, AVERAGES, false>), grid, block, lds, st, p);
}
// Four wavefronts to a block, one to each SIMD, as far as 64 KB of LDS go.  Measured with 1 / 2 / 3 / 4 / 5 / 8 / 10 / 16 at
// n = 128, d = 25.6 M, 2000 events: 35.5 / 34.9 / 35.1 / 33.9 / 34.8 / 34.3 / 35.7 / 36.9 ms; at n = 32, d = 3.0 M with momentum,
// 500 events: 1.37 / 1.40 / 1.49 / 1.36 / 1.40 / 1.38 / 1.43 / 1.56.
template <int kQuads>
hipError_t launch_quads(const ColumnParams& p, bool averages, hipStream_t st) {
    const int64_t strip = static_cast<int64_t>(p.n_rows) * kQuads * 16 * (p.V ? 2 : 1);
    const int waves = static_cast<int>(std::min<int64_t>(4, 65536 / strip));
    const int64_t blocks = ((p.n_vec + kQuads - 1) / kQuads + waves - 1) / waves;
    if (waves < 1 || blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid(static_cast<uint32_t>(blocks)), block(64 * waves);
    const size_t lds = static_cast<size_t>(strip * waves);
    if (p.V && averages) launch_columns<kQuads, true, true>(p, grid, block, lds, st);
    else if (p.V) launch_columns<kQuads, true, false>(p, grid, block, lds, st);
    else if (averages) launch_columns<kQuads, false, true>(p, grid, block, lds, st);
    else launch_columns<kQuads, false, false>(p, grid, block, lds, st);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_column_events(const ColumnArgs& a, hipStream_t st) {
    if (a.batches <= 0 || a.n_rows <= 0) return hipSuccess;
    ColumnParams p;
    p.X = a.X;
    p.V = a.V;
    p.ld = a.ld;
    p.d = a.d;
    p.n_vec = (a.d + 3) / 4;
    p.ops = a.ops;
    p.rows = a.rows;
    p.n_rows = a.n_rows;
    p.batches = a.batches;
    p.key0 = static_cast<uint32_t>(a.synth_seed);
    p.key1 = static_cast<uint32_t>(a.synth_seed >> 32);
    p.synth = synth_scale(a.synth_std);

    p.momentum = a.momentum;
    p.weight_decay = a.weight_decay;
    switch (a.quads) {
        case 4: return launch_quads<4>(p, a.averages, st);
        case 8: return launch_quads<8>(p, a.averages, st);
        case 16: return launch_quads<16>(p, a.averages, st);
        case 32: return launch_quads<32>(p, a.averages, st);
        case 64: return launch_quads<64>(p, a.averages, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace adpsgd_impl
