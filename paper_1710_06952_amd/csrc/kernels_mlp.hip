// Minibatch gradient of the two-layer perceptron  in -> hid (ReLU) -> out with
// softmax cross-entropy (Algorithm 1, gradient step, for the dense-network
// workload).  Parameters are flattened as [W1 (in x hid) | b1 | W2 (hid x out) | b2];
// the gradient reads the bf16 shadow of the stale model and bf16 inputs, and
// accumulates in fp32.  The two large products are dense contractions and run
// on the matrix cores (v_mfma_f32_16x16x32_bf16, 64-lane wavefronts):
//   forward   H  = relu(Xb W1 + b1)        M x in  times  in x hid
//   backward  dW1 = Xb^T dH                in x M  times  M x hid
// The hidden activations and their back-propagated error are rounded to bf16
// before they enter those products.  The second layer (hid x out, out <= 16) is
// small: its products are on the matrix cores in fp32.
//
// Launches per group of gradient operations: forward; softmax with the second-layer
// gradients and the hidden error dH; and, only where a dense gradient is wanted
// (the synchronous schedule, the wait-free variant), dW1.  By default dW1
// is never written out: dH stays in the pending slot and the kernel that applies the
// event (section 4 below) forms the rank-M product tile by tile while it updates the
// model.  The kernels of a round form a serial chain of small grids, so each one
// keeps all its global loads in flight at once instead of looping over them.  Every
// reduction has a fixed order: results do not depend on scheduling.
#include <algorithm>

#include "chains.hpp"
#include "device_common.hpp"
#include "internal.hpp"

namespace adpsgd_impl {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint16_t v8h __attribute__((ext_vector_type(8)));

constexpr int kT = 256;          // 4 wavefronts
constexpr int kMaxM = 64;        // minibatch rows held by one block (4 MFMA row tiles)
constexpr int kMaxOut = 16;
constexpr int kTileH = 64;       // hidden columns per block: 16 per wavefront

struct MlpParams {
    const float* X;
    const uint16_t* Xb;
    int64_t ld;
    int in, hid, out;
    const GradOp* ops;
    int M;
    const int32_t* batch_by_op;   // [op][M] minibatch indices, in the order of ops
    float* slots;
    float gscale;
    float* loss;
    uint16_t* Hb;    // [op][kMaxM][hid]  relu output, bf16
    uint16_t* dHb;   // [op][kMaxM][hid]  error at the hidden pre-activation, bf16, rows >= M zero
    int factored;    // dH goes to the start of the operation's pending slot instead (and stays there
                     // until the update kernel multiplies it with the inputs)
    float* logit_part;  // [op][hid / 32][kMaxM][kMaxOut]  second-layer products of one forward tile
    // Left by the forward kernel for the one that follows, so that its loads depend on nothing but its block index
    // (a kernel of this chain is a few memory round trips long; each dependent load it sheds is one of them):
    int32_t* labels;    // [op][kMaxM]  class of every sample of the minibatch, -1 beyond M
    float* W2f;         // [op][hid][kMaxOut]  the second layer's weights as fp32, zero beyond `out`
    float* b2f;         // [op][kMaxOut]
};

__device__ __forceinline__ v4f mfma_bf16(v8h a, v8h b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// Operand layout of v_mfma_f32_16x16x32_bf16 (D = A B + C, A 16x32, B 32x16):
//   lane l supplies A[l % 16][8 (l / 16) .. +7] and B[8 (l / 16) .. +7][l % 16];
//   lane l receives D[4 (l / 16) + v][l % 16] in element v of its 4 results.

// ---- 0. wait-free variant: the compensated copy of the model a gradient reads ---------------
// For operations that carry a pending gradient g_k' (dense, in slot comp_slot):
//     xrow = bf16(x^i - gamma_k' g_k')        (two fp32 roundings, then round to nearest even)
// grid = (ceil(ld / 1024), n_ops); operations without compensation return at once.
__global__ __launch_bounds__(kT) void mlp_compensated_rows_kernel(const MlpParams p) {
    const GradOp op = p.ops[blockIdx.y];
    if (op.comp_slot < 0 || !op.xrow_bf16) return;
    const int64_t e = 4 * (static_cast<int64_t>(blockIdx.x) * kT + threadIdx.x);
    if (e >= p.ld) return;
    const v4f x = *reinterpret_cast<const v4f*>(p.X + static_cast<int64_t>(op.worker) * p.ld + e);
    const v4f g = *reinterpret_cast<const v4f*>(p.slots + static_cast<int64_t>(op.comp_slot) * p.ld + e);
    v4f c;
    {
#pragma clang fp contract(off)
        const v4f step = g * op.comp_gamma;
        c = x - step;
    }
    uint16_t* __restrict__ dst = static_cast<uint16_t*>(const_cast<void*>(op.xrow_bf16)) + e;
    *reinterpret_cast<v4h*>(dst) = v4h{bf16_rne(c.x), bf16_rne(c.y), bf16_rne(c.z), bf16_rne(c.w)};
}

// ---- 1. forward: H = relu(Xb W1 + b1), grid = (hid / 32, n_ops, ceil(M / 32)) ----------------------
// One block (512 threads) owns a 32 (minibatch) x 32 (hidden) tile of H (two blocks share a weight tile when the
// minibatch has more than 32 samples: a block then pulls 100 KB of operands through its compute unit instead
// of 150 KB, a round of four gradients fills the chip, and the two land on the same XCD).  The contraction over
// the input features is split across the eight wavefronts (k-steps of 32, step s goes to
// wavefront s % 8), each with its own transposed W1 tile in LDS; the operands of up to kFwdDepth
// steps of a wavefront (all of them for 784 inputs) are requested before the first MFMA, so the
// kernel pays the memory latency once.  The eight partial tiles are added through LDS in a fixed order
// -- pairs (w, w + 4) first, then the four sums in sequence -- every thread finishing two elements of the
// tile, and two wavefronts add the block's share of the logits on the matrix cores.  What follows the
// contraction is a chain of short steps: partial tiles in memory of their own and one step instead of two for their sum
// (two barriers instead of five), the logits on the matrix cores instead of 32 products a thread, and two rows of W1 to
// a word where the tile is transposed took 784-1024-10 (M = 64, six gradients) from 11.6 to 9.5 us, 64-256-10 (M = 32) from 5.3
// to 4.6.
// tile handled by block x of a row of G blocks: consecutive tiles on the same XCD (block x runs on XCD x % 8
// when G is a multiple of 8, as it is for every supported hidden size that is a multiple of 256)
__device__ __forceinline__ int xcd_neighbours(int x, int G) { return (G & 7) == 0 ? (x & 7) * (G >> 3) + (x >> 3) : x; }

constexpr int kFwdTileH = 32;
constexpr int kFwdT = 512;
constexpr int kFwdWaves = kFwdT / 64;
constexpr int kFwdDepth = 4;
constexpr int kFwdMT = 2;                  // 16-row minibatch tiles per block
constexpr int kFwdRows = 16 * kFwdMT;      // minibatch rows per block
constexpr int kFwdElems = kFwdMT * 2 * 4;  // accumulator elements per lane: (mt, ht, v)

struct FwdOperands {
    v8h w[2];        // W1 tile 32 (k) x 32 (h): lane holds 2 rows k, 8 columns each
    v8h a[kFwdMT];   // input fragments of the block's 16-row minibatch tiles
};

__global__ __launch_bounds__(kFwdT) void mlp_forward_kernel(const MlpParams p) {
    __shared__ __attribute__((aligned(16))) uint16_t tiles[kFwdWaves][kFwdTileH][40];      // W1 tiles of the wavefronts, [h][k]
    __shared__ float red[kFwdWaves * kFwdElems * 64];                                      // their partial tiles
    __shared__ float W2s[kFwdTileH][kMaxOut];     // this tile's rows of W2, zero beyond `out`
    __shared__ float Hs[kFwdRows][kFwdTileH + 1];  // the finished tile, as the next layer sees it
    const int m0 = kFwdRows * blockIdx.z;          // first minibatch row of this block
    const bool first_rows = blockIdx.z == 0;       // this block also leaves what does not depend on the rows
    const GradOp op = p.ops[blockIdx.y];
    const Global<uint16_t> feat = in_global<uint16_t>(op.features);
    const int32_t* __restrict__ idx = p.batch_by_op + static_cast<int64_t>(blockIdx.y) * p.M;   // independent of op
    const Global<uint16_t> W1 = in_global<uint16_t>(op.xrow_bf16 ? op.xrow_bf16 : p.Xb + static_cast<int64_t>(op.worker) * p.ld);
    const Global<uint16_t> b1 = W1 + static_cast<int64_t>(p.in) * p.hid;
    // Blocks go to the 8 XCDs round robin, each with an L2 of its own, and a 32-column tile of bf16 weights
    // is half a 128-byte line: neighbouring tiles are given to blocks of the same XCD, so that a line of W1
    // is fetched from memory once instead of twice (rocprofv3 FETCH_SIZE at 784-1024-10: 3.8 -> 2.35 MB per
    // gradient, of which 1.6 MB are W1 and 0.8 MB the minibatch inputs once per XCD; the time of this
    // latency-bound kernel does not change).
    const int tile = xcd_neighbours(blockIdx.x, gridDim.x);
    const int h0 = tile * kFwdTileH;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 15, kb = 8 * (lane >> 4);
    // small operands of the epilogue, requested now and used after the contraction
    uint16_t w2raw, b2raw = 0;
    int32_t label = -1;
    const uint16_t b1raw = b1[h0 + 16 * ((wave >> 2) & 1) + li];   // bias of the hidden unit this thread finishes
    {
        const Global<uint16_t> W2 = b1 + p.hid;
        const int hh = threadIdx.x / kMaxOut, o = threadIdx.x % kMaxOut;     // 512 = 32 x 16
        w2raw = o < p.out ? W2[static_cast<int64_t>(h0 + hh) * p.out + o] : static_cast<uint16_t>(0);
        if (tile == 0 && first_rows) {   // one block also leaves the labels and the output bias for the next kernel
            if (threadIdx.x < kMaxM && static_cast<int>(threadIdx.x) < p.M)
                label = in_global<int32_t>(op.targets)[idx[threadIdx.x]];
            if (threadIdx.x < kMaxOut && static_cast<int>(threadIdx.x) < p.out)
                b2raw = W2[static_cast<int64_t>(p.hid) * p.out + threadIdx.x];
        }
    }
    uint16_t(*const Bt)[40] = tiles[wave];

    Global<uint16_t> rowp[kFwdMT];
#pragma unroll
    for (int mt = 0; mt < kFwdMT; ++mt) {
        const int m = m0 + 16 * mt + li;
        rowp[mt] = m < p.M ? feat + static_cast<int64_t>(idx[m]) * op.ld : nullptr;
    }
    const int skk = 2 * (lane >> 2), shh = (lane & 3) * 8;   // staging role inside the wavefront: two rows, which share words in LDS
    auto fetch = [&](int step, FwdOperands& f) {
        const int k0 = 32 * step;
        const v8h zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int k = k0 + skk + r;
            f.w[r] = k < p.in ? *reinterpret_cast<Global<v8h>>(W1 + static_cast<int64_t>(k) * p.hid + h0 + shh) : zero;
        }
#pragma unroll
        for (int mt = 0; mt < kFwdMT; ++mt)
            f.a[mt] = (rowp[mt] && k0 + kb < p.in) ? *reinterpret_cast<Global<v8h>>(rowp[mt] + k0 + kb) : zero;
    };

    v4f acc[kFwdMT][2];
#pragma unroll
    for (int mt = 0; mt < kFwdMT; ++mt)
#pragma unroll
        for (int ht = 0; ht < 2; ++ht) acc[mt][ht] = v4f{0, 0, 0, 0};

    const int steps = (p.in + 31) / 32, iters = (steps + kFwdWaves - 1) / kFwdWaves;   // same trip count for every wavefront
    for (int it0 = 0; it0 < iters; it0 += kFwdDepth) {
        FwdOperands f[kFwdDepth];
#pragma unroll
        for (int u = 0; u < kFwdDepth; ++u)
            if (it0 + u < iters) fetch(wave + kFwdWaves * (it0 + u), f[u]);   // steps beyond the last one fetch zeros
#pragma unroll
        for (int u = 0; u < kFwdDepth; ++u) {
            if (it0 + u < iters) {        // the same for every thread of the block
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    *reinterpret_cast<uint32_t*>(&Bt[shh + e][skk]) = static_cast<uint32_t>(f[u].w[1][e]) << 16 | f[u].w[0][e];
                wave_lds_sync();      // the tile is this wavefront's own: no other wavefront has to wait
                v8h bfrag[2];
#pragma unroll
                for (int ht = 0; ht < 2; ++ht) bfrag[ht] = *reinterpret_cast<const v8h*>(&Bt[16 * ht + li][kb]);
#pragma unroll
                for (int mt = 0; mt < kFwdMT; ++mt)
#pragma unroll
                    for (int ht = 0; ht < 2; ++ht) acc[mt][ht] = mfma_bf16(f[u].a[mt], bfrag[ht], acc[mt][ht]);
                wave_lds_sync();
            }
        }
    }
    {
        const float w2 = bf16_to_float(w2raw);
        W2s[threadIdx.x / kMaxOut][threadIdx.x % kMaxOut] = w2;
        if (first_rows) p.W2f[(static_cast<int64_t>(blockIdx.y) * p.hid + h0) * kMaxOut + threadIdx.x] = w2;     // 32 x 16 floats, contiguous
        if (tile == 0 && first_rows) {
            if (threadIdx.x < kMaxM) p.labels[static_cast<int64_t>(blockIdx.y) * kMaxM + threadIdx.x] = label;
            if (threadIdx.x < kMaxOut) p.b2f[static_cast<int64_t>(blockIdx.y) * kMaxOut + threadIdx.x] = bf16_to_float(b2raw);
        }
    }
    // element q = (mt, ht, v) of lane l of partial tile w at red[(w * kFwdElems + q) * 64 + l]
#pragma unroll
    for (int mt = 0; mt < kFwdMT; ++mt)
#pragma unroll
        for (int ht = 0; ht < 2; ++ht)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(wave * kFwdElems + (mt * 2 + ht) * 4 + v) * 64 + lane] = acc[mt][ht][v];
    __syncthreads();
    // every thread finishes kFwdElems / 8 elements: q = wave + 8 j
#pragma unroll
    for (int j = 0; j < kFwdElems / kFwdWaves; ++j) {
        const int q = wave + kFwdWaves * j;
        float pair[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) pair[w] = red[(w * kFwdElems + q) * 64 + lane] + red[((w + 4) * kFwdElems + q) * 64 + lane];
        const float sum = ((pair[0] + pair[1]) + pair[2]) + pair[3];
        const int mt = q >> 3, ht = (q >> 2) & 1, v = q & 3;
        const int ml = 16 * mt + 4 * (lane >> 4) + v, m = m0 + ml, hh = 16 * ht + li;    // row inside the block, and of the minibatch
        float hval = 0.0f;
        if (m < p.M) {
            const float pre = sum + bf16_to_float(b1raw);
            const uint16_t hb = bf16_rne(pre > 0.0f ? pre : 0.0f);
            p.Hb[(static_cast<int64_t>(blockIdx.y) * kMaxM + m) * p.hid + h0 + hh] = hb;
            hval = bf16_to_float(hb);
        }
        Hs[ml][hh] = hval;
    }
    __syncthreads();
    // this tile's share of the logits, over the 32 hidden units in order: a step of the matrix cores adds its four products one after
    // the other, so an entry has the bits of a chain of fused multiply-adds
    if (wave < kFwdMT) {
        const int lgrp = lane >> 4;
        v4f part = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < kFwdTileH / 4; ++s)
            part = __builtin_amdgcn_mfma_f32_16x16x4f32(Hs[16 * wave + li][4 * s + lgrp], W2s[4 * s + lgrp][li], part, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            p.logit_part[((static_cast<int64_t>(blockIdx.y) * gridDim.x + tile) * kMaxM + m0 + 16 * wave + 4 * lgrp + v) * kMaxOut + li] = part[v];
    }
}

// ---- 2. softmax, second-layer gradients and the hidden error: grid = (hid / 64, n_ops) ----
// 1024 threads.  The grid is small and the work per block is a chain of short dependent steps,
// so the block is wide: every step is spread over 16 wavefronts and every global operand is
// requested before the first one is used.
//   a. thread (m, o) finishes logit o of sample m (sum of the hid / 32 forward-tile contributions
//      in tile order); the 16 lanes of a sample take the softmax together (butterfly max and sum).
//      The 16 blocks of a gradient repeat this small step rather than wait for a kernel of its own.
//   b. wavefront (ht, mt): hidden units 16 ht .. + 15 of the block's 64 and the sample groups mt, mt + 4, mt + 8 and mt + 12
//      of four samples each.  Both products are on the matrix cores in fp32 (16x16x4): the hidden error dH = dl W2^T
//      (rounded to bf16), in four steps over the outputs in order, and dW2 = H^T dl, one step per sample group.
//      A step adds its four products one after the other, so an entry has the bits of a chain of fused multiply-adds, and
//      the sample groups are added as the fixed pairwise tree (g, g + 8), (g, g + 4), (g, g + 2), (g, g + 1): a hidden
//      error next to a boundary of its bf16 rounding falls on the same side whichever unit forms the sums.
//      Operands arrive by rows (a lane's four outputs, its four samples) and are transposed between the four groups of 16
//      lanes in registers.
//   c. the last two steps of the tree through LDS, one thread per (h, o).
// (On the vector ALUs, with a tree of eight barriers over 16 row groups, this kernel took 8.8 us for the rounds of
// 784-1024-10, M = 64, and 7.3 us for those of 64-256-10, M = 32; 6.6 and 5.7 with the products on the matrix cores, 6.4 and 5.5 with
// the softmax's maximum and sum by rotations in a row of 16 lanes instead of trips through LDS.)
constexpr int kBwdT = 1024;

// r[v] of the lanes 16 g .. + 15  <->  r[g] of the lanes 16 v .. + 15
__device__ __forceinline__ void transpose_groups(float (&r)[4]) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(r[v]), __float_as_uint(r[v + 2]), false, false);
        r[v] = __uint_as_float(s[0]);
        r[v + 2] = __uint_as_float(s[1]);
    }
#pragma unroll
    for (int v = 0; v < 4; v += 2) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(r[v]), __float_as_uint(r[v + 1]), false, false);
        r[v] = __uint_as_float(s[0]);
        r[v + 1] = __uint_as_float(s[1]);
    }
}

// the value k lanes further in a row of 16: no trip through LDS.  After k = 8 both halves of a row hold the same, after 4 all quarters,
// so rotations by 8, 4, 2, 1 pair the values that a butterfly pairs.
template <int k>
__device__ __forceinline__ float rotated(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + k, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, rotated<8>(v));
    v = fmaxf(v, rotated<4>(v));
    v = fmaxf(v, rotated<2>(v));
    return fmaxf(v, rotated<1>(v));
}
__device__ __forceinline__ float row_total(float v) {
    v += rotated<8>(v);
    v += rotated<4>(v);
    v += rotated<2>(v);
    return v + rotated<1>(v);
}

__global__ __launch_bounds__(kBwdT) void mlp_backward_small_kernel(const MlpParams p) {
    __shared__ __attribute__((aligned(16))) float dl_s[kMaxM][kMaxOut];   // softmax - onehot, zero beyond M and out
    __shared__ float loss_s[kMaxM];
    __shared__ float red[4][64][kMaxOut];           // shares of dW2, by mt
    __shared__ float red1[4][64];                   // shares of db1
    const GradOp op = p.ops[blockIdx.y];     // needed for the stores only: no load below waits for it
    uint16_t* __restrict__ dH = p.factored ? reinterpret_cast<uint16_t*>(p.slots + static_cast<int64_t>(op.slot) * p.ld)
                                           : p.dHb + static_cast<int64_t>(blockIdx.y) * kMaxM * p.hid;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lrow = lane & 15, lgrp = lane >> 4;
    const int ht = wave & 3, mt = wave >> 2;
    const int hl = 16 * ht + lrow, h = blockIdx.x * 64 + hl;      // this lane's hidden unit ...
    const int m0 = 16 * lgrp + 4 * mt;                            // ... and the first of its four samples
    const int sm = threadIdx.x >> 4, so = threadIdx.x & 15;       // step a: sample and logit

    // ---- all global loads (everything the forward kernel left in the scratch memory, addressed by block index)
    const int label = p.labels[static_cast<int64_t>(blockIdx.y) * kMaxM + sm];      // -1 beyond M
    const int tiles = p.hid / kFwdTileH;
    const float* __restrict__ src = p.logit_part + (static_cast<int64_t>(blockIdx.y) * tiles * kMaxM + sm) * kMaxOut + so;
    constexpr int kTileBatch = 32;
    float part[kTileBatch];
#pragma unroll
    for (int t = 0; t < kTileBatch; ++t) part[t] = t < tiles ? src[static_cast<int64_t>(t) * kMaxM * kMaxOut] : 0.0f;
    const float b2v = p.b2f[static_cast<int64_t>(blockIdx.y) * kMaxOut + so];         // zero beyond `out`
    // outputs 4 lgrp .. + 3 of the hidden unit
    const v4f w2v = *reinterpret_cast<const v4f*>(p.W2f + (static_cast<int64_t>(blockIdx.y) * p.hid + h) * kMaxOut + 4 * lgrp);
    uint16_t hraw[4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
        hraw[v] = p.Hb[(static_cast<int64_t>(blockIdx.y) * kMaxM + min(m0 + v, p.M - 1)) * p.hid + h];

    // ---- a. logits and softmax
    {
        float z = 0.0f;
#pragma unroll
        for (int t = 0; t < kTileBatch; ++t) z += part[t];
        for (int t0 = kTileBatch; t0 < tiles; t0 += kTileBatch) {      // hidden layers wider than 1024
#pragma unroll
            for (int t = 0; t < kTileBatch; ++t) part[t] = (t0 + t < tiles) ? src[static_cast<int64_t>(t0 + t) * kMaxM * kMaxOut] : 0.0f;
#pragma unroll
            for (int t = 0; t < kTileBatch; ++t) z += part[t];
        }
        const bool live = so < p.out;
        const float logit = live ? z + b2v : -INFINITY;
        const float zmax = row_max(logit);
        const float ez = live ? expf(logit - zmax) : 0.0f;
        const float zsum = row_total(ez);
        const int lsrc = (threadIdx.x & 48) + (label >= 0 && label < p.out ? label : 0);   // lane of the labelled class
        const float lsel = __shfl(logit, lsrc, 64);
        dl_s[sm][so] = (live && sm < p.M) ? ez / zsum - (so == label ? 1.0f : 0.0f) : 0.0f;
        if (so == 0) loss_s[sm] = sm < p.M ? -(lsel - zmax - logf(zsum)) : 0.0f;
    }
    // operands of step b that do not come from this step, before the barrier
    float w2[4] = {w2v.x, w2v.y, w2v.z, w2v.w}, hs[4], hv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) hs[v] = hv[v] = m0 + v < p.M ? bf16_to_float(hraw[v]) : 0.0f;
    transpose_groups(w2);         // w2[s]: output 4 s + lgrp
    transpose_groups(hs);         // hs[q]: sample lgrp of group mt + 4 q
    __syncthreads();

    // ---- b. dH and this wavefront's share of dW2
    float* __restrict__ g = p.slots + static_cast<int64_t>(op.slot) * p.ld;
    float* __restrict__ gb1 = g + static_cast<int64_t>(p.in) * p.hid;
    float* __restrict__ gW2 = gb1 + p.hid;
    float* __restrict__ gb2 = gW2 + static_cast<int64_t>(p.hid) * p.out;
    {
        // rows of the product of dH: sample 16 (i / 4) + 4 mt + i % 4 in row i, so a lane's results are its four samples
        const v4f dl4 = *reinterpret_cast<const v4f*>(&dl_s[16 * (lrow >> 2) + 4 * mt + (lrow & 3)][4 * lgrp]);     // zero beyond M and out
        float dl[4] = {dl4.x, dl4.y, dl4.z, dl4.w};
        transpose_groups(dl);
        v4f back = {0, 0, 0, 0};      // entries o >= out are zero in dl and w2
#pragma unroll
        for (int s = 0; s < 4; ++s) back = __builtin_amdgcn_mfma_f32_16x16x4f32(dl[s], w2[s], back, 0, 0, 0);
        v4f share[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            share[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(hs[q], dl_s[16 * q + 4 * mt + lgrp][lrow], v4f{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) red[mt][16 * ht + 4 * lgrp + v][lrow] = (share[0][v] + share[2][v]) + (share[1][v] + share[3][v]);
        float sum_dh = 0.0f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const uint16_t rounded = bf16_rne(back[v] * p.gscale), dh = hv[v] > 0.0f ? rounded : static_cast<uint16_t>(0);
            sum_dh += bf16_to_float(dh);
            dH[static_cast<int64_t>(m0 + v) * p.hid + h] = dh;    // rows m >= M are the zero padding of the dW1 product
        }
        sum_dh += __shfl_xor(sum_dh, 32, 64);
        sum_dh += __shfl_xor(sum_dh, 16, 64);
        if (lgrp == 0) red1[mt][hl] = sum_dh;
    }
    __syncthreads();

    // ---- c. the four shares
    {
        const int hh = threadIdx.x >> 4, o = threadIdx.x & 15;       // 1024 = 64 hidden units x 16 outputs
        const float sum = (red[0][hh][o] + red[2][hh][o]) + (red[1][hh][o] + red[3][hh][o]);
        if (o < p.out) gW2[static_cast<int64_t>(blockIdx.x * 64 + hh) * p.out + o] = sum * p.gscale;
        if (threadIdx.x < 64)
            gb1[blockIdx.x * 64 + threadIdx.x] = (red1[0][threadIdx.x] + red1[2][threadIdx.x]) + (red1[1][threadIdx.x] + red1[3][threadIdx.x]);
    }
    if (blockIdx.x == 0 && wave == 1 && lane < p.out) {
        float sdl = 0.0f;
        for (int m = 0; m < p.M; ++m) sdl += dl_s[m][lane];
        gb2[lane] = sdl * p.gscale;
    }
    if (blockIdx.x == 0 && threadIdx.x == 128 && p.loss) {
        float sl = 0.0f;
        for (int m = 0; m < p.M; ++m) sl += loss_s[m];
        p.loss[op.event] = sl * p.gscale;
    }
}

// ---- 2b. loss only (evaluation of the objective): grid = n_ops, 1024 threads ------------------
// Step a of the backward kernel without the rest: logits, softmax, cross-entropy of the first
// `count` samples of each operation, summed in sample order in fp64.  count_errors: a sample
// contributes 1 when its largest logit (the lowest class on ties) is not its label, else 0.
__global__ __launch_bounds__(kBwdT) void mlp_loss_kernel(const MlpParams p, double* loss_sum, int count_errors) {
    __shared__ float loss_s[kMaxM];
    const GradOp op = p.ops[blockIdx.x];
    const int sm = threadIdx.x >> 4, so = threadIdx.x & 15;
    const int label = p.labels[static_cast<int64_t>(blockIdx.x) * kMaxM + sm];       // left by the forward kernel, -1 beyond M
    const int tiles = p.hid / kFwdTileH;
    const float* __restrict__ src = p.logit_part + (static_cast<int64_t>(blockIdx.x) * tiles * kMaxM + sm) * kMaxOut + so;
    float z = 0.0f;
    for (int t0 = 0; t0 < tiles; t0 += 32) {
        float part[32];
#pragma unroll
        for (int t = 0; t < 32; ++t) part[t] = (t0 + t < tiles) ? src[static_cast<int64_t>(t0 + t) * kMaxM * kMaxOut] : 0.0f;
#pragma unroll
        for (int t = 0; t < 32; ++t) z += part[t];
    }
    const bool live = so < p.out;
    const float logit = live ? z + p.b2f[static_cast<int64_t>(blockIdx.x) * kMaxOut + so] : -INFINITY;
    float zmax = logit;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, off, 64));
    float zsum = live ? expf(logit - zmax) : 0.0f;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) zsum += __shfl_xor(zsum, off, 64);
    const int lsrc = (threadIdx.x & 48) + (label >= 0 && label < p.out ? label : 0);
    const float lsel = __shfl(logit, lsrc, 64);
    int best = live && logit == zmax ? so : kMaxOut;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) best = min(best, __shfl_xor(best, off, 64));
    if (so == 0) loss_s[sm] = count_errors ? (best != label ? 1.0f : 0.0f) : -(lsel - zmax - logf(zsum));
    __syncthreads();
    if (threadIdx.x == 0) {
        const int count = op.count > 0 ? (op.count < p.M ? op.count : p.M) : p.M;
        double s = 0.0;
        for (int m = 0; m < count; ++m) s += loss_s[m];
        loss_sum[blockIdx.x] = s;
    }
}

// ---- 3. dW1 = Xb^T dH ------------------------------------------------------------------
// One 64 (inputs) x 64 (hidden) tile of the product: the minibatch rows of the inputs and of dH
// ([kMaxM][hid] bf16, rows >= M zero) are transposed through LDS, then wavefront w multiplies the
// four 16-row input tiles with hidden columns [16 w, 16 w + 16).  Lane l ends up with
// acc[it][v] = dW1[i0 + 16 it + 4 (l / 16) + v][h0 + 16 w + l % 16].
__device__ __forceinline__ void dw1_tile(Global<uint16_t> feat, int64_t feat_ld, const int32_t* __restrict__ idx,
                                         int M, int in, const uint16_t* __restrict__ dH, int hid, int h0, int i0,
                                         uint16_t (*At)[72], uint16_t (*Bt)[72], v4f acc[4]) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 15, kb = 8 * (lane >> 4);
    {   // stage: thread handles one minibatch row m and 16 consecutive columns
        const int m = threadIdx.x >> 2, seg = (threadIdx.x & 3) * 16;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int c = seg + 8 * half;
            v8h xv = {0, 0, 0, 0, 0, 0, 0, 0};
            if (m < M && i0 + c < in) xv = *reinterpret_cast<Global<v8h>>(feat + static_cast<int64_t>(idx[m]) * feat_ld + i0 + c);
            const v8h dv = *reinterpret_cast<const v8h*>(dH + static_cast<int64_t>(m) * hid + h0 + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                At[c + e][m] = xv[e];
                Bt[c + e][m] = dv[e];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 4; ++it) acc[it] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const v8h bfrag = *reinterpret_cast<const v8h*>(&Bt[16 * wave + li][32 * ks + kb]);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const v8h afrag = *reinterpret_cast<const v8h*>(&At[16 * it + li][32 * ks + kb]);
            acc[it] = mfma_bf16(afrag, bfrag, acc[it]);
        }
    }
}

// dW1 written out as a dense gradient: grid = (hid / 64, ceil(in / 64), n_ops)
__global__ __launch_bounds__(kT) void mlp_dw1_kernel(const MlpParams p) {
    __shared__ __attribute__((aligned(16))) uint16_t At[64][72];   // inputs transposed:  [i][m], 64 m + pad
    __shared__ __attribute__((aligned(16))) uint16_t Bt[64][72];   // hidden error transposed: [h][m]
    const GradOp op = p.ops[blockIdx.z];
    const int h0 = blockIdx.x * kTileH, i0 = blockIdx.y * 64;
    v4f acc[4];
    dw1_tile(in_global<uint16_t>(op.features), op.ld, p.batch_by_op + static_cast<int64_t>(blockIdx.z) * p.M, p.M, p.in,
             p.dHb + static_cast<int64_t>(blockIdx.z) * kMaxM * p.hid, p.hid, h0, i0, At, Bt, acc);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float* __restrict__ g = p.slots + static_cast<int64_t>(op.slot) * p.ld;
    const int h = h0 + 16 * wave + (lane & 15);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + 16 * it + 4 * (lane >> 4) + v;
            if (i < p.in) g[static_cast<int64_t>(i) * p.hid + h] = acc[it][v];
        }
    }
}

// ---- 4. model update with dW1 in factored form ----------------------------------------------
// An event's update  avg = (x^i + x^j) / 2;  x^j <- avg;  x^i <- avg - gamma g  for the
// perceptron, with the first-layer part of g formed here from its factors (the same product
// as above, so the values are those of the dense gradient) and only the small remainder
// (b1, W2, b2) read from the pending slot.  The bf16 shadow of the rows is rewritten.
// A block executes a chain of up to kLinks updates that share rows on its tile: the rows are
// read once, stay in registers from update to update and are written once, and the operands of the
// next product are on their way while one is applied.
// A round is a chain of three kernels with latency for most of its time, so fewer rounds count for more than their length: with
// updates that may follow each other in a round 784-1024-10 (n = 16, M = 64, T_max = 4, 1000 events) takes 175 rounds instead of 296,
// 8.36 -> 6.0 ms when they were written (5.4 now: 9.5 us forward, 6.4 softmax, 15.2 here); 64-256-10 with momentum (n = 16, M = 32,
// 1024 events) 164 rounds instead of 254, 4.0 -> 2.85 ms (2.6 now: 4.6, 5.5, 6.3).  mlp_chain has how long a chain may be.
//   grid = (hid / 64, in_tiles + further rows, chains of the round), in launches of 65 535 rows at most (more than 2 M
//   inputs, or 1 M with dense gradients, need several); row = row0 + blockIdx.y:
//   row <  in_tiles: one 32 x 64 tile of W1.  The tile of g goes through LDS so that
//                 each thread updates float4 pieces of contiguous rows (16 lanes per 256-byte row);
//   row >= in_tiles: 1024 consecutive floats of the remainder (or, where the gradients are dense,
//                 of all parameters), elementwise.
struct MlpApplyParams {
    float* X;
    int64_t ld;
    int64_t d;
    int in, hid, M;
    const UpdateChain* chains;
    const float* slots;
    uint16_t* Xbf16;
    const int32_t* batch_by_op;   // [op][M]
    int in_tiles;            // rows of tiles of W1: ceil(in / 32), or 0 with dense gradients
    int row0;                // first row of blocks of this launch (MORE), else 0
    int64_t dense_from;      // the parameters behind them
    float* V;                // momentum buffers (MOM), else nullptr
    float momentum, weight_decay;
};

constexpr int kApplyRows = 32;              // inputs of a tile

template <int kLinks, bool MOM, bool MORE>
__global__ __launch_bounds__(kT, 4) void mlp_apply_chains_kernel(const MlpApplyParams p) {
    constexpr int kPlaces = kLinks + 1;       // rows of a chain of kLinks operations
    __shared__ __attribute__((aligned(16))) uint16_t At[kApplyRows][72];   // inputs transposed:  [i][m], 64 m + pad
    __shared__ __attribute__((aligned(16))) uint16_t Bt[64][72];           // hidden error transposed: [h][m]
    __shared__ __attribute__((aligned(16))) float Gs[kApplyRows][68];      // the tile of g, [input][hidden]
    const UpdateChain chain = chain_at(p.chains + blockIdx.z);
    const int n_ops = chain.n_ops;
    const int block_row = (MORE ? p.row0 : 0) + static_cast<int>(blockIdx.y);
    if (block_row >= p.in_tiles) {
        // elementwise, with dense gradients from the slots
        const int64_t from = p.dense_from + 4 * kT * (static_cast<int64_t>(block_row - p.in_tiles) * gridDim.x + blockIdx.x);
        const int64_t e = from + 4 * threadIdx.x, left = (p.d + 3) / 4 * 4 - from;       // rows are padded to whole vectors
        if (e >= p.d) return;
        const int bytes = left < 4 * kT ? 4 * static_cast<int>(left) : 16 * kT, offset = 16 * threadIdx.x;
        ChainRows<MOM, kPlaces, 1> c;
#pragma unroll
        for (int q = 0; q < kPlaces; ++q) {
            const int64_t at = static_cast<int64_t>(max(chain.rows[q], 0)) * p.ld + from;
            c.x[q][0] = buffer_load4<false>(buffer_of(p.X + at, chain.rows[q] >= 0 ? bytes : 0), offset);
            if constexpr (MOM) c.v[q][0] = buffer_load4<false>(buffer_of(p.V + at, (chain.steps >> q & 1) != 0 ? bytes : 0), offset);
        }
        v4f g[kLinks][1];
#pragma unroll
        for (int u = 0; u < kLinks; ++u)
            g[u][0] = buffer_load4<false>(buffer_of(p.slots + static_cast<int64_t>(chain.ops[u].slot) * p.ld + from, u < n_ops ? bytes : 0), offset);
#pragma unroll
        for (int u = 0; u < kLinks; ++u)
            if (u == 0 || u < n_ops) c.update(chain.ops[u], p.momentum, p.weight_decay, g[u]);
#pragma unroll
        for (int q = 0; q < kPlaces; ++q) {
            if (chain.rows[q] < 0) continue;
            const int64_t at = static_cast<int64_t>(chain.rows[q]) * p.ld + e;
            const bool steps = MOM && (chain.steps >> q & 1) != 0;
            const v4f w = c.x[q][0], m = MOM ? c.v[MOM ? q : 0][0] : v4f{0, 0, 0, 0};
            const v4h s = {bf16_rne(w.x), bf16_rne(w.y), bf16_rne(w.z), bf16_rne(w.w)};
            if (e + 4 <= p.d) {
                *reinterpret_cast<v4f*>(p.X + at) = w;
                *reinterpret_cast<v4h*>(p.Xbf16 + at) = s;
                if (steps) *reinterpret_cast<v4f*>(p.V + at) = m;
            } else {                                            // entries at and beyond d stay untouched
                const float wv[4] = {w.x, w.y, w.z, w.w}, mv[4] = {m.x, m.y, m.z, m.w};
                const uint16_t sv[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (e + k < p.d) {
                        p.X[at + k] = wv[k];
                        p.Xbf16[at + k] = sv[k];
                        if (steps) p.V[at + k] = mv[k];
                    }
            }
        }
        return;
    }
    const int h0 = blockIdx.x * kTileH, i0 = block_row * kApplyRows;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, kb = 8 * (lane >> 4);
    const int rr = threadIdx.x >> 4, hq = (threadIdx.x & 15) * 4;      // this thread's rows 16 r + rr, columns hq .. hq + 3
    const int m = threadIdx.x >> 2, part = threadIdx.x & 3;            // staging role: sample, quarter of the tile's columns
    const int m_in = min(m, p.M - 1), c_in = min(i0 + 8 * part, p.in - 8);
    const bool live = m < p.M && i0 + 8 * part < p.in;
    const int32_t* const index = p.batch_by_op + static_cast<int64_t>(chain.first) * p.M + m_in;
    struct Factors {
        v8h x, d[2];
    };
    Factors f;
    auto request_error = [&](const UpdateOp& op) {
        const uint16_t* const dH = reinterpret_cast<const uint16_t*>(p.slots + static_cast<int64_t>(op.slot) * p.ld);
#pragma unroll
        for (int half = 0; half < 2; ++half) f.d[half] = *reinterpret_cast<const v8h*>(dH + static_cast<int64_t>(m) * p.hid + h0 + 16 * part + 8 * half);
    };
    auto request_inputs = [&](const UpdateOp& op, int32_t row) {
        f.x = *reinterpret_cast<Global<v8h>>(in_global<uint16_t>(op.features) + static_cast<int64_t>(row) * op.feat_ld + c_in);
    };
    // indices first: loads return in order, and the inputs wait for them
    int32_t row = index[0];
    int32_t row_next = index[static_cast<int64_t>(min(1, n_ops - 1)) * p.M];
    request_error(chain.ops[0]);
    __builtin_amdgcn_sched_barrier(0);
    ChainRows<MOM, kPlaces, 2> c;
    const int64_t corner = static_cast<int64_t>(i0) * p.hid + h0;
    const int bytes = 4 * (min(kApplyRows, p.in - i0) * p.hid - h0), offset = 4 * (rr * p.hid + hq), pitch = 64 * p.hid;
#pragma unroll
    for (int q = 0; q < kPlaces; ++q) {
        const int64_t at = static_cast<int64_t>(max(chain.rows[q], 0)) * p.ld + corner;
        const Buffer x = buffer_of(p.X + at, chain.rows[q] >= 0 ? bytes : 0);
#pragma unroll
        for (int r = 0; r < 2; ++r) c.x[q][r] = buffer_load4<false>(x, offset + r * pitch);
        if constexpr (MOM) {
            const Buffer v = buffer_of(p.V + at, (chain.steps >> q & 1) != 0 ? bytes : 0);
#pragma unroll
            for (int r = 0; r < 2; ++r) c.v[q][r] = buffer_load4<false>(v, offset + r * pitch);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : "+v"(row), "+v"(row_next));       // no address before the rows are requested
    request_inputs(chain.ops[0], row);
#pragma unroll
    for (int u = 0; u < kLinks; ++u) {
        if (u > 0 && u >= n_ops) break;       // the same for the whole block; a chain has one at least
        const UpdateOp& op = chain.ops[u];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            At[8 * part + e][m] = live ? f.x[e] : static_cast<uint16_t>(0);
            Bt[16 * part + e][m] = f.d[0][e];
            Bt[16 * part + 8 + e][m] = f.d[1][e];
        }
        __syncthreads();
        if (u + 1 < kLinks) {
            request_error(chain.ops[u + 1 < kLinks ? u + 1 : u]);
            request_inputs(chain.ops[u + 1 < kLinks ? u + 1 : u], row_next);
            row_next = index[static_cast<int64_t>(min(u + 2, n_ops - 1)) * p.M];
        }
        v4f acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const v8h bfrag = *reinterpret_cast<const v8h*>(&Bt[16 * wave + li][32 * ks + kb]);
#pragma unroll
            for (int it = 0; it < 2; ++it) acc[it] = mfma_bf16(*reinterpret_cast<const v8h*>(&At[16 * it + li][32 * ks + kb]), bfrag, acc[it]);
        }
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int k = 0; k < 4; ++k) Gs[16 * it + 4 * (lane >> 4) + k][16 * wave + li] = acc[it][k];
        __syncthreads();
        const v4f g[2] = {*reinterpret_cast<const v4f*>(&Gs[rr][hq]), *reinterpret_cast<const v4f*>(&Gs[16 + rr][hq])};
        c.update(op, p.momentum, p.weight_decay, g);
    }
#pragma unroll
    for (int q = 0; q < kPlaces; ++q) {
        if (chain.rows[q] < 0) continue;
        const int64_t at = static_cast<int64_t>(chain.rows[q]) * p.ld + corner;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (i0 + 16 * r + rr >= p.in) continue;
            const int64_t e = at + static_cast<int64_t>(16 * r + rr) * p.hid + hq;
            const v4f w = c.x[q][r];
            *reinterpret_cast<v4f*>(p.X + e) = w;
            *reinterpret_cast<v4h*>(p.Xbf16 + e) = v4h{bf16_rne(w.x), bf16_rne(w.y), bf16_rne(w.z), bf16_rne(w.w)};
            if constexpr (MOM) {
                if ((chain.steps >> q & 1) != 0) *reinterpret_cast<v4f*>(p.V + e) = c.v[q][r];
            }
        }
    }
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// scratch memory of a launch group: [Hb][dHb][logit_part][W2f][labels][b2f]
struct ScratchLayout {
    size_t dHb, logit_part, W2f, labels, b2f, total;
};
ScratchLayout scratch_layout(int32_t n_ops, int32_t hid) {
    const size_t ops = static_cast<size_t>(n_ops);
    const size_t act = align256(ops * kMaxM * hid * sizeof(uint16_t));
    ScratchLayout L;
    L.dHb = act;
    L.logit_part = 2 * act;
    L.W2f = L.logit_part + align256(ops * (hid / kFwdTileH) * kMaxM * kMaxOut * 4);
    L.labels = L.W2f + align256(ops * hid * kMaxOut * 4);
    L.b2f = L.labels + align256(ops * kMaxM * 4);
    L.total = L.b2f + align256(ops * kMaxOut * 4);
    return L;
}
void set_scratch(MlpParams& p, void* scratch, int32_t n_ops, int32_t hid) {
    const ScratchLayout L = scratch_layout(n_ops, hid);
    char* s = static_cast<char*>(scratch);
    p.Hb = reinterpret_cast<uint16_t*>(s);
    p.dHb = reinterpret_cast<uint16_t*>(s + L.dHb);
    p.logit_part = reinterpret_cast<float*>(s + L.logit_part);
    p.W2f = reinterpret_cast<float*>(s + L.W2f);
    p.labels = reinterpret_cast<int32_t*>(s + L.labels);
    p.b2f = reinterpret_cast<float*>(s + L.b2f);
}

}  // namespace

size_t mlp_scratch_bytes(int32_t n_ops, int32_t M, int32_t in, int32_t hid, int32_t out) {
    if (n_ops < 1 || M < 1 || M > kMaxM || in < 8 || (in & 7) || hid < kTileH || (hid % kTileH) || out < 1 || out > kMaxOut)
        return 0;
    return scratch_layout(n_ops, hid).total;
}

hipError_t launch_mlp_loss(const MlpGradArgs& a, double* loss_sum, bool count_errors, hipStream_t st) {
    if (a.n_ops <= 0) return hipSuccess;
    if (mlp_scratch_bytes(a.n_ops, a.M, a.in, a.hid, a.out) == 0 || a.n_ops > 65535) return hipErrorInvalidValue;
    MlpParams p{};
    p.X = a.X;
    p.Xb = a.Xbf16;
    p.ld = a.ld;
    p.in = a.in;
    p.hid = a.hid;
    p.out = a.out;
    p.ops = a.ops;
    p.M = a.M;
    p.batch_by_op = a.batch_by_op;
    p.slots = a.slots;
    p.gscale = a.gscale;
    p.loss = nullptr;
    set_scratch(p, a.scratch, a.n_ops, a.hid);
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(a.hid / kFwdTileH, a.n_ops, (a.M + kFwdRows - 1) / kFwdRows), dim3(kFwdT), 0, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_loss_kernel, dim3(a.n_ops), dim3(kBwdT), 0, st, p, loss_sum, count_errors ? 1 : 0);
    return hipGetLastError();
}

bool mlp_can_factor(int32_t in, int32_t hid, int32_t M) {
    // dH (kMaxM x hid bf16) must fit the first-layer part of a pending slot (in x hid fp32)
    return M >= 1 && M <= kMaxM && in >= 32 && (in & 7) == 0 && hid >= kTileH && hid % kTileH == 0;
}

hipError_t launch_mlp_apply_chains(const MlpApplyArgs& a, hipStream_t st) {
    if (a.n_chains <= 0) return hipSuccess;
    if ((a.factored && !mlp_can_factor(a.in, a.hid, a.M)) || a.hid < kTileH || a.n_chains > 65535 || !a.Xbf16) return hipErrorInvalidValue;
    MlpApplyParams p;
    p.X = a.X;
    p.ld = a.ld;
    p.d = a.d;
    p.in = a.in;
    p.hid = a.hid;
    p.M = a.M;
    p.chains = a.chains;
    p.slots = a.slots;
    p.Xbf16 = a.Xbf16;
    p.batch_by_op = a.batch_by_op;
    p.V = a.V;
    p.momentum = a.momentum;
    p.weight_decay = a.weight_decay;
    p.in_tiles = a.factored ? (a.in + kApplyRows - 1) / kApplyRows : 0;
    p.dense_from = a.factored ? static_cast<int64_t>(a.in) * a.hid : 0;
    const int64_t bx = a.hid / kTileH, per_row = bx * kT * 4;                   // floats one grid row of blocks covers
    const int64_t by = p.in_tiles + (a.d - p.dense_from + per_row - 1) / per_row;
    if (by > 0x7FFFFFFF) return hipErrorInvalidValue;
    for (int64_t row0 = 0; row0 < by; row0 += 65535) {
        p.row0 = static_cast<int>(row0);
        const dim3 grid(static_cast<uint32_t>(bx), static_cast<uint32_t>(std::min<int64_t>(by - row0, 65535)), a.n_chains);
        if (row0 > 0 && a.V) hipLaunchKernelGGL((mlp_apply_chains_kernel<3, true, true>), grid, dim3(kT), 0, st, p);
        else if (row0 > 0) hipLaunchKernelGGL((mlp_apply_chains_kernel<3, false, true>), grid, dim3(kT), 0, st, p);
        else if (a.V) hipLaunchKernelGGL((mlp_apply_chains_kernel<3, true, false>), grid, dim3(kT), 0, st, p);
        else if (mlp_chain(false, a.d) == 3) hipLaunchKernelGGL((mlp_apply_chains_kernel<3, false, false>), grid, dim3(kT), 0, st, p);
        else hipLaunchKernelGGL((mlp_apply_chains_kernel<kChain, false, false>), grid, dim3(kT), 0, st, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mlp_gradient(const MlpGradArgs& a, hipStream_t st, int* n_launches) {
    if (a.n_ops <= 0) return hipSuccess;
    if (mlp_scratch_bytes(a.n_ops, a.M, a.in, a.hid, a.out) == 0 || a.n_ops > 65535) return hipErrorInvalidValue;
    MlpParams p;
    p.X = a.X;
    p.Xb = a.Xbf16;
    p.ld = a.ld;
    p.in = a.in;
    p.hid = a.hid;
    p.out = a.out;
    p.ops = a.ops;
    p.M = a.M;
    p.batch_by_op = a.batch_by_op;
    p.slots = a.slots;
    p.gscale = a.gscale;
    p.loss = a.loss;
    p.factored = a.factored ? 1 : 0;
    if (a.factored && !mlp_can_factor(a.in, a.hid, a.M)) return hipErrorInvalidValue;
    set_scratch(p, a.scratch, a.n_ops, a.hid);
    const uint32_t hb = static_cast<uint32_t>(a.hid / kTileH);
    if (a.compensate) {
        if (!a.X || a.factored) return hipErrorInvalidValue;
        const int64_t cb = (a.ld / 4 + kT - 1) / kT;
        hipLaunchKernelGGL(mlp_compensated_rows_kernel, dim3(static_cast<uint32_t>(cb), a.n_ops), dim3(kT), 0, st, p);
        const hipError_t ec = hipGetLastError();
        if (ec != hipSuccess) return ec;
        if (n_launches) *n_launches += 1;
    }
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(a.hid / kFwdTileH, a.n_ops, (a.M + kFwdRows - 1) / kFwdRows), dim3(kFwdT), 0, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_backward_small_kernel, dim3(a.hid / 64, a.n_ops), dim3(kBwdT), 0, st, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.factored) {
        if (n_launches) *n_launches += 2;
        return hipSuccess;
    }
    hipLaunchKernelGGL(mlp_dw1_kernel, dim3(hb, (a.in + 63) / 64, a.n_ops), dim3(kT), 0, st, p);
    if (n_launches) *n_launches += 3;
    return hipGetLastError();
}

}  // namespace adpsgd_impl
