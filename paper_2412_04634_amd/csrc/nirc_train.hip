// Training kernels: fused forward + relative-L2 loss + backward to per-workgroup weight-gradient
// partials, a fixed-order reduction, and Adam with a refresh of the packed weights.
#include "nirc_grad.hpp"
#include "nirc_split.hpp"

namespace nirc {

namespace {

constexpr int kTrainWaves = 4;
constexpr int kChunk = 16 * kTrainWaves;   // samples staged per round
constexpr int kStride = kChunk + 4;        // LDS row stride (floats): conflict-free 16 B reads

template <int W>
struct GradLds {
    static constexpr int kH = 4 * W * kStride;     // h1..h4   [layer][neuron][sample]
    static constexpr int kD = 4 * W * kStride;     // delta1..delta4
    static constexpr int kD5 = 4 * kStride;        // output-layer delta, rows 0..3
    static constexpr int kX = kChunk * kInputs;    // raw inputs [sample][10]
    static constexpr int kTotal = kH + kD + kD5 + kX;
};

// Samples of a workgroup's round in k_grad_split.
__host__ __device__ constexpr int split_round(int64_t batch) { return batch <= 64 * kMaxResidentBlocks ? 64 : 128; }

// Output-pre-activation gradient and loss term of one channel.
// rel: the relative loss (denominator y^2 + eps held constant), else den = 1; fr: the F_r shift of
// the residual-variance loss (0 otherwise)
// sig: sigmoid outputs (dy/dz = y (1 - y)) instead of exp (dy/dz = y)
__device__ inline float out_grad(float z, float t, float dr, bool use_loss, float eps, float k, bool rel,
                                 float fr, bool sig, float &loss_term) {
    const float y = sig ? logistic(z) : expf(z);
    const float dydz = sig ? y * (1.0f - y) : y;
    if (use_loss) {
        const float d = (y - t) + fr, den = rel ? y * y + eps : 1.0f;
        loss_term = d * d / den;
        return k * d / den * dydz;   // k = 2 scale / (3B)
    }
    loss_term = 0.0f;
    return k * dr * dydz;            // k = scale
}

}  // namespace

// One workgroup of 4 waves processes rounds of 64 samples.  Phase 1: each wave runs one
// 16-sample tile forward (the first layer reads all 160 features) and backward with the
// transposed packed weights, keeping activations and deltas in registers, and stages them in
// LDS as [neuron][sample].  Phase 2: each wave owns a fixed set of 16x16 weight-gradient tiles
// (a quarter of every layer's column tiles) held in registers across rounds, and adds the
// round's 64 samples with MFMAs whose K dimension is the sample index.  At the end every tile is
// written once into this workgroup's partial gradient (canonical layout).  For upstream gradients of
// any range (nirc_backward); loss gradients take k_grad_split.
template <int W>
__global__ __launch_bounds__(kTrainWaves * 64) void k_grad_f32(Points pts, Queries q,
                                                               const float *__restrict__ packed,
                                                               TrainArgs args, float *__restrict__ partials,
                                                               float *__restrict__ loss_partials) {
    static_assert(W == 64, "gradient kernel is laid out for width 64");
    constexpr F32Layout L{W};
    constexpr int MT = W / 16, KQ = W / 16;
    using S = GradLds<W>;
    __shared__ f32x4 smem4[(S::kTotal + 3) / 4];
    float *smem = (float *)smem4;
    float *sH = smem;
    float *sD = sH + S::kH;
    float *sD5 = sD + S::kD;
    float *sX = sD5 + S::kD5;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int64_t B = q.count;
    const float kscale = args.loss_scale;

    // owned gradient tiles: first layer input columns {wave, wave+4, wave+8} (< 10), column tile
    // `wave` of W2..W4 and of W5
    f32x4 g1[3][MT], gh[3][MT], g5;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            g1[a][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            gh[a][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    g5 = f32x4{0.f, 0.f, 0.f, 0.f};

    const int64_t n_chunks = (B + kChunk - 1) / kChunk;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
        // ---------------- phase 1: forward + backward of this wave's 16 samples
        {
            const float *pk = opaque(packed);
            const int s = 16 * wave + col;   // sample slot in the chunk
            const int64_t b = chunk * kChunk + s;
            const bool valid = b < B;
            const int64_t bi = valid ? b : B - 1;
            const int64_t p = query_point(q, pts, bi);
            const float xs[7] = {pts.px[p], pts.py[p], pts.pz[p], pts.nx[p], pts.ny[p], pts.nz[p], pts.rough[p]};
            const float ws[3] = {q.wx[bi], q.wy[bi], q.wz[bi]};
            if (g == 0) {
                float *x = sX + s * kInputs;
                x[0] = xs[0]; x[1] = xs[1]; x[2] = xs[2];
                x[3] = ws[0]; x[4] = ws[1]; x[5] = ws[2];
                x[6] = xs[3]; x[7] = xs[4]; x[8] = xs[5]; x[9] = xs[6];
            }
            f32x4 h[4][MT];   // h1..h4
            {
                f32x4 a1[1][MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) a1[0][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                layer1_surface<W>(a1[0], pk + L.offset(SEC_S), xs, lane, g);
                float dx[1] = {ws[0]}, dy[1] = {ws[1]}, dz[1] = {ws[2]};
                layer1_direction<W, 1>(a1, pk + L.offset(SEC_D), dx, dy, dz, lane, g);
                relu_all<W, 1>(a1);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[0][mt] = a1[0][mt];
            }
#pragma unroll
            for (int l = 1; l < 4; ++l) {
                const float *sec = pk + L.offset(SEC_H0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], h[l - 1][kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[l][mt][i] = relu_f32(o[mt][i]);
            }
            f32x4 z5 = f32x4{0.f, 0.f, 0.f, 0.f};
            {
                const float *sec = pk + L.offset(SEC_O);
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    const f32x4 a = *(const f32x4 *)(sec + (kq * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) z5 = mfma4(a[kk], h[3][kq][kk], z5);
                }
            }
            // output delta: rows 0..2 live in lanes 0..15; everything else is zero
            f32x4 d5 = f32x4{0.f, 0.f, 0.f, 0.f};
            if (g == 0 && valid) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float lt;
                    d5[c] = out_grad(z5[c], 0.0f, args.d_rgb[3 * b + c], false, args.loss_eps, kscale, false, 0.0f,
                                     args.sig != 0, lt);
                }
            }
            if (g == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) sD5[c * kStride + s] = d5[c];
            }
            // stage activations
#pragma unroll
            for (int l = 0; l < 4; ++l)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        sH[(l * W + 16 * mt + 4 * g + i) * kStride + s] = h[l][mt][i];
            // backward: delta4 = (W5^T d5) .* [h4 > 0], then through W4^T, W3^T, W2^T
            f32x4 d[MT];
            {
                const float *sec = pk + L.offset(SEC_OT);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 a = *(const f32x4 *)(sec + (mt * 64 + lane) * 4);
                    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) o = mfma4(a[kk], d5[kk], o);
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[mt][i] = h[3][mt][i] > 0.0f ? o[i] : 0.0f;
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) sD[(3 * W + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
#pragma unroll
            for (int l = 3; l >= 1; --l) {   // delta_l = (W_{l+1}^T delta_{l+1}) .* [h_l > 0]
                const float *sec = pk + L.offset(SEC_T0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], d[kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        d[mt][i] = h[l - 1][mt][i] > 0.0f ? o[mt][i] : 0.0f;
                        sD[((l - 1) * W + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
                    }
            }
        }
        __syncthreads();
        // ---------------- phase 2: owned gradient tiles += staged deltas x activations
        // K position (step kk, lane group g) of sample group sq <-> sample 16 sq + 4 g + kk
#pragma unroll 1
        for (int sq = 0; sq < kChunk / 16; ++sq) {
            const int s0 = 16 * sq + 4 * g;
            // hidden layers W2..W4 (a = 0..2) and the output layer: column tile `wave`
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const f32x4 bv = *(const f32x4 *)(sH + (a * W + 16 * wave + col) * kStride + s0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 av = *(const f32x4 *)(sD + ((a + 1) * W + 16 * mt + col) * kStride + s0);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) gh[a][mt] = mfma4(av[kk], bv[kk], gh[a][mt]);
                }
            }
            {
                const f32x4 bv = *(const f32x4 *)(sH + (3 * W + 16 * wave + col) * kStride + s0);
                f32x4 av = f32x4{0.f, 0.f, 0.f, 0.f};
                if (col < 3) av = *(const f32x4 *)(sD5 + col * kStride + s0);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) g5 = mfma4(av[kk], bv[kk], g5);
            }
            // first layer: column tile = input index; features recomputed from staged inputs
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int input = wave + 4 * a;
                if (input >= kInputs) break;
                const int k = col >> 1, sc = col & 1;
                float bv[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    float sn, cs;
                    enc_pair(sX[(s0 + kk) * kInputs + input], k, sn, cs);
                    bv[kk] = sc ? cs : sn;
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 av = *(const f32x4 *)(sD + (16 * mt + col) * kStride + s0);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) g1[a][mt] = mfma4(av[kk], bv[kk], g1[a][mt]);
                }
            }
        }
        __syncthreads();
    }

    // ---------------- write this workgroup's partial gradient (every entry exactly once)
    float *out = partials + (int64_t)blockIdx.x * n_params(W);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int input = wave + 4 * a;
        if (input >= kInputs) break;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[w_offset(W, 0) + (int64_t)(16 * mt + 4 * g + i) * kFeat + 16 * input + col] = g1[a][mt][i];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[w_offset(W, 1 + a) + (int64_t)(16 * mt + 4 * g + i) * W + 16 * wave + col] = gh[a][mt][i];
    if (g == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) out[w_offset(W, 4) + (int64_t)i * W + 16 * wave + col] = g5[i];
    }
    if (threadIdx.x == 0) loss_partials[blockIdx.x] = 0.0f;
}

// ------------------------------------------------------------------------------------------
// Loss gradients of FP32 models.  The forward pass and the deltas stay FP32: a ReLU decision that rounding
// moved would change a sample's gradient by more than rounding does, and an FP16 MFMA cuts the smaller
// products of a group at 2^-24 of the largest, which every sample's deltas would share.  (Layers 1..4 and
// the deltas below the last hidden layer are k_grad_f32's FP32 MFMAs in its order; the output layer and the
// last hidden layer's delta are vector multiply-adds in another.)  The weight gradients' sums over the
// samples take two-term FP16 operands (x s = h + l; h h + h l + l h in three 16x16x32 MFMAs of 16 cycles
// instead of eight FP32 ones of 32): their errors are the samples' own and average out.
//
// Scales: every operand set is scaled by an exact power of two that puts the largest magnitude the
// workgroup has met in it (a layer's activations, a layer's deltas) in [2^14, 2^15), so that a value's
// error is at most 2^-39 of that largest, and 22 bits are kept of a value within 2^-16 of it.  The maxima
// only grow; when one does, the sums held in registers are rescaled (exactly).  An upstream gradient of
// the caller's may span any range and stays with k_grad_f32.
//
// One scale for a layer's units suits models whose units are of like size.  Where the weights into the
// units of a layer, or out of them, differ by more than 2^kSpreadMax from unit to unit (largest magnitudes;
// initialised models 2^2, trained for 150,000 steps up to 2^9), or by more than 2^kSpreadSum over all layers
// (trained 2^22), the sums over the samples are FP32 MFMAs instead, on the same values in the same room of
// the LDS (WIDE): with units 2^40 apart the smaller ones' gradients came out 0.
//
// The weight gradient's operands hold a neuron per lane and samples in registers: each term is turned by
// an MFMA with a 0/1 selection matrix, as in the 16-bit kernels.  A workgroup of 8 waves takes rounds of
// 128 samples, 16 per wave (64 samples, a wave per SIMD, while one round of those covers the batch).
// LDS, 160 KB: the first layer's weights; the hidden layers', whose room takes the transposed ones once
// the forward pass is through and, with the activations' room, the turned inputs at the end; one layer's
// turned activations and deltas.
// 65,536 samples: 116 us (FP32 MFMA throughout, four waves, weights from L2, and 7 more for a kernel that
// drew the samples) -> 86, of which 9 are the samples' gather, 2 x 36 the rounds (17 of MFMA each).
struct GradSplit {
    static constexpr int kW1 = 0, kHT = 2560, kAct = kHT + 3072, kDel = kAct + 2048, kX = kDel + 2048, kW5 = kX + 320,
                         kD5 = kW5 + 48, kMax = kD5 + 96, kLoss = kMax + 18, kTotal = kLoss + 2;   // u32x4
    static constexpr int kRows = 512;   // a turned tile: [K-block][term][lane]
    // kMax: each wave's largest magnitudes of activations h1..h4, the output delta, deltas 1..4
    static constexpr int mH = 0, mD5 = 4, mD = 5, mCount = 9;
};
constexpr int kSplitGradWaves = 8;
constexpr int kSpreadMax = 12, kSpreadSum = 24;
constexpr uint32_t kSpreadMark = 0x53707264u;   // wide[1] once a model's weights have been looked at

// Whether the units of an FP32 model are too far apart for one scale per layer (*wide, see k_grad_split):
// looked at when weights come in from outside.  (Training moves them by a learning rate per step: a spread
// that matters, 2^17 and more, does not come about that way.)  A saved state that holds the answer keeps it, so
// that the resumed model sums as the saved one would have; one written without the mark is looked at.
__global__ __launch_bounds__(512) void k_weight_spread(const float *__restrict__ w, uint32_t *wide, bool saved_state) {
    __shared__ uint32_t most[8][64];   // incoming weights of layers 1..4, outgoing ones (layers 2..5)
    __shared__ uint32_t spread[8];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (saved_state && wide[1] == kSpreadMark) return;
    if (wave >= 4) most[wave][lane] = 0u;
    __syncthreads();
    auto mag = [&](int64_t i) { return __builtin_bit_cast(uint32_t, w[i]) & 0x7FFFFFFFu; };
    // a wave takes every eighth row of each matrix; lane: column
    uint32_t col[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int r = wave + 8 * k;
        const int64_t o = (int64_t)r * kFeat + lane;
        uint32_t in[4] = {max(max(mag(o), mag(o + 64)), lane < kFeat - 128 ? mag(o + 128) : 0u)};
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            in[1 + l] = mag(w_offset(64, 1 + l) + r * 64 + lane);
            col[l] = max(col[l], in[1 + l]);
        }
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            in[l] = wave_max(in[l]);
            if (lane == 0) most[l][r] = in[l];
        }
    }
    if (wave < 3) col[3] = mag(w_offset(64, 4) + wave * 64 + lane);
#pragma unroll
    for (int l = 0; l < 4; ++l) atomicMax(&most[4 + l][lane], col[l]);
    __syncthreads();
    const uint32_t m = most[wave][lane];
    const uint32_t hi = wave_max(m), lo = ~wave_max(m ? ~m : 0u);   // (units without weights do not count)
    if (lane == 0) spread[wave] = hi ? (hi >> 23) - (lo >> 23) : 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t most1 = 0u, in = 0u, out = 0u;
        for (int k = 0; k < 8; ++k) most1 = max(most1, spread[k]);
        for (int k = 0; k < 4; ++k) in += spread[k], out += spread[4 + k];
        wide[0] = most1 > kSpreadMax || max(in, out) > kSpreadSum;
        wide[1] = kSpreadMark;
    }
}

hipError_t launch_weight_spread(const float *w, uint32_t *wide, bool saved_state, hipStream_t s) {
    hipLaunchKernelGGL(k_weight_spread, dim3(1), dim3(512), 0, s, w, wide, saved_state);
    return hipGetLastError();
}

// The workgroup's exponent of a magnitude from its waves' (FP32 bits), within the range that scales can
// follow.
__device__ __forceinline__ int exp_of(const u32x4 *waves) {
    const u32x4 a = waves[0], b = waves[1];
    const uint32_t m = max(max(max(a[0], a[1]), max(a[2], a[3])), max(max(b[0], b[1]), max(b[2], b[3])));
    const int e = (int)(__builtin_amdgcn_readfirstlane(m) >> 23) - 127;
    return e < -100 ? -100 : e;
}
__device__ __forceinline__ float pow2f(int e) { return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23); }
__device__ __forceinline__ uint32_t mag_bits(float x) { return __builtin_bit_cast(uint32_t, x) & 0x7FFFFFFFu; }

// acc += a b over `kb` K-blocks of turned tiles, both operands in two terms.
template <int N, typename A, typename B>
__device__ __forceinline__ void add_split(f32x4 *acc, bool four, const A &a, const B &b) {
    auto block = [&](int k) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = mfma16<NIRC_FP16>(a(i, k, 1), b(i, k, 0), acc[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = mfma16<NIRC_FP16>(a(i, k, 0), b(i, k, 1), acc[i]);
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = mfma16<NIRC_FP16>(a(i, k, 0), b(i, k, 0), acc[i]);
    };
    block(0);
    block(1);
    if (!four) return;
    block(2);
    block(3);
}

// acc += a b over a round's samples in FP32: tiles [16 samples][4 samples][16 units].
template <int N, typename A, typename B>
__device__ __forceinline__ void add_wide(f32x4 *acc, bool four, const A &a, const B &b) {
#pragma unroll 1
    for (int sq = 0; sq < (four ? 8 : 4); ++sq)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const f32x4 av = a(i, sq), bv = b(i, sq);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) acc[i] = mfma4(av[kk], bv[kk], acc[i]);
        }
}

template <bool PLAIN, bool DRAW>
__global__ __launch_bounds__(kSplitGradWaves * 64) void k_grad_split(Points pts, Queries q, TrainDraw draw,
                                                                     const float *__restrict__ packed, TrainArgs args,
                                                                     float *__restrict__ partials,
                                                                     float *__restrict__ loss_partials) {
    using G = GradSplit;
    constexpr F32Layout L{64};
    constexpr int W = 64, MT = 4, KQ = 4, NT = kSplitGradWaves * 64;
    static_assert(L.offset(SEC_S) == 0 && L.offset(SEC_D) + L.size(SEC_D) == 4 * G::kHT &&
                      L.offset(SEC_H0) == 4 * G::kHT && L.offset(SEC_H2) + L.size(SEC_H2) == 4 * G::kAct,
                  "the forward sections are one run");
    static_assert(sizeof(u32x4) * G::kTotal <= 163840, "fits the LDS");
    __shared__ u32x4 smem[G::kTotal];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 15, g = lane >> 4;
    const int64_t B = q.count;
    uint32_t *sMax = (uint32_t *)(smem + G::kMax);
    const bool use_loss = PLAIN || DRAW || args.target != nullptr;
    const float kscale = use_loss ? 2.0f * args.loss_scale / (3.0f * (float)B) : args.loss_scale;
    const uint32_t wide_model = *args.wide;
    const int round_samples = split_round(B);
    const bool four = round_samples == 128, active = four || wave < 4;
    const int64_t n_chunks = (B + round_samples - 1) / round_samples, nblk = gridDim.x;
    auto sample_of = [&](int64_t chunk) {
        const int64_t b = chunk * round_samples + 16 * wave + col;
        return b < B ? b : B;
    };

    // ---------------- prologue: forward weights to LDS, the transposed weights' range, first samples
    TrainSample next;
    DrawnSample drawn;
    if (threadIdx.x < G::mCount * kSplitGradWaves) sMax[threadIdx.x] = 0u;   // (waves without samples leave theirs)
    if constexpr (!DRAW) load_query(q, args, sample_of(blockIdx.x), B, next);
    {
        constexpr int N = G::kAct / NT;
        static_assert(G::kAct % NT == 0, "whole turns");
        u32x4 t[N];
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = ((const u32x4 *)packed)[i * NT + threadIdx.x];
        f32x4 w5 = f32x4{0.f, 0.f, 0.f, 0.f};   // (channel c, K-quad kq, lane group gg): W5[c][16 kq + 4 gg ..]
        const int c5 = (int)threadIdx.x / 16, n5 = threadIdx.x & 15;
        if (threadIdx.x < 48) w5 = *(const f32x4 *)(packed + L.offset(SEC_O) + ((n5 >> 2) * 64 + 16 * (n5 & 3) + c5) * 4);
        if constexpr (DRAW)
            draw_point(pts, draw.keys, min(sample_of(blockIdx.x + g * nblk), B - 1), drawn);
        else
            load_point(pts, q, next);
#pragma unroll
        for (int i = 0; i < N; ++i) smem[i * NT + threadIdx.x] = t[i];
        if (threadIdx.x < 48) ((f32x4 *)(smem + G::kW5))[c5 * 16 + n5] = w5;
        if constexpr (DRAW) draw_target(draw.lobes, draw.keys, drawn);
    }
    __syncthreads();
    // the rounds and the partial gradient, the operands of the sums over the samples in two terms or FP32 (two
    // loops, because the choice inside one costs 4 % of it; this way 1 to 3 %)
    auto rounds = [&](auto wide) {
    constexpr bool WIDE = decltype(wide)::value;
    // this wave's tiles: W2..W4 column tile wave % 4, row tiles 2 (wave / 4) and the next; W5 column
    // tile wave (waves 0..3); W1 row tile wave % 4, inputs wave / 4 + 2 j
    const int own_n = wave & 3, own_m = 2 * (wave >> 2);
    f32x4 gh[3][2], g1[5], g5 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < 3; ++a) gh[a][0] = gh[a][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 5; ++j) g1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the largest exponents met: activations, output delta, deltas
    int eH[4] = {-100, -100, -100, -100}, eD5 = -100, eD[4] = {-100, -100, -100, -100};
    // exponents of the operands in the sums: W1, W2, W3, W4, W5
    int eg[5] = {-1000, -1000, -1000, -1000, -1000};
    auto rescale = [&](int k, int e, f32x4 *acc, int n) {
        if (WIDE) e = 28;   // (the operands carry no scale)
        if (e == eg[k]) return;
        if (eg[k] != -1000)
#pragma unroll
            for (int i = 0; i < n; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][r] = ldexpf(acc[i][r], eg[k] - e);
        eg[k] = e;
    };
    float loss_acc = 0.0f;
    const u32x4 sel[2] = {select_operand<NIRC_FP16>(0, 1.0f, g, col), select_operand<NIRC_FP16>(1, 1.0f, g, col)};
    // both terms of this wave's samples, turned: half an operand of K-block wave / 2
    auto put = [&](u32x4 *tile, const u32x4 &h, const u32x4 &l, const u32x4 &sl) {
        const f32x4 th = mfma16<NIRC_FP16>(h, sl, f32x4{0.f, 0.f, 0.f, 0.f});
        const f32x4 tl = mfma16<NIRC_FP16>(l, sl, f32x4{0.f, 0.f, 0.f, 0.f});
        uint2 *d = (uint2 *)(tile + (wave >> 1) * 128 + lane) + (wave & 1);
        d[0] = make_uint2(pack2<NIRC_FP16>(th[0], th[1]), pack2<NIRC_FP16>(th[2], th[3]));
        d[128] = make_uint2(pack2<NIRC_FP16>(tl[0], tl[1]), pack2<NIRC_FP16>(tl[2], tl[3]));
    };
    // a lane's four units (4 g ..) of its sample, FP32
    auto put_wide = [&](u32x4 *tile, float a, float b, float c, float d) {
        float *o = (float *)(tile + wave * 64 + (col >> 2) * 16 + 4 * g) + (col & 3);
        o[0] = a, o[4] = b, o[8] = c, o[12] = d;
    };
    auto put_layer = [&](u32x4 *tiles, const f32x4 (&v)[MT], float scale) {
        if constexpr (WIDE) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) put_wide(tiles + mt * G::kRows, v[mt][0], v[mt][1], v[mt][2], v[mt][3]);
            return;
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const float x[8] = {v[2 * kb][0],     v[2 * kb][1],     v[2 * kb][2],     v[2 * kb][3],
                                v[2 * kb + 1][0], v[2 * kb + 1][1], v[2 * kb + 1][2], v[2 * kb + 1][3]};
            u32x4 vh, vl;
            split8(x, scale, vh, vl);
            put(tiles + (2 * kb) * G::kRows, vh, vl, sel[0]);
            put(tiles + (2 * kb + 1) * G::kRows, vh, vl, sel[1]);
        }
    };
    auto note_max = [&](int word, uint32_t m) {
        m = wave_max(m);
        if (lane == 0) sMax[word * kSplitGradWaves + wave] = m;
    };
    auto take_max = [&](int &e, int word) { e = max(e, exp_of((const u32x4 *)(sMax + word * kSplitGradWaves))); };
    auto layer_max = [&](const f32x4 (&v)[MT]) {
        uint32_t m = 0u;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float x = v[mt][i], y = v[mt][i + 1];
                m = max(max(m, mag_bits(x)), mag_bits(y));
            }
        return m;
    };
    u32x4 *sAct = smem + G::kAct, *sDel = smem + G::kDel, *sE = smem + G::kHT;
    float *sX = (float *)(smem + G::kX);
    const f32x4 *sW5 = (const f32x4 *)(smem + G::kW5);
    uint16_t *sD5 = (uint16_t *)(smem + G::kD5);   // [K-block][term][lane group][channel][8]

    int round = 0;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += nblk, ++round) {
        const float *pk = opaque(packed);
        const int64_t b = sample_of(chunk);
        const bool valid = b < B, more = chunk + nblk < n_chunks;
        if (round > 0) {   // the hidden layers' weights again, where the turned inputs were
            constexpr int N = (G::kAct - G::kHT) / NT;
            u32x4 t[N];
#pragma unroll
            for (int i = 0; i < N; ++i) t[i] = ((const u32x4 *)pk)[G::kHT + i * NT + threadIdx.x];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < N; ++i) smem[G::kHT + i * NT + threadIdx.x] = t[i];
            __syncthreads();
        }
        f32x4 h[4][MT], d[MT];   // h1..h4; a layer's delta
        float d5[3] = {0.f, 0.f, 0.f};
        if (active) {
            float xs[7], ws[3], tg[3];
            if constexpr (DRAW) {
                if (round > 0 && (round & 3) == 0) {
                    draw_point(pts, draw.keys, min(sample_of(chunk + g * nblk), B - 1), drawn);
                    draw_target(draw.lobes, draw.keys, drawn);
                }
                const int src = 16 * (round & 3) + col;
#pragma unroll
                for (int i = 0; i < 7; ++i) xs[i] = __shfl(drawn.x[i], src, 64);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    ws[i] = __shfl(drawn.w[i], src, 64);
                    tg[i] = __shfl(drawn.t[i], src, 64);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 7; ++i) xs[i] = next.x[i];
#pragma unroll
                for (int i = 0; i < 3; ++i) ws[i] = next.w[i], tg[i] = next.t[i];
                if (more) load_query(q, args, sample_of(chunk + nblk), B, next);
            }
            if (g == 0) {
                float *x = sX + (16 * wave + col) * kInputs;
#pragma unroll
                for (int i = 0; i < 7; ++i) x[i] = xs[i];
#pragma unroll
                for (int i = 0; i < 3; ++i) x[7 + i] = ws[i];
            }
            // ---------------- forward (layers 1..4 operation for operation as k_grad_f32)
            const float *sw = (const float *)smem;
            {
                f32x4 a1[1][MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) a1[0][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                layer1_surface<W>(a1[0], sw + L.offset(SEC_S), xs, lane, g);
                const float dx[1] = {ws[0]}, dy[1] = {ws[1]}, dz[1] = {ws[2]};
                layer1_direction<W, 1>(a1, sw + L.offset(SEC_D), dx, dy, dz, lane, g);
                relu_all<W, 1>(a1);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[0][mt] = a1[0][mt];
            }
            uint32_t mh[4];
            mh[0] = layer_max(h[0]);
#pragma unroll
            for (int l = 1; l < 4; ++l) {
                const float *sec = sw + L.offset(SEC_H0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], h[l - 1][kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[l][mt][i] = relu_f32(o[mt][i]);
                mh[l] = layer_max(h[l]);
            }
            if constexpr (!DRAW)
                if (more) load_point(pts, q, next);
            // output layer and the last layer's delta on the vector units: every lane group has its own
            // 16 neurons of the sample
            f32x4 w5[3][MT];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float z = 0.0f;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    w5[c][mt] = sW5[c * 16 + 4 * mt + g];
#pragma unroll
                    for (int i = 0; i < 4; ++i) z = fmaf(w5[c][mt][i], h[3][mt][i], z);
                }
                z += __shfl_xor(z, 16);
                z += __shfl_xor(z, 32);
                const float t = use_loss ? tg[c] : 0.0f, dr = use_loss ? 0.0f : tg[c];
                float lt;
                d5[c] = PLAIN ? out_grad(z, t, 0.0f, true, args.loss_eps, kscale, true, 0.0f, false, lt)
                              : out_grad(z, t, dr, use_loss, args.loss_eps, kscale, args.loss_kind == NIRC_LOSS_REL_L2,
                                         args.fr ? args.fr[c] : 0.0f, args.sig != 0, lt);
                if (!valid) d5[c] = 0.0f;
                if (g == 0 && valid) loss_acc += lt;
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = fmaf(w5[2][mt][i], d5[2], fmaf(w5[1][mt][i], d5[1], w5[0][mt][i] * d5[0]));
                    d[mt][i] = h[3][mt][i] > 0.0f ? v : 0.0f;
                }
#pragma unroll
            for (int l = 0; l < 4; ++l) note_max(G::mH + l, mh[l]);
            note_max(G::mD5, max(max(mag_bits(d5[0]), mag_bits(d5[1])), mag_bits(d5[2])));
            note_max(G::mD + 3, layer_max(d));
            __syncthreads();   // the maxima; every wave is through its forward pass
        } else {
            __syncthreads();
        }
        // the transposed weights where the hidden layers' were
#pragma unroll
        for (int i = 0; i < (G::kAct - G::kHT) / NT; ++i)
            smem[G::kHT + i * NT + threadIdx.x] = ((const u32x4 *)(pk + L.offset(SEC_T0)))[i * NT + threadIdx.x];
#pragma unroll
        for (int l = 0; l < 4; ++l) take_max(eH[l], G::mH + l);
        take_max(eD5, G::mD5);
        take_max(eD[3], G::mD + 3);
        if (active) {
            if (WIDE && g == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) ((float *)sD5)[128 * c + 16 * wave + col] = d5[c];
            } else if (g == 0) {
                const float f = pow2f(14 - eD5);
                uint16_t *o = sD5 + ((wave >> 1) * 24 + (col >> 2) * 3) * 8 + 4 * (wave & 1) + (col & 3);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    uint32_t hh, ll;
                    split2(d5[c], 0.0f, f, hh, ll);
                    o[c * 8] = (uint16_t)hh;
                    o[96 + c * 8] = (uint16_t)ll;
                }
            }
            put_layer(sAct, h[3], pow2f(14 - eH[3]));
        }
        __syncthreads();
        // ---------------- W5
        if (wave < 4) {
            rescale(4, eD5 + eH[3], &g5, 1);
            if constexpr (WIDE)
                add_wide<1>(&g5, four,
                            [&](int, int sq) {
                                const f32x4 v = *(const f32x4 *)((const float *)sD5 + 128 * (col < 3 ? col : 0) + 16 * sq + 4 * g);
                                return col < 3 ? v : f32x4{0.f, 0.f, 0.f, 0.f};
                            },
                            [&](int, int sq) { return ((const f32x4 *)sAct)[own_n * G::kRows + sq * 64 + lane]; });
            else
                add_split<1>(&g5, four,
                         [&](int, int k, int t) {
                             const u32x4 v = *(const u32x4 *)(sD5 + ((2 * k + t) * 12 + g * 3 + (col < 3 ? col : 0)) * 8);
                             return col < 3 ? v : u32x4{0u, 0u, 0u, 0u};
                         },
                         [&](int, int k, int t) { return sAct[own_n * G::kRows + k * 128 + t * 64 + lane]; });
        }
        __syncthreads();
        // ---------------- layers 4 .. 1: delta_{l+1} in d
#pragma unroll
        for (int l = 3; l >= 0; --l) {
            if (l < 3) take_max(eD[l], G::mD + l);
            if (active) {
                put_layer(sDel, d, pow2f(14 - eD[l]));
                if (l > 0) {
                    put_layer(sAct, h[l > 0 ? l - 1 : 0], pow2f(14 - eH[l > 0 ? l - 1 : 0]));
                } else {
                    // the input features once more, turned (the transposed weights and the activations
                    // are done with)
                    const float *x = sX + (16 * wave + col) * kInputs;
#pragma unroll
                    for (int i = 0; i < 10; i += 2) {
                        float e[8];
                        enc_pair2(x[i], 2 * g, e[0], e[1], e[2], e[3]);
                        enc_pair2(x[i + 1], 2 * g, e[4], e[5], e[6], e[7]);
                        if constexpr (WIDE) {
                            put_wide(sE + i * G::kRows, e[0], e[1], e[2], e[3]);
                            put_wide(sE + (i + 1) * G::kRows, e[4], e[5], e[6], e[7]);
                            continue;
                        }
                        u32x4 eh, el;
                        split8(e, kSplitFeat, eh, el);
                        put(sE + i * G::kRows, eh, el, sel[0]);
                        put(sE + (i + 1) * G::kRows, eh, el, sel[1]);
                    }
                }
            }
            __syncthreads();
            if (l > 0) {
                const int k = l > 0 ? l : 1;
                f32x4 o[MT];
                if (active) {
                    const float *sec = (const float *)(smem + G::kHT) + (k - 1) * L.size(SEC_T0);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kq = 0; kq < KQ; ++kq) {
                        f32x4 a[MT];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], d[kq][kk], o[mt]);
                    }
                }
                rescale(k, eD[k] + eH[k - 1], gh[k - 1], 2);
                if constexpr (WIDE)
                    add_wide<2>(gh[k - 1], four,
                                [&](int m, int sq) { return ((const f32x4 *)sDel)[(own_m + m) * G::kRows + sq * 64 + lane]; },
                                [&](int, int sq) { return ((const f32x4 *)sAct)[own_n * G::kRows + sq * 64 + lane]; });
                else
                    add_split<2>(gh[k - 1], four,
                             [&](int m, int kb, int t) { return sDel[(own_m + m) * G::kRows + kb * 128 + t * 64 + lane]; },
                             [&](int, int kb, int t) { return sAct[own_n * G::kRows + kb * 128 + t * 64 + lane]; });
                if (active) {
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[mt][i] = h[k - 1][mt][i] > 0.0f ? o[mt][i] : 0.0f;
                    note_max(G::mD + k - 1, layer_max(d));
                }
                __syncthreads();
            } else {
                rescale(0, eD[0], g1, 5);
                if constexpr (WIDE)
                    add_wide<5>(g1, four,
                                [&](int, int sq) { return ((const f32x4 *)sDel)[own_n * G::kRows + sq * 64 + lane]; },
                                [&](int j, int sq) {
                                    return ((const f32x4 *)sE)[((wave >> 2) + 2 * j) * G::kRows + sq * 64 + lane];
                                });
                else
                    add_split<5>(g1, four,
                             [&](int, int kb, int t) { return sDel[own_n * G::kRows + kb * 128 + t * 64 + lane]; },
                             [&](int j, int kb, int t) {
                                 return sE[((wave >> 2) + 2 * j) * G::kRows + kb * 128 + t * 64 + lane];
                             });
            }
        }
    }

    // ---------------- this workgroup's partial gradient (every entry exactly once)
    float *out = partials + (int64_t)blockIdx.x * n_params(W);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const int i = (wave >> 2) + 2 * j, input = i < 7 ? surf_input(i) : i - 4;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            out[(16 * own_n + 4 * g + r) * kFeat + 16 * input + col] = ldexpf(g1[j][r], eg[0] - 28);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[w_offset(W, 1 + a) + (16 * (own_m + m) + 4 * g + r) * W + 16 * own_n + col] =
                    ldexpf(gh[a][m][r], eg[1 + a] - 28);
    if (wave < 4 && g == 0) {
#pragma unroll
        for (int r = 0; r < 3; ++r) out[w_offset(W, 4) + r * W + 16 * own_n + col] = ldexpf(g5[r], eg[4] - 28);
    }
#pragma unroll
    for (int dd = 32; dd >= 1; dd >>= 1) loss_acc += __shfl_xor(loss_acc, dd, 64);
    float *sLoss = (float *)(smem + G::kLoss);
    if (lane == 0) sLoss[wave] = loss_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int w = 0; w < kSplitGradWaves; ++w) t += sLoss[w];
        loss_partials[blockIdx.x] = t;
    }
    };
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(wide_model) == 0u, 1))
        rounds(std::false_type{});
    else
        rounds(std::true_type{});
}

// ------------------------------------------------------------------------------------------
// Width 128 (FP32).  Neither the weight-gradient tiles (280 of 16 x 16) nor the staged rows of
// all layers (278 KB) fit one pass, so the batch is swept three times; each sweep recomputes the
// forward and backward of every sample, stages only the rows its tiles need and owns a disjoint
// set of tiles (wave w: column tiles 2w, 2w + 1, or inputs w, w + 4, w + 8):
//   sweep 0: W2, W3    (rows h1, h2, delta2, delta3)
//   sweep 1: W4, W5    (rows h3, h4, delta4, output delta)
//   sweep 2: W1 + loss (rows delta1; features recomputed from the staged raw inputs)
template <int W>
struct GradWideLds {
    static constexpr int kRows = 4 * W + 4;                       // largest sweep
    static constexpr int kTotal = kRows * kStride + kChunk * kInputs;
};

template <int W, int SWEEP>
__global__ __launch_bounds__(kTrainWaves * 64) void k_grad_f32_wide(Points pts, Queries q,
                                                                    const float *__restrict__ packed, TrainArgs args,
                                                                    float *__restrict__ partials,
                                                                    float *__restrict__ loss_partials) {
    static_assert(W == 128, "wide gradient kernel");
    constexpr F32Layout L{W};
    constexpr int MT = W / 16, KQ = W / 16;
    using S = GradWideLds<W>;
    __shared__ f32x4 smem4[(S::kTotal + 3) / 4];
    __shared__ float sLoss[kTrainWaves];
    float *smem = (float *)smem4;
    float *rows = smem;                          // staged rows [row][sample]
    float *sX = smem + S::kRows * kStride;       // raw inputs [sample][10] (sweep 2)
    // row bases: sweep 0: h1 0, h2 W, delta2 2W, delta3 3W; sweep 1: h3 0, h4 W, delta4 2W,
    // d5 3W (4 rows); sweep 2: delta1 0
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int64_t B = q.count;
    const bool use_loss = args.target != nullptr;
    const float kscale = use_loss ? 2.0f * args.loss_scale / (3.0f * (float)B) : args.loss_scale;

    constexpr int NACC = SWEEP == 0 ? 2 * 2 * MT : SWEEP == 1 ? 2 * MT + 2 : 3 * MT;
    f32x4 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float loss_acc = 0.0f;

    const int64_t n_chunks = (B + kChunk - 1) / kChunk;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
        {
            const float *pk = opaque(packed);
            const int s = 16 * wave + col;
            const int64_t b = chunk * kChunk + s;
            const bool valid = b < B;
            const int64_t bi = valid ? b : B - 1;
            const int64_t p = query_point(q, pts, bi);
            const float xs[7] = {pts.px[p], pts.py[p], pts.pz[p], pts.nx[p], pts.ny[p], pts.nz[p], pts.rough[p]};
            const float ws[3] = {q.wx[bi], q.wy[bi], q.wz[bi]};
            if (SWEEP == 2 && g == 0) {
                float *x = sX + s * kInputs;
                x[0] = xs[0]; x[1] = xs[1]; x[2] = xs[2];
                x[3] = ws[0]; x[4] = ws[1]; x[5] = ws[2];
                x[6] = xs[3]; x[7] = xs[4]; x[8] = xs[5]; x[9] = xs[6];
            }
            f32x4 h[4][MT];
            {
                f32x4 a1[1][MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) a1[0][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                layer1_surface<W>(a1[0], pk + L.offset(SEC_S), xs, lane, g);
                float dx[1] = {ws[0]}, dy[1] = {ws[1]}, dz[1] = {ws[2]};
                layer1_direction<W, 1>(a1, pk + L.offset(SEC_D), dx, dy, dz, lane, g);
                relu_all<W, 1>(a1);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[0][mt] = a1[0][mt];
            }
#pragma unroll
            for (int l = 1; l < 4; ++l) {
                const float *sec = pk + L.offset(SEC_H0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], h[l - 1][kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[l][mt][i] = relu_f32(o[mt][i]);
            }
            f32x4 z5 = f32x4{0.f, 0.f, 0.f, 0.f};
            {
                const float *sec = pk + L.offset(SEC_O);
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    const f32x4 a = *(const f32x4 *)(sec + (kq * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) z5 = mfma4(a[kk], h[3][kq][kk], z5);
                }
            }
            f32x4 d5 = f32x4{0.f, 0.f, 0.f, 0.f};
            if (g == 0 && valid) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float t = use_loss ? args.target[3 * b + c] : 0.0f;
                    const float dr = use_loss ? 0.0f : args.d_rgb[3 * b + c];
                    float lt;
                    d5[c] = out_grad(z5[c], t, dr, use_loss, args.loss_eps, kscale, args.loss_kind == NIRC_LOSS_REL_L2,
                                     args.fr ? args.fr[c] : 0.0f, args.sig != 0, lt);
                    loss_acc += lt;
                }
            }
            // stage the activations this sweep needs
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const int base = SWEEP == 0 ? (l < 2 ? l * W : -1) : SWEEP == 1 ? (l >= 2 ? (l - 2) * W : -1) : -1;
                if (base < 0) continue;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) rows[(base + 16 * mt + 4 * g + i) * kStride + s] = h[l][mt][i];
            }
            if (SWEEP == 1 && g == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) rows[(3 * W + c) * kStride + s] = d5[c];
            }
            // backward: delta4 = (W5^T d5) .* [h4 > 0], then through W4^T, W3^T, W2^T
            f32x4 d[MT];
            {
                const float *sec = pk + L.offset(SEC_OT);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 a = *(const f32x4 *)(sec + (mt * 64 + lane) * 4);
                    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) o = mfma4(a[kk], d5[kk], o);
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[mt][i] = h[3][mt][i] > 0.0f ? o[i] : 0.0f;
                }
            }
            if (SWEEP == 1) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) rows[(2 * W + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
            }
#pragma unroll
            for (int l = 3; l >= 1; --l) {   // delta_l = (W_{l+1}^T delta_{l+1}) .* [h_l > 0]
                const float *sec = pk + L.offset(SEC_T0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], d[kq][kk], o[mt]);
                }
                // delta_l rows: sweep 0 keeps delta2 (l = 2) at 2W and delta3 (l = 3) at 3W; sweep 2
                // keeps delta1 (l = 1) at 0
                const int base = SWEEP == 0 ? (l >= 2 ? l * W : -1) : SWEEP == 2 ? (l == 1 ? 0 : -1) : -1;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        d[mt][i] = h[l - 1][mt][i] > 0.0f ? o[mt][i] : 0.0f;
                        if (base >= 0) rows[(base + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
                    }
            }
        }
        __syncthreads();
        // phase 2: K position (step kk, lane group g) of sample group sq <-> sample 16 sq + 4 g + kk
#pragma unroll 1
        for (int sq = 0; sq < kChunk / 16; ++sq) {
            const int s0 = 16 * sq + 4 * g;
            if constexpr (SWEEP == 0) {
                // W2 = delta2 h1^T (rows 2W, 0), W3 = delta3 h2^T (rows 3W, W)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int cc = 0; cc < 2; ++cc) {
                        const int ct = 2 * wave + cc;
                        const f32x4 bv = *(const f32x4 *)(rows + (a * W + 16 * ct + col) * kStride + s0);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            const f32x4 av = *(const f32x4 *)(rows + ((2 + a) * W + 16 * mt + col) * kStride + s0);
                            f32x4 &c = acc[(a * 2 + cc) * MT + mt];
#pragma unroll
                            for (int kk = 0; kk < 4; ++kk) c = mfma4(av[kk], bv[kk], c);
                        }
                    }
            } else if constexpr (SWEEP == 1) {
                // W4 = delta4 h3^T (rows 2W, 0), W5 = d5 h4^T (rows 3W, W)
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    const int ct = 2 * wave + cc;
                    const f32x4 bv = *(const f32x4 *)(rows + (16 * ct + col) * kStride + s0);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const f32x4 av = *(const f32x4 *)(rows + (2 * W + 16 * mt + col) * kStride + s0);
                        f32x4 &c = acc[cc * MT + mt];
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) c = mfma4(av[kk], bv[kk], c);
                    }
                    const f32x4 b4 = *(const f32x4 *)(rows + (W + 16 * ct + col) * kStride + s0);
                    f32x4 a5 = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (col < 3) a5 = *(const f32x4 *)(rows + (3 * W + col) * kStride + s0);
                    f32x4 &c5 = acc[2 * MT + cc];
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) c5 = mfma4(a5[kk], b4[kk], c5);
                }
            } else {
                // W1 = delta1 e^T: column tile = input index, features recomputed from raw inputs
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int input = wave + 4 * a;
                    if (input >= kInputs) break;
                    const int k = col >> 1, sc = col & 1;
                    float bv[4];
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        float sn, cs;
                        enc_pair(sX[(s0 + kk) * kInputs + input], k, sn, cs);
                        bv[kk] = sc ? cs : sn;
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const f32x4 av = *(const f32x4 *)(rows + (16 * mt + col) * kStride + s0);
                        f32x4 &c = acc[a * MT + mt];
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) c = mfma4(av[kk], bv[kk], c);
                    }
                }
            }
        }
        __syncthreads();
    }

    float *out = partials + (int64_t)blockIdx.x * n_params(W);
    if constexpr (SWEEP == 0) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        out[w_offset(W, 1 + a) + (int64_t)(16 * mt + 4 * g + i) * W + 16 * (2 * wave + cc) + col] =
                            acc[(a * 2 + cc) * MT + mt][i];
    } else if constexpr (SWEEP == 1) {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    out[w_offset(W, 3) + (int64_t)(16 * mt + 4 * g + i) * W + 16 * (2 * wave + cc) + col] =
                        acc[cc * MT + mt][i];
            if (g == 0) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    out[w_offset(W, 4) + (int64_t)i * W + 16 * (2 * wave + cc) + col] = acc[2 * MT + cc][i];
            }
        }
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int input = wave + 4 * a;
            if (input >= kInputs) break;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    out[w_offset(W, 0) + (int64_t)(16 * mt + 4 * g + i) * kFeat + 16 * input + col] = acc[a * MT + mt][i];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) loss_acc += __shfl_xor(loss_acc, d, 64);
        if (lane == 0) sLoss[wave] = loss_acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.0f;
            for (int w = 0; w < kTrainWaves; ++w) t += sLoss[w];
            loss_partials[blockIdx.x] = t;
        }
    }
}

// grad[i] = inv_scale * sum_blk partials[blk][i] in a fixed order: a workgroup handles 64 V parameters
// (V consecutive ones per lane) with 16 waves; wave w sums the w-th sixteenth of the partials with
// eight running sums, then the sixteen wave sums are added in a fixed tree.  Raises `bad` on a
// non-finite entry.  Workgroup 0 also reduces the loss.
template <int V>
struct ReduceVec {
    typedef float T __attribute__((ext_vector_type(V)));
};
template <>
struct ReduceVec<1> {
    typedef float T;
};

template <int V>
__device__ __forceinline__ void reduce_grad_block(const float *__restrict__ partials,
                                                  const float *__restrict__ loss_partials, int nblocks, int64_t np,
                                                  float inv_scale, float loss_norm, float *__restrict__ grad,
                                                  float *__restrict__ loss, uint32_t *bad, int blk,
                                                  typename ReduceVec<V>::T (*q)[64], const float *dyn_scale,
                                                  float dyn_batch) {
    using T = typename ReduceVec<V>::T;
    if (dyn_scale) inv_scale = 1.0f / (*dyn_scale * dyn_batch);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t i = ((int64_t)blk * 64 + lane) * V;
    const int per = (nblocks + kReduceWaves - 1) / kReduceWaves;
    const int b0 = min(nblocks, wave * per), b1 = min(nblocks, b0 + per);
    static_assert(kReduceSums == 8, "the tree below adds eight running sums");
    T acc[kReduceSums] = {};
    if (i < np) {
        int b = b0;
        for (; b + kReduceSums <= b1; b += kReduceSums)
#pragma unroll
            for (int u = 0; u < kReduceSums; ++u) acc[u] += *(const T *)(partials + (int64_t)(b + u) * np + i);
        for (int u = 0; b < b1; ++b, ++u) acc[u] += *(const T *)(partials + (int64_t)b * np + i);
    }
    q[wave][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    __syncthreads();
    if (wave == 0 && i < np) {
        T t[kReduceWaves / 2];
#pragma unroll
        for (int k = 0; k < kReduceWaves / 2; ++k) t[k] = q[2 * k][lane] + q[2 * k + 1][lane];
        const T gi = (((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]))) * inv_scale;
        *(T *)(grad + i) = gi;
        bool finite = true;
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const float *e = (const float *)&gi;
            finite = finite && isfinite(e[k]);
        }
        if (bad && !finite) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
    }
    // the loss: lane-strided sums of the partials, then a fixed shuffle tree (one wave, so the
    // loads are in flight together rather than one dependent load per partial)
    if (blk == 0 && wave == 0) {
        float t = 0.0f;
        for (int b = lane; b < nblocks; b += 64) t += loss_partials[b];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) t += __shfl_xor(t, d, 64);
        if (lane == 0) {
            t *= loss_norm;
            if (loss) loss[0] = t;
            if (bad && !isfinite(t)) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
        }
    }
}

__global__ __launch_bounds__(kReduceWaves * 64) void k_reduce_grad(const float *__restrict__ partials,
                                                                   const float *__restrict__ loss_partials,
                                                                   int nblocks, int64_t np, float inv_scale,
                                                                   float loss_norm, float *__restrict__ grad,
                                                                   float *__restrict__ loss, uint32_t *bad,
                                                                   const float *dyn_scale, float dyn_batch) {
    __shared__ float q[kReduceWaves][64];
    reduce_grad_block<1>(partials, loss_partials, nblocks, np, inv_scale, loss_norm, grad, loss, bad, blockIdx.x, q,
                         dyn_scale, dyn_batch);
}

// The reduction of every request of a training work list, with the scale factors each request's own
// step uses (16-bit models: loss_scale * B).  A fixed grid walks the requests' workgroups one after
// the other, whatever the list's length (a grid row for each request that a list may hold: 20,590 of
// 22,720 workgroups of a 6-request list had nothing to do), four parameters per lane.
// 6 x 16,384 samples: 30.4 -> 15.5 us (70 MB).
constexpr int kReduceMultiVec = 4;

__global__ __launch_bounds__(kReduceWaves * 64) void k_reduce_grad_multi(const TrainDesc *__restrict__ desc) {
    constexpr int64_t np = n_params(64);
    constexpr int V = kReduceMultiVec, per = (int)((np + 64 * V - 1) / (64 * V));
    static_assert(np % V == 0, "a lane's parameters are all there or none");
    __shared__ ReduceVec<V>::T q[kReduceWaves][64];
    const int total = desc->n * per;
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const TrainReq &t = desc->req[item / per];
        const float scale = t.loss_scale * (float)t.batch;
        reduce_grad_block<V>(t.partials, t.lpart, t.nb, np, 1.0f / scale, 1.0f / (3.0f * (float)t.batch), t.grad, t.loss,
                             t.bad, item % per, q, t.dyn_scale, (float)t.batch);
        __syncthreads();
    }
}

__global__ void k_check_finite(const float *__restrict__ grad, int64_t np, uint32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < np && !isfinite(grad[i])) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
}

// Adam (Kingma & Ba) with bias correction, t = step + 1; skipped entirely when `bad` is set.
__device__ __forceinline__ void adam_elem(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                                          const float *__restrict__ grad, const int64_t *step, const uint32_t *bad,
                                          int64_t np, float lr, float b1, float b2, float eps, int64_t i) {
    if (i >= np || *bad) return;
    const float t = (float)(*step + 1);
    const float c1 = 1.0f - powf(b1, t), c2 = 1.0f - powf(b2, t);
    float mi = m[i], vi = v[i];
    w[i] = adam_update(w[i], mi, vi, grad[i], c1, c2, lr, b1, b2, eps);
    m[i] = mi;
    v[i] = vi;
}

__global__ void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ grad, const int64_t *step, const uint32_t *bad,
                       int64_t np, float lr, float b1, float b2, float eps) {
    adam_elem(w, m, v, grad, step, bad, np, lr, b1, b2, eps, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Adam on the master weights with the FP32 packed copy refreshed in the same pass: thread i
// updates parameter i (the arithmetic of adam_elem) and stores it into the packed elements that
// hold it (f32_packed_targets; the zero padding is written once, when the weights are set).  A
// skipped step (`bad` set) changes nothing.  The last workgroup to finish (counted in `done`, zero
// between steps) commits the step or records its skip: every other workgroup has read `step` and
// `bad` before it counted itself.
template <int W>
__global__ __launch_bounds__(kAdamThreads) void k_adam_pack32(float *__restrict__ w, float *__restrict__ m,
                                                     float *__restrict__ v, const float *__restrict__ grad,
                                                     int64_t *step, uint32_t *flags, uint32_t *bad, uint32_t *done,
                                                     float *__restrict__ packed, float lr, float b1, float b2,
                                                     float eps) {
    constexpr int64_t np = n_params(W);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = i < np;
    const int64_t j = on ? i : 0;
    float mi = m[j], vi = v[j];
    const float w0 = w[j], gi = grad[j], t = (float)(*step + 1);   // read beside `bad`, not after it
    if (on && *bad == 0u) {
        const float c1 = 1.0f - powf(b1, t), c2 = 1.0f - powf(b2, t);
        const float wi = adam_update(w0, mi, vi, gi, c1, c2, lr, b1, b2, eps);
        m[i] = mi;
        v[i] = vi;
        w[i] = wi;
        int e[2];
        const int n = f32_packed_targets(W, i, e);
        for (int k = 0; k < n; ++k) packed[e[k]] = wi;
    }
    // no fence beyond the workgroup's: see adam_pack16_block
    __syncthreads();
    if (threadIdx.x == 0) {
        if (atomicAdd(done, 1u) == gridDim.x - 1u) {
            commit_step(step, flags, bad, nullptr, nullptr);
            *done = 0u;
        }
    }
}

// ------------------------------------------------------------------------------------------

// Batch estimate of the residual's expectation per channel for the residual-variance loss:
// block b sums t - y over its contiguous share of the batch (each lane a strided run, then a
// fixed tree over the 256 lanes), and one wave adds the kFrBlocks block sums in a fixed tree.
// FP32 throughout; the order never depends on timing, so the result is deterministic.
__global__ __launch_bounds__(256) void k_residual_partials(const float *__restrict__ y, const float *__restrict__ t,
                                                           int64_t B, float *__restrict__ part) {
    __shared__ float sh[3][256];
    const int64_t per = (B + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = (int64_t)blockIdx.x * per, b1 = min(B, b0 + per);
    float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
    for (int64_t b = b0 + threadIdx.x; b < b1; b += 256) {
        a0 += t[3 * b] - y[3 * b];
        a1 += t[3 * b + 1] - y[3 * b + 1];
        a2 += t[3 * b + 2] - y[3 * b + 2];
    }
    sh[0][threadIdx.x] = a0;
    sh[1][threadIdx.x] = a1;
    sh[2][threadIdx.x] = a2;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int c = 0; c < 3; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) part[3 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_residual_final(const float *__restrict__ part, int64_t B,
                                                        float *__restrict__ fr) {
    static_assert(kFrBlocks == 256, "one lane per block sum");
    __shared__ float sh[3][256];
    const int i = threadIdx.x;
    for (int c = 0; c < 3; ++c) sh[c][i] = part[3 * i + c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (i < w)
            for (int c = 0; c < 3; ++c) sh[c][i] += sh[c][i + w];
        __syncthreads();
    }
    if (i < 3) fr[i] = sh[i][0] / (float)B;
}

hipError_t launch_residual_mean(const float *y, const float *t, int64_t B, float *part, float *fr, hipStream_t s) {
    if (B < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_residual_partials, dim3(kFrBlocks), dim3(256), 0, s, y, t, B, part);
    hipLaunchKernelGGL(k_residual_final, dim3(1), dim3(256), 0, s, part, B, fr);
    return hipGetLastError();
}

int grad_blocks32(int W, int64_t batch, bool loss) {
    if (W != 64 || !loss) return train_blocks(batch);
    const int64_t chunks = (batch + split_round(batch) - 1) / split_round(batch);
    return (int)(chunks < 1 ? 1 : chunks > kMaxResidentBlocks ? kMaxResidentBlocks : chunks);
}

int train_blocks(int64_t batch) {
    int64_t chunks = (batch + kChunk - 1) / kChunk;
    if (chunks > kMaxResidentBlocks) chunks = kMaxResidentBlocks;
    return (int)(chunks < 1 ? 1 : chunks);
}

hipError_t launch_grad_partials(int W, const Points &pts, const Queries &q, const float *packed,
                                TrainArgs a, float *partials, float *loss_partials, int nblocks,
                                hipStream_t s, const TrainDraw *draw) {
    if (draw && W != 64) return hipErrorInvalidValue;
    if (W == 128) {
        const dim3 grid(nblocks), block(kTrainWaves * 64);
        hipLaunchKernelGGL((k_grad_f32_wide<128, 0>), grid, block, 0, s, pts, q, packed, a, partials, loss_partials);
        hipLaunchKernelGGL((k_grad_f32_wide<128, 1>), grid, block, 0, s, pts, q, packed, a, partials, loss_partials);
        hipLaunchKernelGGL((k_grad_f32_wide<128, 2>), grid, block, 0, s, pts, q, packed, a, partials, loss_partials);
        return hipGetLastError();
    }
    if (W != 64) return hipErrorInvalidValue;
    // an upstream gradient may span any range: its products stay in FP32
    if (!a.target && !draw) {
        hipLaunchKernelGGL(k_grad_f32<64>, dim3(nblocks), dim3(kTrainWaves * 64), 0, s, pts, q, packed, a, partials,
                           loss_partials);
        return hipGetLastError();
    }
    const bool plain = a.loss_kind == NIRC_LOSS_REL_L2 && !a.fr && !a.sig;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kSplitGradWaves * 64), 0, s, pts, q, draw ? *draw : TrainDraw{},
                           packed, a, partials, loss_partials);
    };
    if (draw && plain) go(k_grad_split<true, true>);
    else if (draw) go(k_grad_split<false, true>);
    else if (plain) go(k_grad_split<true, false>);
    else go(k_grad_split<false, false>);
    return hipGetLastError();
}

hipError_t launch_reduce_grad(int W, const float *partials, const float *loss_partials, int nblocks,
                              float inv_scale, float loss_norm, float *grad, float *loss,
                              uint32_t *bad, hipStream_t s, const float *dyn_scale, float dyn_batch) {
    const int64_t np = n_params(W);
    hipLaunchKernelGGL(k_reduce_grad, dim3((unsigned)((np + 63) / 64)), dim3(kReduceWaves * 64), 0, s, partials,
                       loss_partials, nblocks, np, inv_scale, loss_norm, grad, loss, bad, dyn_scale, dyn_batch);
    return hipGetLastError();
}

hipError_t launch_check_finite(int W, const float *grad, uint32_t *bad, hipStream_t s) {
    const int64_t np = n_params(W);
    hipLaunchKernelGGL(k_check_finite, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, grad, np, bad);
    return hipGetLastError();
}

hipError_t launch_adam(int W, float *master, float *m, float *v, const float *grad, int64_t *step,
                       uint32_t *flags, uint32_t *bad, float lr, float b1, float b2, float eps,
                       float *packed, uint16_t *packed16, int prec, hipStream_t s, uint32_t *done,
                       float *dyn_scale, uint32_t *good_steps) {
    const int64_t np = n_params(W);
    if (packed16)
        return launch_adam_pack16(W, prec, master, m, v, grad, step, flags, bad, dyn_scale, good_steps, done,
                                  packed16, lr, b1, b2, eps, s);
    const dim3 grid((unsigned)((np + kAdamThreads - 1) / kAdamThreads)), block(kAdamThreads);
    if (W == 64)
        hipLaunchKernelGGL(k_adam_pack32<64>, grid, block, 0, s, master, m, v, grad, step, flags, bad, done, packed,
                           lr, b1, b2, eps);
    else if (W == 128)
        hipLaunchKernelGGL(k_adam_pack32<128>, grid, block, 0, s, master, m, v, grad, step, flags, bad, done,
                           packed, lr, b1, b2, eps);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_reduce_grad_multi(const TrainDesc *desc, int W, hipStream_t s) {
    if (W != 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reduce_grad_multi, dim3(2 * kMaxResidentBlocks), dim3(kReduceWaves * 64), 0, s, desc);
    return hipGetLastError();
}

// Explicit-length variants (the hash-grid model's parameter vector).
hipError_t launch_reduce_grad_n(int64_t np, const float *partials, const float *loss_partials, int nblocks,
                                float inv_scale, float loss_norm, float *grad, float *loss, uint32_t *bad,
                                hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_grad, dim3((unsigned)((np + 63) / 64)), dim3(kReduceWaves * 64), 0, s, partials,
                       loss_partials, nblocks, np, inv_scale, loss_norm, grad, loss, bad, (const float *)nullptr, 1.0f);
    return hipGetLastError();
}

hipError_t launch_check_finite_n(int64_t np, const float *grad, uint32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(k_check_finite, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, grad, np, bad);
    return hipGetLastError();
}

// k_adam over four consecutive elements per thread with 16-byte loads and stores (the long
// parameter vectors of the hash-grid model: one streaming pass over w, m, v and the gradient);
// the same arithmetic per element, and element by element in a ragged last group.
__global__ void k_adam4(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                        const float *__restrict__ grad, const int64_t *step, const uint32_t *bad, int64_t np,
                        float lr, float b1, float b2, float eps) {
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (i0 >= np || *bad) return;
    const float t = (float)(*step + 1);
    const float c1 = 1.0f - powf(b1, t), c2 = 1.0f - powf(b2, t);
    if (i0 + 4 <= np) {
        const f32x4 g4 = *(const f32x4 *)(grad + i0);
        f32x4 m4 = *(const f32x4 *)(m + i0), v4 = *(const f32x4 *)(v + i0), w4 = *(const f32x4 *)(w + i0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float mk = m4[k], vk = v4[k];
            w4[k] = adam_update(w4[k], mk, vk, g4[k], c1, c2, lr, b1, b2, eps);
            m4[k] = mk;
            v4[k] = vk;
        }
        *(f32x4 *)(m + i0) = m4;
        *(f32x4 *)(v + i0) = v4;
        *(f32x4 *)(w + i0) = w4;
        return;
    }
    for (int64_t i = i0; i < np; ++i) {
        float mi = m[i], vi = v[i];
        w[i] = adam_update(w[i], mi, vi, grad[i], c1, c2, lr, b1, b2, eps);
        m[i] = mi;
        v[i] = vi;
    }
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

hipError_t launch_adam_n(int64_t np, float *master, float *m, float *v, const float *grad, const int64_t *step,
                         const uint32_t *bad, float lr, float b1, float b2, float eps, hipStream_t s) {
    if (aligned16(master) && aligned16(m) && aligned16(v) && aligned16(grad)) {
        const int64_t groups = (np + 3) / 4;
        hipLaunchKernelGGL(k_adam4, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, master, m, v, grad, step,
                           bad, np, lr, b1, b2, eps);
    } else {
        hipLaunchKernelGGL(k_adam, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, master, m, v, grad, step, bad,
                           np, lr, b1, b2, eps);
    }
    return hipGetLastError();
}

// g[i] *= scale, raising `bad` on a non-finite result.
__global__ void k_scale_check(float *__restrict__ g, int64_t n, float scale, uint32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const float v = g[i] * scale;
        g[i] = v;
        if (bad && !isfinite(v)) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
    }
}

// Four elements per thread with 16-byte accesses where the buffer allows it.
__global__ void k_scale_check4(float *__restrict__ g, int64_t n, float scale, uint32_t *bad) {
    const int64_t i0 = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (i0 >= n) return;
    bool fin = true;
    if (i0 + 4 <= n) {
        f32x4 x = *(const f32x4 *)(g + i0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] *= scale;
            fin = fin && isfinite(x[k]);
        }
        *(f32x4 *)(g + i0) = x;
    } else {
        for (int64_t i = i0; i < n; ++i) {
            const float x = g[i] * scale;
            g[i] = x;
            fin = fin && isfinite(x);
        }
    }
    if (bad && !fin) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
}

__global__ void k_grid_acc_finish(const unsigned long long *__restrict__ acc, const uint32_t *__restrict__ nonfinite,
                                  float *__restrict__ g, int64_t n, float scale, uint32_t *bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = *nonfinite ? __builtin_nanf("") : __ll2float_rn((long long)acc[i]) * 0x1p-36f * scale;
    g[i] = v;
    if (bad && !isfinite(v)) atomicOr(bad, NIRC_FLAG_NONFINITE_GRAD);
}

hipError_t launch_grid_acc_finish(const GridAcc &ga, float *grad, int64_t n, float scale, uint32_t *bad,
                                  hipStream_t s) {
    static_assert(kGridFix == 36, "the finish kernel scales by 2^-36");
    hipLaunchKernelGGL(k_grid_acc_finish, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ga.acc, ga.nonfinite,
                       grad, n, scale, bad);
    return hipGetLastError();
}

hipError_t launch_scale_check(float *g, int64_t n, float scale, uint32_t *bad, hipStream_t s) {
    if (aligned16(g)) {
        const int64_t groups = (n + 3) / 4;
        hipLaunchKernelGGL(k_scale_check4, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, g, n, scale, bad);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scale_check, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, n, scale, bad);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// The hash-grid model in FP32 (width 64): k_grad_f32's two phases with the 64 grid / SH / phi
// inputs staged as rows [canonical input][sample] for the first layer's weight gradient, the grid
// values blended beforehand (bufs.vals).  Each sample's gradient with respect to its 24 grid values
// (W1_grid^T delta1, from the transposed TS32 section) goes to bufs.dvals for the grid-entry sums.
namespace {
struct HashGrad32Lds {
    static constexpr int kH = 4 * 64 * kStride;
    static constexpr int kD = 4 * 64 * kStride;
    static constexpr int kD5 = 4 * kStride;
    static constexpr int kE = kHashIn * kStride;
    static constexpr int kTotal = kH + kD + kD5 + kE;
};
}  // namespace

__global__ __launch_bounds__(kTrainWaves * 64) void k_hash_grad_f32(Queries q, const float *__restrict__ packed,
                                                                    HashGridArgs grid, TrainArgs args,
                                                                    HashTrainBufs bufs, float *__restrict__ partials,
                                                                    float *__restrict__ loss_partials,
                                                                    GridAcc gacc, bool add) {
    constexpr int W = 64, MT = 4, KQ = 4;
    using S = HashGrad32Lds;
    __shared__ f32x4 smem4[(S::kTotal + 3) / 4];
    __shared__ float sLoss[kTrainWaves];
    __shared__ HashLevel s_lv[kHashLevels];
    float *smem = (float *)smem4;
    float *sH = smem;
    float *sD = sH + S::kH;
    float *sD5 = sD + S::kD;
    float *sE = sD5 + S::kD5;
    stage_levels(s_lv, grid);
    __syncthreads();

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int64_t B = q.count, stride = hash_level_stride(B);
    const bool rel = args.loss_kind == NIRC_LOSS_REL_L2;
    // the host passes loss_scale * B: k = 2 loss_scale / 3 per sample
    const float kscale = 2.0f * args.loss_scale / (3.0f * (float)B);

    f32x4 g1[MT], gh[3][MT], g5;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        g1[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < 3; ++a) gh[a][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    g5 = f32x4{0.f, 0.f, 0.f, 0.f};
    float loss_acc = 0.0f;

    const int64_t n_chunks = (B + kChunk - 1) / kChunk;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
        // ---------------- phase 1: forward + backward of this wave's 16 samples
        {
            const float *pk = opaque(packed);
            const int s = 16 * wave + col;
            const int64_t b = chunk * kChunk + s;
            const bool valid = b < B;
            const int64_t bi = valid ? b : B - 1;
            const f32x4 xa = *(const f32x4 *)(bufs.attr + 8 * bi), xb = *(const f32x4 *)(bufs.attr + 8 * bi + 4);
            const float xs[7] = {xa[0], xa[1], xa[2], xa[3], xb[0], xb[1], xb[2]};
            float v[6], ph[4], sd[8];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float2 t = bufs.vals[(3 * g + k) * stride + bi];
                v[2 * k] = t.x;
                v[2 * k + 1] = t.y;
            }
            hash_phi4(xs[3], xs[4], xs[5], xs[6], g, ph);
            hash_dir_values_f32(q.wx[bi], q.wy[bi], q.wz[bi], g, sd);
            // canonical input rows: grid 6 g + k, SH 24 + 4 k + g, phi 49 + 4 j + g
#pragma unroll
            for (int k = 0; k < 6; ++k) sE[(6 * g + k) * kStride + s] = v[k];
#pragma unroll
            for (int k = 0; k < 7; ++k)
                if (4 * k + g < 25) sE[(24 + 4 * k + g) * kStride + s] = sd[k];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (4 * j + g < 15) sE[(49 + 4 * j + g) * kStride + s] = ph[j];

            f32x4 h[4][MT];
            {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[0][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                hash_layer1_surface_f32(h[0], pk, v, ph, lane);
                const float *gD = pk + kHash32S;
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(gD + ((mt * 2 + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) h[0][mt] = mfma4(a[mt][kk], sd[4 * kq + kk], h[0][mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[0][mt][i] = relu_f32(h[0][mt][i]);
            }
#pragma unroll
            for (int l = 1; l < 4; ++l) {
                const float *sec = pk + hash_sec32(SEC_H0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], h[l - 1][kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) h[l][mt][i] = relu_f32(o[mt][i]);
            }
            f32x4 z5 = f32x4{0.f, 0.f, 0.f, 0.f};
            {
                const float *sec = pk + hash_sec32(SEC_O);
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    const f32x4 a = *(const f32x4 *)(sec + (kq * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) z5 = mfma4(a[kk], h[3][kq][kk], z5);
                }
            }
            f32x4 d5 = f32x4{0.f, 0.f, 0.f, 0.f};
            if (g == 0 && valid) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float lt;
                    d5[c] = out_grad(z5[c], args.target[3 * b + c], 0.0f, true, args.loss_eps, kscale, rel, 0.0f,
                                     false, lt);
                    loss_acc += lt;
                }
            }
            if (g == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) sD5[c * kStride + s] = d5[c];
            }
#pragma unroll
            for (int l = 0; l < 4; ++l)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        sH[(l * W + 16 * mt + 4 * g + i) * kStride + s] = h[l][mt][i];
            f32x4 d[MT];
            {
                const float *sec = pk + hash_sec32(SEC_OT);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 a = *(const f32x4 *)(sec + (mt * 64 + lane) * 4);
                    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) o = mfma4(a[kk], d5[kk], o);
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[mt][i] = h[3][mt][i] > 0.0f ? o[i] : 0.0f;
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) sD[(3 * W + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
#pragma unroll
            for (int l = 3; l >= 1; --l) {
                const float *sec = pk + hash_sec32(SEC_T0 + (l - 1));
                f32x4 o[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    f32x4 a[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) a[mt] = *(const f32x4 *)(sec + ((mt * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o[mt] = mfma4(a[mt][kk], d[kq][kk], o[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        d[mt][i] = h[l - 1][mt][i] > 0.0f ? o[mt][i] : 0.0f;
                        sD[((l - 1) * W + 16 * mt + 4 * g + i) * kStride + s] = d[mt][i];
                    }
            }
            // d = delta1; the grid-value gradient of this sample (column col)
            // (rows 16 m + 4 g + i of W1_grid^T delta1: the two values of levels 8 m + 2 g and 8 m + 2 g + 1)
            const float *sec = pk + kHash32TS;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                f32x4 de = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq) {
                    const f32x4 a = *(const f32x4 *)(sec + ((m * KQ + kq) * 64 + lane) * 4);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) de = mfma4(a[kk], d[kq][kk], de);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int level = 8 * m + 2 * g + k;
                    if (valid && level < kHashLevels) {
                        grid_grad_check(gacc, de[2 * k], xs[0], xs[1], xs[2], s_lv[level].res);
                        grid_grad_check(gacc, de[2 * k + 1], xs[0], xs[1], xs[2], s_lv[level].res);
                        bufs.dvals[level * stride + b] = make_float2(de[2 * k], de[2 * k + 1]);
                    }
                }
            }
        }
        __syncthreads();
        // ---------------- phase 2: owned weight-gradient tiles (W1: inputs 16 wave .. 16 wave + 15)
#pragma unroll 1
        for (int sq = 0; sq < kChunk / 16; ++sq) {
            const int s0 = 16 * sq + 4 * g;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const f32x4 bv = *(const f32x4 *)(sH + (a * W + 16 * wave + col) * kStride + s0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 av = *(const f32x4 *)(sD + ((a + 1) * W + 16 * mt + col) * kStride + s0);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) gh[a][mt] = mfma4(av[kk], bv[kk], gh[a][mt]);
                }
            }
            {
                const f32x4 bv = *(const f32x4 *)(sH + (3 * W + 16 * wave + col) * kStride + s0);
                f32x4 av = f32x4{0.f, 0.f, 0.f, 0.f};
                if (col < 3) av = *(const f32x4 *)(sD5 + col * kStride + s0);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) g5 = mfma4(av[kk], bv[kk], g5);
            }
            {
                const f32x4 bv = *(const f32x4 *)(sE + (16 * wave + col) * kStride + s0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 av = *(const f32x4 *)(sD + (16 * mt + col) * kStride + s0);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) g1[mt] = mfma4(av[kk], bv[kk], g1[mt]);
                }
            }
        }
        __syncthreads();
    }

    float *out = partials + (int64_t)blockIdx.x * kHashMlp;
    auto put = [&](int64_t i, float v) { out[i] = add ? out[i] + v : v; };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) put((int64_t)(16 * mt + 4 * g + i) * kHashIn + 16 * wave + col, g1[mt][i]);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                put(W * kHashIn + a * W * W + (int64_t)(16 * mt + 4 * g + i) * W + 16 * wave + col, gh[a][mt][i]);
    if (g == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) put(W * kHashIn + 3 * W * W + (int64_t)i * W + 16 * wave + col, g5[i]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) loss_acc += __shfl_xor(loss_acc, d, 64);
    if (lane == 0) sLoss[wave] = loss_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int w = 0; w < kTrainWaves; ++w) t += sLoss[w];
        loss_partials[blockIdx.x] = add ? loss_partials[blockIdx.x] + t : t;
    }
}

hipError_t launch_hash_grad32(const Queries &q, const float *packed, const HashGridArgs &grid, TrainArgs a,
                              const HashTrainBufs &bufs, float *partials, float *loss_partials, GridAcc gacc,
                              int nblocks, bool add, hipStream_t s) {
    if (!a.target) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_hash_grad_f32, dim3(nblocks), dim3(kTrainWaves * 64), 0, s, q, packed, grid, a, bufs, partials,
                       loss_partials, gacc, add);
    return hipGetLastError();
}

}  // namespace nirc
