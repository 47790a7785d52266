// 16-bit training: fused forward + relative-L2 loss + backward to per-workgroup weight-gradient
// partials with BF16 / FP16 MFMA operands and FP32 accumulation.  Partials use the canonical
// layout of the FP32 kernel, so the fixed-order reduction and Adam (on the FP32 master weights)
// are shared.  The per-sample output gradient is not divided by the batch size inside the
// kernel (the host folds 1/B into the loss scale), which keeps every 16-bit delta near unit
// magnitude whatever the batch; the reduction divides the scale out again.
#include "nirc_grad.hpp"

namespace nirc {

namespace {

// Width 64: workgroups of 8 waves, rounds of two chunks (four 32-sample K-blocks).
constexpr int kWaves64 = 8;

// Width 128: workgroups of 4 waves, rounds of 64 samples (two 32-sample K-blocks).
constexpr int kWaves16 = 4;
constexpr int kChunk16 = 16 * kWaves16;
constexpr int kRow16 = kChunk16 + 8;      // LDS row stride in 16-bit elements (144 B)

template <int PREC>
__device__ __forceinline__ uint16_t to16(float x) {
    return (uint16_t)(pack2<PREC>(x, 0.0f) & 0xFFFFu);
}

// 16-bit element e of an operand (8 values in 4 dwords).
__device__ __forceinline__ uint16_t half_of(const u32x4 &v, int e) {
    return (uint16_t)((v[e >> 1] >> (16 * (e & 1))) & 0xFFFFu);
}

// Stores chained activations (B layout, lane (g, col): K position 8g + j of K-block kb is
// neuron 32 kb + 16 (j / 4) + 4 g + j % 4) as rows [neuron][sample].
template <int W>
__device__ __forceinline__ void stage_chain(uint16_t *rows, const u32x4 (&v)[W / 32], int g, int s) {
#pragma unroll
    for (int kb = 0; kb < W / 32; ++kb)
#pragma unroll
        for (int j = 0; j < 8; ++j) rows[chained_neuron16(kb, g, j) * kRow16 + s] = half_of(v[kb], j);
}

__device__ inline float out_grad16(float z, float t, float dr, bool use_loss, float eps, float k, bool rel, float fr,
                                   bool sig, float &loss_term) {
    const float y = sig ? logistic(z) : expf(z);
    const float dydz = sig ? y * (1.0f - y) : y;
    if (use_loss) {
        const float d = (y - t) + fr, den = rel ? y * y + eps : 1.0f;
        loss_term = d * d / den;
        return k * d / den * dydz;
    }
    loss_term = 0.0f;
    return k * dr * dydz;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Width 64.  A weight gradient dW = sum_s delta_s h_s^T is an MFMA whose K dimension is the sample, so
// its operands hold a neuron per lane and samples in registers, while the layer chain holds a sample
// per lane and neurons in registers.  The change of sides is an MFMA too: with the chained
// activations as the A operand, the product with a 0/1 selection matrix leaves lane (g, c) with neuron
// c of rows 4 g + i - exactly the value each 16-bit operand holds - and the rows of two waves make one
// operand: the even wave's columns are samples 8 (c / 4) + c % 4 of the 32, the odd wave's 4 further, so
// that operand position 8 g + j is sample 8 g + j.
//
// A workgroup of 8 waves takes rounds of two 64-sample chunks, 16 samples per wave, forward and back,
// layer by layer from the last: each wave turns its delta_{l+1} and h_l and puts them in LDS (8-byte stores in
// operand order), and after one barrier each wave adds its own tiles of dW_{l+1} over the round's four
// K-blocks while it goes on to delta_l (two buffers, so that a layer needs one barrier).
// The forward weights are in LDS (51 KB), the transposed ones (28 KB, one CU's L1) in global memory.
// Bound by LDS and VALU work together: per wave and round 78 MFMAs forward and back, 43 to turn the
// operands, 46 for the gradient, against ~600 VALU instructions.
// Of a 65,536-sample BF16 gradient's 26 us (two rounds per workgroup, one workgroup per CU), 5 were the
// weights' and samples' first reads, one after the other, 10.8 and 8.8 the rounds, 2 the partials; with
// the reads side by side and the samples drawn here, a step's kernel takes 29.4 us, 28.6 and 7 with
// samples from a kernel before read back here.
// (Before, four waves staged every value by a two-byte store as [neuron][sample] rows and read all
// weights from L2: 36 us.)
//
// ENC 0: the frequency input (10 input tiles of 16 features).  ENC 1: the hash-grid model's 64 inputs
// (6 tiles: two per K-block of its surface and direction operands; unused columns are not written).
template <int ENC>
struct Grad64 {
    static constexpr int kIn = ENC == 0 ? 10 : 6;           // input tiles
    static constexpr int kInKb = ENC == 0 ? 6 : 3;          // input operands (K-blocks)
    static constexpr int kOwnIn = (4 * kIn + 7) / 8;        // W1 tiles per wave
    // forward sections S, D, H0..H2, O: contiguous in both layouts
    static constexpr int kFwd = ENC == 0 ? H16Layout{64}.offset(SEC_OS) : hash_sec(SEC_OS);   // 16-bit elements
    static constexpr int kFwd4 = kFwd / 8, kE4 = kIn * 4 * 64, kBuf4 = 8 * 4 * 64;             // u32x4
    static constexpr int kTotal4 = kFwd4 + kE4 + 2 * kBuf4;
    __host__ __device__ static constexpr int sec(int s) { return ENC == 0 ? H16Layout{64}.offset(s) : hash_sec(s); }
};

// The chunks (64 samples) of partial slab `blk` of `nblk`: blk, blk + nblk, ..., added in turn.  Up to
// 256 chunks have a slab of one chunk each; beyond 128 a workgroup takes the two that the reduction
// adds first (reduce_grad_block) and stores their sum, so that every batch size has the sums of one
// chunk at a time, whatever a workgroup takes at once.
__host__ __device__ constexpr bool slab_pairs(int64_t B) {
    const int64_t chunks = (B + kChunk16 - 1) / kChunk16;
    return chunks > kReduceSlots && chunks <= 2 * kReduceSlots;
}

template <bool PAIR>
struct SlabChunks {
    int64_t first, step;
    int count;
    __device__ __forceinline__ SlabChunks(int64_t B, int64_t blk, int64_t nblk) {
        const int64_t chunks = (B + kChunk16 - 1) / kChunk16;
        if constexpr (PAIR) {
            const int64_t per = (chunks + kReduceWaves - 1) / kReduceWaves, w = blk / kReduceSums;
            first = w * per + blk % kReduceSums;
            step = kReduceSums;
            const int64_t end = min(chunks, (w + 1) * per);
            count = (first < end ? 1 : 0) + (first + step < end ? 1 : 0);
        } else {
            first = blk;
            step = nblk;
            count = blk < chunks ? (int)((chunks - blk + nblk - 1) / nblk) : 0;
        }
    }
    __device__ __forceinline__ int64_t chunk(int k) const { return first + k * step; }
};

// acc[i] += sum_k a(i, k) b(i, k) over a round's K-blocks: 0, 1 of its first chunk, 2, 3 of its second
// (all zero deltas if it has none), in turn.  PAIR: the second chunk's sum by itself, then added.
template <int PREC, int N, bool PAIR, typename A, typename B>
__device__ __forceinline__ void add_products(f32x4 *acc, const A &a, const B &b) {
    f32x4 t[N];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (PAIR && k >= 2) t[i] = mfma16<PREC>(a(i, k), b(i, k), k == 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : t[i]);
            else acc[i] = mfma16<PREC>(a(i, k), b(i, k), acc[i]);
        }
    if constexpr (PAIR) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += t[i];
    }
}

// Zeroes the 16-bit halves of d whose activation (a ReLU output, never negative) is +0.
__device__ __forceinline__ uint32_t relu_mask2(uint32_t d, uint32_t h) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 hv = __builtin_bit_cast(u16x2, h), one = {1, 1};
    const u16x2 on = hv < one ? hv : one;   // min(h, 1)
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, d) * on));
}

// Block `blk` of `nblk` over the batch (rounds blk, blk + nblk, ...): its partial gradient goes to
// `out` (canonical layout), its loss partial to *loss_out.  smem: Grad64<ENC>::kTotal4; sLoss: kWaves64
// floats.  Ends after a workgroup barrier, so a caller may run the next block on the same LDS.
// PLAIN: the caller guarantees the common case (targets given, relative L2 of eq. 12, no
// residual-variance mean, exp outputs), so the general loss arithmetic is compiled out.
// PAIR: slab_pairs of the batch.  DRAW: the samples are drawn here (keys, lobes) instead of read from
// the queries and targets.
template <int ENC, int PREC, bool PLAIN, bool DRAW, bool PAIR>
__device__ __forceinline__ void grad64_block(const Points &pts, const Queries &q, const uint16_t *packed,
                                             const TrainArgs &args, const HashLevel *s_lv, const HashTrainBufs &bufs,
                                             const GridAcc &gacc, bool add, const DrawKeys &keys,
                                             const nirc_lobes *lobes, float *out, float *loss_out, int64_t blk,
                                             int64_t nblk, u32x4 *smem, float *sLoss) {
    using G = Grad64<ENC>;
    constexpr int MT = 4, KB = 2, W = 64;
    u32x4 *sF = smem, *sE = sF + G::kFwd4, *sB = sE + G::kE4;
    const uint16_t *fw = (const uint16_t *)sF;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int col = lane & 15, g = lane >> 4;
    const int64_t B = q.count, stride = hash_level_stride(B);
    const bool use_loss = PLAIN || DRAW || ENC == 1 || args.target != nullptr;
    // the host passes loss_scale * B for 16-bit models (or the dynamic scale is taken times B):
    // k = 2 loss_scale / 3 per sample
    const float ls = args.dyn_scale ? *args.dyn_scale * (float)B : args.loss_scale;
    const float kscale = use_loss ? 2.0f * ls / (3.0f * (float)B) : ls;

    const SlabChunks<PAIR> sc(B, blk, nblk);
    const int n_rounds = (sc.count + 1) >> 1;
    // this lane's sample of round r: waves 0..3 hold the round's first chunk, 4..7 its second (B: none);
    // the turned rows of a K-block come out in the order of its samples
    auto sample_of = [&](int r) {
        const int k = 2 * r + (wave >> 2);
        const int s = 32 * ((wave >> 1) & 1) + 8 * (col >> 2) + 4 * (wave & 1) + (col & 3);
        const int64_t b = k < sc.count ? sc.chunk(k) * kChunk16 + s : B;
        return b < B ? b : B;
    };
    TrainSample next;
    DrawnSample drawn;
    {   // the forward sections, all their loads in flight together, the first samples' beside them
        constexpr int N = (G::kFwd4 + kWaves64 * 64 - 1) / (kWaves64 * 64);
        const u32x4 *src = (const u32x4 *)packed;
        u32x4 t[N];
        if (ENC == 0 && !DRAW) load_query(q, args, sample_of(0), B, next);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = i * kWaves64 * 64 + (int)threadIdx.x;
            t[i] = src[k < G::kFwd4 ? k : 0];
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ENC == 0 && DRAW) draw_point(pts, keys, min(sample_of(g), B - 1), drawn);
        if constexpr (ENC == 0 && !DRAW) load_point(pts, q, next);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = i * kWaves64 * 64 + (int)threadIdx.x;
            if (k < G::kFwd4) sF[k] = t[i];
        }
        if (ENC == 0 && DRAW) draw_target(*lobes, keys, drawn);
    }
    // this wave's tiles: W2..W4 column tile wave % 4, row tiles 2 (wave / 4) and the next; W5 column
    // tile wave (waves 0..3); W1 row tile wave % 4, input tiles wave / 4 + 2 j
    const int own_n = wave & 3, own_m = 2 * (wave >> 2);
    f32x4 gh[3][2], g1[G::kOwnIn], g5 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < 3; ++a) gh[a][0] = gh[a][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < G::kOwnIn; ++j) g1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float loss_acc = 0.0f;
    const u32x4 sel[2] = {select_operand<PREC>(0, 1.0f, g, col), select_operand<PREC>(1, 1.0f, g, col)};
    // the input features are (sin, 2 cos) pairs, the first layer's gradient takes (sin, cos)
    const u32x4 sel_in[2] = {select_operand<PREC>(0, ENC == 0 ? 0.5f : 1.0f, g, col),
                             select_operand<PREC>(1, ENC == 0 ? 0.5f : 1.0f, g, col)};
    // turned rows of this wave's samples: half an operand of K-block wave / 2
    auto put = [&](u32x4 *slot, const u32x4 &op, const u32x4 &sl) {
        const f32x4 t = mfma16<PREC>(op, sl, f32x4{0.f, 0.f, 0.f, 0.f});
        ((uint2 *)(slot + (wave >> 1) * 64 + lane))[wave & 1] = make_uint2(pack2<PREC>(t[0], t[1]), pack2<PREC>(t[2], t[3]));
    };
    int phase = 0;
    // row slots 0..3 of a buffer: delta; 4..7: activations
    auto buffer = [&]() { return sB + (phase & 1) * G::kBuf4; };

    __syncthreads();
    for (int round = 0; round < n_rounds; ++round) {
        const uint16_t *pk = opaque(packed);
        const int64_t b = sample_of(round);
        const bool valid = b < B;
        const int64_t bi = valid ? b : B - 1;
        const bool more = round + 1 < n_rounds;
        float xs[7], tg[3];
        u32x4 e[G::kInKb];   // input operands
        // FP16: the first layer's gradient takes features rounded once from FP32 (half of a rounded
        // 2 cos may be subnormal and round again, and the second sine is a product, rounded as one)
        constexpr bool kOwnRows = ENC == 0 && PREC == NIRC_FP16;
        if (kOwnRows && round > 0) __syncthreads();   // every wave is done with the previous round's input rows
        if constexpr (ENC == 0) {
            TrainSample cur;
            if constexpr (DRAW) {
                if (round > 0 && (round & 3) == 0) {
                    draw_point(pts, keys, min(sample_of(round + g), B - 1), drawn);
                    draw_target(*lobes, keys, drawn);
                }
                const int src = 16 * (round & 3) + col;
#pragma unroll
                for (int i = 0; i < 7; ++i) cur.x[i] = __shfl(drawn.x[i], src, 64);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    cur.w[i] = __shfl(drawn.w[i], src, 64);
                    cur.t[i] = __shfl(drawn.t[i], src, 64);
                }
            } else {
                cur = next;
                if (more) load_query(q, args, sample_of(round + 1), B, next);
            }
            // scheduling fences between the steps of a round keep their loads and LDS traffic apart
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < 6; ++kb) {
                float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                const int i0 = kb < 4 ? 2 * kb : 2 * (kb - 4);
                const float *v = kb < 4 ? cur.x : cur.w;
                enc_pair2_fast(v[i0], g, f[0], f[1], f[2], f[3]);
                if (i0 + 1 < (kb < 4 ? 7 : 3)) enc_pair2_fast(v[i0 + 1], g, f[4], f[5], f[6], f[7]);
                e[kb] = u32x4{pack2<PREC>(f[0], f[1]), pack2<PREC>(f[2], f[3]), pack2<PREC>(f[4], f[5]),
                              pack2<PREC>(f[6], f[7])};
                if constexpr (kOwnRows) {
                    const uint32_t s0 = to16<PREC>(f[0] * f[1]), s1 = to16<PREC>(f[4] * f[5]);
                    const u32x4 r = {pack2<PREC>(f[0], 0.5f * f[1]), s0 | (uint32_t)to16<PREC>(0.5f * f[3]) << 16,
                                     pack2<PREC>(f[4], 0.5f * f[5]), s1 | (uint32_t)to16<PREC>(0.5f * f[7]) << 16};
                    put(sE + (kb < 4 ? i0 : 7 + i0) * 256, r, sel[0]);
                    if (i0 + 1 < (kb < 4 ? 7 : 3)) put(sE + (kb < 4 ? i0 + 1 : 8 + i0) * 256, r, sel[1]);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) tg[c] = cur.t[c];
        } else {
            const f32x4 xa = *(const f32x4 *)(bufs.attr + 8 * bi), xb = *(const f32x4 *)(bufs.attr + 8 * bi + 4);
            xs[0] = xa[0], xs[1] = xa[1], xs[2] = xa[2], xs[3] = xa[3], xs[4] = xb[0], xs[5] = xb[1], xs[6] = xb[2];
            float v[6];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float2 t = bufs.vals[(3 * g + k) * stride + bi];
                v[2 * k] = t.x;
                v[2 * k + 1] = t.y;
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) tg[c] = args.target[3 * bi + c];
            hash_pack_surface<PREC>(xs, g, v, e[0], e[1]);
            e[2] = sh_operand<PREC>(q.wx[bi], q.wy[bi], q.wz[bi], g);
        }
        __builtin_amdgcn_sched_barrier(0);

        // ---------------- forward
        u32x4 hb[4][KB];   // h1..h4 after ReLU, as chained operands
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            f32x4 h[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) h[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (l == 0) {
                constexpr int SK = ENC == 0 ? 4 : 2, DK = ENC == 0 ? 2 : 1;   // K-blocks of S and D
#pragma unroll
                for (int kb = 0; kb < SK; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        h[mt] = mfma16<PREC>(*(const u32x4 *)(fw + ((mt * SK + kb) * 64 + lane) * 8), e[kb], h[mt]);
                const uint16_t *sD = fw + (ENC == 0 ? H16Layout{64}.offset(SEC_D) : kHashSecD);
#pragma unroll
                for (int kb = 0; kb < DK; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        h[mt] = mfma16<PREC>(*(const u32x4 *)(sD + ((mt * DK + kb) * 64 + lane) * 8), e[SK + kb], h[mt]);
            } else {
                const uint16_t *sec = fw + G::sec(SEC_H0 + (l - 1));
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        h[mt] = mfma16<PREC>(*(const u32x4 *)(sec + ((mt * KB + kb) * 64 + lane) * 8), hb[l - 1][kb], h[mt]);
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) hb[l][kb] = chain_operand<PREC>(h[2 * kb], h[2 * kb + 1]);
        }
        f32x4 z5 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
            z5 = mfma16<PREC>(*(const u32x4 *)(fw + G::sec(SEC_O) + (kb * 64 + lane) * 8), hb[3][kb], z5);
        if constexpr (ENC == 0 && !DRAW) {
            __builtin_amdgcn_sched_barrier(0);
            if (more) load_point(pts, q, next);
        }

        // output delta (channels 0..2 in lane group 0)
        float d5[3] = {0.f, 0.f, 0.f};
        if (g == 0 && valid) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float t = use_loss ? tg[c] : 0.0f, dr = use_loss ? 0.0f : tg[c];
                float lt;
                if constexpr (PLAIN)
                    d5[c] = out_grad16(z5[c], t, 0.0f, true, args.loss_eps, kscale, true, 0.0f, false, lt);
                else
                    d5[c] = out_grad16(z5[c], t, dr, use_loss, args.loss_eps, kscale, args.loss_kind == NIRC_LOSS_REL_L2,
                                       ENC == 0 && args.fr ? args.fr[c] : 0.0f, ENC == 0 && args.sig != 0, lt);
                loss_acc += lt;
            }
        }
        // OT holds output o at K position 8 g + j (j < 4, o = 4 g + j): only lane group 0 carries d5
        const u32x4 d5op = g == 0 ? u32x4{pack2<PREC>(d5[0], d5[1]), pack2<PREC>(d5[2], 0.0f), 0u, 0u}
                                  : u32x4{0u, 0u, 0u, 0u};

        // ---------------- backward and weight gradients, layer by layer
        {
            u32x4 *buf = buffer();
            put(buf, d5op, sel[0]);
#pragma unroll
            for (int n = 0; n < 4; ++n) put(buf + (4 + n) * 256, hb[3][n >> 1], sel[n & 1]);
            __syncthreads();
            if (wave < 4)
                add_products<PREC, 1, PAIR>(&g5, [&](int, int k) { return buf[k * 64 + lane]; },
                                      [&](int, int k) { return buf[(4 + own_n) * 256 + k * 64 + lane]; });
            ++phase;
        }
        // the inputs' turned rows (every wave is past the previous round's last use of them)
#pragma unroll
        for (int i = 0; i < (kOwnRows ? 0 : G::kIn); ++i) {
            // ENC 0: surface inputs 0..6 in K-blocks 0..3, directions 0..2 in 4, 5
            const int kb = ENC == 1 ? i >> 1 : i < 7 ? i >> 1 : 4 + ((i - 7) >> 1);
            const int half = ENC == 1 ? i & 1 : i < 7 ? i & 1 : (i - 7) & 1;
            put(sE + i * 256, e[kb], sel_in[half]);
        }
        f32x4 dl[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            dl[mt] = mfma16<PREC>(*(const u32x4 *)(pk + G::sec(SEC_OT) + (mt * 64 + lane) * 8), d5op,
                                  f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int l = 3; l >= 0; --l) {
            // delta_{l+1} = (W^T delta) .* [h_{l+1} > 0]
            u32x4 db[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const u32x4 d = chain_plain<PREC>(dl[2 * kb], dl[2 * kb + 1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) db[kb][i] = relu_mask2(d[i], hb[l][kb][i]);
            }
            u32x4 *buf = buffer();
#pragma unroll
            for (int m = 0; m < 4; ++m) put(buf + m * 256, db[m >> 1], sel[m & 1]);
            if (l > 0) {
#pragma unroll
                for (int n = 0; n < 4; ++n) put(buf + (4 + n) * 256, hb[l - 1][n >> 1], sel[n & 1]);
            }
            if (l > 0) {
                const uint16_t *sec = pk + G::sec(SEC_T0 + (l - 1));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) dl[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        dl[mt] = mfma16<PREC>(*(const u32x4 *)(sec + ((mt * KB + kb) * 64 + lane) * 8), db[kb], dl[mt]);
            } else if constexpr (ENC == 1) {
                // gradient of the grid values: rows 16 mt + 4 g + i of W1_grid^T delta1 (lane (g, col):
                // levels 8 mt + 2 g and 8 mt + 2 g + 1 of sample col)
                const uint16_t *sec = pk + kHashSecTS;
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    f32x4 de = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb)
                        de = mfma16<PREC>(*(const u32x4 *)(sec + ((mt * KB + kb) * 64 + lane) * 8), db[kb], de);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const int level = 8 * mt + 2 * g + k;
                        if (valid && level < kHashLevels) {
                            const float d0 = de[2 * k], d1 = de[2 * k + 1];
                            grid_grad_check(gacc, d0, xs[0], xs[1], xs[2], s_lv[level].res);
                            grid_grad_check(gacc, d1, xs[0], xs[1], xs[2], s_lv[level].res);
                            bufs.dvals[level * stride + b] = make_float2(d0, d1);
                        }
                    }
                }
            }
            __syncthreads();
            if (l > 0)
                add_products<PREC, 2, PAIR>(gh[l > 0 ? l - 1 : 0],
                                      [&](int m, int k) { return buf[(own_m + m) * 256 + k * 64 + lane]; },
                                      [&](int, int k) { return buf[(4 + own_n) * 256 + k * 64 + lane]; });
            else
                add_products<PREC, G::kOwnIn, PAIR>(
                    g1, [&](int, int k) { return buf[own_n * 256 + k * 64 + lane]; },
                    [&](int j, int k) { return sE[((wave >> 2) + 2 * j) * 256 + k * 64 + lane]; });
            ++phase;
        }
    }

    // ---------------- write this block's partial gradient (every entry exactly once)
    constexpr int IN = ENC == 0 ? kFeat : kHashIn;
    auto store = [&](int i, float v) { out[i] = ENC == 1 && add ? out[i] + v : v; };
#pragma unroll
    for (int j = 0; j < G::kOwnIn; ++j) {
        const int i = (wave >> 2) + 2 * j;
        if (i >= G::kIn) continue;
        int c;   // canonical input of this lane's column, or -1
        if constexpr (ENC == 0) {
            c = 16 * (i < 7 ? surf_input(i) : i - 4) + col;
        } else {
            const int kb = i >> 1, pj = 4 * (i & 1) + (col & 3);
            c = kb < 2 ? hash_surface_input(kb, col >> 2, pj) : hash_direction_input(col >> 2, pj);
        }
        if (c >= 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) store((16 * own_n + 4 * g + r) * IN + c, g1[j][r]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                store(W * IN + a * W * W + (16 * (own_m + m) + 4 * g + r) * W + 16 * own_n + col, gh[a][m][r]);
    if (wave < 4 && g == 0) {
#pragma unroll
        for (int r = 0; r < 3; ++r) store(W * IN + 3 * W * W + r * W + 16 * own_n + col, g5[r]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) loss_acc += __shfl_xor(loss_acc, d, 64);
    if (lane == 0) sLoss[wave] = loss_acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int w = 0; w < kWaves64; ++w) t += sLoss[w];
        *loss_out = ENC == 1 && add ? *loss_out + t : t;
    }
    __syncthreads();
}

template <int PREC, bool PLAIN, bool PAIR>
__global__ __launch_bounds__(kWaves64 * 64) void k_grad_h16(Points pts, Queries q, const uint16_t *__restrict__ packed,
                                                            TrainArgs args, float *__restrict__ partials,
                                                            float *__restrict__ loss_partials) {
    __shared__ u32x4 smem[Grad64<0>::kTotal4];
    __shared__ float sLoss[kWaves64];
    grad64_block<0, PREC, PLAIN, false, PAIR>(pts, q, packed, args, nullptr, HashTrainBufs{}, GridAcc{}, false, DrawKeys{},
                                        nullptr, partials + (int64_t)blockIdx.x * n_params(64),
                                        loss_partials + blockIdx.x, blockIdx.x, gridDim.x, smem, sLoss);
}

// A training frame's step: the same over the `batch` samples it draws.
template <int PREC, bool PLAIN, bool PAIR>
__global__ __launch_bounds__(kWaves64 * 64) void k_grad_h16_draw(Points pts, int64_t batch, TrainDraw draw,
                                                                 const uint16_t *__restrict__ packed, TrainArgs args,
                                                                 float *__restrict__ partials,
                                                                 float *__restrict__ loss_partials) {
    __shared__ u32x4 smem[Grad64<0>::kTotal4];
    __shared__ float sLoss[kWaves64];
    const Queries q{nullptr, nullptr, nullptr, nullptr, batch, nullptr};
    grad64_block<0, PREC, PLAIN, true, PAIR>(pts, q, packed, args, nullptr, HashTrainBufs{}, GridAcc{}, false, draw.keys,
                                       &draw.lobes, partials + (int64_t)blockIdx.x * n_params(64),
                                       loss_partials + blockIdx.x, blockIdx.x, gridDim.x, smem, sLoss);
}

// The gradient step of several models at once (continuous batching of the streams' training
// passes): request r's workgroups are the virtual blocks vb0 .. vb0 + nb - 1 of the list, and a
// fixed grid walks the virtual blocks in order.  Virtual block b of a request computes exactly
// what block b of k_grad_h16_draw computes for that request alone (same chunks, same order), so the
// partials, and everything after them, are bit-identical.
template <int PREC>
__global__ __launch_bounds__(kWaves64 * 64) void k_grad_h16_multi(const TrainDesc *__restrict__ desc, uint32_t step) {
    __shared__ u32x4 smem[Grad64<0>::kTotal4];
    __shared__ float sLoss[kWaves64];
    const int n = desc->n, total = desc->total_vb;
    for (int v = blockIdx.x; v < total; v += gridDim.x) {
        int r = 0;
        while (r + 1 < n && desc->req[r + 1].vb0 <= v) ++r;
        const TrainReq &t = desc->req[r];
        const int b = v - t.vb0;
        const Queries q{nullptr, nullptr, nullptr, nullptr, t.batch, nullptr};
        const TrainArgs a{nullptr, nullptr, t.loss_eps, t.loss_scale * (float)t.batch, t.loss_kind, nullptr,
                          t.output == NIRC_OUTPUT_VISIBILITY, t.dyn_scale};
        const DrawKeys keys{t.key0, t.key1, t.frame, step, t.output};
        float *out = t.partials + (int64_t)b * n_params(64);
        if (slab_pairs(t.batch))
            grad64_block<0, PREC, false, true, true>(t.pts, q, t.packed16, a, nullptr, HashTrainBufs{}, GridAcc{}, false,
                                                     keys, &t.lobes, out, t.lpart + b, b, t.nb, smem, sLoss);
        else
            grad64_block<0, PREC, false, true, false>(t.pts, q, t.packed16, a, nullptr, HashTrainBufs{}, GridAcc{}, false,
                                                      keys, &t.lobes, out, t.lpart + b, b, t.nb, smem, sLoss);
    }
}

// ------------------------------------------------------------------------------------------
// Width 128.  The weight gradient no longer fits in the registers of one workgroup pass (280
// tiles of 16 x 16), so the batch is swept twice, each sweep owning a disjoint set of tiles and
// recomputing the forward and backward of every sample:
//   sweep 0: W2, W3, W4 (wave w owns column tiles 2w, 2w + 1 of each, 48 tiles);
//   sweep 1: W1 (inputs w, w + 4, w + 8) and W5 (column tiles 2w, 2w + 1), and the loss.
// Each sweep stages in LDS only the rows its tiles need.  Weights are read from global memory.
template <int W>
struct Grad16WideLds {
    static constexpr int kRows0 = 6 * W;                  // sweep 0: h1..h3, delta2..delta4
    static constexpr int kRows1 = 2 * W + kFeat + 4;      // sweep 1: h4, delta1, features, d5
    static constexpr int kTotal = (kRows0 > kRows1 ? kRows0 : kRows1) * kRow16;   // 16-bit elements
};

template <int W, int PREC, int SWEEP>
__global__ __launch_bounds__(kWaves16 * 64) void k_grad_h16_wide(Points pts, Queries q,
                                                                 const uint16_t *__restrict__ packed, TrainArgs args,
                                                                 float *__restrict__ partials,
                                                                 float *__restrict__ loss_partials) {
    static_assert(W == 128, "wide gradient kernel");
    constexpr H16Layout L{W};
    constexpr int MT = W / 16, KB = W / 32;
    using S = Grad16WideLds<W>;
    __shared__ u32x4 smem4[(S::kTotal + 7) / 8];
    __shared__ float sLoss[kWaves16];
    uint16_t *smem = (uint16_t *)smem4;
    // sweep 0 rows: h1..h3 at 0..3W, delta2..delta4 at 3W..6W
    // sweep 1 rows: h4 at 0, delta1 at W, features at 2W, d5 at 2W + 160
    uint16_t *rH = smem;
    uint16_t *rD = smem + (SWEEP == 0 ? 3 : 1) * W * kRow16;
    uint16_t *rE = smem + 2 * W * kRow16;
    uint16_t *rD5 = rE + kFeat * kRow16;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int64_t B = q.count;
    const bool use_loss = args.target != nullptr;
    const float ls = args.dyn_scale ? *args.dyn_scale * (float)B : args.loss_scale;
    const float kscale = use_loss ? 2.0f * ls / (3.0f * (float)B) : ls;

    constexpr int NACC = SWEEP == 0 ? 3 * 2 * MT : 3 * MT + 2;
    f32x4 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float loss_acc = 0.0f;

    const int64_t n_chunks = (B + kChunk16 - 1) / kChunk16;
    for (int64_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
        {
            const uint16_t *pk = opaque(packed);
            const int s = 16 * wave + col;
            const int64_t b = chunk * kChunk16 + s;
            const bool valid = b < B;
            const int64_t bi = valid ? b : B - 1;
            const int64_t p = query_point(q, pts, bi);
            const float xs[7] = {pts.px[p], pts.py[p], pts.pz[p], pts.nx[p], pts.ny[p], pts.nz[p], pts.rough[p]};
            const float ws[3] = {q.wx[bi], q.wy[bi], q.wz[bi]};
            float f[44];
#pragma unroll
            for (int i = 0; i < 7; ++i) enc_pair2_fast(xs[i], g, f[4 * i], f[4 * i + 1], f[4 * i + 2], f[4 * i + 3]);
#pragma unroll
            for (int i = 0; i < 3; ++i)
                enc_pair2_fast(ws[i], g, f[28 + 4 * i], f[29 + 4 * i], f[30 + 4 * i], f[31 + 4 * i]);
            if constexpr (SWEEP == 1) {
#pragma unroll
                for (int t = 0; t < 28; ++t)
                    rE[feature_of(true, g, t) * kRow16 + s] = to16<PREC>((t & 1) ? 0.5f * f[t] : f[t]);
#pragma unroll
                for (int t = 0; t < 12; ++t)
                    rE[feature_of(false, g, t) * kRow16 + s] = to16<PREC>((t & 1) ? 0.5f * f[28 + t] : f[28 + t]);
            }

            u32x4 hb[4][KB];
            {
                f32x4 h[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
                const uint16_t *gS = pk + L.offset(SEC_S);
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    const float *fk = f + 8 * kb;
                    const u32x4 bop = kb < 3 ? u32x4{pack2<PREC>(fk[0], fk[1]), pack2<PREC>(fk[2], fk[3]),
                                                     pack2<PREC>(fk[4], fk[5]), pack2<PREC>(fk[6], fk[7])}
                                             : u32x4{pack2<PREC>(fk[0], fk[1]), pack2<PREC>(fk[2], fk[3]), 0u, 0u};
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        h[mt] = mfma16<PREC>(*(const u32x4 *)(gS + ((mt * 4 + kb) * 64 + lane) * 8), bop, h[mt]);
                }
                const float *fd = f + 28;
                const u32x4 bd0 = {pack2<PREC>(fd[0], fd[1]), pack2<PREC>(fd[2], fd[3]), pack2<PREC>(fd[4], fd[5]),
                                   pack2<PREC>(fd[6], fd[7])};
                const u32x4 bd1 = {pack2<PREC>(fd[8], fd[9]), pack2<PREC>(fd[10], fd[11]), 0u, 0u};
                const uint16_t *gD = pk + L.offset(SEC_D);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    h[mt] = mfma16<PREC>(*(const u32x4 *)(gD + ((mt * 2 + 0) * 64 + lane) * 8), bd0, h[mt]);
                    h[mt] = mfma16<PREC>(*(const u32x4 *)(gD + ((mt * 2 + 1) * 64 + lane) * 8), bd1, h[mt]);
                }
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) hb[0][kb] = chain_operand<PREC>(h[2 * kb], h[2 * kb + 1]);
            }
#pragma unroll
            for (int l = 1; l < 4; ++l) {
                const uint16_t *sec = pk + L.offset(SEC_H0 + (l - 1));
                f32x4 h[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) h[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        h[mt] = mfma16<PREC>(*(const u32x4 *)(sec + ((mt * KB + kb) * 64 + lane) * 8), hb[l - 1][kb],
                                             h[mt]);
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) hb[l][kb] = chain_operand<PREC>(h[2 * kb], h[2 * kb + 1]);
            }
            f32x4 z5 = f32x4{0.f, 0.f, 0.f, 0.f};
            {
                const uint16_t *sec = pk + L.offset(SEC_O);
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    z5 = mfma16<PREC>(*(const u32x4 *)(sec + (kb * 64 + lane) * 8), hb[3][kb], z5);
            }
            if constexpr (SWEEP == 0) {
#pragma unroll
                for (int l = 0; l < 3; ++l) stage_chain<W>(rH + l * W * kRow16, hb[l], g, s);
            } else {
                stage_chain<W>(rH, hb[3], g, s);
            }

            float d5[3] = {0.f, 0.f, 0.f};
            if (g == 0 && valid) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const float t = use_loss ? args.target[3 * b + c] : 0.0f;
                    const float dr = use_loss ? 0.0f : args.d_rgb[3 * b + c];
                    float lt;
                    d5[c] = out_grad16(z5[c], t, dr, use_loss, args.loss_eps, kscale, args.loss_kind == NIRC_LOSS_REL_L2,
                                       args.fr ? args.fr[c] : 0.0f, args.sig != 0, lt);
                    loss_acc += lt;
                }
            }
            if constexpr (SWEEP == 1) {
                if (g == 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) rD5[c * kRow16 + s] = to16<PREC>(c < 3 ? d5[c] : 0.0f);
                }
            }

            f32x4 dl[MT];
            {
                const u32x4 bop = g == 0 ? u32x4{pack2<PREC>(d5[0], d5[1]), pack2<PREC>(d5[2], 0.0f), 0u, 0u}
                                         : u32x4{0u, 0u, 0u, 0u};
                const uint16_t *sec = pk + L.offset(SEC_OT);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    dl[mt] = mfma16<PREC>(*(const u32x4 *)(sec + (mt * 64 + lane) * 8), bop, f32x4{0.f, 0.f, 0.f, 0.f});
            }
#pragma unroll
            for (int l = 3; l >= 0; --l) {
                u32x4 db[KB];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint16_t hv = half_of(hb[l][mt >> 1], 4 * (mt & 1) + i);
                        if (hv == 0) dl[mt][i] = 0.0f;
                    }
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) db[kb] = chain_plain<PREC>(dl[2 * kb], dl[2 * kb + 1]);
                // delta_{l+1}: sweep 0 keeps delta2..delta4 (l = 1..3), sweep 1 keeps delta1 (l = 0)
                if constexpr (SWEEP == 0) {
                    if (l >= 1) stage_chain<W>(rD + (l - 1) * W * kRow16, db, g, s);
                } else {
                    if (l == 0) stage_chain<W>(rD, db, g, s);
                }
                if (l == 0) break;
                const uint16_t *sec = pk + L.offset(SEC_T0 + (l - 1));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) dl[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        dl[mt] = mfma16<PREC>(*(const u32x4 *)(sec + ((mt * KB + kb) * 64 + lane) * 8), db[kb], dl[mt]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < kChunk16 / 32; ++kb) {
            const int s0 = 32 * kb + 8 * g;
            if constexpr (SWEEP == 0) {
                // W_{a+2} = delta_{a+2} h_{a+1}^T: A rows of delta (rD slot a), B rows of h (rH slot a)
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int cc = 0; cc < 2; ++cc) {
                        const int ct = 2 * wave + cc;
                        const u32x4 bv = *(const u32x4 *)(rH + (a * W + 16 * ct + col) * kRow16 + s0);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) {
                            const u32x4 av = *(const u32x4 *)(rD + (a * W + 16 * mt + col) * kRow16 + s0);
                            acc[(a * 2 + cc) * MT + mt] = mfma16<PREC>(av, bv, acc[(a * 2 + cc) * MT + mt]);
                        }
                    }
            } else {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int input = wave + 4 * a;
                    if (input >= kInputs) break;
                    const u32x4 bv = *(const u32x4 *)(rE + (16 * input + col) * kRow16 + s0);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const u32x4 av = *(const u32x4 *)(rD + (16 * mt + col) * kRow16 + s0);
                        acc[a * MT + mt] = mfma16<PREC>(av, bv, acc[a * MT + mt]);
                    }
                }
                u32x4 av5 = u32x4{0u, 0u, 0u, 0u};
                if (col < 3) av5 = *(const u32x4 *)(rD5 + col * kRow16 + s0);
#pragma unroll
                for (int cc = 0; cc < 2; ++cc) {
                    const u32x4 bv = *(const u32x4 *)(rH + (16 * (2 * wave + cc) + col) * kRow16 + s0);
                    acc[3 * MT + cc] = mfma16<PREC>(av5, bv, acc[3 * MT + cc]);
                }
            }
        }
        __syncthreads();
    }

    float *out = partials + (int64_t)blockIdx.x * n_params(W);
    if constexpr (SWEEP == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        out[w_offset(W, 1 + a) + (int64_t)(16 * mt + 4 * g + i) * W + 16 * (2 * wave + cc) + col] =
                            acc[(a * 2 + cc) * MT + mt][i];
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
        if (g == 0) {
#pragma unroll
            for (int cc = 0; cc < 2; ++cc)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    out[w_offset(W, 4) + (int64_t)i * W + 16 * (2 * wave + cc) + col] = acc[3 * MT + cc][i];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) loss_acc += __shfl_xor(loss_acc, d, 64);
        if (lane == 0) sLoss[wave] = loss_acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            float t = 0.0f;
            for (int w = 0; w < kWaves16; ++w) t += sLoss[w];
            loss_partials[blockIdx.x] = t;
        }
    }
}

int train_blocks16(int64_t batch) {
    int64_t chunks = (batch + kChunk16 - 1) / kChunk16;
    if (chunks > kMaxResidentBlocks) chunks = kMaxResidentBlocks;
    return (int)(chunks < 1 ? 1 : chunks);
}

int grad_blocks16(int W, int64_t batch) {
    return W == 64 && slab_pairs(batch) ? kReduceSlots : train_blocks16(batch);
}

hipError_t launch_grad_partials16(int W, int prec, const Points &pts, const Queries &q, const void *packed,
                                  TrainArgs a, float *partials, float *loss_partials, int nblocks, hipStream_t s,
                                  const TrainDraw *draw) {
    const uint16_t *pk = (const uint16_t *)packed;
    if (draw && W != 64) return hipErrorInvalidValue;
    if (W == 128) {
        const dim3 grid(nblocks), block(kWaves16 * 64);
        if (prec == NIRC_BF16) {
            hipLaunchKernelGGL((k_grad_h16_wide<128, NIRC_BF16, 0>), grid, block, 0, s, pts, q, pk, a, partials,
                               loss_partials);
            hipLaunchKernelGGL((k_grad_h16_wide<128, NIRC_BF16, 1>), grid, block, 0, s, pts, q, pk, a, partials,
                               loss_partials);
        } else {
            hipLaunchKernelGGL((k_grad_h16_wide<128, NIRC_FP16, 0>), grid, block, 0, s, pts, q, pk, a, partials,
                               loss_partials);
            hipLaunchKernelGGL((k_grad_h16_wide<128, NIRC_FP16, 1>), grid, block, 0, s, pts, q, pk, a, partials,
                               loss_partials);
        }
        return hipGetLastError();
    }
    if (W != 64) return hipErrorInvalidValue;
    const bool plain = (draw || a.target) && a.loss_kind == NIRC_LOSS_REL_L2 && !a.fr && !a.sig;
    auto go = [&](auto P, auto plainc, auto pairc) {
        constexpr int PR = decltype(P)::value;
        constexpr bool PL = decltype(plainc)::value, PA = decltype(pairc)::value;
        const dim3 grid(nblocks), block(kWaves64 * 64);
        if (draw)
            hipLaunchKernelGGL((k_grad_h16_draw<PR, PL, PA>), grid, block, 0, s, pts, q.count, *draw, pk, a, partials,
                               loss_partials);
        else
            hipLaunchKernelGGL((k_grad_h16<PR, PL, PA>), grid, block, 0, s, pts, q, pk, a, partials, loss_partials);
    };
    const bool pair = slab_pairs(q.count);
    auto with_prec = [&](auto P) {
        if (plain && pair) go(P, std::true_type{}, std::true_type{});
        else if (plain) go(P, std::true_type{}, std::false_type{});
        else if (pair) go(P, std::false_type{}, std::true_type{});
        else go(P, std::false_type{}, std::false_type{});
    };
    if (prec == NIRC_BF16) with_prec(std::integral_constant<int, NIRC_BF16>{});
    else with_prec(std::integral_constant<int, NIRC_FP16>{});
    return hipGetLastError();
}

hipError_t launch_train_step_multi(const TrainDesc *desc, int prec, uint32_t step, hipStream_t s) {
    if (prec == NIRC_BF16)
        hipLaunchKernelGGL((k_grad_h16_multi<NIRC_BF16>), dim3(kMaxResidentBlocks), dim3(kWaves64 * 64), 0, s, desc, step);
    else
        hipLaunchKernelGGL((k_grad_h16_multi<NIRC_FP16>), dim3(kMaxResidentBlocks), dim3(kWaves64 * 64), 0, s, desc, step);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_reduce_grad_multi(desc, 64, s);
    if (e == hipSuccess) e = launch_adam_pack16_multi(desc, 64, prec, s);
    return e;
}

// ------------------------------------------------------------------------------------------
// The hash-grid model: grad64_block with the 64 grid / SH / phi inputs, the grid values blended
// beforehand (bufs.vals).  Each sample's gradient with respect to its 24 grid values (W1_grid^T
// delta1, from the TS section) goes to bufs.dvals for the grid-entry sums.
template <int PREC, bool PAIR>
__global__ __launch_bounds__(kWaves64 * 64) void k_hash_grad_h16(Queries q, const uint16_t *__restrict__ packed,
                                                                 HashGridArgs grid, TrainArgs args, HashTrainBufs bufs,
                                                                 float *__restrict__ partials,
                                                                 float *__restrict__ loss_partials, GridAcc gacc,
                                                                 bool add) {
    __shared__ u32x4 smem[Grad64<1>::kTotal4];
    __shared__ float sLoss[kWaves64];
    __shared__ HashLevel s_lv[kHashLevels];
    stage_levels(s_lv, grid);
    __syncthreads();
    grad64_block<1, PREC, false, false, PAIR>(Points{}, q, packed, args, s_lv, bufs, gacc, add, DrawKeys{}, nullptr,
                                        partials + (int64_t)blockIdx.x * kHashMlp, loss_partials + blockIdx.x,
                                        blockIdx.x, gridDim.x, smem, sLoss);
}

hipError_t launch_hash_grad(int prec, const Queries &q, const uint16_t *packed, const HashGridArgs &grid, TrainArgs a,
                            const HashTrainBufs &bufs, float *partials, float *loss_partials, GridAcc gacc,
                            int nblocks, bool add, hipStream_t s) {
    if (!a.target) return hipErrorInvalidValue;
    if (prec != NIRC_BF16 && prec != NIRC_FP16) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(kWaves64 * 64), 0, s, q, packed, grid, a, bufs, partials,
                           loss_partials, gacc, add);
    };
    const bool pair = slab_pairs(q.count);
    if (prec == NIRC_BF16 && pair) go(k_hash_grad_h16<NIRC_BF16, true>);
    else if (prec == NIRC_BF16) go(k_hash_grad_h16<NIRC_BF16, false>);
    else if (pair) go(k_hash_grad_h16<NIRC_FP16, true>);
    else go(k_hash_grad_h16<NIRC_FP16, false>);
    return hipGetLastError();
}

}  // namespace nirc
