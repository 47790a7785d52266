// FP32 layer products on the FP16 matrix units (width 64, frequency input).
//
// Every FP32 operand x of a layer product is held as two FP16 terms, x s = h + l with h the
// nearest FP16 of x s and l the nearest FP16 of the rest, which keeps 22 to 24 significant bits;
// a product x y is h_x h_y + h_x l_y + l_x h_y (l_x l_y is below 2^-22 of it), each exact in the
// FP32 accumulator's input.  Three 16x16x32 MFMAs (3 x 16 cycles for K = 32) replace eight 16x16x4
// FP32 MFMAs (8 x 32 cycles), and a layer's sum is rounded 6 times instead of 16 and more, so
// that the result is closer to 64 bits than the FP32 chain's (predictions of 500,009 queries, rel-L2:
// 0.84e-7 and 1.03e-7 for two models, the FP32 chain 0.95e-7 and 1.30e-7).  Measured: 1080p N = 16
// estimate 8.96 -> 3.52 ms, 500,009 explicit queries 212 -> 92 us.
// The FP16 unit's range is met by exact powers of two:
//   - a layer's weights are scaled so that the largest is in [2^13, 2^14);
//   - activations of layer l are scaled by 2^ea_l so that no unit's bound b_k reaches 2^15.  b_k holds
//     whatever the inputs: the positive weights of the unit's row times the bounds of the layer before
//     (ReLU activations are never negative; of the first layer all weights' magnitudes, for sines and
//     cosines).  Nothing can overflow.
// What the range costs is bounded as well.  A second term resolves 2^-24 of a scaled value, so that a held
// activation errs by at most 2^-25 2^-ea_l beyond its own 2^-22, and a weight of less than 2^-2 as staged by
// 2^-25 as staged.  e_k carries these errors from layer to layer, times the magnitudes of the weights;
// what arrives at z is an error of the prediction, relative to it, that no input can exceed.  A model for
// which it exceeds kSplitFloor takes the FP32 MFMA chain instead: units of a layer far apart, sums that
// cancel, large units that are hardly ever on, layers that have grown in long training; also one with a
// weight that is not finite.  The bound takes all roundings the same way and every unit at its worst; where it
// is 2^-17, independent roundings come to 2^-25, less than FP32's own.  Predictions of 20,000 queries against 64
// bits (bound; rel-L2 here, on the FP32 chain): Glorot weights 2^-22.5, 1.04e-7, 1.29e-7; trained for 30,000 steps
// at a learning rate of 1e-3 2^-20.7, 2.08e-7, 2.44e-7; for 150,000 2^-18.5, 1.64e-7, 2.08e-7; for 3,000 at 1e-2
// 2^-21.9, 1.23e-7, 1.20e-7; for 150,000 2^-10.3: FP32 chain, 1.23e-7.  (Scales from products of the layers' largest
// row sums, without the bound on the error, gave 6.45e-7 for the last, and 2.8e-4 for a model with one unit 2^9
// larger than the others in each of two layers.)
// All this is found once per workgroup, from the packed FP32 weights while they are staged.
#pragma once

#include "nirc_tlmc.hpp"

namespace nirc {

// Staged fragments (A operands of 64 lanes x 8 values, H16Layout's K order; two terms each):
// S 4 row tiles x 4 K-blocks, D 4 x 2, three hidden layers 4 x 2, O 1 x 2.
constexpr int kSplitS = 0, kSplitD = 16, kSplitH = 24, kSplitO = 48, kSplitFrags = 50;
constexpr int kSplitWeights = kSplitFrags * 2 * 64;   // u32x4
constexpr int kSplitSlab = TlmcLds<64>::kSlab + 32 + 48;   // floats per wave (GroupSlab without fa, fb)

// What the workgroup finds about the model while it stages (LDS; a wave's share by row tile).
struct SplitPrep {
    u32x4 wmax[5];     // largest magnitude of a layer's weights, FP32 bits (of the output layer's: [0])
    u32x4 least[5];    // smallest nonzero one, 2 (bits - 1)
    f32x4 bmax[4];     // largest bound of a layer's activations
    float b[4][64];    // a unit's bound
    float e[4][64];    // ... and its activation's error by the format's range
    float ez;          // the outputs' error
};

struct SplitScale {
    float f[4];   // layer l + 1's accumulator times f[l] is its activations' scale
    int ez;       // output accumulator times 2^ez = z
};

constexpr float kSplitFeat = 16384.0f;   // scale of the input features (2^14)

constexpr float kSplitFloor = 0x1p-17f;

// (a f, b f) as packed FP16 pairs h (nearest) and l (nearest of the rest): four v_fma_mix.  The
// empty asm statements keep h one register, so that l reads the same rounding that the matrix
// unit gets.
__device__ __forceinline__ void split2(float a, float b, float f, uint32_t &h, uint32_t &l) {
    _Float16 h0 = (_Float16)(a * f);
    asm("" : "+v"(h0));
    const f16x2 hv = {h0, (_Float16)(b * f)};
    h = __builtin_bit_cast(uint32_t, hv);
    asm("" : "+v"(h));
    const f16x2 hw = __builtin_bit_cast(f16x2, h);
    const f16x2 lv = {(_Float16)__builtin_fmaf(a, f, -(float)hw[0]), (_Float16)__builtin_fmaf(b, f, -(float)hw[1])};
    l = __builtin_bit_cast(uint32_t, lv);
}

__device__ __forceinline__ void split8(const float *x, float f, u32x4 &h, u32x4 &l) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t hh, ll;
        split2(x[2 * i], x[2 * i + 1], f, hh, ll);
        h[i] = hh;
        l[i] = ll;
    }
}

// Sum and maximum over the four lanes of a row (16 apart), and the largest of a wave's 16 rows.
__device__ __forceinline__ float rows_sum(float x) {
    const uint32_t v = __builtin_bit_cast(uint32_t, x);
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t a0 = a[0], a1 = a[1];
    const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1));
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const uint32_t b0 = b[0], b1 = b[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}
__device__ __forceinline__ uint32_t rows_max(uint32_t m) {
    const auto a = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    m = max((uint32_t)a[0], (uint32_t)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return max((uint32_t)b[0], (uint32_t)b[1]);
}
__device__ __forceinline__ uint32_t row_max(uint32_t m) {   // (the same in the four lanes of a row)
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int v = (int)m;
        const int o = st == 0   ? __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false)     // lanes 1 apart
                      : st == 1 ? __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false)     // 2 apart
                      : st == 2 ? __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false)    // mirrored in 8
                                : __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);   // mirrored in 16
        m = max(m, (uint32_t)o);
    }
    return m;
}
__device__ __forceinline__ float row_max(float x) {   // x >= 0
    return __builtin_bit_cast(float, row_max(__builtin_bit_cast(uint32_t, x)));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t m) { return rows_max(row_max(m)); }

// The waves' largest, uniform.
__device__ __forceinline__ uint32_t largest(const u32x4 &v) {
    return __builtin_amdgcn_readfirstlane(max(max(v[0], v[1]), max(v[2], v[3])));
}
__device__ __forceinline__ float largest(const f32x4 &v) {   // (none negative)
    return __builtin_bit_cast(float, largest(__builtin_bit_cast(u32x4, v)));
}

// Stages the split weights of a packed FP32 model (F32Layout{64}) into dst and returns true, or
// returns false when the model needs the FP32 chain (dst is then to be written over).  Called by the whole
// workgroup; ends with a barrier.
// Bounds come layer by layer, so waves 0..3 (a row tile each; lane: row lane % 16, a quarter of its columns)
// go through the layers while waves 4..7 split the weights; every wave has all its reads in flight at once.
template <int WAVES>
__device__ __forceinline__ bool split_stage(const float *packed, u32x4 *dst, SplitPrep *prep, SplitScale &sc) {
    static_assert(WAVES == 8, "four waves for the bounds, four for the terms");
    constexpr F32Layout L{64};
    constexpr int oS = L.offset(SEC_S), oD = L.offset(SEC_D), oH = L.offset(SEC_H0), oO = L.offset(SEC_O);
    constexpr int szH = L.size(SEC_H0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 4, mt = wave & 3, row = 16 * mt + (lane & 15);
    const bool bounds = wave < 4;
    // quads of 16 columns: the first layer's 7 + 3 (waves 4..7), the hidden layers' 4 each, the output's
    // (waves 0 and 4)
    f32x4 u1[10], uh[3][4], uo[4];
    if (!bounds) {
#pragma unroll
        for (int q = 0; q < 10; ++q)
            u1[q] = *(const f32x4 *)(packed + (q < 7 ? oS + (mt * 7 + q) * 256 : oD + (mt * 3 + q - 7) * 256) + 4 * lane);
    }
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int q = 0; q < 4; ++q) uh[l][q] = *(const f32x4 *)(packed + oH + l * szH + (mt * 4 + q) * 256 + 4 * lane);
    if (mt == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) uo[q] = *(const f32x4 *)(packed + oO + q * 256 + 4 * lane);
    }
    float rsum[5];   // a row's sum of magnitudes
    auto look = [&](int l, const f32x4 *u, int nq) {
        uint32_t mx = 0u, mn = ~0u;
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < nq; ++q)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float x = u[q][i], y = u[q][i + 1];   // (a bit cast of a vector's element reads element 0)
                const uint32_t a = __builtin_bit_cast(uint32_t, x), b = __builtin_bit_cast(uint32_t, y);
                mx = max(max(mx, a & 0x7FFFFFFFu), b & 0x7FFFFFFFu);
                mn = min(min(mn, (a - 1u) << 1), (b - 1u) << 1);   // (zeros come out largest)
                sum += fabsf(x);
                sum += fabsf(y);
            }
        rsum[l] = rows_sum(sum);
        mx = wave_max(mx);
        mn = ~wave_max(~mn);
        if (lane == 0) {
            ((uint32_t *)&prep->wmax[l])[mt] = mx;
            ((uint32_t *)&prep->least[l])[mt] = mn;
        }
    };
    if (bounds) {
#pragma unroll
        for (int l = 1; l < 4; ++l) look(l, uh[l - 1], 4);
        if (mt == 0) look(4, uo, 4);
    } else {
        look(0, u1, 10);
        const float n = row_max(rsum[0]);
        if (g == 0) {
            prep->b[0][row] = rsum[0];
            prep->e[0][row] = rsum[0] * (0x1p-25f / kSplitFeat);
        }
        if (lane == 0) ((float *)&prep->bmax[0])[mt] = n;
    }
    __syncthreads();
    bool ok = true;
    int ew[5], ea[5];
    float bmax[5];
#pragma unroll
    for (int l = 0; l < 5; ++l) {
        const uint32_t wm = l < 4 ? largest(prep->wmax[l]) : __builtin_amdgcn_readfirstlane(prep->wmax[4][0]);
        const int e = wm ? (int)(wm >> 23) - 127 : 0;
        ok = ok && wm < 0x7F800000u && e >= -30 && e <= 30;
        ew[l] = 13 - e;
    }
    ea[0] = 14;
    bmax[0] = 1.0f;
    auto take_bmax = [&](int l) {   // activations of layer l + 1
        bmax[l + 1] = 1.001f * largest(prep->bmax[l]);
        const int eb = bmax[l + 1] > 0.0f ? (int)(__builtin_bit_cast(uint32_t, bmax[l + 1]) >> 23) - 127 : 0;
        ok = ok && eb >= -30 && eb <= 30;
        ea[l + 1] = 14 - eb;
        sc.f[l] = ldexpf(1.0f, ea[l + 1] - ea[l] - ew[l]);
    };
    auto put = [&](int frag, const f32x4 &a, const f32x4 &b, float f) {
        const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        u32x4 h, lo;
        split8(x, f, h, lo);
        dst[(2 * frag) * 64 + lane] = h;
        dst[(2 * frag + 1) * 64 + lane] = lo;
    };
    // the magnitude below which layer l's weights are held by their last bits, if it has any (else 0)
    auto small_below = [&](int l) {
        const uint32_t mn = l < 4 ? ~largest(~prep->least[l]) : __builtin_amdgcn_readfirstlane(prep->least[4][0]);
        const float t = ldexpf(0.25f, -ew[l]);
        return (mn >> 1) + 1u < __builtin_bit_cast(uint32_t, t) ? t : 0.0f;
    };
    if (const float t = small_below(0); t > 0.0f) {   // (uniform)
        if (!bounds) {
            float c = 0.0f;
#pragma unroll
            for (int q = 0; q < 10; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) c += u1[q][i] != 0.0f && fabsf(u1[q][i]) < t ? 1.0f : 0.0f;
            c = rows_sum(c);
            if (g == 0) prep->e[0][row] = fmaf(c, ldexpf(0x1p-25f, -ew[0]), rsum[0] * (0x1p-25f / kSplitFeat));
        }
        __syncthreads();
    }
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 1; l < 5; ++l) {
        take_bmax(l - 1);
        if (bounds) {
            if (l < 4 || mt == 0) {
                const float floor = ldexpf(0x1p-25f, -ea[l]);
                float p = 0.0f, e = 0.0f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 bi = *(const f32x4 *)(prep->b[l - 1] + 16 * q + 4 * g);
                    const f32x4 ei = *(const f32x4 *)(prep->e[l - 1] + 16 * q + 4 * g);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float w = l < 4 ? uh[l < 4 ? l - 1 : 0][q][i] : uo[q][i];
                        p = fmaf(fmaxf(w, 0.0f), bi[i], p);
                        e = fmaf(fabsf(w), ei[i], e);
                    }
                }
                const float t = small_below(l);
                if (t > 0.0f) {
                    float c = 0.0f;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 bi = *(const f32x4 *)(prep->b[l - 1] + 16 * q + 4 * g);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float m = fabsf(l < 4 ? uh[l < 4 ? l - 1 : 0][q][i] : uo[q][i]);
                            c += m > 0.0f && m < t ? bi[i] : 0.0f;
                        }
                    }
                    e = fmaf(c, ldexpf(0x1p-25f, -ew[l]), e);
                }
                e = fmaf(floor, rsum[l], rows_sum(e));
                if (l < 4) {
                    p = rows_sum(p);
                    if (g == 0) {
                        prep->b[l < 4 ? l : 0][row] = p;
                        prep->e[l < 4 ? l : 0][row] = e;
                    }
                    p = row_max(p);
                    if (lane == 0) ((float *)&prep->bmax[l < 4 ? l : 0])[mt] = p;
                } else {
                    e = row_max(e);
                    if (lane == 0) prep->ez = e;
                }
            }
        } else {
            const float f = ldexpf(1.0f, ew[l - 1]);
            if (l == 1) {
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) put(kSplitS + mt * 4 + kb, u1[2 * kb], kb < 3 ? u1[2 * kb + 1] : zero, f);
                put(kSplitD + mt * 2, u1[7], u1[8], f);
                put(kSplitD + mt * 2 + 1, u1[9], zero, f);
            } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    put(kSplitH + 8 * (l - 2) + mt * 2 + kb, uh[l > 1 ? l - 2 : 0][2 * kb], uh[l > 1 ? l - 2 : 0][2 * kb + 1], f);
            }
            if (l == 4 && mt == 0) {
                const float fo = ldexpf(1.0f, ew[4]);
                put(kSplitO, uo[0], uo[1], fo);
                put(kSplitO + 1, uo[2], uo[3], fo);
            }
        }
        __syncthreads();
    }
    sc.ez = -(ea[4] + ew[4]);
    return __builtin_amdgcn_readfirstlane(ok && prep->ez <= kSplitFloor);
}

// acc[tt][mt] += K-block kb of a section (first fragment `frag`, KB K-blocks) times the operand
// terms bh, bl of T tiles; the two cross terms first.
template <int T>
__device__ __forceinline__ void split_block(f32x4 (&acc)[T][4], const u32x4 *w, int frag, int KB, int kb,
                                            const u32x4 (&bh)[T], const u32x4 (&bl)[T], int lane) {
    u32x4 ah[4], al[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        ah[mt] = w[2 * (frag + mt * KB + kb) * 64 + lane];
        al[mt] = w[(2 * (frag + mt * KB + kb) + 1) * 64 + lane];
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < T; ++tt) acc[tt][mt] = mfma16<NIRC_FP16>(al[mt], bh[tt], acc[tt][mt]);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < T; ++tt) acc[tt][mt] = mfma16<NIRC_FP16>(ah[mt], bl[tt], acc[tt][mt]);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int tt = 0; tt < T; ++tt) acc[tt][mt] = mfma16<NIRC_FP16>(ah[mt], bh[tt], acc[tt][mt]);
}

// acc += W1_s e_s for T tiles of 16 columns (surface inputs xs[tt], features in B layout).
template <int T>
__device__ __forceinline__ void split_surface(f32x4 (&acc)[T][4], const u32x4 *w, const float (&xs)[T][7], int lane,
                                              int g) {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        u32x4 bh[T], bl[T];
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
            float e[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            enc_pair2(xs[tt][2 * kb], 2 * g, e[0], e[1], e[2], e[3]);
            if (kb < 3) enc_pair2(xs[tt][kb < 3 ? 2 * kb + 1 : 0], 2 * g, e[4], e[5], e[6], e[7]);
            split8(e, kSplitFeat, bh[tt], bl[tt]);
        }
        split_block<T>(acc, w, kSplitS, 4, kb, bh, bl, lane);
    }
}

// The rest of the network for T tiles: acc holds W1_s e_s; adds the direction part, runs the
// hidden layers and returns z as output16_packed leaves it (lane (g, col): queries 4g + i of tile
// col / 3, channel col % 3; other columns zero).
template <int T>
__device__ __forceinline__ f32x4 split_mlp(f32x4 (&acc)[T][4], const u32x4 *w, const SplitScale &sc, const float *dx,
                                           const float *dy, const float *dz, int lane, int g, int col) {
    {
        u32x4 bh[2][T], bl[2][T];
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
            float e[16];
            enc_pair2(dx[tt], 2 * g, e[0], e[1], e[2], e[3]);
            enc_pair2(dy[tt], 2 * g, e[4], e[5], e[6], e[7]);
            enc_pair2(dz[tt], 2 * g, e[8], e[9], e[10], e[11]);
            e[12] = e[13] = e[14] = e[15] = 0.0f;
            split8(e, kSplitFeat, bh[0][tt], bl[0][tt]);
            split8(e + 8, kSplitFeat, bh[1][tt], bl[1][tt]);
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) split_block<T>(acc, w, kSplitD, 2, kb, bh[kb], bl[kb], lane);
    }
    u32x4 bh[2][T], bl[2][T];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        // ReLU and the next layer's operand terms
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                float x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = relu_f32(acc[tt][2 * kb + (i >> 2)][i & 3]);
                split8(x, sc.f[l], bh[kb][tt], bl[kb][tt]);
            }
        if (l == 3) break;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[tt][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) split_block<T>(acc, w, kSplitH + 8 * l, 2, kb, bh[kb], bl[kb], lane);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
    }
    // output layer: Y = H W5^T; tile tt's copy of W5^T sits in columns 3 tt .. 3 tt + 2 (the staged
    // fragment has W5 in columns 0..2 and zeros elsewhere, read with the lanes shifted)
    f32x4 y0 = f32x4{0.f, 0.f, 0.f, 0.f}, y1 = y0, y2 = y0;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int tt = 0; tt < T; ++tt) {
            const int o = 2 * (kSplitO + kb) * 64 + 16 * g + ((col - 3 * tt) & 15);
            const u32x4 oh = w[o], ol = w[o + 64];
            y0 = mfma16<NIRC_FP16>(bl[kb][tt], oh, y0);
            y1 = mfma16<NIRC_FP16>(bh[kb][tt], ol, y1);
            y2 = mfma16<NIRC_FP16>(bh[kb][tt], oh, y2);
        }
    f32x4 z;
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = ldexpf((y0[i] + y1[i]) + y2[i], sc.ez);
    return z;
}

}  // namespace nirc
