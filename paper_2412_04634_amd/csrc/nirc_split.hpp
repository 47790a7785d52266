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
//   - activations of layer l are scaled by 2^ea_l with B_l 2^ea_l < 2^15, where B_l bounds every
//     activation whatever the inputs: B_0 = 1 (sines and cosines), B_l = B_{l-1} times the largest
//     row sum of the positive weights (of all weights' magnitudes in the first layer; ReLU
//     activations are never negative).  Nothing can overflow, and the second term's resolution,
//     2^-24 of a scale whose typical activation is 2^2..2^9, stays below FP32 rounding.
// The scales are found once per workgroup from the packed FP32 weights while they are staged.
// Models the scales do not suit (a weight that is not finite, layer norms beyond 2^+-30, a nonzero
// weight row more than 2^12 below its layer's largest weight) take the FP32 MFMA chain instead.
#pragma once

#include "nirc_tlmc.hpp"

namespace nirc {

// Staged fragments (A operands of 64 lanes x 8 values, H16Layout's K order; two terms each):
// S 4 row tiles x 4 K-blocks, D 4 x 2, three hidden layers 4 x 2, O 1 x 2.
constexpr int kSplitS = 0, kSplitD = 16, kSplitH = 24, kSplitO = 48, kSplitFrags = 50;
constexpr int kSplitWeights = kSplitFrags * 2 * 64;   // u32x4
constexpr int kSplitSlab = TlmcLds<64>::kSlab + 32 + 48;   // floats per wave (GroupSlab without fa, fb)

// Weight norms gathered by the workgroup (FP32 bits; magnitudes order like their bits).
struct SplitNorms {
    uint32_t wmax[5];   // largest magnitude of a layer
    uint32_t rmin[5];   // smallest nonzero row maximum of a layer
    uint32_t row[4];    // largest row sum
};

struct SplitScale {
    int ew[5];    // weights of layer l + 1 carry 2^ew[l]
    float f[4];   // layer l + 1's accumulator times f[l] is its activations' scale
    int ez;       // output accumulator times 2^ez = z
};

constexpr float kSplitFeat = 16384.0f;   // scale of the input features (2^14)

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

// Scales from the norms; false when the model has to take the FP32 chain.  Uniform.
__device__ __forceinline__ bool split_scales(const SplitNorms &n, SplitScale &sc) {
    bool ok = true;
    float B = 1.0f;
    int ea = 14;
#pragma unroll
    for (int l = 0; l < 5; ++l) {
        const uint32_t wm = __builtin_amdgcn_readfirstlane(n.wmax[l]);
        const uint32_t rm = __builtin_amdgcn_readfirstlane(n.rmin[l]);
        const int e = wm ? (int)(wm >> 23) - 127 : 0;
        ok = ok && wm < 0x7F800000u && e >= -30 && e <= 30 && (rm == ~0u || rm >= wm - (12u << 23));
        sc.ew[l] = 13 - e;
        if (l < 4) {
            B *= 1.001f * __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(n.row[l]));
            const int eb = B > 0.0f ? (int)(__builtin_bit_cast(uint32_t, B) >> 23) - 127 : 0;
            ok = ok && eb >= -30 && eb <= 30;
            sc.f[l] = ldexpf(1.0f, (14 - eb) - ea - sc.ew[l]);
            ea = 14 - eb;
        }
    }
    sc.ez = -(ea + sc.ew[4]);
    return ok;
}

// Stages the split weights of a packed FP32 model (F32Layout{64}) into dst and returns true, or
// returns false (dst unwritten) when the model needs the FP32 chain.  Called by the whole
// workgroup; barriers inside, none at the end.
template <int WAVES>
__device__ __forceinline__ bool split_stage(const float *packed, u32x4 *dst, SplitNorms *norms, SplitScale &sc) {
    constexpr F32Layout L{64};
    constexpr int oS = L.offset(SEC_S), oD = L.offset(SEC_D), oH = L.offset(SEC_H0), oO = L.offset(SEC_O);
    constexpr int szH = L.size(SEC_H0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (threadIdx.x < 5) {
        norms->wmax[threadIdx.x] = 0u;
        norms->rmin[threadIdx.x] = ~0u;
        if (threadIdx.x < 4) norms->row[threadIdx.x] = 0u;
    }
    __syncthreads();
    // a wave takes whole row tiles (lane: row lane % 16, a quarter of its columns)
    for (int c = wave; c < 17; c += WAVES) {
        const int layer = c < 4 ? 0 : c < 16 ? 1 + ((c - 4) >> 2) : 4, mt = c < 16 ? c & 3 : 0;
        uint32_t mx = 0u;
        float row = 0.0f;
        auto take = [&](int o, bool first) {
            const f32x4 a = *(const f32x4 *)(packed + o + 4 * lane);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float v = a[k];   // (a bit cast of the vector's element itself reads element 0)
                mx = max(mx, __builtin_bit_cast(uint32_t, v) & 0x7FFFFFFFu);
                row += first ? fabsf(v) : fmaxf(v, 0.0f);
            }
        };
        if (layer == 0) {
#pragma unroll
            for (int q = 0; q < 7; ++q) take(oS + (mt * 7 + q) * 256, true);
#pragma unroll
            for (int q = 0; q < 3; ++q) take(oD + (mt * 3 + q) * 256, true);
        } else {
            const int base = layer < 4 ? oH + (layer - 1) * szH : oO;
#pragma unroll
            for (int q = 0; q < 4; ++q) take(base + (mt * 4 + q) * 256, false);
        }
#pragma unroll
        for (int d = 16; d <= 32; d <<= 1) {
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, d));
            row += __shfl_xor(row, d);
        }
        uint32_t mn = mx ? mx : ~0u;
#pragma unroll
        for (int d = 1; d <= 8; d <<= 1) {
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, d));
            mn = min(mn, (uint32_t)__shfl_xor((int)mn, d));
            row = fmaxf(row, __shfl_xor(row, d));
        }
        if (lane == 0) {
            atomicMax(&norms->wmax[layer], mx);
            atomicMin(&norms->rmin[layer], mn);
            if (layer < 4) atomicMax(&norms->row[layer], __builtin_bit_cast(uint32_t, row));
        }
    }
    __syncthreads();
    if (!split_scales(*norms, sc)) return false;
    for (int i = wave; i < kSplitFrags; i += WAVES) {
        int o, layer;
        bool pair = true;   // the K-block's second quad exists (else zero padding)
        if (i < kSplitD) {
            o = oS + ((i >> 2) * 7 + 2 * (i & 3)) * 256;
            pair = (i & 3) < 3;
            layer = 0;
        } else if (i < kSplitH) {
            o = oD + (((i - kSplitD) >> 1) * 3 + 2 * (i & 1)) * 256;
            pair = (i & 1) == 0;
            layer = 0;
        } else if (i < kSplitO) {
            const int h = i - kSplitH;
            o = oH + (h >> 3) * szH + (((h >> 1) & 3) * 4 + 2 * (h & 1)) * 256;
            layer = 1 + (h >> 3);
        } else {
            o = oO + 2 * (i - kSplitO) * 256;
            layer = 4;
        }
        const f32x4 a = *(const f32x4 *)(packed + o + 4 * lane);
        const f32x4 b = pair ? *(const f32x4 *)(packed + o + 256 + 4 * lane) : f32x4{0.f, 0.f, 0.f, 0.f};
        const int ew = layer == 0 ? sc.ew[0] : layer == 1 ? sc.ew[1] : layer == 2 ? sc.ew[2] : layer == 3 ? sc.ew[3] : sc.ew[4];
        const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        u32x4 h, l;
        split8(x, ldexpf(1.0f, ew), h, l);
        dst[(2 * i) * 64 + lane] = h;
        dst[(2 * i + 1) * 64 + lane] = l;
    }
    return true;
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
