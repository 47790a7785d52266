// Pieces of the fused estimator that the 16-bit chain and the split FP32 chain share: a point
// group's LDS slab, the sums over a pass's outputs and the per-point combine.
#pragma once

#include "nirc_h16.hpp"

namespace nirc {

// Per-wave scratch of the estimator's point group (LDS).
struct GroupSlab {
    float *hs;     // [16 points][W] surface projection
    float *db;     // [3][kDirSlots] staged directions
    float *psum;   // [16 points][4] cache-level sums
    float *yres;   // [16 points][4] residual-direction predictions
    float *qbuf;   // [2][3 channels][16 quads of a pass] sums of a lane's queries (general N only)
    float *nrm;    // [3][16] normals of the group's points
    u32x4 *fa;     // [4 tiles][4 lane groups][16 queries] direction features, first K-block
    uint2 *fb;     // [4 tiles][4 lane groups][16 queries] direction features, second K-block
};

// Direction features of a 4-tile pass are staged in the slab at width 64 only; wider models
// compute each tile's direction operands in the lanes that use them (and give the room to their
// hidden-layer weights).
template <int W>
struct Tlmc16Lds {
    static constexpr int kSlab = TlmcLds<W>::kSlab + 32 + 48 + (lds_weights(W) ? 4 * 64 * 4 + 4 * 64 * 2 : 0);   // floats
};

__device__ inline GroupSlab group_slab(float *base, int W) {
    GroupSlab gs;
    gs.hs = base;
    gs.db = gs.hs + 16 * W;
    gs.psum = gs.db + 3 * kDirSlots;
    gs.yres = gs.psum + 64;
    gs.qbuf = gs.yres + 64;
    gs.nrm = gs.qbuf + 96;
    gs.fa = (u32x4 *)(gs.nrm + 48);
    gs.fb = (uint2 *)(gs.fa + 4 * 64);
    return gs;
}

// The outputs of a pass of T tiles (first tile T0, staged directions from batch slot s0): z as
// output16_packed leaves it.  A lane exponentiates its four queries of one tile and channel, adds
// cache tiles to the per-point sums and leaves the residual tile's predictions in the slab.
// LIBEXP: the library's exponential for sigmoid outputs (the FP32 models).
// FEW: the sums of N = 1, 2, 4, 8 are laid out before the general ones.  That suits the 16-bit estimate of one
// request, whose passes are short (BF16, 230,399 points: N = 2 65.4 us behind them, 63.6 before; N = 12 131.8 and
// 132.2).  FP32 and the batched lists want the other order (FP32, N = 31: 798 us and 820; five streams of 83,566
// points, N = 12, with their training: 291 and 298).
template <int T, bool OCC, bool N16, bool LIBEXP, bool FEW = false>
__device__ __forceinline__ void tlmc_sums(const f32x4 &z, int T0, int s0, int n_cache, DivN dn, const GroupSlab &gs,
                                          int lane, int g, int col, const Points &pts, int64_t p0, int mode,
                                          const nirc_lobes &lobes) {
    // lane (g, col): tile tt = col / 3, channel c = col % 3, queries 4g + i of that tile
    const int tt = col / 3, c = col - 3 * (col / 3);
    const bool valid = col < 3 * T;
    const int Tt = T0 + tt;
    const int q0 = 4 * g;   // first query (row) of this lane within its tile
    float e0, e1, e2, e3;
    if (OCC && mode == NIRC_OUTPUT_VISIBILITY) {
        // uniform: predicted visibility times channel c of the known radiance, for this lane's
        // four queries (their staged directions and their points' positions)
        const int ts = min(tt, T - 1);   // lanes past the pass's tiles compute an unused value
        const int Ts = T0 + ts;
        float ev[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int qi = 16 * (s0 + ts) + q0 + i;
            const int j = (Ts < n_cache) ? (int)div_n((uint32_t)(16 * Ts + q0 + i), dn) : q0 + i;
            const int64_t pj = min(p0 + j, pts.count - 1);
            const float Lc = field_channel(lobes, c, pts.px[pj], pts.py[pj], pts.pz[pj], gs.db[qi],
                                           gs.db[kDirSlots + qi], gs.db[2 * kDirSlots + qi]);
            ev[i] = LIBEXP ? Lc * logistic(z[i]) : Lc / (1.0f + __expf(-z[i]));
        }
        e0 = ev[0];
        e1 = ev[1];
        e2 = ev[2];
        e3 = ev[3];
    } else {
        e0 = __expf(z[0]);
        e1 = __expf(z[1]);
        e2 = __expf(z[2]);
        e3 = __expf(z[3]);
    }
    if (N16 || (n_cache & 15) == 0) {
        float sum = (e0 + e1) + (e2 + e3);
        sum += __shfl_xor(sum, 16);
        sum += __shfl_xor(sum, 32);
        // one point per tile, N / 16 consecutive tiles per point.  A pass of T = 2 or 4 tiles
        // starts at a tile index divisible by T, so its tiles of one point are neighbours in the
        // pass: fold them into the lane of the run's last tile (tile tt sits 3 columns after tile
        // tt - 1), which then adds to the point's sum; every storing lane has its own point.
        bool last = true;
        if constexpr (T >= 2) {
            const int tpp = n_cache >> 4;
            if (tpp >= 2) {
                sum += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, sum), 0x113, 0xF,
                                                                           0xF, true));   // row_shr:3
                if (T == 4 && tpp >= 4)
                    sum += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, sum), 0x116,
                                                                               0xF, 0xF, true));   // row_shr:6
                last = ((tt + 1) & (min(tpp, T) - 1)) == 0;
            }
        }
        if (valid && last && g == 0 && Tt < n_cache) gs.psum[div_n((uint32_t)(16 * Tt), dn) * 4 + c] += sum;
    } else if constexpr (!N16) {
        if (FEW ? __builtin_expect(n_cache <= 8 && (n_cache & (n_cache - 1)) == 0, 1)
                : n_cache <= 8 && (16 % n_cache) == 0) {
            // every point of a cache tile lies inside the tile: plain stores of complete sums
            if (valid && Tt < n_cache) {
                const int pbase = (int)div_n((uint32_t)(16 * Tt + q0), dn);   // point of this lane's first query
                if (n_cache == 1) {
                    gs.psum[(pbase + 0) * 4 + c] = e0;
                    gs.psum[(pbase + 1) * 4 + c] = e1;
                    gs.psum[(pbase + 2) * 4 + c] = e2;
                    gs.psum[(pbase + 3) * 4 + c] = e3;
                } else if (n_cache == 2) {
                    gs.psum[(pbase + 0) * 4 + c] = e0 + e1;
                    gs.psum[(pbase + 1) * 4 + c] = e2 + e3;
                } else if (n_cache == 4) {
                    gs.psum[pbase * 4 + c] = (e0 + e1) + (e2 + e3);
                }
            }
            if (n_cache == 8) {
                float sum = (e0 + e1) + (e2 + e3);
                sum += __shfl_xor(sum, 16);
                if (valid && Tt < n_cache && (g & 1) == 0) gs.psum[((16 * Tt + q0) / 8) * 4 + c] = sum;
            }
        } else {
            // any other N (3, 5, 6, 7, 9, ...): a lane's four consecutive queries belong to at most
            // two points (4 <= N + 1), so it leaves one sum per point in the slab; then one lane per
            // (point, channel) adds the quads of its point: at most one that it enters in the middle
            // and the ones that start in it.  Bound by LDS latency: independent reads, one update
            // per point and pass (FP16, 230,399 points, N = 5: 110 us with one lane per channel adding
            // query by query onto the slab, a dependent read and write each; 86 so)
            const int nq = 4 * min(T, n_cache - T0);   // cache quads of this pass (may be <= 0)
            const int base = 16 * T0;                  // its first query
            {
                const int q = base + 16 * tt + q0;
                const int left = n_cache - (q - (int)div_n((uint32_t)(valid ? q : 0), dn) * n_cache);
                const float a = e0 + (left > 1 ? e1 : 0.0f) + (left > 2 ? e2 : 0.0f) + (left > 3 ? e3 : 0.0f);
                const float b = (left > 1 ? 0.0f : e1) + (left > 2 ? 0.0f : e2) + (left > 3 ? 0.0f : e3);
                if (valid) {
                    gs.qbuf[16 * c + 4 * tt + g] = a;
                    gs.qbuf[48 + 16 * c + 4 * tt + g] = b;
                }
            }
            wave_sync();
            const int ch = lane % 3;
            const int pt = (nq > 0 ? (int)div_n((uint32_t)base, dn) : 0) + lane / 3;
            const int lo = pt * n_cache - base, hi = lo + n_cache;   // the point's queries, from the pass's first
            if (pt < 16 && lo < 4 * nq) {
                float sum = 0.0f;
                if (lo > 0 && (lo & 3)) sum = gs.qbuf[48 + 16 * ch + (lo >> 2)];
                const int u1 = min((hi + 3) >> 2, nq);
#pragma unroll 4
                for (int u = lo > 0 ? (lo + 3) >> 2 : 0; u < u1; ++u) sum += gs.qbuf[16 * ch + u];
                gs.psum[pt * 4 + ch] += sum;
            }
            wave_sync();
        }
    }
    // residual tile: predictions at each point's residual direction (query j = point j)
    if (valid && Tt == n_cache) {
        gs.yres[(q0 + 0) * 4 + c] = e0;
        gs.yres[(q0 + 1) * 4 + c] = e1;
        gs.yres[(q0 + 2) * 4 + c] = e2;
        gs.yres[(q0 + 3) * 4 + c] = e3;
    }
}

// NaN if a point's attribute is.
__device__ __forceinline__ float attr_sum(const float x[7]) {
    return ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + x[6]);
}

// The residual sample and the store of one point group (16 points from p0; the wave's sums and
// residual predictions are in the slab, each lane holds its column's point and residual direction).
// nans (bit: point): all results of a point whose attributes are not numbers (the split FP32 chain's
// predictions are numbers then: see k_infer_split).
template <bool OCC>
__device__ __forceinline__ void tlmc_finish(const GroupSlab &gs, const float xs[7], float rdx, float rdy, float rdz,
                                            int64_t p0, int64_t P, int64_t pc, int n_cache, int mode,
                                            const float *rrad, float *out_tl, float *out_c, float *out_r,
                                            const nirc_lobes &lobes, int g, int col, uint32_t nans = 0u) {
    // residual sample: the caller's radiance (uniform branch), or the field: lane group g
    // evaluates lobe g at its column's point and residual direction, and the four lobes are
    // summed across the lane groups
    float Lr[3];
    if (rrad) {
        Lr[0] = rrad[3 * pc];
        Lr[1] = rrad[3 * pc + 1];
        Lr[2] = rrad[3 * pc + 2];
    } else {
        field_lobe(lobes, g, xs[0], xs[1], xs[2], rdx, rdy, rdz, Lr);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            Lr[c] += __shfl_xor(Lr[c], 16);
            Lr[c] += __shfl_xor(Lr[c], 32);
        }
        if (OCC && mode != NIRC_OUTPUT_RADIANCE) {   // the occluded scene's residual sample V L
            const float V = visibility(lobes, xs[0], rdx, rdy, rdz);
            Lr[0] *= V;
            Lr[1] *= V;
            Lr[2] *= V;
        }
    }
    if (g == 0 && p0 + col < P) {
        float inv_n = 1.0f / (float)n_cache;
        if ((nans >> col) & 1u) inv_n = Lr[0] = Lr[1] = Lr[2] = __builtin_nanf("");
        const float *ps = gs.psum + 4 * col, *yr = gs.yres + 4 * col;
        store_estimate(p0 + col, inv_n, ps[0], ps[1], ps[2], Lr[0] - yr[0], Lr[1] - yr[1], Lr[2] - yr[2], out_tl,
                       out_c, out_r);
    }
}

}  // namespace nirc
