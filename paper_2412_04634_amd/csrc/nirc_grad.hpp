// Pieces that the gradient kernels of width 64 share: a round's samples and the change of sides of
// their operands.
#pragma once

#include "nirc_hash.hpp"

namespace nirc {

// Packs two result tiles into a chained B operand without ReLU (backward deltas).
template <int PREC>
__device__ __forceinline__ u32x4 chain_plain(const f32x4 &lo, const f32x4 &hi) {
    return u32x4{pack2<PREC>(lo[0], lo[1]), pack2<PREC>(lo[2], lo[3]), pack2<PREC>(hi[0], hi[1]),
                 pack2<PREC>(hi[2], hi[3])};
}

// One sample's inputs to a training round: its point's attributes, its direction and its
// target (or output gradient).  Loaded ahead of use in two steps, so that neither the point
// index nor the attributes that depend on it are waited for: the query's own values one round
// ahead (load_query), the point's attributes half a round ahead (load_point).
struct TrainSample {
    float x[7], w[3], t[3];
    int64_t bi;   // the query (the batch's last one for the slots past its end)
    int64_t j;    // its point index as given (bi itself when the queries carry none)
    bool valid;
};

__device__ __forceinline__ void load_query(const Queries &q, const TrainArgs &args, int64_t b, int64_t B,
                                             TrainSample &o) {
    o.valid = b < B;
    o.bi = o.valid ? b : B - 1;
    o.j = q.point ? (int64_t)q.point[o.bi] : o.bi;
    o.w[0] = q.wx[o.bi], o.w[1] = q.wy[o.bi], o.w[2] = q.wz[o.bi];
    const float *t = args.target ? args.target : args.d_rgb;
#pragma unroll
    for (int c = 0; c < 3; ++c) o.t[c] = t[3 * o.bi + c];
}

__device__ __forceinline__ void load_point(const Points &pts, const Queries &q, TrainSample &o) {
    // the checks of query_point on the index loaded before
    int64_t p = o.j;
    if (p < 0 || p >= pts.count) {
        if (q.err) atomicOr(q.err, NIRC_FLAG_BAD_POINT_INDEX);
        p = p < 0 ? 0 : pts.count - 1;
    }
    o.x[0] = pts.px[p], o.x[1] = pts.py[p], o.x[2] = pts.pz[p];
    o.x[3] = pts.nx[p], o.x[4] = pts.ny[p], o.x[5] = pts.nz[p], o.x[6] = pts.rough[p];
}

// A training frame's sample, drawn where it is used: the lanes of a wave draw 64 samples together,
// lane (g, c) that of slot c in the workgroup's g-th next round, and each round takes its own lanes'.
struct DrawnSample {
    float x[7], u1, u2, w[3], t[3];
};

__device__ __forceinline__ void draw_point(const Points &pts, const DrawKeys &keys, int64_t b, DrawnSample &o) {
    const int64_t p = train_point(pts.count, (uint32_t)b, keys, o.u1, o.u2);
    o.x[0] = pts.px[p], o.x[1] = pts.py[p], o.x[2] = pts.pz[p];
    o.x[3] = pts.nx[p], o.x[4] = pts.ny[p], o.x[5] = pts.nz[p], o.x[6] = pts.rough[p];
}

__device__ __forceinline__ void draw_target(const nirc_lobes &lobes, const DrawKeys &keys, DrawnSample &o) {
    cosine_dir(o.x[3], o.x[4], o.x[5], o.u1, o.u2, o.w[0], o.w[1], o.w[2]);
    train_target(lobes, keys.mode, o.x[0], o.x[1], o.x[2], o.w[0], o.w[1], o.w[2], o.t);
}

// Selection operands (B: lane (g, c) holds K positions 8 g + j of column c): column c takes K position
// 8 (c / 4) + c % 4 + 4 half, times `odd` where c is odd.  (0 x inf and 0 x NaN are NaN: a value that is not
// finite spoils its sample's other positions of the operand too, so that such a sample leaves more entries of the
// gradient not finite than it would by itself.  It leaves some in any case, and the step is skipped.)
template <int PREC>
__device__ __forceinline__ u32x4 select_operand(int half, float odd, int g, int col) {
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    const uint32_t one = pack2<PREC>((col & 1) ? odd : 1.0f, 0.0f) & 0xFFFFu;
    const uint32_t w = (col & 1) ? one << 16 : one;
    if (g == (col >> 2)) {
        const int d = 2 * half + ((col & 3) >> 1);
        v = u32x4{d == 0 ? w : 0u, d == 1 ? w : 0u, d == 2 ? w : 0u, d == 3 ? w : 0u};
    }
    return v;
}

}  // namespace nirc
