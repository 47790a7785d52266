// The hash grid's part of a training step, around the gradient kernels (which see a sample's grid
// values as 24 plain inputs and return the loss gradient of each):
//   k_hash_points, k_hash_gather
//                    gather every sample's point and corner features and blend them, once, with
//                    the chip's full occupancy (inside the gradient kernels, at one wave per SIMD,
//                    the dependent random reads were exposed), and note which slice of its level
//                    each cell touches;
//   k_hash_scatter   sums the gradient of a slice of one level in LDS (64-bit fixed point, integer
//                    adds: the same sums in any order) and applies Adam to the slice, or writes its
//                    gradient: no accumulator in memory to clear, add to and read back;
//   k_hash_merge     the same for the small levels, whose slices several workgroups share.
// BF16, 65,536 samples, the default grid: 1.42 -> 0.57 ms per 4-step frame; per step the gather takes
// 11 + 24 us (the samples drawn on the way; 7 + 8 + 24 with a kernel of their own), the gradient kernel
// 24 (280 with gather and atomics inside), the sums with Adam 61 + 10 (clearing the accumulators,
// converting them and a separate Adam pass alone took 47).
// Sums by global 64-bit atomics (k_hash_scatter_atomic) serve the grids the slices do not suit: the
// memory side performs them at 16 G cache-line operations/s whatever the occupancy or the placement
// (65,536 samples x 12 levels: 192 us measured alone; 12.6 M adds).
#include "nirc_hash.hpp"

namespace nirc {

namespace {

constexpr int kScatThreads = 1024;
constexpr int kScatPer = kSliceEntries / kScatThreads;   // entries per thread

// Weight of corner (bx, by, bz), in hash_entry's order of products.
__device__ __forceinline__ float corner_weight(const HashCell &h, int bx, int by, int bz) {
    return (bx ? h.f[0] : 1.0f - h.f[0]) * (by ? h.f[1] : 1.0f - h.f[1]) * (bz ? h.f[2] : 1.0f - h.f[2]);
}

}  // namespace

bool hash_scatter_plan(const HashGridArgs &grid, int64_t B, HashScatterPlan *p) {
    int task = 0;
    p->merged_elems = 0;
    for (int l = kHashLevels - 1; l >= 0; --l) {   // the large levels' tasks come first
        const HashLevel &lv = grid.lv[l];
        HashScatterLevel &s = p->lv[l];
        const int64_t n1 = (int64_t)lv.res + 1;
        if (lv.dense) {
            // whole x rows per slice, so that a corner pair (c0, c0 + 1) stays in one slice
            if (n1 > kSliceEntries) return false;
            s.rows = (int32_t)(kSliceEntries / n1);
            s.magic = (uint32_t)((0x100000000ull + (uint64_t)s.rows - 1) / (uint64_t)s.rows);
            const int64_t rows = n1 * n1;
            if (rows > (1 << 17)) return false;   // the magic division's range
            s.slices = (int32_t)((rows + s.rows - 1) / s.rows);
        } else {
            // c0 + 1 <= res < kSliceEntries changes only the index's bits below a slice's size
            if (lv.res >= kSliceEntries) return false;
            const int64_t T = (int64_t)grid.tmask + 1;
            s.rows = 0;
            s.magic = 0;
            s.slices = (int32_t)((T + kSliceEntries - 1) / kSliceEntries);
        }
        if (s.slices > 256) return false;   // slice codes are bytes
        // a slice with more corner pairs than one CU's share of all of them (4 B per level; not below
        // 8192) is split over the samples, so that no workgroup is left walking at the end: with the
        // default grid's coarse levels in one piece each, 330 tasks took 80 us, 256 of them 47
        const int64_t pairs = 4 * B / s.slices;
        const int64_t share = 4 * B * kHashLevels / 256 > 8192 ? 4 * B * kHashLevels / 256 : 8192;
        int64_t reps = (pairs + share - 1) / share;
        if (reps < 1) reps = 1;
        if (reps > 32) reps = 32;
        s.reps = (int32_t)reps;
        s.per = (int32_t)(((B + reps - 1) / reps + 63) / 64 * 64);
        s.task0 = task;
        task += s.slices * s.reps;
        if (s.reps > 1) {
            s.merge0 = (int32_t)p->merged_elems;
            p->merged_elems += 2 * (lv.dense ? n1 * n1 * n1 : (int64_t)grid.tmask + 1);
        } else {
            s.merge0 = -1;
        }
    }
    p->tasks = task;
    p->first = 0;
    for (int l = kHashLevels - 1; l >= 0; --l)
        if (p->lv[l].reps > 1) {
            p->first = p->lv[l].task0;
            break;
        }
    return true;
}

// The samples' point attributes attr[B][8] (position, normal, roughness, 0), gathered once by point
// index; clears the merged levels' accumulators and the non-finite flag.  DRAW: a training frame's
// samples are drawn here, their directions and targets written for the gradient kernel.
template <bool DRAW>
__global__ __launch_bounds__(256) void k_hash_points(Points pts, Queries q, TrainDraw draw, HashDrawn drawn,
                                                     int64_t merged_elems, HashTrainBufs bufs, GridAcc gacc,
                                                     bool first) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nt = (int64_t)gridDim.x * blockDim.x;
    if (first && tid == 0) *gacc.nonfinite = 0u;
    for (int64_t i = tid; i < merged_elems; i += nt) gacc.acc[i] = 0ull;
    if (tid >= q.count) return;
    float u1 = 0.0f, u2 = 0.0f;
    const int64_t p = DRAW ? train_point(pts.count, (uint32_t)tid, draw.keys, u1, u2) : query_point(q, pts, tid);
    const float x0 = pts.px[p], x1 = pts.py[p], x2 = pts.pz[p], n0 = pts.nx[p], n1 = pts.ny[p], n2 = pts.nz[p];
    f32x4 *a = (f32x4 *)(bufs.attr + 8 * tid);
    a[0] = f32x4{x0, x1, x2, n0};
    a[1] = f32x4{n1, n2, pts.rough[p], 0.0f};
    if constexpr (DRAW) {
        float x, y, z, L[3];
        cosine_dir(n0, n1, n2, u1, u2, x, y, z);
        train_target(draw.lobes, draw.keys.mode, x0, x1, x2, x, y, z, L);
        drawn.wx[tid] = x;
        drawn.wy[tid] = y;
        drawn.wz[tid] = z;
#pragma unroll
        for (int c = 0; c < 3; ++c) drawn.target[3 * tid + c] = L[c];
    }
}

// Blended grid values vals[level][stride] and, per level, the slices of a cell's four (y, z) corner
// rows, one byte each, codes[level][stride].  EXACT: the cells' fractions from the unrounded position
// product (FP32 models; 16-bit models round the blended values to 16 bits).
// Bound by the 96 random 8-byte reads per sample.  Workgroups go to the eight XCDs in turn, and each
// XCD has its own 4 MB L2: workgroups x, x + 8, ... take level 11 - x (a hashed level of the default
// grid is 2 MB) and half of the samples of one coarse level, so that a table is read into one L2
// only (every XCD reading every level's 18.7 MB misses it: 47 us at 65,536 samples).  The placement
// is a matter of speed alone.
template <bool EXACT>
__global__ __launch_bounds__(256) void k_hash_gather(int64_t B, const float2 *__restrict__ table, HashGridArgs grid,
                                                     HashScatterPlan plan, bool sliced, HashTrainBufs bufs) {
    const int x = blockIdx.x & 7;
    const int64_t stride = hash_level_stride(B), half = (B + 1) / 2;
    const int64_t nt = (int64_t)(gridDim.x >> 3) * blockDim.x;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const int level = part == 0 ? kHashLevels - 1 - x : (kHashLevels - 1 - 8) - (x >> 1);
        HashLevel lv = grid.lv[0];
        HashScatterLevel sl = plan.lv[0];
#pragma unroll
        for (int l = 1; l < kHashLevels; ++l)   // constant indices: the argument structs stay in scalar registers
            if (level == l) {
                lv = grid.lv[l];
                sl = plan.lv[l];
            }
        const uint32_t n1 = (uint32_t)lv.res + 1u;
        const int64_t b0 = part == 1 && (x & 1) ? half : 0, b1 = part == 1 && !(x & 1) ? half : B;
#pragma unroll 2
        for (int64_t b = b0 + (int64_t)(blockIdx.x >> 3) * blockDim.x + threadIdx.x; b < b1; b += nt) {
            const f32x4 pos = *(const f32x4 *)(bufs.attr + 8 * b);
            float2 t[8];
            hash_fetch8(lv, grid.tmask, table, pos[0], pos[1], pos[2], t);
            if (sliced) {
                const HashCell h = hash_cell<EXACT>(pos[0], pos[1], pos[2], lv.res);
                uint32_t code = 0u;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t v1 = (uint32_t)h.c[1] + (r & 1), v2 = (uint32_t)h.c[2] + (r >> 1);
                    const uint32_t row = v1 + n1 * v2;
                    const uint32_t hashed = (((v1 * 2654435761u) ^ (v2 * 805459861u)) & grid.tmask) / kSliceEntries;
                    code |= (lv.dense ? (sl.rows == 1 ? row : __umulhi(row, sl.magic)) : hashed) << (8 * r);
                }
                bufs.codes[level * stride + b] = code;
            }
            bufs.vals[level * stride + b] = hash_blend2<EXACT>(lv, pos[0], pos[1], pos[2], t);
        }
    }
}

// One workgroup per task of the plan: slice `slice` of a level over samples [s0, s1).  The workgroup
// walks the samples' slice codes, a wave queues those that touch the slice and adds 64 at a time
// into LDS (both corners of a matching row, both features).  Then, for a slice of its own, Adam on
// its entries (ADAM; parameters and moments were requested before the walk, so that their HBM
// latency lies under it) or the gradient; a shared slice goes to the merged accumulators.
// LDS holds one workgroup per CU (128 KB of sums), so the walk's latencies are covered by 16 waves:
// of a hashed slice's 34 us (256 at once), 9 are the parameters' reads from HBM, 17 the walk, 4 the
// last adds and 4 Adam and the stores.
template <bool ADAM>
__global__ __launch_bounds__(kScatThreads) void k_hash_scatter(HashGridArgs grid, HashScatterPlan plan,
                                                               HashTrainBufs bufs, GridAcc gacc, int64_t B, float scale,
                                                               float *__restrict__ grad, HashAdam ad) {
    __shared__ u32x4 s_acc4[kSliceEntries];   // two 64-bit sums per entry
    __shared__ uint2 s_q[kScatThreads / 64][128];   // (sample, slice code xor the slice's)
    unsigned long long *s_acc = (unsigned long long *)s_acc4;
    // the shared slices' tasks are dispatched first: they are the short ones
    int task = (int)blockIdx.x + plan.first;
    if (task >= plan.tasks) task -= plan.tasks;
    // the task's level: constant indices only, so that the argument structs stay in registers
    int level = 0;
    HashLevel lv = grid.lv[0];
    HashScatterLevel sl = plan.lv[0];
#pragma unroll
    for (int l = 1; l < kHashLevels; ++l)
        if (task < plan.lv[l - 1].task0) {
            level = l;
            lv = grid.lv[l];
            sl = plan.lv[l];
        }
    const int rel = task - sl.task0;
    const int slice = rel / sl.reps, rep = rel - slice * sl.reps;
    const uint32_t n1 = (uint32_t)lv.res + 1u, T = grid.tmask + 1u;
    const uint32_t row0 = (uint32_t)slice * (uint32_t)sl.rows;
    uint32_t base, count;   // the slice's entries within its level
    if (lv.dense) {
        base = row0 * n1;
        count = min((uint32_t)sl.rows * n1, n1 * n1 * n1 - base);
    } else {
        base = (uint32_t)slice * kSliceEntries;
        count = min((uint32_t)kSliceEntries, T - base);
    }
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t e0 = 2 * (size_t)(lv.off + base);   // the slice's first grid parameter
    float2 pw[kScatPer], pm[kScatPer], pv[kScatPer];
    if (ADAM && sl.reps == 1) {
#pragma unroll
        for (int k = 0; k < kScatPer; ++k) {
            const uint32_t e = (uint32_t)(tid + k * kScatThreads);
            if (e < count) {
                pw[k] = *(const float2 *)(ad.w + e0 + 2 * e);
                pm[k] = *(const float2 *)(ad.m + e0 + 2 * e);
                pv[k] = *(const float2 *)(ad.v + e0 + 2 * e);
            }
        }
    }
    if (ADAM) {
        const uint32_t nonfinite = *gacc.nonfinite;
        if (nonfinite && blockIdx.x == 0 && tid == 0) atomicOr(ad.bad, NIRC_FLAG_NONFINITE_GRAD);
        if (nonfinite || *ad.bad != 0u) return;   // (the same for every workgroup)
    }
    for (uint32_t e = tid; e < count; e += kScatThreads) s_acc4[e] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    const uint32_t pat = (uint32_t)slice * 0x01010101u;
    const int64_t stride = hash_level_stride(B);
    const uint32_t *codes = bufs.codes + level * stride;
    const float2 *dE = bufs.dvals + level * stride;
    const uint32_t lmask = min(T, (uint32_t)kSliceEntries) - 1u;
    uint2 *queue = s_q[wave];
    // 2^36 v to the nearest integer (ties to even, as llrintf): exactly the sum's low bits when the
    // FP64 unit adds it to 1.5 x 2^52; in range for |v| < 2^14, beyond it by the library
    auto fix36 = [](float v) -> unsigned long long {
        if (fabsf(v) >= 0x1p14f) return (unsigned long long)llrintf(v * 0x1p36f);
        return __builtin_bit_cast(unsigned long long, __builtin_fma((double)v, 0x1p36, 0x1.8p52)) - 0x4338000000000000ull;
    };
    auto add = [&](uint32_t e, float w, float2 d) {   // in range: checked by the gradient kernel
        atomicAdd(s_acc + 2 * e, fix36(w * d.x));
        atomicAdd(s_acc + 2 * e + 1, fix36(w * d.y));
    };
    int queued = 0;
    auto push = [&](bool hit, uint32_t b, uint32_t x) {
        const uint64_t mask = __ballot(hit);
        if (hit)
            queue[queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = make_uint2(b, x);
        queued += __popcll(mask);
    };
    // 64 queued samples at a time, one per lane: a batch's loads are issued when it is full and its
    // adds made when the next one is, so that their latency lies under the walk
    struct Batch {
        uint32_t b, x;   // no byte of x zero: nothing to add
        float2 d;
        f32x4 pos;
    };
    Batch cur{0u, ~0u, make_float2(0.f, 0.f), f32x4{0.f, 0.f, 0.f, 0.f}};
    auto load = [&](int n) {   // takes the first n <= 64 entries off the queue
        wave_sync();
        const uint2 e = queue[lane], rest = queue[64 + lane];
        Batch t{0u, ~0u, make_float2(0.f, 0.f), f32x4{0.f, 0.f, 0.f, 0.f}};
        if (lane < n) {
            t.b = e.x;
            t.x = e.y;
            t.d = dE[e.x];
            t.pos = *(const f32x4 *)(bufs.attr + 8 * (size_t)e.x);
        }
        wave_sync();
        queued -= n;
        if (lane < queued) queue[lane] = rest;
        wave_sync();
        return t;
    };
    auto rows = [](uint32_t x) { return (x - 0x01010101u) & ~x & 0x80808080u; };   // lowest flag: a zero byte
    // adds a matching corner row (two corners, two features) of each loaded sample, again while many
    // lanes have one (a coarse level's rows share a slice); the few that are left (6 % of a hashed
    // level's samples have a second row) go back to the queue instead of holding the wave
    auto drain = [&](Batch t) {
        const HashCell h = hash_cell(t.pos[0], t.pos[1], t.pos[2], lv.res);
        const uint32_t c0 = (uint32_t)h.c[0];
        do {
            const uint32_t z = rows(t.x);
            if (z) {
                const int sh = __builtin_ctz(z) & 24, r = sh >> 3;
                t.x |= 0xFFu << sh;
                const uint32_t v1 = (uint32_t)h.c[1] + (r & 1), v2 = (uint32_t)h.c[2] + (r >> 1);
                const float w0 = corner_weight(h, 0, r & 1, r >> 1), w1 = corner_weight(h, 1, r & 1, r >> 1);
                uint32_t i0, i1;
                if (lv.dense) {
                    i0 = (v1 + n1 * v2 - row0) * n1 + c0;
                    i1 = i0 + 1u;
                } else {
                    const uint32_t y = (v1 * 2654435761u) ^ (v2 * 805459861u);
                    i0 = (c0 ^ y) & lmask;
                    i1 = ((c0 + 1u) ^ y) & lmask;
                }
                add(i0, w0, t.d);
                add(i1, w1, t.d);
            }
        } while (__popcll(__ballot(rows(t.x) != 0u)) > 24);
        push(rows(t.x) != 0u, t.b, t.x);
    };
    // the walk: four consecutive samples per lane and step, the next step's codes loaded ahead
    // (a level's codes and the parts' bounds are 16-byte aligned; past the end nothing matches)
    const int64_t s0 = (int64_t)rep * sl.per, s1 = min(B, s0 + sl.per);
    auto fetch = [&](int64_t b) {
        u32x4 c = u32x4{~pat, ~pat, ~pat, ~pat};
        if (b < s1) c = *(const u32x4 *)(codes + b);
        if (b + 4 > s1)
#pragma unroll
            for (int j = 0; j < 4; ++j) c[j] = b + j < s1 ? c[j] : ~pat;
        return c;
    };
    int64_t b0 = s0 + 256 * wave + 4 * lane;
    u32x4 next = fetch(b0);
    for (int64_t w0 = s0 + 256 * wave; w0 < s1; w0 += 4 * kScatThreads, b0 += 4 * kScatThreads) {
        const u32x4 now = next;
        next = fetch(b0 + 4 * kScatThreads);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = now[j] ^ pat;
            push(rows(x) != 0u, (uint32_t)(b0 + j), x);   // at most 63 + 64 queued
            while (queued >= 64) {   // every turn takes a row off each sample it drains
                const Batch full = load(64);
                drain(cur);          // (pushes at most 64 behind the at most 63 left)
                cur = full;
            }
        }
    }
    drain(cur);
    while (queued > 0) drain(load(min(queued, 64)));
    __syncthreads();

    if (sl.reps > 1) {
        unsigned long long *out = gacc.acc + sl.merge0 + 2 * (size_t)base;
        for (uint32_t i = tid; i < 2 * count; i += kScatThreads) {
            const unsigned long long a = s_acc[i];
            if (a) atomicAdd(out + i, a);
        }
        return;
    }
    const float t = ADAM ? (float)(*ad.step + 1) : 0.0f;
    const float c1 = ADAM ? 1.0f - powf(ad.b1, t) : 0.0f, c2 = ADAM ? 1.0f - powf(ad.b2, t) : 0.0f;
    const bool nan = !ADAM && *gacc.nonfinite != 0u;
#pragma unroll
    for (int k = 0; k < kScatPer; ++k) {
        const uint32_t e = (uint32_t)(tid + k * kScatThreads);
        if (e >= count) continue;
        const float gx = __ll2float_rn((long long)s_acc[2 * e]) * 0x1p-36f * scale;
        const float gy = __ll2float_rn((long long)s_acc[2 * e + 1]) * 0x1p-36f * scale;
        if constexpr (ADAM) {
            const float wx = adam_update(pw[k].x, pm[k].x, pv[k].x, gx, c1, c2, ad.lr, ad.b1, ad.b2, ad.eps);
            const float wy = adam_update(pw[k].y, pm[k].y, pv[k].y, gy, c1, c2, ad.lr, ad.b1, ad.b2, ad.eps);
            *(float2 *)(ad.w + e0 + 2 * e) = make_float2(wx, wy);
            *(float2 *)(ad.m + e0 + 2 * e) = pm[k];
            *(float2 *)(ad.v + e0 + 2 * e) = pv[k];
        } else {
            const float a = nan ? __builtin_nanf("") : gx, b = nan ? __builtin_nanf("") : gy;
            grad[e0 + 2 * e] = a;
            grad[e0 + 2 * e + 1] = b;
            if (!isfinite(a) || !isfinite(b)) atomicOr(ad.bad, NIRC_FLAG_NONFINITE_GRAD);
        }
    }
}

// The merged levels' parameters (accumulator i: parameter i of the level that holds it) and, with
// ADAM, the MLP's (their reduced gradients in mlp_grad): Adam, or the gradient of the merged levels.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_hash_merge(HashGridArgs grid, HashScatterPlan plan, GridAcc gacc, float scale,
                                                    const float *__restrict__ mlp_grad, float *__restrict__ grad,
                                                    HashAdam ad) {
    const int64_t mlp = ADAM ? kHashMlp : 0;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= mlp + plan.merged_elems) return;
    if (ADAM && *ad.bad) return;
    int64_t o = 0;   // offset from the grid's first parameter (the MLP's are below it)
    float g;
    if (i < mlp) {
        o = i - kHashMlp;
        g = mlp_grad[i];
    } else {
        const int64_t j = i - mlp;
#pragma unroll
        for (int l = 0; l < kHashLevels; ++l) {   // merge0 falls with the level
            const int m0 = plan.lv[l].merge0;
            const int64_t n1 = (int64_t)grid.lv[l].res + 1;
            const int64_t n = 2 * (grid.lv[l].dense ? n1 * n1 * n1 : (int64_t)grid.tmask + 1);
            if (m0 >= 0 && j >= m0 && j < m0 + n) o = 2 * (int64_t)grid.lv[l].off + (j - m0);
        }
        g = !ADAM && *gacc.nonfinite ? __builtin_nanf("") : __ll2float_rn((long long)gacc.acc[j]) * 0x1p-36f * scale;
    }
    if constexpr (ADAM) {
        const float t = (float)(*ad.step + 1);
        const float c1 = 1.0f - powf(ad.b1, t), c2 = 1.0f - powf(ad.b2, t);
        float m = ad.m[o], v = ad.v[o];
        ad.w[o] = adam_update(ad.w[o], m, v, g, c1, c2, ad.lr, ad.b1, ad.b2, ad.eps);
        ad.m[o] = m;
        ad.v[o] = v;
    } else {
        grad[o] = g;
        if (!isfinite(g)) atomicOr(ad.bad, NIRC_FLAG_NONFINITE_GRAD);
    }
}

// Grids without a plan: the 16 values of one (sample, level) - 8 corners x 2 features - in 16
// consecutive lanes, corners along x (neighbouring entries) in consecutive lane pairs, so that an
// instruction's adds to one cache line travel together; zeros are skipped.
__global__ __launch_bounds__(256) void k_hash_scatter_atomic(HashGridArgs grid, HashTrainBufs bufs, GridAcc gacc,
                                                             int64_t B) {
    __shared__ HashLevel s_lv[kHashLevels];
    stage_levels(s_lv, grid);
    __syncthreads();
    const int lane = threadIdx.x & 63, corner = (lane & 15) >> 1, f = lane & 1;
    const int64_t n = B * kHashLevels, step = (int64_t)gridDim.x * blockDim.x / 16;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 16; i < n; i += step) {
        const int level = (int)(i / B);
        const int64_t b = i - level * B;
        const float2 d = bufs.dvals[level * hash_level_stride(B) + b];
        const float *x = bufs.attr + 8 * b;
        const HashLevel lv = s_lv[level];
        const HashCell cell = hash_cell(x[0], x[1], x[2], lv.res);
        float w;
        const uint32_t e = hash_entry(lv, grid.tmask, cell, corner, w);
        grid_acc_add(gacc, 2 * (size_t)e + f, w * (f ? d.y : d.x));
    }
}

hipError_t launch_hash_prep(const Points &pts, const Queries &q, const float *table, const HashGridArgs &grid,
                            const HashScatterPlan &plan, bool sliced, bool exact, bool first, const HashTrainBufs &bufs,
                            GridAcc gacc, hipStream_t s, const TrainDraw *draw, const HashDrawn &drawn) {
    static_assert(kHashLevels == 12, "8 XCDs: 8 levels, and two workgroup sets on each of the other 4");
    const dim3 pg((unsigned)((q.count + 255) / 256));
    const int64_t merged = sliced ? plan.merged_elems : 0;
    if (draw)
        hipLaunchKernelGGL(k_hash_points<true>, pg, dim3(256), 0, s, pts, q, *draw, drawn, merged, bufs, gacc, first);
    else
        hipLaunchKernelGGL(k_hash_points<false>, pg, dim3(256), 0, s, pts, q, TrainDraw{}, drawn, merged, bufs, gacc,
                           first);
    int64_t per = (q.count + 255) / 256;   // workgroups per XCD
    if (per > 128) per = 128;
    const dim3 nb((unsigned)(8 * per)), block(256);
    const float2 *t2 = (const float2 *)table;
    if (exact) hipLaunchKernelGGL(k_hash_gather<true>, nb, block, 0, s, q.count, t2, grid, plan, sliced, bufs);
    else hipLaunchKernelGGL(k_hash_gather<false>, nb, block, 0, s, q.count, t2, grid, plan, sliced, bufs);
    return hipGetLastError();
}

hipError_t launch_hash_scatter(const HashGridArgs &grid, const HashScatterPlan &plan, const HashTrainBufs &bufs,
                               GridAcc gacc, int64_t B, float scale, const float *mlp_grad, float *grad,
                               const HashAdam &ad, bool adam, hipStream_t s) {
    const int64_t rest = plan.merged_elems + (adam ? kHashMlp : 0);
    const dim3 tasks(plan.tasks), block(kScatThreads), merge((unsigned)((rest + 255) / 256));
    if (adam) hipLaunchKernelGGL(k_hash_scatter<true>, tasks, block, 0, s, grid, plan, bufs, gacc, B, scale, grad, ad);
    else hipLaunchKernelGGL(k_hash_scatter<false>, tasks, block, 0, s, grid, plan, bufs, gacc, B, scale, grad, ad);
    if (rest == 0) return hipGetLastError();
    if (adam)
        hipLaunchKernelGGL(k_hash_merge<true>, merge, dim3(256), 0, s, grid, plan, gacc, scale, mlp_grad, grad, ad);
    else
        hipLaunchKernelGGL(k_hash_merge<false>, merge, dim3(256), 0, s, grid, plan, gacc, scale, mlp_grad, grad, ad);
    return hipGetLastError();
}

hipError_t launch_hash_scatter_atomic(const HashGridArgs &grid, const HashTrainBufs &bufs, GridAcc gacc, int64_t B,
                                      hipStream_t s) {
    int64_t nb = (B * kHashLevels * 16 + 255) / 256;
    if (nb > 2048) nb = 2048;
    hipLaunchKernelGGL(k_hash_scatter_atomic, dim3((unsigned)nb), dim3(256), 0, s, grid, bufs, gacc, B);
    return hipGetLastError();
}

}  // namespace nirc
