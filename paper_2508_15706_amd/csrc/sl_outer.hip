// Dense outer steps of the DiLoCo family (Eq. (1): DiLoCo's Nesterov outer
// momentum; Section 3.2: DiLoCo-LOM; appendix "Exact algorithmic description of
// DiLoCo variants").  They are the dense counterparts of the sparse aggregate
// in sl_apply.hip and walk the same chunk work list, so that elements of the
// arenas that belong to no tensor are never touched.
//
//   k_lom_direction   m <- mu*m + delta ; dir <- delta + mu*m         (one worker)
//   k_dense_avg_apply avg = (1/R) sum_r dirs[r], r ascending from +0.0f;
//                     [m <- mu*m + avg ; avg <- avg + mu*m] ; theta <- theta - lr*avg
//
// Every "c*y + z" is one fp32 fused multiply-add.  Both kernels are pure
// streams, bound by memory: one wavefront owns one chunk and moves it in two halves
// of eight 16-byte accesses per lane per stream, all loads of a stream under way before the first result -
// in partial chunks too, where a lane whose four columns exist still moves them with one access (200 x 530 matrices
// and the like, 3.4M elements, four directions: element by element 60 us, so 23; with momentum 72 and 30).
#include <type_traits>

#include "sl_device.h"
#include "sl_internal.h"

// 16-byte accesses per lane and stream that are in flight together (half a chunk; a quarter
// and a whole chunk measured the same within the run-to-run spread of these kernels)
#ifndef SL_LOM_STEP
#define SL_LOM_STEP 8
#endif
#ifndef SL_DENSE_STEP
#define SL_DENSE_STEP 8
#endif
// LDS that a workgroup asks for and does not use: two of them fit a compute unit then (the compute unit's 160 KB are handed out
// in pieces of 1280 bytes, and three times 43 of these are more).  With more waves the memory has more rows open
// than it keeps, and is slower (direction / four directions averaged, ms, with as many workgroups as the registers allow, three (53,760
// bytes), two: 1.8B list 5.06 / 7.66, 4.86 / 7.66, 4.84 / 7.40; 400,000 x 1000 1.85 / 2.27, 1.64 / 2.26, 1.56 / 2.16; 178M list and
// 786,432 x 768 within 2 %).  The average with momentum has registers for two workgroups only and takes the same time either way.
#ifndef SL_STREAM_LDS
#define SL_STREAM_LDS 54272
#endif
namespace {

struct LomArgs {
    const SlChunkDesc *desc;
    float *m;
    const float *delta;
    float *dir;
    float mu;
    long long n_chunks;
    unsigned order;          // sl_work_group
};

// KEEP: without the streaming hint (sl_rows_unaligned).
template <bool KEEP>
__global__ void __launch_bounds__(256) k_lom_direction(LomArgs A)
{
    const int lane = threadIdx.x & 63;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long c = (long long)sl_work_group(blockIdx.x, A.order) * (blockDim.x >> 6) + wave;
    if (c >= A.n_chunks) return;
    const SlChunkDesc d = A.desc[c];
    float *mc = A.m + d.base;
    const float *dc = A.delta + d.base;
    float *oc = A.dir + d.base;
    const int lr = lane >> 4, lc = (lane & 15) * 4;
    const unsigned stride = (unsigned)d.stride;
    if (d.flags & SLC_FULL) {
        const unsigned o0 = 4u * (lr * stride + lc), step = 16u * stride;
        constexpr int S = SL_LOM_STEP;
#pragma unroll
        for (int q = 0; q < 16 / S; ++q) {
            sl_f4 mv[S], dv[S];
#pragma unroll
            for (int u = 0; u < S; ++u) mv[u] = sl_load_stream_at<KEEP>(mc, (S * q + u) * step, o0);
#pragma unroll
            for (int u = 0; u < S; ++u) dv[u] = sl_load_stream_at<KEEP>(dc, (S * q + u) * step, o0);
#pragma unroll
            for (int u = 0; u < S; ++u) {
                sl_f4 m = mv[u], g = dv[u], o;
                m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
                m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
                o.x = fmaf(A.mu, m.x, g.x), o.y = fmaf(A.mu, m.y, g.y);
                o.z = fmaf(A.mu, m.z, g.z), o.w = fmaf(A.mu, m.w, g.w);
                sl_store_stream_at<KEEP>(mc, (S * q + u) * step, o0, m);
                sl_store_stream_at<KEEP>(oc, (S * q + u) * step, o0, o);
            }
        }
    } else {
        const int rows = d.rows, cols = d.cols, last_cols = d.last_cols;
        constexpr int S = SL_LOM_STEP;
#pragma unroll
        for (int q = 0; q < 16 / S; ++q) {
            sl_f4 mv[S], dv[S];
            sl_load_partial<S, false, KEEP>(A.m, d, S * q, lane, mv);
            sl_load_partial<S, false, KEEP>(A.delta, d, S * q, lane, dv);
#pragma unroll
            for (int u = 0; u < S; ++u) {
                const int row = 4 * (S * q + u) + lr, n = (row < rows - 1 ? cols : row == rows - 1 ? last_cols : 0) - lc;
                sl_f4 m = mv[u], g = dv[u], o;
                m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
                m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
                o.x = fmaf(A.mu, m.x, g.x), o.y = fmaf(A.mu, m.y, g.y);
                o.z = fmaf(A.mu, m.z, g.z), o.w = fmaf(A.mu, m.w, g.w);
                sl_store_edge<KEEP>(mc + (row * stride + lc), n, m);
                sl_store_edge<KEEP>(oc + (row * stride + lc), n, o);
            }
        }
    }
}

struct DenseArgs {
    const SlChunkDesc *desc;
    float *theta;
    float *mom;              // global momentum (Eq. (1)), or null
    float neg_lr, inv_R, mu;
    int R;
    long long n_chunks;
    unsigned order;          // sl_work_group
    const float *dirs[SL_MAX_WORKERS];
};

// SHORT: without it the compiler waits for a worker's first loads before it requests the last three, two trips to memory per
// worker.  Lists that give every compute unit a few waves only pay for that (us, so / SHORT, four directions and four with momentum: 864
// chunks 17.0 / 14.9 and 22.4 / 20.5, 1024 20.6 / 19.3 and 27.7 / 27.0, 4200 75.5 / 73.3 and 101.0 / 98.8); long ones are faster
// with fewer loads open at a time (6144 98.6 / 99.5, 16384 260 / 273, 1.8B list 7362 / 7454), and so are ragged ones at every length (32,000 x
// 100 19.0 / 20.0, 200 x 530 15.4 / 16.2): the loads of their partial chunks come one by one, and neighbours that share lines should
// meet.  The line lies between the two.
template <bool NESTEROV, bool SHORT, bool KEEP>
__global__ void __launch_bounds__(256) k_dense_avg_apply(DenseArgs A)
{
    const int lane = threadIdx.x & 63;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long c = (long long)sl_work_group(blockIdx.x, A.order) * (blockDim.x >> 6) + wave;
    if (c >= A.n_chunks) return;
    const SlChunkDesc d = A.desc[c];
    float *tc = A.theta + d.base;
    float *mc = NESTEROV ? A.mom + d.base : nullptr;
    const int lr = lane >> 4, lc = (lane & 15) * 4;
    const unsigned stride = (unsigned)d.stride;
    const int R = A.R;
    const int rows = d.rows, cols = d.cols, last_cols = d.last_cols;
    const unsigned o0 = 4u * (lr * stride + lc), step = 16u * stride;
    constexpr int S = SL_DENSE_STEP;
    auto part = [&](int q, auto is_full) __attribute__((always_inline)) {
        constexpr bool full = decltype(is_full)::value;
        // access u of this step: elements 4 (S q + u) + lr, lc .. lc + 3 of the chunk
        auto exist = [&](int u) -> int {                    // how many of them (partial chunks)
            const int row = 4 * (S * q + u) + lr;
            return (row < rows - 1 ? cols : row == rows - 1 ? last_cols : 0) - lc;
        };
        auto load = [&](const float *p, sl_f4 (&v)[S]) __attribute__((always_inline)) {
            if (full) {
#pragma unroll
                for (int u = 0; u < S; ++u) v[u] = sl_load_stream_at<KEEP>(p, (S * q + u) * step, o0);
            } else {
#pragma unroll
                for (int u = 0; u < S; ++u) v[u] = sl_load_edge<KEEP>(p + ((4 * (S * q + u) + lr) * stride + lc), exist(u));
            }
        };
        sl_f4 th[S], mo[NESTEROV ? S : 1], acc[S];
        load(tc, th);
        if constexpr (NESTEROV) load(mc, mo);
#pragma unroll
        for (int u = 0; u < S; ++u) acc[u] = sl_f4{0.f, 0.f, 0.f, 0.f};
        for (int r = 0; r < R; ++r) {                       // r ascending: the order is part of the result
            sl_f4 g[S];
            load(A.dirs[r] + d.base, g);
            if (full && SHORT) __builtin_amdgcn_sched_barrier(0);       // (all eight requested before the first is waited for)
#pragma unroll
            for (int u = 0; u < S; ++u) acc[u] = acc[u] + g[u];
        }
#pragma unroll
        for (int u = 0; u < S; ++u) {
            auto store = [&](float *p, sl_f4 v) __attribute__((always_inline)) {
                if (full) sl_store_stream_at<KEEP>(p, (S * q + u) * step, o0, v);
                else sl_store_edge<KEEP>(p + ((4 * (S * q + u) + lr) * stride + lc), exist(u), v);
            };
            sl_f4 g = acc[u] * A.inv_R;
            if constexpr (NESTEROV) {
                sl_f4 m = mo[u];
                m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
                m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
                store(mc, m);
                g.x = fmaf(A.mu, m.x, g.x), g.y = fmaf(A.mu, m.y, g.y);
                g.z = fmaf(A.mu, m.z, g.z), g.w = fmaf(A.mu, m.w, g.w);
            }
            sl_f4 v = th[u];
            v.x = fmaf(A.neg_lr, g.x, v.x), v.y = fmaf(A.neg_lr, g.y, v.y);
            v.z = fmaf(A.neg_lr, g.z, v.z), v.w = fmaf(A.neg_lr, g.w, v.w);
            store(tc, v);
        }
    };
    if (d.flags & SLC_FULL) {
#pragma unroll 1
        for (int q = 0; q < 16 / S; ++q) part(q, std::true_type{});
    } else {
#pragma unroll 1
        for (int q = 0; q < 16 / S; ++q) part(q, std::false_type{});
    }
}

int check_launch()
{
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}

}  // namespace

int slk_lom_direction(const sl_plan *p, float *m, const float *delta, float mu, float *dir, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    LomArgs A;
    A.desc = p->d_desc;
    A.m = m;
    A.delta = delta;
    A.dir = dir;
    A.mu = mu;
    A.n_chunks = p->n_chunks;
    const dim3 grid((unsigned)((p->n_chunks + 3) / 4)), block(256);
    A.order = sl_order(p, grid.x);
    hipLaunchKernelGGL(sl_rows_unaligned(p, SL_DIRECTION_KEPT_FROM) ? k_lom_direction<true> : k_lom_direction<false>, grid, block, SL_STREAM_LDS, st, A);
    return check_launch();
}

int slk_dense_avg_apply(const sl_plan *p, float *theta, float *mom, const float *const *dirs, int R, float lr,
                        float mu, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    DenseArgs A;
    A.desc = p->d_desc;
    A.theta = theta;
    A.mom = mom;
    A.neg_lr = -lr;
    A.inv_R = 1.0f / (float)R;
    A.mu = mu;
    A.R = R;
    A.n_chunks = p->n_chunks;
    for (int r = 0; r < SL_MAX_WORKERS; ++r) A.dirs[r] = r < R ? dirs[r] : nullptr;
    const dim3 grid((unsigned)((p->n_chunks + 3) / 4)), block(256);
    A.order = sl_order(p, grid.x);
    const bool is_short = p->n_chunks < SL_DENSE_SHORT_BELOW && p->n_partial * 32 < p->n_chunks;
    typedef void (*kernel_t)(DenseArgs);
#define SL_DENSE_KINDS(KEEP) {{k_dense_avg_apply<false, false, KEEP>, k_dense_avg_apply<false, true, KEEP>}, \
                              {k_dense_avg_apply<true, false, KEEP>, k_dense_avg_apply<true, true, KEEP>}}
    static const kernel_t table[2][2][2] = {SL_DENSE_KINDS(false), SL_DENSE_KINDS(true)};
#undef SL_DENSE_KINDS
    hipLaunchKernelGGL(table[sl_rows_unaligned(p, sl_dense_kept_from(p)) ? 1 : 0][mom ? 1 : 0][is_short ? 1 : 0], grid, block, SL_STREAM_LDS, st, A);
    return check_launch();
}
