// The aggregate + outer update (Algorithm 1, "Aggregate + Outer Update"; Eq. (2) lines 3-4) on short lists, over plain and
// coded payloads: what sl_apply.hip and sl_apply_coded.hip do with a wave per chunk, with all waves of a workgroup on ONE chunk.
//
// What bounds a short list is the chain of one wave (see sl_select_group.hip).  Here wave w owns 1 / WAVES of the chunk's positions:
// their theta, accumulators and outer update.  The payloads are decoded by worker, one wave each (w, w + WAVES, ..), into lists
// of (position, value) in LDS; behind one barrier every wave adds the entries of its own positions, worker after
// worker in the order r = 0 .. R - 1 - a part of each list, as the indices of a record ascend (where they do not, the whole list is
// looked through).  Same order of additions, same bits.
#include "sl_coded.h"

namespace {

struct GroupApplyArgs {
    const SlChunkDesc *desc;
    const SlCodedDesc *cdesc;
    float *theta;
    float *mom;              // global outer momentum buffer (Nesterov variant), else null
    float mu, neg_lr, inv_R;
    int R;
    int k, bits, hdr_bytes, rec_bytes;
    SlCodedGeom G;
    int stage_bytes;         // coded: LDS of a wave's words and running sums
    int off_list, off_bounds;        // LDS offsets of the lists and of each worker's parts
    const unsigned char *payload[SL_MAX_WORKERS];
    unsigned sec_words[SL_MAX_WORKERS];      // coded: words of each payload's quotient section
};

// CODED: payloads in the coded wire format.  NESTEROV: with DiLoCo's global Nesterov momentum (Eq. (1)).
template <int WAVES, bool CODED, bool NESTEROV>
__global__ void __launch_bounds__(64 * WAVES) k_apply_group(GroupApplyArgs A)
{
    constexpr int NA = 16 / WAVES, PART_LOG2 = WAVES == 8 ? 9 : 10;        // 16-byte accesses per lane; log2 of a wave's positions
    static_assert((WAVES << PART_LOG2) == SL_CHUNK, "parts of a chunk");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = sl_uniform(tid >> 6);
    const int k = A.k, bits = A.bits;
    float *acc = reinterpret_cast<float *>(smem);
    uint2 *const list = reinterpret_cast<uint2 *>(smem + A.off_list);
    unsigned short *const bounds = reinterpret_cast<unsigned short *>(smem + A.off_bounds);     // [worker][first | end][part]
#pragma unroll
    for (int u = 0; u < NA; ++u) reinterpret_cast<float4 *>(acc)[64 * (NA * wave + u) + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    const long long c = blockIdx.x;
    const SlChunkDesc d = A.desc[c];

    // ---- theta, and what the lanes keep of worker `lane`: its payload and where it has the chunk's bit vector
    const int lr = lane >> 4, lc = (lane & 15) * 4;
    const unsigned stride = (unsigned)d.stride, o0 = 4u * ((4u * NA * wave + lr) * stride + lc), step = 16u * stride;
    const bool full = d.flags & SLC_FULL;
    float *tc = A.theta + d.base, *mc = NESTEROV ? A.mom + d.base : nullptr;
    sl_f4 th[NA], mo[NA];
    // (The streaming hint stays on unaligned rows too: with / without it, us, 1001 columns, k = 64, R = 4, plain 256 chunks 8.4 / 9.1, 512 10.3 / 11.4, 1024 14.9 / 15.3, coded 1024
    // 16.6 / 17.6; with the momentum 256 10.3 / 11.4, 512 15.4 / 15.1, 1024 23.9 / 19.7, the one form that would gain.)
    if (full) {
#pragma unroll
        for (int u = 0; u < NA; ++u) th[u] = sl_load_stream_at(tc, u * step, o0);
        if constexpr (NESTEROV) {
#pragma unroll
            for (int u = 0; u < NA; ++u) mo[u] = sl_load_stream_at(mc, u * step, o0);
        }
    } else {
        sl_partial_request(A.theta, d, NA * wave, lane, th);
        if constexpr (NESTEROV) sl_partial_request(A.mom, d, NA * wave, lane, mo);
    }
    SlCodedDesc cd;
    unsigned v_word = 0;     // first word of the vector, from the start of the section
    int v_meta = 0;          // (first bit inside that word) | (bits << 5)
    if constexpr (CODED) {
        cd = A.cdesc[c];
        if (lane < A.R) {
            const sl_gbytes p = reinterpret_cast<sl_gbytes>(reinterpret_cast<unsigned long long>(A.payload[lane]));
            const SlVecPlace P = sl_coded_dir_entry(A.G, p + cd.dir_off, cd.pos);
            v_word = P.run_word + (unsigned)(P.start_bit >> 5);
            v_meta = (P.start_bit & 31) | (P.nbits << 5);
        }
    }

    // ---- decoding
    // Entry m of worker r: to its list, and which entries lie in which part.
    int prev, last_part;     // index of the entry before, and its part
    bool ascending;
    auto put = [&](int r, int m, bool live, unsigned j, float v) __attribute__((always_inline)) {
        const int before = sl_lane_read((int)j, lane - 1), up = lane ? before : prev, part = (int)(j >> PART_LOG2);
        const int from = m == 0 ? -1 : lane ? before >> PART_LOG2 : last_part;
        if (live) {
            list[r * k + m] = make_uint2(4u * j, __float_as_uint(v));
            unsigned short *first = bounds + 2 * WAVES * r, *end = first + WAVES;
            for (int q = from + 1; q <= part; ++q) {
                first[q] = (unsigned short)m;
                if (q) end[q - 1] = (unsigned short)m;
            }
        }
        ascending = ascending && sl_ballot(live && m > 0 && (int)j <= up) == 0;
        prev = __builtin_amdgcn_readlane((int)j, 63);
        last_part = prev >> PART_LOG2;
    };
    auto begin = [&]() __attribute__((always_inline)) { prev = -1, last_part = -1, ascending = true; };
    auto finish = [&](int r, int last) __attribute__((always_inline)) {     // last: the part of entry k - 1
        unsigned short *first = bounds + 2 * WAVES * r, *end = first + WAVES;
        sl_wave_sync();
        if (lane < WAVES) {
            if (lane > last || !ascending) first[lane] = (unsigned short)(ascending ? k : 0);
            if (lane >= last || !ascending) end[lane] = (unsigned short)k;
        }
    };
    // What is requested of a payload ahead of the decode of the one before it: the first 64 entries of a plain record, or a word per
    // lane of the bit vector and of the remainders, and the first 64 value fields.  Taken apart only when its turn comes.
    struct Ahead {
        unsigned w0, w1, f;
        unsigned char b0, b1;
        float table;
    };
    auto load_field = [&](const unsigned char *fields, int m, Ahead &h) __attribute__((always_inline)) {
        if (bits == 32) {
            h.f = reinterpret_cast<const unsigned *>(fields)[m];
        } else {
            const int at = (m * bits) >> 3;  // (the last byte holds the end of the last code)
            h.b0 = fields[at], h.b1 = fields[min(at + 1, ((k * bits) >> 3) - 1)];
        }
    };
    auto value_of = [&](const Ahead &h, float table, int m) __attribute__((always_inline)) {
        if (bits == 32) return __uint_as_float(h.f);
        const unsigned code = ((h.b0 | (unsigned)h.b1 << 8) >> ((m * bits) & 7)) & ((1u << (bits & 31)) - 1u);
        return __int_as_float(sl_lane_read(__float_as_int(table), (int)code));
    };
    const int n_fields = bits == 32 ? 0 : 1 << bits, nrw = A.G.rem_bytes >> 2, b = A.G.b;
    auto vector_word = [&](const unsigned char *p, int r, int w) __attribute__((always_inline)) {
        const unsigned long long at = (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)v_word, r) + (unsigned)w;
        return at < A.sec_words[r] ? reinterpret_cast<const unsigned *>(p + A.G.section)[at] : 0xFFFFFFFFu;   // (beyond the end: no entries)
    };
    auto request = [&](int r, Ahead &h) __attribute__((always_inline)) {
        const unsigned char *p = A.payload[r];
        const int m = min(lane, k - 1);
        h.table = 0.f;
        if constexpr (CODED) {
            h.w0 = vector_word(p, r, min(lane, A.G.ua));
            h.w1 = reinterpret_cast<const unsigned *>(p + cd.fix_off)[min(lane, max(nrw - 1, 0))];
            load_field(p + cd.fix_off + A.G.rem_bytes, m, h);
            if (n_fields) h.table = reinterpret_cast<const float *>(p + cd.lut_off)[min(lane, n_fields - 1)];
        } else {
            h.w0 = *reinterpret_cast<const u16_any *>(p + d.rec_off + ((3 * m) >> 1));
            load_field(p + d.rec_off + 3 * k / 2, m, h);
            if (n_fields) h.table = reinterpret_cast<const float *>(p + sl_lut_off(d, A.hdr_bytes, A.rec_bytes))[min(lane, n_fields - 1)];
        }
    };
    auto decode_plain = [&](int r, const Ahead &h) __attribute__((always_inline)) {
        const unsigned char *rec = A.payload[r] + d.rec_off, *fields = rec + 3 * k / 2;
        begin();
        auto entry = [&](int m, const Ahead &x) __attribute__((always_inline)) {
            const int mm = min(m, k - 1);    // (lanes beyond the last entry repeat it)
            put(r, m, m < k, (mm & 1) ? x.w0 >> 4 : x.w0 & 0xFFFu, value_of(x, h.table, mm));
        };
        entry(lane, h);
        constexpr int U = 4;                 // further passes whose loads are under way together
        for (int m0 = 64; m0 < k; m0 += 64 * U) {
            Ahead x[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (m0 + 64 * u < k) {
                    const int m = min(m0 + 64 * u + lane, k - 1);
                    x[u].w0 = *reinterpret_cast<const u16_any *>(rec + ((3 * m) >> 1));
                    load_field(fields, m, x[u]);
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (m0 + 64 * u < k) entry(m0 + 64 * u + lane, x[u]);
        }
        finish(r, last_part);
    };
    auto decode_coded = [&](int r, const Ahead &h) __attribute__((always_inline)) {
        // the bit vector and the remainders in LDS, value fields straight from the payload
        unsigned *raw = reinterpret_cast<unsigned *>(smem + SL_CHUNK * sizeof(float) + (size_t)wave * A.stage_bytes);
        unsigned *rem = raw + A.G.ua + 1;
        unsigned short *sums = reinterpret_cast<unsigned short *>(rem + nrw + 1);
        const unsigned char *p = A.payload[r], *fix = p + cd.fix_off;
        const int meta = __builtin_amdgcn_readlane(v_meta, r), sh = meta & 31, n = meta >> 5;
        sl_wave_sync();
        if (lane <= A.G.ua) raw[lane] = h.w0;
        for (int w = lane + 64; w <= A.G.ua; w += 64) raw[w] = vector_word(p, r, w);
        if (lane <= nrw) rem[lane] = lane < nrw ? h.w1 : 0u;
        if (lane == 0 && nrw >= 64) rem[64] = 0u;                // (64 words at most)
        for (int m = lane; m < k; m += 64) sums[m] = 0;          // (a vector with too few zeros)
        sl_wave_sync();
        // bit by bit: the i-th zero, at bit z, ends entry i, whose quotients so far sum to z - i
        for (int z0 = 0, i0 = 0; z0 < n; z0 += 64) {
            const int z = z0 + lane, at = sh + z;
            const bool zero = z < n && !((raw[min(at >> 5, A.G.ua)] >> (at & 31)) & 1u);
            const unsigned long long mask = sl_ballot(zero);
            const int i = i0 + sl_mbcnt(mask);
            if (zero && i < k) sums[i] = (unsigned short)(z - i);
            i0 += sl_popc(mask);
        }
        sl_wave_sync();
        begin();
        int carry = 0;
        Ahead x = h;
        for (int m0 = 0; m0 < k; m0 += 64) {
            const int m = m0 + lane, mm = min(m, k - 1), bit = mm * b, wi = bit >> 5;
            if (m0) load_field(fix + A.G.rem_bytes, mm, x);
            const unsigned f = __builtin_amdgcn_alignbit(rem[wi + (b ? 1 : 0)], rem[wi], (unsigned)(bit & 31)) & ((1u << b) - 1u);
            const int incl = sl_wave_iscan(m < k ? (int)f : 0) + carry;
            carry = __builtin_amdgcn_readlane(incl, 63);
            // index of entry m, cut to 12 bits: a malformed payload stays inside the chunk
            put(r, m, m < k, (unsigned)(mm + ((int)sums[mm] << b) + incl) & 0xFFFu, value_of(x, h.table, mm));
        }
        finish(r, last_part);
    };

    // ---- the workers
    Ahead next;
    if (wave < A.R) request(wave, next);
    for (int r = wave; r < A.R; r += WAVES) {
        const Ahead h = next;
        if (r + WAVES < A.R) request(r + WAVES, next);
        if constexpr (CODED) decode_coded(r, h);
        else decode_plain(r, h);
    }
    __syncthreads();
    // this wave's part of the list of worker `lane`
    int lo = 0, hi = 0;
    if (lane < A.R) lo = bounds[2 * WAVES * lane + wave], hi = bounds[2 * WAVES * lane + WAVES + wave];
    auto add = [&](int m, int end, uint2 e) __attribute__((always_inline)) {
        if (m < end && (int)(e.x >> (PART_LOG2 + 2)) == wave) {
            float *at = reinterpret_cast<float *>(smem + e.x);
            *at = *at + __uint_as_float(e.y);
        }
        sl_wave_sync();                      // worker r is complete before worker r + 1 is added
    };
    constexpr int U = 4;                     // workers whose first entries are read together
    for (int r0 = 0; r0 < A.R; r0 += U) {
        uint2 e[U];
        int first[U], end[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = min(r0 + u, A.R - 1);
            first[u] = __builtin_amdgcn_readlane(lo, r), end[u] = __builtin_amdgcn_readlane(hi, r);
            e[u] = list[r * k + min(first[u] + lane, k - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r0 + u < A.R) {
                add(first[u] + lane, end[u], e[u]);
                for (int m = first[u] + 64; m < end[u]; m += 64) add(m + lane, end[u], list[(r0 + u) * k + min(m + lane, k - 1)]);
            }
    }

    // ---- theta <- theta - lr * average
    if (!full) {
        sl_partial_place(d, NA * wave, lane, th);
        if constexpr (NESTEROV) sl_partial_place(d, NA * wave, lane, mo);
    }
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const float4 a = reinterpret_cast<const float4 *>(acc)[64 * (NA * wave + u) + lane];
        sl_f4 g;
        g.x = a.x * A.inv_R, g.y = a.y * A.inv_R, g.z = a.z * A.inv_R, g.w = a.w * A.inv_R;
        const int n = full ? 4 : sl_partial_exist(d, lr, lc, NA * wave + u);
        const unsigned at = (4u * (NA * wave + u) + lr) * stride + lc;
        if constexpr (NESTEROV) {
            sl_f4 m = mo[u];
            m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
            m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
            if (full) sl_store_stream_at(mc, u * step, o0, m);
            else sl_store_edge(mc + at, n, m);
            g.x = fmaf(A.mu, m.x, g.x), g.y = fmaf(A.mu, m.y, g.y);
            g.z = fmaf(A.mu, m.z, g.z), g.w = fmaf(A.mu, m.w, g.w);
        }
        sl_f4 v = th[u];
        v.x = fmaf(A.neg_lr, g.x, v.x), v.y = fmaf(A.neg_lr, g.y, v.y);
        v.z = fmaf(A.neg_lr, g.z, v.z), v.w = fmaf(A.neg_lr, g.w, v.w);
        if (full) sl_store_stream_at(tc, u * step, o0, v);
        else sl_store_edge(tc + at, n, v);
    }
}

}  // namespace

// bytes != null: coded payloads
int slk_apply_group(const sl_plan *p, float *theta, float *mom, float mu, const void *const *payloads, const size_t *bytes, int R, float lr,
                    int waves, hipStream_t st)
{
    GroupApplyArgs A;
    const SlCodedGeom &G = p->cg;
    A.desc = p->d_desc;
    A.cdesc = p->d_cdesc;
    A.theta = theta;
    A.mom = mom;
    A.mu = mu;
    A.neg_lr = -lr;
    A.inv_R = 1.0f / (float)R;
    A.R = R;
    A.k = p->k;
    A.bits = p->bits;
    A.hdr_bytes = p->hdr_bytes;
    A.rec_bytes = p->rec_bytes;
    A.G = G;
    for (int r = 0; r < SL_MAX_WORKERS; ++r) {
        A.payload[r] = r < R ? static_cast<const unsigned char *>(payloads[r]) : nullptr;
        const size_t sec = bytes && r < R && bytes[r] > (size_t)G.section ? (bytes[r] - (size_t)G.section) >> 2 : 0;
        A.sec_words[r] = sec > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned)sec;
    }
    auto up16 = [](size_t v) { return (v + 15) & ~(size_t)15; };
    A.stage_bytes = bytes ? (int)up16(4 * (size_t)(G.ua + 1 + (G.rem_bytes >> 2) + 1) + 2 * (size_t)p->k) : 0;
    size_t at = SL_CHUNK * sizeof(float) + (size_t)waves * A.stage_bytes;
    A.off_list = (int)at;
    at += sizeof(uint2) * (size_t)R * p->k;
    A.off_bounds = (int)at;
    at = up16(at + 2 * 2 * (size_t)waves * R);
    typedef void (*kernel_t)(GroupApplyArgs);
    static const kernel_t table[2][2][2] = {{{k_apply_group<4, false, false>, k_apply_group<4, false, true>},
                                             {k_apply_group<4, true, false>, k_apply_group<4, true, true>}},
                                            {{k_apply_group<8, false, false>, k_apply_group<8, false, true>},
                                             {k_apply_group<8, true, false>, k_apply_group<8, true, true>}}};
    const kernel_t fn = table[waves == 8 ? 1 : 0][bytes ? 1 : 0][mom ? 1 : 0];
    if (at > 65536) return SL_ERR_INVALID_ARG;           // (sl_apply_waves sends no such call)
    hipLaunchKernelGGL(fn, dim3((unsigned)p->n_chunks), dim3(64 * waves), at, st, A);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}
