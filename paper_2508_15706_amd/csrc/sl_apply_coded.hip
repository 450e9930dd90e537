// sl_decompress_avg_apply_coded (short lists: sl_apply_group.hip): the aggregate + outer update (Algorithm 1, "Aggregate + Outer
// Update"; Eq. (2) lines 3-4) over R payloads in the CODED wire format (sl_coded.h; the
// appendix "Compression of indices in Top-k" is where the index coder enters the method).
//
// One wavefront owns one chunk, as in sl_apply.hip: fp32 accumulators of the chunk in LDS,
// workers added in the order r = 0..R-1, theta streamed through registers once.  What differs is
// how a worker's k (index, value) entries are found:
//   1. lane r reads worker r's directory entry: where the chunk's quotient bit vector lies;
//   2. the workers' fixed records (table, remainders, value fields) and bit vectors are staged
//      in LDS with coalesced loads, the first of them fetched ahead of the theta loads;
//   3. every lane takes one 32-bit word of some worker's vector, counts its zero bits and, from one
//      prefix sum over the counts, writes down where every eighth zero of the vector lies (the byte,
//      and how many zeros of that byte come before it);
//   4. every lane takes 8 consecutive entries of some worker: it finds the first one's zero bit from that
//      note, the others in the 64 bits behind it; the i-th zero of a vector, at bit z, ends entry i,
//      whose quotients so far sum to z - i.  The entries' remainders are b bytes of the record, a prefix
//      sum over the lanes of a worker completes idx_i = i + ((z_i - i) << b) + r_0 + ... + r_i;
//   5. the same lanes add their entries, worker by worker.
// With few entries per chunk (LISTS) step 3 lists every zero of the words instead, step 4 turns that
// list into one of 16-bit indices and step 5 adds an entry per lane from it: more work, a shorter chain.
// Steps 3 and 4 run for all workers of a batch at once, so their cost per chunk hardly grows
// with R; only step 5 is a chain over the workers.
// What bounds it: above R * k of about 1024 entries per chunk the number of instructions, two waves per
// SIMD sharing the issue slots (LDS: 16 KB of accumulators per wave).  A chunk at k = 256, R = 16 takes 3183 vector,
// 821 scalar and 488 LDS instructions (50 vector lane slots per entry), and its wave issues in 47 % of
// its cycles (1174 us for 123,505 chunks); with lists everywhere, a lane per word of the longest possible vector and
// as many turns as the fullest word has zeros, it took 3500, 1233 and 538 (1404 us).
#include "sl_coded.h"

namespace {

#ifndef SL_CAPPLY_STAGE
#define SL_CAPPLY_STAGE 4096      // LDS bytes for one batch of staged workers
#endif
// Up to k = 128 with fewer than so many entries per chunk (R * k) the entries go through index lists in
// LDS: the decode is short there and hidden behind the theta loads, what is left is the length of its
// chain (24,000 chunks, lists / the other form: k = 64, R = 8 165 / 167 us; k = 128, R = 8 174 / 170;
// k = 96, R = 16 243 / 178; k = 64, R = 32 245 / 214).  Up to k = 16 at 2 bits that holds whatever R: two lanes
// per worker add while the others wait (k = 16, R = 64 272 / 299; 1, 3, 4 and 32 bits 315, 341, 403 and 355 with
// lists, 281, 295, 355 and 309 without).
#ifndef SL_CAPPLY_LISTS_BELOW
#define SL_CAPPLY_LISTS_BELOW 1024
#endif
#ifndef SL_CAPPLY_PFF
#define SL_CAPPLY_PFF 4           // words per lane fetched ahead of the theta loads: tables and fixed records,
#endif
#ifndef SL_CAPPLY_PFU
#define SL_CAPPLY_PFU 2           // ... bit vectors
#endif

struct CodedApplyArgs {
    SlCodedGeom G;
    const SlChunkDesc *desc;
    const SlCodedDesc *cdesc;
    float *theta;
    float *mom;              // global outer momentum buffer (Nesterov variant), else null
    float mu, neg_lr, inv_R;
    int R;
    int batch;               // workers staged at a time
    int slot_bytes;          // LDS bytes of one staged worker
    int fwp;                 // words of (table header + fixed record)
    unsigned magic_l;        // floor(2^32 / d) + 1 for d = lanes per worker in step 4
    int lpw_log2;            // staging: log2 of the lanes that fetch one worker's words (64 / lanes >= batch)
    int uwp_log2;            // log2 of the slots per worker in step 3 (a power of two >= G.ua)
    int E;                   // index lists: entries per lane in step 4, 8, or 4 when k is not a multiple of 8
    int off_t, off_q, off_h; // a slot's table of every eighth zero, its value pairs, its index list (bytes)
    int lds_per_wave;
    long long n_chunks;
    unsigned order;          // sl_work_group
    const unsigned char *payload[SL_MAX_WORKERS];
    unsigned sec_words[SL_MAX_WORKERS];   // words of each payload's quotient section
};

SL_DEV void acc_add(float *acc, unsigned j, float q) { acc[j] = acc[j] + q; }

// NESTEROV: with DiLoCo's global Nesterov momentum (Eq. (1)).
// LISTS (few entries): steps 3 to 5 go through index lists in LDS, see the top of the file.
// KEEP: the arenas' accesses without the streaming hint (sl_rows_unaligned).
template <bool TWO_BIT, bool NESTEROV, bool LISTS, bool KEEP>
__global__ void __launch_bounds__(256) k_apply_coded(CodedApplyArgs A)
{
    extern __shared__ __align__(16) unsigned char smem_all[];
    const SlCodedGeom &G = A.G;
    const int lane = threadIdx.x & 63, k = G.k, b = G.b;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long c = (long long)sl_work_group(blockIdx.x, A.order) * (blockDim.x >> 6) + wave;
    if (c >= A.n_chunks) return;
    unsigned char *smem = smem_all + (size_t)wave * A.lds_per_wave;
    float *acc = reinterpret_cast<float *>(smem);
    unsigned char *stage = smem + SL_CHUNK * sizeof(float);
    const SlChunkDesc d = A.desc[c];
    const SlCodedDesc cd = A.cdesc[c];
    const int bits = TWO_BIT ? 2 : G.bits;
    const int hdr = TWO_BIT ? 16 : G.hdr, hdrw = hdr >> 2;
    const int fwp = A.fwp, uraw = G.ua + 1;
    // one staged worker: [table header][fixed record][uraw words of the bit vector][where every eighth zero
    // lies, 16 bits each][step 5 by the lanes of step 4, 2-bit codes: the 16 pairs of values][else: indices]
    const int off_u = 4 * fwp, off_t = A.off_t, off_q = A.off_q, off_h = A.off_h;

    float *tc = A.theta + d.base;
    const int lr = lane >> 4, lc = (lane & 15) * 4;
    const unsigned stride = (unsigned)d.stride;
    const bool full = d.flags & SLC_FULL;

    // lane l keeps worker l's payload pointer and section size; the others read them across lanes
    static_assert(SL_MAX_WORKERS <= 64, "one payload per lane");
    const unsigned long long my_ptr = reinterpret_cast<unsigned long long>(A.payload[lane]);
    const unsigned my_words = A.sec_words[lane];
    asm volatile("" ::"v"(my_words));   // arrives with the pointer: no later wait may count it among the prefetches
    auto payload_of = [&](int r) -> sl_gbytes {
        const unsigned lo = (unsigned)sl_lane_read((int)(unsigned)my_ptr, r);
        const unsigned hi = (unsigned)sl_lane_read((int)(unsigned)(my_ptr >> 32), r);
        return reinterpret_cast<sl_gbytes>(((unsigned long long)hi << 32) | lo);
    };
    // Step 1, once for all workers: lane r < R learns where worker r keeps the chunk's bit vector:
    // first word (bounded by the section's size when it is used), shift and length.  This is the one
    // load that the loads of the vectors depend on.
    unsigned v_word = 0;         // first word of the vector, from the start of the section
    int v_meta = k << 5;         // (first bit inside that word) | (bits << 5)
    if (lane < A.R) {
        const SlVecPlace P = sl_coded_dir_entry(G, reinterpret_cast<sl_gbytes>(my_ptr) + cd.dir_off, cd.pos);
        v_word = P.run_word + (unsigned)(P.start_bit >> 5);
        v_meta = (P.start_bit & 31) | (P.nbits << 5);
    }
    // Staging.  A batch's workers share the wave's lanes: lanes [rs * LPW, (rs + 1) * LPW) fetch the words
    // of the batch's worker rs, LPW words at a time, so a lane needs its worker's pointer, vector place and
    // section size once per batch (four lane reads) and its addresses step by a constant.  Two parts per
    // worker, each fetched by straight-line code: fwp words of (table header, fixed record) and uraw words
    // of the bit vector (all ones beyond a payload's end: no entries).
    const int LPW = 1 << A.lpw_log2, rs = lane >> A.lpw_log2, qs = lane & (LPW - 1);
    unsigned char *const my_stage = stage + rs * A.slot_bytes;
    struct StageSrc {
        sl_gbytes p;
        unsigned word0, limit;
        bool live;
    };
    auto stage_src = [&](int r0, int nb) -> StageSrc {
        StageSrc S;
        S.live = rs < nb;
        const int r = S.live ? r0 + rs : r0;
        S.p = payload_of(r);
        S.word0 = (unsigned)sl_lane_read((int)v_word, r);
        S.limit = (unsigned)sl_lane_read((int)my_words, r);
        return S;
    };
    auto src_fixed = [&](const StageSrc &S, int u) -> unsigned {
        const int q = qs + (u << A.lpw_log2);
        const bool valid = S.live && q < fwp;
        const long long at = q < hdrw ? cd.lut_off + 4 * q : cd.fix_off + 4 * (q - hdrw);
        return valid ? *reinterpret_cast<sl_gwords>(S.p + at) : 0u;
    };
    auto src_vector = [&](const StageSrc &S, int u) -> unsigned {
        const int q = qs + (u << A.lpw_log2);
        const unsigned long long at = (unsigned long long)S.word0 + (unsigned)q;
        return (S.live && q < uraw && at < S.limit) ? reinterpret_cast<sl_gwords>(S.p + G.section)[at] : 0xFFFFFFFFu;
    };
    auto park_fixed = [&](int nb, int u, unsigned v) {
        const int q = qs + (u << A.lpw_log2);
        if (rs < nb && q < fwp) reinterpret_cast<unsigned *>(my_stage)[q] = v;
    };
    auto park_vector = [&](int nb, int u, unsigned v) {
        const int q = qs + (u << A.lpw_log2);
        if (rs < nb && q < uraw) reinterpret_cast<unsigned *>(my_stage + off_u)[q] = v;
    };

    constexpr int PFF = SL_CAPPLY_PFF, PFU = SL_CAPPLY_PFU;
    unsigned pf_f[PFF], pf_u[PFU], pn_f[PFF], pn_u[PFU];
    const int nb0 = min(A.batch, A.R);

    sl_f4 th[16], mo[NESTEROV ? 16 : 1];
    float *mc = NESTEROV ? A.mom + d.base : nullptr;
    // The first 64 * PF words of the first batch are fetched BEFORE the theta loads: loads complete in
    // order, so the decode then waits for these few words only and runs while the chunk's 16 KB of
    // theta are in flight.  (Tried: the directory entry one chunk ahead, a wave taking several chunks
    // in turn - the loop costs more registers than a wave has next to a second one; and half of the
    // theta loads ahead of these words, which leaves too little of the stream behind the decode.)
    {
        const StageSrc S = stage_src(0, nb0);
#pragma unroll
        for (int u = 0; u < PFF; ++u) pf_f[u] = src_fixed(S, u);
#pragma unroll
        for (int u = 0; u < PFU; ++u) pf_u[u] = src_vector(S, u);
    }
    // Sixteen loads are issued for EVERY chunk, so that the wait in front of the words fetched above
    // is "all but the last sixteen" whatever the chunk: a ragged chunk (a tensor's edge) reads its own
    // descriptor sixteen times instead, and then loads its elements (sl_load_partial).  Were the
    // sixteen under a condition, the number of loads behind those words would be unknown and the
    // wait would be for all of them on the full chunks too.
    {
        const float *none = reinterpret_cast<const float *>(A.desc + c);
        const float *ts = full ? tc : none, *ms = (NESTEROV && full) ? mc : none;
        const unsigned o0 = full ? 4u * (lr * stride + lc) : 0u, step = full ? 16u * stride : 0u;
#pragma unroll
        for (int i = 0; i < 16; ++i) th[i] = sl_load_stream_at<KEEP>(ts, i * step, o0);
        if constexpr (NESTEROV) {
#pragma unroll
            for (int i = 0; i < 16; ++i) mo[i] = sl_load_stream_at<KEEP>(ms, i * step, o0);
        }
    }
    if (!full) {
        sl_load_partial<16, false, KEEP>(A.theta, d, 0, lane, th);
        if constexpr (NESTEROV) sl_load_partial<16, false, KEEP>(A.mom, d, 0, lane, mo);
        // (waited for here: loads of this block in flight behind it would be counted by the wait in front of the staged words
        // on full chunks too: 24,000 of them, k = 256, R = 16, 238 us without this, 229 with it)
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
        reinterpret_cast<float4 *>(acc)[i * 64 + lane] = make_float4(0.f, 0.f, 0.f, 0.f);

    const int L = (k + 7) >> 3;                   // step 4: lanes per worker, eight entries each (without lists)
    const int uwp = 1 << A.uwp_log2;
    // One batch of workers: staged, decoded, added.  The first batch is processed by straight-line code
    // of its own ahead of the loop over the others: inside a loop the wait in front of the staged words
    // is for every outstanding load, the theta loads included, and the decode would start only once the
    // whole chunk has arrived; ahead of the loop it is for the words alone.
    auto do_batch = [&](const int r0, const bool first) __attribute__((always_inline)) {
        const int nb = min(A.batch, A.R - r0);
        sl_wave_sync();
        // ---- step 2: stage the batch.  The first words of both parts are in registers: fetched ahead of
        // the theta loads for the first batch (pf_*), while the previous batch was decoded for the others
        // (pn_*: registers of their own, so that the wait in front of the first batch's words stays
        // "everything but the theta loads" - one array written on both paths would make it "everything").
        {
            if (first) {
#pragma unroll
                for (int u = 0; u < PFF; ++u) park_fixed(nb, u, pf_f[u]);
#pragma unroll
                for (int u = 0; u < PFU; ++u) park_vector(nb, u, pf_u[u]);
            } else {
#pragma unroll
                for (int u = 0; u < PFF; ++u) park_fixed(nb, u, pn_f[u]);
#pragma unroll
                for (int u = 0; u < PFU; ++u) park_vector(nb, u, pn_u[u]);
            }
            if ((PFF << A.lpw_log2) < fwp || (PFU << A.lpw_log2) < uraw) {      // what the registers did not hold
                const StageSrc S = stage_src(r0, nb);
                for (int u = PFF; (u << A.lpw_log2) < fwp; u += 2) {
                    const unsigned v0 = src_fixed(S, u), v1 = src_fixed(S, u + 1);
                    park_fixed(nb, u, v0);
                    park_fixed(nb, u + 1, v1);
                }
                for (int u = PFU; (u << A.lpw_log2) < uraw; u += 2) {
                    const unsigned v0 = src_vector(S, u), v1 = src_vector(S, u + 1);
                    park_vector(nb, u, v0);
                    park_vector(nb, u + 1, v1);
                }
                // (every load of this block has been waited for by a lane that parked its word; said once
                // more for all of them, so that the registers they used are not taken to be in flight by
                // code that follows - which would put a wait for the theta loads in front of steps 4 and 5
                // on the lists that never come here)
                __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
            }
            if (r0 + A.batch < A.R) {
                const StageSrc S = stage_src(r0 + A.batch, min(A.batch, A.R - r0 - A.batch));
#pragma unroll
                for (int u = 0; u < PFF; ++u) pn_f[u] = src_fixed(S, u);
#pragma unroll
                for (int u = 0; u < PFU; ++u) pn_u[u] = src_vector(S, u);
            }
            sl_wave_sync();
        }
        // the dequantised value of a staged worker's entry m
        auto value_at = [&](const unsigned char *slot, int m) -> float {
            const float *lutp = reinterpret_cast<const float *>(slot);
            const unsigned char *vals = slot + 4 * hdrw + G.rem_bytes;
            if (TWO_BIT) return lutp[(vals[m >> 2] >> (2 * (m & 3))) & 3u];
            if (bits == 32) return reinterpret_cast<const float *>(vals)[m];
            return lutp[sl_code_at(vals, m, bits)];
        };
        // ---- no remainders (b = 0, k above 1419): a gap is its quotient, the vector is the chunk's bit map -
        // bit p is zero exactly where index p is selected - and the entries are added straight from it, the
        // i-th zero with the i-th value, worker after worker.  (Steps 3 to 5 would give the same sums.)
        if (b == 0) {
            const int passes = (G.ua + 63) >> 6;
            for (int r = 0; r < nb; ++r) {
                const unsigned char *slot = stage + r * A.slot_bytes;
                const unsigned *raw = reinterpret_cast<const unsigned *>(slot + off_u);
                const int meta = sl_lane_read(v_meta, r0 + r);
                const int sh = meta & 31, n = meta >> 5;
                int carry = 0;
                for (int t = 0; t < passes; ++t) {
                    const int j = 64 * t + lane;
                    unsigned zeros = 0;
                    if (j < G.ua) {
                        const unsigned w = __builtin_amdgcn_alignbit(raw[j + 1], raw[j], (unsigned)sh);
                        const int left = n - 32 * j;
                        const unsigned mask = left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u;
                        zeros = ~w & mask;
                    }
                    const int nz = __builtin_popcount(zeros);
                    const int incl = sl_wave_iscan(nz);
                    int lo = carry + incl - nz, hi = lo + nz - 1;    // entries of the word's lowest and highest zero
                    carry += __builtin_amdgcn_readlane(incl, 63);
                    // Two zeros per turn, one from each end of the word: two independent chains, their LDS
                    // reads issued together.  (An entry beyond k - 1 can only come from a malformed vector
                    // and takes the last entry's value.)
                    if constexpr (TWO_BIT) {
                        // the word's nz two-bit codes, entry `lo` at bit 0 of a 64-bit window
                        const unsigned *cw = reinterpret_cast<const unsigned *>(slot + 4 * hdrw + G.rem_bytes);
                        const int e0 = min(lo, k - 1), wi = (2 * e0) >> 5, csh = (2 * e0) & 31;
                        const unsigned c0 = cw[wi], c1 = cw[wi + 1], c2 = cw[wi + 2];
                        unsigned long long wl = ((unsigned long long)__builtin_amdgcn_alignbit(c2, c1, (unsigned)csh) << 32) |
                                                __builtin_amdgcn_alignbit(c1, c0, (unsigned)csh);
                        unsigned long long wh = nz ? wl << (64 - 2 * nz) : 0ull;      // entry `hi` in the two top bits
                        const float *lutp = reinterpret_cast<const float *>(slot);
                        while (zeros) {
                            const int pl = __builtin_ctz(zeros), ph = 31 - __builtin_clz(zeros);
                            const float q_lo = lutp[(unsigned)wl & 3u], q_hi = lutp[(unsigned)(wh >> 62)];
                            const unsigned j_lo = (unsigned)(32 * j + pl), j_hi = (unsigned)(32 * j + ph);
                            const float a_lo = acc[j_lo], a_hi = acc[j_hi];
                            acc[j_lo] = a_lo + q_lo;
                            if (ph != pl) acc[j_hi] = a_hi + q_hi;
                            zeros &= zeros - 1u;
                            zeros &= ~(1u << ph);
                            wl >>= 2, wh <<= 2;
                        }
                    } else {
                        while (zeros) {
                            const int pl = __builtin_ctz(zeros), ph = 31 - __builtin_clz(zeros);
                            const float q_lo = value_at(slot, min(lo, k - 1));
                            const float q_hi = value_at(slot, min(hi, k - 1));
                            acc_add(acc, (unsigned)(32 * j + pl), q_lo);
                            if (ph != pl) acc_add(acc, (unsigned)(32 * j + ph), q_hi);
                            zeros &= zeros - 1u;
                            zeros &= ~(1u << ph);
                            ++lo, --hi;
                        }
                    }
                }
                sl_wave_sync();               // worker r is complete before worker r+1 is added
            }
            return;
        }
        if constexpr (LISTS) {
        // ---- step 3 with lists: the zero bits of the vectors -> running quotient sums, by entry
        {
            const int slots = nb << A.uwp_log2;
            int carry = 0;
            for (int s0 = 0; s0 < slots; s0 += 64) {
                const int slot = s0 + lane;
                const int r = slot >> A.uwp_log2, j = slot & (uwp - 1);
                const bool live = slot < slots && j < G.ua;
                const int meta = sl_lane_read(v_meta, live ? r0 + r : 0);
                const int sh = meta & 31, n = meta >> 5;
                unsigned zeros = 0;
                unsigned short *hs = reinterpret_cast<unsigned short *>(stage + (live ? r : 0) * A.slot_bytes + off_h);
                if (live) {
                    const unsigned *raw = reinterpret_cast<const unsigned *>(stage + r * A.slot_bytes + off_u);
                    const unsigned w = __builtin_amdgcn_alignbit(raw[j + 1], raw[j], (unsigned)sh);
                    const int left = n - 32 * j;
                    const unsigned mask = left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u;
                    zeros = ~w & mask;
                }
                const int nz = __builtin_popcount(zeros);
                const int incl = sl_wave_iscan(nz);
                int rank;
                if (uwp <= 64) {
                    const int seg = lane & ~(uwp - 1);                 // first lane of this worker's words
                    const int before = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
                    rank = incl - nz - (seg > 0 ? before : 0);
                } else {
                    if ((s0 & (uwp - 1)) == 0) carry = 0;              // a new worker starts with this pass
                    rank = carry + incl - nz;
                    carry += __builtin_amdgcn_readlane(incl, 63);
                }
                // The word's zero bits, two from each end per turn of the loop (four independent chains; the
                // length of this loop - the word with the most zeros - is on the chunk's critical path).  Entry
                // `rank` is the word's lowest zero, entry `rank + nz - 1` its highest; when one zero is left both
                // ends write the same value to the same place.  A vector with more than k zeros (malformed)
                // takes the loop that checks every store.
                if (__builtin_amdgcn_ballot_w64(rank + nz > k) == 0) {
                    // (byte addresses and values as plain integers the compiler may not take apart again:
                    // it would rebuild each of them from j and rank in every turn)
                    unsigned lo = (unsigned)(size_t)(hs + rank), hi = (unsigned)(size_t)(hs + rank + nz - 1);
                    int vlo = 32 * j - rank, vhi = 32 * j + 31 - (rank + nz - 1);
                    asm volatile("" : "+v"(lo), "+v"(hi), "+v"(vlo), "+v"(vhi));
                    auto put = [](unsigned at, int v) {
                        *reinterpret_cast<unsigned short __attribute__((address_space(3))) *>(at) = (unsigned short)v;
                    };
                    while (zeros) {
                        const int pl = __builtin_ctz(zeros), ch = __builtin_clz(zeros);
                        put(lo, vlo + pl);
                        put(hi, vhi - ch);
                        zeros &= (zeros - 1u) & ~(0x80000000u >> ch);
                        if (zeros) {
                            const int pl2 = __builtin_ctz(zeros), ch2 = __builtin_clz(zeros);
                            put(lo + 2, vlo - 1 + pl2);
                            put(hi - 2, vhi + 1 - ch2);
                            zeros &= (zeros - 1u) & ~(0x80000000u >> ch2);
                        }
                        lo += 4, hi -= 4, vlo -= 2, vhi += 2;
                    }
                } else {
                    int rk = rank;
                    while (zeros) {
                        const int pl = __builtin_ctz(zeros);
                        if (rk < k) hs[rk] = (unsigned short)(32 * j + pl - rk);
                        zeros &= zeros - 1u;
                        ++rk;
                    }
                }
            }
            sl_wave_sync();
        }
        // ---- step 4 with lists: remainders, their prefix sums, the indices
        {
            const int L = k / A.E, E = A.E;             // lanes per worker, entries per lane
            const int wpp = L <= 64 ? 64 / L : 1;       // workers per pass
            const int ppw = (L + 63) >> 6;              // passes per worker (1 unless L > 64)
            const unsigned fmask = (1u << b) - 1u;
            for (int rb = 0; rb < nb; rb += wpp) {
                int carry = 0;
                for (int ps = 0; ps < ppw; ++ps) {
                    // (lane / L; the multiplier does not exist for L = 1)
                    const int rl = L == 1 ? lane : L <= 64 ? (int)__umulhi((unsigned)lane, A.magic_l) : 0;
                    const int o = L <= 64 ? lane - rl * L : 64 * ps + lane;
                    const int r = rb + rl;
                    const bool live = rl < wpp && r < nb && o < L;
                    unsigned char *slot = stage + (live ? r : 0) * A.slot_bytes;
                    int pre[8];
                    int total = 0;
                    if (live) {
                        // (the two words behind the one that holds the first field are read whether or not
                        // the fields reach them: they lie inside the worker's slot)
                        const unsigned *rem = reinterpret_cast<const unsigned *>(slot + 4 * hdrw);
                        const int bit = o * E * b, wi = bit >> 5;
                        const unsigned w0 = rem[wi], w1 = rem[wi + 1], w2 = rem[wi + 2];
                        const unsigned lo = __builtin_amdgcn_alignbit(w1, w0, (unsigned)(bit & 31));
                        const unsigned hi = __builtin_amdgcn_alignbit(w2, w1, (unsigned)(bit & 31));
                        const unsigned long long win = ((unsigned long long)hi << 32) | lo;
                        int t = 0;
                        if (b <= 8) {
                            // four fields fit a word: entries 0..3 from the window's low word, 4..7 from
                            // the word that starts at field 4
                            const unsigned lo4 = (unsigned)(win >> (4 * b));
#pragma unroll
                            for (int e = 0; e < 4; ++e) pre[e] = (t += (int)__builtin_amdgcn_ubfe(lo, (unsigned)(e * b), (unsigned)b));
#pragma unroll
                            for (int e = 0; e < 4; ++e) pre[4 + e] = (t += (int)__builtin_amdgcn_ubfe(lo4, (unsigned)(e * b), (unsigned)b));
                        } else {
#pragma unroll
                            for (int e = 0; e < 8; ++e) pre[e] = (t += (int)((unsigned)(win >> (e * b)) & fmask));
                        }
                        total = E == 8 ? pre[7] : pre[3];
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) pre[e] = 0;
                    }
                    const int incl = sl_wave_iscan(total);
                    int excl;
                    if (L <= 64) {
                        const int seg = rl * L;
                        const int before = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
                        excl = incl - total - (seg > 0 ? before : 0);
                    } else {
                        excl = carry + incl - total;
                        carry += __builtin_amdgcn_readlane(incl, 63);
                    }
                    if (live) {
                        unsigned short *hs = reinterpret_cast<unsigned short *>(slot + off_h) + o * E;
                        unsigned short hv[8];
                        if (E == 8) {
                            const uint4 q4 = *reinterpret_cast<const uint4 *>(hs);
                            hv[0] = (unsigned short)q4.x, hv[1] = (unsigned short)(q4.x >> 16);
                            hv[2] = (unsigned short)q4.y, hv[3] = (unsigned short)(q4.y >> 16);
                            hv[4] = (unsigned short)q4.z, hv[5] = (unsigned short)(q4.z >> 16);
                            hv[6] = (unsigned short)q4.w, hv[7] = (unsigned short)(q4.w >> 16);
                        } else {
                            const uint2 q2 = *reinterpret_cast<const uint2 *>(hs);
                            hv[0] = (unsigned short)q2.x, hv[1] = (unsigned short)(q2.x >> 16);
                            hv[2] = (unsigned short)q2.y, hv[3] = (unsigned short)(q2.y >> 16);
                            hv[4] = hv[5] = hv[6] = hv[7] = 0;
                        }
                        // two indices per word, cut to 12 bits each after packing: a malformed payload stays
                        // inside the chunk (a valid one never reaches bit 12)
                        unsigned pw[4];
                        const unsigned base = (unsigned)(o * E) + (unsigned)excl;
#pragma unroll
                        for (int e = 0; e < 8; e += 2) {
                            const unsigned i0 = base + (unsigned)e + ((unsigned)hv[e] << b) + (unsigned)pre[e];
                            const unsigned i1 = base + (unsigned)(e + 1) + ((unsigned)hv[e + 1] << b) + (unsigned)pre[e + 1];
                            pw[e >> 1] = (i0 | (i1 << 16)) & 0x0FFF0FFFu;
                        }
                        if (E == 8)
                            *reinterpret_cast<uint4 *>(hs) = make_uint4(pw[0], pw[1], pw[2], pw[3]);
                        else
                            *reinterpret_cast<uint2 *>(hs) = make_uint2(pw[0], pw[1]);
                    }
                }
            }
            sl_wave_sync();
        }
        } else {
        // ---- step 3: where every eighth zero of the vectors lies
        {
            const int slots = nb << A.uwp_log2;
            int carry = 0;
            for (int s0 = 0; s0 < slots; s0 += 64) {
                const int slot = s0 + lane;
                const int r = slot >> A.uwp_log2, j = slot & (uwp - 1);
                // (a lane without a word reads the first one of some worker and finds no zeros in it)
                const int rr = r < nb ? r : 0, jj = j < G.ua ? j : 0;
                const int meta = sl_lane_read(v_meta, r0 + rr);
                const int sh = meta & 31;
                unsigned char *base = stage + rr * A.slot_bytes;
                const unsigned *raw = reinterpret_cast<const unsigned *>(base + off_u) + jj;
                const int left = r < nb && j < G.ua ? (meta >> 5) - 32 * j : 0;
                const unsigned mask = left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u;
                const unsigned zeros = ~__builtin_amdgcn_alignbit(raw[1], raw[0], (unsigned)sh) & mask;
                const int nz = __builtin_popcount(zeros);
                const int incl = sl_wave_iscan(nz);
                int rank;
                if (uwp <= 64) {
                    const int seg = lane & ~(uwp - 1);                 // first lane of this worker's words
                    const int before = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
                    rank = incl - nz - (seg > 0 ? before : 0);
                } else {
                    if ((s0 & (uwp - 1)) == 0) carry = 0;              // a new worker starts with this pass
                    rank = carry + incl - nz;
                    carry += __builtin_amdgcn_readlane(incl, 63);
                }
                // zeros rank .. rank + nz - 1 of the vector lie in this word: each of its four bytes holds at
                // most one whose number is a multiple of eight (a vector with more than k zeros is malformed:
                // the rest is left out)
                unsigned short *table = reinterpret_cast<unsigned short *>(base + off_t);
                int from = rank;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int to = q < 3 ? rank + __builtin_popcount(zeros & ((1u << (8 * (q + 1))) - 1u)) : rank + nz;
                    const int m = (from + 7) & ~7;
                    // (no such zero: entry L of the table takes the write, nobody reads it)
                    table[m < to && m < k ? m >> 3 : L] = (unsigned short)(((4 * j + q) << 3) | (m - from));
                    from = to;
                }
            }
            sl_wave_sync();
        }
        // ---- steps 4 and 5
        {
            const int wpp = L <= 64 ? 64 / L : 1;       // workers per pass
            const int ppw = (L + 63) >> 6;              // passes per worker (1 unless L > 64)
            const unsigned fmask = (1u << b) - 1u;
            if constexpr (TWO_BIT) {
                // the values of two consecutive codes, by their four bits
                for (int q = lane; q < 16 * nb; q += 64) {
                    unsigned char *slot = stage + (q >> 4) * A.slot_bytes;
                    const float *lutp = reinterpret_cast<const float *>(slot);
                    reinterpret_cast<float2 *>(slot + off_q)[q & 15] = make_float2(lutp[q & 3], lutp[(q >> 2) & 3]);
                }
                sl_wave_sync();
            }
            for (int rb = 0; rb < nb; rb += wpp) {
                int carry = 0;
                for (int ps = 0; ps < ppw; ++ps) {
                    // (lane / L; the multiplier does not exist for L = 1)
                    const int rl = L == 1 ? lane : L <= 64 ? (int)__umulhi((unsigned)lane, A.magic_l) : 0;
                    const int o = L <= 64 ? lane - rl * L : 64 * ps + lane;
                    const int r = rb + rl;
                    const bool live = rl < wpp && r < nb && o < L;
                    unsigned char *slot = stage + (live ? r : 0) * A.slot_bytes;
                    const int meta = sl_lane_read(v_meta, live ? r0 + r : 0);
                    const int oo = live ? o : 0;         // (a lane without entries decodes some worker's first ones)
                    int pre[8];                          // r_0 + ... + r_e, plus e - (e << b): what entry e's index holds
                                                         // besides the lane's part and its zero's place
                    int total;
                    {
                        // (the two words behind the one that holds the first field are read whether or not
                        // the fields reach them: they lie inside the worker's slot)
                        const unsigned *rem = reinterpret_cast<const unsigned *>(slot + 4 * hdrw);
                        const int bit = oo * 8 * b, wi = bit >> 5;
                        const unsigned w0 = rem[wi], w1 = rem[wi + 1], w2 = rem[wi + 2];
                        const unsigned lo = __builtin_amdgcn_alignbit(w1, w0, (unsigned)(bit & 31));
                        const unsigned hi = __builtin_amdgcn_alignbit(w2, w1, (unsigned)(bit & 31));
                        // entries 0..2 from the window's low word, 3 from the word that starts at its field (b is
                        // at most 9), 4..7 from the word that starts at field 4 (b = 9 is k = 4: no such entries)
                        const unsigned lo3 = __builtin_amdgcn_alignbit(hi, lo, (unsigned)(3 * b));
                        const unsigned lo4 = (unsigned)((((unsigned long long)hi << 32) | lo) >> (4 * b));
                        const int step = 1 - (1 << b);
                        int t = 0;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const unsigned f = e < 3 ? __builtin_amdgcn_ubfe(lo, (unsigned)(e * b), (unsigned)b)
                                               : e == 3 ? lo3 & fmask : __builtin_amdgcn_ubfe(lo4, (unsigned)((e - 4) * b), (unsigned)b);
                            t = e ? t + (int)f + step : (int)f;
                            pre[e] = t;
                        }
                        total = t - 7 * step;
                    }
                    const int incl = sl_wave_iscan(total);
                    int excl;
                    if (L <= 64) {
                        const int seg = rl * L;
                        const int before = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
                        excl = incl - total - (seg > 0 ? before : 0);
                    } else {
                        excl = carry + incl - total;
                        carry += __builtin_amdgcn_readlane(incl, 63);
                    }
                    // the eight zeros: the first from the table, the others in the 64 bits behind it (20 of them on
                    // average, whatever k: the Rice parameter follows it; 32 would not do for one lane in a hundred)
                    const unsigned *raw = reinterpret_cast<const unsigned *>(slot + off_u);
                    int p[8];                            // places of the zeros, from the first one's on
                    int start = 0;                       // place of the first in the vector
                    unsigned z, zh;
                    {
                        const unsigned note = reinterpret_cast<const unsigned short *>(slot + off_t)[oo];
                        const int byte = min((int)(note >> 3), 4 * G.ua - 1);      // (beyond: a vector with too few zeros)
                        const int at = (meta & 31) + 8 * byte, wi = at >> 5;
                        const unsigned w0 = raw[wi], w1 = raw[wi + 1], w2 = raw[wi + 2];
                        const unsigned lo = ~__builtin_amdgcn_alignbit(w1, w0, (unsigned)(at & 31));
                        const unsigned hi = ~__builtin_amdgcn_alignbit(w2, w1, (unsigned)(at & 31));
                        const unsigned skip = (unsigned)sl_place_in_byte(lo & 0xFFu, (int)(note & 7u));
                        start = 8 * byte + (int)skip;
                        z = __builtin_amdgcn_alignbit(hi, lo, skip);
                        zh = hi >> skip;                 // (57 bits at least)
                    }
                    const int want = min(8, k - 8 * o);
                    if (__builtin_amdgcn_ballot_w64(live && __builtin_popcount(z) + __builtin_popcount(zh) < want) == 0) {
                        p[0] = 0;
                        int off = 0;
#pragma unroll
                        for (int e = 1; e < 8; ++e) {
                            if (e == 4) z = want == 8 && live ? z : 0x1Fu;       // (the last four of a lane that has four: any)
                            if (e == 1) z = live ? z : 0x1Fu;
                            z &= z - 1u;
                            const bool next = z == 0u;                   // on to the upper word (once at most)
                            z = next ? zh : z;
                            off = next ? 32 : off;
                            p[e] = __builtin_ctz(z) + off;
                        }
                    } else {
                        // a lane's eight zeros reach further (clustered supports): word by word
                        int q = start;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            for (int turn = 0; turn < 130; ++turn) {     // (at most 128 words: a malformed vector ends the search)
                                const int at = (meta & 31) + q, wi = min(at >> 5, G.ua);
                                const unsigned w = ~__builtin_amdgcn_alignbit(raw[wi + 1], raw[wi], (unsigned)(at & 31));
                                if (w != 0u) {
                                    q += __builtin_ctz(w);
                                    break;
                                }
                                q += 32;
                            }
                            p[e] = q - start;
                            ++q;
                        }
                    }
                    const int base = excl + 8 * oo + ((start - 8 * oo) << b);
                    // index of entry e, cut to 12 bits: a malformed payload stays inside the chunk (a valid one
                    // never reaches bit 12)
                    unsigned idx[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) idx[e] = (unsigned)(base + (pre[e] + (p[e] << b))) & 0xFFFu;
                    // ---- step 5: these lanes add their entries, worker after worker.  The positions of
                    // one record are distinct: the reads, then the writes, are issued together.
                    float v[8];
                    const unsigned char *vals = slot + 4 * hdrw + G.rem_bytes;
                    if constexpr (TWO_BIT) {
                        const unsigned cw = reinterpret_cast<const unsigned short *>(vals)[oo];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float2 q2 = reinterpret_cast<const float2 *>(slot + off_q)[(cw >> (4 * e)) & 15u];
                            v[2 * e] = q2.x, v[2 * e + 1] = q2.y;
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = e < want ? value_at(slot, min(8 * o + e, k - 1)) : 0.f;
                    }
                    for (int w = 0; w < wpp; ++w) {
                        if (live && rl == w) {
                            float t[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e) t[e] = acc[idx[e]];
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (e < 4 || want == 8) acc[idx[e]] = t[e] + v[e];
                        }
                        sl_wave_sync();   // worker r is complete before worker r+1 is added
                    }
                }
            }
            sl_wave_sync();
        }
        }
        if constexpr (LISTS) {
            // ---- step 5 with lists: the entries of up to eight workers are fetched first (independent LDS
            // reads), then added worker by worker: the additions form a chain of LDS round trips
            for (int rb = 0; rb < nb; rb += 8) {
                unsigned jj[8][2];
                float qq[8][2];
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2) {
                        const int m = lane + 64 * s2;
                        jj[u][s2] = 0xFFFFu;
                        qq[u][s2] = 0.0f;
                        if (rb + u < nb && m < k) {
                            const unsigned char *slot = stage + (rb + u) * A.slot_bytes;
                            jj[u][s2] = reinterpret_cast<const unsigned short *>(slot + off_h)[m];
                            qq[u][s2] = value_at(slot, m);
                        }
                    }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (rb + u < nb) {
#pragma unroll
                        for (int s2 = 0; s2 < 2; ++s2)
                            if (jj[u][s2] != 0xFFFFu) acc_add(acc, jj[u][s2], qq[u][s2]);
                        sl_wave_sync();   // worker r is complete before worker r+1 is added
                    }
                }
            }
        }
    };
    do_batch(0, true);
    for (int r0 = A.batch; r0 < A.R; r0 += A.batch) do_batch(r0, false);

    if (full) {
        const unsigned o0 = 4u * (lr * stride + lc), step = 16u * stride;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float4 a = reinterpret_cast<const float4 *>(acc)[i * 64 + lane];
            sl_f4 g;
            g.x = a.x * A.inv_R, g.y = a.y * A.inv_R, g.z = a.z * A.inv_R, g.w = a.w * A.inv_R;
            if constexpr (NESTEROV) {
                sl_f4 m = mo[i];
                m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
                m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
                sl_store_stream_at<KEEP>(mc, i * step, o0, m);
                g.x = fmaf(A.mu, m.x, g.x), g.y = fmaf(A.mu, m.y, g.y);
                g.z = fmaf(A.mu, m.z, g.z), g.w = fmaf(A.mu, m.w, g.w);
            }
            sl_f4 v = th[i];
            v.x = fmaf(A.neg_lr, g.x, v.x);
            v.y = fmaf(A.neg_lr, g.y, v.y);
            v.z = fmaf(A.neg_lr, g.z, v.z);
            v.w = fmaf(A.neg_lr, g.w, v.w);
            sl_store_stream_at<KEEP>(tc, i * step, o0, v);
        }
    } else {
        const int rows = d.rows, cols = d.cols, last_cols = d.last_cols;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = 4 * i + lr;
            const int lim = row < rows - 1 ? cols : (row == rows - 1 ? last_cols : 0);
            const unsigned o0 = row * stride + lc;
            const float4 a = reinterpret_cast<const float4 *>(acc)[i * 64 + lane];
            sl_f4 g;
            g.x = a.x * A.inv_R, g.y = a.y * A.inv_R, g.z = a.z * A.inv_R, g.w = a.w * A.inv_R;
            sl_f4 m = sl_f4{0.f, 0.f, 0.f, 0.f};
            if constexpr (NESTEROV) {
                m = mo[i];
                m.x = fmaf(A.mu, m.x, g.x), m.y = fmaf(A.mu, m.y, g.y);
                m.z = fmaf(A.mu, m.z, g.z), m.w = fmaf(A.mu, m.w, g.w);
                g.x = fmaf(A.mu, m.x, g.x), g.y = fmaf(A.mu, m.y, g.y);
                g.z = fmaf(A.mu, m.z, g.z), g.w = fmaf(A.mu, m.w, g.w);
            }
            sl_f4 v = th[i];
            v.x = fmaf(A.neg_lr, g.x, v.x), v.y = fmaf(A.neg_lr, g.y, v.y);
            v.z = fmaf(A.neg_lr, g.z, v.z), v.w = fmaf(A.neg_lr, g.w, v.w);
            if (lc + 3 < lim) {
                if constexpr (NESTEROV) sl_store_stream_u<KEEP>(mc + o0, m);
                sl_store_stream_u<KEEP>(tc + o0, v);
            } else {
#pragma unroll
                for (int cc = 0; cc < 4; ++cc)
                    if (lc + cc < lim) {
                        if constexpr (NESTEROV) mc[o0 + cc] = m[cc];
                        tc[o0 + cc] = v[cc];
                    }
            }
        }
    }
}

int pow2_log2_at_least(int n)
{
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

}  // namespace

// mom != null: with the global momentum
int slk_apply_coded(const sl_plan *p, float *theta, float *mom, float mu, const void *const *payloads, const size_t *bytes,
                    int R, float lr, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    if (const int waves = sl_apply_waves(p, R, true, mom != nullptr); waves > 1) return slk_apply_group(p, theta, mom, mu, payloads, bytes, R, lr, waves, st);
    CodedApplyArgs A;
    A.G = p->cg;
    A.desc = p->d_desc;
    A.cdesc = p->d_cdesc;
    A.theta = theta;
    A.mom = mom;
    A.mu = mu;
    A.neg_lr = -lr;
    A.inv_R = 1.0f / (float)R;
    A.R = R;
    const SlCodedGeom &G = p->cg;
    A.fwp = (G.hdr + G.cfix) >> 2;
    const bool few = (long long)R * G.k < SL_CAPPLY_LISTS_BELOW || (G.k <= 16 && G.bits == 2);
    const bool lists = G.k <= 128 && few;
    A.E = (G.k & 7) ? 4 : 8;
    const int L = lists ? G.k / A.E : (G.k + 7) / 8;
    auto up16 = [](int v) { return (v + 15) & ~15; };
    A.off_t = A.off_q = A.off_h = up16(4 * A.fwp + 4 * (G.ua + 1));
    if (lists) {
        A.slot_bytes = up16(A.off_h + 2 * G.k);
    } else {
        A.off_q = up16(A.off_t + 2 * (L + 1));
        A.slot_bytes = A.off_q + (G.bits == 2 ? 128 : 0);
    }
    A.uwp_log2 = pow2_log2_at_least(G.ua);
    int batch = SL_CAPPLY_STAGE / A.slot_bytes;
    // (a whole number of passes of step 3, where a pass holds several workers' vectors)
    const int per_pass = A.uwp_log2 < 6 ? 64 >> A.uwp_log2 : 1;
    if (batch > per_pass) batch -= batch % per_pass;
    // Without lists the batch follows two things more (24,000 chunks each).  `cap`: no more workers than have all
    // their words fetched ahead (SL_CAPPLY_PFF and _PFU words by each of a worker's 64 / batch lanes; below two
    // workers per batch that cannot be had) - but not where that leaves more than a third of step 4's lanes without
    // a worker, i.e. with wide tables or values at small k (k = 64: at 4 bits, R = 64 660 us with the cap, 468
    // without, 504 with lists; at 32 bits, R = 16 306, 219 and 238).  And workers left over after whole passes of
    // step 4 cost a pass: they wait for the next batch where that makes passes and batches fewer (k = 72, R = 40:
    // 380 us with eight at a time, 310 with seven at 1 bit, 300 and 266 at 2).
    if (!lists) {
        int lanes = 1;
        while (lanes < 32 && (SL_CAPPLY_PFF * lanes < A.fwp || SL_CAPPLY_PFU * lanes < G.ua + 1)) lanes <<= 1;
        const int cap = 64 / lanes, wpp = L <= 64 ? 64 / L : 1;
        if (batch > cap && 2 * wpp <= 3 * cap) batch = cap;
        auto turns = [&](int b) { return R / b * (1 + (b + wpp - 1) / wpp) + (R % b ? 1 + (R % b + wpp - 1) / wpp : 0); };
        const int whole = batch - batch % wpp;
        if (batch > wpp && turns(whole) < turns(batch)) batch = whole;
    }
    if (batch < 1) batch = 1;
    if (batch > R) batch = R;
    A.batch = batch;
    A.lpw_log2 = 6 - pow2_log2_at_least(batch);
    A.magic_l = L > 1 ? (unsigned)(0x100000000ull / (unsigned)L + 1) : 0u;
    A.n_chunks = p->n_chunks;
    for (int r = 0; r < SL_MAX_WORKERS; ++r) {
        A.payload[r] = r < R ? static_cast<const unsigned char *>(payloads[r]) : nullptr;
        const size_t sec = r < R && bytes[r] > (size_t)G.section ? (bytes[r] - (size_t)G.section) >> 2 : 0;
        A.sec_words[r] = sec > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned)sec;
    }
    A.lds_per_wave = (int)((SL_CHUNK * sizeof(float) + (size_t)batch * A.slot_bytes + 15) & ~(size_t)15);
    int wpb = sl_chunks_per_group(p);
    while (wpb > 1 && (size_t)A.lds_per_wave * wpb > (size_t)p->max_lds) wpb >>= 1;
    const size_t lds = (size_t)A.lds_per_wave * wpb;
    typedef void (*kernel_t)(CodedApplyArgs);
#define SL_CAPPLY_KINDS(KEEP)                                                                             \
    {{{k_apply_coded<false, false, false, KEEP>, k_apply_coded<false, true, false, KEEP>},                   \
      {k_apply_coded<false, false, true, KEEP>, k_apply_coded<false, true, true, KEEP>}},                    \
     {{k_apply_coded<true, false, false, KEEP>, k_apply_coded<true, true, false, KEEP>},                     \
      {k_apply_coded<true, false, true, KEEP>, k_apply_coded<true, true, true, KEEP>}}}
    static const kernel_t table[2][2][2][2] = {SL_CAPPLY_KINDS(false), SL_CAPPLY_KINDS(true)};
#undef SL_CAPPLY_KINDS
    const kernel_t fn = table[sl_rows_unaligned(p, sl_apply_kept_from(p, mom != nullptr)) ? 1 : 0][p->bits == 2 ? 1 : 0][lists ? 1 : 0][mom ? 1 : 0];
    if (lds > 65536) {
        hipError_t aerr = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (aerr != hipSuccess) {
            sl_note_hip_error(aerr);
            return SL_ERR_HIP;
        }
    }
    const dim3 grid((unsigned)((p->n_chunks + wpb - 1) / wpb)), block(64 * wpb);
    A.order = sl_order(p, grid.x);
    hipLaunchKernelGGL(fn, grid, block, lds, st, A);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}
