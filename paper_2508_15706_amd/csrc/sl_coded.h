// The coded wire format ("SLRICE02") on the device: what a wavefront needs to write and to
// read one chunk of it.  (The paper's appendix "Compression of indices in Top-k" names its index
// coder - Rice coding - and the rates it reaches, not the format; this one is the library's.)
//
// A chunk's ascending index list idx_0 < ... < idx_(k-1) is coded as gaps g_0 = idx_0,
// g_i = idx_i - idx_(i-1) - 1, each split by the Rice parameter b = floor(log2(2839 / k)) into a
// quotient q_i = g_i >> b and a remainder of b bits.  The two halves are stored apart:
//   * remainders: k fields of b bits (LSB first) at the start of the chunk's FIXED RECORD, padded
//     to 4 bytes, followed there by the k value fields as they stand in a plain record;
//   * quotients: one BIT VECTOR per chunk, the unary codes back to back - q_i one-bits, then a
//     zero bit - so entry i ends at the vector's i-th zero bit, at position
//     z_i = i + q_0 + ... + q_i, and the vector has k + Q bits, Q = sum of the q_i.
// So idx_i = i + ((z_i - i) << b) + r_0 + ... + r_i: every entry follows from the position of its
// own zero bit and a prefix sum of remainders, and a wave decodes a chunk's entries side by side.
//
// Buffer: "SLRICE02", uint64 total bytes; per tensor a 16-byte aligned block [table header]
// [directory][fixed records] at offsets that follow from the tensor list alone; then the
// quotient section: per group of 16 consecutive chunks of a tensor one run of their bit vectors,
// back to back, zero-padded to a 4-byte word.  A directory entry = uint32 offset of the group's
// run (in words from the start of the section) + the 16 chunks' Q (1 byte each while the
// largest possible Q is below 256, else 2).
#pragma once
#include "sl_device.h"
#include "sl_internal.h"

typedef unsigned __attribute__((address_space(3))) *sl_lds_words;

// LDS word |= v, &= v (the lanes of a wave may hit one word together)
SL_DEV void sl_lds_or(unsigned *p, unsigned v)
{
    __hip_atomic_fetch_or((sl_lds_words)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
SL_DEV void sl_lds_and(unsigned *p, unsigned v)
{
    __hip_atomic_fetch_and((sl_lds_words)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Lane i reads lane i - S of its row of 16 lanes, 0 where there is none (S = 1, 2, 4, 8).
template <int S>
SL_DEV int sl_row_shr(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x110 + S, 0xF, 0xF, true); }

// Inclusive prefix sum over the 64 lanes (all active): four steps inside each row of 16 lanes,
// then the totals of the rows below are added (read from the rows' last lanes).
SL_DEV int sl_wave_iscan(int v)
{
    v += sl_row_shr<1>(v);
    v += sl_row_shr<2>(v);
    v += sl_row_shr<4>(v);
    v += sl_row_shr<8>(v);
    const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31),
              t2 = __builtin_amdgcn_readlane(v, 47);
    const int row = (int)(threadIdx.x & 63) >> 4;
    return v + (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
}

// Place of the set bit of byte x that has n set bits below it, by halving.
SL_DEV int sl_place_in_byte(unsigned x, int n)
{
    const int c4 = __builtin_popcount(x & 15u);
    const bool up4 = n >= c4;
    n -= up4 ? c4 : 0;
    x = up4 ? x >> 4 : x;
    const int c2 = __builtin_popcount(x & 3u);
    const bool up2 = n >= c2;
    n -= up2 ? c2 : 0;
    x = up2 ? x >> 2 : x;
    return (up4 ? 4 : 0) + (up2 ? 2 : 0) + (n >= (int)(x & 1u) ? 1 : 0);
}

// Value of lane `src` (any lane; all lanes call this together).
SL_DEV int sl_lane_read(int v, int src) { return __builtin_amdgcn_ds_bpermute(4 * src, v); }

// ---------------------------------------------------------------------------------- writer
// Codes the k ascending indices idx[0..k) (LDS) of one chunk.  uv (LDS, G.ua words) receives
// the bit vector, bits beyond its k + Q left as ones; rw (LDS, G.rem_bytes / 4 words) the
// remainder fields, padding zero.  Returns Q (uniform).  Called by all 64 lanes; the caller
// orders its own earlier LDS accesses before the call and reads uv / rw after it.
// Indices that are not strictly ascending (a malformed plain record - a compressor never
// produces one) are coded as gap 0, and a vector that would outgrow k + qmax bits is cut there.
// (The _filled form: uv holds ones and rw zeros already.)
SL_DEV int sl_coded_emit_filled(const SlCodedGeom &G, int lane, const unsigned short *idx, unsigned *uv, unsigned *rw)
{
    const int k = G.k, b = G.b;
    const int limit = k + G.qmax;            // bits of the longest vector
    // A lane owns ceil(k / 64) CONSECUTIVE entries: one wave scan for the whole chunk, and the lanes of one
    // store instruction are that many entries apart, so that at high densities they land in different
    // words of the vector (64 neighbouring entries would share two or three words, and the LDS atomics on
    // one word take turns).
    const int E = (k + 63) >> 6, m0 = lane * E, m1 = min(k, m0 + E);
    const int first_prev = (m0 > 0 && m0 < k) ? (int)idx[m0 - 1] : -1;
    int prev = first_prev, qsum = 0;
    for (int m = m0; m < m1; ++m) {
        const int cur = (int)idx[m];
        qsum += max(cur - prev - 1, 0) >> b;
        prev = cur;
    }
    const int incl = sl_wave_iscan(qsum);
    int qrun = incl - qsum;                  // quotients of all entries before the lane's first
    prev = first_prev;
    for (int m = m0; m < m1; ++m) {
        const int cur = (int)idx[m];
        const int gap = max(cur - prev - 1, 0);
        prev = cur;
        qrun += gap >> b;
        const unsigned r = (unsigned)gap & ((1u << b) - 1u);
        const int z = qrun + m;              // position of entry m's zero bit
        if (z < limit) sl_lds_and(&uv[z >> 5], ~(1u << (z & 31)));
        if (b) {
            const int bit = m * b, sh = bit & 31;
            sl_lds_or(&rw[bit >> 5], r << sh);
            if (sh + b > 32) sl_lds_or(&rw[(bit >> 5) + 1], r >> (32 - sh));
        }
    }
    const int carry = __builtin_amdgcn_readlane(incl, 63);
    sl_wave_sync();
    return min(carry, G.qmax);
}
SL_DEV int sl_coded_emit(const SlCodedGeom &G, int lane, const unsigned short *idx, unsigned *uv, unsigned *rw)
{
    for (int w = lane; w < G.ua; w += 64) uv[w] = 0xFFFFFFFFu;
    for (int w = lane; w < (G.rem_bytes >> 2); w += 64) rw[w] = 0u;
    sl_wave_sync();
    return sl_coded_emit_filled(G, lane, idx, uv, rw);
}

// ---------------------------------------------------------------------------------- reader
// One directory entry (16-byte loads need only 4-byte alignment): for the chunk at position
// `pos` of its group, the word offset of the group's run, the bit at which the chunk's vector
// starts inside the run and the vector's length.  Quotient sums are clamped to qmax, so that
// a malformed entry still describes a vector of at most k + qmax bits that starts below
// 15 (k + qmax).
struct SlVecPlace {
    unsigned run_word;      // the group's run, in words from the start of the quotient section
    int start_bit;          // first bit of the chunk's vector inside the run
    int nbits;              // k + Q
};

// words and halfwords of records, which start at any byte where their size is odd
typedef unsigned __attribute__((aligned(1))) u32_any;
typedef unsigned short __attribute__((aligned(1))) u16_any;

// pointers into global memory, for addresses that are put together from integers (a generic
// pointer would turn every access into a flat load that LDS waits have to sit out)
typedef const unsigned char __attribute__((address_space(1))) *sl_gbytes;
typedef const unsigned __attribute__((address_space(1))) *sl_gwords;
typedef unsigned sl_u4u __attribute__((ext_vector_type(4), aligned(4)));
typedef const sl_u4u __attribute__((address_space(1))) *sl_gu4;

// The words of a directory entry as loaded (the loads are issued here; nothing waits for them
// until sl_coded_dir_parse reads the words).
struct SlDirWords {
    unsigned run_word;
    sl_u4u lo, hi;          // the 16 quotient sums: 16 bytes, or 32 when they are two bytes each
};

SL_DEV SlDirWords sl_coded_dir_load(const SlCodedGeom &G, sl_gbytes entry)
{
    SlDirWords W;
    const sl_gwords e = reinterpret_cast<sl_gwords>(entry);
    W.run_word = e[0];
    W.lo = *reinterpret_cast<sl_gu4>(e + 1);
    W.hi = sl_u4u{0u, 0u, 0u, 0u};
    if (G.qf == 2) W.hi = *reinterpret_cast<sl_gu4>(e + 5);
    return W;
}

// Field j (0..15) of a directory entry's quotient sums, j a compile-time constant.
template <int J>
SL_DEV unsigned sl_dir_field(int qf, sl_u4u lo, sl_u4u hi)
{
    if (qf == 2) {
        const sl_u4u v = J < 8 ? lo : hi;
        const unsigned w = ((J >> 1) & 3) == 0 ? v.x : ((J >> 1) & 3) == 1 ? v.y : ((J >> 1) & 3) == 2 ? v.z : v.w;
        return (w >> (16 * (J & 1))) & 0xFFFFu;
    }
    const unsigned w = (J >> 2) == 0 ? lo.x : (J >> 2) == 1 ? lo.y : (J >> 2) == 2 ? lo.z : lo.w;
    return (w >> (8 * (J & 3))) & 0xFFu;
}

template <int J>
SL_DEV void sl_dir_sum(int qf, int qmax, sl_u4u lo, sl_u4u hi, int pos, int &before, int &own)
{
    if constexpr (J < SL_RICE_GROUP) {
        const int qc = min((int)sl_dir_field<J>(qf, lo, hi), qmax);
        before += J < pos ? qc : 0;
        own = J == pos ? qc : own;
        sl_dir_sum<J + 1>(qf, qmax, lo, hi, pos, before, own);
    }
}

SL_DEV SlVecPlace sl_coded_dir_parse(const SlCodedGeom &G, unsigned run_word, sl_u4u lo, sl_u4u hi, int pos)
{
    SlVecPlace P;
    P.run_word = run_word;
    int before = 0, own = 0;
    sl_dir_sum<0>(G.qf, G.qmax, lo, hi, pos, before, own);
    P.start_bit = pos * G.k + before;
    P.nbits = G.k + own;
    return P;
}

SL_DEV SlVecPlace sl_coded_dir_entry(const SlCodedGeom &G, sl_gbytes entry, int pos)
{
    const SlDirWords W = sl_coded_dir_load(G, entry);
    return sl_coded_dir_parse(G, W.run_word, W.lo, W.hi, pos);
}

// ---------------------------------------------------------------------------------- placement
// The variable-length part of a buffer.  The writers leave each chunk's bit vector and quotient sum
// in the workspace; then, each step reading what the one before wrote:
//   sl_coded_scan_block    one workgroup per SL_SCAN_BLOCK groups: words of each group's run and their exclusive prefix inside
//                          the block, whatever tensors it spans (by tensor, a workgroup had 8192 groups of a large matrix to go
//                          through alone while tensors of one group had one each);
//   sl_coded_place         one wave per group: the words of the blocks before its own summed up, the 16 vectors
//                          shifted into one run, the run and the directory entry written; the last one writes the buffer header.
// The compressor runs them as extra workgroups of the quantizer's launches (sl_quant.hip), on lists of
// many tensors and in the transcoder they are launches of their own (sl_coded.hip).
struct SlCodedArgs {
    SlCodedGeom G;
    const SlTensorDev *tensors;
    const SlGroup *groups;
    long long n_groups;
    int ua_log2;                    // log2 of a power of two >= G.ua
    const unsigned *uvec;           // [n_chunks][G.ua] bit vectors as the writers left them
    const unsigned short *qsum;     // [n_chunks]
    unsigned *gwords;               // [n_groups] words of each group's run
    unsigned *goff;                 // [n_groups] word offset of the run inside its block of SL_SCAN_BLOCK groups
    unsigned char *out;             // the coded buffer
};

inline SlCodedArgs sl_coded_args(const sl_plan *p, unsigned char *out, unsigned char *ws)
{
    SlCodedArgs A;
    A.G = p->cg;
    A.tensors = p->d_tensors;
    A.groups = p->d_groups;
    A.n_groups = p->n_groups;
    A.ua_log2 = 0;
    while ((1 << A.ua_log2) < p->cg.ua) ++A.ua_log2;
    A.uvec = reinterpret_cast<const unsigned *>(ws + p->ws_uvec);
    A.qsum = reinterpret_cast<const unsigned short *>(ws + p->ws_qsum);
    A.gwords = reinterpret_cast<unsigned *>(ws + p->ws_gwords);
    A.goff = reinterpret_cast<unsigned *>(ws + p->ws_goff);
    A.out = out;
    return A;
}

// Words of a group's run, from the chunks' quotient sums (sixteen are read whether or not the group has them: behind the last lie
// other parts of the workspace).
typedef unsigned sl_u4h __attribute__((ext_vector_type(4), aligned(2)));
SL_DEV unsigned sl_coded_group_words(const SlCodedArgs &A, const SlGroup &g)
{
    const sl_u4h *q = reinterpret_cast<const sl_u4h *>(A.qsum + g.chunk0);
    const sl_u4h lo = q[0], hi = q[1];
    unsigned bits = (unsigned)(g.n_chunks * A.G.k);
#pragma unroll
    for (int i = 0; i < SL_RICE_GROUP; ++i) {
        const unsigned w = i < 8 ? lo[(i >> 1) & 3] : hi[(i >> 1) & 3];
        bits += i < g.n_chunks ? (w >> (16 * (i & 1))) & 0xFFFFu : 0u;
    }
    return (bits + 31u) >> 5;
}

// Block `block` of SL_SCAN_BLOCK groups; called by all threads of a workgroup of THREADS; `wsum` (LDS) THREADS / 64 words.
#define SL_SCAN_BLOCK 1024
inline long long sl_scan_blocks(long long n_groups) { return (n_groups + SL_SCAN_BLOCK - 1) / SL_SCAN_BLOCK; }
template <int THREADS>
SL_DEV void sl_coded_scan_block(const SlCodedArgs &A, long long block, unsigned *wsum)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned carry = 0;                          // words of the block before this tile (a group has below 2^13)
    for (int first = 0; first < SL_SCAN_BLOCK; first += THREADS) {
        if (block * SL_SCAN_BLOCK + first >= A.n_groups) return;
        const long long g = block * SL_SCAN_BLOCK + first + tid;
        const unsigned v = g < A.n_groups ? sl_coded_group_words(A, A.groups[g]) : 0u;
        const unsigned incl = (unsigned)sl_wave_iscan((int)v);
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        unsigned before = carry;
#pragma unroll
        for (int q = 0; q < THREADS / 64; ++q) {
            before += q < wave ? wsum[q] : 0u;
            carry += wsum[q];
        }
        if (g < A.n_groups) {
            A.gwords[g] = v;
            A.goff[g] = before + incl - v;
        }
        __syncthreads();
    }
}

// The buffer header and the zero padding that rounds the buffer up to 16 bytes, for a section of so many words.  One
// wave (or its first four lanes).
SL_DEV void sl_coded_header(unsigned long long words, long long section, unsigned char *out)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long end = (unsigned long long)section + 4ull * words;
    const unsigned long long total = (end + 15ull) & ~15ull;
    if (lane == 0) {
        unsigned long long *h = reinterpret_cast<unsigned long long *>(out);
        h[0] = 0x3230454349524C53ull;                      // "SLRICE02", little endian
        h[1] = total;
    }
    if (end + 4ull * lane < total) *reinterpret_cast<unsigned *>(out + end + 4ull * lane) = 0u;
}

// Words of the section in front of group gi, after sl_coded_scan_block.  One wave; uniform.
SL_DEV unsigned long long sl_coded_words_before(const SlCodedArgs &A, long long gi)
{
    const long long block = gi / SL_SCAN_BLOCK;
    unsigned long long v = 0;
    if (block > 0) {
        for (long long b = threadIdx.x & 63; b < block; b += 64) {
            const long long last = b * SL_SCAN_BLOCK + SL_SCAN_BLOCK - 1;
            v += A.goff[last] + A.gwords[last];
        }
#pragma unroll
        for (int l = 0; l < 6; ++l) v += sl_partner(v, l);
    }
    return v + A.goff[gi];
}

// Words of LDS that sl_coded_place needs per wave.
inline size_t sl_coded_place_words(const SlCodedGeom &G) { return (size_t)SL_RICE_GROUP * G.ua + 1; }

// Group g, whose run of nw words begins at word `base` of the section (below 2^32 by the plan's check; one wave; `run`: its LDS): the chunks' vectors, as the writers left them (G.ua words each,
// bits beyond k + Q undefined), are shifted to their bit offsets inside the run in LDS; the run and
// the directory entry go to the buffer.  A lane takes one (chunk, word) pair per turn, so that the
// loads of several chunks are under way together (a chunk per turn left most lanes idle and waited
// for memory sixteen times in a row: 33 us for 443,569 chunks of k = 64).  From k = 356 (33 words and
// more) a chunk's words fill the wave by themselves, and pairs spend a third of it on words beyond the
// vectors: a chunk per turn (304 chunks, k = 1024, whole transcode: pairs 27.5 us, so 25.5; k = 512 19.5 and 19.0).
#ifndef SL_PLACE_BY_CHUNK
#define SL_PLACE_BY_CHUNK 6               // log2 of the words of the longest vector, rounded up
#endif
SL_DEV void sl_coded_place_at(const SlCodedArgs &A, const SlGroup &g, unsigned long long base, unsigned nw, unsigned *run)
{
    const int lane = threadIdx.x & 63;
    const SlCodedGeom &G = A.G;
    const SlTensorDev td = A.tensors[g.tensor];
    const long long c0 = g.chunk0;
    const int nc = g.n_chunks;

    const int q = lane < nc ? (int)A.qsum[c0 + lane] : 0;
    const int nbits = lane < nc ? G.k + q : 0;
    const int start = sl_wave_iscan(nbits) - nbits;                      // lanes 0..15 matter
    for (unsigned w = lane; w < nw + 1u; w += 64) run[w] = 0u;
    sl_wave_sync();
    const bool by_chunk = A.ua_log2 >= SL_PLACE_BY_CHUNK;
    for (int i = 0; by_chunk && i < nc; ++i) {
        const int s = __builtin_amdgcn_readlane(start, i), n = __builtin_amdgcn_readlane(nbits, i), sh = s & 31;
        const unsigned *src = A.uvec + (size_t)(c0 + i) * G.ua;
        for (int j = lane; 32 * j < n; j += 64) {
            const int left = n - 32 * j;         // bits of this word that belong to the vector
            const unsigned w = src[j] & (left < 32 ? (1u << left) - 1u : 0xFFFFFFFFu);
            sl_lds_or(&run[(s >> 5) + j], w << sh);
            if (sh) sl_lds_or(&run[(s >> 5) + j + 1], w >> (32 - sh));
        }
    }
    const int slots = by_chunk ? 0 : nc << A.ua_log2;
    constexpr int U = 2;                         // turns whose loads are issued together
    for (int s0 = 0; s0 < slots; s0 += 64 * U) {
        unsigned v[U];
        int at[U];                               // first bit of the word inside the run, or -1
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int slot = s0 + 64 * u + lane, i = min(slot >> A.ua_log2, SL_RICE_GROUP - 1), j = slot & ((1 << A.ua_log2) - 1);
            const int n = sl_lane_read(nbits, i), left = n - 32 * j;     // bits of this word that belong to the vector
            const int first = sl_lane_read(start, i);
            at[u] = slot < slots && left > 0 ? first + 32 * j : -1;
            v[u] = at[u] >= 0 ? A.uvec[(size_t)(c0 + i) * G.ua + j] & (left < 32 ? (1u << left) - 1u : 0xFFFFFFFFu) : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (at[u] >= 0) {
                const int sh = at[u] & 31;
                sl_lds_or(&run[at[u] >> 5], v[u] << sh);
                if (sh) sl_lds_or(&run[(at[u] >> 5) + 1], v[u] >> (32 - sh));
            }
        }
    }
    sl_wave_sync();
    unsigned *dst = reinterpret_cast<unsigned *>(A.out + G.section) + base;
    for (unsigned w = lane; w < nw; w += 64) dst[w] = run[w];
    unsigned char *entry = A.out + td.cdir_off + (long long)g.local_group * G.dent;
    if (lane == 0) *reinterpret_cast<unsigned *>(entry) = (unsigned)base;
    if (lane < SL_RICE_GROUP) {
        if (G.qf == 1) entry[4 + lane] = (unsigned char)q;
        else reinterpret_cast<unsigned short *>(entry + 4)[lane] = (unsigned short)q;
    }
}

// Group gi (one wave; `run`: its LDS), after sl_coded_scan_block.  The wave of the last group writes the buffer header too.
SL_DEV void sl_coded_place(const SlCodedArgs &A, long long gi, unsigned *run)
{
    const unsigned long long base = sl_coded_words_before(A, gi);
    const unsigned nw = A.gwords[gi];
    if (gi == A.n_groups - 1) sl_coded_header(base + nw, A.G.section, A.out);
    sl_coded_place_at(A, A.groups[gi], base, nw, run);
}
