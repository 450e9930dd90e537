// Coded wire format: the passes that place the variable-length part (the chunks' quotient bit
// vectors), and the transcoder from a plain payload (sl_rice_encode).  The format is described
// in sl_coded.h; the appendix "Compression of indices in Top-k" of the paper is where an index
// coder enters the method.
//
// The writers of a coded buffer (kernel A of sl_compress_coded, or k_rice_chunks below for a
// payload that already exists) put everything whose place follows from the tensor list - table
// headers, remainder and value fields - straight into the buffer, and leave each chunk's bit
// vector and quotient sum Q in the workspace, from where the placement steps of sl_coded.h take them.
#include <algorithm>

#include "sl_coded.h"

int sl_rice_param(int k)
{
    const int q = 2839 / k;
    int b = 0;
    while ((2 << b) <= q) ++b;
    return q < 1 ? 0 : b;
}

namespace {

__global__ void __launch_bounds__(SL_SCAN_BLOCK) k_coded_scan(SlCodedArgs A)
{
    __shared__ unsigned wsum[SL_SCAN_BLOCK / 64];
    sl_coded_scan_block<SL_SCAN_BLOCK>(A, (long long)blockIdx.x, wsum);
}

__global__ void __launch_bounds__(256) k_coded_place(SlCodedArgs A)
{
    extern __shared__ __align__(16) unsigned place_lds[];
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long gi = (long long)blockIdx.x * (blockDim.x >> 6) + wave;
    if (gi < A.n_groups) sl_coded_place(A, gi, place_lds + (size_t)wave * (SL_RICE_GROUP * A.G.ua + 1));
}

// The header of a buffer without groups.
__global__ void __launch_bounds__(64) k_coded_empty(SlCodedArgs A) { sl_coded_header(0, A.G.section, A.out); }

// Both placement steps in one: every workgroup sums up the words of the groups before its own.  That is quadratic in the groups, but up
// to SL_PLACE_FUSED_UPTO it takes two turns of 1024 threads, less than a launch of the scan (sl_rice_encode at k = 64, scan and placement /
// this, us: 16 groups 8.6 / 7.7, 1024 9.9 / 8.9, 2048 11.65 / 10.95, 4096 14.7 / 14.75, 8192 20.7 / 25.3; 9.7, 16.3, 25.5, 44.0 and 80.6 us
// when one workgroup went through all groups of a tensor).  The waves behind the first `placing` only help to sum up.
__global__ void __launch_bounds__(1024) k_coded_place_fused(SlCodedArgs A, int placing)
{
    extern __shared__ __align__(16) unsigned place_lds[];
    __shared__ unsigned long long part[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = sl_uniform(tid >> 6);
    const long long first = (long long)blockIdx.x * placing;
    unsigned long long sum = 0;
    for (long long g = tid; g < first; g += 1024) sum += sl_coded_group_words(A, A.groups[g]);
#pragma unroll
    for (int l = 0; l < 6; ++l) sum += sl_partner(sum, l);
    if (lane == 0) part[wave] = sum;
    // (meanwhile: the words of the workgroup's own groups, by lane)
    const unsigned own = lane < placing && first + lane < A.n_groups ? sl_coded_group_words(A, A.groups[first + lane]) : 0u;
    const unsigned upto = (unsigned)sl_wave_iscan((int)own);
    __syncthreads();
    const long long gi = first + wave;
    if (wave >= placing || gi >= A.n_groups) return;
    unsigned long long base = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) base += part[w];
    const unsigned nw = (unsigned)__builtin_amdgcn_readlane((int)own, wave);
    base += (unsigned)__builtin_amdgcn_readlane((int)upto, wave) - nw;
    if (gi == A.n_groups - 1) sl_coded_header(base + nw, A.G.section, A.out);
    sl_coded_place_at(A, A.groups[gi], base, nw, place_lds + (size_t)wave * (SL_RICE_GROUP * A.G.ua + 1));
}

// ------------------------------------------------------------------ transcoders
// Both take several consecutive chunks of a coding group per wave, as many as fill its lanes at E consecutive entries
// each (8; 4 where k is no multiple of 8): 16 chunks up to k = 32, 4 at k = 128, one from k = 264 on, then in
// passes of 64 * E entries.  They are bound by the instructions of a wave and the length of its chain of memory and LDS
// trips, so a wave with a quarter of its lanes at work pays four times (a chunk per wave before; 125,100 chunks of k = 128:
// encode 50 -> 21 us, decode 128 -> 27).  What belongs to the chunks of a wave lies in one piece in both formats and in the
// workspace: records, fixed records, bit vectors.
struct TransArgs {
    SlCodedGeom G;
    const SlTensorDev *tensors;
    const SlGroup *groups;
    long long n_groups;
    int rec_bytes;
    int s_log2;              // chunks per wave: 1 << s_log2, one pass where that is above 1
    int L;                   // lanes per chunk: k / E
    unsigned magic_l, magic_v;   // floor(2^32 / d) + 1 for d = L and the words of a chunk's value fields (0: d = 1)
    int lds_words;           // of one wave
    int run_words;           // decode: words of the longest run of bit vectors of a wave
    const unsigned char *in;
    unsigned sec_words;      // decode: words of the buffer's quotient section
    unsigned char *out;
    unsigned *uvec;          // encode
    unsigned short *qsum;
};

SL_DEV int div_by(int n, unsigned magic) { return magic ? (int)__umulhi((unsigned)n, magic) : n; }

// The chunks of a wave.
struct WaveChunks {
    SlTensorDev td;
    int pos;                 // place of the first one in its group
    long long local, gi;     // its index in the tensor, the group's in the list
    int n;                   // how many there are (0: none)
};

SL_DEV WaveChunks wave_chunks(const TransArgs &A)
{
    WaveChunks W;
    const long long w = (long long)blockIdx.x * (blockDim.x >> 6) + sl_uniform((int)(threadIdx.x >> 6));
    W.gi = w >> (4 - A.s_log2);
    W.n = 0;
    if (W.gi >= A.n_groups) return W;
    const SlGroup g = A.groups[W.gi];
    W.td = A.tensors[g.tensor];
    W.pos = (int)(w & ((SL_RICE_GROUP >> A.s_log2) - 1)) << A.s_log2;
    W.local = (long long)g.local_group * SL_RICE_GROUP + W.pos;
    const long long left = W.td.n_chunks - W.local;
    W.n = left <= 0 ? 0 : (int)min((long long)(1 << A.s_log2), left);
    return W;
}

// Plain -> coded: a lane reads its E indices from the record, codes their gaps and puts its remainder fields and
// its piece of the bit vector (64 bits hold them but for clustered supports, which go bit by bit) into
// LDS; from there and from the value fields the chunks' fixed records and vectors leave in whole words.
template <int E>
__global__ void __launch_bounds__(256) k_rice_encode(TransArgs A)
{
    extern __shared__ __align__(16) unsigned trans_lds[];
    const int lane = threadIdx.x & 63;
    const SlCodedGeom &G = A.G;
    const WaveChunks W = wave_chunks(A);
    if (W.n == 0) return;
    const SlTensorDev &td = W.td;
    const int k = G.k, b = G.b, L = A.L, nf = G.cfix >> 2;
    unsigned *fx = trans_lds + (size_t)sl_uniform((int)(threadIdx.x >> 6)) * A.lds_words;       // fixed records
    unsigned *uv = fx + (nf << A.s_log2);                                                       // bit vectors
    const unsigned char *rec = A.in + td.pay_off + G.hdr + W.local * A.rec_bytes;
    const long long c0 = td.chunk0 + W.local;
    // a lane's part of the index stream, E * 12 bits
    auto load_idx = [&](int s, unsigned (&w)[3]) __attribute__((always_inline)) {
        const int i = div_by(s, A.magic_l), o = s - i * L;
        w[0] = w[1] = w[2] = 0u;
        if (s < W.n * L) {
            const unsigned char *at = rec + i * A.rec_bytes + o * (E * 12 / 8);
            w[0] = *reinterpret_cast<const u32_any *>(at);
            if constexpr (E == 8) {
                w[1] = *reinterpret_cast<const u32_any *>(at + 4);
                w[2] = *reinterpret_cast<const u32_any *>(at + 8);
            } else {
                w[1] = *reinterpret_cast<const u16_any *>(at + 4);
            }
        }
    };
    unsigned iw[3];
    load_idx(lane, iw);
    for (int w = lane; w < W.n * nf; w += 64) fx[w] = 0u;
    for (int w = lane; w < W.n * G.ua; w += 64) uv[w] = 0xFFFFFFFFu;
    sl_wave_sync();
    // the value fields
    if ((G.val_bytes & 3) == 0) {
        const int vw = G.val_bytes >> 2;
        for (int q = lane; q < W.n * vw; q += 64) {
            const int i = div_by(q, A.magic_v), w = q - i * vw;
            fx[i * nf + (G.rem_bytes >> 2) + w] = *reinterpret_cast<const u32_any *>(rec + i * A.rec_bytes + 3 * k / 2 + 4 * w);
        }
    } else {
        for (int i = 0; i < W.n; ++i)
            for (int q = lane; q < G.val_bytes; q += 64)
                reinterpret_cast<unsigned char *>(fx + i * nf)[G.rem_bytes + q] = rec[i * A.rec_bytes + 3 * k / 2 + q];
    }
    const int limit = k + G.qmax;            // bits of the longest vector
    int q_carry = 0, last_carry = -1;        // one chunk in several passes: quotients and last index so far
    for (int s0 = 0; s0 < W.n * L; s0 += 64) {
        const int s = s0 + lane, i = div_by(s, A.magic_l), o = s - i * L;
        const bool live = s < W.n * L;
        if (s0) load_idx(s, iw);
        int idx[E];
        idx[0] = (int)(iw[0] & 0xFFFu), idx[1] = (int)((iw[0] >> 12) & 0xFFFu);
        idx[2] = (int)((iw[0] >> 24) | ((iw[1] & 0xFu) << 8)), idx[3] = (int)((iw[1] >> 4) & 0xFFFu);
        if constexpr (E == 8) {
            idx[4] = (int)((iw[1] >> 16) & 0xFFFu), idx[5] = (int)((iw[1] >> 28) | ((iw[2] & 0xFFu) << 4));
            idx[6] = (int)((iw[2] >> 8) & 0xFFFu), idx[7] = (int)(iw[2] >> 20);
        }
        int prev = sl_lane_read(idx[E - 1], lane - 1);
        if (lane == 0) prev = last_carry;
        if (o == 0) prev = -1;
        last_carry = __builtin_amdgcn_readlane(idx[E - 1], 63);
        // gaps; remainders as one field of E * b bits, zero bits by their distance from the lane's first code
        unsigned long long rem = 0;
        int z[E], run = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int gap = max(idx[e] - prev - 1, 0);       // (a malformed record's descending index: gap 0)
            prev = idx[e];
            run += gap >> b;
            z[e] = run + e;
            rem |= (unsigned long long)((unsigned)gap & ((1u << b) - 1u)) << (e * b);
        }
        if (!live) run = 0;
        const int incl = sl_wave_iscan(run);
        int before;                              // quotients of the chunk's entries before the lane's
        if (A.s_log2) {
            const int seg = i * L, under = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
            before = incl - run - (seg > 0 ? under : 0);
        } else {
            before = q_carry + incl - run;
            q_carry += __builtin_amdgcn_readlane(incl, 63);
        }
        unsigned *cf = fx + i * nf, *cv = uv + i * G.ua;
        if (live && b) {
            const int bit = o * E * b, sh = bit & 31;
            const unsigned lo = (unsigned)rem, hi = (unsigned)(rem >> 32);
            const unsigned r1 = sh ? __builtin_amdgcn_alignbit(hi, lo, 32 - sh) : hi, r2 = sh ? hi >> (32 - sh) : 0u;
            sl_lds_or(&cf[bit >> 5], lo << sh);
            if (r1) sl_lds_or(&cf[(bit >> 5) + 1], r1);
            if (r2) sl_lds_or(&cf[(bit >> 5) + 2], r2);
        }
        const int at = before + o * E, sh = at & 31;         // the lane's first code in the vector
        if (__builtin_amdgcn_ballot_w64(live && (sh + z[E - 1] >= 64 || at + z[E - 1] >= limit)) == 0) {
            unsigned long long zeros = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) zeros |= 1ull << ((sh + z[e]) & 63);
            const unsigned lo = (unsigned)zeros, hi = (unsigned)(zeros >> 32);
            if (live && lo) sl_lds_and(&cv[at >> 5], ~lo);
            if (live && hi) sl_lds_and(&cv[(at >> 5) + 1], ~hi);
        } else if (live) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int p = at + z[e];
                if (p < limit) sl_lds_and(&cv[p >> 5], ~(1u << (p & 31)));
            }
        }
        // quotient sums: in one pass the chunk's last lane knows its own
        if (A.s_log2 && live && o == L - 1) A.qsum[c0 + i] = (unsigned short)min(before + run, G.qmax);
    }
    if (A.s_log2 == 0 && lane == 0) A.qsum[c0] = (unsigned short)min(q_carry, G.qmax);
    sl_wave_sync();
    unsigned *fix = reinterpret_cast<unsigned *>(A.out + td.cfix_off + W.local * (long long)G.cfix);
    for (int w = lane; w < W.n * nf; w += 64) fix[w] = fx[w];
    unsigned *uvo = A.uvec + (size_t)c0 * G.ua;
    for (int w = lane; w < W.n * G.ua; w += 64) uvo[w] = uv[w];
    if (W.local == 0)                                              // the table header
        for (int w = lane; 4 * w < G.hdr; w += 64)
            reinterpret_cast<unsigned *>(A.out + td.cblk_off)[w] = reinterpret_cast<const unsigned *>(A.in + td.pay_off)[w];
    if (W.local + W.n == td.n_chunks) {                            // zero padding of the block
        const long long used = (td.cfix_off - td.cblk_off) + td.n_chunks * (long long)G.cfix;
        for (long long q = used + lane; q < td.cblk_bytes; q += 64) A.out[td.cblk_off + q] = 0;
    }
}

// Coded -> plain.  The wave's bit vectors are one run of bits, and in it the zero that ends entry m of chunk i is
// number i * k + m: a lane per word of the run notes where every E-th zero lies (the window of E bits, which
// holds at most one such zero, and how many of its zeros come before), then a lane takes E consecutive
// entries: their zeros from the 64 bits behind the note (20 are needed on average at E = 8 and every k; where some
// lane's reach further, all search word by word), their remainders from the fixed record, and one prefix sum completes
// idx_i = i + ((z_i - i) << b) + r_0 + ... + r_i.  A malformed buffer gives indices cut into the chunk.
// (Registers for eight waves per SIMD.)
template <int E>
__global__ void __launch_bounds__(256, 8) k_rice_decode(TransArgs A)
{
    extern __shared__ __align__(16) unsigned trans_lds[];
    const int lane = threadIdx.x & 63;
    const SlCodedGeom &G = A.G;
    const WaveChunks W = wave_chunks(A);
    if (W.n == 0) return;
    const SlTensorDev &td = W.td;
    const int k = G.k, b = G.b, L = A.L, slots = W.n * L;
    unsigned *raw = trans_lds + (size_t)sl_uniform((int)(threadIdx.x >> 6)) * A.lds_words;      // the run's words, three of ones
    unsigned short *note = reinterpret_cast<unsigned short *>(raw + A.run_words + 3);           // one per E entries, one for all others
    const unsigned char *fix = A.in + td.cfix_off + W.local * (long long)G.cfix;
    unsigned char *rec = A.out + td.pay_off + G.hdr + W.local * A.rec_bytes;
    // the directory entry: lane l holds chunk l's quotient sum (cut to the largest possible one)
    const unsigned char *dir = A.in + td.cdir_off + W.gi * (long long)G.dent - td.group0 * (long long)G.dent;
    const unsigned run_word = *reinterpret_cast<const unsigned *>(dir);
    int q = 0;
    if (lane < SL_RICE_GROUP)
        q = min(G.qf == 1 ? (int)dir[4 + lane] : (int)reinterpret_cast<const unsigned short *>(dir + 4)[lane], G.qmax);
    // the three words that hold a lane's remainder fields (those behind the last field are cut off: any word will do)
    auto load_rem = [&](int s, unsigned (&w)[3]) __attribute__((always_inline)) {
        const int i = div_by(s, A.magic_l), o = s - i * L, wi = (o * E * b) >> 5, top = (G.cfix >> 2) - 1;
        const unsigned *f = reinterpret_cast<const unsigned *>(fix + (s < slots ? i : 0) * G.cfix);
#pragma unroll
        for (int u = 0; u < 3; ++u) w[u] = f[s < slots ? min(wi + u, top) : 0];
    };
    unsigned rw[3];
    load_rem(lane, rw);
    // the value fields, as they stand
    const bool whole = ((G.val_bytes | A.rec_bytes | (3 * k / 2)) & 3) == 0;
    const int vw = G.val_bytes >> 2;
    if (whole) {
        for (int v = lane; v < W.n * vw; v += 64) {
            const int i = div_by(v, A.magic_v), w = v - i * vw;
            reinterpret_cast<unsigned *>(rec + i * A.rec_bytes + 3 * k / 2)[w] =
                reinterpret_cast<const unsigned *>(fix + i * G.cfix + G.rem_bytes)[w];
        }
    } else {
        for (int i = 0; i < W.n; ++i)
            for (int v = lane; v < G.val_bytes; v += 64)
                rec[i * A.rec_bytes + 3 * k / 2 + v] = fix[i * G.cfix + G.rem_bytes + v];
    }
    int start;                                    // lane l: first bit of chunk l's vector in the group's run
    {
        int v = q;
        v += sl_row_shr<1>(v);
        v += sl_row_shr<2>(v);
        v += sl_row_shr<4>(v);
        v += sl_row_shr<8>(v);
        start = lane * k + v - q;
    }
    const int first = __builtin_amdgcn_readlane(start, W.pos);
    const int end = __builtin_amdgcn_readlane(start + k + q, W.pos + W.n - 1);
    const unsigned long long word0 = (unsigned long long)run_word + (unsigned)(first >> 5);
    const int org = first & 31, bits = org + end - first, nw = (bits + 31) >> 5;      // the run in bits of its words
    const unsigned *sec = reinterpret_cast<const unsigned *>(A.in + G.section);
    if (lane < 3) raw[nw + lane] = 0xFFFFFFFFu;
    for (int j0 = 0, carry = 0; j0 < nw; j0 += 64) {
        const int j = j0 + lane;
        unsigned w = 0xFFFFFFFFu;
        if (j < nw && word0 + (unsigned)j < A.sec_words) w = sec[word0 + (unsigned)j];
        if (j < nw) raw[j] = w;
        if (j == 0) w |= (1u << org) - 1u;
        const int left = bits - 32 * j;
        const unsigned zeros = ~w & (left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u);
        const int nz = __builtin_popcount(zeros), incl = sl_wave_iscan(nz), rank = carry + incl - nz;
        carry += __builtin_amdgcn_readlane(incl, 63);
        int from = rank;
#pragma unroll
        for (int u = 0; u < 32 / E; ++u) {
            const int to = u < 32 / E - 1 ? rank + __builtin_popcount(zeros & ((1u << (E * (u + 1))) - 1u)) : rank + nz;
            const int m = (from + E - 1) & ~(E - 1);
            note[m < to && m < W.n * k ? m / E : (L << A.s_log2)] = (unsigned short)(((j * (32 / E) + u) << 3) | (m - from));
            from = to;
        }
    }
    sl_wave_sync();
    int r_carry = 0;                              // one chunk in several passes: remainders so far
    for (int s0 = 0; s0 < slots; s0 += 64) {
        const int s = s0 + lane, ii = div_by(s, A.magic_l);
        const bool live = s < slots;
        const int i = live ? ii : 0, o = live ? s - ii * L : 0;         // (a lane without entries decodes the first ones)
        if (s0) load_rem(s, rw);
        int pre[E];                               // r_0 + ... + r_e, plus e - (e << b): what entry e's index holds
                                                  // besides the lane's part and its zero's place
        int total;
        {
            const unsigned sh = (unsigned)(o * E * b) & 31u;
            const unsigned lo = __builtin_amdgcn_alignbit(rw[1], rw[0], sh), hi = __builtin_amdgcn_alignbit(rw[2], rw[1], sh);
            // entries 0..2 from the window's low word, 3 from the word that starts at its field (b is at most 9),
            // 4..7 from the word that starts at field 4 (b = 9 is k = 4: no such entries)
            const unsigned lo3 = __builtin_amdgcn_alignbit(hi, lo, (unsigned)(3 * b));
            const unsigned lo4 = (unsigned)((((unsigned long long)hi << 32) | lo) >> (4 * b));
            const int step = 1 - (1 << b);
            int t = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const unsigned f = e < 3 ? __builtin_amdgcn_ubfe(lo, (unsigned)(e * b), (unsigned)b)
                                   : e == 3 ? lo3 & ((1u << b) - 1u) : __builtin_amdgcn_ubfe(lo4, (unsigned)((e - 4) * b), (unsigned)b);
                t = e ? t + (int)f + step : (int)f;
                pre[e] = t;
            }
            total = live ? t - (E - 1) * step : 0;
        }
        const int incl = sl_wave_iscan(total);
        int excl;
        if (A.s_log2) {
            const int seg = i * L, under = sl_lane_read(incl, seg > 0 ? seg - 1 : 0);
            excl = incl - total - (seg > 0 ? under : 0);
        } else {
            excl = r_carry + incl - total;
            r_carry += __builtin_amdgcn_readlane(incl, 63);
        }
        const int vec = sl_lane_read(start, W.pos + i) - first + org;      // first bit of the chunk's vector
        int at;                                   // bit of the lane's first zero
        unsigned z, zh;
        {
            const unsigned n = note[live ? s : 0];
            const int win = min((int)(n >> 3), nw * (32 / E) - 1), wi = (win * E) >> 5;   // (beyond: a run with too few zeros)
            const unsigned sh = (unsigned)(win * E) & 31u;
            const unsigned lo = ~__builtin_amdgcn_alignbit(raw[wi + 1], raw[wi], sh);
            const unsigned hi = ~__builtin_amdgcn_alignbit(raw[wi + 2], raw[wi + 1], sh);
            // bits of an earlier lane's words in front of the run are no zeros of it
            const unsigned skip_bits = win * E < org ? (unsigned)(org - win * E) : 0u;      // below E: the window holds a zero
            const unsigned skip = (unsigned)sl_place_in_byte(lo & ((1u << E) - 1u) & (0xFFFFFFFFu << skip_bits), (int)(n & 7u));
            at = win * E + (int)skip;
            z = __builtin_amdgcn_alignbit(hi, lo, skip);
            zh = hi >> skip;                      // (57 bits at least)
        }
        int p[E];                                 // places of the zeros, from the first one's on
        if (__builtin_amdgcn_ballot_w64(live && __builtin_popcount(z) + __builtin_popcount(zh) < E) == 0) {
            p[0] = 0;
            int off = 0;
            z = live ? z : (2u << E) - 1u;
#pragma unroll
            for (int e = 1; e < E; ++e) {
                z &= z - 1u;
                const bool next = z == 0u;        // on to the upper word (once at most)
                z = next ? zh : z;
                off = next ? 32 : off;
                p[e] = __builtin_ctz(z) + off;
            }
        } else {
            int t = at;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                for (int wi = t >> 5; wi < nw; ++wi) {
                    const unsigned v = ~raw[wi] & (wi == t >> 5 ? 0xFFFFFFFFu << (t & 31) : 0xFFFFFFFFu);
                    if (v) {
                        t = 32 * wi + __builtin_ctz(v);
                        break;
                    }
                }
                p[e] = t - at;
                ++t;
            }
        }
        const int base = excl + E * o + ((at - vec - E * o) << b);
        unsigned idx[E];
#pragma unroll
        for (int e = 0; e < E; ++e) idx[e] = (unsigned)(base + (pre[e] + (p[e] << b))) & 0xFFFu;
        // the plain record's 12-bit index stream: eight entries are twelve bytes
        if (live) {
            unsigned char *dst = rec + i * A.rec_bytes + o * (E * 12 / 8);
            *reinterpret_cast<u32_any *>(dst) = idx[0] | (idx[1] << 12) | (idx[2] << 24);
            if constexpr (E == 8) {
                *reinterpret_cast<u32_any *>(dst + 4) = (idx[2] >> 8) | (idx[3] << 4) | (idx[4] << 16) | (idx[5] << 28);
                *reinterpret_cast<u32_any *>(dst + 8) = (idx[5] >> 4) | (idx[6] << 8) | (idx[7] << 20);
            } else {
                *reinterpret_cast<u16_any *>(dst + 4) = (unsigned short)((idx[2] >> 8) | (idx[3] << 4));
            }
        }
    }
    if (W.local == 0)                                              // the table header
        for (int w = lane; 4 * w < G.hdr; w += 64)
            reinterpret_cast<unsigned *>(A.out + td.pay_off)[w] = reinterpret_cast<const unsigned *>(A.in + td.cblk_off)[w];
    if (W.local + W.n == td.n_chunks)                              // zero padding of the block
        for (long long v = G.hdr + td.n_chunks * (long long)A.rec_bytes + lane; v < td.block_bytes; v += 64) A.out[td.pay_off + v] = 0;
}

int launched()
{
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}

}  // namespace

#ifndef SL_PLACE_FUSED_UPTO
#define SL_PLACE_FUSED_UPTO 2048
#endif
// The steps that finish a coded buffer once its writers have run, as launches of their own.
int slk_coded_finish(const sl_plan *p, unsigned char *out, unsigned char *ws, hipStream_t st)
{
    const SlCodedArgs A = sl_coded_args(p, out, ws);
    const size_t per_wave = sl_coded_place_words(p->cg) * sizeof(unsigned);
    if (p->n_groups == 0) {
        hipLaunchKernelGGL(k_coded_empty, dim3(1), dim3(64), 0, st, A);
        return launched();
    }
    if (p->n_groups <= SL_PLACE_FUSED_UPTO) {
        const int placing = (int)std::max<size_t>(1, std::min<size_t>(16, 49152 / per_wave));
        hipLaunchKernelGGL(k_coded_place_fused, dim3((unsigned)((p->n_groups + placing - 1) / placing)), dim3(1024), placing * per_wave, st, A,
                           placing);
        return launched();
    }
    hipLaunchKernelGGL(k_coded_scan, dim3((unsigned)sl_scan_blocks(p->n_groups)), dim3(SL_SCAN_BLOCK), 0, st, A);
    if (const int rc = launched()) return rc;
    int wpb = 4;
    while (wpb > 1 && per_wave * wpb > 65536) wpb >>= 1;
    hipLaunchKernelGGL(k_coded_place, dim3((unsigned)((p->n_groups + wpb - 1) / wpb)), dim3(64 * wpb), per_wave * wpb, st, A);
    return launched();
}

namespace {

// What both transcoders need; returns the entries per lane.
int trans_args(const sl_plan *p, const unsigned char *in, unsigned char *out, TransArgs &A)
{
    const SlCodedGeom &G = p->cg;
    const int E = G.k & 7 ? 4 : 8;
    A.G = G;
    A.tensors = p->d_tensors;
    A.groups = p->d_groups;
    A.n_groups = p->n_groups;
    A.rec_bytes = p->rec_bytes;
    A.L = G.k / E;
    A.s_log2 = 4;
    while (A.s_log2 > 0 && (A.L << A.s_log2) > 64) --A.s_log2;
    auto magic = [](int d) { return d > 1 ? (unsigned)(0x100000000ull / (unsigned)d + 1) : 0u; };
    A.magic_l = magic(A.L);
    A.magic_v = magic(G.val_bytes >> 2);
    A.run_words = 0;
    A.in = in;
    A.sec_words = 0;
    A.out = out;
    A.uvec = nullptr;
    A.qsum = nullptr;
    return E;
}

// Four waves per workgroup, fewer where their LDS passes what a launch may ask for without further notice (the encoder's
// whole fixed records: fp32 values from k = 3976 on, 67,584 bytes at k = 4096).
int trans_launch(void (*fn)(TransArgs), const TransArgs &A, hipStream_t st)
{
    const long long waves = A.n_groups << (4 - A.s_log2);
    const size_t per_wave = (size_t)A.lds_words * sizeof(unsigned);
    int wpb = 4;
    while (wpb > 1 && per_wave * wpb > 65536) wpb >>= 1;
    hipLaunchKernelGGL(fn, dim3((unsigned)((waves + wpb - 1) / wpb)), dim3(64 * wpb), per_wave * wpb, st, A);
    return launched();
}

}  // namespace

int slk_rice_encode(const sl_plan *p, const unsigned char *payload, unsigned char *out,
                    unsigned char *ws, hipStream_t st)
{
    if (p->n_chunks > 0) {
        TransArgs A;
        const int E = trans_args(p, payload, out, A);
        A.uvec = reinterpret_cast<unsigned *>(ws + p->ws_uvec);
        A.qsum = reinterpret_cast<unsigned short *>(ws + p->ws_qsum);
        A.lds_words = ((A.G.cfix >> 2) + A.G.ua) << A.s_log2;
        const int rc = trans_launch(E == 8 ? k_rice_encode<8> : k_rice_encode<4>, A, st);
        if (rc) return rc;
    }
    return slk_coded_finish(p, out, ws, st);
}

int slk_rice_decode(const sl_plan *p, const unsigned char *in, size_t in_bytes, unsigned char *payload, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    TransArgs A;
    const int E = trans_args(p, in, payload, A);
    const size_t sec = in_bytes > (size_t)A.G.section ? (in_bytes - (size_t)A.G.section) >> 2 : 0;
    A.sec_words = sec > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned)sec;
    A.run_words = (31 + ((A.G.k + A.G.qmax) << A.s_log2) + 31) / 32;
    A.lds_words = A.run_words + 3 + ((A.L << A.s_log2) + 2) / 2;
    return trans_launch(E == 8 ? k_rice_decode<8> : k_rice_decode<4>, A, st);
}
