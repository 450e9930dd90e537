// Kernel A of sl_compress on short lists: error-feedback accumulate and chunk-wise Top-k as in sl_select_kernel.h (Eq. (2)
// lines 1 and 2; Section 3.3 last paragraph), with all waves of a workgroup on ONE chunk.
//
// What bounds a short list is the chain of instructions of one wave, not memory: alone on its SIMD a wave issues a dependent
// instruction every eight cycles or so, and one that passes from the vector to the scalar unit and back (a ballot, its count, a
// new threshold) takes some hundred.  Here wave w owns accesses NA w .. NA w + NA - 1 of the chunk (access i of lane l: local indices
// 256 i + 4 l ..), so that every pass over the chunk is an eighth as long, and the searches are not made step by step:
//   * the lanes of a wave hold 64 thresholds, the waves share the keys they are compared with (ranks): one exchange through
//     LDS gives 64 ranks, which stand for six steps of a bisection;
//   * the bound below which nothing is selected is one of 64 of the group maxima, the bracket of the k-th largest candidate
//     lies between two of 64 candidates, and few steps, if any, are left;
//   * above k = 512 a sample takes the place of the maxima and the candidates are the keys inside its bracket.
// The outputs (index stream and values, coded form, sums) are written by different waves side by side.  Same selection, same
// order, same trees: every byte is the other form's.
#include <cmath>

#include "sl_coded.h"
#include "sl_search.h"
#include "sl_select.h"

namespace {

constexpr int CAND_CAP = 1024, CAND_SLOTS = CAND_CAP / 64, CAND_PAD = 32;
constexpr int SAMPLE = 512;                      // keys of the sample

// LDS, in this order (sizes are multiples of 16 bytes)
constexpr int LDS_TABLE = 128;                   // (tallies of the waves: two sets) centroids of the pending record
constexpr int LDS_RANKS = LDS_TABLE + 64;        // partial ranks, 64 per wave
constexpr int LDS_VEC = LDS_RANKS + 2048;        // the coded form: bit vector and remainder words, 192 at most
constexpr int LDS_LIST = LDS_VEC + 768;          // maxima or sample
constexpr int lds_buffer(int m) { return LDS_LIST + 4 * (m > SAMPLE ? m : SAMPLE); }      // pending values | candidates
constexpr int LDS_CAND = 6 * CAND_CAP + 4 * CAND_PAD;    // keys, then index and sign in 16 bits

// M: group maxima that bound the threshold from below, at least 2k of them; 0: no such bound (k > 512).
// KEEP: the arenas' accesses without the streaming hint (sl_access_load).
template <int WAVES, int M, bool KEEP>
// (Registers for four waves per SIMD above k = 512, where the sums of 64 entries per lane would take more; below, a bound on them that is
// met anyway changes the schedule for the worse: 2048 chunks, k = 64, sl_compress 38.7 us without, 41.8 with it.)
__global__ void __launch_bounds__(64 * WAVES, M > 0 ? 1 : 4) k_select_group(SelectArgs A, int sub, int sel_off, int margin)
{
    constexpr int THREADS = 64 * WAVES, NA = 16 / WAVES, NR = 4 * NA;      // 16-byte accesses and registers per lane
    constexpr int PAD = 4 * WAVES;           // a list of candidates is padded to so many
    static_assert(PAD <= CAND_PAD && WAVES <= 8, "room in LDS");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = sl_uniform(tid >> 6);
    const long long c = blockIdx.x;
    // (what only the outputs need of the arguments is read when they are written: read at the start it costs scalar registers
    // all along, and the searches spill theirs; A is the first parameter, so the kernel's arguments begin with it)
    typedef const SelectArgs __attribute__((address_space(4))) *ArgsPtr;
    ArgsPtr late = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const SlChunkDesc d = A.desc[c];
    const int k = A.k, bits = A.bits;
    const bool coded = A.coded != nullptr, pend = A.pending != nullptr;
    const long long fix_off = coded ? A.cdesc[c].fix_off : 0;
    int *tally = reinterpret_cast<int *>(smem);
    float *table = reinterpret_cast<float *>(smem + LDS_TABLE);
    int *partial = reinterpret_cast<int *>(smem + LDS_RANKS);
    unsigned *vec = reinterpret_cast<unsigned *>(smem + LDS_VEC);
    int *list = reinterpret_cast<int *>(smem + LDS_LIST);
    unsigned char *buffer = smem + lds_buffer(M);
    float *corr = reinterpret_cast<float *>(buffer);
    int *ckey = reinterpret_cast<int *>(buffer);
    unsigned short *cidx = reinterpret_cast<unsigned short *>(ckey + CAND_CAP + CAND_PAD);
    float *sel_val = reinterpret_cast<float *>(smem + sel_off);
    unsigned short *sel_idx = reinterpret_cast<unsigned short *>(sel_val + k);

    // what needs no input: the pending values' array (+0.0f where nothing is pending, see pend_half in sl_select_kernel.h) and the
    // coded form's words
    if (pend) {
#pragma unroll
        for (int u = 0; u < NA; ++u) reinterpret_cast<float4 *>(corr)[THREADS * u + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (coded && tid < 192) vec[tid] = tid < A.G.ua ? 0xFFFFFFFFu : 0u;

    // ---------------------------------------------------------------- loads
    const int lr = lane >> 4, lc = (lane & 15) * 4;
    const unsigned stride = (unsigned)d.stride;
    const bool full = d.flags & SLC_FULL, need_e = !A.frozen;
    float *ec = A.e + d.base;
    sl_f4 ev[NA], dv[NA], tv[NA];
    const unsigned o0 = 4u * ((4u * NA * wave + lr) * stride + lc), step = 16u * stride;
    if (full) {
        if (need_e) {
#pragma unroll
            for (int u = 0; u < NA; ++u) ev[u] = sl_load_stream_at<KEEP>(ec, u * step, o0);
        }
        if (!sub) {
#pragma unroll
            for (int u = 0; u < NA; ++u) dv[u] = sl_load_stream_at<KEEP>(A.delta + d.base, u * step, o0);
        }
        if (A.theta_local) {
#pragma unroll
            for (int u = 0; u < NA; ++u) tv[u] = sl_load_stream_at<KEEP>(A.theta_local + d.base, u * step, o0);
        }
    } else {
        if (need_e) sl_partial_request<KEEP>(A.e, d, NA * wave, lane, ev);
        if (!sub) sl_partial_request<KEEP>(A.delta, d, NA * wave, lane, dv);
        if (A.theta_local) sl_partial_request<KEEP>(A.theta_local, d, NA * wave, lane, tv);
    }
    // The pending record, an entry per thread (k <= 512); above, where records are whole words, eight entries.
    if (pend) {
        const unsigned char *prec = A.pending + d.rec_off, *pcodes = prec + 3 * k / 2;
        float p_table = 0.f;
        if (bits != 32)
            p_table = reinterpret_cast<const float *>(A.pending + sl_lut_off(d, A.hdr_bytes, A.rec_bytes))[min(tid, (1 << bits) - 1)];
        auto value_of = [&](unsigned field) -> float { return table[field & ((1u << bits) - 1u)]; };
        const bool octets = M == 0 && (A.rec_bytes & 3) == 0 && (k & 7) == 0;
        bool first = true;
        // (the table is in place once the first entries have arrived)
        auto settle = [&]() __attribute__((always_inline)) {
            if (first) {
                if (bits != 32 && tid < (1 << bits)) table[tid] = p_table;
                __syncthreads();
                first = false;
            }
        };
        if (octets) {
            for (int o0 = 0; o0 < (k >> 3); o0 += THREADS) {
                const int o = min(o0 + tid, (k >> 3) - 1);       // (a thread without an octet repeats the last one)
                const unsigned *q = reinterpret_cast<const unsigned *>(prec) + 3 * o;
                const unsigned w0 = q[0], w1 = q[1], w2 = q[2];
                unsigned cw = 0;
                if (bits != 32) {
                    unsigned char b[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) b[i] = pcodes[o * bits + min(i, bits - 1)];
                    cw = b[0] | (unsigned)b[1] << 8 | (unsigned)b[2] << 16 | (unsigned)b[3] << 24;
                }
                settle();
                auto put = [&](int e, unsigned j) __attribute__((always_inline)) {
                    corr[j] = bits == 32 ? reinterpret_cast<const float *>(pcodes)[8 * o + e] : value_of(cw >> (e * bits));
                };
                put(0, w0 & 0xFFFu);
                put(1, (w0 >> 12) & 0xFFFu);
                put(2, (w0 >> 24) | ((w1 & 0xFu) << 8));
                put(3, (w1 >> 4) & 0xFFFu);
                put(4, (w1 >> 16) & 0xFFFu);
                put(5, (w1 >> 28) | ((w2 & 0xFFu) << 4));
                put(6, (w2 >> 8) & 0xFFFu);
                put(7, w2 >> 20);
            }
        } else {
            for (int m0 = 0; m0 < k; m0 += THREADS) {
                const int m = min(m0 + tid, k - 1);              // (a thread without an entry repeats the last one)
                const unsigned i = *reinterpret_cast<const u16_any *>(prec + ((3 * m) >> 1));
                unsigned v;
                if (bits == 32) {
                    v = reinterpret_cast<const unsigned *>(pcodes)[m];
                } else {
                    const int at = (m * bits) >> 3;              // (the last byte holds the end of the last code)
                    v = pcodes[at] | (unsigned)pcodes[min(at + 1, ((k * bits) >> 3) - 1)] << 8;
                }
                settle();
                corr[(m & 1) ? i >> 4 : i & 0xFFFu] = bits == 32 ? __uint_as_float(v) : value_of(v >> ((m * bits) & 7));
            }
        }
        __syncthreads();
    }
    // ---------------------------------------------------------------- a = beta * e + delta
    if (!full) {
        if (need_e) sl_partial_place(d, NA * wave, lane, ev);
        if (!sub) sl_partial_place(d, NA * wave, lane, dv);
        if (A.theta_local) sl_partial_place(d, NA * wave, lane, tv);
    }
    float a[NR];
    int key[NR];                             // magnitudes, -1 outside the tensor
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        sl_f4 v;
        if (sub) {
            v = ev[u];
        } else {
            v = A.theta_local ? dv[u] - tv[u] : dv[u];
            if (need_e) {
                sl_f4 x = ev[u];
                if (pend) {
                    const float4 q = reinterpret_cast<const float4 *>(corr)[64 * (NA * wave + u) + lane];
                    x.x = x.x - q.x, x.y = x.y - q.y, x.z = x.z - q.z, x.w = x.w - q.w;
                }
                v.x = fmaf(A.beta, x.x, v.x), v.y = fmaf(A.beta, x.y, v.y);
                v.z = fmaf(A.beta, x.z, v.z), v.w = fmaf(A.beta, x.w, v.w);
            }
        }
        int n = 4;
        if (full) {
            if (need_e && !sub) sl_store_stream_at<KEEP>(ec, u * step, o0, v);
        } else {
            n = sl_partial_exist(d, lr, lc, NA * wave + u);
            if (need_e && !sub) sl_store_edge<KEEP>(ec + ((4u * (NA * wave + u) + lr) * stride + lc), n, v);
        }
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
            a[4 * u + cc] = v[cc];
            key[4 * u + cc] = cc < n ? key_of(v[cc]) : -1;
        }
    }

    // ---------------------------------------------------------------- tools
    // How many of the keys at `l` (LDS, `per` per wave, a multiple of 4) reach this lane's value t: the same in all waves.
    auto ranks = [&](const int *l, int per, int t) __attribute__((always_inline)) {
        int n = 0;
        const int4 *q = reinterpret_cast<const int4 *>(l + wave * per);
#pragma unroll 4
        for (int j = 0; j < (per >> 2); ++j) {
            const int4 x = q[j];
            n += (x.x >= t ? 1 : 0) + (x.y >= t ? 1 : 0) + (x.z >= t ? 1 : 0) + (x.w >= t ? 1 : 0);
        }
        partial[64 * wave + lane] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) n += partial[64 * w + lane];
        return n;
    };
    // Every wave's value to all waves.  (Sets are used in turn: a wave that writes one again has passed a barrier behind everyone's
    // reads of it.)
    int turn = 0;
    auto gather = [&](int mine, int (&all)[WAVES]) __attribute__((always_inline)) {
        int *set = tally + WAVES * turn;
        if (lane == 0) set[wave] = mine;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) all[w] = sl_uniform(set[w]);
        turn ^= 1;
    };
    auto sum_of = [&](const int (&v)[WAVES]) __attribute__((always_inline)) {
        int n = v[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) n += v[w];
        return n;
    };
    auto count_all = [&](auto test) __attribute__((always_inline)) {
        int mine = 0, all[WAVES];
#pragma unroll
        for (int r = 0; r < NR; ++r) mine += sl_popc(sl_ballot(test(key[r])));
        gather(mine, all);
        return sum_of(all);
    };

    // ---------------------------------------------------------------- the candidates: keys in [from, upto)
    // First the keys that reach a bound given by the group maxima; where there are too many of them (partial chunks with fewer groups
    // than k), and above k = 512, those inside the bracket of a sample; where that misses or holds too many (ties without
    // number), none.
    int from = 0, upto, place[NA], base, ncand, n_above, all[WAVES];
    auto inside = [&](int x) { return x >= from && (x < upto || upto == 0x7FFFFFFF); };    // (the largest key belongs to an open range)
    bool have = false;
    for (int attempt = M > 0 ? 0 : 1; !have && attempt < 2; ++attempt) {
        upto = 0x7FFFFFFF;
        if (attempt == 0) {
            // a group is a lane's registers, a part of them, or spread over neighbouring lanes
            constexpr int MM = M > 0 ? M : 64, PER = MM / THREADS;
            if constexpr (PER > 0) {
#pragma unroll
                for (int g = 0; g < PER; ++g) {
                    int m = key[g];
#pragma unroll
                    for (int r = g + PER; r < NR; r += PER) m = max(m, key[r]);
                    list[THREADS * g + tid] = m;
                }
            } else {
                constexpr int SHARE = PER > 0 ? 1 : THREADS / MM;
                static_assert(M == 0 || SHARE == 1 || SHARE == 2 || SHARE == 4, "lanes of a group");
                int m = key[0];
#pragma unroll
                for (int r = 1; r < NR; ++r) m = max(m, key[r]);
                m = max(m, sl_dpp<SL_DPP_XOR1>(m));
                if constexpr (SHARE == 4) m = max(m, sl_dpp<SL_DPP_XOR2>(m));
                list[tid / SHARE] = m;       // (all lanes of the group write the same value)
            }
            __syncthreads();                 // (the pending values have been read by now, too)
            constexpr int EVERY = MM / 64;
            const int t = list[EVERY * lane + (lane & (EVERY - 1))];
            const int n = ranks(list, MM / WAVES, t);
            from = max(sl_wave_max(n >= k ? t : -1), 0);
        } else {
            // one key in eight (of all residues of row and column), k / 8 of the k largest among them
#pragma unroll
            for (int g = 0; g < SAMPLE / THREADS; ++g) {
                int x = key[8 * g];
#pragma unroll
                for (int r = 1; r < 8; ++r) x = (tid & 7) == r ? key[8 * g + r] : x;
                list[THREADS * g + tid] = x;
            }
            __syncthreads();
            constexpr int EVERY = SAMPLE / 64;
            const int t = list[EVERY * lane + (lane & (EVERY - 1))];
            const int n = ranks(list, SAMPLE / WAVES, t), ks = k / (SL_CHUNK / SAMPLE);
            from = max(sl_wave_max(n >= ks + margin ? t : -1), 0);
            const int over = sl_wave_min(n <= ks - margin ? t : 0x7FFFFFFF);
            upto = over > from ? over : 0x7FFFFFFF;
        }
        // how many of its four elements of every access a lane gives, summed over the lanes below for two accesses at a time
        // (halfwords), then over the waves
        int n4[NA], scan[NA / 2], over = 0, mine = 0;
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            n4[u] = 0;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) n4[u] += inside(key[4 * u + cc]) ? 1 : 0;
        }
        if (upto != 0x7FFFFFFF) {
#pragma unroll
            for (int r = 0; r < NR; ++r) over += sl_popc(sl_ballot(key[r] >= upto));
        }
#pragma unroll
        for (int h = 0; h < NA / 2; ++h) scan[h] = sl_wave_iscan(n4[2 * h] | n4[2 * h + 1] << 16);
#pragma unroll
        for (int u = 0; u < NA; ++u) {       // where the lane's elements go, from the wave's first on
            place[u] = mine + ((scan[u >> 1] >> (16 * (u & 1))) & 0xFFFF) - n4[u];
            mine += (__builtin_amdgcn_readlane(scan[u >> 1], 63) >> (16 * (u & 1))) & 0xFFFF;
        }
        gather(mine | over << 16, all);
        base = ncand = n_above = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            base += w < wave ? all[w] & 0xFFFF : 0;
            ncand += all[w] & 0xFFFF;
            n_above += all[w] >> 16;
        }
        have = ncand <= CAND_CAP && n_above < k && n_above + ncand >= k;
    }
    int T = 0, n_gt = 0;                     // the threshold; where more than k keys reach it, how many lie above
    bool exact = false;
    if (have) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            int to = base + place[u];
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const int x = key[4 * u + cc];
                const bool in = inside(x);
                if (in) {
                    ckey[to] = x;
                    cidx[to] = (unsigned short)((256 * (NA * wave + u) + 4 * lane + cc) | (__float_as_uint(a[4 * u + cc]) >> 31) << 15);
                }
                to += in ? 1 : 0;
            }
        }
        if (tid < PAD) ckey[ncand + tid] = -1;
        __syncthreads();
        // the k'-th largest of the list lies between two of 64 of its keys
        const int kk = k - n_above;
        const int t = ckey[(lane * ncand) >> 6];
        const int per = ((ncand + PAD - 1) / PAD) * 4;
        const int n = ranks(ckey, per, t);
        const int lo = max(sl_wave_max(n >= kk ? t : -1), from), hi = sl_wave_min(n < kk ? t : 0x7FFFFFFF);
        exact = sl_ballot(n == kk) != 0;     // (then lo is that lane's)
        T = lo;
        if (!exact) {
            const int nslots = (ncand + 63) >> 6;
            int ck[CAND_SLOTS];
#pragma unroll
            for (int s = 0; s < CAND_SLOTS; s += 4) {
                ck[s] = ck[s + 1] = ck[s + 2] = ck[s + 3] = -1;
                if (s < nslots) {            // (reads beyond the list stay inside its place)
#pragma unroll
                    for (int q = s; q < s + 4; ++q) ck[q] = ckey[64 * q + lane];
#pragma unroll
                    for (int q = s; q < s + 4; ++q) ck[q] = 64 * q + lane < ncand ? ck[q] : -1;
                }
            }
            auto count_cand = [&](int x) {
                int m = 0;
#pragma unroll
                for (int s = 0; s < CAND_SLOTS; s += 4)
                    if (s < nslots) {
#pragma unroll
                        for (int q = s; q < s + 4; ++q) m += sl_popc(sl_ballot(ck[q] >= x));
                    }
                return m;
            };
            // (plain halving: an interpolated step takes four times as long here and saves less)
            const unsigned long long at_hi = sl_ballot(t == hi);
            int beyond = hi;
            n_gt = at_hi ? __builtin_amdgcn_readlane(n, __builtin_ctzll(at_hi)) : count_cand(hi);
            if (n_gt >= kk) T = hi, exact = n_gt == kk, n_gt = 0;        // (NaNs)
            while (!exact && beyond - T > 1) {
                const int mid = T + ((beyond - T) >> 1), m = count_cand(mid);
                if (m >= kk) T = mid;
                else beyond = mid, n_gt = m;
                exact = m == kk;
            }
            n_gt += n_above;
        }
    } else {
        // Ties without number: the waves count their own registers.  Mostly the keys that are too many are those at `from` itself (zeros,
        // values of few levels): where k keys reach it and fewer lie above, it is the threshold (chunks of eight values among zeros, k = 64, us: 2048
        // deferred 37.5, with a wave per chunk 66.6; 512 frozen 18.1 and 50.5, searched here too 63.1).
        auto reach = [&](int x) { return count_all([&](int y) { return y >= x; }); };
        const int above = n_above + ncand >= k ? count_all([&](int y) { return y > from; }) : k;
        if (above < k) {
            T = from, n_gt = above, exact = n_above + ncand == k;
        } else {
            int lmax = key[0];
#pragma unroll
            for (int r = 1; r < NR; ++r) lmax = max(lmax, key[r]);
            gather(sl_wave_max(lmax), all);
            int hi = all[0];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) hi = max(hi, all[w]);
            if (sl_sample_serves(hi)) {
                int n_lo = reach(0), beyond = hi + 1;
                T = sl_find_kth(0, beyond, n_lo, n_gt, k, reach, exact);
            } else {
                T = sl_bisect_kth(0, hi, k, reach, exact);
                if (!exact) {
                    exact = reach(T) == k;
                    n_gt = count_all([&](int y) { return y > T; });
                }
            }
        }
    }
    const int need = exact ? 0 : k - n_gt;   // ties to take, lowest indices first

    // ---------------------------------------------------------------- the selected entries, in ascending local index
    if (have && n_above == 0) {
        // from the list: 64 candidates at a time, each wave its share
        const int nslots = (ncand + 63) >> 6;
        int at = 0, tbase = 0;
        constexpr int S = M > 0 && M <= 128 ? 2 : 4;             // slots that are read together
        for (int s = 0; s < nslots; s += S) {
            int x[S];
#pragma unroll
            for (int q = 0; q < S; ++q) x[q] = ckey[64 * (s + q) + lane];        // (reads beyond the list stay inside its place)
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const int p = 64 * (s + q) + lane;
                const bool in = p < ncand;
                unsigned long long m;
                if (exact) {
                    m = sl_ballot(in && x[q] >= T);
                } else {
                    const bool eq = in && x[q] == T;
                    const unsigned long long me = sl_ballot(eq);
                    m = sl_ballot((in && x[q] > T) || (eq && tbase + sl_mbcnt(me) < need));
                    tbase += sl_popc(me);
                }
                if (((s + q) & (WAVES - 1)) == wave) {
                    const int pos = at + sl_mbcnt(m);
                    if (((m >> lane) & 1ull) && pos < k) {
                        const unsigned i = cidx[p];
                        sel_val[pos] = __uint_as_float((unsigned)x[q] | (i & 0x8000u) << 16);
                        sel_idx[pos] = (unsigned short)(i & 0xFFFu);
                    }
                }
                at += sl_popc(m);
            }
        }
    } else {
        // from the registers
        int gt = 0, eq = 0;                  // this wave's keys that are taken in any case, and its ties
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            gt += sl_popc(sl_ballot(exact ? key[r] >= T : key[r] > T));
            eq += exact ? 0 : sl_popc(sl_ballot(key[r] == T));
        }
        gather(gt << 16 | eq, all);
        int at = 0, tbase = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int e = all[w] & 0xFFFF;
            if (w < wave) {
                at += (all[w] >> 16) + min(e, max(need - tbase, 0));
                tbase += e;
            }
        }
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            bool f[4], tie[4];
            int trank = tbase;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                tie[cc] = !exact && key[4 * u + cc] == T;
                const unsigned long long m = sl_ballot(tie[cc]);
                trank += sl_mbcnt(m);
                tbase += sl_popc(m);
            }
            int pos = at;
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                f[cc] = key[4 * u + cc] > T || (exact && key[4 * u + cc] == T) || (tie[cc] && trank < need);
                trank += tie[cc] ? 1 : 0;
                const unsigned long long m = sl_ballot(f[cc]);
                pos += sl_mbcnt(m);
                at += sl_popc(m);
            }
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
                if (f[cc] && pos < k) {
                    sel_val[pos] = a[4 * u + cc];
                    sel_idx[pos] = (unsigned short)(256 * (NA * wave + u) + 4 * lane + cc);
                    ++pos;
                }
        }
    }
    __syncthreads();

    if (sub) {
        // m - Top-k(m): x - x = +0.0 at the selected positions, the rest stays as it is
        for (int p = tid; p < k; p += THREADS) {
            const unsigned j = sel_idx[p];
            ec[(j >> 6) * stride + (j & 63u)] = 0.0f;
        }
        return;
    }

    // ---------------------------------------------------------------- outputs: wave 1 the coded form, wave 2 the sums, the others
    // index stream and values
    asm volatile("" : "+s"(late));
    if (wave == 2) {
        double s1, s2;
        double *const leaf = late->leafA;
        sl_chunk_trees<(M == 0 ? 64 : M <= 128 ? 1 : M / 128)>(k, lane, sel_val, s1, s2);
        if (lane == 0) {
            leaf[c] = s1;
            leaf[late->n_chunks + c] = s2;
        }
        return;
    }
    if (coded && wave == 1) {
        SlCodedGeom C;                       // (what the coder uses of it)
        C.k = k, C.b = late->G.b, C.qmax = late->G.qmax, C.ua = late->G.ua;
        C.rem_bytes = late->G.rem_bytes, C.val_bytes = late->G.val_bytes, C.cfix = late->G.cfix;
        unsigned *uv = vec, *rw = vec + C.ua;
        const int Q = sl_coded_emit_filled(C, lane, sel_idx, uv, rw);
        unsigned char *fix = late->coded + fix_off;
        for (int w = lane; w < (C.rem_bytes >> 2); w += 64) reinterpret_cast<unsigned *>(fix)[w] = rw[w];
        if (bits == 32) {
            // unquantized: the values follow the remainders as they follow the indices of a plain record
            for (int m = lane; m < k; m += 64) reinterpret_cast<float *>(fix + C.rem_bytes)[m] = sel_val[m];
        } else if ((C.val_bytes & 3) && lane == 0) {
            // the record's last word holds value fields and padding: cleared here, the codes come later
            *reinterpret_cast<unsigned *>(fix + C.cfix - 4) = 0u;
        }
        unsigned *uvo = late->uvec + (size_t)c * C.ua;
        const int words = (k + Q + 31) >> 5;
        for (int w = lane; w < words; w += 64) uvo[w] = uv[w];
        if (lane == 0) late->qsum[c] = (unsigned short)Q;
        return;
    }
    float *const vals = late->vals;
    unsigned char *rec = late->payload + d.rec_off;
    // (the waves that are left: 0, 3, 4, .., and 1 without the coded form)
    const int share = coded ? WAVES - 2 : WAVES - 1, me = 64 * (wave == 0 ? 0 : wave == 1 ? share - 1 : wave - 2) + lane;
    float *recv = bits == 32 ? reinterpret_cast<float *>(rec + 3 * k / 2) : nullptr;
    for (int p = me; p < k; p += 64 * share) {
        vals[c * k + p] = sel_val[p];
        if (recv) recv[p] = sel_val[p];
    }
    const int last = 64 * share - 1 - me;    // (the index stream from the other end: with few entries other waves take it)
    if ((k & 15) == 0) {
        // 12-bit index stream, one 32-bit word per lane (see sl_select_kernel.h for records on 2 bytes)
        for (int w = last; w < 3 * k / 8; w += 64 * share) {
            const int bit0 = 32 * w;
            int m = bit0 / 12;
            unsigned word = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q, ++m) {
                const int sh = 12 * m - bit0;
                if (m < k && sh < 32) {
                    const unsigned v = sel_idx[m];
                    word |= sh >= 0 ? v << sh : v >> (-sh);
                }
            }
            reinterpret_cast<u32_any *>(rec)[w] = word;
        }
    } else {
        for (int b = last; b < 3 * k / 2; b += 64 * share) {
            const int m = 8 * b / 12, sh = 8 * b - 12 * m;       // 0, 4 or 8
            unsigned v = (unsigned)sel_idx[m] >> sh;
            if (sh == 8 && m + 1 < k) v |= (unsigned)sel_idx[m + 1] << 4;
            rec[b] = (unsigned char)v;
        }
    }
}

}  // namespace

int slk_select_group(const SelectArgs &A, bool sub_only, int waves, bool keep, hipStream_t st)
{
    const int k = A.k, m = k <= 64 ? 128 : k <= 128 ? 256 : k <= 256 ? 512 : k <= 512 ? 1024 : 0;
    size_t at = lds_buffer(m) + (A.pending ? SL_CHUNK * sizeof(float) : (size_t)LDS_CAND);
    const int sel_off = (int)at;
    at += 6 * (size_t)k;
    // two and a half standard deviations of how many of the k largest are among the sample
    const double share = (double)k / SL_CHUNK;
    int margin = (int)(2.5 * std::sqrt(SAMPLE * share * (1.0 - share))) + 1;
    const dim3 grid((unsigned)A.n_chunks);
    const int sub = sub_only ? 1 : 0;
    typedef void (*kernel_t)(SelectArgs, int, int, int);
#define SL_GROUP_KINDS(W, KEEP) \
    {k_select_group<W, 128, KEEP>, k_select_group<W, 256, KEEP>, k_select_group<W, 512, KEEP>, k_select_group<W, 1024, KEEP>, k_select_group<W, 0, KEEP>}
    static const kernel_t table[2][2][5] = {{SL_GROUP_KINDS(4, false), SL_GROUP_KINDS(4, true)}, {SL_GROUP_KINDS(8, false), SL_GROUP_KINDS(8, true)}};
#undef SL_GROUP_KINDS
    const kernel_t fn = table[waves == 8 ? 1 : 0][keep ? 1 : 0][m == 128 ? 0 : m == 256 ? 1 : m == 512 ? 2 : m == 1024 ? 3 : 4];
    hipLaunchKernelGGL(fn, grid, dim3(64 * waves), at, st, A, sub, sel_off, margin);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}
