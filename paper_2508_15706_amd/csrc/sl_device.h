// Wave64 helpers for the gfx950 kernels: ballots, cross-lane butterflies and
// the fixed-shape fp64 summation tree.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sl_internal.h"

#define SL_DEV __device__ __forceinline__

SL_DEV unsigned long long sl_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Number of set bits of `m` below this lane.
SL_DEV int sl_mbcnt(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Orders this wavefront's own LDS accesses: the hardware executes one wave's LDS
// instructions in order, so only the compiler has to be kept from moving
// memory operations across this point.  What waves of a workgroup share needs
// __syncthreads().
SL_DEV void sl_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef float sl_f4 __attribute__((ext_vector_type(4)));
// The same vector in memory that is only 4-byte aligned (rows of a matrix whose column
// count is not a multiple of 4): still one 16-byte access - global memory accesses need
// no more than dword alignment on this target - so every streaming access below goes
// through it and a full tile of any matrix takes the vector path.
typedef float sl_f4u __attribute__((ext_vector_type(4), aligned(4)));

// Streaming (non-temporal) 16-byte accesses for data that is touched once.
// The *_at forms take a wave-uniform base and a 32-bit byte offset, which the
// compiler turns into scalar-base + 32-bit vector-offset addressing (one VGPR
// per address instead of two).
SL_DEV sl_f4 sl_load_stream(const float *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const sl_f4 *>(p));
}
SL_DEV void sl_store_stream(float *p, sl_f4 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<sl_f4 *>(p));
}

// KEEP: without the streaming hint, for rows that do not begin on a 64-byte piece of memory.  The pieces that two tiles share - one in
// four or five of each - are read and written by two waves; a streamed piece is given up between the two, so that it is read twice and,
// worse, written back in parts that the memory has to merge (24,576 chunks, us, streamed / kept: 1001 columns, aggregate 241 / 161, of
// coded payloads 223 / 178, direction 445 / 377, two directions averaged 388 / 314, accumulate 304 / 285; 1000 columns 194 / 157, 189 / 167,
// 379 / 358, 351 / 309, 297 / 295; 127 columns 257 / 180, 259 / 206, 552 / 440, 435 / 350, 367 / 324).  Aligned rows want the hint: 1024
// columns 132 / 146, 132 / 144, 270 / 299, 264 / 292, 226 / 254; 1008 columns (64-byte rows) 149 / 155, 158 / 167, 311 / 339, 303 / 308, 263 / 291.  So do
// reads alone (Sub-k, 1001 columns 132 / 139).  Kept loads with streamed stores lie in between.
template <bool KEEP>
SL_DEV sl_f4 sl_access_load(const sl_f4u *p)
{
    if constexpr (KEEP) return *p;
    else return __builtin_nontemporal_load(p);
}
template <bool KEEP>
SL_DEV void sl_access_store(sl_f4u *p, sl_f4 v)
{
    if constexpr (KEEP) *p = v;
    else __builtin_nontemporal_store(v, p);
}

// (`row_off` is a wave-uniform byte offset and goes into the scalar base, so
// that all accesses of a chunk share the single vector offset `lane_off`.)
template <bool KEEP = false>
SL_DEV sl_f4 sl_load_stream_at(const float *base, unsigned row_off, unsigned lane_off)
{
    const char *row = reinterpret_cast<const char *>(base) + row_off;
    return sl_access_load<KEEP>(reinterpret_cast<const sl_f4u *>(row + lane_off));
}
template <bool KEEP = false>
SL_DEV void sl_store_stream_at(float *base, unsigned row_off, unsigned lane_off, sl_f4 v)
{
    char *row = reinterpret_cast<char *>(base) + row_off;
    sl_access_store<KEEP>(reinterpret_cast<sl_f4u *>(row + lane_off), v);
}

// 16-byte streaming accesses at an address that is only 4-byte aligned.
template <bool KEEP = false>
SL_DEV sl_f4 sl_load_stream_u(const float *p)
{
    return sl_access_load<KEEP>(reinterpret_cast<const sl_f4u *>(p));
}
template <bool KEEP = false>
SL_DEV void sl_store_stream_u(float *p, sl_f4 v)
{
    sl_access_store<KEEP>(reinterpret_cast<sl_f4u *>(p), v);
}

// Four elements at p of which `n` exist (any n; none below 1): one access where all four do, else element by
// element; what does not exist is read as +0.0f and not written.
template <bool KEEP = false>
SL_DEV sl_f4 sl_load_edge(const float *p, int n)
{
    sl_f4 v = sl_f4{0.f, 0.f, 0.f, 0.f};
    if (n >= 4) {
        v = sl_load_stream_u<KEEP>(p);
    } else {
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
            if (cc < n) v[cc] = p[cc];
    }
    return v;
}
template <bool KEEP = false>
SL_DEV void sl_store_edge(float *p, int n, sl_f4 v)
{
    if (n >= 4) {
        sl_store_stream_u<KEEP>(p, v);
    } else {
#pragma unroll
        for (int cc = 0; cc < 4; ++cc)
            if (cc < n) p[cc] = v[cc];
    }
}

// Moves the elements of such loads into place: `exist` and `place` of access u (sl_partial_exist, sl_partial_origin).
template <bool ZERO, int N, class Exist, class Place>
SL_DEV void sl_partial_settle(const SlChunkDesc &d, int lc, int room, Exist exist, Place place, sl_f4 (&v)[N])
{
    // the four elements from the one that lies `by` places into a load on
    auto moved = [&](sl_f4 w, bool one, bool two) -> sl_f4 {
        const float x0 = one ? w.y : w.x, x1 = one ? w.z : w.y, x2 = one ? w.w : w.z;
        return sl_f4{two ? x2 : x0, two ? w.w : x1, x2, w.w};
    };
    auto kept = [&](sl_f4 w, int n) -> sl_f4 {
        if constexpr (!ZERO) return w;
        return sl_f4{n > 0 ? w.x : 0.f, n > 1 ? w.y : 0.f, n > 2 ? w.z : 0.f, n > 3 ? w.w : 0.f};
    };
    const bool cut = ((d.cols | d.last_cols) & 3) != 0;
    if (cut && d.cols == d.last_cols && room) {              // a tile: the same columns in every row
        const int n0 = d.cols - lc;
        const int by = n0 > 0 && n0 < 4 ? 4 - n0 : 0;
        const bool one = by & 1, two = by & 2;
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = kept(moved(v[u], one, two), exist(u));
    } else if (cut) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int n = exist(u), by = n > 0 && n < 4 ? sl_partial_back(n, place(u)) : 0;
            v[u] = kept(moved(v[u], by & 1, by & 2), n);
        }
    } else if constexpr (ZERO) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const bool in = exist(u) > 0;
            v[u] = sl_f4{in ? v[u].x : 0.f, in ? v[u].y : 0.f, in ? v[u].z : 0.f, in ? v[u].w : 0.f};
        }
    }
}

// Accesses i0 .. i0 + N - 1 of a lane to a partial chunk of `arena` (access i: elements lc .. lc + 3 of row 4 i + lr); what
// does not exist comes as +0.0f (ZERO) or as any value.  Every lane issues one 16-byte load per row, and all are under way
// together; with them under the conditions the compiler waits for memory once per row (aggregate of three plain / coded
// payloads, k = 32, us: 1155 chunks of a 67-column matrix 12.2 -> 10.0 / 12.8 -> 13.0, 900 of 530 columns 20.4 -> 10.6 / 17.4 -> 13.9,
// 12,000 of 67 columns 112 -> 66 / 89 -> 80, 24,000 of 1000 columns 257 -> 189 / 235 -> 187, the last also by the order of the
// chunks; with momentum 2000 chunks of 100 columns are 4 % slower, all others faster).
// Where the edge cuts through a lane's columns, the load ends with the row's last element (sl_partial_load_at) and its elements are
// moved into place afterwards.
// (One function, not the two below: with them the aggregates' full chunks take 11 to 15 registers more; 178M list, momentum, fp32
// values 488 / 506.)
template <int N, bool ZERO = false, bool KEEP = false>
SL_DEV void sl_load_partial(const float *arena, const SlChunkDesc &d, int i0, int lane, sl_f4 (&v)[N])
{
    const int lr = lane >> 4, lc = (lane & 15) * 4, room = sl_partial_room(d);
    const float *p = arena + (d.base - room);
    const unsigned o0 = sl_partial_origin(d, lr, lc, room), step = 16u * (unsigned)d.stride;
    auto exist = [&](int u) -> int { return sl_partial_exist(d, lr, lc, i0 + u); };
    auto place = [&](int u) -> unsigned { return o0 + (unsigned)(i0 + u) * step; };
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = sl_load_stream_at<KEEP>(p, 0u, sl_partial_load_at(exist(u), place(u), room));
    sl_partial_settle<ZERO>(d, lc, room, exist, place, v);
}

// The same in two steps, for several streams: all requested before the first is moved into place.  What does not exist comes as any value.
template <bool KEEP = false, int N>
SL_DEV void sl_partial_request(const float *arena, const SlChunkDesc &d, int i0, int lane, sl_f4 (&v)[N])
{
    const int lr = lane >> 4, lc = (lane & 15) * 4, room = sl_partial_room(d);
    const float *p = arena + (d.base - room);
    const unsigned o0 = sl_partial_origin(d, lr, lc, room), step = 16u * (unsigned)d.stride;
#pragma unroll
    for (int u = 0; u < N; ++u)
        v[u] = sl_load_stream_at<KEEP>(p, 0u, sl_partial_load_at(sl_partial_exist(d, lr, lc, i0 + u), o0 + (unsigned)(i0 + u) * step, room));
}
template <int N>
SL_DEV void sl_partial_place(const SlChunkDesc &d, int i0, int lane, sl_f4 (&v)[N])
{
    const int lr = lane >> 4, lc = (lane & 15) * 4, room = sl_partial_room(d);
    const unsigned o0 = sl_partial_origin(d, lr, lc, room), step = 16u * (unsigned)d.stride;
    sl_partial_settle<false>(d, lc, room, [&](int u) -> int { return sl_partial_exist(d, lr, lc, i0 + u); },
                             [&](int u) -> unsigned { return o0 + (unsigned)(i0 + u) * step; }, v);
}

SL_DEV int sl_popc(unsigned long long m) { return __builtin_popcountll(m); }

SL_DEV int sl_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Which group of adjacent chunks workgroup `i` of a kernel that streams arenas takes: windows of SL_ORDER_WINDOW
// groups are walked at two places together, half a window apart, by the even and the odd XCDs (workgroups
// reach the eight XCDs in turn).  `order` (sl_order) is the number of groups in whole windows, the rest is taken in
// list order; its bit 0 turns the four groups of a place by one from one four to the next.
// What it is for is the memory's: walked at one place by all XCDs, the rows that are open at a time
// crowd on part of its channels.  Accumulate pass / aggregate of coded payloads / dense aggregate of four (k = 64, R = 8), list
// order and this one, us: 178M list 404 / 264 / 786 and 376 / 236 / 754, 510M 1066 / 705 / 2188 and 1002 / 663 / 2062, MoE
// 1424 / 920 / 2877 and 1350 / 865 / 2771, 1.8B 3582 / 2484 / 7616 and 3572 / 2364 / 7424, the same as flat runs 3972 / 2671 /
// 7925 and 3753 / 2490 / 7624; the plain aggregate of the 1.8B list (rows 8 KB apart) 2372 and 2390, the only one that
// lost.  The halves of the whole list in place of windows: the same, but 2470 for the 1.8B coded aggregate (neighbouring chunks
// share lines of the payloads); windows of 256 groups lose 1 % on the accumulate pass; four or eight places 1 - 3 %
// behind two except on flat runs; a third, a sixth or random places are worse than list order.
SL_DEV unsigned sl_work_group(unsigned i, unsigned order)
{
    if (i >= (order & ~1u)) return i;
    const unsigned j = i % SL_ORDER_WINDOW;
    unsigned o = j >> 1;
    if (order & 1u) o = (o & ~3u) | ((o + (o >> 2)) & 3u);
    return i - j + (j & 1u) * (SL_ORDER_WINDOW / 2) + o;
}

// Cross-lane moves inside a row of 16 lanes as data-parallel-primitive modifiers (no trip
// through the LDS crossbar, unlike a shuffle).  With all 64 lanes active:
//   SL_DPP_XOR1, SL_DPP_XOR2  lane i reads lane i ^ 1, i ^ 2 (quad permutations);
//   SL_DPP_HALF_MIRROR        lane i reads lane 7 - i of its group of 8: a lane of the other quad;
//   SL_DPP_MIRROR             lane i reads lane 15 - i of its row: a lane of the other group of 8.
// In a butterfly whose earlier levels left the same value in every lane of a quad (a group of
// 8), the mirrors therefore deliver exactly what lane i ^ 4 (i ^ 8) would.
#define SL_DPP_XOR1 0xB1
#define SL_DPP_XOR2 0x4E
#define SL_DPP_HALF_MIRROR 0x141
#define SL_DPP_MIRROR 0x140
// (every lane has a source lane, so there is no old value to keep: the move needs no copy of v first and
// can become an operand of the instruction that uses it)
template <int CTRL>
SL_DEV int sl_dpp(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true); }
template <int CTRL>
SL_DEV double sl_dpp(double v)
{
    return __hiloint2double(sl_dpp<CTRL>(__double2hiint(v)), sl_dpp<CTRL>(__double2loint(v)));
}
template <int CTRL>
SL_DEV unsigned long long sl_dpp(unsigned long long v)
{
    const unsigned lo = (unsigned)sl_dpp<CTRL>((int)(unsigned)v), hi = (unsigned)sl_dpp<CTRL>((int)(unsigned)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
// Level l (0..5) of a butterfly over the wave: the value of the partner lane.
template <class T>
SL_DEV T sl_partner(T v, int l)
{
    switch (l) {
    case 0: return sl_dpp<SL_DPP_XOR1>(v);
    case 1: return sl_dpp<SL_DPP_XOR2>(v);
    case 2: return sl_dpp<SL_DPP_HALF_MIRROR>(v);
    case 3: return sl_dpp<SL_DPP_MIRROR>(v);
    default: return __shfl_xor(v, 1 << l);
    }
}

// (all 64 lanes active)
SL_DEV int sl_wave_max(int v)
{
#pragma unroll
    for (int l = 0; l < 4; ++l) v = max(v, sl_partner(v, l));       // every lane: its row's maximum
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

SL_DEV int sl_wave_min(int v)
{
#pragma unroll
    for (int l = 0; l < 4; ++l) v = min(v, sl_partner(v, l));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

SL_DEV int sl_pow2ceil(int n)
{
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// Adjacent-pair tree over the 64 lanes' values, `levels` levels (1 <= 2^levels
// <= 64): afterwards every lane whose index is a multiple of 2^levels holds the
// sum of its aligned group in the fixed pairing (v[2i] + v[2i+1] at each level).
// (All 64 lanes active.  a + b and b + a are the same double, so both lanes of a pair end
// up with the same sum, and after level l all 2^(l+1) lanes of a group hold the group's.)
SL_DEV double sl_wave_tree(double v, int levels)
{
#pragma unroll
    for (int l = 0; l < 6; ++l)
        if (l < levels) v = v + sl_partner(v, l);
    return v;
}

SL_DEV double sl_lane0(double v)
{
    int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
    int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    return __hiloint2double(hi, lo);
}

SL_DEV double sl_lane(double v, int l)
{
    int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// sl_wave_tree's result in lane 0, as a wave-uniform value.  The four levels inside a row of
// 16 lanes leave each row's sum in every lane of the row; the two levels above them pair rows
// (0, 1), (2, 3) and then the pairs, read lane by lane instead of being shuffled.
SL_DEV double sl_wave_tree0(double v, int levels)
{
    v = sl_wave_tree(v, min(levels, 4));
    if (levels <= 4) return sl_lane0(v);
    const double r01 = sl_lane(v, 0) + sl_lane(v, 16);
    if (levels == 5) return r01;
    return r01 + (sl_lane(v, 32) + sl_lane(v, 48));
}

// Adjacent-pair trees of x and x*x over the E consecutive floats at v (E a power of two, v
// aligned for the widest read used); entries from index n on count as +0.0 and are not read
// (n a multiple of 4, or of 2 when E = 2: a read never straddles n).
template <int E>
SL_DEV void sl_lane_trees(const float *v, int n, double &sx, double &sxx)
{
    if constexpr (E == 2) {
        float2 q = make_float2(0.f, 0.f);
        if (n > 0) q = *reinterpret_cast<const float2 *>(v);
        const double x0 = q.x, x1 = q.y;
        sx = x0 + x1;
        sxx = x0 * x0 + x1 * x1;
    } else if constexpr (E == 4) {
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        if (n > 0) q = *reinterpret_cast<const float4 *>(v);
        const double x0 = q.x, x1 = q.y, x2 = q.z, x3 = q.w;
        sx = (x0 + x1) + (x2 + x3);
        sxx = (x0 * x0 + x1 * x1) + (x2 * x2 + x3 * x3);
    } else {
        double a, aa, b, bb;
        sl_lane_trees<E / 2>(v, n, a, aa);
        sl_lane_trees<E / 2>(v + E / 2, n - E / 2, b, bb);
        sx = a + b;
        sxx = aa + bb;
    }
}

// Fixed summation trees of one chunk's k selected values x (canonical order, in LDS at
// `val`, 16-byte aligned; k a multiple of 4) and of their squares: the leaves of the
// two-level sums.  Each sequence is padded with +0.0 to P = pow2ceil(k) and reduced by adjacent
// pairs.  Lane l owns the P/64 consecutive entries from l*P/64 on - a subtree, summed in
// the lane - and one butterfly over the lanes finishes both trees.  MAXE bounds P/64 (the
// instantiation's largest k / 64, rounded up to a power of two).  The results are uniform.
template <int MAXE>
SL_DEV void sl_chunk_trees(int k, int lane, const float *val, double &sum_x, double &sum_xx)
{
    const int P = sl_pow2ceil(k);
    double x = 0.0, xx = 0.0;
    int levels = 6;
    if (P <= 64) {
        levels = 0;
        while ((1 << levels) < P) ++levels;
        x = lane < k ? (double)val[lane] : 0.0;
        xx = x * x;
    } else {
        const int E = P >> 6, n = k - lane * E;
        const float *v = val + lane * E;
        if (MAXE >= 2 && E == 2) sl_lane_trees<2>(v, n, x, xx);
        else if (MAXE >= 4 && E == 4) sl_lane_trees<4>(v, n, x, xx);
        else if (MAXE >= 8 && E == 8) sl_lane_trees<8>(v, n, x, xx);
        else if (MAXE >= 16 && E == 16) sl_lane_trees<16>(v, n, x, xx);
        else if (MAXE >= 32 && E == 32) sl_lane_trees<32>(v, n, x, xx);
        else if (MAXE >= 64 && E == 64) sl_lane_trees<64>(v, n, x, xx);
    }
    sum_x = sl_wave_tree0(x, levels);
    sum_xx = sl_wave_tree0(xx, levels);
}
