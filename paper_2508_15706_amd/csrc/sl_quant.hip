// Kernels B-E of sl_compress: the per-tensor 2-bit statistical quantizer
// (Section 4, experimental set-up) and the error-feedback residual (Eq. (2)
// line 2, Algorithm 1 error update).
//
//   B  per tensor: fixed-tree fp64 sums of x and x*x over its selected values
//      -> mean mu and variance;
//   C  per chunk: 2-bit codes from (x - mu)^2 vs T, codes packed into the
//      payload record, per-bin partial sums and counts;
//   D  per tensor: fixed-tree sums per bin -> centroid LUT, written as the
//      tensor block's header;
//   E  per chunk: e[idx] = a - LUT[code] at the k selected positions.
//
// Sums over a tensor are two-level: a tree over each chunk's k entries (the
// leaves, produced by kernels A and C) and a tree over the chunk leaves in
// chunk order.  Both trees pad with +0.0 to a power of two and add adjacent
// pairs, so the result does not depend on scheduling.
#include <algorithm>

#include "sl_coded.h"

namespace {

constexpr int RED_THREADS = 1024, RED_WAVES = RED_THREADS / 64;
constexpr int RED_TILE = 4 * RED_THREADS;   // leaves that the block's threads read at a time
constexpr int RED_TILES = 16;               // tiles whose partial sums are kept before they are summed in turn

typedef double red_d2 __attribute__((ext_vector_type(2), aligned(8)));   // one 16-byte access, 8-byte aligned

struct RedShared {
    double part[2][RED_TILES * RED_WAVES];  // sums of 256 consecutive leaves
    double stack[2][40];
    double result[2];
    unsigned long long cnt[RED_WAVES];
};

// Sum w of super `su` (65536 leaves) of tree s, pushed on its binary-counter stack; the last one leaves the tree's sum.  One lane.
SL_DEV void red_push(RedShared &sh, int s, long long su, long long supers, double w)
{
    auto push = [&](long long idx, double x) {
        int lvl = 0;
        while (idx & 1) {
            x = sh.stack[s][lvl] + x;
            idx >>= 1;
            ++lvl;
        }
        sh.stack[s][lvl] = x;
    };
    push(su, w);
    if (su == supers - 1) {
        long long P = 1;
        int top = 0;
        while (P < supers) P <<= 1, ++top;
        for (long long i = supers; i < P; ++i) push(i, 0.0);      // +0.0 padding
        sh.result[s] = sh.stack[s][top];
    }
}

// Adjacent-pair trees over leaf[s][0 .. n), s < NS, padded with +0.0 to a power of two (of at least
// 65536; extra +0.0 leaves do not change a sum).  Called by all RED_THREADS threads of the block;
// the sums come back to every thread.
// What bounds it: latency, one block per tensor and bin; with hundreds of small tensors the number of
// instructions of a block.  The waves read all tiles of 4096 leaves without waiting for each other,
// four loads of 32 bytes per lane under way together, and meet once per 65536 leaves (with a barrier
// pair per tile and one sum after the other the statistics of a 25,152-chunk tensor took 17.7 us, the
// centroids 21); a wave without leaves only writes its zero.
template <int NS>
__device__ void block_tree_sums(const double *const (&leaf)[NS], long long n, RedShared &sh, double (&sum)[NS])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr long long SUPER = (long long)RED_TILE * RED_TILES;
    const long long supers = n > SUPER ? (n + SUPER - 1) / SUPER : 1;
    for (long long su = 0; su < supers; ++su) {
        const long long rest = n - su * SUPER;
        const int tiles = (int)min((long long)RED_TILES, (rest + RED_TILE - 1) / RED_TILE);
        constexpr int U = 4 / NS;
        for (int t0 = 0; t0 < tiles; t0 += U) {
            const long long first = su * SUPER + (long long)t0 * RED_TILE + 256ll * wave;     // this wave's first leaf
            if (first >= n) {                                      // (then the later tiles of the wave are empty too)
                if (lane < U)
#pragma unroll
                    for (int s = 0; s < NS; ++s) sh.part[s][(t0 + lane) * RED_WAVES + wave] = 0.0;
                continue;
            }
            double x[U][NS][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long long b = first + (long long)u * RED_TILE + 4ll * lane;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) x[u][s][q] = 0.0;
                    if (b + 3 < n) {
                        const red_d2 lo = *reinterpret_cast<const red_d2 *>(leaf[s] + b), hi = *reinterpret_cast<const red_d2 *>(leaf[s] + b + 2);
                        x[u][s][0] = lo.x, x[u][s][1] = lo.y, x[u][s][2] = hi.x, x[u][s][3] = hi.y;
                    } else if (b < n) {
                        x[u][s][0] = leaf[s][b];
                        if (b + 1 < n) x[u][s][1] = leaf[s][b + 1];
                        if (b + 2 < n) x[u][s][2] = leaf[s][b + 2];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u < tiles) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const double v = sl_wave_tree((x[u][s][0] + x[u][s][1]) + (x[u][s][2] + x[u][s][3]), 6);
                        if (lane == 0) sh.part[s][(t0 + u) * RED_WAVES + wave] = v;
                    }
                }
        }
        __syncthreads();
        if (wave < NS) {
            const int have = tiles * RED_WAVES;
            double p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = 4 * lane + q < have ? sh.part[wave][4 * lane + q] : 0.0;
            const double w = sl_wave_tree((p[0] + p[1]) + (p[2] + p[3]), 6);
            if (lane == 0) red_push(sh, wave, su, supers, w);
        }
        __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) sum[s] = sh.result[s];
}

// ---- large tensors
// One workgroup reads the leaves of a tensor at the rate of one compute unit: 64 us for the statistics of 131,072 chunks, 50 for a
// bin.  Where a tensor has more than SL_SPLIT_TENSOR chunks, a launch before B and one before D sum up pieces of 256
// leaves, one wave each, and B and D read the pieces' sums; the plan has a table of the pieces, as other tensors' leaves are not looked at.
// (sl_compress, error feedback frozen, k = 64, whole tensors / pieces, us: one matrix of 10,496 chunks, 2 bits 66.4 / 65.1, 4 bits 74.2 / 73.6, 16,384 89.2 / 85.5,
// 98.4 / 94.0, 25,600 127.2 / 117.3, 140.3 / 132.1; one of 12,288 beside 60 of 768 233.4 / 232.8, 262.2 / 261.9, one of 25,600 beside 60 of 512
// 234.8 / 226.4, 260.9 / 253.9; 1.8B list, two of 25,152 chunks, 1600 / 1596, 1775 / 1771, 1605 and 1796 where the launch went over all groups
// of the list; MoE list, one of 12,576, 605.4 / 606.5, 693.5 / 691.9.)
// B and D are instantiations of their own where a list has pieces (PIECES): with the choice made in one kernel lists without any were up to a microsecond slower
// (sl_compress, frozen, us, one kernel / two: 10,240 chunks 61.6 / 60.9, 178M list, 4 bits 192.2 / 191.3, 700 tensors of 3 chunks, 4 bits 84.3 / 79.5).
struct RedPieces {
    double *sum;            // [columns][stride]; null: no tensor of the list is split
    unsigned *cnt;          // (D only)
    long long stride;       // (the number of pieces)
    SL_DEV bool split(const SlTensorDev &td) const { return sum && td.piece0 >= 0; }
};

__global__ void __launch_bounds__(256)
k_piece_sums(const SlPiece *pieces, const double *leaf, const unsigned *cnt, long long n_chunks_total, RedPieces P)
{
    const int lane = threadIdx.x & 63;
    const long long pi = 4ll * blockIdx.x + sl_uniform((int)(threadIdx.x >> 6));
    if (pi >= P.stride) return;
    const SlPiece g = pieces[pi];
    const int n = g.n_chunks, b = 4 * lane;
    leaf += blockIdx.y * n_chunks_total + g.chunk0;
    double x[4] = {0.0, 0.0, 0.0, 0.0};
    unsigned c = 0;
    if (b + 3 < n) {
        const red_d2 lo = *reinterpret_cast<const red_d2 *>(leaf + b), hi = *reinterpret_cast<const red_d2 *>(leaf + b + 2);
        x[0] = lo.x, x[1] = lo.y, x[2] = hi.x, x[3] = hi.y;
    } else if (b < n) {
        x[0] = leaf[b];
        if (b + 1 < n) x[1] = leaf[b + 1];
        if (b + 2 < n) x[2] = leaf[b + 2];
    }
    if (P.cnt) {
        cnt += blockIdx.y * n_chunks_total + g.chunk0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (64 * q + lane < n) c += cnt[64 * q + lane];
#pragma unroll
        for (int l = 0; l < 6; ++l) c += (unsigned)sl_partner((int)c, l);
    }
    const double v = sl_wave_tree((x[0] + x[1]) + (x[2] + x[3]), 6);
    if (lane == 0) {
        const long long at = blockIdx.y * P.stride + pi;
        P.sum[at] = v;
        if (P.cnt) P.cnt[at] = c;
    }
}

// The trees of block_tree_sums over n leaves, from the sums of their pieces; wave s takes tree s.
template <int NS>
__device__ void block_piece_sums(const double *const (&piece)[NS], long long n, RedShared &sh, double (&sum)[NS])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long pieces = (n + SL_PIECE - 1) / SL_PIECE, supers = (pieces + 255) / 256;
    if (wave < NS) {
        const double *const src = NS == 1 || wave == 0 ? piece[0] : piece[NS - 1];
        double p[4], next[4];
        auto load = [&](long long su, double (&x)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const long long i = 256 * su + 4 * lane + q;
                x[q] = i < pieces ? src[i] : 0.0;
            }
        };
        load(0, next);
        for (long long su = 0; su < supers; ++su) {
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = next[q];
            load(su + 1, next);
            const double w = sl_wave_tree((p[0] + p[1]) + (p[2] + p[3]), 6);
            if (lane == 0) red_push(sh, wave, su, supers, w);
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) sum[s] = sh.result[s];
}

// Mean and population variance of m values from their sum and sum of squares.
SL_DEV SlTensorStat stat_of(long long m, double sum, double squares)
{
    const double M = (double)m;
    const double mu = sum / M;
    const double q = squares / M;
    const double p = mu * mu;
    double var = q - p;
    if (var < 0.0) var = 0.0;
    SlTensorStat s;
    s.mu = mu;
    s.var = var;
    return s;
}

// A wave's own statistics of a tensor of at most SL_SHORT_TENSOR chunks: the trees of block_tree_sums over its leaves, all
// of them loaded before the first is added.  Uniform.
#define SL_SHORT_TENSOR 1024
SL_DEV SlTensorStat wave_stats(const SlTensorDev &td, const double *leafA, long long n_chunks_total, int k)
{
    constexpr int TILES = SL_SHORT_TENSOR / 256;
    const int lane = threadIdx.x & 63, n = (int)td.n_chunks;
    double x[2][TILES][4], sum[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < TILES; ++q) {
            const double *leaf = leafA + s * n_chunks_total + td.chunk0;
            const int i = 256 * q + 4 * lane;
#pragma unroll
            for (int u = 0; u < 4; ++u) x[s][q][u] = 0.0;
            if (i + 3 < n) {
                const red_d2 lo = *reinterpret_cast<const red_d2 *>(leaf + i), hi = *reinterpret_cast<const red_d2 *>(leaf + i + 2);
                x[s][q][0] = lo.x, x[s][q][1] = lo.y, x[s][q][2] = hi.x, x[s][q][3] = hi.y;
            } else if (i < n) {
                x[s][q][0] = leaf[i];
                if (i + 1 < n) x[s][q][1] = leaf[i + 1];
                if (i + 2 < n) x[s][q][2] = leaf[i + 2];
            }
        }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        double t[TILES];
#pragma unroll
        for (int q = 0; q < TILES; ++q) {
            t[q] = 0.0;
            if (256 * q < n) t[q] = sl_wave_tree0((x[s][q][0] + x[s][q][1]) + (x[s][q][2] + x[s][q][3]), 6);
        }
        sum[s] = (t[0] + t[1]) + (t[2] + t[3]);
    }
    return stat_of(td.n_chunks * (long long)k, sum[0], sum[1]);
}

// ------------------------------------------------------------------ kernel B
// One workgroup per tensor: its statistics.  With the coded format, up to SL_PLACE_SHARED_UPTO, further
// workgroups take the first placement step (independent of the statistics, and a launch of its
// own would cost more than its work).
template <bool PIECES>
__global__ void __launch_bounds__(RED_THREADS, 8)
k_tensor_stats(const SlTensorDev *tensors, int n_tensors, const double *leafA, long long n_chunks_total, int k,
               SlTensorStat *tstat, SlCodedArgs C, RedPieces P)
{
    __shared__ RedShared sh;
    if ((int)blockIdx.x >= n_tensors) {
        sl_coded_scan_block<RED_THREADS>(C, (int)blockIdx.x - n_tensors, reinterpret_cast<unsigned *>(sh.part[0]));
        return;
    }
    const SlTensorDev td = tensors[blockIdx.x];
    double S[2];
    if (PIECES && P.split(td)) {
        const double *const piece = P.sum + td.piece0;
        const double *const both[2] = {piece, piece + P.stride};
        block_piece_sums<2>(both, td.n_chunks, sh, S);
    } else {
        const double *const leaf[2] = {leafA + td.chunk0, leafA + n_chunks_total + td.chunk0};
        block_tree_sums<2>(leaf, td.n_chunks, sh, S);
    }
    if (threadIdx.x == 0) tstat[blockIdx.x] = stat_of(td.n_chunks * (long long)k, S[0], S[1]);
}

// ------------------------------------------------------------------ kernel C
struct CodeArgs {
    const SlChunkDesc *desc;
    const SlTensorStat *tstat;
    const float *vals;
    double *leafC;          // [4][n_chunks] per-chunk tree sums of the values of each bin
    unsigned *cnt;          // [4][n_chunks] entries per bin
    unsigned char *payload;
    long long n_chunks;
    int k;
    // coded wire format next to the plain record (null: not wanted): the value fields of a chunk are
    // the same bytes in both, in the coded buffer they follow the chunk's remainder fields
    unsigned char *coded;
    const SlCodedDesc *cdesc;
    int rem_bytes;
    int passes;             // passes of 512 entries over a chunk (1 up to k = 512)
    // SHORT: what kernel B would have read; the workgroups behind the chunks' `code_blocks` take its placement step
    unsigned code_blocks;
    const double *leafA;
    const SlTensorDev *tensors;
    SlCodedArgs C;
};

// Value of lane i ^ (1 << L), exactly (sl_partner's mirrors only do where the lanes of a quad hold the
// same value): inside a row of 16 lanes as DPP moves, across rows as a shuffle.
template <int L>
SL_DEV int xor_lane(int v)
{
    if constexpr (L == 0) return sl_dpp<SL_DPP_XOR1>(v);
    else if constexpr (L == 1) return sl_dpp<SL_DPP_XOR2>(v);
    else if constexpr (L == 2) return sl_dpp<SL_DPP_HALF_MIRROR>(sl_dpp<0x1B>(v));     // i ^ 3, then ^ 7
    else if constexpr (L == 3) return sl_dpp<0x128>(v);     // a rotation by eight inside the row
    else return __shfl_xor(v, 1 << L);
}
template <int L>
SL_DEV double xor_lane(double v)
{
    return __hiloint2double(xor_lane<L>(__double2hiint(v)), xor_lane<L>(__double2loint(v)));
}

// Levels L .. LOG_LPC-1 of the adjacent-pair trees of N bins over groups of 2^LOG_LPC lanes.  While a
// lane still holds several bins, a level halves them: the lanes of a pair exchange the bins they give
// up, so that N bins cost N/2 + N/4 + ... exchanges instead of N per level.  (a + b = b + a bit for
// bit, so it does not matter which lane of a pair adds.)  Afterwards r[0 .. max(1, N >> LOG_LPC)) of a
// lane are the bins from bin_of_lane on.
template <int N, int L, int LOG_LPC, int NB>
SL_DEV void reduce_bins(double (&r)[NB], int lane)
{
    if constexpr (L < LOG_LPC) {
        if constexpr (N > 1) {
            const bool up = (lane >> L) & 1;
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                const double lo = r[i], hi = r[i + N / 2], keep = up ? hi : lo, give = up ? lo : hi;
                r[i] = keep + xor_lane<L>(give);
            }
            reduce_bins<N / 2, L + 1, LOG_LPC>(r, lane);
        } else {
            r[0] = r[0] + xor_lane<L>(r[0]);
            reduce_bins<1, L + 1, LOG_LPC>(r, lane);
        }
    }
}

// Is the value at distance dlt from the mean at or beyond inner edge j (1 <= j < 2^BITS) of the
// 2^BITS uniform bins over [-6 sigma, 6 sigma]?  The edge sits at c_j sigma, c_j = 12 j / 2^BITS - 6
// (exact in fp64); decided on squares against (c_j c_j) var.
template <int BITS>
SL_DEV bool edge_reached(int j, double dlt, double dd, double var)
{
    const double cj = (double)j * (12.0 / (double)(1 << BITS)) - 6.0;    // exact: small integer times a power-of-two multiple of 3
    const double Tj = (cj * cj) * var;
    const bool nonneg = dlt >= 0.0;
    return cj < 0.0 ? (nonneg || dd <= Tj) : cj == 0.0 ? nonneg : (nonneg && dd >= Tj);
}

// The code of a value = the number of inner edges it has reached.  The edges ascend, so "reached"
// holds for a prefix of them and the count is found by bisection (BITS decisions instead of 2^BITS - 1).
template <int BITS>
SL_DEV int code_of(double dlt, double var)
{
    const double dd = dlt * dlt;
    int code = 0;
#pragma unroll
    for (int s = BITS - 1; s >= 0; --s) {
        const int mid = code + (1 << s);
        code = edge_reached<BITS>(mid, dlt, dd, var) ? mid : code;
    }
    return code;
}

// The bins of eight consecutive values.  With two bits a bin is the side of the mean and whether the
// value lies beyond 3 sigma, decided by compares against T = 9 var; both stay lane masks, and so do
// the tests for a bin that follow from them.
template <int BITS>
struct Bins {
    int code[8];
    SL_DEV void find(const float *x, double mu, double var)
    {
#pragma unroll
        for (int j = 0; j < 8; ++j) code[j] = code_of<BITS>((double)x[j] - mu, var);
    }
    SL_DEV bool in(int j, int bin) const { return code[j] == bin; }
    SL_DEV unsigned of(int j) const { return (unsigned)code[j]; }
};
template <>
struct Bins<2> {
    bool neg[8], far[8];
    SL_DEV void find(const float *x, double mu, double var)
    {
        const double T = 9.0 * var;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const double dlt = (double)x[j] - mu, dd = dlt * dlt;
            neg[j] = dlt < 0.0;
            far[j] = neg[j] ? dd > T : dd >= T;
        }
    }
    SL_DEV bool in(int j, int bin) const
    {
        return bin == 0 ? neg[j] && far[j] : bin == 1 ? neg[j] && !far[j] : bin == 2 ? !neg[j] && !far[j] : !neg[j] && far[j];
    }
    SL_DEV unsigned of(int j) const { return (neg[j] ? 0u : 2u) + (unsigned)(neg[j] != far[j]); }
};

// Adjacent-pair tree over entries j .. j+N-1 of a lane's eight, entries of other bins counting as +0.0.
template <int N, int BITS>
SL_DEV double lane_tree(const float *x, const Bins<BITS> &B, int j, int bin)
{
    if constexpr (N == 1) return B.in(j, bin) ? (double)x[j] : 0.0;
    else return lane_tree<N / 2>(x, B, j, bin) + lane_tree<N / 2>(x, B, j + N / 2, bin);
}

// 2^LOG_LPC lanes per chunk, eight consecutive entries per lane: 8 << LOG_LPC = pow2ceil(k), at
// least 8, up to 512 (entries from k on are the +0.0 padding of the tree); above, the wave takes the
// chunk's entries in 2, 4 or 8 passes of 512.  A lane finds its entries' codes and sums them bin by
// bin (a subtree of the fixed tree); the lanes of a chunk finish the trees of all bins together
// (reduce_bins).
// What bounds it: on long lists reading the values, at the rate any kernel this short reads
// memory that was written before the last gigabyte was (113 MB in 54 us at 443,569 chunks of k = 64,
// 506 MB in 143 us at 123,505 chunks of k = 1024; with the arithmetic taken out 41 and 145 us); on
// short lists the latency of one chain descriptor - statistics - arithmetic.  Eight entries per lane
// need no transposition through LDS and no deep stacks of partial sums in registers, and the
// cross-lane levels are shared by 64 / 2^LOG_LPC chunks.  A lane per chunk with such stacks, which
// this replaces up to k = 128 and at 1, 3 and 4 bits, took 88 us at k = 64, 2 bits, and, four bins
// per pass, 176 us for 46,537 chunks of k = 128 at 4 bits (here 30) and 1900 us for 300 chunks of
// k = 1024 (here 25), where it left most of the chip without a wave.  Waves that stay for
// several steps and fetch ahead are slower: the registers cost more waves than the overlap gains.
// SHORT (short lists of short tensors, slk_quantize): there is no kernel B; a wave finds the statistics of its chunks'
// tensors by itself from at most 16 KB of leaves each, which costs less than the launch (sl_compress at k = 64, plain / coded, us: 64 chunks 20.4 -> 19.1 / 23.0 -> 21.1, 512 22.1 -> 20.8 / 24.7 -> 22.9, 1024 26.3 -> 25.3 / 29.2 -> 27.4).
template <int BITS, int LOG_LPC, bool SHORT>
__global__ void __launch_bounds__(256) k_codes(CodeArgs A)
{
    constexpr int E = 8, LPC = 1 << LOG_LPC, CPW = 64 / LPC, NB = 1 << BITS, LEFT = NB >> LOG_LPC > 0 ? NB >> LOG_LPC : 1;
    constexpr bool WIDE = E * LPC > 128;     // a bin's count needs more than 8 bits
    const int lane = threadIdx.x & 63, k = A.k;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    if constexpr (SHORT) {
        if (blockIdx.x >= A.code_blocks) {
            __shared__ unsigned wsum[4];
            sl_coded_scan_block<256>(A.C, (int)(blockIdx.x - A.code_blocks), wsum);
            return;
        }
    }
    const long long cw = ((long long)blockIdx.x * (blockDim.x >> 6) + wave) * CPW;
    if (cw >= A.n_chunks) return;
    const int sub = lane & (LPC - 1);
    const long long c = cw + (lane >> LOG_LPC);
    const bool live = c < A.n_chunks;
    const long long cl = live ? c : cw;          // (a lane without a chunk reads the wave's first one and writes nothing)
    const int mine = live ? k : 0;

    const float *vin = A.vals + cl * k;
    const SlChunkDesc d = A.desc[cl];
    double mu = 0.0, var = 0.0;
    if constexpr (SHORT) {
        const int t0 = __builtin_amdgcn_readlane(d.tensor, 0), t1 = __builtin_amdgcn_readlane(A.desc[min(cw + CPW, A.n_chunks) - 1].tensor, 0);
        for (int t = t0; t <= t1; ++t) {
            const SlTensorStat s = wave_stats(A.tensors[t], A.leafA, A.n_chunks, k);
            mu = d.tensor == t ? s.mu : mu;
            var = d.tensor == t ? s.var : var;
        }
    } else {
        mu = A.tstat[d.tensor].mu, var = A.tstat[d.tensor].var;
    }
    unsigned char *const out1 = A.payload + d.rec_off + 3 * k / 2;
    unsigned char *const out2 = A.coded ? A.coded + A.cdesc[cl].fix_off + A.rem_bytes : nullptr;

    constexpr int BY = NB >= 8 ? NB / 4 : 1;
    unsigned by[BY];                             // entries per bin, bytes (two bits: one word; more: word 2h + p
#pragma unroll                                   // holds bins 8h + p, + 2, + 4, + 6; one bit: 16-bit fields)
    for (unsigned &q : by) q = 0;
    double r[NB], left1 = 0.0, left2 = 0.0, left4 = 0.0;     // (left*: roots of 512, 1024 and 2048 entries, above k = 512)
    struct Values {
        sl_f4 a, b;
    };
    auto values_at = [&](int m0) -> Values {     // entries m0 .. m0+7 of the chunk, +0.0f from entry k on
        Values v;
        v.a = v.b = sl_f4{0.f, 0.f, 0.f, 0.f};
        if (m0 < mine) v.a = sl_load_stream(vin + m0);
        if (m0 + 4 < mine) v.b = sl_load_stream(vin + m0 + 4);
        return v;
    };
    Values next = values_at(E * sub);
#pragma unroll 1
    for (int p = 0, m0 = E * sub; p == 0 || (LOG_LPC == 6 && p < A.passes); ++p, m0 += E * LPC) {
        const int n = min(max(mine - m0, 0), E);             // entries of this lane: a multiple of 4
        const Values now = next;
        if constexpr (LOG_LPC == 6) {
            if (p + 1 < A.passes) next = values_at(m0 + E * LPC);
        }
        const float x[E] = {now.a.x, now.a.y, now.a.z, now.a.w, now.b.x, now.b.y, now.b.z, now.b.w};
        Bins<BITS> B;
        B.find(x, mu, var);
        // ---- the code fields: eight entries are BITS whole bytes
        unsigned w = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) w |= B.of(j) << (BITS * j);
        auto store_codes = [&](unsigned char *out) __attribute__((always_inline)) {
            unsigned char *o = out + (m0 >> 3) * BITS;
            if (n == E) {
                if constexpr (BITS == 4) {                   // 4-byte aligned: k is a multiple of 8
                    *reinterpret_cast<unsigned *>(o) = w;
                } else if (BITS == 2 && (k & 7) == 0) {      // 2-byte aligned
                    *reinterpret_cast<unsigned short *>(o) = (unsigned short)w;
                } else {
#pragma unroll
                    for (int q = 0; q < BITS; ++q) o[q] = (unsigned char)(w >> (8 * q));
                }
            } else if (BITS == 2 && n == 4) {
                o[0] = (unsigned char)w;
            }
        };
        store_codes(out1);
        if (A.coded) store_codes(out2);
        // ---- entries per bin
        if constexpr (NB <= 4) {                 // from the packed fields
            const unsigned v = w & ((1u << (BITS * n)) - 1u);
            if constexpr (NB == 2) {
                const unsigned ones = (unsigned)__builtin_popcount(v);
                by[0] += (unsigned)n - ones + (ones << 16);
            } else {
                const unsigned lo = v & 0x5555u, hi = (v >> 1) & 0x5555u, both = lo & hi;
                const unsigned n3 = (unsigned)__builtin_popcount(both), n1 = (unsigned)__builtin_popcount(lo ^ both),
                               n2 = (unsigned)__builtin_popcount(hi ^ both);
                by[0] += (unsigned)n - n1 - n2 - n3 + (n1 << 8) + (n2 << 16) + (n3 << 24);
            }
        } else {
            unsigned long long nib = 0;          // four bits per bin hold the counts of eight entries
#pragma unroll
            for (int j = 0; j < 8; ++j) nib += j < n ? 1ull << (4 * B.of(j)) : 0ull;
#pragma unroll
            for (int h = 0; h < NB / 8; ++h) {
                const unsigned v = (unsigned)(nib >> (32 * h));
                by[2 * h] += v & 0x0F0F0F0Fu;
                by[2 * h + 1] += (v >> 4) & 0x0F0F0F0Fu;
            }
        }
        // ---- sums per bin
#pragma unroll
        for (int b = 0; b < NB; ++b) r[b] = lane_tree<8>(x, B, 0, b);
        reduce_bins<NB, 0, LOG_LPC>(r, lane);
        if constexpr (LOG_LPC == 6) {            // passes pair up like any other neighbours of the tree
            if (p & 1) {
                r[0] = left1 + r[0];
                if (p & 2) {
                    r[0] = left2 + r[0];
                    if (p & 4) r[0] = left4 + r[0];
                    else left4 = r[0];
                } else {
                    left2 = r[0];
                }
            } else {
                left1 = r[0];
            }
        }
    }

    // ---- the counts of the chunk: all its lanes end up with the sums
    constexpr int CW = (NB >= 8 ? NB / 4 : 1) * (WIDE && NB > 2 ? 2 : 1);
    unsigned cnt[CW];
    if constexpr (CW == BY) {
#pragma unroll
        for (int w = 0; w < CW; ++w) cnt[w] = by[w];
    } else {                                     // 16 bits: word 2w + s holds bytes s and s + 2 of word w
#pragma unroll
        for (int w = 0; w < BY; ++w) cnt[2 * w] = by[w] & 0x00FF00FFu, cnt[2 * w + 1] = (by[w] >> 8) & 0x00FF00FFu;
    }
#pragma unroll
    for (int w = 0; w < CW; ++w)
#pragma unroll
        for (int l = 0; l < LOG_LPC; ++l) cnt[w] += (unsigned)sl_partner((int)cnt[w], l);
    auto count_of = [&](int bin) -> unsigned {
        if constexpr (NB == 2) return (cnt[0] >> (16 * bin)) & 0xFFFFu;
        const int byte = NB == 4 ? bin : (bin >> 1) & 3, word = NB == 4 ? 0 : 2 * (bin >> 3) + (bin & 1);
        const int at = WIDE ? 2 * word + (byte & 1) : word;
        // (masks instead of a choice: the compiler turns a choice among array elements into an indexed
        // read of a copy of the array in memory)
        unsigned v = 0;
#pragma unroll
        for (int w = 0; w < CW; ++w) v |= cnt[w] & (CW == 1 || at == w ? 0xFFFFFFFFu : 0u);
        return WIDE ? (v >> (16 * (byte >> 1))) & 0xFFFFu : (v >> (8 * byte)) & 0xFFu;
    };

    int bin0 = 0;                                // first bin that this lane ended up with
#pragma unroll
    for (int l = 0; l < BITS && l < LOG_LPC; ++l) bin0 += ((lane >> l) & 1) * (NB >> (l + 1));
    if (live && (sub >> BITS) == 0) {
#pragma unroll
        for (int i = 0; i < LEFT; ++i) {
            A.leafC[(long long)(bin0 + i) * A.n_chunks + c] = r[i];
            A.cnt[(long long)(bin0 + i) * A.n_chunks + c] = count_of(bin0 + i);
        }
    }
}

typedef void (*codes_kernel)(CodeArgs);

template <int BITS, bool SHORT>
codes_kernel codes_for(int log_lpc)
{
    static const codes_kernel table[7] = {k_codes<BITS, 0, SHORT>, k_codes<BITS, 1, SHORT>, k_codes<BITS, 2, SHORT>,
                                          k_codes<BITS, 3, SHORT>, k_codes<BITS, 4, SHORT>, k_codes<BITS, 5, SHORT>,
                                          k_codes<BITS, 6, SHORT>};
    return table[log_lpc];
}
template <bool SHORT>
codes_kernel codes_for(int bits, int log_lpc)
{
    return bits == 1 ? codes_for<1, SHORT>(log_lpc) : bits == 2 ? codes_for<2, SHORT>(log_lpc)
           : bits == 3 ? codes_for<3, SHORT>(log_lpc) : codes_for<4, SHORT>(log_lpc);
}

// ------------------------------------------------------------------ kernel D
// One workgroup per (tensor, bin): fixed-tree sum of the bin's leaves, integer count, centroid ->
// LUT[b] in the tensor block's header.  With the placement steps in these launches (PLACE) further
// workgroups take the last of them, `place_waves` groups each.
template <bool PLACE, bool PIECES>
__global__ void __launch_bounds__(RED_THREADS, 8)
k_tensor_lut(const SlTensorDev *tensors, int n_tensors, const double *leafC, const unsigned *cnt,
             long long n_chunks_total, int hdr_bytes, int rec_bytes, int nbins, unsigned char *payload,
             unsigned char *coded, int cfix, SlCodedArgs C, int place_waves, RedPieces P)
{
    __shared__ RedShared sh;
    extern __shared__ __align__(16) unsigned place_lds[];
    const int tid = threadIdx.x;
    const int b = blockIdx.y;
    if (PLACE && (int)blockIdx.x >= n_tensors) {
        const int wave = sl_uniform(tid >> 6);
        const long long gi = ((long long)((int)blockIdx.x - n_tensors) * nbins + b) * place_waves + wave;
        if (wave < place_waves && gi < C.n_groups) sl_coded_place(C, gi, place_lds + (size_t)wave * (SL_RICE_GROUP * C.G.ua + 1));
        return;
    }
    const SlTensorDev &td = tensors[blockIdx.x];             // (read again behind the sums: it would be kept in scratch memory across them)
    unsigned long long part = 0;
    const bool split = PIECES && P.split(td);
    const long long piece = b * P.stride + td.piece0;
    const unsigned *cb = split ? P.cnt + piece : cnt + b * n_chunks_total + td.chunk0;
    const long long counts = split ? (td.n_chunks + SL_PIECE - 1) / SL_PIECE : td.n_chunks;
    for (long long i = tid; i < counts; i += RED_THREADS) part += cb[i];
    if (64 * (tid >> 6) < counts) {                        // (a wave without chunks has nothing to add)
#pragma unroll
        for (int l = 0; l < 6; ++l) part += sl_partner(part, l);
    }
    if ((tid & 63) == 0) sh.cnt[tid >> 6] = part;
    double S[1];
    if (split) {                                                // (the barriers of both are behind the additions above)
        const double *const sums[1] = {P.sum + piece};
        block_piece_sums<1>(sums, td.n_chunks, sh, S);
    } else {
        const double *const leaf[1] = {leafC + b * n_chunks_total + td.chunk0};
        block_tree_sums<1>(leaf, td.n_chunks, sh, S);
    }
    const double Sb = S[0];
    unsigned long long nb = tid < RED_WAVES ? sh.cnt[tid] : 0ull;
    if (tid < 64) {
#pragma unroll
        for (int l = 0; l < 4; ++l) nb += sl_partner(nb, l);
    }
    if (tid == 0) {
        float cen = nb ? (float)(Sb / (double)nb) : 0.0f;
        if (cen == 0.0f) cen = 0.0f;        // never -0.0f on the wire
        reinterpret_cast<float *>(payload + td.pay_off)[b] = cen;
        if (coded) reinterpret_cast<float *>(coded + td.cblk_off)[b] = cen;
    }
    // zero the padding that rounds the header (two floats at 1 bit) and the tensor block up to 16 bytes
    if (b == 0 && tid >= nbins && 4 * tid < hdr_bytes) {
        reinterpret_cast<float *>(payload + td.pay_off)[tid] = 0.0f;
        if (coded) reinterpret_cast<float *>(coded + td.cblk_off)[tid] = 0.0f;
    }
    const long long used = hdr_bytes + td.n_chunks * (long long)rec_bytes;
    if (b == 0 && tid < td.block_bytes - used) payload[td.pay_off + used + tid] = 0;
    // the same table and padding in the coded buffer's block
    const long long cused = (td.cfix_off - td.cblk_off) + td.n_chunks * (long long)cfix;
    if (coded && b == 0 && tid < td.cblk_bytes - cused) coded[td.cblk_off + cused + tid] = 0;
}

// Unquantized values: there is no table, only the block padding is left to write.
__global__ void __launch_bounds__(64)
k_pad_blocks(const SlTensorDev *tensors, int rec_bytes, unsigned char *payload, unsigned char *coded, int cfix)
{
    const SlTensorDev td = tensors[blockIdx.x];
    const long long used = td.n_chunks * (long long)rec_bytes;
    if ((long long)threadIdx.x < td.block_bytes - used) payload[td.pay_off + used + threadIdx.x] = 0;
    const long long cused = (td.cfix_off - td.cblk_off) + td.n_chunks * (long long)cfix;
    if (coded && (long long)threadIdx.x < td.cblk_bytes - cused) coded[td.cblk_off + cused + threadIdx.x] = 0;
}

// ------------------------------------------------------------------ kernel E
struct ResidualArgs {
    const SlChunkDesc *desc;
    const float *vals;              // the selected values a, or null: read them from e
    const unsigned char *payload;
    float *e;
    long long n_chunks;
    int k, bits, hdr_bytes, rec_bytes;
};

__global__ void __launch_bounds__(256) k_residual(ResidualArgs A)
{
    const int lane = threadIdx.x & 63, k = A.k;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long c = (long long)blockIdx.x * (blockDim.x >> 6) + wave;
    if (c >= A.n_chunks) return;
    const SlChunkDesc d = A.desc[c];
    const float *lut = reinterpret_cast<const float *>(A.payload + sl_lut_off(d, A.hdr_bytes, A.rec_bytes));
    const unsigned char *rec = A.payload + d.rec_off;
    const unsigned char *codes = rec + 3 * k / 2;       // or the k fp32 values (4-byte aligned)
    float *ec = A.e + d.base;
    for (int m = lane; m < k; m += 64) {
        const int b = (3 * m) >> 1;
        const unsigned w = (unsigned)rec[b] | ((unsigned)rec[b + 1] << 8);
        const unsigned j = (m & 1) ? (w >> 4) : (w & 0xFFFu);
        const float q = A.bits == 32 ? reinterpret_cast<const float *>(codes)[m]
                                     : lut[sl_code_at(codes, m, A.bits)];
        float *dst = ec + ((j >> 6) * (unsigned)d.stride + (j & 63u));
        const float a = A.vals ? A.vals[c * k + m] : *dst;
        *dst = a - q;
    }
}

}  // namespace

static int check_launch()
{
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}

static int launch_residual(const sl_plan *p, float *e, const float *vals, const unsigned char *payload,
                           hipStream_t st)
{
    ResidualArgs R;
    R.desc = p->d_desc;
    R.vals = vals;
    R.payload = payload;
    R.e = e;
    R.k = p->k;
    R.bits = p->bits;
    R.hdr_bytes = p->hdr_bytes;
    R.rec_bytes = p->rec_bytes;
    R.n_chunks = p->n_chunks;
    const int wpb = 4;
    const unsigned nblk = (unsigned)((p->n_chunks + wpb - 1) / wpb);
    hipLaunchKernelGGL(k_residual, dim3(nblk), dim3(64 * wpb), 0, st, R);
    return check_launch();
}

int slk_residual(const sl_plan *p, float *e, const unsigned char *payload, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    return launch_residual(p, e, nullptr, payload, st);
}

// The coded format's placement steps share the launches of B, C and D up to so many (tensors x (bins + 4)): one or two
// launches are saved, but in D every tensor's workgroups pay for the registers and the LDS of the placement (tensors of 3
// chunks, k = 64, shared / launches of their own: 2 bits, 100 tensors 22.0 / 23.7 us, 300 34.5 / 33.6, 3000 201 / 171; 1 bit, 100 19.4 / 22.0,
// 300 30.6 / 30.2; 4 bits, 100 35.6 / 33.8, 500 94.6 / 76.6; tensors of 40 chunks, 2 bits, 300 130.0 / 130.5, 1000 374 / 367).
#ifndef SL_PLACE_SHARED_UPTO
#define SL_PLACE_SHARED_UPTO 2000
#endif

// Lists up to so many chunks whose tensors have at most SL_SHORT_TENSOR go without kernel B where no wave of the code kernel
// meets more than two tensors: it takes their statistics one after the other, about 1 us each, and the launch is
// worth 2 (sl_compress, kernel B / without, us: one wave among 164 with 2 tensors 21.2 / 20.9, with 3 21.2 / 21.7, 4 21.2 / 22.6, 8 21.3 / 26.4;
// every wave with 2, k = 64, 24.5 / 24.4, with 3 30.1 / 31.2; a run of 57 one-chunk tensors at k = 8 25.8 / 56.7; 3.4M elements in
// matrices of odd sides and their vectors, five in a wave, k = 32, 39.2 / 41.0; one tensor of 3 chunks 17.9 / 16.5).
#define SL_SHORT_LIST 8192
#define SL_SHORT_WAVE_TENSORS 2

int slk_quantize(const sl_plan *p, float *e, int skip_residual, unsigned char *payload, unsigned char *coded,
                 unsigned char *ws, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    const int k = p->k;
    const SlCodedArgs placing = sl_coded_args(p, coded, ws);     // (used only with `coded`)
    const bool shared = coded && p->bits != 32 && (long long)p->n_tensors * ((1 << p->bits) + 4) <= SL_PLACE_SHARED_UPTO;
    const float *vals = reinterpret_cast<const float *>(ws + p->ws_vals);
    double *leafA = reinterpret_cast<double *>(ws + p->ws_leafA);
    double *leafC = reinterpret_cast<double *>(ws + p->ws_leafC);
    unsigned *cnt = reinterpret_cast<unsigned *>(ws + p->ws_cnt);
    SlTensorStat *tstat = reinterpret_cast<SlTensorStat *>(ws + p->ws_tstat);
    int rc;

    if (p->bits == 32) {
        // nothing to quantize: kernel A wrote the values into the records
        hipLaunchKernelGGL(k_pad_blocks, dim3(p->n_tensors), dim3(64), 0, st, p->d_tensors, p->rec_bytes, payload, coded, p->cg.cfix);
        if ((rc = check_launch())) return rc;
        sl_prof_mark(p, SL_PROF_LUT, st);
        if (!skip_residual) {
            if ((rc = launch_residual(p, e, vals, payload, st))) return rc;
            sl_prof_mark(p, SL_PROF_RESIDUAL, st);
        }
        if (coded) {
            if ((rc = slk_coded_finish(p, coded, ws, st))) return rc;
            sl_prof_mark(p, SL_PROF_INDEX, st);
        }
        return SL_OK;
    }

    const int log_lpc = sl_code_lanes_log2(k);
    const bool few = p->max_tensor_chunks <= SL_SHORT_TENSOR && p->n_chunks <= SL_SHORT_LIST &&
                     p->max_wave_tensors <= SL_SHORT_WAVE_TENSORS;
    // Sums of pieces of large tensors: those of kernel A's leaves stand where C writes its own later, those of C's where A's have been.
    // (They fit: a split tensor has two hundred times as many chunks as pieces.)
    const bool split = p->n_pieces > 0;
    const long long stride = p->n_pieces;
    const RedPieces PB = {split ? leafC : nullptr, nullptr, stride};
    const RedPieces PD = {split ? leafA : nullptr, reinterpret_cast<unsigned *>(leafA + (stride << p->bits)), stride};
    const unsigned piece_blocks = (unsigned)((p->n_pieces + 3) / 4);
    const unsigned scan_blocks = shared ? (unsigned)sl_scan_blocks(p->n_groups) : 0;
    if (split) {
        hipLaunchKernelGGL(k_piece_sums, dim3(piece_blocks, 2), dim3(256), 0, st, p->d_pieces, leafA, nullptr, (long long)p->n_chunks, PB);
        if ((rc = check_launch())) return rc;
    }
    if (!few) {
        hipLaunchKernelGGL(split ? k_tensor_stats<true> : k_tensor_stats<false>, dim3(p->n_tensors + scan_blocks), dim3(RED_THREADS), 0, st, p->d_tensors, p->n_tensors, leafA,
                            (long long)p->n_chunks, k, tstat, placing, PB);
        if ((rc = check_launch())) return rc;
    }
    sl_prof_mark(p, SL_PROF_STATS, st);

    CodeArgs C;
    C.desc = p->d_desc;
    C.tstat = tstat;
    C.vals = vals;
    C.leafC = leafC;
    C.cnt = cnt;
    C.payload = payload;
    C.n_chunks = p->n_chunks;
    C.k = k;
    C.coded = coded;
    C.cdesc = p->d_cdesc;
    C.rem_bytes = p->cg.rem_bytes;
    C.passes = 1;
    while (512 * C.passes < k) C.passes <<= 1;
    const codes_kernel fn = few ? codes_for<true>(p->bits, log_lpc) : codes_for<false>(p->bits, log_lpc);
    const long long per_block = 4ll * (64 >> log_lpc);
    C.code_blocks = (unsigned)((p->n_chunks + per_block - 1) / per_block);
    C.leafA = leafA;
    C.tensors = p->d_tensors;
    C.C = placing;
    hipLaunchKernelGGL(fn, dim3(C.code_blocks + (few ? scan_blocks : 0)), dim3(256), 0, st, C);
    if ((rc = check_launch())) return rc;
    sl_prof_mark(p, SL_PROF_CODES, st);

    const int nbins = 1 << p->bits;
    if (split) {
        hipLaunchKernelGGL(k_piece_sums, dim3(piece_blocks, nbins), dim3(256), 0, st, p->d_pieces, leafC, cnt, (long long)p->n_chunks, PD);
        if ((rc = check_launch())) return rc;
    }
    const size_t per_wave_lds = sl_coded_place_words(p->cg) * sizeof(unsigned);
    const int place_waves = shared ? (int)std::max<size_t>(1, std::min<size_t>(RED_WAVES, 49152 / per_wave_lds)) : 0;
    const long long per_column = (long long)place_waves * nbins;      // groups that one column of workgroups takes
    const long long place_columns = shared ? (p->n_groups + per_column - 1) / per_column : 0;
    const auto lut = split ? (shared ? k_tensor_lut<true, true> : k_tensor_lut<false, true>) : (shared ? k_tensor_lut<true, false> : k_tensor_lut<false, false>);
    hipLaunchKernelGGL(lut, dim3((unsigned)(p->n_tensors + place_columns), nbins), dim3(RED_THREADS),
                       place_waves * per_wave_lds, st, p->d_tensors, p->n_tensors, leafC, cnt, (long long)p->n_chunks,
                       p->hdr_bytes, p->rec_bytes, nbins, payload, coded, p->cg.cfix, placing, place_waves, PD);
    if ((rc = check_launch())) return rc;
    sl_prof_mark(p, SL_PROF_LUT, st);

    if (!skip_residual) {
        if ((rc = launch_residual(p, e, vals, payload, st))) return rc;
        sl_prof_mark(p, SL_PROF_RESIDUAL, st);
    }
    if (coded && !shared) {
        if ((rc = slk_coded_finish(p, coded, ws, st))) return rc;
        sl_prof_mark(p, SL_PROF_INDEX, st);
    }
    return SL_OK;
}
