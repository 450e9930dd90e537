// Internal structures shared by the host API and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sparseloco.h"

// One 4096-element chunk seen as a 64-row view: element (row, col) of the view
// is arena[base + row*stride + col].  A FLAT chunk is the view with stride 64.
// `rows` valid rows; every valid row has `cols` valid columns except the last
// valid row, which has `last_cols`.  Everything a kernel needs to know about a
// chunk comes with one 32-byte scalar load.
struct SlChunkDesc {
    long long base;
    int stride;
    unsigned char rows, cols, last_cols, flags;
    long long rec_off;      // byte offset of the chunk's record inside a payload
    int tensor;             // index of the tensor in the list
    int local_chunk;        // index of the chunk inside its tensor
};
static_assert(sizeof(SlChunkDesc) == 32, "descriptor is one 32-byte load");
enum { SLC_FULL = 1 };   // all 4096 positions valid (rows need not be 16-byte aligned)

struct SlTensorDev {
    long long chunk0;       // first chunk of the tensor in list order
    long long n_chunks;
    long long pay_off;      // byte offset of the tensor's block in a payload
    long long block_bytes;  // align16(16 + n_chunks * record_bytes)
    long long group0;       // first directory group (16 chunks) of the tensor, list order
    // coded format: byte offsets inside a coded buffer of the tensor's block (table header first),
    // of its directory and of its first fixed record; size of the block
    long long cblk_off, cdir_off, cfix_off, cblk_bytes;
    long long piece0;       // first of its pieces (SlPiece), -1 where its leaves are summed without
};

enum { SL_RICE_GROUP = 16 };  // chunks per directory entry of the coded format

// Where a chunk's parts lie in a coded buffer (byte offsets that follow from the tensor list):
// what the coded aggregate needs about a chunk besides its SlChunkDesc, in one 32-byte load.
struct SlCodedDesc {
    long long lut_off;      // table header of the chunk's tensor block
    long long dir_off;      // directory entry of the chunk's group
    long long fix_off;      // the chunk's fixed record
    int pos;                // position of the chunk in its group, 0..15
    int reserved;
};
static_assert(sizeof(SlCodedDesc) == 32, "descriptor is one 32-byte load");

// Sizes of the coded format that follow from k and the value width (see sl_coded.h).
struct SlCodedGeom {
    int k, bits;
    int b;                  // Rice parameter
    int qmax;               // largest possible sum of a chunk's quotients, (4096 - k) >> b
    int qf;                 // bytes of a quotient-sum field in the directory: 1 or 2
    int dent;               // bytes of a directory entry: 4 + 16 * qf
    int rem_bytes;          // the k remainders, padded to 4 bytes
    int val_bytes;          // the k value fields: k * bits / 8
    int cfix;               // fixed record: rem_bytes + val_bytes padded to 4
    int hdr;                // table header of a tensor block
    int ua;                 // words of a chunk's longest bit vector: ceil((k + qmax) / 32)
    long long section;      // byte offset of the quotient section (end of the last block)
};

struct SlGroup {            // one coding group of the index coder
    int tensor;
    int local_group;
    int chunk0, n_chunks;   // its chunks, list order
};

struct SlPiece {            // so many leaves of a tensor that are summed up by a wave of their own (k_piece_sums)
    int chunk0, n_chunks;   // its chunks, list order
};
enum { SL_PIECE = 256 };
// The pieces of the tensors of more than SL_SPLIT_TENSOR chunks, and each tensor's first one.
#define SL_SPLIT_TENSOR 10240
template <class Tensors, class Pieces>
inline void sl_make_pieces(Tensors &tensors, Pieces &pieces)
{
    for (SlTensorDev &t : tensors) {
        const bool split = t.n_chunks > SL_SPLIT_TENSOR;
        t.piece0 = split ? (long long)pieces.size() : -1;
        for (long long c = 0; split && c < t.n_chunks; c += SL_PIECE)
            pieces.push_back(SlPiece{(int)(t.chunk0 + c), (int)(t.n_chunks - c < SL_PIECE ? t.n_chunks - c : SL_PIECE)});
    }
}

// Per-tensor quantizer state produced during sl_compress.
struct SlTensorStat {
    double mu;      // mean of the selected values
    double var;     // their population variance (bin edges sit at multiples of sigma)
};
static_assert(sizeof(SlTensorStat) == 16, "");

// Sizes of the wire format for `bits` value bits (1..4, or 32 = unquantized
// fp32 values): look-up table header of a tensor block and one chunk record.
__host__ __device__ inline int sl_hdr_bytes(int bits)
{
    return bits == 32 ? 0 : ((4 << bits) < 16 ? 16 : (4 << bits));
}
__host__ __device__ inline int sl_rec_bytes(int k, int bits) { return 3 * k / 2 + k * bits / 8; }

// Code of entry m in a little-endian stream of `bits`-wide fields (bits <= 4).
__host__ __device__ inline unsigned sl_code_at(const unsigned char *codes, int m, int bits)
{
    const int bit = m * bits, sh = bit & 7;
    unsigned w = codes[bit >> 3];
    if (sh + bits > 8) w |= (unsigned)codes[(bit >> 3) + 1] << 8;
    return (w >> sh) & ((1u << bits) - 1u);
}

struct sl_plan {
    int k;
    int bits;                   // value bits: 1..4, or 32 for unquantized fp32 values
    int rec_bytes, hdr_bytes;   // sl_rec_bytes(k, bits), sl_hdr_bytes(bits)
    int n_tensors;
    int device;
    int max_lds;                // largest LDS allocation of one workgroup, bytes
    int64_t n_chunks;
    int64_t n_elements;
    int64_t n_partial;          // chunks without SLC_FULL
    int64_t n_unaligned;        // chunks whose rows do not all begin on a multiple of 16 elements
    int64_t max_tensor_chunks;  // chunks of the tensor that has most
    int max_wave_tensors;       // tensors that a wave of the code kernel meets among its chunks, at most
    size_t payload_bytes;
    size_t ws_bytes;
    // workspace sections (byte offsets)
    size_t ws_vals, ws_leafA, ws_leafC, ws_cnt, ws_tstat;
    // device tables
    SlChunkDesc *d_desc;
    SlCodedDesc *d_cdesc;
    SlTensorDev *d_tensors;
    SlGroup *d_groups;
    int64_t n_groups;
    SlPiece *d_pieces;
    int64_t n_pieces;
    size_t rice_max_bytes;      // upper bound of a coded buffer, 0 when the list is beyond the coded format
    SlCodedGeom cg;
    // workspace sections of the coded path: per-chunk bit vectors (cg.ua words each) and quotient
    // sums, per-group run lengths (words) and offsets in a block of groups (words)
    size_t ws_uvec, ws_qsum, ws_gwords, ws_goff;
    // host copies
    SlTensorDev *h_tensors;
    // optional per-kernel timing (sl_profile_begin / sl_profile_end)
    struct SlProfile *prof;
};

// log2 of the lanes that the code kernel gives to a chunk, eight entries each; a wave takes 64 >> this consecutive chunks.
inline int sl_code_lanes_log2(int k)
{
    int l = 0;
    while (l < 6 && (8 << l) < k) ++l;
    return l;
}

// Byte offset of the LUT header of the chunk's tensor block inside a payload.
__host__ __device__ inline long long sl_lut_off(const SlChunkDesc &d, int hdr_bytes, int rec_bytes)
{
    return d.rec_off - hdr_bytes - (long long)d.local_chunk * rec_bytes;
}

// Chunks (waves) per workgroup of the aggregates, and of the selection up to k = 128, with a wave per chunk: four adjacent ones, so that a workgroup streams
// 1 KB of every matrix row it touches; but one on lists so short that workgroups of four, dealt to the compute units in one turn or two,
// would leave a third of the places without any.  Four / one, us, one call on buffers that no cache holds (768-column matrices): plain, k = 512, R = 4
// 504 chunks 11.7 / 11.1, 1020 13.2 / 13.0, 1536 15.0 / 15.6, 2040 17.3 / 18.1, 4092 33.2 / 34.4; k = 64, R = 16 504 12.2 / 11.9, 2040 16.8 / 17.3, 4092 32.4 / 34.2; coded, k =
// 256, R = 4 504 12.3 / 11.6, 1272 15.2 / 15.0, 3072 25.5 / 25.6.  Sub-k, k = 64 1360 18.4 / 18.0, k = 16 15.7 / 15.5 (1024 columns 19.7 / 18.3, 17.0 / 15.5).  (Rows of 1024 columns want one up to 3072 chunks, plain, k = 64, R = 16 1024 16.7 / 13.7, 2048 22.1 /
// 17.2; those of 64, 1088 and 2048 do not.)  Not where one chunk in 32 or more is partial: rows then begin anywhere in a line of memory, and the neighbours
// that share a line should share an L2 (coded, k = 64, R = 8, 594 chunks of a 530-column matrix 17.5 / 18.7; plain, k = 256, 1024 of 1001 columns 19.3 / 21.3).
#define SL_COMPUTE_UNITS 256
inline int sl_chunks_per_group(const sl_plan *p)
{
    const int64_t groups = (p->n_chunks + 3) / 4, turns = (groups + SL_COMPUTE_UNITS - 1) / SL_COMPUTE_UNITS;
    return turns <= 2 && 3 * groups <= 2 * SL_COMPUTE_UNITS * turns && p->n_partial * 32 < p->n_chunks ? 1 : 4;
}

#define SL_DENSE_SHORT_BELOW 5120         // see k_dense_avg_apply

// Do the accesses of this list go without the streaming hint (sl_access_load)?  Unaligned rows lose up to half with it, aligned ones a tenth
// without, so it is a matter of their share, `percent` of the chunks at least.  On buffers that no cache holds, rows of 1001 columns among aligned ones, with
// the hint / without, us: aggregates (k = 64, R = 4) 1920 chunks, 25 % 18.4 / 20.1, 50 % 19.7 / 20.3, 75 % 20.7 / 20.3; 9600, 15 % 62.8 / 65.3, 25 % 66.5 / 66.5, 35 %
// 69.7 / 66.9, 25,600, 25 % 171 / 160; with momentum 1920, 35 % 32.9 / 34.2, 50 % 34.6 / 34.3, 5120, 25 % 76.4 / 76.2, 35 % 79.8 / 76.8.  Dense streams: direction 5120, 25 % 76.7 / 79.8, 35 % 79.9 / 80.7, 50 % 84.3 /
// 82.6; average of four 9600, 25 % 185 / 192, 35 % 188 / 190, 50 % 194 / 188.  (Arenas that do not begin on 64 bytes are not looked at.)
inline bool sl_rows_unaligned(const sl_plan *p, int percent) { return 100 * p->n_unaligned >= percent * p->n_chunks; }
inline int sl_apply_kept_from(const sl_plan *p, bool mom) { return p->n_chunks > (mom ? 4096 : 8192) ? 25 : 50; }     // aggregates
inline int sl_dense_kept_from(const sl_plan *p) { return p->n_chunks < SL_DENSE_SHORT_BELOW ? 25 : 40; }              // dense average
#define SL_DIRECTION_KEPT_FROM 40

// The same for the accumulate (`streams` as for sl_select_waves; none gains that only reads: frozen, 25,600 chunks, all unaligned, k = 32 136 / 140, 12,800 79.2 / 78.4):
// deferred, k = 128 2560 chunks, 25 % 48.5 / 50.9, 50 % 50.9 / 51.4, 75 % 51.9 / 51.4; 9600, 25 % 120 / 122, 50 % 124 / 123, 75 % 133 / 127; k = 64 25,600, 25 % 272 / 283,
// 50 % 289 / 277, 75 % 307 / 283.  Where the update follows, k = 64 9600, 25 % 140 / 147, 75 % 155 / 146, 25,600, 25 % 330 / 371, 75 % 361 / 363, all 374 / 362; k = 512 5120, 25 % 132 /
// 120, 9600, 25 % 225 / 197, 12,160, 25 % 265 / 251, 16,000, 75 % 384 / 358, 25,600, 25 % 551 / 580, 50 % 520 / 583, 75 % 609 / 591, all 643 / 628; from parameters k = 64 25,600, 25 %
// 405 / 459, 75 % 465 / 457; k = 512 9600, 25 % 231 / 235, 75 % 252 / 242.
inline bool sl_select_unaligned(const sl_plan *p, int streams, bool update_follows, bool params)
{
    if (streams == 1) return false;
    if (update_follows && p->n_chunks > 12288) return sl_rows_unaligned(p, 75);
    return sl_rows_unaligned(p, update_follows && !params && p->k > 256 && p->k <= 1536 ? 25 : 50);
}

// Waves per chunk of kernel A: several (sl_select_group.hip) on lists so short that the chain of a wave's instructions is longer than the
// stream, one where the compute units are full without.  The work that each wave of a chunk repeats grows with k, and the less a call moves
// the sooner one wave is enough: `streams` is 1 where it reads one arena and writes none or single entries (error feedback frozen, Sub-k), 2 for the
// accumulate with the error update deferred, 3 where the update follows or the pseudo-gradient is formed from parameters.  A workgroup per chunk goes in turns over
// the compute units, so the lines lie at multiples of 256.  One wave / several, us, one call on buffers that no cache holds, full chunks of 1024 columns, of 768:
// frozen k = 64 512 18.5 / 17.0, 1280 32.9 / 30.2, 32.4 / 30.3, 1360 32.9 / 34.0, 32.8 / 34.0; k = 136 1280 35.8 / 33.7, 34.8 / 33.7; k = 256 768 31.0 / 29.4, 31.4 / 29.4; k = 264 768
// 35.7 / 31.7, 35.2 / 31.6; k = 1024 1280 54.2 / 51.8, 53.2 / 51.8, 1536 55.0 / 54.3, 54.0 / 54.1, 1792 56.6 / 57.6, 55.8 / 57.0; Sub-k k = 64 1280 19.4 / 16.1, 18.2 / 16.1, 1360
// 19.7 / 19.3, 18.4 / 18.3, 2048 22.2 / 22.6, 21.0 / 22.1; k = 256 768 20.1 / 18.8, 19.4 / 18.9, 896 20.6 / 20.6, 20.0 / 20.8; k = 512 768 25.3 / 23.8, 24.8 / 24.2; k = 1024 1280 37.1 / 36.2,
// 37.4 / 36.1, 1536 38.4 / 38.5.  Deferred k = 136 1536 45.5 / 42.8, 43.8 / 42.7, 1792 48.0 / 45.7, 44.8 / 46.2; k = 256 1280 46.4 / 39.8, 43.4 / 40.0, 1536 46.8 / 45.4, 44.2 / 45.6;
// k = 1024 2304 79.5 / 70.8, 73.7 / 71.2, 2560 80.3 / 75.0, 74.6 / 74.1, 2816 83.7 / 77.9, 76.1 / 77.7.  Matrices of 64 rows: deferred, k = 64 256 21.1 / 16.7, 1024 25.1 / 24.1, 2048 34.0 / 34.7,
// 6144 70.4 / 69.0 (1024 columns 2048 41.2 / 36.3, 6144 77.6 / 72.9); k = 512 1024 33.0 / 34.3; with the update k = 64 512 26.6 / 23.1, 2048 44.6 / 41.5, 6144 94.4 / 88.7, k = 256 2048 55.2 / 54.1, k = 512 768
// 41.5 / 41.1, 1536 54.7 / 58.0, k = 1024 2048 82.1 / 77.2, 3072 100.1 / 99.1.  Eight waves against four (deferred, k = 64): 256 chunks 16.9 -> 16.1, 512 18.8 -> 19.0, 768 20.8 -> 21.3.
// Above k = 1928 the LDS of a compute unit holds two workgroups of the one-wave form, not three, which a list of 2049 chunks and more feels: frozen, k = 2048 2048 chunks
// 64.2 / 66.6, 2220 87.1 / 74.9, Sub-k 2880 62.2 / 56.3.  Lists with partial chunks (`ragged`: one chunk in 32 or more) gain whatever the call reads, narrow tiles most: columns 200, frozen, k = 256 780 49.6 / 30.6, Sub-k
// 916 37.2 / 20.7, deferred, k = 200 1360 61.0 / 45.5; columns 1001, frozen, k = 32 3120 40.5 / 37.5; 900 of 530 columns, k = 32 37.4 / 27.3; 1155 of 67, k = 64 55.4 / 30.3.
inline int sl_select_waves(int64_t n_chunks, int k, int streams, bool ragged)
{
    if (n_chunks <= 512) return 8;
    int64_t upto = k <= 128 ? 6144 : k <= 256 ? 2048 : k <= 512 ? 768 : 3072;
    if (!ragged && k <= 1928) {
        if (streams == 1) upto = k <= 160 || k > 512 ? 1280 : 768;
        else if (streams == 2) upto = k <= 128 ? 6144 : k <= 256 ? 1536 : k <= 512 ? 768 : 2560;
    }
    return n_chunks <= upto ? 4 : 1;
}

// Does the accumulate leave the streaming hint out because the error update follows, which writes at the selected places?  It pays where
// those are many and the buffer is still in the caches then, and fits them beside the pseudo-gradient; it costs the accumulate what the hint is worth, most where
// little is selected.  sl_compress on buffers that no cache holds before the call, with the hint / without, us: k = 16 4096 chunks 57.9 / 63.7, k = 64 64.0 / 67.8,
// k = 256 79.2 / 81.6, k = 512 3072 79.9 / 80.7, 4096 99.8 / 97.8, 6144 144 / 132, 9216 201 / 185, 10,240 199 / 203, k = 1024 4096 129 / 126, 9216 237 / 218, k = 1536 8192 222 / 209, k = 2048
// 6144 206 / 208; fp32 values, k = 512 6144 131 / 113; from parameters k = 512 4096 102 / 107, k = 1024 9216 238 / 245.  (Called again on the same buffers it pays
// at every k, as the next call then finds them in the caches: 4096, k = 64 62.0 / 53.3.  A training step between two calls leaves nothing there.)
inline bool sl_update_kept(int64_t n_chunks, int k, bool params)
{
    return !params && k > 256 && k <= 1536 && n_chunks >= 4096 && n_chunks <= 9216;
}

// Does Sub-k write whole 64-byte pieces back?  Where the caches do not hold the buffer, a write of four bytes costs the memory a read and a write of its piece;
// with few of them looking at every piece costs more.  Single entries / pieces, us, buffers that no cache holds: k = 4 16,384 chunks 51.8 / 55.3, 49,152 147 / 152, k = 8 16,384 56.9 / 58.8,
// 49,152 159 / 162, k = 16 16,384 64.1 / 63.4, 49,152 177 / 172, k = 64 12,288 64.7 / 58.5, 16,384 84.1 / 74.2, 49,152 258 / 195, k = 128 49,152 348 / 220, k = 512 16,384 167 / 117, 49,152 496 / 311.
// (Just written before the call: k = 64 12,288 54.6 / 60.4, 16,384 73.8 / 76.2, 20,480 94.7 / 91.6.)
inline bool sl_subk_pieces(int64_t n_chunks, int k) { return k >= 16 && n_chunks >= 16384; }

// Waves per chunk of the aggregates: several (sl_apply_group.hip) on short lists with few workers, one else.  With a wave per worker
// and a list of entries for each the work grows with R, and with k, where the other routes' does less.  One wave and the number taken
// here, us, one call on buffers that no cache holds, full chunks of 1024-column matrices, lr update: plain, k = 64, R = 4 64 chunks 8.6 -> 7.2, 512 9.7 -> 8.7,
// 1024 14.4 -> 10.6, 2048 21.8 -> 17.6; R = 8 256 9.1 -> 8.8, 1024 15.1 -> 12.1, 2048 22.0 -> 20.5; k = 200, R = 8 512 22.3 -> 11.1; k = 256, R = 4 256 9.9 -> 10.0, 512 11.0 ->
// 10.8, 1024 15.4 -> 12.9, R = 8 512 11.9 -> 11.8, with momentum 1024 25.1 -> 21.8, 4 bits 19.6 -> 17.1, fp32 values 23.5 -> 15.6; coded, k = 64, R = 4 256 11.6 -> 10.2, 1024
// 16.2 -> 13.6, R = 8 256 12.1 -> 10.9; k = 128, R = 4 1024 16.5 -> 14.5.  Beyond the lines: plain, k = 256, two bits (one wave decodes eight entries a lane), R =
// 5 768 14.0 -> 14.8, R = 8 1024 16.3 -> 17.0 (1001 columns 19.2 -> 21.3); k = 512, R = 3 256 10.0 -> 12.9; k = 16, R = 16 512 11.5 -> 12.0; k = 64, R = 8 4096 30.6 -> 32.9; coded, k = 64, R = 8
// 1280 15.4 -> 17.4, k = 128, R = 8 512 12.2 -> 13.3; k = 256, R = 4 256 11.0 -> 12.8.  (Called again and again in a graph, everything in the caches, k = 64, R = 4: 512 chunks 5.1 -> 4.5,
// 1024 9.0 -> 5.8, 2048 16.9 -> 13.6.)
inline int sl_apply_waves(const sl_plan *p, int R, bool coded, bool mom)
{
    const int64_t n = p->n_chunks;
    const int k = p->k;
    if (coded) return k > 128 ? 1 : n <= 256 && R <= 8 ? 8 : n <= 1024 && R <= 4 ? 4 : 1;
    if (k > 256 || R > 8) return 1;
    if (n <= 512) return 8;
    if (k == 256 && p->bits == 2 && R > 4 && !mom) return 1;
    if (n <= 1024) return 4;
    return R * k <= 1024 && n <= (p->n_partial * 32 >= n ? 1280 : 2048) ? 4 : 1;
}

// sl_work_group's `order` for a grid of so many groups.  Where a list has many partial chunks - the last column of a
// matrix's tiles: one group in every few - the slow groups would all come to one or two of the XCDs, so the groups
// are turned (columns 1000 and 2730, a chunk in 25 partial, plain aggregate of 8: list order 475, paired 488, turned 471 us;
// on full chunks the turn costs up to 3 %).
#define SL_ORDER_WINDOW 1024u             // groups of a window: whole windows only are walked in another order than the list's
static_assert((SL_ORDER_WINDOW & (SL_ORDER_WINDOW - 1)) == 0 && SL_ORDER_WINDOW >= 8, "sl_work_group permutes halves and fours");
inline unsigned sl_order(const sl_plan *p, unsigned groups)
{
    const unsigned whole = p->n_chunks < 4 * SL_ORDER_WINDOW ? 0u : groups & ~(SL_ORDER_WINDOW - 1);
    return whole | (whole && p->n_partial * 32 >= p->n_chunks ? 1u : 0u);
}

// Where a lane's 16-byte loads of a partial chunk begin (sl_load_partial; access i: elements lc .. lc + 3 of row 4 i + lr).
// A lane whose four columns exist loads them; one that the row's end cuts through loads the four elements that
// end there, begun up to three earlier; one without elements the chunk's first four (a chunk holds at least that many).  Elements
// before a row's first belong to the tensor too - another row or chunk - but for its first row's, so in a tensor's first
// chunk no load begins before that chunk: memory outside the tensors is the caller's.
// (Functions of plain values: the same arithmetic as methods of a struct led to other registers in the aggregates' full chunks; 510M
// list, coded aggregate, us, so / with the struct: k = 256, R = 16 1172 / 1197, k = 128, R = 16 772 / 804, k = 64, R = 32 1042 / 1069.)
#define SL_HD __host__ __device__ __attribute__((always_inline)) inline
// elements before the chunk that a load may begin at
SL_HD int sl_partial_room(const SlChunkDesc &d) { return d.local_chunk ? 4 : 0; }
// how many of access i's four elements exist (none below 1)
SL_HD int sl_partial_exist(const SlChunkDesc &d, int lr, int lc, int i)
{
    const int row = 4 * i + lr;
    return (row < d.rows - 1 ? d.cols : row == d.rows - 1 ? d.last_cols : 0) - lc;
}
// bytes from `room` elements before the chunk to access 0; 16 * stride more for each further one
SL_HD unsigned sl_partial_origin(const SlChunkDesc &d, int lr, int lc, int room)
{
    return 4u * ((unsigned)lr * (unsigned)d.stride + (unsigned)(lc + room));
}
// elements between the first of the load and the first of the access at `place`, 1 <= exist <= 3
SL_HD int sl_partial_back(int exist, unsigned place)
{
    const int n = 4 - exist, m = (int)(place >> 2);
    return n < m ? n : m;
}
// where the load begins
SL_HD unsigned sl_partial_load_at(int exist, unsigned place, int room)
{
    return exist >= 4 ? place : exist > 0 ? place - 4u * (unsigned)sl_partial_back(exist, place) : 4u * (unsigned)room;
}

// Records an event after the kernel of `phase` (phase < 0: start of a call).
void sl_prof_mark(const sl_plan *p, int phase, hipStream_t st);

// sl_compress and its variants behind one argument check (sl_api.hip)
// (coded != null: the coded wire format is written as well, `coded_capacity` bytes available)
int sl_compress_impl(sl_plan *p, float *e, const float *delta, const float *theta_local, float beta,
                     int flags, const void *pending, void *payload, void *workspace, void *stream,
                     bool random = false, unsigned seed = 0u, void *coded = nullptr, size_t coded_capacity = 0);

// device address of the library's own scratch array on `device` (the current device), sl_noalloc.hip
int sl_noalloc_scratch(int device, void **out);

// launchers (defined next to their kernels)
int slk_select(const sl_plan *p, float *e, const float *delta, const float *theta_local, float beta,
               int frozen, const unsigned char *pending, unsigned char *payload, unsigned char *coded,
               unsigned char *ws, bool update_follows, hipStream_t st);       // update_follows: slk_quantize takes step E
// the same with Random-k in place of Top-k
int slk_select_random(const sl_plan *p, float *e, const float *delta, float beta, int frozen,
                      const unsigned char *pending, unsigned char *payload, unsigned char *ws, unsigned seed,
                      hipStream_t st);
// B, C, D and (unless skip_residual) E; with `coded` also the placement steps of the coded buffer
int slk_quantize(const sl_plan *p, float *e, int skip_residual, unsigned char *payload, unsigned char *coded,
                 unsigned char *ws, hipStream_t st);
// E on its own: e[idx] -= LUT[code] for the entries of `payload`
int slk_residual(const sl_plan *p, float *e, const unsigned char *payload, hipStream_t st);
// mom != null: DiLoCo's global Nesterov momentum on top of the aggregate
int slk_apply(const sl_plan *p, float *theta, float *mom, float mu, const void *const *payloads, int R,
              float lr, hipStream_t st);
// dense outer steps of the DiLoCo family (sl_outer.hip) and Sub-k (sl_select.hip)
int slk_lom_direction(const sl_plan *p, float *m, const float *delta, float mu, float *dir, hipStream_t st);
int slk_dense_avg_apply(const sl_plan *p, float *theta, float *mom, const float *const *dirs, int R, float lr,
                        float mu, hipStream_t st);
int slk_sub_topk(const sl_plan *p, float *m, hipStream_t st);
int slk_validate(const sl_plan *p, const unsigned char *payload, int *flag, hipStream_t st);
int slk_pack(const uint16_t *idx, const uint8_t *codes, int64_t n_chunks, int k, unsigned char *out,
             hipStream_t st);
int slk_pack_bits(const uint16_t *idx, const uint8_t *codes, const float *values, int64_t n_chunks, int k,
                  int bits, unsigned char *out, hipStream_t st);
int slk_rice_encode(const sl_plan *p, const unsigned char *payload, unsigned char *out,
                    unsigned char *ws, hipStream_t st);
int slk_rice_decode(const sl_plan *p, const unsigned char *in, size_t in_bytes, unsigned char *payload, hipStream_t st);
// coded wire format: the steps that place the quotient bit vectors once a buffer's writers have run
int slk_coded_finish(const sl_plan *p, unsigned char *out, unsigned char *ws, hipStream_t st);
// theta update from R coded payloads (mom != null: with the global momentum)
int slk_apply_coded(const sl_plan *p, float *theta, float *mom, float mu, const void *const *payloads, const size_t *bytes,
                    int R, float lr, hipStream_t st);
// either of them with several waves per chunk (bytes != null: coded payloads)
int slk_apply_group(const sl_plan *p, float *theta, float *mom, float mu, const void *const *payloads, const size_t *bytes, int R, float lr,
                    int waves, hipStream_t st);
int sl_rice_param(int k);
void sl_note_hip_error(hipError_t e);
