// Arguments of kernel A of sl_compress, shared by its two forms: a wavefront per chunk (sl_select_kernel.h) and, on short
// lists, a workgroup per chunk (sl_select_group.hip).
#pragma once
#include "sl_device.h"
#include "sl_internal.h"

#ifndef SL_SELECT_BOUND_BITS
#define SL_SELECT_BOUND_BITS 12   // bits of the pruning bound that are decided (0 = all)
#endif
struct SelectArgs {
    const SlChunkDesc *desc;
    float *e;
    const float *delta;             // the pseudo-gradient, or theta_outer when theta_local is set
    const float *theta_local;       // non-null: delta = theta_outer - theta_local, formed on the fly
    const unsigned char *pending;   // payload whose values are still to be subtracted from e
    float beta;
    int frozen;
    int k;
    int bits, hdr_bytes, rec_bytes; // value width of the payloads and the sizes that follow from it
    unsigned seed_hash;     // Random-k: fmix32(seed), see random_key
    int sample_margin;      // select_general: ranks of the sample's bracket, k / 8 -+ this (0: no sample)
    int pieces;             // Sub-k: whole 64-byte pieces are written back
    int lds_per_wave;
    int pend_off;           // offset of the pending-correction tables in a wave's LDS
    int pend_words;         // the pending record is staged in LDS as whole words (large k), see pend_half
    float *vals;            // [n_chunks * k] selected values, canonical order
    double *leafA;          // [2][n_chunks] per-chunk tree sums of x and x*x
    unsigned char *payload;
    long long n_chunks;
    unsigned order;          // sl_work_group
    // coded wire format written next to the plain record (null: not wanted): the remainder fields go
    // to their place in the buffer, the chunk's quotient bit vector and quotient sum to the workspace
    unsigned char *coded;
    const SlCodedDesc *cdesc;
    SlCodedGeom G;
    unsigned *uvec;
    unsigned short *qsum;
};

SL_DEV int key_of(float x) { return (int)(__float_as_uint(x) & 0x7FFFFFFFu); }

// Waves per chunk: several on lists so short that the chain of a wave's instructions is longer than the stream, one where the
// compute units are full without.  The work that each wave of a chunk repeats grows with k, so the line falls.  sl_compress_coded /
// sl_compress, full chunks, one wave and the number taken here, us: 64 chunks, k = 32 20.0 -> 15.7 / 20.0 -> 16.8; 256, k = 64
// 21.4 -> 17.3 / 21.9 -> 18.7, k = 1024 55.9 -> 37.8 / 46.2 -> 34.3; 512, k = 256 30.8 -> 26.2 / 31.1 -> 28.9; 1024, k = 64 28.0 -> 24.2 /
// 30.0 -> 27.6, k = 1024 63.1 -> 49.7 / 61.5 -> 50.7; 2048, k = 128 42.9 -> 40.6 / 48.2 -> 43.4, k = 256 48.0 -> 48.1 / 54.1 -> 51.0; 4096, k = 64
// 56.7 -> 55.3 / 65.3 -> 60.4; beyond the lines 4096, k = 256 64.9 -> 69.5 / 79.2 -> 79.7; 1024, k = 512 43.0 -> 41.5 / 43.7 -> 46.0; 8192, k = 64
// 94.5 -> 94.6 / 108.2 -> 105.9, k = 128 96.8 -> 99.6; 5120, k = 1024 124 -> 135.  Eight waves against four: 256, k = 64 18.0 -> 17.3; 512 20.7 ->
// 20.4; 768 23.1 -> 23.8.  Partial chunks gain more, their loads do not come row by row here: 900 chunks of 530 columns, k = 32
// 37.4 -> 27.3; 1155 of 67, k = 64 55.4 -> 30.3.
inline int sl_select_waves(int64_t n_chunks, int k)
{
    if (n_chunks <= 512) return 8;
    return n_chunks <= (k <= 128 ? 6144 : k <= 256 ? 2048 : k <= 512 ? 768 : 3072) ? 4 : 1;
}

// The workgroup-per-chunk form (sl_select_group.hip), `waves` 4 or 8, `keep`: without the streaming hint; A as for the other one but for the LDS.
int slk_select_group(const SelectArgs &A, bool sub_only, int waves, bool keep, hipStream_t st);

// The wave-per-chunk form without the streaming hint (sl_select_kept.hip).
void (*sl_select_kept(int k, bool two_bit, bool params))(SelectArgs);
