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

// The workgroup-per-chunk form (sl_select_group.hip), `waves` 4 or 8, `keep`: without the streaming hint; A as for the other one but for the LDS.
int slk_select_group(const SelectArgs &A, bool sub_only, int waves, bool keep, hipStream_t st);

// The wave-per-chunk form without the streaming hint (sl_select_kept.hip).
void (*sl_select_kept(int k, bool two_bit, bool params))(SelectArgs);
