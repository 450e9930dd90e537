// Launches of kernel A of sl_compress in its different forms: a wave per chunk (sl_select_kernel.h), several waves per chunk
// on short lists (sl_select_group.hip), Random-k and Sub-k.
#include <cmath>

#include "sl_select_kernel.h"

static unsigned host_fmix32(unsigned h)
{
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

static int launch_select(const sl_plan *p, float *e, const float *delta, const float *theta_local, float beta,
                         int frozen, const unsigned char *pending, unsigned char *payload, unsigned char *coded,
                         unsigned char *ws, bool update_follows, bool sub_only, bool random, unsigned seed, hipStream_t st)
{
    if (p->n_chunks == 0) return SL_OK;
    const int k = p->k;
    const bool pruned = k <= 512;
    SelectArgs A;
    A.desc = p->d_desc;
    A.e = e;
    A.delta = delta;
    A.theta_local = theta_local;
    A.pending = pending;
    A.beta = beta;
    A.frozen = frozen;
    A.k = k;
    A.bits = p->bits;
    A.hdr_bytes = p->hdr_bytes;
    A.rec_bytes = p->rec_bytes;
    A.seed_hash = host_fmix32(seed);
    {
        const double share = (double)k / SL_CHUNK;
        const int margin = (int)(2.5 * std::sqrt(512.0 * share * (1.0 - share))) + 1;
        A.sample_margin = k > 512 && p->n_chunks >= SL_SAMPLE_FROM && k / 8 + margin < 511 ? margin : 0;
    }
    {
        size_t b = pruned ? sizeof(uint2) * cand_cap(k > 256 ? 16 : 8) : sizeof(int) * SL_SELECT_LIST_CAP;
        // (the coded form's bit vector and remainder words reuse this first part: at most 128 + 64 words)
        b += (6 * (size_t)k + 7) & ~(size_t)7;
        b = (b + 15) & ~(size_t)15;
        // k > 256: a pending record of whole words and whole groups of eight entries is staged in LDS
        A.pend_words = pending && k > 256 && (p->rec_bytes & 3) == 0 && (k & 7) == 0 && p->rec_bytes <= 8192;
        // the pending tables are dead before the selection starts: they share its LDS
        A.pend_off = 0;
        if (pending) {
            const size_t pb = (SL_CHUNK / 2) * sizeof(float) + 16 * sizeof(float) +
                              (A.pend_words ? (size_t)p->rec_bytes : 0);
            if (b < pb) b = pb;
        }
        A.lds_per_wave = (int)((b + 15) & ~(size_t)15);
    }
    A.pieces = sub_only && sl_subk_pieces(p->n_chunks, k);
    A.vals = sub_only ? nullptr : reinterpret_cast<float *>(ws + p->ws_vals);
    A.leafA = sub_only ? nullptr : reinterpret_cast<double *>(ws + p->ws_leafA);
    A.payload = payload;
    A.n_chunks = p->n_chunks;
    A.coded = sub_only ? nullptr : coded;
    A.cdesc = p->d_cdesc;
    A.G = p->cg;
    A.uvec = (sub_only || !coded) ? nullptr : reinterpret_cast<unsigned *>(ws + p->ws_uvec);
    A.qsum = (sub_only || !coded) ? nullptr : reinterpret_cast<unsigned short *>(ws + p->ws_qsum);
    const int streams = sub_only || frozen ? 1 : update_follows || theta_local ? 3 : 2;
    const int waves = random ? 1 : sl_select_waves(p->n_chunks, k, streams, p->n_partial * 32 >= p->n_chunks);
    // Without the streaming hint: unaligned rows, and error buffers that the caches still hold when the update follows (sl_update_kept).  With several
    // waves per chunk unaligned rows gain from it on longer lists only (deferred, k = 32: 4000 chunks of 1001 columns 70.3 / 60.2, 900 of 530 29.4 / 30.7).
    const bool keep = update_follows && sl_update_kept(p->n_chunks, k, theta_local != nullptr);
    const bool unaligned = sl_select_unaligned(p, streams, update_follows, theta_local != nullptr);
    if (waves > 1) return slk_select_group(A, sub_only, waves, unaligned && p->n_chunks > 2048, st);
    // (one chunk per workgroup where the LDS of four does not fit)
    const int wpb = 4 * (size_t)A.lds_per_wave > 65536 ? 1 : k <= 128 ? sl_chunks_per_group(p) : 4;
    const dim3 grid((unsigned)((p->n_chunks + wpb - 1) / wpb)), block(64 * wpb);
    A.order = sl_order(p, grid.x);
    const size_t lds = (size_t)A.lds_per_wave * wpb;
    const bool two = p->bits == 2;
    select_kernel fn;
    if (sub_only) fn = select_for<2, false, false>(k);
    else if (random) fn = two ? k_select<0, 0, true, false, true> : k_select<0, 0, false, false, true>;
    else fn = keep || unaligned ? sl_select_kept(k, two, theta_local != nullptr) : select_for<false>(k, two, theta_local != nullptr);
    hipLaunchKernelGGL(fn, grid, block, lds, st, A);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
        sl_note_hip_error(err);
        return SL_ERR_HIP;
    }
    return SL_OK;
}

int slk_select(const sl_plan *p, float *e, const float *delta, const float *theta_local, float beta,
               int frozen, const unsigned char *pending, unsigned char *payload, unsigned char *coded,
               unsigned char *ws, bool update_follows, hipStream_t st)
{
    return launch_select(p, e, delta, theta_local, beta, frozen, pending, payload, coded, ws, update_follows, false, false, 0u, st);
}

int slk_select_random(const sl_plan *p, float *e, const float *delta, float beta, int frozen,
                      const unsigned char *pending, unsigned char *payload, unsigned char *ws, unsigned seed,
                      hipStream_t st)
{
    return launch_select(p, e, delta, nullptr, beta, frozen, pending, payload, nullptr, ws, false, false, true, seed, st);
}

int slk_sub_topk(const sl_plan *p, float *m, hipStream_t st)
{
    return launch_select(p, m, nullptr, nullptr, 1.0f, 0, nullptr, nullptr, nullptr, nullptr, false, true, false, 0u, st);
}
