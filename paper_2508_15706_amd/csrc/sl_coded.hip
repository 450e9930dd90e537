// Coded wire format: the passes that place the variable-length part (the chunks' quotient bit
// vectors), and the transcoder from a plain payload (sl_rice_encode).  The format is described
// in sl_coded.h; the appendix "Compression of indices in Top-k" of the paper is where an index
// coder enters the method.
//
// The writers of a coded buffer (kernel A of sl_compress_coded, or k_rice_chunks below for a
// payload that already exists) put everything whose place follows from the tensor list - table
// headers, remainder and value fields - straight into the buffer, and leave each chunk's bit
// vector and quotient sum Q in the workspace, from where the placement steps of sl_coded.h take them.
#include "sl_coded.h"

int sl_rice_param(int k)
{
    const int q = 2839 / k;
    int b = 0;
    while ((2 << b) <= q) ++b;
    return q < 1 ? 0 : b;
}

namespace {

// Threads per tensor: 1024 read the groups of a large tensor in few turns (one of 24,000 chunks, k = 64, whole
// transcode: 29.1 us, with 256 threads 30.5); with more tensors than such workgroups fit the chip together (two per
// compute unit) they only take each other's places (tensors of 3 chunks: 700 19.0 / 16.8 us, 3000 50.3 / 40.4).
#ifndef SL_SCAN_WIDE_UPTO
#define SL_SCAN_WIDE_UPTO 512
#endif
template <int THREADS>
__global__ void __launch_bounds__(THREADS) k_coded_scan_tensor(SlCodedArgs A)
{
    __shared__ unsigned wsum[THREADS / 64];
    sl_coded_scan_tensor<THREADS>(A, (int)blockIdx.x, wsum);
}

__global__ void __launch_bounds__(64) k_coded_scan_list(SlCodedArgs A)
{
    sl_coded_scan_list(A.twords, A.n_tensors, A.G.section, A.out);
}

__global__ void __launch_bounds__(256) k_coded_place(SlCodedArgs A)
{
    extern __shared__ __align__(16) unsigned place_lds[];
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long gi = (long long)blockIdx.x * (blockDim.x >> 6) + wave;
    if (gi >= A.n_groups) return;
    sl_coded_place(A, gi, place_lds + (size_t)wave * (SL_RICE_GROUP * A.G.ua + 1));
}

// ------------------------------------------------------------------ transcoder, plain -> coded
// One wave per chunk: the record's 12-bit indices are unpacked into LDS and coded by the same
// routine as in kernel A of the compressor; the value fields and the table header are copied.
struct ChunksArgs {
    SlCodedGeom G;
    const SlChunkDesc *desc;
    const SlTensorDev *tensors;
    long long n_chunks;
    int rec_bytes;
    const unsigned char *payload;
    unsigned char *out;
    unsigned *uvec;
    unsigned short *qsum;
};

__global__ void __launch_bounds__(256) k_rice_chunks(ChunksArgs A)
{
    extern __shared__ __align__(16) unsigned char chunks_lds[];
    const int lane = threadIdx.x & 63;
    const int wave = sl_uniform((int)(threadIdx.x >> 6));
    const long long c = (long long)blockIdx.x * (blockDim.x >> 6) + wave;
    if (c >= A.n_chunks) return;
    const SlCodedGeom &G = A.G;
    const int k = G.k, nrw = G.rem_bytes >> 2;
    const size_t per_wave = ((size_t)2 * k + 4 * ((size_t)G.ua + nrw) + 15) & ~(size_t)15;
    unsigned char *smem = chunks_lds + (size_t)wave * per_wave;
    unsigned *uv = reinterpret_cast<unsigned *>(smem);
    unsigned *rw = uv + G.ua;
    unsigned short *idx = reinterpret_cast<unsigned short *>(rw + nrw);
    const SlChunkDesc d = A.desc[c];
    const SlTensorDev td = A.tensors[d.tensor];
    const unsigned char *rec = A.payload + d.rec_off;
    for (int m = lane; m < k; m += 64) {
        const int b0 = (3 * m) >> 1;
        const unsigned w = (unsigned)rec[b0] | ((unsigned)rec[b0 + 1] << 8);
        idx[m] = (unsigned short)((m & 1) ? (w >> 4) : (w & 0xFFFu));
    }
    sl_wave_sync();
    const int Q = sl_coded_emit(G, lane, idx, uv, rw);
    unsigned char *fix = A.out + td.cfix_off + (long long)d.local_chunk * G.cfix;
    for (int w = lane; w < nrw; w += 64) reinterpret_cast<unsigned *>(fix)[w] = rw[w];
    // the value fields byte for byte, then the record's zero padding
    const unsigned char *vals = rec + 3 * k / 2;
    for (int i = lane; i < G.cfix - G.rem_bytes; i += 64) fix[G.rem_bytes + i] = i < G.val_bytes ? vals[i] : 0;
    unsigned *uvo = A.uvec + (size_t)c * G.ua;
    const int words = (k + Q + 31) >> 5;
    for (int w = lane; w < words; w += 64) uvo[w] = uv[w];
    if (lane == 0) A.qsum[c] = (unsigned short)Q;
    if (d.local_chunk == 0)                                        // the table header
        for (int i = lane; 4 * i < G.hdr; i += 64)
            reinterpret_cast<unsigned *>(A.out + td.cblk_off)[i] =
                reinterpret_cast<const unsigned *>(A.payload + td.pay_off)[i];
    if (d.local_chunk == td.n_chunks - 1) {                        // zero padding of the block
        const long long used = (td.cfix_off - td.cblk_off) + td.n_chunks * (long long)G.cfix;
        for (long long i = used + lane; i < td.cblk_bytes; i += 64) A.out[td.cblk_off + i] = 0;
    }
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

int slk_coded_scan(const sl_plan *p, unsigned char *out, unsigned char *ws, hipStream_t st)
{
    if (p->n_tensors <= SL_SCAN_WIDE_UPTO)
        hipLaunchKernelGGL(k_coded_scan_tensor<1024>, dim3(p->n_tensors), dim3(1024), 0, st, sl_coded_args(p, out, ws));
    else
        hipLaunchKernelGGL(k_coded_scan_tensor<256>, dim3(p->n_tensors), dim3(256), 0, st, sl_coded_args(p, out, ws));
    return launched();
}

int slk_coded_place(const sl_plan *p, unsigned char *out, unsigned char *ws, hipStream_t st)
{
    int wpb = 4;
    const size_t per_wave = sl_coded_place_words(p->cg) * sizeof(unsigned);
    while (wpb > 1 && per_wave * wpb > 65536) wpb >>= 1;
    hipLaunchKernelGGL(k_coded_place, dim3((unsigned)((p->n_groups + wpb - 1) / wpb)), dim3(64 * wpb), per_wave * wpb, st,
                       sl_coded_args(p, out, ws));
    return launched();
}

// The steps that finish a coded buffer once its writers have run, as launches of their own.
int slk_coded_finish(const sl_plan *p, unsigned char *out, unsigned char *ws, hipStream_t st)
{
    int rc;
    if (p->n_groups > 0 && (rc = slk_coded_scan(p, out, ws, st))) return rc;
    hipLaunchKernelGGL(k_coded_scan_list, dim3(1), dim3(64), 0, st, sl_coded_args(p, out, ws));
    if ((rc = launched())) return rc;
    return p->n_groups > 0 ? slk_coded_place(p, out, ws, st) : SL_OK;
}

int slk_rice_encode(const sl_plan *p, const unsigned char *payload, unsigned char *out,
                    unsigned char *ws, hipStream_t st)
{
    if (p->n_chunks > 0) {
        ChunksArgs C;
        C.G = p->cg;
        C.desc = p->d_desc;
        C.tensors = p->d_tensors;
        C.n_chunks = p->n_chunks;
        C.rec_bytes = p->rec_bytes;
        C.payload = payload;
        C.out = out;
        C.uvec = reinterpret_cast<unsigned *>(ws + p->ws_uvec);
        C.qsum = reinterpret_cast<unsigned short *>(ws + p->ws_qsum);
        const size_t per_wave = ((size_t)2 * p->k + 4 * ((size_t)p->cg.ua + (p->cg.rem_bytes >> 2)) + 15) & ~(size_t)15;
        hipLaunchKernelGGL(k_rice_chunks, dim3((unsigned)((p->n_chunks + 3) / 4)), dim3(256), per_wave * 4, st, C);
        const int rc = launched();
        if (rc) return rc;
    }
    return slk_coded_finish(p, out, ws, st);
}
