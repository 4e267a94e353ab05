// k_archive.hip -- the archive format (its sections are laid out in encode_dev.h,
// the header written in k_outlier.hip), statuses, descriptor upload.
//
// Archive format v2 (little-endian, 128-byte header, every section starts on
// a 16-byte boundary, padding is zero):
//   Huffman: u8 len[n_bins] | u16 sbits[n_sub] | u32 words[n_words]
//            (sbits: bit count of every sub-chunk of hs = min(hc, 256)
//            symbols; chunks of hc symbols start on a word, their sub-chunks
//            follow each other without padding)
//   RLE:     u16 val[n_runs] | u32 len[n_runs]
//   RLE+VLE: u8 len[n_bins] | u16 sbits | u32 words (the run values as a
//            Huffman stream of their own) | u32 rlen[n_runs]
//   all:     u32 outlier_index[n_out] | i32 outlier_delta[n_out]
// The paper leaves the container unspecified; the header records everything
// a decoder needs (dims, chunking, codec, step, section counts).
#include "ebc_dev.h"
#include "ebc_launch.h"

namespace ebc {

__global__ void k_status(const FieldDesc* __restrict__ F, int32_t* __restrict__ st)
{
    *st = F[0].dyn->status;
}

__global__ void k_batch_status(const FieldDesc* __restrict__ F, int nf, int32_t* __restrict__ st)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nf) return;
    st[F[k].slot] = F[k].dyn->status;
}

// Upload up to kDescPerLaunch descriptors passed by value.
__global__ void k_put_desc(DescBlob blob, FieldDesc* __restrict__ dst)
{
    const int k = threadIdx.x;
    if (k < blob.count) dst[blob.first + k] = blob.d[k];
}

hipError_t launch_status(const FieldDesc* F, int32_t* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_status, dim3(1), dim3(1), 0, s, F, st);
    return hipGetLastError();
}

hipError_t launch_batch_status(const FieldDesc* F, int nf, int32_t* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_status, dim3((nf + 63) / 64), dim3(64), 0, s, F, nf, st);
    return hipGetLastError();
}

hipError_t upload_descs(const FieldDesc* host, int nf, FieldDesc* dev, hipStream_t s)
{
    for (int first = 0; first < nf; first += kDescPerLaunch) {
        DescBlob b;
        b.first = first;
        b.count = min(kDescPerLaunch, nf - first);
        for (int k = 0; k < b.count; ++k) b.d[k] = host[first + k];
        hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(kDescPerLaunch), 0, s, b, dev);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ebc
