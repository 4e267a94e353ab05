// k_archive.hip -- the archive format (its sections are laid out in encode_dev.h,
// the header written in k_outlier.hip) and the descriptor upload.
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

// Upload up to kDescPerLaunch descriptors passed by value, a word per thread
// (a descriptor per thread took 5 us for eight).  For a decompression (init) the
// fields' device scalars start from the header values and their code-0 counters
// from zero.
__global__ __launch_bounds__(kBlock) void k_put_desc(DescBlob blob, FieldDesc* __restrict__ dst, int init)
{
    // the arguments as memory: indexing the parameter itself by thread would
    // copy it to scratch first
    const auto* src = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr() +
                      offsetof(DescBlob, d) / 4;
    const uint32_t words = (uint32_t)blob.count * (sizeof(FieldDesc) / 4);
    uint32_t* out = (uint32_t*)(dst + blob.first);
    for (uint32_t i = threadIdx.x; i < words; i += kBlock) out[i] = src[i];
    if (!init) return;
    const auto* fds = (const __attribute__((address_space(4))) FieldDesc*)src;
    for (int k = threadIdx.x / kWave; k < blob.count; k += kWavesPerBlock) {
        const auto& fd = fds[__builtin_amdgcn_readfirstlane(k)];
        if (fd.codec_hdr != ARC_CONST) fd.zslot[lane_id() * kZeroStride] = 0;
        if (lane_id() != 0) continue;
        FieldDyn d = {};
        d.status = ST_OK;
        d.codec = fd.codec_hdr;
        d.ebx2 = fd.ebx2_hdr;
        d.n_out = fd.n_out_hdr;
        *fd.dyn = d;
    }
}
static_assert(sizeof(FieldDesc) % 8 == 0 && offsetof(DescBlob, d) % 8 == 0, "copied as words");

hipError_t upload_descs(const FieldDesc* host, int nf, FieldDesc* dev, bool init, hipStream_t s)
{
    for (int first = 0; first < nf; first += kDescPerLaunch) {
        DescBlob b;
        b.first = first;
        b.count = min(kDescPerLaunch, nf - first);
        for (int k = 0; k < b.count; ++k) b.d[k] = host[first + k];
        hipLaunchKernelGGL(k_put_desc, dim3(1), dim3(kBlock), 0, s, b, dev, init ? 1 : 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ebc
