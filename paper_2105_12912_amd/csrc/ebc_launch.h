// ebc_launch.h -- host-side launchers of the HIP kernels (one per kernel
// family); each enqueues on the given stream and returns hipGetLastError().
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ebc_types.h"

namespace ebc {

// Records a failure detail for ebc_last_error() (calling thread) and returns status.
int set_error(int status, const char* fmt, ...);

constexpr uint64_t kMaxThreads = 1ull << 32;  // a launch has to have fewer

constexpr int kDescPerLaunch = 8;
struct DescBlob {
    int first;
    int count;
    FieldDesc d[kDescPerLaunch];
};

// scan
constexpr uint32_t kScanMax = 0xFFFFF000u;  // longest array (a multiple of the scan's tile)
uint32_t scan_tmp_words(uint32_t n);
// exclusive scan, total in a[n]; direct_max: tile count up to which each
// tile's workgroup adds the sums of the tiles before it (0: the default),
// above which the tile sums are scanned by one workgroup first
hipError_t launch_scan(uint32_t* a, uint32_t n, uint32_t* tmp, hipStream_t s, uint32_t direct_max = 0);

// quantisation
hipError_t launch_range(const FieldDesc* F, int nf, uint32_t units, bool f64, hipStream_t s);
hipError_t launch_params(const FieldDesc* F, int nf, hipStream_t s);
// a field's rows: shorter than a quad (rank 2 and 3), any, 16-byte aligned
enum { kRowsShort = 0, kRowsAny = 1, kRowsVec = 2 };
uint32_t construct_resident_blocks(int rank, int rows, uint32_t n_bins, bool f64);
hipError_t launch_construct(const FieldDesc* F, int nf, int rank, int rows, bool f64, uint32_t wg_tiles,
                            uint32_t blocks, uint32_t n_bins, uint32_t* seg_cnt, hipStream_t s);
hipError_t launch_hist_reduce(const FieldDesc* F, int nf, uint32_t n_bins, hipStream_t s);

// codebook
size_t codebook_lds_bytes(uint32_t n_bins);
// direct: the partial histograms are added up here (no histogram reduce before)
hipError_t launch_codebook(const FieldDesc* F, int nf, uint32_t n_bins, int pass, bool direct, hipStream_t s);
// decompression prologue; direct: no field has more than kPrepDirect chunks
hipError_t launch_dec_prep(const FieldDesc* F, int nf, uint32_t units, bool direct, uint8_t* tabs, size_t stride,
                           uint32_t* wcnt, uint32_t* soff, hipStream_t s);
size_t codebook_wide_scratch_bytes(uint32_t n_bins);

// compressibility estimates (histogram bounds; madogram over `samples` pairs)
hipError_t launch_estimate(const FieldDesc* F, int nf, EstDev* est, uint64_t samples, uint64_t seed,
                           hipStream_t s);

// Huffman
size_t huff_write_lds_bytes(uint32_t n_bins, uint32_t hc);
// count pass of the Huffman chunks (which: 0 Huffman fields, 1 RLE+VLE fields)
// and, with rt_units, of the run-length tiles
hipError_t launch_encode_count(const FieldDesc* F, int nf, uint32_t units, uint32_t hc, uint32_t n_bins,
                               uint32_t* wcnt, int which, uint32_t rt_units, uint32_t* rcnt, hipStream_t s);
hipError_t launch_huff_write(const FieldDesc* F, int nf, uint32_t units, uint32_t hc, uint32_t n_bins,
                             const uint32_t* soff, const uint32_t* woff, const uint32_t* roff, hipStream_t s);
void huff_decode_split(uint64_t n_sub, uint32_t* per_wave, uint32_t* lanes, uint32_t* groups);
hipError_t launch_huff_decode(const FieldDesc* F, int nf, uint32_t units, uint32_t per_wave, uint32_t lanes,
                              const uint32_t* woff, const uint32_t* soff, const uint8_t* tabs,
                              size_t tab_stride, hipStream_t s);

// RLE
hipError_t launch_rle_count(const FieldDesc* F, int nf, uint32_t units, uint32_t* rcnt, hipStream_t s);
// RLE+VLE: the run-value stream, its length and its histogram
hipError_t launch_rle_vle_prep(const FieldDesc* F, int nf, uint32_t units, const uint32_t* roff,
                               uint32_t n_bins, hipStream_t s);
hipError_t launch_rle_decode(const FieldDesc* F, int nf, uint32_t rl_units, uint32_t rt_units,
                             uint32_t* starts, uint32_t* tmap, uint32_t* tmp, uint32_t n_starts,
                             uint32_t scan_direct, bool expand, hipStream_t s);
hipError_t launch_rle_reconstruct(const FieldDesc* F, int nf, uint32_t rt_units, const uint32_t* starts,
                                  const uint32_t* tmap, hipStream_t s);

// outliers
uint32_t outlier_write_segs(uint32_t n_seg);
hipError_t launch_outlier_write(const FieldDesc* F, int nf, uint32_t units, const uint32_t* soff,
                                hipStream_t s);
// headers, result records (res: 16 bytes per field in the caller's order, or
// NULL), runs of run-length fields (rt_units tiles, if any) and outlier lists
hipError_t launch_finish(const FieldDesc* F, int nf, uint32_t rt_units, uint32_t ow_units, const uint32_t* soff,
                         const uint32_t* woff, const uint32_t* roff, uint64_t* res, hipStream_t s);
hipError_t launch_outlier_scatter(const FieldDesc* F, int nf, uint32_t units, const uint32_t* starts,
                                  const uint32_t* tmap, hipStream_t s);

// reconstruction
hipError_t launch_reconstruct(const FieldDesc* F, int nf, int rank, bool vec, bool f64, uint32_t wg_tiles,
                              hipStream_t s);
hipError_t launch_reconstruct3(const FieldDesc* F, int nf, uint32_t units, hipStream_t s);
// st: statuses in the caller's order (device), or NULL
hipError_t launch_recon_check(const FieldDesc* F, int nf, int32_t* st, hipStream_t s);
hipError_t launch_fill_const(const FieldDesc* F, int nf, uint32_t units, hipStream_t s);

// archive
// init: a decompression's device scalars as well
hipError_t upload_descs(const FieldDesc* host, int nf, FieldDesc* dev, bool init, hipStream_t s);

}  // namespace ebc
