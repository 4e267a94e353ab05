// k_outlier.hip -- ordered outlier list (compaction at compression, scatter at
// decompression) and the archive headers, written in the same launch.
//
// Sec. IV-B.1 (modified quantisation): an out-of-range delta keeps its code
// slot as the placeholder 0 and is stored exactly in a separate list; before
// reconstruction the list is fused back (Algorithm 1, decompression half).
// The list is ordered by linear index.  Compression already counted the
// outliers of every row segment (the x-extent of one construct wave-tile);
// after a scan of those counts, each segment with outliers is compacted by
// a group of lanes.  Decompression scatters the list into a
// dense delta scratch and validates it against the codes.
#include "encode_dev.h"
#include "rle_dev.h"
#include "ebc_launch.h"

namespace ebc {

constexpr uint32_t kSegLane = 8;  // elements of a segment per lane

// Segments per workgroup.  Where most segments hold no outlier a workgroup's time is
// that of looking at them: 256, one per thread (18 us with 64 against 10 us on the 1M
// segments of 512^3).  Where many hold some, 64 (62 us against 37 us on the 2e5 of a
// rough 100x500x500 field).  The host does not know the density, so the line is the
// size at which 256 still make 2048 workgroups.  (A rough field above it was not
// measured.)
uint32_t outlier_write_segs(uint32_t n_seg) { return n_seg > (1u << 19) ? kBlock : kWave; }

// element range [a, b) of segment s
__device__ __forceinline__ void seg_range(const FieldDesc& fd, uint32_t s, uint64_t& a, uint64_t& b)
{
    if (fd.rank == 1) {
        a = (uint64_t)s * 256;
        b = min(a + 256, fd.n);
    } else {
        const uint32_t xs = fd.xs;
        const uint64_t row = s / fd.nxb;
        const uint32_t xb = s % fd.nxb;
        a = row * fd.nx + (uint64_t)xb * xs;
        b = row * fd.nx + min((uint64_t)(xb + 1) * xs, (uint64_t)fd.nx);
    }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

// A workgroup looks at its segments (xs elements each, a power of two
// from 32 to 256) and lists those that hold outliers; a field without many
// ends there.  Listed segments are then compacted 256 * 8 / xs at a time, xs / 8
// lanes to a segment and eight elements to a lane, two such groups in flight:
// codes by 16-byte loads (any alignment) and the deltas along with them, or if
// outliers are rare only those of the lanes that turn out to hold one, and a scan
// of the lanes' counts gives every outlier its place.  With a thread per segment,
// each walking up to 256 elements, the kernel took 77 us on a 100x500x500 field
// most of whose segments hold outliers (15 us on 256x256).
// offsets(): the list's two sections, asked for only when there is something
// to write.
struct OutlierLds {
    uint32_t seg[kBlock], pos[kBlock], n[kWavesPerBlock];
};
struct OutlierOut {
    EBC_G uint32_t* oidx;
    EBC_G int32_t* oval;
    bool ok;
};
template <class OFFSETS>
__device__ __forceinline__ void outlier_unit(const FieldDesc& fd, uint32_t t, const uint32_t* __restrict__ soff,
                                             OutlierLds& sm, OFFSETS offsets)
{
    const uint32_t l = lane_id(), w = threadIdx.x / kWave;
    {
        const uint32_t sg = (t - fd.ow_base) * fd.ow_segs + threadIdx.x;
        const uint32_t* off = soff + fd.seg_base;
        uint32_t o0 = 0, o1 = 0;
        if (threadIdx.x < fd.ow_segs && sg < fd.n_seg) o0 = off[sg], o1 = off[sg + 1];
        const uint64_t m = ballot(o0 != o1);
        if (l == 0) sm.n[w] = __popcll(m);
        __syncthreads();
        uint32_t k = __popcll(m & ((1ull << l) - 1));
#pragma unroll
        for (uint32_t v = 0; v < (uint32_t)kWavesPerBlock - 1; ++v) k += v < w ? sm.n[v] : 0u;
        if (o0 != o1) {
            sm.seg[k] = sg;
            sm.pos[k] = o0 - kcount(off, 0);
        }
    }
    __syncthreads();
    const uint32_t n = sm.n[0] + sm.n[1] + sm.n[2] + sm.n[3];
    if (n == 0) return;
    const OutlierOut to = offsets();
    if (!to.ok) return;
    EBC_G uint32_t* const oidx = to.oidx;
    EBC_G int32_t* const oval = to.oval;
    const EBC_G uint16_t* __restrict__ q = fd.q;
    const EBC_G int32_t* __restrict__ dsc = fd.dsc;
    // lanes per segment: as the segment's width asks for, 1 .. 32; rows shorter than a
    // segment take fewer (4M rows of 2: 79 us with xs / 8 lanes each, 37 so)
    const uint32_t row = fd.rank == 1 || fd.nx >= fd.xs ? fd.xs
                         : fd.nx <= kSegLane            ? kSegLane
                                                        : 1u << (32 - __builtin_clz(fd.nx - 1));
    const uint32_t g = row / kSegLane;
    // outliers in more than one of 16 elements: nearly every lane needs its deltas
    const bool dense = 16 * (uint64_t)(kcount(soff, (uint64_t)fd.seg_base + fd.n_seg) - kcount(soff, fd.seg_base)) > fd.n;
    const uint32_t sub = threadIdx.x / g, gl = threadIdx.x % g, per = kBlock / g;
    for (uint32_t k0 = 0; k0 < n; k0 += 2 * per) {
        u32x4 c[2], d0[2], d1[2];
        uint64_t i[2];
        uint32_t p[2];
        bool full[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t k = k0 + h * per + sub;
            uint64_t a = 0, b = 0;
            p[h] = 0;
            if (k < n) {
                seg_range(fd, sm.seg[k], a, b);
                p[h] = sm.pos[k];
            }
            i[h] = a + gl * kSegLane;
            c[h] = u32x4{0x00010001u, 0x00010001u, 0x00010001u, 0x00010001u};
            d0[h] = d1[h] = u32x4{0u, 0u, 0u, 0u};
            full[h] = i[h] + kSegLane <= b;
            if (full[h]) {
                c[h] = *(const EBC_G u32x4_a2*)(q + i[h]);
                if (dense) {
                    d0[h] = *(const EBC_G u32x4_a4*)(dsc + i[h]);
                    d1[h] = *(const EBC_G u32x4_a4*)(dsc + i[h] + 4);
                }
            } else if (i[h] < b) {  // the row's end
#pragma unroll
                for (uint32_t e = 0; e < kSegLane - 1; ++e) {
                    if (i[h] + e < b) {
                        const uint32_t sh = 16 * (e & 1);
                        c[h][e / 2] = (c[h][e / 2] & ~(0xFFFFu << sh)) | ((uint32_t)q[i[h] + e] << sh);
                    }
                }
            }
        }
        uint32_t zm[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            zm[h] = 0;
#pragma unroll
            for (uint32_t e = 0; e < kSegLane; ++e)
                zm[h] |= (((c[h][e / 2] >> (16 * (e & 1))) & 0xFFFFu) == 0 ? 1u : 0u) << e;
            // (the workspace goes on past the field's last delta)
            if (!dense || !full[h]) {
                if (zm[h] & 0x0Fu) d0[h] = *(const EBC_G u32x4_a4*)(dsc + i[h]);
                if (zm[h] & 0xF0u) d1[h] = *(const EBC_G u32x4_a4*)(dsc + i[h] + 4);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // rank of the lane's outliers inside its segment
            const uint32_t cnt = __popc(zm[h]), excl = wave_incl_scan_u32(cnt) - cnt;
            const uint32_t first = (uint32_t)__shfl((int)excl, (int)(l - l % g));
            if (zm[h]) {
                uint32_t pos = p[h] + excl - first;
#pragma unroll
                for (uint32_t e = 0; e < kSegLane; ++e) {
                    if ((zm[h] >> e) & 1u) {
                        oidx[pos] = (uint32_t)(i[h] + e);
                        oval[pos] = (int32_t)(e < 4 ? d0[h][e & 3] : d1[h][e & 3]);
                        ++pos;
                    }
                }
            }
        }
    }
}

// the outlier list at the offsets recorded in the field's scalars (inspection
// entry point)
__global__ __launch_bounds__(kBlock) void k_outlier_write(const FieldDesc* __restrict__ F, int nf,
                                                          const uint32_t* __restrict__ soff)
{
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::ow_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || dy->codec == ARC_CONST || dy->n_out == 0) return;
    __shared__ OutlierLds sm;
    outlier_unit(fd, t, soff, sm, [&] {
        return OutlierOut{(EBC_G uint32_t*)(fd.arc + dy->off_oidx), (EBC_G int32_t*)(fd.arc + dy->off_oval), true};
    });
}

__device__ __forceinline__ void zero_gap(EBC_G uint8_t* a, uint64_t from, uint64_t to)
{
    for (uint64_t i = from + threadIdx.x; i < to; i += kBlock) a[i] = 0;
}

// The field's scalars, header bytes, Huffman length section, the zero padding
// between sections, and the result record of the async calls (archive bytes, 0
// on error; status; codec).  One workgroup.
__device__ __forceinline__ void write_header(const FieldDesc& fd, const uint32_t* soff, const uint32_t* woff,
                                             const uint32_t* roff, uint64_t* __restrict__ res)
{
    EBC_G FieldDyn* dyn = fd.dyn;
    const auto* dy = kconst(fd.dyn);
    int32_t status = dy->status;
    const int32_t codec = dy->codec;
    Layout y = {};
    if (status == ST_OK) {
        y = layout_of(fd, codec, soff, woff, roff);
        if (y.total > fd.arc_cap) status = ST_ERR_OUT_TOO_SMALL;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (dy->status == ST_OK) {
            dyn->status = status;
            dyn->total = y.total;
            dyn->n_out = y.n_out, dyn->n_words = y.n_words, dyn->n_runs = y.n_runs;
            dyn->off_sbits = y.off_sbits, dyn->off_words = y.off_words, dyn->off_rlen = y.off_rlen;
            dyn->off_oidx = y.off_oidx, dyn->off_oval = y.off_oval;
        }
        if (res) {
            uint64_t* r = res + 2ull * fd.slot;
            r[0] = status == ST_OK ? y.total : 0ull;
            r[1] = (uint64_t)(uint32_t)status | ((uint64_t)(uint32_t)codec << 32);
        }
    }
    if (status != ST_OK) return;
    EBC_G uint8_t* a = fd.arc;
    const uint32_t l = threadIdx.x;
    __shared__ uint32_t h[32];
    if (l == 0) {
        h[0] = 0x31434245u;  // "EBC1"
        h[1] = 2u;           // version 2, flags 0
        h[2] = (uint32_t)fd.rank | ((uint32_t)codec << 8) | ((uint32_t)fd.eb_mode << 16) |
               ((uint32_t)fd.dtype << 24);
        h[3] = fd.n_bins;
        const uint64_t dims[3] = {fd.nx, fd.ny, fd.nz};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            h[4 + 2 * k] = (uint32_t)dims[k];
            h[5 + 2 * k] = (uint32_t)(dims[k] >> 32);
        }
        h[10] = fd.rank == 1 ? 256u : fd.rank == 2 ? 16u : 8u;
        h[11] = fd.rank == 1 ? 1u : fd.rank == 2 ? 16u : 8u;
        h[12] = fd.rank == 3 ? 8u : 1u;
        h[13] = fd.hc;
        const double dd[3] = {fd.eb, dy->eb_abs, dy->ebx2};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint64_t b = (uint64_t)__double_as_longlong(dd[k]);
            h[14 + 2 * k] = (uint32_t)b;
            h[15 + 2 * k] = (uint32_t)(b >> 32);
        }
        // constant value as f64 (exact for an fp32 field)
        const uint64_t cb = codec == ARC_CONST ? (uint64_t)__double_as_longlong((double)dy->mn) : 0ull;
        h[20] = (uint32_t)cb;
        h[21] = (uint32_t)(cb >> 32);
        const uint64_t na = codec == ARC_HUFFMAN ? (uint64_t)fd.n_hch : y.n_runs;  // RLE, RLE+VLE: runs
        const uint64_t v[4] = {y.n_out, codec == ARC_CONST ? 0ull : na, y.n_words, y.total};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            h[22 + 2 * k] = (uint32_t)v[k];
            h[23 + 2 * k] = (uint32_t)(v[k] >> 32);
        }
        h[30] = huff_codec(codec) ? fd.hs : 0u;
        h[31] = 0;
    }
    __syncthreads();
    if (l < 32) ((EBC_G uint32_t*)a)[l] = h[l];
    if (codec == ARC_CONST) return;
    if (huff_codec(codec)) {
        const bool vle = codec == ARC_RLE_VLE;
        const uint64_t nsub = vle ? (y.n_runs + fd.hs - 1) / fd.hs : fd.n_sub;
        const EBC_G uint32_t* len4 = (const EBC_G uint32_t*)fd.len;  // lengths are 256-byte aligned
#pragma unroll 4
        for (uint32_t s = l; s < fd.n_bins / 4; s += kBlock) ((EBC_G uint32_t*)(a + kHdr))[s] = len4[s];
        for (uint32_t s = (fd.n_bins & ~3u) + l; s < fd.n_bins; s += kBlock) a[kHdr + s] = fd.len[s];
        zero_gap(a, kHdr + fd.n_bins, y.off_sbits);
        zero_gap(a, y.off_sbits + 2ull * nsub, y.off_words);
        const uint64_t words_end = y.off_words + 4ull * y.n_words;
        if (vle) {
            zero_gap(a, words_end, y.off_rlen);
            zero_gap(a, y.off_rlen + 4ull * y.n_runs, y.off_oidx);
        } else {
            zero_gap(a, words_end, y.off_oidx);
        }
    } else {
        zero_gap(a, kHdr + 2ull * y.n_runs, y.off_rlen);
        zero_gap(a, y.off_rlen + 4ull * y.n_runs, y.off_oidx);
    }
    zero_gap(a, y.off_oidx + 4ull * y.n_out, y.off_oval);
    zero_gap(a, y.off_oval + 4ull * y.n_out, y.total);
}

// Last launch of a compression: the header of every field (workgroups below
// nf), the runs of run-length fields (the next rt_blocks workgroups) and the
// outlier lists.  One launch of small pieces: each by itself is a launch of 3 to
// 8 us that most fields need little of.
__global__ __launch_bounds__(kBlock) void k_finish(const FieldDesc* __restrict__ F, int nf, uint32_t rt_blocks,
                                                   uint32_t rt_units, uint32_t first,
                                                   const uint32_t* __restrict__ soff,
                                                   const uint32_t* __restrict__ woff,
                                                   const uint32_t* __restrict__ roff,
                                                   uint64_t* __restrict__ res)
{
    __shared__ OutlierLds sm;
    uint32_t t = first + blockIdx.x;
    if (t < (uint32_t)nf) {
        write_header(F[t], soff, woff, roff, res);
        return;
    }
    t -= (uint32_t)nf;
    if (t < rt_blocks) {
        rle_write_tiles(F, nf, soff, woff, roff, rt_units, kRleValArc | kRleLen,
                        t * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave),
                        rt_blocks * kWavesPerBlock);
        return;
    }
    t -= rt_blocks;
    const int f = find_field<&FieldDesc::ow_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    const int32_t codec = dy->codec, status = dy->status;
    // (the header's workgroup may report a small buffer while the waves of this one
    // get here: they all go on, and find that out by themselves)
    if ((status != ST_OK && status != ST_ERR_OUT_TOO_SMALL) || codec == ARC_CONST) return;
    outlier_unit(fd, t, soff, sm, [&] {
        const Layout y = layout_of(fd, codec, soff, woff, roff);
        return OutlierOut{(EBC_G uint32_t*)(fd.arc + y.off_oidx), (EBC_G int32_t*)(fd.arc + y.off_oval),
                          y.total <= fd.arc_cap};
    });
}

// ------------------------------------------------------------- decoding
// one thread per listed outlier: index in range, strictly ascending, code 0
// (the code of a 1D run-length coded field is looked up among its tile's runs)
__global__ __launch_bounds__(kBlock) void k_outlier_scatter(const FieldDesc* __restrict__ F, int nf,
                                                            const uint32_t* __restrict__ starts,
                                                            const uint32_t* __restrict__ tmap)
{
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::sc_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    EBC_G FieldDyn* dy = fd.dyn;
    if (dy->status != ST_OK || fd.codec_hdr == ARC_CONST) return;
    const uint64_t k = (uint64_t)(t - fd.sc_base) * kBlock + threadIdx.x;
    if (k >= fd.n_out_hdr) return;
    const EBC_G uint32_t* oidx = (const EBC_G uint32_t*)(fd.arc + fd.off_oidx);
    const EBC_G int32_t* oval = (const EBC_G int32_t*)(fd.arc + fd.off_oval);
    const uint32_t i = oidx[k];
    bool bad = i >= fd.n || (k > 0 && oidx[k - 1] >= i);
    if (!bad) {
        if (fd.rank == 1 && rle_codec(fd.codec_hdr)) bad = run_value(fd, i, starts, tmap) != 0;
        else bad = fd.q[i] != 0;
    }
    if (bad) {
        atomicMin(&dy->status, ST_ERR_ARCHIVE);
        return;
    }
    fd.dsc[i] = oval[k];
}

hipError_t launch_outlier_write(const FieldDesc* F, int nf, uint32_t units, const uint32_t* soff,
                                hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_outlier_write, dim3(units), dim3(kBlock), 0, s, F, nf, soff);
    return hipGetLastError();
}

hipError_t launch_finish(const FieldDesc* F, int nf, uint32_t rt_units, uint32_t ow_units, const uint32_t* soff,
                         const uint32_t* woff, const uint32_t* roff, uint64_t* res, hipStream_t s)
{
    // a wave per tile; up to 2048 workgroups, of which the device holds 1792 at a time
    const uint32_t rb = min((rt_units + kWavesPerBlock - 1) / kWavesPerBlock, kEncBlocks);
    // the outlier lists of a field of nearly 2^32 segments go by themselves
    const uint64_t all = (uint64_t)nf + rb + ow_units;
    const uint32_t one = all * kBlock < kMaxThreads ? (uint32_t)all : nf + rb;
    hipLaunchKernelGGL(k_finish, dim3(one), dim3(kBlock), 0, s, F, nf, rb, rt_units, 0u, soff, woff, roff, res);
    if (one < all) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_finish, dim3(ow_units), dim3(kBlock), 0, s, F, nf, rb, rt_units, one, soff, woff, roff,
                           res);
    }
    return hipGetLastError();
}

hipError_t launch_outlier_scatter(const FieldDesc* F, int nf, uint32_t units, const uint32_t* starts,
                                  const uint32_t* tmap, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_outlier_scatter, dim3(units), dim3(kBlock), 0, s, F, nf, starts, tmap);
    return hipGetLastError();
}

}  // namespace ebc
