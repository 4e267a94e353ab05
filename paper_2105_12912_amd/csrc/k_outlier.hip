// k_outlier.hip -- ordered outlier list: compaction at compression, scatter
// at decompression.
//
// Sec. IV-B.1 (modified quantisation): an out-of-range delta keeps its code
// slot as the placeholder 0 and is stored exactly in a separate list; before
// reconstruction the list is fused back (Algorithm 1, decompression half).
// The list is ordered by linear index.  Compression already counted the
// outliers of every row segment (the x-extent of one construct wave-tile);
// after a scan of those counts, each segment with outliers is compacted by
// a group of lanes.  Decompression scatters the list into a
// dense delta scratch and validates it against the codes.
#include "ebc_dev.h"
#include "ebc_launch.h"

namespace ebc {

constexpr uint32_t kSegPerBlock = kWave;  // segments per workgroup
constexpr uint32_t kSegLane = 8;          // elements of a segment per lane

uint32_t outlier_write_units(uint32_t n_seg) { return (n_seg + kSegPerBlock - 1) / kSegPerBlock; }

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

// A workgroup looks at kSegPerBlock segments (xs elements each, a power of two
// from 32 to 256) and lists those that hold outliers; a field without many
// ends there.  Listed segments are then compacted 256 * 8 / xs at a time, xs / 8
// lanes to a segment and eight elements to a lane: codes and deltas come in one
// round trip of 16-byte loads (any alignment), and a scan of the lanes' counts
// gives every outlier its place.  With a thread per segment, each walking up to
// 256 elements, the kernel took 77 us on a 100x500x500 field most of whose
// segments hold outliers (15 us on 256x256).
__global__ __launch_bounds__(kBlock) void k_outlier_write(const FieldDesc* __restrict__ F, int nf,
                                                          const uint32_t* __restrict__ soff)
{
    __shared__ uint32_t s_seg[kSegPerBlock], s_pos[kSegPerBlock];
    __shared__ uint32_t s_n;
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::ow_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || dy->codec == ARC_CONST || dy->n_out == 0) return;
    const uint32_t l = lane_id();
    if (threadIdx.x < (uint32_t)kWave) {
        const uint32_t sg = (t - fd.ow_base) * kSegPerBlock + l;
        const uint32_t* off = soff + fd.seg_base;
        uint32_t o0 = 0, o1 = 0;
        if (sg < fd.n_seg) o0 = off[sg], o1 = off[sg + 1];
        const uint64_t m = ballot(o0 != o1);
        if (o0 != o1) {
            const uint32_t k = __popcll(m & ((1ull << l) - 1));
            s_seg[k] = sg;
            s_pos[k] = o0 - off[0];
        }
        if (l == 0) s_n = __popcll(m);
    }
    __syncthreads();
    const uint32_t n = s_n;
    if (n == 0) return;
    EBC_G uint32_t* oidx = (EBC_G uint32_t*)(fd.arc + dy->off_oidx);
    EBC_G int32_t* oval = (EBC_G int32_t*)(fd.arc + dy->off_oval);
    const EBC_G uint16_t* __restrict__ q = fd.q;
    const EBC_G int32_t* __restrict__ dsc = fd.dsc;
    const uint32_t g = fd.xs / kSegLane;  // lanes per segment: 4 .. 32
    const uint32_t sub = threadIdx.x / g, gl = threadIdx.x % g;
    for (uint32_t k0 = 0; k0 < n; k0 += kBlock / g) {
        const uint32_t k = k0 + sub;
        uint64_t a = 0, b = 0;
        if (k < n) seg_range(fd, s_seg[k], a, b);
        const uint64_t i = a + gl * kSegLane;
        u32x4 c = {0x00010001u, 0x00010001u, 0x00010001u, 0x00010001u};
        u32x4 d0 = {0u, 0u, 0u, 0u}, d1 = {0u, 0u, 0u, 0u};
        if (i + kSegLane <= b) {
            c = *(const EBC_G u32x4_a2*)(q + i);
            d0 = *(const EBC_G u32x4_a4*)(dsc + i);
            d1 = *(const EBC_G u32x4_a4*)(dsc + i + 4);
        } else if (i < b) {  // the row's end
#pragma unroll
            for (uint32_t e = 0; e < kSegLane - 1; ++e) {
                if (i + e < b) {
                    const uint32_t sh = 16 * (e & 1);
                    c[e / 2] = (c[e / 2] & ~(0xFFFFu << sh)) | ((uint32_t)q[i + e] << sh);
                    if (e < 4) d0[e & 3] = (uint32_t)dsc[i + e];
                    else d1[e & 3] = (uint32_t)dsc[i + e];
                }
            }
        }
        uint32_t zm = 0;
#pragma unroll
        for (uint32_t e = 0; e < kSegLane; ++e) zm |= (((c[e / 2] >> (16 * (e & 1))) & 0xFFFFu) == 0 ? 1u : 0u) << e;
        // rank of the lane's outliers inside its segment
        const uint32_t cnt = __popc(zm), excl = wave_incl_scan_u32(cnt) - cnt;
        const uint32_t first = (uint32_t)__shfl((int)excl, (int)(l - l % g));
        if (zm) {
            uint32_t pos = s_pos[k] + excl - first;
#pragma unroll
            for (uint32_t e = 0; e < kSegLane; ++e) {
                if ((zm >> e) & 1u) {
                    oidx[pos] = (uint32_t)(i + e);
                    oval[pos] = (int32_t)(e < 4 ? d0[e & 3] : d1[e & 3]);
                    ++pos;
                }
            }
        }
    }
}

// ------------------------------------------------------------- decoding
// one thread per listed outlier: index in range, strictly ascending, code 0
__global__ __launch_bounds__(kBlock) void k_outlier_scatter(const FieldDesc* __restrict__ F, int nf)
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
    if (!bad) bad = fd.q[i] != 0;
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

hipError_t launch_outlier_scatter(const FieldDesc* F, int nf, uint32_t units, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_outlier_scatter, dim3(units), dim3(kBlock), 0, s, F, nf);
    return hipGetLastError();
}

}  // namespace ebc
