// k_rle.hip -- run-length encoding of the quant-codes and its inverse.
//
// Sec. III-B: a run of equal symbols is stored as a (value, count) tuple; the
// run lengths are metadata.  Runs are maximal and taken over the whole code
// array in row-major order.  Encoding marks run starts (a code differing from
// its predecessor), counts them per tile, scans the counts, and writes
// (value, length) pairs in order (encode_dev.h).  Decoding scans the stored
// lengths into starts and expands each output tile from the runs that overlap
// it.
#include "encode_dev.h"
#include "rle_dev.h"
#include "ebc_launch.h"

namespace ebc {

__global__ __launch_bounds__(kBlock) void k_rle_count(const FieldDesc* __restrict__ F, int nf,
                                                      uint32_t* __restrict__ rcnt, uint32_t units)
{
    __shared__ RleShared sh;
    rle_count_tiles(F, nf, rcnt, units, sh);
}

// RLE+VLE: the run values before their codebook exists
__global__ __launch_bounds__(kBlock) void k_rle_write(const FieldDesc* __restrict__ F, int nf,
                                                      const uint32_t* __restrict__ soff,
                                                      const uint32_t* __restrict__ woff,
                                                      const uint32_t* __restrict__ roff, uint32_t units,
                                                      int what)
{
    rle_write_tiles(F, nf, soff, woff, roff, units, what,
                    blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave),
                    gridDim.x * kWavesPerBlock);
}

// RLE+VLE compress: histogram of the run values, kRleTile values per
// workgroup, privatised in LDS (the codes' histogram of Sec. II-A step 5,
// taken over the value stream).
__global__ __launch_bounds__(kBlock) void k_rle_vhist(const FieldDesc* __restrict__ F, int nf,
                                                      uint32_t units)
{
    extern __shared__ uint32_t sh[];
    for (uint32_t t = blockIdx.x; t < units; t += gridDim.x) {
        const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
        const FieldDesc& fd = F[f];
        const auto* dy = kconst(fd.dyn);
        const uint64_t R = dy->n_runs;
        const uint64_t lo = (uint64_t)(t - fd.rt_base) * kRleTile;
        if (dy->status != ST_OK || dy->codec != ARC_RLE_VLE || lo >= R) {
            t = skip_field(fd, t) - gridDim.x;
            continue;
        }
        // wide bins: LDS slots as in construction (code 0, then a window
        // around the centre), other values counted in HBM directly
        const uint32_t nb = fd.n_bins, ns = hist_slots(nb), wlo = hist_win_lo(nb);
        const bool wide = nb > kMaxBins;
        for (uint32_t b = threadIdx.x; b < ns; b += kBlock) sh[b] = 0;
        __syncthreads();
        const uint64_t hi = min(lo + (uint64_t)kRleTile, R);
        for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) {
            const uint32_t v = fd.vsym[i];
            if (!wide) {
                atomicAdd(&sh[v], 1u);
            } else {
                const uint32_t dj = v - wlo;  // codes below the window wrap to large values
                if (v == 0) atomicAdd(&sh[0], 1u);
                else if (dj < kHistWin - 1) atomicAdd(&sh[dj + 1], 1u);
                else atomicAdd(&fd.vhist[v], 1u);
            }
        }
        __syncthreads();
        for (uint32_t b = threadIdx.x; b < ns; b += kBlock)
            if (sh[b]) atomicAdd(&fd.vhist[wide && b ? wlo + b - 1 : b], sh[b]);
        __syncthreads();
    }
}

// ------------------------------------------------------------- decoding
// Run lengths from the archive into the batch-wide array.  A run must be
// non-empty and no longer than the field; the scan that follows works modulo
// 2^32, so the cover check below also needs the starts to increase.
__global__ __launch_bounds__(kBlock) void k_rle_prep(const FieldDesc* __restrict__ F, int nf,
                                                     uint32_t* __restrict__ starts)
{
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::rl_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const uint32_t k = (t - fd.rl_base) * kBlock + threadIdx.x;
    if (!rle_codec(fd.codec_hdr) || k >= fd.n_runs_hdr) return;
    const uint32_t L = ((const EBC_G uint32_t*)(fd.arc + fd.off_rlen))[k];
    if (L == 0 || (uint64_t)L > fd.n) atomicMin(&fd.dyn->status, ST_ERR_ARCHIVE);
    starts[fd.rle_base + k] = L;
}

// After the scan, two things in one launch.
//
// Check, one thread per run (workgroups below rl_units): the runs must cover
// the field exactly.  With every length in [1, n], the relative starts (mod
// 2^32) increase strictly exactly when no prefix sum wrapped, and then the last
// one is the true total, which must equal n.
//
// Tile map, one thread per output tile (the other workgroups): the run that
// holds the tile's first element (the largest r with start[r] <= tile start)
// and the number of runs it overlaps, so that every tile's searches are in
// flight at once rather than one thread per workgroup searching while the
// others wait.  The searches stay inside the run array whatever it holds.
// tmap[2t] = first run, or the run's value if it is the only one; tmap[2t + 1] =
// run count.
__global__ __launch_bounds__(kBlock) void k_rle_map(const FieldDesc* __restrict__ F, int nf, uint32_t rl_units,
                                                    uint32_t rt_units, const uint32_t* __restrict__ starts,
                                                    uint32_t* __restrict__ tmap)
{
    if (blockIdx.x < rl_units) {
        const uint32_t t = blockIdx.x;
        const int f = find_field<&FieldDesc::rl_base>(F, nf, t);
        const FieldDesc& fd = F[f];
        const uint32_t k = (t - fd.rl_base) * kBlock + threadIdx.x;
        if (!rle_codec(fd.codec_hdr) || k >= fd.n_runs_hdr) return;
        const uint32_t* S = starts + fd.rle_base;
        const uint32_t s0 = S[0];
        const uint32_t a = S[k] - s0, b = S[k + 1] - s0;
        bool bad = b <= a;
        if (k + 1 == fd.n_runs_hdr && (uint64_t)b != fd.n) bad = true;
        if (bad) atomicMin(&fd.dyn->status, ST_ERR_ARCHIVE);
        return;
    }
    const uint32_t t = (blockIdx.x - rl_units) * kBlock + threadIdx.x;
    if (t >= rt_units) return;
    const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    if (!rle_codec(fd.codec_hdr)) return;
    const uint32_t* S = starts + fd.rle_base;
    const uint32_t s0 = S[0];
    const uint64_t lo = (uint64_t)(t - fd.rt_base) * kRleTile;
    const uint64_t hi = min(lo + (uint64_t)kRleTile, fd.n);
    // the runs holding the tile's first and last element, searched side by side
    // (each step waits for a load: 14 us one after the other on 120M elements, 10 here)
    uint32_t a = 0, b = fd.n_runs_hdr - 1, c = 0, d = b;
    while (a < b || c < d) {
        const uint32_t m = a + ((b - a + 1) >> 1), k = c + ((d - c + 1) >> 1);  // (the sums may pass 2^32)
        const uint32_t sm = S[m] - s0, sk = S[k] - s0;
        if (a < b) {
            if ((uint64_t)sm <= lo) a = m;
            else b = m - 1;
        }
        if (c < d) {
            if ((uint64_t)sk <= hi - 1) c = k;
            else d = k - 1;
        }
    }
    tmap[2 * t] = c == a ? fd.rval[a] : a;
    tmap[2 * t + 1] = c - a + 1;
}

// Expansion of 2D and 3D fields into the code array (1D fields are reconstructed
// from their runs, see k_rle_reconstruct).
__global__ __launch_bounds__(kBlock) void k_rle_expand(const FieldDesc* __restrict__ F, int nf,
                                                       const uint32_t* __restrict__ starts,
                                                       const uint32_t* __restrict__ tmap)
{
    __shared__ RleStage sm;
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    if (fd.dyn->status != ST_OK || !rle_codec(fd.codec_hdr) || fd.rank == 1) return;
    uint16_t c[kRleItems];
    const uint64_t i0 = (uint64_t)(t - fd.rt_base) * kRleTile + (uint64_t)threadIdx.x * kRleItems;
    const uint32_t rlo = tmap[2 * t], nr = tmap[2 * t + 1];
    if (nr == 1) {  // rlo is the value
#pragma unroll
        for (int k = 0; k < kRleItems; ++k) c[k] = (uint16_t)rlo;
    } else {
        expand_tile(fd, t, rlo, nr, starts, sm, c);
    }
    EBC_G uint16_t* __restrict__ q = fd.q;
    if (i0 + kRleItems <= fd.n) {
        *(EBC_G uint4*)(q + i0) = pack8(c);
        *(EBC_G uint4*)(q + i0 + 8) = pack8(c + 8);
    } else {
        for (int k = 0; k < kRleItems; ++k)
            if (i0 + k < fd.n) q[i0 + k] = c[k];
    }
}

hipError_t launch_rle_count(const FieldDesc* F, int nf, uint32_t units, uint32_t* rcnt, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_rle_count, dim3(min(units, kEncBlocks)), dim3(kBlock), 0, s, F, nf, rcnt, units);
    return hipGetLastError();
}

hipError_t launch_rle_vle_prep(const FieldDesc* F, int nf, uint32_t units, const uint32_t* roff,
                               uint32_t n_bins, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_rle_write, dim3(min(units, kEncBlocks)), dim3(kBlock), 0, s, F, nf, roff, roff, roff,
                       units, kRleValSym);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t g = units < kPersistentBlocks ? units : kPersistentBlocks;
    hipLaunchKernelGGL(k_rle_vhist, dim3(g), dim3(kBlock), (size_t)hist_slots(n_bins) * 4, s, F, nf, units);
    return hipGetLastError();
}

hipError_t launch_rle_decode(const FieldDesc* F, int nf, uint32_t rl_units, uint32_t rt_units,
                             uint32_t* starts, uint32_t* tmap, uint32_t* tmp, uint32_t n_starts,
                             uint32_t scan_direct, bool expand, hipStream_t s)
{
    if (!rl_units) return hipSuccess;
    hipLaunchKernelGGL(k_rle_prep, dim3(rl_units), dim3(kBlock), 0, s, F, nf, starts);
    hipError_t e = launch_scan(starts, n_starts, tmp, s, scan_direct);
    if (e != hipSuccess) return e;
    const uint32_t maps = (rt_units + kBlock - 1) / kBlock;
    if (((uint64_t)rl_units + maps) * kBlock < kMaxThreads) {
        hipLaunchKernelGGL(k_rle_map, dim3(rl_units + maps), dim3(kBlock), 0, s, F, nf, rl_units, rt_units, starts,
                           tmap);
    } else {  // nearly 2^32 runs: the checks by themselves
        hipLaunchKernelGGL(k_rle_map, dim3(rl_units), dim3(kBlock), 0, s, F, nf, rl_units, rt_units, starts, tmap);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_rle_map, dim3(maps), dim3(kBlock), 0, s, F, nf, 0u, rt_units, starts, tmap);
    }
    if (rt_units && expand)
        hipLaunchKernelGGL(k_rle_expand, dim3(rt_units), dim3(kBlock), 0, s, F, nf, starts, tmap);
    return hipGetLastError();
}

}  // namespace ebc
