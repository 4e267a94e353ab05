// encode_dev.h -- device code shared by the encode kernels: section offsets and
// the run-length passes (which run in launches that other work needs too).
#pragma once

#include "ebc_dev.h"

namespace ebc {

// Section offsets and total size of a field's archive from the scanned counts.
// Every kernel that writes into the archive works them out itself (a few
// scalar loads) instead of waiting for a launch that does.
struct Layout {
    uint64_t n_out, n_words, n_runs;
    uint64_t off_sbits, off_words, off_rlen, off_oidx, off_oval, total;
};

__device__ __forceinline__ uint32_t kcount(const uint32_t* p, uint64_t i)
{
    return ((const __attribute__((address_space(4))) uint32_t*)p)[i];
}

// soff, woff, roff: the scanned outlier, word and run counts
__device__ __forceinline__ Layout layout_of(const FieldDesc& fd, int32_t codec, const uint32_t* soff,
                                            const uint32_t* woff, const uint32_t* roff)
{
    if (codec == ARC_CONST) return Layout{0, 0, 0, 0, 0, 0, 0, 0, kHdr};
    const bool huff = huff_codec(codec), rle = rle_codec(codec);
    const uint64_t no = kcount(soff, (uint64_t)fd.seg_base + fd.n_seg) - kcount(soff, fd.seg_base);
    uint32_t R = 0, nw = 0;
    if (rle) R = kcount(roff, (uint64_t)fd.rt_base + fd.n_rt) - kcount(roff, fd.rt_base);
    // the Huffman stream: the N codes, or the R run values
    const uint32_t nch = rle ? (uint32_t)(((uint64_t)R + fd.hc - 1) / fd.hc) : fd.n_hch;
    const uint32_t nsub = rle ? (uint32_t)(((uint64_t)R + fd.hs - 1) / fd.hs) : fd.n_sub;
    if (huff) nw = kcount(woff, (uint64_t)fd.hch_base + nch) - kcount(woff, fd.hch_base);
    const uint64_t sbits = huff ? align16(kHdr + fd.n_bins) : 0, words = huff ? align16(sbits + 2ull * nsub) : 0;
    // run values (RLE) or the stream's words, then run lengths, then outliers
    const uint64_t first = huff ? align16(words + 4ull * nw) : align16(kHdr + 2ull * R);
    const uint64_t rlen = rle ? first : 0, oidx = rle ? align16(first + 4ull * R) : first;
    const uint64_t oval = align16(oidx + 4ull * no);
    return Layout{no, nw, R, sbits, words, rlen, oidx, oval, align16(oval + 4ull * no)};
}

// --------------------------------------------------------- run-length passes
// Runs are maximal and taken over the whole code array in row-major order
// (Sec. III-B).  Both passes stride over tiles of kRleTile codes.

constexpr int kRleItems = kRleTile / kBlock;

struct RleShared {  // double-buffered by tile, so that one barrier per tile does
    uint32_t cnt[2][kWavesPerBlock], first[2][kWavesPerBlock];
};

// Grid-stride step past field fd's RLE tiles (those of a field that is not
// run-length coded): the first tile index of this workgroup's stride at or
// beyond the field's end, so such a field costs one iteration per workgroup.
__device__ __forceinline__ uint32_t skip_field(const FieldDesc& fd, uint32_t t)
{
    const uint32_t end = fd.rt_base + fd.n_rt;
    return t + ((end - t + gridDim.x - 1) / gridDim.x) * gridDim.x;
}

// the thread's 16 codes from element i0 on (zeros past the field)
__device__ __forceinline__ void rle_codes(const FieldDesc& fd, uint64_t i0, uint16_t c[kRleItems])
{
    const EBC_G uint16_t* __restrict__ q = fd.q;
    if (i0 + kRleItems <= fd.n) {
        const uint4 a = *(const EBC_G uint4*)(q + i0);
        const uint4 b = *(const EBC_G uint4*)(q + i0 + 8);
        const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) c[2 * k] = w[k] & 0xFFFF, c[2 * k + 1] = w[k] >> 16;
    } else {
#pragma unroll
        for (int k = 0; k < kRleItems; ++k) c[k] = i0 + k < fd.n ? q[i0 + k] : 0;
    }
}

// bit k: element i0 + k starts a run (differs from its predecessor).  Every
// lane of the wave takes part.
__device__ __forceinline__ uint32_t run_flags(const FieldDesc& fd, uint64_t i0, const uint16_t c[kRleItems])
{
    // the last code of the lane before (wave_shr:1); a wave's first lane loads it
    uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c[kRleItems - 1], 0x138, 0xF, 0xF, false);
    if (lane_id() == 0 && i0 > 0 && i0 < fd.n) prev = fd.q[i0 - 1];
    uint32_t flags = 0;
#pragma unroll
    for (int k = 0; k < kRleItems; ++k) {
        flags |= (c[k] != prev ? 1u : 0u) << k;
        prev = c[k];
    }
    if (i0 == 0) flags |= 1u;
    const uint32_t nv = i0 >= fd.n ? 0u : (uint32_t)min<uint64_t>(kRleItems, fd.n - i0);
    return flags & ((1u << nv) - 1u);
}

// Count pass, 16 codes per thread: run starts per tile, each tile's first one and, where the
// workspace has room (rflag), the flags themselves, an eighth of the codes'
// bytes, so that the write pass need not read all codes again.
__device__ __forceinline__ void rle_count_tiles(const FieldDesc* __restrict__ F, int nf,
                                                uint32_t* __restrict__ rcnt, uint32_t units, RleShared& sh)
{
    const uint32_t w = threadIdx.x / kWave;
    uint32_t par = 0;
    for (uint32_t t = blockIdx.x; t < units;) {
        const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
        const FieldDesc& fd = F[f];
        const auto* dy = kconst(fd.dyn);
        if (dy->status != ST_OK || !rle_codec(dy->codec)) {
            t = skip_field(fd, t);
            continue;
        }
        const uint32_t tl = t - fd.rt_base;
        const uint64_t i0 = (uint64_t)tl * kRleTile + threadIdx.x * kRleItems;
        uint16_t c[kRleItems];
        rle_codes(fd, i0, c);
        const uint32_t flags = run_flags(fd, i0, c);
        if (fd.rflag) fd.rflag[(uint64_t)tl * kBlock + threadIdx.x] = (uint16_t)flags;
        const uint32_t cnt = wave_sum_u32(__popc(flags));
        const uint64_t fb = ballot(flags != 0);
        uint32_t first = 0xFFFFFFFFu;
        if (fb) {
            const int L = __builtin_ctzll(fb);
            first = (w * kWave + L) * kRleItems + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)flags, L));
        }
        if (lane_id() == 0) sh.cnt[par][w] = cnt, sh.first[par][w] = first;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0, fs = 0xFFFFFFFFu;
            for (int k = 0; k < kWavesPerBlock; ++k) tot += sh.cnt[par][k], fs = min(fs, sh.first[par][k]);
            rcnt[t] = tot;
            fd.rfirst[tl] = fs;
        }
        par ^= 1;
        t += gridDim.x;
    }
}

// what: kRleValArc writes the run values into the archive (RLE codec),
// kRleValSym into the run-value stream of the Huffman pass (RLE+VLE codec,
// whose run count it also records), kRleLen the run lengths (both codecs).
constexpr int kRleValArc = 1, kRleValSym = 2, kRleLen = 4;

// run-start flags of the 64 codes from element i0 on, read from the codes
__device__ __forceinline__ uint64_t run_flags64(const FieldDesc& fd, uint64_t i0)
{
    const EBC_G uint16_t* __restrict__ q = fd.q;
    if (i0 >= fd.n) return 0;
    uint32_t prev = i0 > 0 ? q[i0 - 1] : 0u;
    uint64_t m = 0;
    for (uint32_t g = 0; g < 4; ++g) {
        uint16_t c[kRleItems];
        rle_codes(fd, i0 + g * kRleItems, c);
        uint32_t flags = 0;
#pragma unroll
        for (int k = 0; k < kRleItems; ++k) {
            flags |= (c[k] != prev ? 1u : 0u) << k;
            prev = c[k];
        }
        m |= (uint64_t)flags << (16 * g);
    }
    if (i0 == 0) m |= 1u;
    return fd.n - i0 < 64 ? m & ((1ull << (fd.n - i0)) - 1) : m;
}

// Runs of a tile from which the wave writes them 64 codes at a time instead of a lane
// its own: a lane's runs follow each other, each a load and two stores of their own.
// (A compression of 4M noise values, nearly each a run: 238 us without, 145 with.)
constexpr uint32_t kDenseRuns = 1024;

// Write pass: (value, length) of the runs that start in each tile, a wave per
// tile and 64 codes per lane, so that waves need no barrier and many tiles are
// in flight (the pass is a chain of short loads: a workgroup per tile took 53 us
// on 1.2e8 codes with 9.5e5 runs).  A run ends where the next one starts: in the
// same lane, a later lane, or the next tile that has a run start (found in the
// scanned counts).  Waves `wave` of `waves` share the tiles.
__device__ __forceinline__ void rle_write_tiles(const FieldDesc* __restrict__ F, int nf,
                                                const uint32_t* __restrict__ soff,
                                                const uint32_t* __restrict__ woff,
                                                const uint32_t* __restrict__ roff, uint32_t units, int what,
                                                uint32_t wave, uint32_t waves)
{
    const uint32_t lane = lane_id();
    int cur = -1;
    bool val_arc = false, val_sym = false, lens = false, skip = true;
    uint64_t off_rlen = 0;
    for (uint32_t t = wave; t < units;) {
        const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
        const FieldDesc& fd = F[f];
        if (f != cur) {
            cur = f;
            const auto* dy = kconst(fd.dyn);
            const int32_t codec = dy->codec;
            val_arc = (what & kRleValArc) && codec == ARC_RLE;
            val_sym = (what & kRleValSym) && codec == ARC_RLE_VLE;
            lens = (what & kRleLen) && rle_codec(codec);
            skip = dy->status != ST_OK || !(val_arc || val_sym || lens);
            if (!skip && (val_arc || lens)) {
                const Layout y = layout_of(fd, codec, soff, woff, roff);
                skip = y.total > fd.arc_cap;
                off_rlen = y.off_rlen;
            }
        }
        if (skip) {
            const uint32_t end = fd.rt_base + fd.n_rt;
            t += ((end - t + waves - 1) / waves) * waves;
            continue;
        }
        const uint32_t tl = t - fd.rt_base, r0 = kcount(roff, fd.rt_base);
        const uint32_t a = kcount(roff, t), b = kcount(roff, (uint64_t)t + 1);
        t += waves;
        if (val_sym && tl == 0 && lane == 0)
            fd.dyn->n_runs = kcount(roff, (uint64_t)fd.rt_base + fd.n_rt) - r0;
        if (a == b) continue;  // no run starts here
        const uint64_t i0 = (uint64_t)tl * kRleTile + lane * 64;
        uint64_t m = fd.rflag ? ((const EBC_G uint64_t*)fd.rflag)[(uint64_t)tl * kWave + lane] : run_flags64(fd, i0);
        // where the tile's last run ends: the first tile after this one whose
        // scanned count moves on
        uint32_t after = (uint32_t)fd.n;
        if (lens) {
            uint32_t lo = tl + 1, hi = fd.n_rt;
            if (lo < hi && kcount(roff, (uint64_t)fd.rt_base + lo + 1) != b) hi = lo;
            while (lo < hi) {
                const uint32_t md = (lo + hi) >> 1;
                if (kcount(roff, (uint64_t)fd.rt_base + md + 1) != b) hi = md;
                else lo = md + 1;
            }
            if (lo < fd.n_rt) after = lo * kRleTile + fd.rfirst[lo];
        }
        const uint32_t cnt = __popcll(m);
        uint32_t pos = a - r0 + wave_incl_scan_u32(cnt) - cnt;
        // the first start of a later lane
        const uint64_t fb = ballot(m != 0);
        const uint32_t mine = m ? (uint32_t)i0 + __builtin_ctzll(m) : 0u;
        const uint64_t later = lane == kWave - 1 ? 0ull : fb >> (lane + 1);
        const uint32_t nl = (uint32_t)__shfl((int)mine, later ? (int)(lane + 1 + __builtin_ctzll(later)) : (int)lane);
        if (later) after = nl;
        EBC_G uint16_t* val = val_arc ? (EBC_G uint16_t*)(fd.arc + kHdr) : fd.vsym;
        EBC_G uint32_t* len = (EBC_G uint32_t*)(fd.arc + off_rlen);
        if (b - a > kDenseRuns) {
            // 64 consecutive codes per step, so that loads and stores are contiguous
            uint32_t at = a - r0;
#pragma unroll 4
            for (uint32_t g = 0; g < kWave; ++g) {
                const uint64_t mg = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), g) << 32 |
                                    (uint32_t)__builtin_amdgcn_readlane((int)m, g);
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)after, g);
                const uint32_t p = tl * kRleTile + g * 64 + lane;
                if ((mg >> lane) & 1u) {
                    const uint64_t next = mg >> lane >> 1;
                    const uint32_t o = at + __popcll(mg & ((1ull << lane) - 1));
                    if (val_arc || val_sym) val[o] = fd.q[p];
                    if (lens) len[o] = (next ? p + 1 + __builtin_ctzll(next) : end) - p;
                }
                at += __popcll(mg);
            }
            continue;
        }
        while (m) {
            const uint32_t k = __builtin_ctzll(m);
            m &= m - 1;
            if (val_arc || val_sym) val[pos] = fd.q[i0 + k];
            if (lens) len[pos] = (m ? (uint32_t)i0 + __builtin_ctzll(m) : after) - ((uint32_t)i0 + k);
            ++pos;
        }
    }
}

}  // namespace ebc
