// k_codebook.hip -- canonical Huffman codebook on the device, one workgroup
// per field, plus the adaptive RLE/Huffman decision and the decoder tables.
//
// Sec. II-A steps 6-7 build a canonical Huffman codebook from the histogram
// (the earlier single-thread build is named as a bottleneck in Sec. I); the
// paper does not fix the construction, so this path uses the deterministic
// two-queue method: leaves ordered by (frequency, symbol), internal nodes in
// a FIFO, the leaf wins ties.  Lengths come from the leaf counts that the merge
// leaves behind; canonical codes are assigned in (length, symbol) order, first
// code 0, code_{k+1} = (code_k + 1) << (len_{k+1} - len_k).
//
// Decision (Sec. I contribution list, Sec. III-B.2): run-length encoding when
// the Huffman average bit length is <= 1.09, i.e. 100 * sum(f*len) <= 109 * N
// in exact integers.
#include "ebc_dev.h"
#include "ebc_launch.h"

namespace ebc {

// The codebook and the decoder tables run as one workgroup per field of kCb
// threads: nothing in them is long, so one item per thread keeps each step to a
// few dependent LDS reads.
constexpr uint32_t kCb = 1024;
constexpr int kCbWaves = kCb / kWave;

// Lanes of a wave with the same value of an NB-bit number (NB ballots); a lane
// whose `on` is false is in no group.
template <int NB>
__device__ __forceinline__ uint64_t match_bits(uint32_t v, bool on)
{
    uint64_t m = ballot(on);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint64_t s = ballot((v >> b) & 1u);
        m &= (v >> b) & 1u ? s : ~s;
    }
    return m;
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Exclusive prefix over the workgroup's waves of one value per wave, and its sum.
__device__ __forceinline__ uint32_t waves_before(uint32_t v, uint32_t* s_w, uint32_t* total)
{
    const uint32_t w = threadIdx.x / kWave;
    if (lane_id() == 0) s_w[w] = v;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (uint32_t k = 0; k < (uint32_t)kCbWaves; ++k) {
        const uint32_t x = s_w[k];
        off += k < w ? x : 0u;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return off;
}

// Stable sort of m (count, symbol) pairs by count, in place in LDS: eight-bit
// digits, one pass per digit that the largest count needs.  A wave owns a
// contiguous share of at most E * 64 pairs, held in registers while the pass
// ranks them (eight ballots find the lanes with an equal digit).  dig: LDS,
// kCbWaves * 256 counters.
template <int E>
__device__ __forceinline__ void sort_by_count(uint32_t* cnt, uint16_t* sym, uint32_t m, uint32_t maxcnt,
                                              uint16_t* dig, uint32_t* s_w)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
    const uint32_t per = (m + kCb - 1) / kCb;  // batches of 64 per wave, <= E
    for (uint32_t shift = 0; shift < 32 && (maxcnt >> shift) != 0; shift += 8) {
        for (uint32_t i = threadIdx.x; i < kCbWaves * 256 / 2; i += kCb) ((uint32_t*)dig)[i] = 0;
        __syncthreads();
        uint32_t c[E], rk[E];
        uint16_t y[E];
        uint16_t* my = dig + w * 256;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t i = (w * per + e) * kWave + lane;
            const bool on = (uint32_t)e < per && i < m;
            c[e] = on ? cnt[i] : 0u;
            y[e] = on ? sym[i] : (uint16_t)0;
            if ((uint32_t)e < per) {
                const uint32_t d = (c[e] >> shift) & 255u;
                const uint64_t g = match_bits<8>(d, on);
                const uint32_t r = lanes_below(g);
                rk[e] = on ? my[d] + r : 0u;
                // the wave's LDS accesses complete in order: the counters move
                // on after every lane has read its own
                if (on && r == 0) my[d] = (uint16_t)(my[d] + __popcll(g));
            }
        }
        __syncthreads();
        // first place of every digit, and of every wave inside it
        uint32_t tot = 0;
        if (threadIdx.x < 256) {
#pragma unroll
            for (uint32_t k = 0; k < (uint32_t)kCbWaves; ++k) {
                const uint32_t x = dig[k * 256 + threadIdx.x];
                dig[k * 256 + threadIdx.x] = (uint16_t)tot;
                tot += x;
            }
        }
        const uint32_t inc = wave_incl_scan_u32(tot);
        uint32_t all;
        const uint32_t base = waves_before((uint32_t)__builtin_amdgcn_readlane((int)inc, 63), s_w, &all) + inc - tot;
        if (threadIdx.x < 256) {
#pragma unroll
            for (uint32_t k = 0; k < (uint32_t)kCbWaves; ++k) dig[k * 256 + threadIdx.x] += (uint16_t)base;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t i = (w * per + e) * kWave + lane;
            if ((uint32_t)e < per && i < m) {
                const uint32_t pos = my[(c[e] >> shift) & 255u] + rk[e];
                cnt[pos] = c[e];
                sym[pos] = y[e];
            }
        }
        __syncthreads();
    }
}

// value of lane (l ^ J)
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    const int i = (int)v;
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0xB1, 0xF, 0xF, false);
    else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0x4E, 0xF, 0xF, false);
    else if constexpr (J == 4) {
        // lanes 0-3 and 8-11 of a row take lane + 4, the others lane - 4
        const int t = __builtin_amdgcn_update_dpp(i, i, 0x104, 0xF, 0x5, false);
        return (uint32_t)__builtin_amdgcn_update_dpp(t, i, 0x114, 0xF, 0xA, false);
    } else if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(i, i, 0x128, 0xF, 0xF, false);
    else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return lane_id() & 16 ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return lane_id() & 32 ? r[0] : r[1];
    }
}
template <int J>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v)
{
    return ((uint64_t)lane_xor<J>((uint32_t)(v >> 32)) << 32) | lane_xor<J>((uint32_t)v);
}
template <int J, class K>
__device__ __forceinline__ K merge_step(K v)
{
    const K u = lane_xor<J>(v);
    return lane_id() & J ? max(u, v) : min(u, v);
}
template <class K>
__device__ __forceinline__ K key_at(K v, int lane)
{
    if constexpr (sizeof(K) == 4) return (K)__builtin_amdgcn_readlane((int)v, lane);
    else
        return ((K)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}

// Two-queue Huffman merge of m sorted leaf weights, by one wave, in rounds.
// Let t be the weight of the next internal node (the sum of the two lightest
// available items).  Every available item of weight <= t is picked before that
// node and before any later one, so all of them can be paired in merged order
// at once (ties: leaf before internal node, older internal node before newer);
// an odd one out waits for the next round.  This reproduces the sequential
// picks exactly.
//
// A round takes the next 64 leaves and 64 internal nodes into registers, a lane
// each, with keys 2 * weight + (1 for internal nodes), and merges the two sorted
// lists by a bitonic merge of lane exchanges without LDS; neighbours then are
// pairs.  Of a list with more items than its 64, only what is not above the last
// loaded key takes part.  Rounds that looked every item's place up by a binary
// search in LDS took 4200 cycles each (24 of them for 1024 symbols, 66 us for the
// kernel).  leaf(i), node(i): weights; put(i, w, l): internal node i weighs w and
// l leaves were picked before its pair.  K: 32 bits if the total is below 2^31 - 1.
template <class K, class LEAF, class NODE, class PUT>
__device__ __forceinline__ void two_queue_merge(uint32_t m, LEAF leaf, NODE node, PUT put)
{
    constexpr K kInf = ~(K)0;
    const uint32_t lane = lane_id();
    uint32_t li = 0, ih = 0, ni = 0;
    while (ni + 1 < m) {
        const uint32_t i = li + lane, j = ih + (kWave - 1) - lane;
        const K a = i < m ? (K)leaf(i) * 2 : kInf;
        const K b = j < ni ? (K)node(j) * 2 + 1 : kInf;
        const K cap_a = m - li > (uint32_t)kWave ? key_at(a, kWave - 1) : kInf;
        const K cap_b = ni - ih > (uint32_t)kWave ? key_at(b, 0) : kInf;
        // leaves ascending, nodes descending: lower and upper half, then each
        // half sorted
        K lo = min(a, b), hi = max(a, b);
        lo = merge_step<32>(lo), hi = merge_step<32>(hi);
        lo = merge_step<16>(lo), hi = merge_step<16>(hi);
        lo = merge_step<8>(lo), hi = merge_step<8>(hi);
        lo = merge_step<4>(lo), hi = merge_step<4>(hi);
        lo = merge_step<2>(lo), hi = merge_step<2>(hi);
        lo = merge_step<1>(lo), hi = merge_step<1>(hi);
        const K t = (key_at(lo, 0) >> 1) + (key_at(lo, 1) >> 1);
        const K cap = min(min(cap_a, cap_b), t * 2 + 1);
        const uint32_t cnt = __popcll(ballot(lo <= cap)) + __popcll(ballot(hi <= cap));
        const uint32_t np = cnt / 2;  // at least 1: the two lightest always pair
        if (np == 0) break;           // (bounds the loop)
        const uint64_t la = ballot((lo & 1) == 0), lb = ballot((hi & 1) == 0);  // leaves
        const uint32_t wl = (uint32_t)(lo >> 1), wh = (uint32_t)(hi >> 1);
        const uint32_t sl = wl + lane_xor<1>(wl), sh = wh + lane_xor<1>(wh);
        const uint32_t k = lane / 2;
        if ((lane & 1) == 0) {
            if (k < np) put(ni + k, sl, li + lanes_below(la));
            if (k + 32 < np) put(ni + k + 32, sh, li + __popcll(la) + lanes_below(lb));
        }
        // leaves among the first 2 np items
        const uint32_t n0 = min(2 * np, 64u), n1 = 2 * np - n0;
        const uint64_t m0 = n0 == 64 ? ~0ull : (1ull << n0) - 1, m1 = n1 == 64 ? ~0ull : (1ull << n1) - 1;
        const uint32_t dl = __popcll(la & m0) + __popcll(lb & m1);
        li += dl, ih += 2 * np - dl, ni += np;
    }
}

// Leaf depths from the leaf counts picked before each internal node's pair.
// Depths fall along both queues, so a level's internal nodes are a range
// [a, b) and its children the picks 2a .. 2b - 1: leaves from picked(a) on, and
// the internal nodes [2a - picked(a), a).  One thread: bnd[d] = first leaf (in
// sorted order) of depth d + 1; returns the number of levels.
template <class PICKED>
__device__ __forceinline__ uint32_t leaf_levels(uint32_t m, uint32_t* bnd, PICKED picked)
{
    if (m == 1) {  // a lone symbol gets one bit
        bnd[0] = 0;
        return 1;
    }
    uint32_t a = m - 2, d = 0;
    for (;;) {
        const uint32_t p = picked(a);
        bnd[d++] = p;
        const uint32_t na = 2 * a - p;
        if (na >= a || d == 64) break;
        a = na;
    }
    return d;
}

// Canonical codes in (length, symbol) order from the symbols' lengths, the
// encoder's tables, the payload bits and, for the codes' own pass, the codec
// decision.  A wave owns a contiguous share of the symbols.  len(s): length of
// symbol s; bnd, nlev: leaves per depth (leaf_levels); wc: LDS,
// kCbWaves * 64 counters.
template <class LEN>
__device__ __forceinline__ void canonical_codes(const FieldDesc& fd, EBC_G FieldDyn* dy, int pass, uint32_t m,
                                                const uint32_t* bnd, uint32_t nlev, uint32_t* wc,
                                                uint64_t* first, uint64_t* s_bits, int32_t* s_codec,
                                                const EBC_G uint32_t* __restrict__ hist, LEN len)
{
    const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
    const uint32_t nb = fd.n_bins;
    const uint32_t per = (nb + kCb - 1) / kCb;  // batches of 64 symbols per wave
    uint32_t* my = wc + w * 64;
    my[lane] = 0;
    for (uint32_t e = 0; e < per; ++e) {
        const uint32_t s = (w * per + e) * kWave + lane;
        const uint32_t L = s < nb ? len(s) : 0u;
        if (L) atomicAdd(&my[L], 1u);
    }
    if (threadIdx.x == 0) {
        // first code of each length; length L = d + 1 has the leaves from
        // bnd[d] to the previous level's
        uint64_t c = 0;
        uint32_t end = m;
        for (uint32_t d = 0; d < nlev; ++d) {
            first[d + 1] = c;
            const uint32_t p = bnd[d];
            c = (c + (end - p)) << 1;
            end = p;
        }
        dy->max_len = nlev;
        dy->n_used = m;
    }
    __syncthreads();
    if (threadIdx.x < 64) {  // symbols of each length in the waves before
        uint32_t x[kCbWaves], run = 0;
#pragma unroll
        for (int k = 0; k < kCbWaves; ++k) x[k] = wc[k * 64 + threadIdx.x];
#pragma unroll
        for (int k = 0; k < kCbWaves; ++k) {
            wc[k * 64 + threadIdx.x] = run;
            run += x[k];
        }
    }
    __syncthreads();
    uint64_t bits = 0;
    for (uint32_t e = 0; e < per; ++e) {
        const uint32_t s = (w * per + e) * kWave + lane;
        const uint32_t L = s < nb ? len(s) : 0u;
        const uint64_t g = match_bits<6>(L, L != 0);
        const uint32_t r = lanes_below(g);
        uint64_t packed = 0;
        if (L) {
            packed = ((uint64_t)L << 56) | (first[L] + my[L] + r);
            bits += (uint64_t)hist[s] * L;
            // after every lane has read its counter (LDS accesses of a wave
            // complete in order)
            if (r == 0) my[L] += __popcll(g);
        }
        if (s < nb) fd.code[s] = packed, fd.len[s] = (uint8_t)L;
    }
    bits = wave_sum_u64(bits);
    if (lane == 0) s_bits[w] = bits;
    __syncthreads();
    if (threadIdx.x == 0 && pass == 0) {
        uint64_t tb = 0;
        for (int k = 0; k < kCbWaves; ++k) tb += s_bits[k];
        dy->huff_bits = tb;
        // the 1.09-bit rule picks the run-length workflow; with VLE requested
        // its run values are Huffman-coded as well
        const bool rle = 100ull * tb <= 109ull * fd.n;
        int codec;
        switch (fd.codec_req) {
        case REQ_AUTO: codec = rle ? ARC_RLE : ARC_HUFFMAN; break;
        case REQ_AUTO_VLE: codec = rle ? ARC_RLE_VLE : ARC_HUFFMAN; break;
        case REQ_HUFFMAN: codec = ARC_HUFFMAN; break;
        case REQ_RLE: codec = ARC_RLE; break;
        default: codec = ARC_RLE_VLE; break;
        }
        dy->codec = codec;
        dy->n_out = fd.hist[0];
        *s_codec = codec;
    }
    if (pass == 0 && fd.vhist) {
        // cleared here for the histogram of the run values
        __syncthreads();
        if (*s_codec == ARC_RLE_VLE)
            for (uint32_t s = threadIdx.x; s < nb; s += kCb) fd.vhist[s] = 0;
    }
}

// The used symbols in symbol order through put(position, count, symbol); returns
// their number, and the largest count.
template <class HIST, class PUT>
__device__ __forceinline__ uint32_t compact_used(HIST hist, uint32_t nb, uint32_t* s_w, uint32_t* maxcnt, PUT put)
{
    uint32_t m = 0, mx = 0;
    for (uint32_t b0 = 0; b0 < nb; b0 += kCb) {
        const uint32_t s = b0 + threadIdx.x;
        const uint32_t h = s < nb ? hist(s) : 0u;
        const uint64_t g = ballot(h != 0);
        uint32_t tot;
        const uint32_t pos = m + waves_before(__popcll(g), s_w, &tot) + lanes_below(g);
        if (h) put(pos, h, s);
        mx = max(mx, h);
        m += tot;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o));
    if (lane_id() == 0) s_w[threadIdx.x / kWave] = mx;
    __syncthreads();
    for (int k = 0; k < kCbWaves; ++k) mx = max(mx, s_w[k]);
    __syncthreads();
    *maxcnt = mx;
    return m;
}

// LDS of the two codebook kernels, carved from one block: leaf counts and
// symbols, internal weights and picked-leaf counts (narrow bins keep all of
// them for every bin, and the code lengths), the sort's digit counters.
size_t codebook_lds_bytes(uint32_t n_bins) { return (size_t)15 * ((n_bins + 63) & ~63u) + kCbWaves * 256 * 2; }

// pass 0: the codebook of the quant-codes and the codec decision; pass 1
// (RLE+VLE fields only): the codebook of the run values, from their own
// histogram, which replaces the first in code / len.
__global__ __launch_bounds__(kCb) void k_codebook(const FieldDesc* __restrict__ F, int pass, bool direct)
{
    const FieldDesc& fd = F[blockIdx.x];
    EBC_G FieldDyn* dy = fd.dyn;
    if (dy->status != ST_OK || dy->codec == ARC_CONST) return;
    if (pass == 1 && dy->codec != ARC_RLE_VLE) return;
    const EBC_G uint32_t* __restrict__ hist = pass == 0 ? fd.hist : fd.vhist;
    const uint32_t nb = fd.n_bins, na = (nb + 63) & ~63u;
    extern __shared__ uint32_t lds32[];
    uint32_t* lw = lds32;                       // leaf weights, ascending
    uint32_t* iw = lw + na;                     // internal weights
    uint32_t* pk = iw + na;                     // leaves picked before each internal node's pair
    uint16_t* sym = (uint16_t*)(pk + na);       // leaf symbols
    uint16_t* dig = sym + na;                   // digit counters
    uint8_t* len_s = (uint8_t*)(dig + kCbWaves * 256);
    __shared__ uint32_t s_w[kCbWaves];
    __shared__ uint32_t bnd[64];
    __shared__ uint32_t s_lev;
    __shared__ uint64_t first[65];
    __shared__ uint64_t s_bits[kCbWaves];
    __shared__ int32_t s_codec;
    __shared__ uint32_t wc[kCbWaves * 64];
    uint32_t maxcnt;
    auto count = [&](uint32_t s) -> uint32_t {
        if (!direct) return hist[s];
        // few partial rows (kHistDirect): added up here instead of in a launch
        uint32_t h = 0;
#pragma unroll 8
        for (uint32_t r = 0; r < fd.hrows; ++r) h += fd.hpart[(uint64_t)r * nb + s];
        fd.hist[s] = h;
        return h;
    };
    const uint32_t m = compact_used(count, nb, s_w, &maxcnt, [&](uint32_t p, uint32_t h, uint32_t s) {
        lw[p] = h;
        sym[p] = (uint16_t)s;
    });
    if (m == 0) {
        if (threadIdx.x == 0) dy->status = ST_ERR_ARCHIVE;
        return;
    }
    sort_by_count<kMaxBins / kCb>(lw, sym, m, maxcnt, dig, s_w);
    if (threadIdx.x < (uint32_t)kWave) {
        auto leaf = [&](uint32_t i) { return lw[i]; };
        auto node = [&](uint32_t i) { return iw[i]; };
        auto put = [&](uint32_t i, uint32_t v, uint32_t l) { iw[i] = v, pk[i] = l; };
        if (fd.n < 0x7FFFFFFFull) two_queue_merge<uint32_t>(m, leaf, node, put);
        else two_queue_merge<uint64_t>(m, leaf, node, put);
        if (threadIdx.x == 0) s_lev = leaf_levels(m, bnd, [&](uint32_t i) { return pk[i]; });
    }
    for (uint32_t s = threadIdx.x; s < na / 4; s += kCb) ((uint32_t*)len_s)[s] = 0;
    __syncthreads();
    const uint32_t nlev = s_lev;
    for (uint32_t i = threadIdx.x; i < m; i += kCb) {
        uint32_t L = 1;
        for (uint32_t d = 0; d < nlev; ++d) L += bnd[d] > i ? 1u : 0u;
        len_s[sym[i]] = (uint8_t)L;
    }
    __syncthreads();
    canonical_codes(fd, dy, pass, m, bnd, nlev, wc, first, s_bits, &s_codec, hist,
                    [&](uint32_t s) { return (uint32_t)len_s[s]; });
}

// ------------------------------------------------- wide bins (> kMaxBins)
// The same construction for n_bins up to 65536.  Leaves are sorted in LDS when
// at most kWideSort symbols are used (a field with many bins seldom uses all
// of them), otherwise by a bitonic sort of 64-bit keys in a per-field scratch
// of the workspace; the merge reads its leaves from where they were sorted.
// Pending internal nodes (at most half the leaves) live in an LDS ring, the
// picked-leaf counts in the scratch.

constexpr uint32_t kWideSort = 16384;
constexpr uint32_t kWideRing = 32768;

size_t codebook_wide_scratch_bytes(uint32_t n_bins)
{
    size_t P = 1;
    while (P < n_bins) P <<= 1;
    return 8 * P + 4 * P;  // sort keys, picked-leaf counts
}

// LDS, in bytes: either leaf counts, symbols, digit counters and a ring of
// kWideSort / 2 nodes, or a ring of kWideRing nodes
constexpr uint32_t kWideLds = kWideSort * 6 + kCbWaves * 256 * 2 + kWideSort / 2 * 4;
static_assert(kWideLds >= kWideRing * 4, "either use fits");

__global__ __launch_bounds__(kCb) void k_codebook_wide(const FieldDesc* __restrict__ F, int pass)
{
    const FieldDesc& fd = F[blockIdx.x];
    EBC_G FieldDyn* dy = fd.dyn;
    if (dy->status != ST_OK || dy->codec == ARC_CONST) return;
    if (pass == 1 && dy->codec != ARC_RLE_VLE) return;
    const EBC_G uint32_t* __restrict__ hist = pass == 0 ? fd.hist : fd.vhist;
    const uint32_t nb = fd.n_bins;
    uint32_t P0 = 1;
    while (P0 < nb) P0 <<= 1;
    EBC_G uint64_t* keys = (EBC_G uint64_t*)fd.cbs;  // (count << 16) | symbol
    EBC_G uint32_t* pk = (EBC_G uint32_t*)(keys + P0);
    extern __shared__ uint32_t lds32[];
    uint32_t* lw = lds32;
    uint16_t* sym = (uint16_t*)(lw + kWideSort);
    uint16_t* dig = sym + kWideSort;
    __shared__ uint32_t s_w[kCbWaves];
    __shared__ uint32_t bnd[64];
    __shared__ uint32_t s_lev;
    __shared__ uint64_t first[65];
    __shared__ uint64_t s_bits[kCbWaves];
    __shared__ int32_t s_codec;
    __shared__ uint32_t wc[kCbWaves * 64];
    uint32_t maxcnt;
    auto count = [&](uint32_t s) { return hist[s]; };
    const uint32_t m = compact_used(count, nb, s_w, &maxcnt, [&](uint32_t p, uint32_t h, uint32_t s) {
        keys[p] = ((uint64_t)h << 16) | s;
        if (p < kWideSort) lw[p] = h, sym[p] = (uint16_t)s;
    });
    if (m == 0) {
        if (threadIdx.x == 0) dy->status = ST_ERR_ARCHIVE;
        return;
    }
    const bool in_lds = m <= kWideSort;
    if (in_lds) {
        sort_by_count<kWideSort / kCb>(lw, sym, m, maxcnt, dig, s_w);
    } else {
        // ascending bitonic sort of the m keys, padded to a power of two
        uint32_t P = 1;
        while (P < m) P <<= 1;
        for (uint32_t i = m + threadIdx.x; i < P; i += kCb) keys[i] = ~0ull;
        for (uint32_t k = 2; k <= P; k <<= 1) {
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                __syncthreads();
                for (uint32_t i = threadIdx.x; i < P; i += kCb) {
                    const uint32_t q = i ^ j;
                    if (q > i) {
                        const uint64_t a = keys[i], b = keys[q];
                        const bool up = (i & k) == 0;
                        if ((a > b) == up) keys[i] = b, keys[q] = a;
                    }
                }
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < (uint32_t)kWave) {
        uint32_t* iw = in_lds ? (uint32_t*)(dig + kCbWaves * 256) : lds32;
        const uint32_t mask = in_lds ? kWideSort / 2 - 1 : kWideRing - 1;
        auto leaf = [&](uint32_t i) { return in_lds ? lw[i] : (uint32_t)(keys[i] >> 16); };
        auto node = [&](uint32_t i) { return iw[i & mask]; };
        auto put = [&](uint32_t i, uint32_t v, uint32_t l) { iw[i & mask] = v, pk[i] = l; };
        if (fd.n < 0x7FFFFFFFull) two_queue_merge<uint32_t>(m, leaf, node, put);
        else two_queue_merge<uint64_t>(m, leaf, node, put);
    }
    __syncthreads();  // the counts in the scratch are seen by the workgroup
    if (threadIdx.x == 0) s_lev = leaf_levels(m, bnd, [&](uint32_t i) { return pk[i]; });
    for (uint32_t s = threadIdx.x; s < nb; s += kCb) fd.len[s] = 0;
    __syncthreads();
    const uint32_t nlev = s_lev;
    for (uint32_t i = threadIdx.x; i < m; i += kCb) {
        uint32_t L = 1;
        for (uint32_t d = 0; d < nlev; ++d) L += bnd[d] > i ? 1u : 0u;
        fd.len[in_lds ? (uint32_t)sym[i] : (uint32_t)keys[i] & 0xFFFFu] = (uint8_t)L;
    }
    __syncthreads();
    canonical_codes(fd, dy, pass, m, bnd, nlev, wc, first, s_bits, &s_codec, hist,
                    [&](uint32_t s) { return (uint32_t)fd.len[s]; });
}

// ------------------------------------------------------- decoder tables
// From the code lengths stored in an archive: per-length counts, first codes
// and offsets, the symbol permutation in (length, symbol) order and the two
// lookup levels.  One workgroup per field, every table entry computed by
// itself from the lengths' code-space ends: the shortest length whose end lies
// above a window is the length of the codeword it starts with.  A search over
// the lengths for every entry and a scan for the long prefixes took 18 us for
// 1024 bins (36 us for 16384).
__device__ __forceinline__ void build_dectab(const FieldDesc& fd, DecTab* T)
{
    EBC_G FieldDyn* dy = fd.dyn;
    if (dy->status != ST_OK || !huff_codec(dy->codec)) return;
    const uint32_t nb = fd.n_bins;
    const bool narrow = nb <= kMaxBins;  // the permutation is kept in LDS too
    __shared__ uint32_t wc[kCbWaves * 64];
    __shared__ uint32_t cntL[65];
    __shared__ uint64_t first[65];
    __shared__ uint32_t offs[65];
    __shared__ uint32_t end1[kLutBits + 1];   // code-space ends in first-level windows
    __shared__ uint32_t end2[kL2MaxBits + 1]; // in second-level windows, lengths above kLutBits
    __shared__ uint16_t perm_s[kMaxBins];
    __shared__ uint32_t t1[1u << kLutBits];
    __shared__ int s_bad;
    __shared__ uint32_t s_maxl;
    const uint32_t lane = lane_id(), w = threadIdx.x / kWave;
    const uint32_t per = (nb + kCb - 1) / kCb;  // batches of 64 symbols per wave
    const EBC_G uint8_t* alen = fd.arc + kHdr;
    uint32_t* my = wc + w * 64;
    my[lane] = 0;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    for (uint32_t e = 0; e < per; ++e) {
        const uint32_t s = (w * per + e) * kWave + lane;
        const uint32_t L = s < nb ? alen[s] : 0u;
        if (L > (uint32_t)kMaxDecodeLen) s_bad = 1;
        else if (L) atomicAdd(&my[L], 1u);
    }
    __syncthreads();
    if (s_bad) {
        if (threadIdx.x == 0) dy->status = ST_ERR_ARCHIVE;
        return;
    }
    if (threadIdx.x < 64) {  // symbols of each length in the waves before
        uint32_t x[kCbWaves], run = 0;
#pragma unroll
        for (int k = 0; k < kCbWaves; ++k) x[k] = wc[k * 64 + threadIdx.x];
#pragma unroll
        for (int k = 0; k < kCbWaves; ++k) {
            wc[k * 64 + threadIdx.x] = run;
            run += x[k];
        }
        cntL[threadIdx.x] = run;
        if (threadIdx.x == 0) cntL[64] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // canonical first codes; the lengths must satisfy Kraft's inequality
        // (first[L] + count[L] <= 2^L at every length), otherwise the archive
        // is corrupt and no table lookup below may be trusted
        uint64_t c = 0;
        uint32_t off = 0, maxl = 0;
        int bad = 0;
        first[0] = 0, offs[0] = 0;
        // counts read 16 at a time so that the chain waits on LDS four times
        for (int L0 = 1; L0 <= 64; L0 += 16) {
            uint32_t cl[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) cl[u] = cntL[L0 + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int L = L0 + u;
                const uint32_t n = cl[u];
                first[L] = c;
                offs[L] = off;
                off += n;
                if (L <= kMaxDecodeLen && c + n > (1ull << L)) bad = 1;
                c = L <= kMaxDecodeLen ? (c + n) << 1 : 0;
                if (n) maxl = L;
            }
        }
        T->max_len = maxl;
        s_maxl = maxl;
        if (maxl == 0 || bad) dy->status = ST_ERR_ARCHIVE;
        s_bad = bad | (maxl == 0);
    }
    __syncthreads();
    if (s_bad) return;
    const uint32_t maxl = s_maxl;
    for (uint32_t e = 0; e < per; ++e) {
        const uint32_t s = (w * per + e) * kWave + lane;
        const uint32_t L = s < nb ? alen[s] : 0u;
        const uint64_t g = match_bits<6>(L, L != 0);
        const uint32_t r = lanes_below(g);
        if (L) {
            const uint32_t pos = offs[L] + my[L] + r;
            if (narrow) perm_s[pos] = (uint16_t)s;
            T->perm[pos] = (uint16_t)s;
            // after every lane has read its counter (LDS accesses of a wave
            // complete in order)
            if (r == 0) my[L] += __popcll(g);
        }
    }
    // Longer codewords are numerically larger, so the prefixes that start one
    // longer than kLutBits are the top nlong windows, and the decoder computes
    // a second-level index from the stream bits alone.
    const uint32_t end12 = (uint32_t)(first[kLutBits] + cntL[kLutBits]);
    const uint32_t nlong = (1u << kLutBits) - end12;
    uint32_t l2k = 0;
    if (maxl > (uint32_t)kLutBits && nlong > 0) {
        l2k = min(kL2MaxBits, maxl - (uint32_t)kLutBits);
        while (l2k > 0 && (nlong << l2k) > kL2Size) --l2k;
    }
    const uint32_t l2n = l2k ? nlong << l2k : 0u;
    if (threadIdx.x <= 64) {
        const uint32_t L = threadIdx.x;
        // left-aligned ends of the code space of lengths <= L (monotone in L)
        T->endv[L] = L >= 1 && L < maxl ? (first[L] + cntL[L]) << (64 - L) : ~0ull;
        T->first[L] = first[L];
        T->offset[L] = offs[L];
        if (L <= (uint32_t)kLutBits) end1[L] = L ? (uint32_t)(first[L] + cntL[L]) << (kLutBits - L) : 0u;
        else if (L <= kLutBits + l2k) end2[L - kLutBits] = (uint32_t)(first[L] + cntL[L]) << (kLutBits + l2k - L);
        if (L == 0) T->l2k = l2k, T->l2n = l2n;
    }
    __syncthreads();
    auto perm = [&](uint32_t i) -> uint32_t { return narrow ? perm_s[i] : T->perm[i]; };
    // t1[p]: the codeword of at most kLutBits bits that the window p starts
    // with, as (length << 16) | symbol, or 0
    uint32_t ends[kLutBits];
#pragma unroll
    for (int l = 1; l < kLutBits; ++l) ends[l] = end1[l];
    for (uint32_t p = threadIdx.x; p < (1u << kLutBits); p += kCb) {
        uint32_t L = 1;
#pragma unroll
        for (int l = 1; l < kLutBits; ++l) L += p >= ends[l] ? 1u : 0u;
        t1[p] = p < end12 ? (L << 16) | perm(offs[L] + (p >> (kLutBits - L)) - (uint32_t)first[L]) : 0u;
    }
    for (uint32_t i = threadIdx.x; i < l2n; i += kCb) {
        const uint32_t v = (end12 << l2k) + i;  // kLutBits + l2k bits
        uint32_t k = 1;
        for (uint32_t l = 1; l < l2k; ++l) k += v >= end2[l] ? 1u : 0u;
        uint32_t e = 0;
        if (v < end2[l2k]) {
            const uint32_t L = kLutBits + k;
            e = (L << 16) | perm(offs[L] + (v >> (l2k - k)) - (uint32_t)first[L]);
        }
        T->l2[i] = e;
    }
    __syncthreads();
    // An entry chains up to three t1 lookups; a window with only r valid
    // leading bits (the rest zero) still decodes a codeword of length <= r
    // correctly, because such a codeword depends on its own bits only.
    for (uint32_t p = threadIdx.x; p < (1u << kLutBits); p += kCb) {
        uint64_t e = 0;
        uint32_t pos = 0, n = 0;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const uint32_t v = t1[(p << pos) & ((1u << kLutBits) - 1)];
            const uint32_t L = v >> 16;
            const bool ok = n == (uint32_t)u && L != 0 && L <= (uint32_t)kLutBits - pos;
            e |= ok ? (uint64_t)(v & 0xFFFFu) << (16 * u) : 0ull;
            pos += ok ? L : 0u;
            n += ok ? 1u : 0u;
        }
        T->lut[p] = e | ((uint64_t)pos << 48) | ((uint64_t)(2 * n) << 54);
    }
}

// Chunk c of a field: the start bits of its sub-chunks inside it (the running
// sums of the stored sub-chunk bit counts); returns its word count.
__device__ __forceinline__ uint32_t chunk_words(const FieldDesc& fd, uint32_t c, uint32_t* __restrict__ soff)
{
    const EBC_G uint16_t* __restrict__ sb = (const EBC_G uint16_t*)(fd.arc + fd.off_sbits);
    const uint32_t k = fd.hc / fd.hs;  // sub-chunks per chunk
    const uint32_t s0 = c * k, s1 = min(s0 + k, fd.n_sub);
    uint32_t run = 0;
    uint32_t s = s0;
    for (; s + 4 <= s1; s += 4) {
        uint32_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = sb[s + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            soff[fd.sub_base + s + u] = run;
            run += x[u];
        }
    }
    for (; s < s1; ++s) {
        soff[fd.sub_base + s] = run;
        run += sb[s];
    }
    return (run + 31) / 32;
}

// Huffman decompression prologue: the decoder tables of every field (workgroups
// below nf), and the offsets of its sub-chunks.  DIRECT (no field has more than
// kPrepDirect chunks): one workgroup per field scans the word counts as well,
// and no scan launches follow.  Otherwise a thread per chunk stores its word
// count for the scan.  (Tables, counts, two scan launches and a check of their
// sum were five launches, 23 us on 256x256.)
template <bool DIRECT>
__global__ __launch_bounds__(kCb) void k_dec_prep(const FieldDesc* __restrict__ F, int nf,
                                                  uint8_t* __restrict__ tabs, size_t stride,
                                                  uint32_t* __restrict__ wcnt, uint32_t* __restrict__ soff)
{
    uint32_t t = blockIdx.x;
    if (t < (uint32_t)nf) {
        build_dectab(F[t], (DecTab*)(tabs + (size_t)t * stride));
        return;
    }
    t -= (uint32_t)nf;
    if (DIRECT) {
        __shared__ uint32_t s_w[kCbWaves];
        const FieldDesc& fd = F[t];
        if (!huff_codec(fd.codec_hdr)) return;
        constexpr uint32_t kPer = kPrepDirect / kCb;
        const uint32_t c0 = threadIdx.x * kPer;
        uint32_t words[kPer], sum = 0;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) {
            words[k] = c0 + k < fd.n_hch ? chunk_words(fd, c0 + k, soff) : 0u;
            sum += words[k];
        }
        const uint32_t inc = wave_incl_scan_u32(sum);
        uint32_t tot;
        uint32_t off = waves_before((uint32_t)__builtin_amdgcn_readlane((int)inc, 63), s_w, &tot) + inc - sum;
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) {
            if (c0 + k < fd.n_hch) wcnt[fd.hch_base + c0 + k] = off;
            off += words[k];
        }
        if (threadIdx.x == 0) wcnt[fd.hch_base + fd.n_hch] = tot;
    } else {
        const int f = find_field<&FieldDesc::hpwg_base>(F, nf, t);
        const FieldDesc& fd = F[f];
        const uint32_t c = (t - fd.hpwg_base) * kCb + threadIdx.x;
        if (!huff_codec(fd.codec_hdr)) return;
        if (c == 0) wcnt[fd.hch_base + fd.n_hch] = 0;
        if (c < fd.n_hch) wcnt[fd.hch_base + c] = chunk_words(fd, c, soff);
    }
}

hipError_t launch_codebook(const FieldDesc* F, int nf, uint32_t n_bins, int pass, bool direct, hipStream_t s)
{
    if (n_bins > kMaxBins) hipLaunchKernelGGL(k_codebook_wide, dim3(nf), dim3(kCb), kWideLds, s, F, pass);
    else hipLaunchKernelGGL(k_codebook, dim3(nf), dim3(kCb), codebook_lds_bytes(n_bins), s, F, pass, direct);
    return hipGetLastError();
}

hipError_t launch_dec_prep(const FieldDesc* F, int nf, uint32_t units, bool direct, uint8_t* tabs, size_t stride,
                           uint32_t* wcnt, uint32_t* soff, hipStream_t s)
{
    if (direct)
        hipLaunchKernelGGL(k_dec_prep<true>, dim3(2 * nf), dim3(kCb), 0, s, F, nf, tabs, stride, wcnt, soff);
    else
        hipLaunchKernelGGL(k_dec_prep<false>, dim3(nf + units), dim3(kCb), 0, s, F, nf, tabs, stride, wcnt, soff);
    return hipGetLastError();
}

}  // namespace ebc
