// k_huffman.hip -- chunked canonical Huffman encoding and decoding.
//
// Sec. II-A steps 7-8: encode the quant-codes with the codebook and
// concatenate ("deflate") the codewords.  The stream is cut into chunks of hc
// symbols so both directions run chunk-parallel; each chunk starts on a 32-bit
// word, bits are packed MSB-first, and the per-chunk bit counts are stored so
// a decoder can locate every chunk (Sec. III-B.2 mentions the chunk-wise
// metadata).  Sec. V-C notes that writing a word only once it is full saves
// DRAM stores: here every chunk is assembled in LDS and leaves with
// coalesced full-word stores.
//
// Encode: one wavefront per chunk (k_huff_bits counts bits; after a scan of
// the word counts k_huff_write packs with LDS atomic ORs and copies out).
// Decode: one lane per sub-chunk; a kLutBits-wide table yields up to three short
// codewords per lookup, longer codewords use a second table or the canonical
// limit test.
#include "encode_dev.h"
#include "ebc_launch.h"

namespace ebc {


// words of a wave's buffer in the write pass: 32 bits per symbol of a chunk (a
// chunk of more is packed in two rounds: that takes a field of some 1e8
// elements, most of one code); the passes of chunks longer than kPassHc keep room
// for 64
__host__ __device__ constexpr uint32_t huff_buf_words(uint32_t hc) { return hc <= kPassHc ? hc + 2 : 2 * kPassHc; }

size_t huff_write_lds_bytes(uint32_t n_bins, uint32_t hc)
{
    // code table (none for wide bins, whose table stays in HBM), then the word
    // buffers
    return (size_t)(n_bins > kMaxBins ? 0 : n_bins) * 8 + (size_t)huff_cpw(hc) * huff_buf_words(hc) * 4;
}

// The writer's table entry for symbol s (see write_entry), for wide bins
// built from the codebook in HBM on every lookup.
__device__ __forceinline__ uint64_t write_entry(uint64_t packed);

// Symbols [lo, lo + S) of a chunk (S = hc / 64, owned by one lane), kept as
// raw 16-byte blocks so that the loads can be issued one work unit ahead and
// unpacked only when the unit is processed.
template <uint32_t S>
struct SymRaw {
    static constexpr uint32_t NV = S >= 8 ? S / 8 : 1;
    uint4 v[NV];
    __device__ __forceinline__ uint32_t at(uint32_t k) const
    {
        const uint4& b = v[k / 8];
        const uint32_t h = (k % 8) / 2;
        const uint32_t w = h == 0 ? b.x : h == 1 ? b.y : h == 2 ? b.z : b.w;
        return (w >> (16 * (k & 1))) & 0xFFFFu;
    }
};

template <uint32_t S>
__device__ __forceinline__ void load_raw(const EBC_G uint16_t* __restrict__ q, uint64_t lo, uint64_t n,
                                         SymRaw<S>& r)
{
    if (S >= 8 && lo + S <= n) {
#pragma unroll
        for (uint32_t k = 0; k < SymRaw<S>::NV; ++k) r.v[k] = *(const EBC_G uint4*)(q + lo + 8 * k);
    } else {  // short chunks and the field's tail: assembled here
        uint32_t w[4 * SymRaw<S>::NV];
#pragma unroll
        for (uint32_t k = 0; k < 4 * SymRaw<S>::NV; ++k) w[k] = 0;
#pragma unroll
        for (uint32_t k = 0; k < S; ++k)
            if (lo + k < n) w[k / 2] |= (uint32_t)q[lo + k] << (16 * (k & 1));
#pragma unroll
        for (uint32_t k = 0; k < SymRaw<S>::NV; ++k)
            r.v[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
    }
}

// The coded stream of a field: its quant-codes (Huffman codec) or its run values
// (RLE+VLE codec, as many as the run count found on the device); `which` selects
// the codecs a launch covers: 0 Huffman, 1 RLE+VLE, 2 both.  A workgroup keeps
// it while it stays in the field's work units [lo, hi): looked up for every
// unit, the chain of scalar loads through descriptor and device scalars was
// most of a unit's time.
struct EncField {
    int f;
    uint32_t lo, hi;
    bool ok;                         // field is being Huffman-coded by this launch
    const EBC_G uint16_t* src;       // symbols of the stream
    uint64_t cnt;                    // symbols in the stream
    uint32_t nch, nsub;              // its chunks and sub-chunks
    uint32_t hch;                    // its first entry among the word counts
};

__device__ __forceinline__ EncField enc_field(const FieldDesc* __restrict__ F, int nf, uint32_t t, int which)
{
    EncField e;
    e.f = find_field<&FieldDesc::hwg_base>(F, nf, t);
    const FieldDesc& fd = F[e.f];
    const auto* dk = kconst(fd.dyn);
    const int32_t codec = dk->codec;
    e.lo = fd.hwg_base, e.hi = fd.hwg_base + fd.hwg_units;
    e.ok = dk->status == ST_OK &&
           (which == 0 ? codec == ARC_HUFFMAN : which == 1 ? codec == ARC_RLE_VLE : huff_codec(codec));
    const bool vle = codec == ARC_RLE_VLE;
    e.src = vle ? fd.vsym : fd.q;
    e.cnt = vle ? dk->n_runs : fd.n;
    e.nch = vle ? (uint32_t)((e.cnt + fd.hc - 1) / fd.hc) : fd.n_hch;
    e.nsub = vle ? (uint32_t)((e.cnt + fd.hs - 1) / fd.hs) : fd.n_sub;
    e.hch = fd.hch_base;
    return e;
}

// One encode work unit: huff_cpw(hc) chunks, one per wavefront.
struct EncUnit {
    EncField e;
    uint32_t c;   // this wave's chunk
    uint32_t wo;  // its scanned word offset (write pass)
    bool ok;
};

// The first unit from t on, in this workgroup's stride, that the launch codes;
// the units of a field that it does not code (or past a short value stream)
// are stepped over at once.  Past the end the unit is dead (ok false, the
// stream of whatever unit it held or passed last).
template <uint32_t S>
__device__ __forceinline__ uint32_t enc_seek(const FieldDesc* __restrict__ F, int nf, uint32_t t, uint32_t units,
                                             int which, const uint32_t* __restrict__ woff, EncUnit& u)
{
    constexpr uint32_t kCpw = huff_cpw(64 * S);
    u.ok = false;
    while (t < units) {
        if (t < u.e.lo || t >= u.e.hi) u.e = enc_field(F, nf, t, which);
        if (u.e.ok && (t - u.e.lo) * kCpw < u.e.nch) {
            // blockDim = 64 * cpw; the chunk index is wave-uniform (scalar)
            u.c = (t - u.e.lo) * kCpw + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
            if (woff) u.wo = kcount(woff, (uint64_t)u.e.hch + min(u.c, u.e.nch - 1));
            u.ok = true;
            return t;
        }
        t += ((u.e.hi - t + gridDim.x - 1) / gridDim.x) * gridDim.x;
    }
    return t;
}

// For S >= 8 the loads are unconditional (a lane with nothing to load reads
// the start of the stream instead), so every pipeline stage issues the same
// number of loads and the compiler's wait counts never have to assume a stage
// without them.  Symbols past the stream's end are masked by the users; the
// tail chunk's last lane may read up to 30 bytes past the stream, which the
// workspace always follows with other scratch.
template <uint32_t S>
__device__ __forceinline__ void enc_issue(const EncUnit& u, SymRaw<S>& r)
{
    const uint64_t lo = (uint64_t)u.c * (64 * S) + (uint64_t)lane_id() * S;
    const bool live = u.ok && u.c < u.e.nch && lo < u.e.cnt;
    if (S >= 8) {
        const EBC_G uint16_t* p = u.e.src + (live ? lo : 0);
#pragma unroll
        for (uint32_t k = 0; k < SymRaw<S>::NV; ++k) r.v[k] = *(const EBC_G uint4*)(p + 8 * k);
    } else if (live) {
        load_raw<S>(u.e.src, lo, u.e.cnt, r);
    }
}

// Grid-stride walk over the work units with the next unit's symbols in
// flight while the current one is processed (two static buffers, so no
// register copy ever waits on a load).  proc(unit, symbols) must treat the
// workgroup uniformly (it may synchronise).  woff: scanned word offsets, or NULL.
template <uint32_t S, class Proc>
__device__ __forceinline__ void enc_pipeline(const FieldDesc* __restrict__ F, int nf, uint32_t units,
                                             int which, const uint32_t* __restrict__ woff, Proc& proc)
{
    SymRaw<S> A, B;
    EncUnit ua;
    ua.e.lo = ua.e.hi = 0, ua.wo = 0;
    uint32_t t = enc_seek<S>(F, nf, blockIdx.x, units, which, woff, ua);
    if (t >= units) return;
    EncUnit ub = ua;  // a dead unit still names a stream that can be read
    enc_issue<S>(ua, A);
    for (;;) {
        // the next stage's loads are always issued (a dead unit past the end)
        t = enc_seek<S>(F, nf, t + gridDim.x, units, which, woff, ub);
        enc_issue<S>(ub, B);
        proc(ua, A);
        if (t >= units) break;
        t = enc_seek<S>(F, nf, t + gridDim.x, units, which, woff, ua);
        enc_issue<S>(ua, A);
        proc(ub, B);
        if (t >= units) break;
    }
}

// Both encode kernels are persistent: a workgroup walks groups of
// huff_cpw(hc) chunks with a grid stride and reloads the code table in LDS
// only when it moves to another field.
// W: wide bins (n_bins > kMaxBins), whose lengths are read from HBM
template <uint32_t S, bool W>
struct BitsProc {
    const FieldDesc* F;
    uint32_t* wcnt;
    uint8_t* len_s;
    int cur;
    const EBC_G uint8_t* len;
    __device__ __forceinline__ void operator()(const EncUnit& u, const SymRaw<S>& r)
    {
        if (!u.ok) return;
        if (u.e.f != cur) {
            const FieldDesc& fd = F[u.e.f];
            len = fd.len;
            if (!W) {
                __syncthreads();
                for (uint32_t s = threadIdx.x; s < fd.n_bins; s += kWave * huff_cpw(64 * S)) len_s[s] = len[s];
                __syncthreads();
            }
            cur = u.e.f;
        }
        if (u.c >= u.e.nch) return;
        const uint64_t lo = (uint64_t)u.c * (64 * S) + (uint64_t)lane_id() * S;
        // symbols past the stream's end count zero bits; every lookup is
        // issued before any is used
        const uint32_t m = lo < u.e.cnt ? (uint32_t)min<uint64_t>(S, u.e.cnt - lo) : 0u;
        uint32_t bits = 0;
        if (__all(m == S)) {
            // every lane holds S symbols (all chunks but a field's last)
#pragma unroll
            for (uint32_t k = 0; k < S; ++k) bits += W ? len[r.at(k)] : len_s[r.at(k)];
        } else {
#pragma unroll
            for (uint32_t k = 0; k < S; ++k) {
                const uint32_t L = W ? len[k < m ? r.at(k) : 0u] : len_s[k < m ? r.at(k) : 0u];
                bits += k < m ? L : 0u;
            }
        }
        bits = wave_sum_u32(bits);
        if (lane_id() == 0) wcnt[u.e.hch + u.c] = (bits + 31) / 32;
    }
};

// Bits of the Huffman fields' chunks; with rt_units (workgroups of kBlock
// threads), run starts of the run-length fields' tiles as well, which saves a
// launch that most fields have no use for.
template <uint32_t S, bool W>
__global__ __launch_bounds__(kBlock) void k_huff_bits(const FieldDesc* __restrict__ F, int nf,
                                                      uint32_t* __restrict__ wcnt, uint32_t units,
                                                      int which, uint32_t rt_units,
                                                      uint32_t* __restrict__ rcnt)
{
    __shared__ uint8_t len_s[W ? 1 : kMaxBins];
    __shared__ RleShared sh;
    if (rt_units) rle_count_tiles(F, nf, rcnt, rt_units, sh);
    BitsProc<S, W> proc{F, wcnt, len_s, -1, nullptr};
    enc_pipeline<S>(F, nf, units, which, nullptr, proc);
}

// append the low `take` (<= 32) bits of v to a window that starts on a word
// boundary; full words are ORed into the chunk's LDS word buffer
__device__ __forceinline__ void put_bits(uint64_t& acc, uint32_t& nacc, uint32_t& w, uint32_t* wbuf,
                                         uint64_t v, uint32_t take)
{
    acc |= v << (64 - nacc - take);
    nacc += take;
    if (nacc >= 32) {
        atomicOr(&wbuf[w], (uint32_t)(acc >> 32));
        ++w;
        acc <<= 32;
        nacc -= 32;
    }
}

// The writer's LDS copy of the codebook: a codeword of at most 32 bits sits
// left-aligned in the high word with its length in the low byte, so that
// appending it is one shift and one OR; a longer codeword keeps only its
// length here and is read from the codebook itself.
__device__ __forceinline__ uint64_t write_entry(uint64_t packed)
{
    const uint32_t L = (uint32_t)(packed >> 56);
    if (L == 0 || L > 32) return L;
    return ((uint64_t)((uint32_t)packed << (32 - L)) << 32) | L;
}

// The entry of lanes with at most 16 symbols: the codeword right-aligned in the
// high word (a longer one than 32 bits as its length only), its length below.
__device__ __forceinline__ uint64_t join_entry(uint64_t packed)
{
    const uint32_t L = (uint32_t)(packed >> 56);
    return ((uint64_t)(L <= 32 ? (uint32_t)packed : 0u) << 32) | L;
}

// OR a piece of L <= 64 bits, right-aligned in v, into the word buffer at bit b
__device__ __forceinline__ void or_bits(uint32_t* wbuf, uint32_t b, uint64_t v, uint32_t L)
{
    const uint64_t x = v << ((64 - L) & 63);  // left-aligned (an empty piece is 0)
    const uint32_t hi = (uint32_t)(x >> 32), lo = (uint32_t)x, s = b & 31;
    uint32_t* w = wbuf + (b >> 5);
    atomicOr(w, hi >> s);
    if (s + L > 32) {
        atomicOr(w + 1, __builtin_amdgcn_alignbit(hi, lo, s));
        if (s + L > 64) atomicOr(w + 2, __builtin_amdgcn_alignbit(lo, 0u, s));
    }
}

// OR the part of a codeword of 1 <= L <= 56 bits at bit b that lies in the n words
// from word `from` on into a buffer of those words
__device__ __forceinline__ void or_long(uint32_t* wbuf, uint32_t from, uint32_t n, uint32_t b, uint64_t cw, uint32_t L)
{
    const uint64_t x = cw << (64 - L);
    const uint32_t hi = (uint32_t)(x >> 32), lo = (uint32_t)x, s = b & 31;
    const uint32_t w = (b >> 5) - from;  // (words before `from` wrap to large values)
    if (w < n) atomicOr(wbuf + w, hi >> s);
    if (s + L > 32 && w + 1 < n) atomicOr(wbuf + (w + 1), __builtin_amdgcn_alignbit(hi, lo, s));
    if (s + L > 64 && w + 2 < n) atomicOr(wbuf + (w + 2), __builtin_amdgcn_alignbit(lo, 0u, s));
}

// append a codeword of L <= 32 bits given left-aligned in cw
__device__ __forceinline__ void put_left(uint64_t& acc, uint32_t& nacc, uint32_t& w, uint32_t* wbuf,
                                         uint32_t cw, uint32_t L)
{
    acc |= (uint64_t)cw << (32 - nacc);
    nacc += L;
    if (nacc >= 32) {
        atomicOr(&wbuf[w], (uint32_t)(acc >> 32));
        ++w;
        acc <<= 32;
        nacc -= 32;
    }
}

template <uint32_t S, bool W>
struct WriteProc {
    const FieldDesc* F;
    const uint32_t *soff, *woff, *roff;
    uint64_t* lds64;
    int cur;
    bool fits;                  // field cur's archive fits into its buffer
    EBC_G uint32_t* words;      // its sections
    EBC_G uint16_t* sbits;
    uint32_t wfirst;            // scanned word offset of its first chunk
    const EBC_G uint64_t* code;
    uint32_t tab;               // entries of the LDS code table
    // Lanes of up to 16 symbols keep their table entries in registers and join
    // them by shifts before they touch the word buffer; wider lanes look them up
    // twice and append them one by one.
    static constexpr bool kKeep = S <= 16;
    __device__ __forceinline__ static uint64_t make_entry(uint64_t packed)
    {
        return kKeep ? join_entry(packed) : write_entry(packed);
    }
    __device__ __forceinline__ uint64_t entry(const uint64_t* code_s, uint32_t sym) const
    {
        return W ? make_entry(code[sym]) : code_s[sym];
    }
    // The lane's symbols as pieces of neighbours: pairs of at most 32 bits, fours
    // and eights of at most 64.  A wave whose pieces all fit ORs one (S <= 8) or
    // two pieces of eight per lane into its buffer, or fours where eights are too
    // long: 7 vector instructions per symbol instead of 24 for appending the
    // codewords one by one behind a branch (512^3: 109 to 100 us; 64M walk 41 to 31).
    // False: a pair or a four is too long (or a codeword is).
    __device__ __forceinline__ static bool join(const uint64_t (&e)[kKeep ? S : 1], uint64_t (&p4)[(S + 3) / 4],
                                                uint32_t (&l4)[(S + 3) / 4], uint32_t& bits)
    {
        bool ok = true;
        bits = 0;
#pragma unroll
        for (uint32_t g = 0; g < (S + 3) / 4; ++g) {
            uint32_t c[4] = {0, 0, 0, 0}, L[4] = {0, 0, 0, 0};
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (4 * g + k < S) c[k] = (uint32_t)(e[4 * g + k] >> 32), L[k] = (uint32_t)e[4 * g + k];
            const uint32_t la = L[0] + L[1], lb = L[2] + L[3];
            ok = ok && max(la, lb) <= 32;
            const uint32_t a = (c[0] << (L[1] & 31)) | c[1], b = (c[2] << (L[3] & 31)) | c[3];
            p4[g] = ((uint64_t)a << (lb & 63)) | b;
            l4[g] = la + lb;
            bits += l4[g];
        }
        return ok;
    }
    __device__ __forceinline__ void operator()(const EncUnit& u, const SymRaw<S>& r)
    {
        if (!u.ok) return;
        constexpr uint32_t hc = 64 * S, hs = hc < kSubMax ? hc : kSubMax;
        uint64_t* code_s = lds64;
        if (u.e.f != cur) {
            const FieldDesc& fd = F[u.e.f];
            const Layout y = layout_of(fd, kconst(fd.dyn)->codec, soff, woff, roff);
            fits = y.total <= fd.arc_cap;
            words = (EBC_G uint32_t*)(fd.arc + y.off_words);
            wfirst = kcount(woff, u.e.hch);
            sbits = (EBC_G uint16_t*)(fd.arc + y.off_sbits);
            code = fd.code;
            tab = W ? 0u : fd.n_bins;
            if (!W) {
                __syncthreads();
                for (uint32_t s = threadIdx.x; s < tab; s += kWave * huff_cpw(hc)) code_s[s] = make_entry(code[s]);
                __syncthreads();
            }
            cur = u.e.f;
        }
        if (!fits) return;
        // Each wave packs its chunk in a word buffer of its own, and a wave's
        // LDS accesses complete in order, so clearing, packing and copying
        // out need no barrier; only a new field's code table (shared by the
        // workgroup, whose waves all work on one field) does.
        uint32_t* wbuf = (uint32_t*)(lds64 + tab) + (threadIdx.x / kWave) * huff_buf_words(hc);
        const bool live = u.c < u.e.nch;
        const uint64_t lo = (uint64_t)u.c * hc + (uint64_t)lane_id() * S;
        // symbols past the stream's end take the empty entry
        const uint32_t m = live && lo < u.e.cnt ? (uint32_t)min<uint64_t>(S, u.e.cnt - lo) : 0u;
        uint64_t e[kKeep ? S : 1];
        uint32_t mybits = 0;
        if (__all(m == S)) {
            // every lane holds S symbols (all chunks but a field's last)
#pragma unroll
            for (uint32_t k = 0; k < S; ++k) {
                const uint64_t v = entry(code_s, r.at(k));
                if (kKeep) e[kKeep ? k : 0] = v;
                else mybits += (uint32_t)v & 0xFFu;
            }
        } else {
#pragma unroll
            for (uint32_t k = 0; k < S; ++k) {
                const uint64_t v0 = entry(code_s, k < m ? r.at(k) : 0u);
                const uint64_t v = k < m ? v0 : 0ull;
                if (kKeep) e[kKeep ? k : 0] = v;
                else mybits += (uint32_t)v & 0xFFu;
            }
        }
        constexpr uint32_t kFours = (S + 3) / 4;
        uint64_t p4[kFours];
        uint32_t l4[kFours];
        bool joined = false;
        if constexpr (kKeep) joined = __all(join(e, p4, l4, mybits));
        if (!live) return;
        const uint32_t incl = wave_incl_scan_u32(mybits);
        const uint32_t b0 = incl - mybits;
        const uint32_t nw = ((uint32_t)__builtin_amdgcn_readlane((int)incl, 63) + 31) / 32;  // the chunk's words
        // Offsets count modulo 2^32, from whatever the counts scanned before this
        // field's add up to (those of a field that is not coded are never written):
        // only the difference of two offsets of one field is a place.
        EBC_G uint32_t* dst = words + (uint32_t)(u.wo - wfirst);
        // sub-chunk bit counts (u16): one per kSubMax symbols of the chunk, or
        // one for the whole chunk when it is shorter; a sub-chunk's count is
        // the scan at its last lane minus b0 at its first
        constexpr uint32_t kLps = kSubMax / S < 64 ? kSubMax / S : 64u;
        const uint32_t sb = (uint32_t)__shfl((int)incl, (int)min<uint32_t>(lane_id() + kLps - 1, 63)) - b0;
        const uint64_t sub = (uint64_t)u.c * (hc / hs) + lane_id() / kLps;
        if (lane_id() % kLps == 0 && lo < u.e.cnt && sub < u.e.nsub) sbits[sub] = (uint16_t)sb;
        if (__builtin_expect(nw > hc, 0)) {
            // more than 32 bits per symbol: as many words as the buffer has at a time
            for (uint32_t from = 0; from < nw; from += hc) {
                for (uint32_t i = lane_id(); i < hc; i += kWave) wbuf[i] = 0;
                uint32_t b = b0;
                for (uint32_t k = 0; k < m; ++k) {
                    const uint64_t cw = code[u.e.src[lo + k]];
                    const uint32_t L = (uint32_t)(cw >> 56);
                    or_long(wbuf, from, hc, b, cw & ((1ull << 56) - 1), L);
                    b += L;
                }
                for (uint32_t i = lane_id(); i < min(nw - from, hc); i += kWave) dst[from + i] = wbuf[i];
            }
            return;
        }
        for (uint32_t i = lane_id(); i < nw; i += kWave) wbuf[i] = 0;
        if (joined) {
            uint32_t b = b0;
            uint32_t longest = 0;
#pragma unroll
            for (uint32_t g = 0; g + 1 < kFours; g += 2) longest = max(longest, l4[g] + l4[g + 1]);
            if (kFours > 1 && __all(longest <= 64)) {
#pragma unroll
                for (uint32_t g = 0; g < kFours; g += 2) {
                    const uint32_t g1 = g + 1 < kFours ? g + 1 : g;
                    const uint32_t L = l4[g] + l4[g1];
                    // (a second four of 64 bits leaves none for the first)
                    const uint64_t v = (l4[g1] < 64 ? p4[g] << (l4[g1] & 63) : 0ull) | p4[g1];
                    or_bits(wbuf, b, v, L);
                    b += L;
                }
            } else {
#pragma unroll
                for (uint32_t g = 0; g < kFours; ++g) {
                    or_bits(wbuf, b, p4[g], l4[g]);
                    b += l4[g];
                }
            }
        } else {
            uint32_t w = b0 >> 5, nacc = b0 & 31;
            uint64_t acc = 0;
#pragma unroll
            for (uint32_t k = 0; k < S; ++k) {
                const uint64_t v = kKeep ? e[kKeep ? k : 0] : (k < m ? entry(code_s, r.at(k)) : 0ull);
                const uint32_t L = (uint32_t)v & 0xFFu;
                if (L <= 32) {
                    const uint32_t c = (uint32_t)(v >> 32);
                    put_left(acc, nacc, w, wbuf, kKeep ? (L ? c << (32 - L) : 0u) : c, L);
                } else {
                    const uint64_t cw = code[r.at(k)] & ((1ull << 56) - 1);
                    put_bits(acc, nacc, w, wbuf, cw >> 32, L - 32);
                    put_bits(acc, nacc, w, wbuf, cw & 0xFFFFFFFFull, 32);
                }
            }
            if (nacc) atomicOr(&wbuf[w], (uint32_t)(acc >> 32));
        }
        for (uint32_t i = lane_id(); i < nw; i += kWave) dst[i] = wbuf[i];
    }
};

// A wave looks up its chunk's codewords, packs them in LDS and copies the words out.
// Bound by latency (table and word buffer in LDS, an atomic OR per piece) at 20
// waves per CU; 25 KB of LDS per workgroup of 1024 bins and the field's pointers kept
// from unit to unit gave 100 -> 88 us on 512^3 against 40 KB and a walk through the
// descriptors for every unit, the fifth workgroup per CU 80 us (two bytes per symbol
// read at the copy rate: 52).  64M walk 30 -> 23, batch of 16 fields 67 -> 58.
template <uint32_t S, bool W>
__global__ __launch_bounds__(kBlock) void k_huff_write(const FieldDesc* __restrict__ F, int nf,
                                                       const uint32_t* __restrict__ soff,
                                                       const uint32_t* __restrict__ woff,
                                                       const uint32_t* __restrict__ roff, uint32_t units)
{
    extern __shared__ uint64_t lds64[];
    WriteProc<S, W> proc{F, soff, woff, roff, lds64, -1, false, nullptr, nullptr, 0, nullptr, 0};
    enc_pipeline<S>(F, nf, units, 2, woff, proc);
}

// ------------------------------------------------ chunks longer than kPassHc
// One wave per chunk, in passes of kPassHc symbols (64 per lane).  The bit
// count pass sums code lengths per sub-chunk (4 lanes) and per chunk; the
// write pass packs each pass into an LDS word buffer starting at the bit
// offset the previous passes reached (its partial last word carried over as
// the buffer's first word), copies out the complete words and keeps the
// partial one for the next pass.
constexpr uint32_t kPassPerLane = kPassHc / kWave;  // 64 symbols
static_assert(kSubMax % kPassPerLane == 0, "a sub-chunk is a whole number of lanes");

// a work unit: one chunk
struct LongUnit {
    int f;
    uint32_t c;
    bool ok;
    const EBC_G uint16_t* src;
    uint64_t cnt;
    uint32_t nch;
};
__device__ __forceinline__ LongUnit long_unit(const FieldDesc* __restrict__ F, int nf, uint32_t t, int which)
{
    const EncField e = enc_field(F, nf, t, which);
    return LongUnit{e.f, t - e.lo, e.ok, e.src, e.cnt, e.nch};
}

__device__ __forceinline__ void load_pass(const LongUnit& u, uint64_t lo, uint32_t sym[kPassPerLane])
{
    const uint64_t i0 = lo + (uint64_t)lane_id() * kPassPerLane;
    if (i0 + kPassPerLane <= u.cnt) {
#pragma unroll
        for (uint32_t k = 0; k < kPassPerLane / 8; ++k) {
            const uint4 v = *(const EBC_G uint4*)(u.src + i0 + 8 * k);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int h = 0; h < 4; ++h) sym[8 * k + 2 * h] = w[h] & 0xFFFF, sym[8 * k + 2 * h + 1] = w[h] >> 16;
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < kPassPerLane; ++k) sym[k] = i0 + k < u.cnt ? u.src[i0 + k] : 0xFFFFFFFFu;
    }
}

template <bool W>
__global__ __launch_bounds__(kWave) void k_huff_bits_long(const FieldDesc* __restrict__ F, int nf,
                                                          uint32_t* __restrict__ wcnt, uint32_t units,
                                                          int which)
{
    __shared__ uint8_t len_s[W ? 1 : kMaxBins];
    int cur = -1;
    for (uint32_t t = blockIdx.x; t < units; t += gridDim.x) {
        const LongUnit u = long_unit(F, nf, t, which);
        if (!u.ok) continue;
        const FieldDesc& fd = F[u.f];
        if (!W && u.f != cur) {
            for (uint32_t s = threadIdx.x; s < fd.n_bins; s += kWave) len_s[s] = fd.len[s];
            cur = u.f;
        }
        if (u.c >= u.nch) continue;
        uint64_t bits = 0;
        for (uint32_t p = 0; p < fd.hc / kPassHc; ++p) {
            const uint64_t lo = (uint64_t)u.c * fd.hc + (uint64_t)p * kPassHc;
            if (lo >= u.cnt) break;
            uint32_t sym[kPassPerLane];
            load_pass(u, lo, sym);
            uint32_t b = 0;
#pragma unroll
            for (uint32_t k = 0; k < kPassPerLane; ++k)
                b += sym[k] == 0xFFFFFFFFu ? 0u : (W ? fd.len[sym[k]] : len_s[sym[k]]);
            bits += wave_sum_u32(b);
        }
        if (lane_id() == 0) {
            wcnt[fd.hch_base + u.c] = (uint32_t)((bits + 31) / 32);
        }
    }
}

template <bool W>
__global__ __launch_bounds__(kWave) void k_huff_write_long(const FieldDesc* __restrict__ F, int nf,
                                                           const uint32_t* __restrict__ soff,
                                                           const uint32_t* __restrict__ woff,
                                                           const uint32_t* __restrict__ roff,
                                                           uint32_t units)
{
    extern __shared__ uint64_t lds64[];
    int cur = -1;
    for (uint32_t t = blockIdx.x; t < units; t += gridDim.x) {
        const LongUnit u = long_unit(F, nf, t, 2);
        if (!u.ok) continue;
        const FieldDesc& fd = F[u.f];
        const auto* dy = kconst(fd.dyn);
        const uint32_t nb = fd.n_bins;
        uint64_t* code_s = lds64;
        uint32_t* wbuf = (uint32_t*)(lds64 + (W ? 0 : nb));
        if (!W && u.f != cur) {
            for (uint32_t s = threadIdx.x; s < nb; s += kWave) code_s[s] = write_entry(fd.code[s]);
            cur = u.f;
        }
        auto entry = [&](uint32_t sym) { return W ? write_entry(fd.code[sym]) : code_s[sym]; };
        if (u.c >= u.nch) continue;
        const Layout y = layout_of(fd, dy->codec, soff, woff, roff);
        if (y.total > fd.arc_cap) continue;
        const uint32_t wo = woff[fd.hch_base + u.c] - woff[fd.hch_base];
        EBC_G uint32_t* dst = (EBC_G uint32_t*)(fd.arc + y.off_words) + wo;
        EBC_G uint16_t* sbits = (EBC_G uint16_t*)(fd.arc + y.off_sbits);
        uint64_t done = 0;      // bits of the chunk already packed
        uint32_t carry = 0;     // the partial word at bit (done & ~31)
        uint32_t words_out = 0; // complete words stored
        for (uint32_t p = 0; p < fd.hc / kPassHc; ++p) {
            const uint64_t lo = (uint64_t)u.c * fd.hc + (uint64_t)p * kPassHc;
            if (lo >= u.cnt) break;
            uint32_t sym[kPassPerLane];
            load_pass(u, lo, sym);
            uint32_t mybits = 0;
#pragma unroll
            for (uint32_t k = 0; k < kPassPerLane; ++k)
                mybits += sym[k] == 0xFFFFFFFFu ? 0u : (uint32_t)entry(sym[k]) & 0xFFu;
            const uint32_t incl = wave_incl_scan_u32(mybits);
            const uint32_t pass_bits = (uint32_t)__shfl((int)incl, kWave - 1);
            // sub-chunk counts: 4 lanes of 64 symbols per 256-symbol sub-chunk
            constexpr uint32_t kLps = kSubMax / kPassPerLane;
            const uint32_t sb = (uint32_t)__shfl((int)incl, (int)min<uint32_t>(lane_id() + kLps - 1, 63)) -
                                (incl - mybits);
            const uint64_t sub = lo / fd.hs + lane_id() / kLps;
            const uint64_t l0 = lo + (uint64_t)lane_id() * kPassPerLane;
            if (lane_id() % kLps == 0 && l0 < u.cnt) sbits[sub] = (uint16_t)sb;
            // buffer word 0 holds the carried partial word
            const uint32_t head = (uint32_t)(done & 31);
            const uint32_t nbw = (head + pass_bits + 31) / 32;
            for (uint32_t i = lane_id(); i < nbw + 1; i += kWave) wbuf[i] = i == 0 ? carry : 0u;
            const uint32_t b0 = head + incl - mybits;
            uint32_t w = b0 >> 5, nacc = b0 & 31;
            uint64_t acc = 0;
#pragma unroll
            for (uint32_t k = 0; k < kPassPerLane; ++k) {
                if (sym[k] == 0xFFFFFFFFu) continue;
                const uint64_t v = entry(sym[k]);
                const uint32_t L = (uint32_t)v & 0xFFu;
                if (L <= 32) {
                    put_left(acc, nacc, w, wbuf, (uint32_t)(v >> 32), L);
                } else {
                    const uint64_t cw = fd.code[sym[k]] & ((1ull << 56) - 1);
                    put_bits(acc, nacc, w, wbuf, cw >> 32, L - 32);
                    put_bits(acc, nacc, w, wbuf, cw & 0xFFFFFFFFull, 32);
                }
            }
            if (nacc) atomicOr(&wbuf[w], (uint32_t)(acc >> 32));
            // complete words leave; the last partial one is carried
            const uint32_t full = (head + pass_bits) / 32;
            for (uint32_t i = lane_id(); i < full; i += kWave) dst[words_out + i] = wbuf[i];
            carry = wbuf[full];  // a wave's LDS accesses complete in order
            words_out += full;
            done += pass_bits;
        }
        if ((done & 31) && lane_id() == 0) dst[words_out] = carry;
    }
}

// ------------------------------------------------------------- decoding

__device__ __forceinline__ uint32_t word_at(const EBC_G uint32_t* __restrict__ w, uint32_t nw, uint32_t i)
{
    return i < nw ? w[i] : 0u;
}

// 64 stream bits starting at bit `pos` (zero beyond the lane's words)
__device__ __forceinline__ uint64_t window_at(const EBC_G uint32_t* __restrict__ w, uint32_t nw,
                                              uint32_t pos)
{
    const uint32_t k = pos >> 5, s = pos & 31;
    uint64_t a = ((uint64_t)word_at(w, nw, k) << 32) | word_at(w, nw, k + 1);
    if (s) a = (a << s) | (word_at(w, nw, k + 2) >> (32 - s));
    return a;
}

// The canonical search for the codeword at the head of a window, among the
// lengths from `from` on: its length is `from` plus the number of code-space
// ends the window lies at or above.  Returns the length (0 if the bits are not a
// codeword) and the symbol.
struct LongCode {
    uint32_t maxl;
    const uint64_t* s_endv;
    const uint64_t* s_first;
    const uint32_t* s_off;
    const uint16_t* perm;  // global: only codewords longer than both table levels get here
    __device__ __forceinline__ uint32_t decode(uint64_t w, uint32_t from, uint32_t& sym) const
    {
        uint32_t L = from;
        for (uint32_t l = from; l < maxl; ++l) L += w >= s_endv[l] ? 1u : 0u;
        // the window is at or above the first length-L code by construction;
        // it must also be below the end of the length-L codes
        const uint64_t d = (w >> (64 - L)) - s_first[L];
        if (d >= (uint64_t)(s_off[L + 1] - s_off[L])) return 0;
        sym = perm[s_off[L] + (uint32_t)d];
        // wait for the symbol here: where the paths merge, a wait would also
        // cover every stream load and output store in flight
        asm volatile("" ::"v"(sym));
        return L;
    }
};

// Output staging: each lane collects its decoded symbols in an LDS row and
// the wave moves them to HBM in blocks of kFlush symbols per lane.  A block
// leaves when every lane still decoding holds one; the copy is transposed
// (four consecutive threads write one lane's 64-byte block), so a store
// instruction writes sixteen whole 64-byte segments.  A lane too far ahead of
// its last flush skips groups of steps until the slower lanes have caught up,
// which never delays the wave: the waiting lane is ahead of the slowest one.
constexpr uint32_t kFlush = 32;
constexpr uint32_t kParts = kFlush / 8;    // 16-byte pieces of a flushed block
constexpr uint32_t kSteps = 4;             // table steps per group
constexpr uint32_t kRowWords = 29;         // row stride (odd: no bank conflicts across lanes)
constexpr uint32_t kGroupSyms = 1 + 3 * kSteps;  // symbols a group adds at most
// symbols up to which a lane goes on: a group's last step writes three slots
// from its start, at most kGroupSyms - 3 symbols after the group's
constexpr uint32_t kRowGo = 2 * kRowWords - (kGroupSyms - 3) - 3;
static_assert(kRowGo >= kFlush, "a waiting lane always holds a whole block");
constexpr uint32_t kTailWords = (kRowGo + kGroupSyms - kFlush + 1) / 2;  // kept past a block, at most
static_assert(kFlush / 2 + kTailWords <= kRowWords, "the kept words lie in the row");

// LDS of a decode workgroup: the tables, then a row per lane.  The first-level
// table sits at LDS address 0 (its index needs no base).
struct DecLds {
    uint64_t lut[1u << kLutBits];
    uint32_t l2s[kL2Size + 2];  // entry l2n: 0
    uint64_t first[65];
    uint64_t endv[65];
    uint32_t off[65];
    uint32_t next;     // work groups of this workgroup handed out
    uint32_t rows[1];  // lanes * kRowWords
};
uint32_t huff_decode_lds_bytes(uint32_t lanes) { return (uint32_t)offsetof(DecLds, rows) + lanes * kRowWords * 4; }

// LDS at a byte address (the workgroup's dynamic LDS starts at 0: the kernel
// has no static LDS), without an addition of a base.  The rows are written as
// halfwords and words and read as words: the types may alias.
typedef uint16_t __attribute__((may_alias)) u16_lds;
typedef uint32_t __attribute__((may_alias)) u32_lds;
typedef uint64_t __attribute__((may_alias)) u64_lds;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#if defined(__HIP_DEVICE_COMPILE__)
#define EBC_LDS(T, a) (*(__attribute__((address_space(3))) T*)(uint32_t)(a))
#else
#define EBC_LDS(T, a) (*(T*)(uintptr_t)(a))
#endif

// One lane per sub-chunk (hs = min(hc, 256) symbols, its bit count and its
// start from the archive's sub-chunk counts), blockDim.x lanes per workgroup,
// of which each wave's first per_wave ones work.
// The decoded stream is the field's quant-codes, or its run values (RLE+VLE).
//
// The loop runs groups of kSteps table steps.  A group starts with the 64-bit
// window at the lane's position, cut from the two 16-byte blocks of the stream
// that the lane holds in registers (a third is in flight).  A step shifts the
// window by the bits used so far, reads one table entry (up to three whole
// codewords), stores its three symbol slots at the row's end (only the decoded
// ones count) and adds the counts up: 13 vector instructions and three LDS
// ones.  The slots go as one aligned dword and the halfword before or after
// it: an LDS access across its alignment costs 64 cycles, a lane at a time,
// against 8 for these two together.  kSteps * kLutBits bits never exceed the window.  A codeword longer than the
// table makes its lane stand still to the end of the group (its entry counts
// nothing); the next group first decodes it through the second-level table or
// the canonical search.  A lane that passes its last symbol stops; the bits of
// the at most kGroupSyms - 1 symbols too many are taken back after the loop.
// Codewords longer than 32 bits leave for an exact path that reads windows
// straight from the stream.  Flushed blocks are stored non-temporally: they
// are not read before the kernel ends, and kept in the L2 they push out the
// stream's lines, each of which a lane comes back to eight times (22 us more on the
// 512^3 field).
//
// With the former step (bit buffer topped up from an LDS ring, exact clipping
// and both table levels in every step: about 60 vector instructions) a wave
// needed 900 cycles per step by itself and the kernel 257-290 us on a 512^3
// field at 3.8 bits per symbol, 82 us on 256x256; now 178-212 and 50 us.  What
// bounds it now is latency: a wave waits half of its time (table reads that
// depend on each other, stream blocks), and the LDS rows allow 16 waves per CU.
// Three, four or five steps per group make no difference on the large field.
__global__ __launch_bounds__(1024) void k_huff_decode(const FieldDesc* __restrict__ F, int nf,
                                                      const uint32_t* __restrict__ woff,
                                                      const uint32_t* __restrict__ soff,
                                                      const uint8_t* __restrict__ tabs, size_t tab_stride,
                                                      uint32_t per_wave)
{
    extern __shared__ uint64_t lds64[];
    DecLds& sm = *(DecLds*)lds64;
    const uint32_t lanes = blockDim.x;
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::hdwg_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    EBC_G FieldDyn* dy = fd.dyn;
    // EBC_LDS counts from the start of LDS: static LDS of this kernel, which there must
    // be none of, would come first
    if ((uint32_t)(uintptr_t)lds64 != 0) {
        if (threadIdx.x == 0) atomicMin(&dy->status, (int32_t)ST_ERR_UNSUPPORTED);
        return;
    }
    // One thread reads the status for all waves: workgroups of the field that find
    // the archive corrupt change it while this launch runs, and a wave that left by
    // itself would be missed at loading the tables.
    if (threadIdx.x == 0) sm.next = dy->status == ST_OK && huff_codec(dy->codec) ? 0u : 1u;
    __syncthreads();
    if (sm.next != 0) return;  // (the queue starts behind the next barrier)
    // the chunks' words must add up to the header's count
    const uint32_t tot = woff[fd.hch_base + fd.n_hch] - woff[fd.hch_base];
    if ((uint64_t)tot != fd.n_words_hdr) {
        if (threadIdx.x == 0) atomicMin(&dy->status, (int32_t)ST_ERR_ARCHIVE);
        return;
    }
    const DecTab* __restrict__ T = (const DecTab*)(tabs + (size_t)f * tab_stride);
    const uint32_t l2k = T->l2k, l2n = T->l2n;
    const uint32_t l2sub = (1u << (kLutBits + l2k)) - l2n;  // first long prefix << l2k
    {
        const uint4* src = (const uint4*)T->lut;
        uint4* dst = (uint4*)sm.lut;
#pragma unroll 8
        for (uint32_t i = threadIdx.x; i < (1u << kLutBits) / 2; i += lanes) dst[i] = src[i];
        for (uint32_t i = threadIdx.x; i <= l2n; i += lanes) sm.l2s[i] = i < l2n ? T->l2[i] : 0u;
        for (uint32_t i = threadIdx.x; i < 65; i += lanes) {
            sm.first[i] = T->first[i];
            sm.endv[i] = T->endv[i];
            sm.off[i] = T->offset[i];
        }
    }
    const uint32_t maxl = T->max_len;
    __syncthreads();
    // from here on LDS is also reached by byte address (EBC_LDS)
    asm volatile("" ::"v"((uint32_t)(uintptr_t)lds64) : "memory");
    const uint32_t lane = lane_id();
    const uint32_t hs = fd.hs, per = fd.hc / hs;
    const EBC_G uint8_t* arc = fd.arc;
    const EBC_G uint32_t* stream = (const EBC_G uint32_t*)(arc + fd.off_words);
    const LongCode lc{maxl, sm.endv, sm.first, sm.off, T->perm};
    // LDS byte addresses of the lane's row
    const uint32_t row = (uint32_t)offsetof(DecLds, rows) + threadIdx.x * (kRowWords * 4);
    const uint32_t lim_go = row + 2 * kRowGo, lim_flush = row + 2 * kFlush;
    // this lane's 16-byte piece of a flushed block: row lane / 4 of each
    // sixteen, part lane % 4
    const uint32_t fsrc = (uint32_t)offsetof(DecLds, rows) +
                          ((threadIdx.x - lane + lane / kParts) * kRowWords + (lane % kParts) * 4) * 4;
    auto row16b = [](uint32_t a) {
        return u32x4{EBC_LDS(const u32_lds, a), EBC_LDS(const u32_lds, a + 4), EBC_LDS(const u32_lds, a + 8),
                     EBC_LDS(const u32_lds, a + 12)};
    };
    // The field's groups of per_wave sub-chunks go to its workgroups in turn (so that
    // each has a mix of dense and sparse parts), and a workgroup's waves take
    // its groups as they finish: waves differ by a factor of three in steps.
    const uint32_t n_grp = (fd.n_sub + per_wave - 1) / per_wave;
    for (;;) {
        uint32_t gi = 0;
        if (lane == 0) gi = atomicAdd(&sm.next, 1u);
        gi = __builtin_amdgcn_readfirstlane(gi);
        const uint32_t g = gi * fd.hdwg_units + (t - fd.hdwg_base);
        if (gi >= n_grp || g >= n_grp) break;
        const uint32_t sub0 = g * per_wave;
        const uint32_t sub = sub0 + lane;
        bool live = lane < per_wave && sub < fd.n_sub;
        const uint32_t c = live ? sub / per : 0;
        const uint32_t nbits = live ? ((const EBC_G uint16_t*)(arc + fd.off_sbits))[sub] : 0u;
        // start bit of the sub-chunk inside the field's word stream
        const uint64_t b0 = live ? (uint64_t)(woff[fd.hch_base + c] - woff[fd.hch_base]) * 32 +
                                       soff[fd.sub_base + sub]
                                 : 0ull;
        const uint64_t lo = (uint64_t)sub * hs;
        const uint32_t skip = (uint32_t)(b0 & 31);
        const uint32_t nwl = live ? (skip + nbits + 31) / 32 : 0u;  // words the lane may read
        // The sum of the chunks' words was checked modulo 2^32 only; with stored
        // counts that wrap it, a sub-chunk may lie anywhere.
        if (live && (b0 >> 5) + nwl > fd.n_words_hdr) {
            atomicMin(&dy->status, (int32_t)ST_ERR_ARCHIVE);
            live = false;
        }
        const uint32_t want = live ? (uint32_t)min<uint64_t>(hs, fd.hn - lo) : 0u;
        const EBC_G uint32_t* __restrict__ words = stream + (live ? (uint32_t)(b0 >> 5) : 0u);

        // Stream position: pm = (bit position) - 1, counted from the first bit
        // of block A, so that the window from the next bit on is two funnel
        // shifts by ~pm.  The blocks are 16-byte aligned and start one word
        // before the lane's first (the archive's header and sections lie before
        // the words), which keeps pm from going below zero.  Blocks past the
        // lane's words are not read (the last one is read again instead; its
        // bits count for nothing).
        const uintptr_t wa = (uintptr_t)words - 4;
        const uint32_t ob = (uint32_t)((wa & 15u) >> 2);
        const EBC_G uint4* __restrict__ blk = (const EBC_G uint4*)(wa & ~(uintptr_t)15u);
        const uint32_t last = (ob + 1 + nwl + 3) / 4 - 1;
        uint4 A = make_uint4(0u, 0u, 0u, 0u), B = A, P = A;
        if (live) A = blk[0], B = blk[min(1u, last)], P = blk[min(2u, last)];
        uint32_t jb = 0;  // A is block jb
        uint32_t pm = 32 * (ob + 1) + skip - 1;

        uint32_t sp = row;              // the next symbol's place
        uint32_t endp = row + 2 * want; // where the last symbol ends (moves with the flushes)
        uint32_t over = 0;    // symbols decoded past the last one
        uint32_t nflush = 0;  // flushes the wave has made
        bool stuck = false;   // a codeword longer than the table is next
        bool slow = false;
        bool act = want > 0;
        EBC_G uint16_t* const fdst = fd.hsym + (uint64_t)(sub0 + lane / kParts) * hs + (lane % kParts) * 8;

        while (__any(act)) {
            if (pm >= 128) {
                A = B;
                B = P;
                pm -= 128;
                ++jb;
                P = blk[min(jb + 2, last)];
            }
            // words pm / 32 .. pm / 32 + 3 of A and B
            const bool k2 = (pm & 64u) != 0, k1 = (pm & 32u) != 0;
            const uint32_t u0 = k2 ? A.z : A.x, u1 = k2 ? A.w : A.y, u2 = k2 ? B.x : A.z, u3 = k2 ? B.y : A.w;
            const uint32_t x0 = k1 ? u1 : u0, x1 = k1 ? u2 : u1, x2 = k1 ? u3 : u2;
            uint32_t hi = __builtin_amdgcn_alignbit(x0, x1, ~pm), lw = __builtin_amdgcn_alignbit(x1, x2, ~pm);
            bool go = act && sp <= lim_go;
            if (go && stuck) {
                // the prefixes that start a codeword longer than the table are
                // the top ones and own consecutive blocks in prefix order, so
                // the second-level index follows from the bits (entry l2n,
                // which is 0, for any other)
                const uint32_t v = sm.l2s[min((hi >> (32 - kLutBits - l2k)) - l2sub, l2n)];
                uint32_t sym = v, L = v >> 16;
                if (L == 0) L = lc.decode(((uint64_t)hi << 32) | lw, kLutBits + 1, sym);
                EBC_LDS(u16_lds, sp) = (uint16_t)sym;
                sp += 2;
                // the window moves on by L bits (13 to 32)
                const uint32_t u4 = k2 ? B.z : B.x, x3 = k1 ? u4 : u3;
                const uint32_t l2w = __builtin_amdgcn_alignbit(x2, x3, ~pm);
                hi = __builtin_amdgcn_alignbit(hi, lw, 32 - L);
                lw = __builtin_amdgcn_alignbit(lw, l2w, 32 - L);
                pm += L;
                if (__builtin_expect(L == 0 || L > 32, 0)) {
                    sp -= 2;
                    pm -= L;
                    slow = true;
                    act = go = false;
                }
            }
            if (go) {
                const uint64_t buf = ((uint64_t)hi << 32) | lw;
                uint32_t acc = 0;  // low six bits: bits used in this group
                uint32_t n2 = 0;
#pragma unroll
                for (uint32_t u = 0; u < kSteps; ++u) {
                    const uint32_t wh = (uint32_t)((buf << (acc & 63u)) >> 32);
                    const uint64_t e =
                        EBC_LDS(const u64_lds, (wh >> (32 - kLutBits - 3)) & (((1u << kLutBits) - 1) << 3));
                    const uint32_t eh = (uint32_t)(e >> 32);
                    // odd places (sp % 4 == 2): the halfword s0 at sp, the dword
                    // s1 s2 after it; even ones: the dword s0 s1 at sp, then s2
                    const uint32_t odd = sp & 2u;
                    EBC_LDS(u32_lds, sp + odd) = __builtin_amdgcn_alignbit(eh, (uint32_t)e, sp << 3);
                    EBC_LDS(u16_lds, sp + 4 - 2 * odd) = (uint16_t)(odd ? (uint32_t)e : eh);
                    acc += eh >> 16;
                    n2 = (eh >> 22) & 7u;
                    sp += n2;
                }
                pm += acc & 63u;
                stuck = n2 == 0;
            }
            if (act && sp >= endp) {
                over = (sp - endp) / 2;
                sp = endp;
                act = false;
            }
            // a block of kFlush symbols leaves when every lane still decoding
            // has one
            if (__all(sp >= lim_flush || !act)) {
                // every lane holding a block has taken part in every flush so
                // far (a lane left out had stopped decoding with fewer than
                // kFlush symbols and never gains more), so its offset is
                // wave-uniform
                const uint64_t has = ballot(sp >= lim_flush);
                EBC_G uint16_t* dst = fdst + nflush * kFlush;
#pragma unroll
                for (uint32_t k = 0; k < kParts; ++k) {
                    if ((has >> (k * (kWave / kParts) + lane / kParts)) & 1u)
                        __builtin_nontemporal_store(row16b(fsrc + k * (kWave / kParts) * kRowWords * 4),
                                                    (EBC_G u32x4*)(dst + k * (kWave / kParts) * hs));
                }
                ++nflush;
                if (sp >= lim_flush) {
                    // the symbols past the block move to the front of the row
#pragma unroll
                    for (uint32_t w = 0; w < kTailWords; ++w)
                        EBC_LDS(u32_lds, row + 4 * w) = EBC_LDS(const u32_lds, row + 2 * kFlush + 4 * w);
                    sp -= 2 * kFlush;
                    endp -= 2 * kFlush;
                }
            }
        }
        // position after the lane's last symbol, counted from word w0
        uint32_t pos = 128 * jb + pm + 1 - 32 * (ob + 1);
        const EBC_G uint8_t* lens = arc + kHdr;  // code lengths, one byte per symbol
        for (uint32_t i = 0; i < over; ++i) pos -= lens[EBC_LDS(const u16_lds, sp + 2 * i)];
        // exact path, one codeword at a time from a window read straight from
        // the stream (lanes that met a codeword longer than 32 bits)
        uint32_t spi = (sp - row) / 2;
        uint32_t left = (endp - sp) / 2;  // symbols still to decode (0 unless slow)
        uint32_t flushed = want - left - spi;
        EBC_G uint16_t* __restrict__ out = fd.hsym + lo;
        bool bad = false;
        if (slow) {
            for (uint32_t k = 0; k < spi; ++k) out[flushed + k] = EBC_LDS(const u16_lds, row + 2 * k);
            flushed += spi;
            spi = 0;
            for (; left > 0; --left) {
                uint32_t sym = 0;
                const uint32_t L = lc.decode(window_at(words, nwl, pos), 1, sym);
                if (L == 0) {
                    bad = true;
                    break;
                }
                out[flushed++] = (uint16_t)sym;
                pos += L;
            }
        }
        if (live) {
            // what is left in the row: whole 16-byte groups, then single symbols
            uint32_t k = 0;
            for (; k + 8 <= spi; k += 8) *(EBC_G u32x4*)(out + flushed + k) = row16b(row + 2 * k);
            for (; k < spi; ++k) out[flushed + k] = EBC_LDS(const u16_lds, row + 2 * k);
        }
        // the sub-chunk must take exactly its stored bit count
        if (live && (bad || pos != skip + nbits)) atomicMin(&dy->status, ST_ERR_ARCHIVE);
    }
}

#define EBC_HC_DISPATCH(KERNEL, W, ...)                                                     \
    switch (hc) {                                                                           \
    case 64: hipLaunchKernelGGL((KERNEL<1, W>), __VA_ARGS__); break;                        \
    case 128: hipLaunchKernelGGL((KERNEL<2, W>), __VA_ARGS__); break;                       \
    case 256: hipLaunchKernelGGL((KERNEL<4, W>), __VA_ARGS__); break;                       \
    case 512: hipLaunchKernelGGL((KERNEL<8, W>), __VA_ARGS__); break;                       \
    case 1024: hipLaunchKernelGGL((KERNEL<16, W>), __VA_ARGS__); break;                     \
    case 2048: hipLaunchKernelGGL((KERNEL<32, W>), __VA_ARGS__); break;                     \
    case 4096: hipLaunchKernelGGL((KERNEL<64, W>), __VA_ARGS__); break;                     \
    default: return hipErrorInvalidValue;                                                   \
    }

// Compute units of an MI355X as one partition; on a part of it the grids and splits
// below are too large, which costs time only.
constexpr uint32_t kCus = 256;

// persistent grid: enough workgroups to fill the device several times over
static uint32_t persistent_grid(uint32_t units) { return units < kPersistentBlocks ? units : kPersistentBlocks; }

// Workgroups of kBlock threads (chunks of at most 1024 symbols) take the
// run-length tiles along; with longer chunks these get a launch of their own.
static bool takes_runs(uint32_t hc) { return kWave * huff_cpw(hc) == (uint32_t)kBlock; }

hipError_t launch_encode_count(const FieldDesc* F, int nf, uint32_t units, uint32_t hc, uint32_t n_bins,
                               uint32_t* wcnt, int which, uint32_t rt_units, uint32_t* rcnt, hipStream_t s)
{
    if (rt_units && (!takes_runs(hc) || !units)) {
        const hipError_t e = launch_rle_count(F, nf, rt_units, rcnt, s);
        if (e != hipSuccess) return e;
        rt_units = 0;
    }
    if (!units) return hipSuccess;
    const bool wide = n_bins > kMaxBins;
    const dim3 g(max(persistent_grid(units), min(rt_units, kEncBlocks)));
    if (hc > kPassHc) {
        if (wide) hipLaunchKernelGGL(k_huff_bits_long<true>, g, dim3(kWave), 0, s, F, nf, wcnt, units, which);
        else hipLaunchKernelGGL(k_huff_bits_long<false>, g, dim3(kWave), 0, s, F, nf, wcnt, units, which);
        return hipGetLastError();
    }
    const dim3 b(kWave * huff_cpw(hc));
    if (wide) {
        EBC_HC_DISPATCH(k_huff_bits, true, g, b, 0, s, F, nf, wcnt, units, which, rt_units, rcnt)
    } else {
        EBC_HC_DISPATCH(k_huff_bits, false, g, b, 0, s, F, nf, wcnt, units, which, rt_units, rcnt)
    }
    return hipGetLastError();
}

hipError_t launch_huff_write(const FieldDesc* F, int nf, uint32_t units, uint32_t hc, uint32_t n_bins,
                             const uint32_t* soff, const uint32_t* woff, const uint32_t* roff, hipStream_t s)
{
    if (!units) return hipSuccess;
    const bool wide = n_bins > kMaxBins;
    const size_t sh = huff_write_lds_bytes(n_bins, hc);
    // The short-chunk kernels' registers allow five workgroups per CU: with up to
    // five workgroups' tables and buffers in a CU's LDS the grid is as many (512^3:
    // 80 us, with four 88, with eight and thus a second, partial round 86).
    const bool five = hc <= 1024 && 5 * sh <= 160u * 1024;
    const dim3 g(min(units, five ? 5 * kCus : kPersistentBlocks));
    if (hc > kPassHc) {
        if (wide) hipLaunchKernelGGL(k_huff_write_long<true>, g, dim3(kWave), sh, s, F, nf, soff, woff, roff, units);
        else hipLaunchKernelGGL(k_huff_write_long<false>, g, dim3(kWave), sh, s, F, nf, soff, woff, roff, units);
        return hipGetLastError();
    }
    const dim3 b(kWave * huff_cpw(hc));
    if (wide) {
        EBC_HC_DISPATCH(k_huff_write, true, g, b, sh, s, F, nf, soff, woff, roff, units)
    } else {
        EBC_HC_DISPATCH(k_huff_write, false, g, b, sh, s, F, nf, soff, woff, roff, units)
    }
    return hipGetLastError();
}

// Decode workgroups of a call whose streams make n_sub sub-chunks: sub-chunks per
// wave, lanes per workgroup, and waves' worth of work that a workgroup takes.  The
// tables take 42 KB of LDS per workgroup and a lane 116 bytes, so a CU holds one
// workgroup of 1024 lanes (16 waves) or two of 256.  Above 4096 waves' worth of work
// (64 sub-chunks each) a workgroup of 1024 lanes takes a 256th of the sum, so that the
// tables are loaded once per CU and the waves even out; between 2048 and 4096, 16, and
// some CUs stay idle.  Every field of a batch rounds up to whole workgroups of its own,
// so there may be more of them than CUs.  A call of up to two workgroups of 256 lanes
// per CU is split over all of them, up to 65536 sub-chunks with half of each wave's
// lanes idle: four waves load the tables, and a wave waits for the slowest of 32 lanes
// only (one wave of 64 per workgroup: 256x256 55 us, here 50; 1800x3600 44 and 40;
// 1501x2999 with 16384 bins 87 and 81).  16 sub-chunks per wave gain nothing more on
// those, 8 lose once the workgroups do not fit at once (1800x3600: 58 us).
void huff_decode_split(uint64_t n_sub, uint32_t* per_wave, uint32_t* lanes, uint32_t* groups)
{
    *per_wave = n_sub <= 32 * 4 * 2 * kCus ? 32 : 64;
    const uint64_t n_grp = (n_sub + *per_wave - 1) / *per_wave;
    if (n_grp <= 2 * kCus * 4) *lanes = 256, *groups = 4;
    else *lanes = 1024, *groups = n_grp <= kCus * 16 ? 16 : (uint32_t)((n_grp + kCus - 1) / kCus);
}

hipError_t launch_huff_decode(const FieldDesc* F, int nf, uint32_t units, uint32_t per_wave, uint32_t lanes,
                              const uint32_t* woff, const uint32_t* soff, const uint8_t* tabs,
                              size_t tab_stride, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_huff_decode, dim3(units), dim3(lanes), huff_decode_lds_bytes(lanes), s, F, nf, woff,
                       soff, tabs, tab_stride, per_wave);
    return hipGetLastError();
}

}  // namespace ebc
