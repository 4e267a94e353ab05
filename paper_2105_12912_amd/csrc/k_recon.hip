// k_recon.hip -- Lorenzo reconstruction as an N-D partial sum, with the
// outlier fuse and dequantisation folded in.
//
// Sec. IV-B.2: with q' = q - r (outliers substituted, Sec. IV-B.1), the
// reconstructed integers are the inclusive N-D prefix sum of q' within each
// chunk, and the N-D sum splits into one-axis passes (x, then y, then z;
// Algorithm 1, decompression half).  Output = d * (2 eb) rounded once to fp32.
//
// Mapping: a lane owns four consecutive x.  The x pass is a within-lane prefix
// plus the totals of the quads to its left in the chunk row (DPP row shifts in
// 2D and 3D, a full-wave scan for the 256-long 1D chunk); the y pass is a running
// sum in registers as the wave walks the chunk's rows, the z pass a scan over groups
// of lanes.  Integer sums wrap modulo 2^32 exactly as the CPU recurrence truncated to
// int32 does.
#include "ebc_dev.h"
#include "ebc_launch.h"
#include "rle_dev.h"

namespace ebc {

// Four codes kept packed (two per 32-bit word) so that a whole tile's loads
// fit in few registers; codes of absent elements read as 1 (never the
// outlier placeholder).
__device__ __forceinline__ u32x2 load_packed(const EBC_G uint16_t* __restrict__ q, uint64_t i, int nvalid)
{
    if (nvalid == 4 && (i & 1) == 0) return *(const EBC_G u32x2_a4*)(q + i);  // dword-aligned
    uint32_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = k < nvalid ? q[i + k] : 1u;
    u32x2 t;
    t.x = c[0] | (c[1] << 16);
    t.y = c[2] | (c[3] << 16);
    return t;
}

__device__ __forceinline__ void unpack4(u32x2 t, uint32_t c[4])
{
    c[0] = t.x & 0xFFFF, c[1] = t.x >> 16, c[2] = t.y & 0xFFFF, c[3] = t.y >> 16;
}

template <bool VEC>
__device__ __forceinline__ void store_quad(EBC_G float* __restrict__ o, uint64_t i, int nvalid,
                                           const float v[4])
{
    if (VEC && nvalid == 4) {
        st_nt_f4(o + i, f32x4{v[0], v[1], v[2], v[3]});
    } else if (nvalid == 4) {
        *(EBC_G f32x4_a4*)(o + i) = f32x4{v[0], v[1], v[2], v[3]};  // dword-aligned
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nvalid) o[i + k] = v[k];
    }
}

// q' for a quad: code - r, or the exact outlier delta where the code is 0
__device__ __forceinline__ void fuse4(const uint32_t c[4], int nvalid, int32_t r,
                                      const EBC_G int32_t* __restrict__ dsc, uint64_t i, uint32_t qp[4],
                                      uint32_t& zeros)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (c[k] == 0 && k < nvalid) {
            qp[k] = (uint32_t)dsc[i + k];
            // consume the loaded value inside the (rare) branch, so that the
            // wait for it stays here and the common path never waits on the
            // loads and stores in flight
            asm volatile("" ::"v"(qp[k]));
            ++zeros;
        } else {
            qp[k] = c[k] - (uint32_t)r;
        }
    }
}

__device__ __forceinline__ void dequant4(const uint32_t s[4], double ebx2, float v[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (float)((double)(int32_t)s[k] * ebx2);
}

// fp64 archives: the product rounded once, in binary64
__device__ __forceinline__ void dequant4(const uint32_t s[4], double ebx2, double v[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (double)(int32_t)s[k] * ebx2;
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef f64x2 f64x2_a8 __attribute__((aligned(8)));

// an fp64 quad: two 16-byte stores (non-temporal on 16-byte aligned rows)
template <bool VEC>
__device__ __forceinline__ void store_quad(EBC_G double* __restrict__ o, uint64_t i, int nvalid,
                                           const double v[4])
{
    if (nvalid == 4) {
        if (VEC) {
            __builtin_nontemporal_store(f64x2{v[0], v[1]}, (EBC_G f64x2*)(o + i));
            __builtin_nontemporal_store(f64x2{v[2], v[3]}, (EBC_G f64x2*)(o + i + 2));
        } else {
            *(EBC_G f64x2_a8*)(o + i) = f64x2{v[0], v[1]};
            *(EBC_G f64x2_a8*)(o + i + 2) = f64x2{v[2], v[3]};
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nvalid) o[i + k] = v[k];
    }
}

// output element type of a field: fp32, or fp64 for fp64 archives
template <class OT> __device__ __forceinline__ EBC_G OT* field_out(const FieldDesc& fd);
template <> __device__ __forceinline__ EBC_G float* field_out<float>(const FieldDesc& fd) { return fd.outf; }
template <> __device__ __forceinline__ EBC_G double* field_out<double>(const FieldDesc& fd) { return fd.outd; }

// 1D: this lane's quads of one workgroup tile, one in each of the wave's four
// 256-long chunks.
struct RTile {
    static constexpr int NQ = 4;
    u32x2 raw[NQ];
};

// lane geometry of a tile: first element of quad k and its valid count
__device__ __forceinline__ void rquad(const FieldDesc& fd, uint32_t tl, int k, uint64_t& i0, int& nv)
{
    const int l = lane_id();
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t wt = tl * kWavesPerBlock + w;
    i0 = (uint64_t)wt * 1024 + k * 256 + 4 * l;
    nv = (wt >= fd.n_wave_tiles || i0 >= fd.n) ? 0 : (int)min<uint64_t>(4, fd.n - i0);
    if (nv == 0) i0 = 0;
}

// With 16-byte rows (VEC) every quad is loaded with one unconditional vector
// load (an absent quad reads the start of the code array; the tail quad of a
// 1D field may read up to 6 bytes past the codes, into the outlier scratch
// that follows them), so the number of memory operations per tile is fixed
// and the compiler never has to wait for stores before a load's use.
template <bool VEC>
__device__ __forceinline__ void rtile_load(const FieldDesc& fd, uint32_t tl, RTile& T)
{
#pragma unroll
    for (int k = 0; k < RTile::NQ; ++k) {
        uint64_t i0;
        int nv;
        rquad(fd, tl, k, i0, nv);
        if (VEC) T.raw[k] = ld_nt_u2(fd.q + (nv > 0 ? i0 : 0));
        else T.raw[k] = load_packed(fd.q, i0, nv);
    }
}

template <bool VEC, class OT>
__device__ __forceinline__ void rtile_process(const FieldDesc& fd, uint32_t tl, const RTile& T,
                                              double ebx2, uint32_t& zeros)
{
    const int32_t r = (int32_t)(fd.n_bins / 2);
    const EBC_G int32_t* __restrict__ dsc = fd.dsc;
    EBC_G OT* __restrict__ out = field_out<OT>(fd);
#pragma unroll
    for (int k = 0; k < RTile::NQ; ++k) {
        uint64_t i0;
        int nv;
        rquad(fd, tl, k, i0, nv);
        uint32_t c[4], s[4];
        unpack4(T.raw[k], c);
        if (VEC) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j >= nv) c[j] = 1u;  // absent: never the outlier placeholder
        }
        fuse4(c, nv, r, dsc, i0, s, zeros);
        s[1] += s[0], s[2] += s[1], s[3] += s[2];  // x pass within the quad
        // exclusive prefix of the lane totals over the 256-long chunk
        const uint32_t excl = wave_incl_scan_u32(s[3]) - s[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += excl;
        OT v[4];
        dequant4(s, ebx2, v);
        if constexpr (VEC && sizeof(OT) == 4) {
            // one unconditional vector store (absent quads go to the sink);
            // a partial quad (1D tail only) is then written element-wise
            st_nt_f4(nv == 4 ? out + i0 : fd.sink, f32x4{v[0], v[1], v[2], v[3]});
            if (nv > 0 && nv < 4) {
                for (int j = 0; j < nv; ++j) out[i0 + j] = v[j];
            }
        } else {
            store_quad<VEC>(out, i0, nv, v);
        }
    }
}

// Zero codes seen by this workgroup for field fd, added to one of the field's
// counters (their sum is checked against the outlier count by k_recon_check).
__device__ __forceinline__ void flush_zeros(const FieldDesc& fd, uint32_t zeros, uint32_t* s_z)
{
    const uint32_t zs = wave_sum_u32(zeros);
    if (lane_id() == 0) s_z[threadIdx.x / kWave] = zs;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t z = s_z[0] + s_z[1] + s_z[2] + s_z[3];
        if (z) atomicAdd(&fd.zslot[(blockIdx.x % kZeroSlots) * kZeroStride], z);
    }
}

// 1D: one workgroup per tile, which measured faster than a resident-size grid that
// strides over the tiles with the next one's codes in flight.
template <bool VEC, class OT>
__global__ __launch_bounds__(kBlock) void k_reconstruct(const FieldDesc* __restrict__ F, int nf)
{
    __shared__ uint32_t s_z[kWavesPerBlock];
    const uint32_t t = blockIdx.x;
    const FieldDesc& fd = F[find_field<&FieldDesc::wg_base>(F, nf, t)];
    const uint32_t tl = t - fd.wg_base;
    RTile T;
    rtile_load<VEC>(fd, tl, T);  // on the way while the field's scalars are read
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || dy->codec == ARC_CONST) return;
    uint32_t zeros = 0;
    rtile_process<VEC, OT>(fd, tl, T, dy->ebx2, zeros);
    flush_zeros(fd, zeros, s_z);
}

// A tile inside one run, of code v (not the outlier placeholder): its chunks are
// alike, s = (x + 1) (v - r).
template <class OT>
__device__ __forceinline__ void constant_tile(const FieldDesc& fd, uint32_t tl, uint32_t v, double ebx2)
{
    EBC_G OT* __restrict__ out = field_out<OT>(fd);
    uint32_t s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = (4 * lane_id() + j + 1) * (v - fd.n_bins / 2);
    OT o[4];
    dequant4(s, ebx2, o);
    const bool vec = ((uintptr_t)out & 15u) == 0;
#pragma unroll
    for (int k = 0; k < RTile::NQ; ++k) {
        uint64_t i0;
        int nv;
        rquad(fd, tl, k, i0, nv);
        if (vec) store_quad<true>(out, i0, nv, o);
        else store_quad<false>(out, i0, nv, o);
    }
}

// 1D run-length coded fields: a workgroup expands one tile of runs and
// reconstructs it, so the codes (2 bytes per element, written and read back) never
// leave the CU.  A thread expands 16 consecutive codes and a lane reconstructs
// quads, so the codes of a wave's 1024 elements change hands through LDS.  Tiles
// inside one run, most of a field that is worth run-length coding, need neither.
// Bound by the stores: 86 us for a mostly constant field of 120M elements (a plain
// fill of that size takes 73), where expansion and reconstruction took 68 + 105.
union RleLds {
    RleStage run;
    uint4 code[kRleTile / 8];
};
template <class OT>
__device__ __forceinline__ void rle_tile(const FieldDesc& fd, uint32_t t, uint32_t rlo, uint32_t nr,
                                         const uint32_t* __restrict__ starts, double ebx2, RleLds& sm,
                                         uint32_t* s_z)
{
    const uint32_t tl = t - fd.rt_base;
    if (nr == 1 && rlo != 0) {
        constant_tile<OT>(fd, tl, rlo, ebx2);
        return;
    }
    RTile T;
    if (nr == 1) {
#pragma unroll
        for (int k = 0; k < RTile::NQ; ++k) T.raw[k] = u32x2{0u, 0u};
    } else {
        uint16_t c[kRleItems];
        expand_tile(fd, t, rlo, nr, starts, sm.run, c);
        __syncthreads();
        uint4* s_code = sm.code;
        s_code[2 * threadIdx.x] = pack8(c);
        s_code[2 * threadIdx.x + 1] = pack8(c + 8);
        __syncthreads();
        const uint32_t w = threadIdx.x / kWave;
#pragma unroll
        for (int k = 0; k < RTile::NQ; ++k)
            T.raw[k] = ((const u32x2*)s_code)[(w * RTile::NQ + k) * kWave + lane_id()];
    }
    uint32_t zeros = 0;
    if (((uintptr_t)field_out<OT>(fd) & 15u) == 0) rtile_process<true, OT>(fd, tl, T, ebx2, zeros);
    else rtile_process<false, OT>(fd, tl, T, ebx2, zeros);
    flush_zeros(fd, zeros, s_z);
}

__global__ __launch_bounds__(kBlock) void k_rle_reconstruct(const FieldDesc* __restrict__ F, int nf,
                                                            const uint32_t* __restrict__ starts,
                                                            const uint32_t* __restrict__ tmap)
{
    __shared__ RleLds sm;
    __shared__ uint32_t s_z[kWavesPerBlock];
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::rt_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || !rle_codec(fd.codec_hdr) || fd.rank != 1) return;
    const uint32_t rlo = tmap[2 * t], nr = tmap[2 * t + 1];  // (the value itself where nr is 1)
    if (fd.dtype == 1) rle_tile<double>(fd, t, rlo, nr, starts, dy->ebx2, sm, s_z);
    else rle_tile<float>(fd, t, rlo, nr, starts, dy->ebx2, sm, s_z);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// running minimum of the two codes packed in each word (a zero half stays)
__device__ __forceinline__ uint32_t min_halves(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                  __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ bool has_zero_half(uint32_t w) { return (w & 0xFFFFu) == 0 || (w >> 16) == 0; }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

// 2D: a wave owns a tile of xs = 64 wx elements along x by 16 * 4 / wx rows; a
// lane is a quad along x and walks the 16 rows of its chunk row, so a row of the
// tile is one contiguous load and store, the y pass a running sum in registers
// and the x pass a prefix over the four lanes of a 16-wide chunk.  All rows are
// loaded at once (the kernel is bound by that round trip on fields of a few
// million values, by traffic on larger ones).  Deltas are loaded for eight rows at
// a time, only if some lane holds an outlier there.  With the 16 rows across the
// lanes of a DPP row a load touched 16 rows by 32 bytes, and every outlier waited
// for its own delta: 32 us on 1800x3600, against the 8 us that its bytes take.
template <bool VEC, class OT>
__global__ __launch_bounds__(kWave) void k_reconstruct2(const FieldDesc* __restrict__ F, int nf)
{
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::wg_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || dy->codec == ARC_CONST) return;
    const uint32_t tl = t - fd.wg_base, nxb = fd.nxb;
    const uint32_t l = lane_id(), lx = fd.xs / 4;  // lanes along x: 16, 32 or 64
    const uint32_t nx = fd.nx, ny = fd.ny;
    const uint32_t x0 = (tl % nxb) * fd.xs + 4 * (l & (lx - 1));
    const uint32_t y0 = (tl / nxb * (kWave / lx) + l / lx) * 16;
    const uint32_t nv = x0 < nx && y0 < ny ? min<uint32_t>(4, nx - x0) : 0u;
    const uint32_t rows = nv ? min<uint32_t>(16, ny - y0) : 0u;
    const uint64_t i0 = nv ? (uint64_t)y0 * nx + x0 : 0;
    const EBC_G uint16_t* __restrict__ q = fd.q + i0;
    const EBC_G int32_t* __restrict__ dsc = fd.dsc + i0;
    EBC_G OT* __restrict__ out = field_out<OT>(fd) + i0;
    const uint32_t r = fd.n_bins / 2;
    const double ebx2 = dy->ebx2;
    u32x2 raw[16];
#pragma unroll
    for (uint32_t y = 0; y < 16; ++y) {
        raw[y] = u32x2{0x00010001u, 0x00010001u};  // absent codes read as 1
        if (y < rows) {
            if (nv == 4) {
                if (VEC) raw[y] = ld_nt_u2(q + (uint64_t)y * nx);
                else raw[y] = *(const EBC_G u32x2_a2*)(q + (uint64_t)y * nx);
            } else {
                uint32_t c[3] = {1u, 1u, 1u};
#pragma unroll
                for (uint32_t k = 0; k < 3; ++k)
                    if (k < nv) c[k] = q[(uint64_t)y * nx + k];
                raw[y] = u32x2{c[0] | (c[1] << 16), c[2] | 0x00010000u};
            }
        }
    }
    const uint32_t m1 = (l & 3) >= 1 ? ~0u : 0u, m2 = (l & 3) >= 2 ? ~0u : 0u;
    uint32_t yprev[4] = {0, 0, 0, 0};
    uint32_t zeros = 0;
#pragma unroll
    for (uint32_t h = 0; h < 16; h += 8) {
        uint32_t low = 0xFFFFFFFFu;
#pragma unroll
        for (uint32_t y = h; y < h + 8; ++y) low = min_halves(low, min_halves(raw[y].x, raw[y].y));
        const bool any = __any(has_zero_half(low));
        u32x4 d[8];
        if (any) {
#pragma unroll
            for (uint32_t y = h; y < h + 8; ++y) {
                d[y - h] = u32x4{0u, 0u, 0u, 0u};
                // (the workspace goes on past the field's last delta)
                if (has_zero_half(min_halves(raw[y].x, raw[y].y)))
                    d[y - h] = *(const EBC_G u32x4_a4*)(dsc + (uint64_t)y * nx);
            }
        }
#pragma unroll
        for (uint32_t y = h; y < h + 8; ++y) {
            uint32_t c[4], s[4];
            unpack4(raw[y], c);
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] = c[k] - r;
            if (any) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    s[k] = c[k] == 0 ? d[y - h][k] : s[k];
                    zeros += c[k] == 0;
                }
            }
            s[1] += s[0], s[2] += s[1], s[3] += s[2];  // x pass within the quad
            uint32_t inc = s[3];
            inc += dpp_shr_u<1>(inc) & m1;
            inc += dpp_shr_u<2>(inc) & m2;
            const uint32_t left = inc - s[3];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[k] += left + yprev[k];  // y pass
                yprev[k] = s[k];
            }
            OT v[4];
            dequant4(s, ebx2, v);
            if (y < rows) store_quad<VEC>(out, (uint64_t)y * nx, (int)nv, v);
        }
    }
    const uint32_t zs = wave_sum_u32(zeros);
    if (l == 0 && zs) atomicAdd(&fd.zslot[(t % kZeroSlots) * kZeroStride], zs);
}

// fp32 quads are stored non-temporally (512^3: 143 us against 144, a batch of 16
// fields 55 against 56), fp64 ones, two stores each, are not (100x500x500: 96 against
// 87)
__device__ __forceinline__ void store_quad3(EBC_G float* __restrict__ o, const float v[4])
{
    __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, (EBC_G f32x4_a4*)o);
}
__device__ __forceinline__ void store_quad3(EBC_G double* __restrict__ o, const double v[4])
{
    store_quad<false>(o, 0, 4, v);
}

// The chunks of a wave's blocks from their codes and deltas (see k_reconstruct3).
// full: both planes of the lane's quad lie in the field, single: the first does; nvz:
// the quad's elements inside the field, by plane.  Returns the lane's outlier count.
template <class OT, uint32_t GP>
__device__ __forceinline__ uint32_t block_sums(const FieldDesc& fd, const u32x2 (&c)[2][8],
                                                    const u32x4 (&d)[2][8], uint32_t y0, uint64_t i0, bool full,
                                                    bool single, const int (&nvz)[2], double ebx2)
{
    const uint32_t nx = fd.nx, ny = fd.ny, r = fd.n_bins / 2, g = (lane_id() >> 4) % GP;
    const uint64_t plane = (uint64_t)ny * nx;
    EBC_G OT* __restrict__ out = field_out<OT>(fd);
    uint32_t yprev[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    uint32_t zeros = 0;
    const uint32_t odd = lane_id() & 1 ? ~0u : 0u, g1 = g & 1 ? ~0u : 0u, g2 = g & 2 ? ~0u : 0u;
#pragma unroll
    for (uint32_t y = 0; y < 8; ++y) {
        if (y0 + y >= ny) continue;  // uniform
        uint32_t s[2][4];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t cv[4];
            unpack4(c[p][y], cv);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                zeros += cv[k] == 0;
                s[p][k] = cv[k] == 0 ? d[p][y][k] : cv[k] - r;
            }
            s[p][1] += s[p][0], s[p][2] += s[p][1], s[p][3] += s[p][2];  // x pass within the quad
            const uint32_t left = dpp_shr_u<1>(s[p][3]) & odd;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[p][k] += left + yprev[p][k];  // y pass
                yprev[p][k] = s[p][k];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s[1][k] += s[0][k];
            // z pass: the totals of the block's lanes with a lower g
            if constexpr (GP > 1) {
                const auto t = __builtin_amdgcn_permlane16_swap(s[1][k], s[1][k], false, false);
                uint32_t below = t[0] & g1;
                if constexpr (GP > 2) {
                    const uint32_t both = t[0] + t[1];
                    below += __builtin_amdgcn_permlane32_swap(both, both, false, false)[0] & g2;
                }
                s[0][k] += below, s[1][k] += below;
            }
        }
        const uint64_t i = i0 + (uint64_t)y * nx;
        OT v[2][4];
        dequant4(s[0], ebx2, v[0]);
        dequant4(s[1], ebx2, v[1]);
        if (full) {
            store_quad3(out + i, v[0]);
            store_quad3(out + i + plane, v[1]);
        } else if (single) {
            store_quad3(out + i, v[0]);
        } else if (nvz[0] > 0) {
            store_quad<false>(out, i, nvz[0], v[0]);
            store_quad<false>(out, i + plane, nvz[1], v[1]);
        }
    }
    return zeros;
}

// 3D: a wave owns a block of 64 x 8 x 8, eight chunks along x.  Lane (g, xq) =
// (l / 16, l % 16) holds a quad along x of the planes 2g and 2g + 1 and walks y, so a
// row of the block is one access of 16 lanes: the x pass is in-lane plus the total of
// the pair lane, the y pass a running sum, the z pass a sum of the lane's two planes
// and a scan over the four g.  All codes are loaded at once, behind one branch (with
// one per row the loads were spread out and everything a third slower), then, if some
// lane holds an outlier, the deltas (for quads without one the field's first delta, so
// that no access depends on the lane).  Bound by the traffic, and by the two round
// trips on fields of a few million values.
//
// A wave per 256 x 8 x 8 that kept running sums over all planes, with the chunks that
// hold outliers left to a second kernel, took 158 + 18 us on 512^3, 40 + 90 on a rough
// fp64 field of 100x500x500 and 83 + 43 on the 3D fields of a batch; this one takes
// 143, 87 and 55.
//
// GP: 16-lane groups per block.  A last layer of one or two planes has work for one
// group of a block, of three or four for two: the wave then takes the four or two
// next blocks along x (recon3_groups).  With one block per wave in every layer such
// fields took 79 us (1x4096x4096), 85 (2), 112 (3) and 227 (9 planes), longer than a
// wave per 256 x 8 had (35, 44, 58, 181); so they take 25, 42, 65 and 182.
template <class OT, uint32_t GP>
__device__ __forceinline__ uint32_t recon3_wave(const FieldDesc& fd, uint32_t xb, uint32_t yb, uint32_t zb,
                                             double ebx2)
{
    const uint32_t nx = fd.nx, ny = fd.ny, nz = fd.nz;
    const uint32_t l4 = lane_id() >> 4, zz = zb * 8 + 2 * (l4 % GP), y0 = yb * 8;
    const uint32_t x0 = (xb * (4 / GP) + l4 / GP) * 64 + (lane_id() & 15) * 4;
    const int nv = x0 < nx ? (int)min<uint32_t>(4, nx - x0) : 0;
    const EBC_G uint16_t* __restrict__ q = fd.q;
    const EBC_G int32_t* __restrict__ dsc = fd.dsc;
    const uint64_t i0 = ((uint64_t)zz * ny + y0) * nx + x0, plane = (uint64_t)ny * nx;
    const bool full = nv == 4 && zz + 1 < nz, single = nv == 4 && zz + 1 == nz;
    const int nvz[2] = {zz < nz ? nv : 0, zz + 1 < nz ? nv : 0};
    u32x2 c[2][8];
    u32x4 d[2][8];
#pragma unroll
    for (uint32_t y = 0; y < 8; ++y) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            c[p][y] = u32x2{0x00010001u, 0x00010001u};
            d[p][y] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    if (full) {
#pragma unroll
        for (uint32_t y = 0; y < 8; ++y) {
            if (y0 + y >= ny) break;  // uniform
#pragma unroll
            for (int p = 0; p < 2; ++p) c[p][y] = *(const EBC_G u32x2_a2*)(q + i0 + p * plane + (uint64_t)y * nx);
        }
    } else if (single) {
        // the field's last plane
#pragma unroll
        for (uint32_t y = 0; y < 8; ++y) {
            if (y0 + y >= ny) break;
            c[0][y] = *(const EBC_G u32x2_a2*)(q + i0 + (uint64_t)y * nx);
        }
    } else if (nvz[0] > 0) {
        // the field's last, partial quad along x
#pragma unroll
        for (uint32_t y = 0; y < 8; ++y) {
            if (y0 + y >= ny) break;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint64_t i = i0 + p * plane + (uint64_t)y * nx;
                uint32_t e[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) e[k] = k < nvz[p] ? q[i + k] : 1u;
                c[p][y] = u32x2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
            }
        }
    }
    uint32_t low = 0xFFFFFFFFu;  // smallest code halves met
#pragma unroll
    for (uint32_t y = 0; y < 8; ++y)
#pragma unroll
        for (int p = 0; p < 2; ++p) low = min_halves(low, min_halves(c[p][y].x, c[p][y].y));
    const bool met = has_zero_half(low);
    if (__any(met)) {
        if (full || single) {  // (an absent plane holds no outlier code)
#pragma unroll
            for (uint32_t y = 0; y < 8; ++y) {
                if (y0 + y >= ny) break;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const bool z = has_zero_half(min_halves(c[p][y].x, c[p][y].y));
                    d[p][y] = *(const EBC_G u32x4_a4*)(dsc + (z ? i0 + p * plane + (uint64_t)y * nx : 0));
                }
            }
        } else if (met) {
#pragma unroll
            for (uint32_t y = 0; y < 8; ++y) {
                if (y0 + y >= ny) break;
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        d[p][y][k] = k < nvz[p] ? (uint32_t)dsc[i0 + p * plane + (uint64_t)y * nx + k] : 0u;
            }
        }
    }
    return block_sums<OT, GP>(fd, c, d, y0, i0, full, single, nvz, ebx2);
}

// wave b of a field: its blocks in the order x, y, z, a last layer of few planes with
// several blocks per wave
template <class OT>
__device__ __forceinline__ uint32_t recon3_blocks(const FieldDesc& fd, uint32_t b, double ebx2)
{
    const uint32_t nxb = fd.nxb, nyb = fd.nyb, layer = nxb * nyb;
    const uint32_t zb = min(b / layer, fd.nzb - 1), gp = recon3_groups(fd.nz - zb * 8);
    b -= zb * layer;
    const uint32_t w = (nxb + 4 / gp - 1) / (4 / gp);  // waves along x
    const uint32_t xb = b % w, yb = b / w;
    if (yb >= nyb) return 0;
    if (gp == 4) return recon3_wave<OT, 4>(fd, xb, yb, zb, ebx2);
    if (gp == 2) return recon3_wave<OT, 2>(fd, xb, yb, zb, ebx2);
    return recon3_wave<OT, 1>(fd, xb, yb, zb, ebx2);
}

__global__ __launch_bounds__(kBlock) void k_reconstruct3(const FieldDesc* __restrict__ F, int nf)
{
    const uint32_t t = blockIdx.x;
    const int f = find_field<&FieldDesc::r3_base>(F, nf, t);
    const FieldDesc& fd = F[f];
    const auto* dy = kconst(fd.dyn);
    if (dy->status != ST_OK || dy->codec == ARC_CONST) return;
    const uint32_t b = (t - fd.r3_base) * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t zeros =
        fd.dtype == 1 ? recon3_blocks<double>(fd, b, dy->ebx2) : recon3_blocks<float>(fd, b, dy->ebx2);
    const uint32_t zs = wave_sum_u32(zeros);
    if (lane_id() == 0 && zs) atomicAdd(&fd.zslot[(b % kZeroSlots) * kZeroStride], zs);
}

// decompression epilogue, one wave per field: the code-0 count must equal the
// outlier count; the field's status into the caller's slot (st may be NULL)
static_assert(kZeroSlots == kWave, "one lane per counter");
__global__ __launch_bounds__(kWave) void k_recon_check(const FieldDesc* __restrict__ F, int32_t* __restrict__ st)
{
    const FieldDesc& fd = F[blockIdx.x];
    EBC_G FieldDyn* dy = fd.dyn;
    int32_t status = dy->status;
    if (status == ST_OK && fd.codec_hdr != ARC_CONST) {
        const uint64_t z = wave_sum_u64(fd.zslot[lane_id() * kZeroStride]);
        if (z != fd.n_out_hdr) status = ST_ERR_ARCHIVE;
    }
    if (lane_id() != 0) return;
    dy->status = status;
    if (st) st[fd.slot] = status;
}

// constant field (range zero): every element is the stored value
__global__ __launch_bounds__(kBlock) void k_fill_const(const FieldDesc* __restrict__ F, int nf)
{
    const uint32_t u = blockIdx.x;
    const int f = find_field<&FieldDesc::range_base>(F, nf, u);
    const FieldDesc& fd = F[f];
    if (fd.codec_hdr != ARC_CONST || fd.dyn->status != ST_OK) return;
    const uint64_t lo = (uint64_t)(u - fd.range_base) * kRangeUnit;
    const uint64_t hi = min(lo + (uint64_t)kRangeUnit, fd.n);
    if (fd.dtype == 1) {
        for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) fd.outd[i] = fd.cval;
    } else {
        for (uint64_t i = lo + threadIdx.x; i < hi; i += kBlock) fd.outf[i] = (float)fd.cval;
    }
}

template <class OT>
static void reconstruct_launch(const FieldDesc* F, int nf, int rank, bool vec, uint32_t wg_tiles, hipStream_t s)
{
    const dim3 g(wg_tiles);
    if (rank == 1) {
        const dim3 b(kBlock);
        if (vec) hipLaunchKernelGGL((k_reconstruct<true, OT>), g, b, 0, s, F, nf);
        else hipLaunchKernelGGL((k_reconstruct<false, OT>), g, b, 0, s, F, nf);
    } else {
        const dim3 b(kWave);  // one wave per tile
        if (vec) hipLaunchKernelGGL((k_reconstruct2<true, OT>), g, b, 0, s, F, nf);
        else hipLaunchKernelGGL((k_reconstruct2<false, OT>), g, b, 0, s, F, nf);
    }
}

hipError_t launch_reconstruct(const FieldDesc* F, int nf, int rank, bool vec, bool f64, uint32_t wg_tiles,
                              hipStream_t s)
{
    if (wg_tiles == 0) return hipSuccess;
    if (f64) reconstruct_launch<double>(F, nf, rank, vec, wg_tiles, s);
    else reconstruct_launch<float>(F, nf, rank, vec, wg_tiles, s);
    return hipGetLastError();
}

hipError_t launch_rle_reconstruct(const FieldDesc* F, int nf, uint32_t rt_units, const uint32_t* starts,
                                  const uint32_t* tmap, hipStream_t s)
{
    hipLaunchKernelGGL(k_rle_reconstruct, dim3(rt_units), dim3(kBlock), 0, s, F, nf, starts, tmap);
    return hipGetLastError();
}

hipError_t launch_reconstruct3(const FieldDesc* F, int nf, uint32_t units, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_reconstruct3, dim3(units), dim3(kBlock), 0, s, F, nf);
    return hipGetLastError();
}

hipError_t launch_recon_check(const FieldDesc* F, int nf, int32_t* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_recon_check, dim3(nf), dim3(kWave), 0, s, F, st);
    return hipGetLastError();
}

hipError_t launch_fill_const(const FieldDesc* F, int nf, uint32_t units, hipStream_t s)
{
    if (!units) return hipSuccess;
    hipLaunchKernelGGL(k_fill_const, dim3(units), dim3(kBlock), 0, s, F, nf);
    return hipGetLastError();
}

}  // namespace ebc
