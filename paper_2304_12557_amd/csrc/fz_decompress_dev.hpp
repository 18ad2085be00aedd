// fz_decompress_dev.hpp -- device code of the decompressor, shared by the
// per-field kernel (fz_decompress.hip) and the batched one (fz_batch.hip).
//
// The inverse of the compression pass (Sec. 4.4 calls the two pipelines
// symmetric).  A workgroup per chunk, its 16 steps shared out over the waves
// (8 waves of 2 steps, or 16 of 1; several chunks of a thin last layer to a
// workgroup).  Each lane loads its steps' words of its
// nonzero bricks (their positions follow from the bit flags by popcount and
// mbcnt, Sec. 3.4), undoes the bitshuffle with the same in-register
// transpose, decodes the sign-magnitude codes (Sec. 3.2), and inverts the
// Lorenzo predictor as inclusive prefix sums: along the patch in registers,
// across lanes for the carries, along the sweep dimension over the wave's own
// steps in registers and over the waves through LDS (the sum of a wave's
// steps is what it adds to every later one).  Then it dequantizes (one fp32
// multiply, Sec. 2.3) and stores.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fz_device.hpp"
#include "fz_format.hpp"
#include "fz_kernels.hpp"

namespace fz {

// The stream's header as 32-bit words.
struct Header {
    uint32_t w[kHeaderBytes / 4];
};
__device__ __forceinline__ Header load_header(const uint8_t* __restrict__ s)
{
    const ConstMem<uint32_t>* hw = const_mem<uint32_t>(s);
    Header h;
#pragma unroll
    for (int i = 0; i < kHeaderBytes / 4; i++) h.w[i] = hw[i];
    return h;
}

// dtype: 0 for an fp32 output, 1 for fp64; predictor: the header byte 15
// the caller handles (0 chunk-local Lorenzo, 1 field-global); s_bytes: the
// bytes readable at s (at least the header, table and flags, checked on the
// host)
__device__ __forceinline__ uint32_t check_header(const Header& h, const Geom& g, int rank, int dtype, int predictor,
                                                 uint64_t s_bytes)
{
    const uint32_t (&w)[kHeaderBytes / 4] = h.w;
    auto byte_at = [&](int off) { return (w[off / 4] >> (8 * (off % 4))) & 0xFFu; };
    auto u64_at = [&](int off) { return (uint64_t)w[off / 4] | ((uint64_t)w[off / 4 + 1] << 32); };
    bool bad = byte_at(kOffDtype) != (uint32_t)dtype || byte_at(kOffRank) != (uint32_t)rank ||
               byte_at(kOffEbMode) > (dtype ? 1u : 2u) || byte_at(kOffPredictor) != (uint32_t)predictor;
    if (dtype) {  // 2 eb as a normal, finite double
        const double e2 = __longlong_as_double((long long)u64_at(kOffEbx2F64));
        bad |= !(e2 >= 2.2250738585072014e-308 && e2 <= 1.7976931348623157e308);
    }
    const float st = __uint_as_float(w[kOffEbx2 / 4]);  // the point-wise mode's step: an integer in [2, 2^24)
    bad |= byte_at(kOffEbMode) == 2 && (!(st >= 2.0f && st < 16777216.0f) || st != __builtin_floorf(st));
#pragma unroll
    for (int i = 0; i < 3; i++) bad |= u64_at(kOffDims + 8 * i) != (uint64_t)g.n[i];
    bad |= w[kOffNChunks / 4] != (uint32_t)g.n_chunks;
    const uint64_t total = u64_at(kOffTotal);
    bad |= total < (uint64_t)g.payload_off || ((total - g.payload_off) & 15) != 0 || total > s_bytes;
    // the codes in the order of their precedence
    return w[kOffMagic / 4] != kMagic ? 6u                                                          // FZ_ERR_STREAM
         : w[kOffVersion / 4] != ((uint32_t)kVersion | ((uint32_t)kHeaderBytes << 16)) ? 7u  // FZ_ERR_VERSION
         : w[kOffStatus / 4] != 0u ? 8u                                                      // FZ_ERR_STATUS
         : bad ? 6u : 0u;
}

// Sign-magnitude decode (Sec. 3.2): P[i] holds the codes of cells i and
// i + 16 (sign in bit 15), decoded in packed 16-bit arithmetic, d = (m ^ s) - s
// with s = 0 or -1, and widened (where the sums that follow allow it, inside
// their adds).
__device__ __forceinline__ void decode_codes(const uint32_t (&P)[16], int (&d)[32])
{
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const fz_short2 s = __builtin_bit_cast(fz_short2, P[i]) >> 15;
        const fz_short2 m = __builtin_bit_cast(fz_short2, P[i] & 0x7FFF7FFFu);
        const fz_short2 r = (m ^ s) - s;
        d[i] = r.x;
        d[i + 16] = r.y;
    }
}

// Orders one wave's LDS accesses to its own tile (writes before the reads of
// other lanes, reads before the next rewrite): the compiler may not move
// memory operations across it, and the wave waits for its LDS operations.
// A workgroup barrier is not needed (no other wave touches the tile) and not
// possible where the waves of a workgroup run different numbers of steps.
__device__ __forceinline__ void wave_lds_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// LDS of one wave (kRegionWords 32-bit words): first its share of the carry
// exchange (2048 ints), then the tile through which it stores a step, so that
// every store instruction writes whole rows: 3-D, 32 rows of 64 values, the
// 16-byte pieces of row r exchanged by XOR with r / 4 (a lane's patch row;
// without it the 8 lanes of a column of patches write to the same banks:
// half of the kernel's LDS cycles were conflicts); 2-D and 1-D, the step's
// 2048 values in order with 4 words of padding after every 32.  Both spread a
// wave's 16-byte accesses over the banks.  fp64 steps pass through it half by
// half.
constexpr int kRegionWords = 2048 + 4 * (2048 / 32);
constexpr int kRegionBad = 2048;  // beside the carry: whether the wave found a bad escape
// places in a 2-D or 1-D tile, written so that all but the lane's part is an
// immediate offset: value i sits at i + 4 (i / 32), double i (of 1024, which
// fill a region) at i + 2 (i / 16)
template <int RANK>
__device__ __forceinline__ int run_put(int j, int lane)  // the j-th 4 of a lane's 32 values
{
    return RANK == 2 ? 1152 * (j >> 2) + 16 * lane + 4 * (lane >> 1) + 4 * (j & 3) : 36 * lane + 4 * j;
}
__device__ __forceinline__ int run_get(int i, int lane) { return 288 * i + 4 * lane + 4 * (lane >> 3); }  // values 256 i + 4 lane ..
__device__ __forceinline__ int run_put64(int j, int lane) { return 18 * lane + 2 * j; }  // the j-th 2 of a lane's 16 doubles
__device__ __forceinline__ int run_get64(int i, int lane) { return 144 * i + 2 * lane + 2 * (lane >> 3); }  // doubles 128 i + 2 lane ..

// an offset past the range of any resource below: the store is dropped
constexpr uint32_t kNoStore = 0xFFFFFFF0u;

// What a step of a chunk covers of the output: `rows` x `cols` values from
// `base`, row pitch `nx` (3-D: a plane; 2-D: two rows; 1-D: one run).
template <typename T>
struct StepOut {
    T* base;
    int64_t nx;
    int rows, cols;
};

template <int RANK, typename T>
__device__ __forceinline__ StepOut<T> step_out(T* __restrict__ y, const Geom& g, const int64_t (&org)[3],
                                               const int64_t (&ext)[3], int st)
{
    // uniform, and kept in scalar registers: a resource built from a vector
    // register would put a loop around each store
    auto uni = [](int64_t v) { return __builtin_amdgcn_readfirstlane((int)v); };
    if (RANK == 3)
        return {as_global(y + ((org[0] + st) * g.n[1] + org[1]) * g.n[2] + org[2]), g.n[2], uni(ext[1]), uni(ext[2])};
    if (RANK == 2)
        return {as_global(y + (org[0] + 2 * st) * g.n[1] + org[1]), g.n[1], min(2, uni(ext[0]) - 2 * st), uni(ext[1])};
    return {as_global(y + org[0] + (int64_t)kStepCodes * st), 0, 1, min(kStepCodes, uni(ext[0]) - kStepCodes * st)};
}

// Store one step of 32-bit values (fp32, or the integers), held as 32 words
// per lane, through the wave's tile.  Store instruction i writes 16 bytes per
// lane: 4 rows of 64 values of a 3-D plane, or 1 KiB of a 2-D row or 1-D run.
// stream: nontemporal stores, for whole lines only (kCacheStream); 4-byte
// alignment suffices for a 16-byte buffer store.  edge: the step is cut by
// the field's edge (uniform); pieces outside are skipped, a piece straddling the end of
// a row is stored value by value.
template <int RANK, typename T>
__device__ __forceinline__ void store_step32(const StepOut<T>& o, bool stream, bool edge, const uint32_t (&d)[32], int lane,
                                             uint32_t* tile)
{
    static_assert(sizeof(T) == 4, "32-bit values");
    if (RANK == 3) {
        const int py = lane & 7, px = lane >> 3;
        uint32_t* t = tile + 256 * py;
        const int p0 = 4 * ((2 * px) ^ py), p1 = 4 * ((2 * px + 1) ^ py);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            *reinterpret_cast<uint4*>(t + 64 * r + p0) = make_uint4(d[8 * r], d[8 * r + 1], d[8 * r + 2], d[8 * r + 3]);
            *reinterpret_cast<uint4*>(t + 64 * r + p1) = make_uint4(d[8 * r + 4], d[8 * r + 5], d[8 * r + 6], d[8 * r + 7]);
        }
    } else {
        // 2-D: lane l has columns 16 l .. of both rows; 1-D: values 32 l ..
#pragma unroll
        for (int j = 0; j < 8; j++)
            *reinterpret_cast<uint4*>(tile + run_put<RANK>(j, lane)) = make_uint4(d[4 * j], d[4 * j + 1], d[4 * j + 2], d[4 * j + 3]);
    }
    wave_lds_sync();  // orders the tile's writes before its reads
    // offsets stay below 2^32 - 16: at most 32 rows of a contiguous extent
    // below 2^25
    const uint32_t nx = (uint32_t)o.nx;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        o.base, (short)0, !edge ? -1 : o.rows > 0 ? (int)(4u * ((uint32_t)(o.rows - 1) * nx + (uint32_t)o.cols)) : 0,
        kBufferFlags);
    auto piece = [&](int i) {
        return *reinterpret_cast<const fz_u32x4*>(RANK == 3 ? tile + 64 * (4 * i + (lane >> 4)) + 4 * ((lane & 15) ^ i)
                                                            : tile + run_get(i, lane));
    };
    if (!edge) {
        const uint32_t voff = RANK == 3 ? 4u * ((uint32_t)(lane >> 4) * nx + 4u * (uint32_t)(lane & 15)) : 16u * (uint32_t)lane;
        auto soff = [&](int i) {
            return RANK == 3 ? 16u * (uint32_t)i * nx : RANK == 2 ? 4u * (uint32_t)(i >> 2) * nx + 1024u * (i & 3) : 1024u * i;
        };
        fz_u32x4 w[8];
#pragma unroll
        for (int i = 0; i < 8; i++) w[i] = piece(i);
        if (stream) {
#pragma unroll
            for (int i = 0; i < 8; i++) __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, voff, soff(i), kCacheStream);
        } else {
#pragma unroll
            for (int i = 0; i < 8; i++) __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, voff, soff(i), 0);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int row = RANK == 3 ? 4 * i + (lane >> 4) : RANK == 2 ? i >> 2 : 0;
            const int col = RANK == 3 ? 4 * (lane & 15) : RANK == 2 ? 256 * (i & 3) + 4 * lane : 256 * i + 4 * lane;
            const int n = row < o.rows ? o.cols - col : 0;  // values of the piece inside the field
            const uint32_t voff = 4u * ((uint32_t)row * nx + (uint32_t)col);
            const fz_u32x4 w = piece(i);
            __builtin_amdgcn_raw_buffer_store_b128(w, rs, n >= 4 ? voff : kNoStore, 0u, 0);
            if (o.cols & 3) {  // uniform: rows that end inside a piece
                __builtin_amdgcn_raw_buffer_store_b32(w.x, rs, n > 0 && n < 4 ? voff : kNoStore, 0u, 0);
                __builtin_amdgcn_raw_buffer_store_b32(w.y, rs, n > 1 && n < 4 ? voff + 4u : kNoStore, 0u, 0);
                __builtin_amdgcn_raw_buffer_store_b32(w.z, rs, n == 3 ? voff + 8u : kNoStore, 0u, 0);
            }
        }
    }
    wave_lds_sync();  // the tile is rewritten by the next step
}

// The same for doubles, in two halves: rows 4 py + 2 h, + 1 of every patch
// (3-D), row h (2-D), values 16 h .. 16 h + 15 of every lane's 32 (1-D).
// Store instruction i writes 16 bytes per lane, whole 128-byte lines: 2 rows
// of 64 doubles, 1 KiB of a row, or 8 runs of 16 doubles.
template <int RANK>
__device__ __forceinline__ void store_step64(const StepOut<double>& o, bool stream, bool edge, const int (&d)[32], double ebx2,
                                             int lane, uint32_t* tile)
{
    double* t64 = reinterpret_cast<double*>(tile);
#pragma unroll
    for (int h = 0; h < 2; h++) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int i = 16 * h + 2 * j;
            double* t = RANK == 3 ? t64 + 128 * (lane & 7) + 64 * (j >> 2) + 2 * ((4 * (lane >> 3) + (j & 3)) ^ (lane & 7))
                                  : t64 + run_put64(j, lane);
            *reinterpret_cast<double2*>(t) = make_double2((double)d[i] * ebx2, (double)d[i + 1] * ebx2);
        }
        wave_lds_sync();  // orders the tile's writes before its reads
        fz_u32x4 w[8];
#pragma unroll
        for (int i = 0; i < 8; i++)
            w[i] = *reinterpret_cast<const fz_u32x4*>(RANK == 3 ? t64 + 64 * (2 * i + (lane >> 5)) + 2 * ((lane & 31) ^ i)
                                                                : t64 + run_get64(i, lane));
        const uint32_t pitch = RANK == 3 ? (uint32_t)o.nx : 0u;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            // the instruction's first row is uniform: its resource starts there
            const int at = 128 * i + 2 * lane;  // 2-D, 1-D: the value's place in the half
            const int row0 = RANK == 3 ? 4 * i + 2 * h : RANK == 2 ? h : 0, row = row0 + (RANK == 3 ? lane >> 5 : 0);
            const int col = RANK == 3 ? 2 * (lane & 31) : RANK == 2 ? at : 32 * (at >> 4) + 16 * h + (at & 15);
            const int left = o.rows - row0;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                o.base + (int64_t)row0 * o.nx, (short)0,
                !edge ? -1 : left > 0 ? (int)(8u * ((left > 1 ? pitch : 0u) + (uint32_t)o.cols)) : 0, kBufferFlags);
            const uint32_t voff = 8u * ((RANK == 3 ? (uint32_t)(lane >> 5) * pitch : 0u) + (uint32_t)col);
            if (!edge) {
                if (stream) __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, voff, 0u, kCacheStream);
                else __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, voff, 0u, 0);
            } else {
                const int n = row < o.rows ? o.cols - col : 0;  // values of the piece inside the field
                __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, n >= 2 ? voff : kNoStore, 0u, 0);
                if (o.cols & 1)  // uniform: rows that end inside a piece
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_shufflevector(w[i], w[i], 0, 1), rs, n == 1 ? voff : kNoStore, 0u, 0);
            }
        }
        wave_lds_sync();  // the tile is rewritten by the next half
    }
}

// 3-D: inclusive prefix of one plane of deltas along x, then y (the lane's
// 4x8 patch at rows 4 py.., columns 8 px..): inside the patch, with the carry
// across the lanes 8 apart (DPP and lane swaps) along x and across lanes -1,
// -2, -4 (a shift inside the 16-lane row) along y.
__device__ __forceinline__ void plane_prefix3(int (&d)[32], int lane)
{
    const int py = lane & 7;
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int cc = 1; cc < 8; cc++) d[8 * r + cc] += d[8 * r + cc - 1];
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const int ex_ = excl_scan_stride8(d[8 * r + 7], lane);
#pragma unroll
        for (int cc = 0; cc < 8; cc++) d[8 * r + cc] += ex_;
    }
#pragma unroll
    for (int r = 1; r < 4; r++)
#pragma unroll
        for (int cc = 0; cc < 8; cc++) d[8 * r + cc] += d[8 * (r - 1) + cc];
    // the carry over the 8 lanes of a column of patches: a shift by 1 and by 2
    // inside the 16-lane row, lanes whose value would reach the next 8 cleared
    // first, so that each shift fuses with its add; a shift by 4 into the
    // upper half of each 8 only (a bank mask)
    const int m1 = py == 7 ? 0 : -1, m2 = py >= 6 ? 0 : -1;
#pragma unroll
    for (int cc = 0; cc < 8; cc++) {
        const int C = d[24 + cc];
        int inc = C + row_shr<1>(C & m1);
        inc += row_shr<2>(inc & m2);
        inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xf, 0xa, false);
        const int ex_ = inc - C;
#pragma unroll
        for (int r = 0; r < 4; r++) d[8 * r + cc] += ex_;
    }
}

// 2-D: inclusive prefix along x of one row held as 16 values per lane (lane
// l has columns 16 l .. 16 l + 15)
__device__ __forceinline__ void row_prefix2(int* d, int lane)
{
#pragma unroll
    for (int cc = 1; cc < 16; cc++) d[cc] += d[cc - 1];
    const int tot = d[15];
    const int ex_ = wave_incl_scan(tot) - tot;
#pragma unroll
    for (int cc = 0; cc < 16; cc++) d[cc] += ex_;
}

// Workgroup-shared state of a decompression workgroup of NW waves.
template <int NW>
struct DecompressLds {
    __attribute__((aligned(16))) uint32_t region[NW][kRegionWords];  // per wave: its carry, then its tile
};

// A step's escape codes (sign set, magnitude 0; they decode to 0), one bit per
// cell, from the words of its 16 bit planes (plane 15: the signs).
__device__ __forceinline__ uint32_t escape_mask(const uint32_t (&P)[16])
{
    uint32_t mag = 0u;
#pragma unroll
    for (int b = 0; b < 15; b++) mag |= P[b];
    return P[15] & ~mag;
}

// The logged deltas of one step's escape codes (emask), added to d.  Pairs
// are strictly ascending in the code index; those of the wave's steps are
// pairs lo .. hi - 1.  Each lane takes pairs and scatters the step's deltas
// into the wave's (zeroed) LDS region, from where every lane reads the ones of
// its cells: no branch per cell and one round trip for all of them.  Returns
// nonzero unless the step's pairs and its escape codes are the same cells and
// every one of the pairs lies in the wave's `codes` codes from `first`.
__device__ __forceinline__ uint32_t add_escapes(uint32_t emask, int (&d)[32], const uint32_t* __restrict__ pairs,
                                                uint32_t lo, uint32_t hi, uint32_t first, uint32_t codes, uint32_t n0,
                                                int lane, uint32_t* region)
{
    int left = __popc(emask);
    uint32_t bad = 0;
#pragma unroll
    for (int j = 0; j < 8; j++) *reinterpret_cast<uint4*>(region + 256 * j + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_sync();  // zeros before the scatter
    for (uint32_t j0 = lo; j0 < hi; j0 += 64) {
        const uint32_t j = j0 + (uint32_t)lane;
        uint32_t at = 0xFFFFFFFFu, delta = 0u;  // relative to the step: past it for a lane without a pair
        if (j < hi) {
            const uint32_t n = pairs[2 * j];
            delta = pairs[2 * j + 1];
            bad |= n - first >= codes || (j + 1 < hi && pairs[2 * j + 2] <= n) ? 1u : 0u;
            at = n - n0;
        }
        const bool mine = at < (uint32_t)kStepCodes;
        const uint32_t patch = (at >> 5) & 63u, cell = at & 31u;
        const uint32_t em = (uint32_t)lane_value((int)emask, (int)patch);
        if (mine) {
            bad |= ((em >> cell) & 1u) ^ 1u;
            region[256 * (cell >> 2) + 4 * patch + (cell & 3u)] = delta;
            left--;
        }
    }
    wave_lds_sync();  // the scatter before the reads
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const uint4 v = *reinterpret_cast<const uint4*>(region + 256 * j + 4 * lane);
        d[4 * j] += (int)v.x;
        d[4 * j + 1] += (int)v.y;
        d[4 * j + 2] += (int)v.z;
        d[4 * j + 3] += (int)v.w;
    }
    wave_lds_sync();  // the region is written again
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) left += __shfl_xor(left, sh);
    return bad | (left != 0 ? 1u : 0u);
}

// In-plane part of the inverse predictor (the sums along the sweep dimension
// follow): 3-D along x and y; 2-D along x, then the second row on the first;
// 1-D along x over the step.
template <int RANK>
__device__ __forceinline__ void step_prefix(int (&d)[32], int lane)
{
    if (RANK == 3) {
        plane_prefix3(d, lane);
    } else if (RANK == 2) {
        row_prefix2(d, lane);
        row_prefix2(d + 16, lane);
#pragma unroll
        for (int cc = 0; cc < 16; cc++) d[16 + cc] += d[cc];
    } else {
#pragma unroll
        for (int m = 1; m < 32; m++) d[m] += d[m - 1];
        const int tot = d[31];
        const int ex_ = wave_incl_scan(tot) - tot;
#pragma unroll
        for (int m = 0; m < 32; m++) d[m] += ex_;
    }
}

// A following chunk's payload is brought into the L2 up to this size (32 KB):
// those of the 64 chunks at work on an XCD then take up to half of its 4 MB.
// Measured (us, cached / cold, none / up to 32 KB / all): 512^3 of 23 KB a chunk
// 109.9 / 136.6, 107.7 / 118.1, 106.6 / 118.7; of 37 KB 114.0 / 137.7, 111.9 /
// 134.7, 121.6 / 128.6.
constexpr uint32_t kWarmUnits = 32768 / 16;

// Decompress chunk c of a field with `waves` waves of a workgroup, whose LDS
// regions are S; wave w runs the 16 / NW steps from w * 16 / NW, and waves = NW
// unless the chunk has no cells past the steps of fewer.  A stream that fails a
// check writes an fz_status code to *d_err (if given) and leaves the chunk's
// output untouched.  No byte at or past s + s_bytes is read: the header's total
// is checked against s_bytes, and every chunk's payload against the total.
// All checks give the same result in every wave of a chunk, so they return
// together; between the waves of a workgroup's other chunks, which go on, the
// barriers only count those left.
//
// Sweep dimension: what a step adds to the later ones is its last in-plane
// prefix (3-D: the plane; 2-D: its second row; 1-D: its last value).  Each
// wave sums its own steps in registers, leaves the sum in its LDS region, and
// after a barrier adds the regions of the waves before it.  Holding every
// step in registers, no step is decoded twice and none waits for the one
// before it.
//
// What bounds it: VALU issue (584 instructions per step and wave, 68 % of the
// cycles on 512^3) with the stores behind it; two workgroups per CU overlap
// one's loads and barriers with the other's arithmetic.  Measured against one
// wave per chunk (4 waves for at most 512 chunks) before, REL 1e-3, buffers in
// turn / from cold caches: 512^3 113 -> 101 / 127 -> 116 us, 100x500x500 50 -> 30 /
// 54 -> 32, 8192^2 55 -> 51 / 59 -> 59, 2^26 values 63 -> 53 / 70 -> 62, 1800x3600
// 19 -> 12 / 26 -> 15, 64^3 17 -> 10 / 26 -> 13.  Without the reads ahead (next_c)
// the large ones were slower from cold caches: 512^3 141, 8192^2 70 us.
//
// WARM: next_c is the chunk that takes this one's place on the device (-1: none).  Its
// flags and payload are brought into the L2 while this one is worked on: the
// chain of a chunk starts with two reads one after the other (table and flags,
// then bricks), whose latency from HBM two workgroups a CU do not cover.
template <int RANK, typename T, int NW, bool WARM = false>
__device__ __forceinline__ void decompress_chunk(const uint8_t* __restrict__ s, uint64_t s_bytes, T* __restrict__ y,
                                                 bool stream, const Geom& g, uint32_t* d_err, int64_t c, int wave, int lane,
                                                 DecompressLds<NW>& S, int64_t next_c = -1, int waves = NW)
{
    static_assert(NW == 8 || NW == 16, "2 or 1 steps per wave");
    constexpr int NS = kSteps / NW;
    constexpr bool F64 = sizeof(T) == 8;
    constexpr bool INT = std::is_integral_v<T>;
    // lane i holds flag word i of the chunk (layer i / 16, plane i % 16); the
    // wave's own layer's words also come as scalars
    const uint8_t* flags = s + g.flags_off + (int64_t)kFlagBytesPerChunk * c;
    const uint64_t f = reinterpret_cast<const uint64_t*>(flags)[lane];
    // words 0 .. 2 of the next chunk's place in the table on lanes 0 .. 2: its
    // offset, and (not for the last chunk) the next one's
    uint32_t next_tab = 0u;
    if constexpr (WARM)
        next_tab = __builtin_amdgcn_raw_buffer_load_b32(
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(s) + g.table_off + 8 * max(next_c, (int64_t)0), (short)0,
                                              next_c < 0 ? 0 : next_c + 1 < g.n_chunks ? 12 : 8, kBufferFlags),
            4u * (uint32_t)lane, 0u, 0);
    const int s0 = NS * wave, k = s0 >> 2;
    const ConstMem<uint64_t>* fk = const_mem<uint64_t>(flags + 8 * kPlanes * k);
    uint64_t F[kPlanes];
#pragma unroll
    for (int b = 0; b < kPlanes; b++) F[b] = fk[b];
    const ConstMem<uint32_t>* tab = const_mem<uint32_t>(s + g.table_off + 8 * c);
    const uint32_t off = tab[0], nout = tab[1], next_off = tab[2];  // (behind the last chunk's: padding or its flags)
    const Header h = load_header(s);
    // WARM: what the chunk starts from, all on its way before any of it is looked
    // at; left to itself the compiler puts each load behind the check before
    // it, and from HBM each waits in turn.
    if constexpr (WARM)
        asm volatile("" ::"s"(F[0]), "s"(F[1]), "s"(F[2]), "s"(F[3]), "s"(F[4]), "s"(F[5]), "s"(F[6]), "s"(F[7]), "s"(F[8]), "s"(F[9]),
                     "s"(F[10]), "s"(F[11]), "s"(F[12]), "s"(F[13]), "s"(F[14]), "s"(F[15]), "s"(off), "s"(nout), "s"(next_off),
                     "s"(h.w[kOffMagic / 4]), "s"(h.w[kOffStatus / 4]), "s"(h.w[kOffDims / 4]), "s"(h.w[kOffEbx2 / 4]),
                     "s"(h.w[kOffNChunks / 4]), "s"(h.w[kOffTotal / 4]));
    const uint32_t hdr_err = check_header(h, g, RANK, F64 ? 1 : 0, INT ? 1 : 0, s_bytes);
    if (hdr_err) {
        if (c == 0 && wave == 0 && lane == 0 && d_err) atomicCAS(d_err, 0u, hdr_err);
        return;
    }
    const uint64_t total = (uint64_t)h.w[kOffTotal / 4] | ((uint64_t)h.w[kOffTotal / 4 + 1] << 32);
    const uint64_t payload_units = (total - g.payload_off) / 16;
    int64_t org[3], ext[3];
    chunk_box(g, c, org, ext);
    const int L = layers_of(RANK, ext[0]);
    const int cnt = __popcll(f);
    const int incl = wave_incl_scan(cnt);
    const uint32_t nnz = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    // the table is the exclusive prefix sum of the chunks' units (Sec. 3.4):
    // this chunk's offset plus its units (from the flags' popcounts and its
    // escape count) is the next chunk's offset, or the payload's end.  Chunks
    // are checked independently, so each also checks that it ends inside the
    // payload.
    const uint64_t next = c + 1 < g.n_chunks ? (uint64_t)next_off : payload_units;
    const uint64_t end = (uint64_t)off + nnz + (nout + 1) / 2;
    const bool bad = nout > (uint32_t)kChunkOutlierCap || end != next || end > payload_units || (c == 0 && off != 0) ||
                     __ballot(f != 0 && lane >= L * kPlanes) != 0;
    if (bad) {
        if (wave == 0 && lane == 0 && d_err) atomicCAS(d_err, 0u, 6u);
        return;
    }

    // The wave's words: plane b of this lane's brick holds the words of steps
    // s0 .. s0 + NS - 1 at byte voff of the chunk's payload.  A zero brick
    // gets an offset beyond the resource's range, where the load returns 0
    // without touching memory.
    const uint4* pay = reinterpret_cast<const uint4*>(s + g.payload_off) + off;
    const uint32_t skip = 4u * (uint32_t)(s0 & 3);  // the step's word in a brick, in the resource's base
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<uint8_t*>(const_cast<uint4*>(pay)) + skip, (short)0, nnz ? (int)(16u * nnz - skip) : 0, kBufferFlags);
    uint32_t base = (uint32_t)__builtin_amdgcn_readlane(incl - cnt, k * kPlanes);
    uint32_t W[NS][16];
#pragma unroll
    for (int b = 0; b < 16; b++) {
        const uint32_t at = (base + mbcnt(F[b])) << 4;
        const uint32_t voff = __builtin_amdgcn_inverse_ballot_w64(F[b]) ? at : 0x80000000u;
        base += (uint32_t)__builtin_popcountll(F[b]);
        if constexpr (NS == 2) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, 0u, 0);
            W[0][b] = t[0];
            W[1][b] = t[1];
        } else {
            W[0][b] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, 0u, 0);
        }
    }

    // One load per line, issued behind the words and used by nothing (held to
    // the end below).  A wave's two steps have at most 64 lines.
    uint32_t warm = 0u, warm_flags = 0u;
    if constexpr (WARM) {
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)next_tab, 0);
        const uint64_t to = next_c + 1 < g.n_chunks ? (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)next_tab, 2) : payload_units;
        const uint32_t units = next_c >= 0 && to > at && to <= payload_units && to - at <= kWarmUnits ? (uint32_t)(to - at) : 0u;
        warm = __builtin_amdgcn_raw_buffer_load_b32(
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(s) + g.payload_off + 16 * (int64_t)at, (short)0,
                                              (int)(16u * units), kBufferFlags),
            128u * (uint32_t)(64 * wave + lane), 0u, 0);
        warm_flags = __builtin_amdgcn_raw_buffer_load_b32(
            __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint8_t*>(s) + g.flags_off + (int64_t)kFlagBytesPerChunk * max(next_c, (int64_t)0), (short)0,
                next_c >= 0 && wave == 0 ? kFlagBytesPerChunk : 0, kBufferFlags),
            128u * (uint32_t)lane, 0u, 0);
    }

    // steps of the chunk inside the field (the others hold no cell of it)
    const int live = (int)(RANK == 3 ? ext[0] : RANK == 2 ? (ext[0] + 1) / 2 : (ext[0] + kStepCodes - 1) / kStepCodes);
    // escape pairs are in code-index order: those of this wave's steps are the
    // ones from `seen` (indices below its first code) to `seen_end`
    const uint32_t* pairs = reinterpret_cast<const uint32_t*>(pay + nnz);
    uint32_t seen = 0, seen_end = 0, esc_bad = 0;
    const uint32_t first = (uint32_t)s0 * kStepCodes;
    if (nout) {
        uint32_t n0 = 0, n1 = 0;
        for (uint32_t j = (uint32_t)lane; j < nout; j += 64) {
            const uint32_t at = pairs[2 * j];
            n0 += at < first ? 1u : 0u;
            n1 += at < first + (uint32_t)NS * kStepCodes ? 1u : 0u;
            esc_bad |= at >= (uint32_t)live * kStepCodes ? 1u : 0u;
        }
#pragma unroll
        for (int sh = 32; sh > 0; sh >>= 1) {
            n0 += (uint32_t)__shfl_xor((int)n0, sh);
            n1 += (uint32_t)__shfl_xor((int)n1, sh);
        }
        seen = n0;
        seen_end = n1;
    }

    int d[NS][32];
#pragma unroll
    for (int t = 0; t < NS; t++) {
        if (s0 + t < live) {
            if (nout) {
                const uint32_t emask = escape_mask(W[t]);
                transpose16(W[t]);
                decode_codes(W[t], d[t]);
                esc_bad |= add_escapes(emask, d[t], pairs, seen, seen_end, first, (uint32_t)NS * kStepCodes,
                                       (uint32_t)(s0 + t) * kStepCodes, lane, S.region[wave]);
                step_prefix<RANK>(d[t], lane);
            } else {  // without the branch inside, the widening of the codes goes into the adds
                transpose16(W[t]);
                decode_codes(W[t], d[t]);
                step_prefix<RANK>(d[t], lane);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 32; i++) d[t][i] = 0;
        }
        __builtin_amdgcn_sched_barrier(0);  // one step's arrays at a time: 128 registers
    }
    // sums along the sweep dimension: what the wave's steps add to later ones
    // goes to its region, those of the waves before are added to its first
    // step, and that one to its second
    constexpr int NC = RANK == 3 ? 8 : 4;   // a wave's sum (2-D, 3-D): NC x 4 values per lane
    constexpr int C0 = RANK == 3 ? 0 : 16;  // from value C0 of a step
    auto put_sum = [&]() {
        int* xw = reinterpret_cast<int*>(S.region[wave]);
#pragma unroll
        for (int j = 0; j < NC; j++) {
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; i++) q[i] = d[NS - 1][C0 + 4 * j + i] + (NS == 2 ? d[0][C0 + 4 * j + i] : 0);
            *reinterpret_cast<int4*>(xw + 256 * j + 4 * lane) = make_int4(q[0], q[1], q[2], q[3]);
        }
    };
    auto add_sum = [&](int j) {
        const int* xj = reinterpret_cast<const int*>(S.region[j]);
#pragma unroll
        for (int i = 0; i < NC; i++) {
            const int4 v = *reinterpret_cast<const int4*>(xj + 256 * i + 4 * lane);
            d[0][4 * i] += v.x;
            d[0][4 * i + 1] += v.y;
            d[0][4 * i + 2] += v.z;
            d[0][4 * i + 3] += v.w;
            if (RANK == 2) {
                d[0][16 + 4 * i] += v.x;
                d[0][16 + 4 * i + 1] += v.y;
                d[0][16 + 4 * i + 2] += v.z;
                d[0][16 + 4 * i + 3] += v.w;
            }
        }
    };
    if (RANK >= 2) put_sum();
    else if (lane == 63) S.region[wave][0] = (uint32_t)(d[NS - 1][31] + (NS == 2 ? d[0][31] : 0));
    if (nout) {
        const bool any = __ballot(esc_bad != 0u) != 0;
        if (lane == 0) S.region[wave][kRegionBad] = any ? 1u : 0u;
    }
    __syncthreads();
    if (nout && __ballot(S.region[lane < waves ? lane : 0][kRegionBad] != 0u)) {
        // not every escape code has its pair, or not every pair its escape code
        if (wave == 0 && lane == 0 && d_err) atomicCAS(d_err, 0u, 6u);
        return;
    }
    if (RANK >= 2) {
        // in groups of 4 waves: first the waves before in the group, then the
        // groups before, whose sum their last wave leaves in its region (no
        // wave has read that one yet): 16 region reads per chunk, not 28
#pragma unroll 1
        for (int j = wave & ~3; j < wave; j++) add_sum(j);
        if ((wave & 3) == 3 && wave < NW - 1) put_sum();
        __syncthreads();
#pragma unroll 1
        for (int j = 3; j < (wave & ~3); j += 4) add_sum(j);
    } else {
        int carry = lane < wave ? (int)S.region[lane < NW ? lane : 0][0] : 0;
#pragma unroll
        for (int sh = 8; sh > 0; sh >>= 1) carry += __shfl_xor(carry, sh);  // the waves' lanes 0 .. 15
        carry = __builtin_amdgcn_readfirstlane(carry);
#pragma unroll
        for (int i = 0; i < 32; i++) d[0][i] += carry;
    }
    if (NS == 2) {
        const int last = RANK == 1 ? __builtin_amdgcn_readlane(d[0][31], 63) : 0;
#pragma unroll
        for (int i = 0; i < 32; i++) d[NS - 1][i] += RANK == 3 ? d[0][i] : RANK == 2 ? d[0][16 + (i & 15)] : last;
    }
    __syncthreads();  // the regions become the waves' tiles
    if constexpr (WARM) asm volatile("" ::"v"(warm), "v"(warm_flags));

    const uint32_t mode = (const_mem<uint32_t>(s)[kOffEbMode / 4] >> (8 * (kOffEbMode % 4))) & 0xFFu;
#pragma unroll
    for (int t = 0; t < NS; t++) {
        if (s0 + t >= live) break;
        const StepOut<T> o = step_out<RANK, T>(y, g, org, ext, s0 + t);
        const bool edge = RANK == 3 ? o.rows < 32 || o.cols < 64 : RANK == 2 ? o.rows < 2 || o.cols < 1024 : o.cols < kStepCodes;
        if constexpr (F64) {
            const double ebx2 = *const_mem<double>(s + kOffEbx2F64);
            store_step64<RANK>(o, stream, edge, d[t], ebx2, lane, S.region[wave]);
        } else {
            // Dequantization (Sec. 2.3): q * 2eb, one fp32 multiply, or in the
            // point-wise relative mode the inverse of the bit-pattern
            // transform with the stream's step (checked by check_header); the
            // integers themselves for the field-global predictor
            uint32_t v[32];
            const float ebx2 = *const_mem<float>(s + kOffEbx2);
            if (INT) {
#pragma unroll
                for (int i = 0; i < 32; i++) v[i] = (uint32_t)d[t][i];
            } else if (mode == 2) {
                const uint32_t step = (uint32_t)ebx2;
#pragma unroll
                for (int i = 0; i < 32; i++) v[i] = __float_as_uint(pw_dequant(d[t][i], step));
            } else {
#pragma unroll
                for (int i = 0; i < 32; i++) v[i] = __float_as_uint((float)d[t][i] * ebx2);
            }
            store_step32<RANK>(o, stream, edge, v, lane, S.region[wave]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The chunk of block b of an fp32-sized decompression.  Plain stores: in runs
// per XCD (xcd_order).  Streaming stores fill whole lines, which no two chunks
// share: in order.
template <bool STREAM>
__device__ __forceinline__ int64_t in_place_chunk(const Geom& g, uint32_t b)
{
    return STREAM ? (int64_t)b : xcd_order(b, g.n_chunks);
}

// The same where more chunks than are at work at once make up n chunks in whole
// layers.  With streaming stores each XCD (every eighth block) would write the
// same columns of every row and plane, in 2-D where rows are multiples of 32 KB
// the same 4 KB modulo 32 KB.  So in 3-D the rows of chunks are turned against one
// another, and such 2-D fields take runs of 8 per XCD.  Measured, in order /
// turned / (runs of 8): 64x1024x2048 114.7 / 108.3 / (110.3) us, 32x2048x2048 109.6
// / 102.3 / (103.3), 2048x256x256 108.8 / 100.3 / (106.0), 512^3 101.0 / 100.5 /
// (104.6); 2-D 64x2^20 70.7 / - / (58.7), 32x2^20 39.1 / - / (33.9), 1000x100000
// 73.4 / - / (78.5).  fp64 rows that are no whole lines share them as plain fp32
// stores do, and short rows of chunks lose by turning: runs (fp64, turned / runs:
// 32x1024x2048 104.6 / 118.7, 256x512x512 106.9 / 109.9, 1024x256x256 107.4 / 97.8).
// With plain divisions: by multiply-high on the scalar unit the turned order
// measured 111.8, 107.1, 104.0 and 104.3 in the four fp32 fields.
template <int RANK, typename T, bool STREAM>
__device__ __forceinline__ int64_t turned_chunk(const Geom& g, uint32_t b, int64_t n)
{
    const uint32_t row_bytes = (uint32_t)g.n[RANK - 1] * (uint32_t)sizeof(T);  // (2-D, 3-D: below 2^28)
    if (!STREAM || (RANK == 2 && (row_bytes & 32767u) == 0)) return xcd_order(b, n);
    if (sizeof(T) == 8 && RANK >= 2 && ((row_bytes & 127u) != 0 || (RANK == 3 && g.grid[2] < (int)kXcdRun)))
        return xcd_order(b, n);
    if (RANK != 3) return b;
    const uint32_t nx = (uint32_t)g.grid[2], ny = (uint32_t)g.grid[1];
    const uint32_t row = b / nx, x = b - row * nx, z = row / ny, y = row - z * ny;
    const uint32_t by = (3 * y + 5 * z) % nx;
    return row * nx + (x + by < nx ? x + by : x + by - nx);
}

// The last layer of a field's chunks (2-D, 3-D), if the field reaches at most 8
// of their 16 steps: as waves take two steps each, 1, 2 or 4 of them run such a
// chunk, and a workgroup of 8 several chunks.  With all 8 on one chunk, those
// without a step only hold wave slots and LDS (1x2048x2048: 19.8 us, now 11.0;
// 4x2048x2048: 27.4, now 17.7; 33x2016x1984, a third of whose chunks have one
// plane: 116.6, now 103.6).
struct ThinLayer {
    uint32_t full;  // chunks before it, one per block
    int lg;         // log2 of the waves that run one of its chunks
    uint32_t blocks(const Geom& g) const
    {
        const uint32_t per = 8u >> lg;
        return full + ((uint32_t)g.n_chunks - full + per - 1) / per;
    }
};
// at_once: the blocks at work at once.  Chunks that find room in the last round
// of the blocks before them are better spread over the CUs it leaves idle
// (100x500x500: 34.3 us shared, 30.0 not).
inline ThinLayer thin_layer(const Geom& g, uint32_t at_once)
{
    const ThinLayer none{(uint32_t)g.n_chunks, 3};
    if (g.rank == 1) return none;
    const int64_t e = g.n[0] - (g.grid[0] - 1) * g.box[0], steps = g.rank == 3 ? e : (e + 1) / 2;
    if (steps > 8) return none;
    const ThinLayer t{(uint32_t)(g.n_chunks - g.grid[1] * g.grid[2]), steps > 4 ? 2 : steps > 2 ? 1 : 0};
    const uint32_t last = t.full % at_once, room = t.full && !last ? 0u : at_once - last;
    return none.full - t.full > room ? t : none;
}

// The per-field kernel (fp32, fp64) for fields of more chunks than are at work at
// once (`ahead`): a workgroup reads ahead for the chunk that takes its place,
// chunks are taken in turned_chunk's order, and a thin last layer shares
// workgroups.  first: the launch's first block of the field (launch_chunks).
// fp64, one wave a chunk / 8 waves / this, us: 32x1024x2048 104 / 118 / 105, cold
// 107 / 128 / 115; 4096x8192 cold 58 / 61 / 56; 40x1000000 cold 75 / 80 / 72.
template <int RANK, typename T, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress_ahead(const uint8_t* __restrict__ s, uint64_t sb,
                                                             T* __restrict__ y, Geom g, uint32_t* d_err, uint32_t first,
                                                             uint32_t ahead, ThinLayer thin)
{
    __shared__ DecompressLds<8> S;
    int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = 8, w0 = 0;
    const uint32_t b = first + blockIdx.x;
    int64_t c, next = -1;
    if (b < thin.full) {
        c = turned_chunk<RANK, T, STREAM>(g, b, thin.full);
        if (b + ahead < thin.full) next = turned_chunk<RANK, T, STREAM>(g, b + ahead, thin.full);
    } else {
        const int lg = thin.lg, per = 8 >> lg;
        c = (int64_t)thin.full + (int64_t)(b - thin.full) * per + (wave >> lg);
        if (c >= g.n_chunks) return;
        if (c + (int64_t)ahead * per < g.n_chunks) next = c + (int64_t)ahead * per;
        waves = 1 << lg;
        w0 = wave & ~(waves - 1);
        wave -= w0;
    }
    decompress_chunk<RANK, T, 8, true>(s, sb, y, STREAM, g, d_err, c, wave, threadIdx.x & 63,
                                           *reinterpret_cast<DecompressLds<8>*>(S.region[w0]), next, waves);
}

template <int RANK, typename T, bool STREAM>
inline hipError_t launch_ahead(const uint8_t* s, uint64_t sb, T* y, const Geom& g, uint32_t* d_err, uint32_t at_once,
                               hipStream_t st)
{
    const ThinLayer thin = thin_layer(g, at_once);
    return launch_chunks(thin.blocks(g), [&](uint32_t first, dim3 blocks) {
        hipLaunchKernelGGL((k_decompress_ahead<RANK, T, STREAM>), blocks, dim3(512), 0, st, s, sb, y, g, d_err, first, at_once,
                           thin);
    });
}

}  // namespace fz
