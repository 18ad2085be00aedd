// fz_device.hpp -- device helpers shared by the compression and
// decompression kernels of libfzmi (wave64 cross-lane moves, the in-register
// 16x16 bit transpose used for the bitshuffle, loaders).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fz_format.hpp"

namespace fz {

// raw buffer resources: dword 3 of the descriptor (gfx9 data format 32); a
// load at an offset of num_records bytes or more returns 0
constexpr int kBufferFlags = 0x00020000;
typedef uint32_t fz_u32x4 __attribute__((ext_vector_type(4)));
typedef float fz_f32x4 __attribute__((ext_vector_type(4)));
typedef double fz_f64x2 __attribute__((ext_vector_type(2)));

// cache policy of a buffer access: nontemporal (the nt bit).  Used where a
// kernel streams data it never touches again -- the reconstructed field,
// the range pass over the input -- so that the lines do not displace what
// the next kernel reads.  fp32 stores use it only where every instruction fills
// whole 128-byte lines, as partial lines lose the merging in the L2; which
// outputs are streamed, and both sides measured: stream_stores.
constexpr int kCacheStream = 2;
// lane l receives lane l-1's value (DPP wave_shr:1).  Lane 0 receives an
// unspecified value: the compiler may leave the DPP destination of a lane
// without a source uninitialized, so callers mask it.
__device__ __forceinline__ int shift_up1_raw(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, false);
}
// the same with 0 on lane 0 (a following `&` takes the shift in as its operand)
__device__ __forceinline__ uint32_t shift_up1_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
}

// value of `v` held by lane - SH within the same row of 16 lanes (0 for the
// first SH lanes of a row)
template <int SH>
__device__ __forceinline__ int row_shr(int v)
{
    static_assert(SH >= 1 && SH <= 15, "row shift");
    return __builtin_amdgcn_update_dpp(0, v, 0x110 + SH, 0xf, 0xf, true);
}

// value of `v` held by lane (i + 8) mod 16 of the same 16-lane row
__device__ __forceinline__ int row_ror8(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false);
}

// Exclusive prefix sum of `v` over the 8 lanes with the same lane & 7, in
// the order of lane >> 3 (lanes 8 apart).  Within a 16-lane row the two
// halves are paired by DPP; the rows' totals are combined with the lane
// swaps (with both operands x, permlane16_swap gives the rows (x0, x0, x2,
// x2) and (x1, x1, x3, x3), permlane32_swap gives (x0, x1, x0, x1)).
__device__ __forceinline__ int excl_scan_stride8(int v, int lane)
{
    const int s1 = v + row_shr<8>(v);                   // upper half: its pair's inclusive sum
    const int r8 = row_ror8(s1);                         // on every lane: a lane shift under a branch
    const int u = (lane & 8) ? s1 : r8;                  // would read inactive lanes; the row's total
    const auto p = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const int a = (int)p[0];                             // rows: R0, R0, R2, R2
    const int c = a + (int)p[1];                         // rows: R0+R1, R0+R1, R2+R3, R2+R3
    const auto q = __builtin_amdgcn_permlane32_swap((uint32_t)c, (uint32_t)c, false, false);
    const int row = lane >> 4;
    int o = (row & 1) ? a : 0;                           // rows 1, 3: R0, R2
    o += (row & 2) ? (int)q[0] : 0;                      // rows 2, 3: + R0+R1
    return o + s1 - v;
}

// value of `v` held by lane `src` (any lane; indices wrap modulo 64)
__device__ __forceinline__ int lane_value(int v, int src)
{
    return __builtin_amdgcn_ds_bpermute(src << 2, v);
}

// v of lane `to` (a constant) set to a uniform value.  The intrinsic by its
// name, as clang has no builtin for it (inline assembly would miss the wait
// states between a compare that wrote the value and this read of it).
extern "C" __device__ uint32_t fz_writelane(uint32_t value, uint32_t to, uint32_t v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ void set_lane(uint32_t& v, int to, uint32_t value)
{
    v = fz_writelane(value, (uint32_t)to, v);
}

__device__ __forceinline__ uint32_t mbcnt(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// inclusive prefix sum over the 64 lanes: within each row of 16 by DPP row
// shifts, then the last lane of the row before (rows 1 and 3) and of lane 31
// (rows 2 and 3) broadcast into the next rows
__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += row_shr<1>(v);
    v += row_shr<2>(v);
    v += row_shr<4>(v);
    v += row_shr<8>(v);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Prequantization (Sec. 2.3): q = rint(x * inv), fp32 multiply then round
// half to even.  `acc` collects max(|p|) as shifted bits so that one compare
// per step detects NaN/Inf or |p| >= 2^31.
__device__ __forceinline__ int prequant(float v, float inv, uint32_t& acc)
{
    float p = v * inv;
    acc = max(acc, __float_as_uint(p) << 1);
    return (int)__builtin_rintf(p);
}

__device__ __forceinline__ uint32_t absu(int d) { return d < 0 ? 0u - (uint32_t)d : (uint32_t)d; }

// how k_compress turns its input words into the integers q: fp32 values on
// the grid 2eb (Sec. 2.3), fp32 values through the point-wise relative
// transform, or words that already hold q (fp64 input, prequantized by a
// pass of its own)
constexpr int kQuantGrid = 0, kQuantPw = 1, kQuantInt = 2;

// The quantizer a stream records.  step == 0: the 2eb grid of the ABS and REL
// modes, q = rint(x * inv).  step > 0: the point-wise relative mode, where
// the data's logarithmic transform is the float's bit pattern b (exponent and
// mantissa, a piecewise-linear log2 exact in integers) and q = sign(x) *
// floor((b + floor(step / 2)) / step).  inv is 0 in that mode, so x * inv
// flags exactly the non-finite inputs.
struct Quant {
    float inv;
    uint32_t step;
    uint32_t magic;  // floor(2^32 / step): the division by step as a multiply-high
};

__device__ __forceinline__ Quant quant_of(const uint8_t* hdr)
{
    Quant z;
    z.inv = *reinterpret_cast<const float*>(hdr + kOffInv);
    const bool pw = hdr[kOffEbMode] == 2;
    z.step = pw ? (uint32_t)*reinterpret_cast<const float*>(hdr + kOffEbx2) : 0u;
    z.magic = pw ? (uint32_t)(0x100000000ull / (uint64_t)z.step) : 0u;
    return z;
}

// q of the point-wise relative mode.  n < 2^32, so the multiply-high estimate
// is floor(n / step) or one less, and one compare corrects it (Granlund and
// Montgomery's division by an invariant integer).
__device__ __forceinline__ int pw_quant(float x, const Quant& z)
{
    const uint32_t bits = __float_as_uint(x);
    const uint32_t n = (bits & 0x7FFFFFFFu) + (z.step >> 1);
    uint32_t a = __umulhi(n, z.magic);
    a += (n - a * z.step >= z.step) ? 1u : 0u;
    return (bits >> 31) ? -(int)a : (int)a;
}

// its inverse: the float with the sign of q and the bits min(|q| * step, the
// largest finite float)
__device__ __forceinline__ float pw_dequant(int q, uint32_t step)
{
    const uint64_t m = (uint64_t)absu(q) * step;
    const uint32_t b = m > 0x7F7FFFFFull ? 0x7F7FFFFFu : (uint32_t)m;
    return __uint_as_float(b | (q < 0 ? 0x80000000u : 0u));
}

typedef short fz_short2 __attribute__((ext_vector_type(2)));

// Sign-magnitude 16-bit codes of packed 16-bit deltas, in place (Sec. 3.2:
// sign in the MSB, magnitude below); -32768 becomes the escape code 0x8000.
__device__ __forceinline__ void sign_magnitude(uint32_t (&P)[16])
{
#pragma unroll
    for (int i = 0; i < 16; i++) {
        const fz_short2 x = __builtin_bit_cast(fz_short2, P[i]);
        const fz_short2 mag = __builtin_elementwise_max(x, (fz_short2)0 - x);
        P[i] = __builtin_bit_cast(uint32_t, mag) | (P[i] & 0x80008000u);
    }
}
constexpr uint32_t kEscapeLimit = 65534u;  // d + 32767 above this (as unsigned): an escape

// In-register bit transpose: on entry P[i] holds code i (low half) and code
// i+16 (high half); on exit P[b] bit m = bit b of code m (Sec. 3.3's
// bitshuffle of 32 codes).  The transform is its own inverse.
// One bit-field insert per result, named in assembly: from the masked form
// the compiler merges the masks of neighbouring stages into up to three ands
// and ors per result (measured: about 190 instead of 112 instructions per
// transpose).
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t on, uint32_t off)
{
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(mask), "v"(on), "v"(off));
    return r;
}
template <int S, uint32_t M>
__device__ __forceinline__ void tswap(uint32_t& a, uint32_t& b)
{
    const uint32_t na = bfi(M, a, b << S);
    const uint32_t nb = bfi(M, a >> S, b);
    a = na;
    b = nb;
}

// the byte stage of the transpose: two byte permutes per pair of words
__device__ __forceinline__ void tswap8(uint32_t& a, uint32_t& b)
{
    const uint32_t na = __builtin_amdgcn_perm(b, a, 0x06020400u);  // a0 b0 a2 b2
    const uint32_t nb = __builtin_amdgcn_perm(b, a, 0x07030501u);  // a1 b1 a3 b3
    a = na;
    b = nb;
}

__device__ __forceinline__ void transpose16(uint32_t (&P)[16])
{
#pragma unroll
    for (int i = 0; i < 8; i++) tswap8(P[i], P[i + 8]);
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = (j & 3) | ((j & 4) << 1);
        tswap<4, 0x0F0F0F0Fu>(P[i], P[i + 4]);
    }
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = (j & 1) | ((j & 6) << 1);
        tswap<2, 0x33333333u>(P[i], P[i + 2]);
    }
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int i = 2 * j;
        tswap<1, 0x55555555u>(P[i], P[i + 1]);
    }
}

// order-preserving unsigned key of a float (-0 counts as +0)
__device__ __forceinline__ uint32_t float_key(float v)
{
    uint32_t b = __float_as_uint(v == 0.0f ? 0.0f : v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// a value that is the same on every lane, in scalar registers
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// A uniform pointer read from memory (a batch's job), as one to global memory
// in scalar registers: the compiler cannot see either by itself and would use
// flat accesses, per lane.
template <typename T>
__device__ __forceinline__ T* as_global(T* p)
{
    return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)uniform64((int64_t)(uintptr_t)p);
}

// Memory that a kernel only reads, at a uniform address: read with scalar
// loads, whatever else the kernel writes.
template <typename T>
using ConstMem = const __attribute__((address_space(4))) T;
template <typename T>
__device__ __forceinline__ ConstMem<T>* const_mem(const void* p)
{
    return (ConstMem<T>*)(uintptr_t)uniform64((int64_t)(uintptr_t)p);
}

__device__ __forceinline__ uint32_t div_by(uint32_t n, const Divisor& d)
{
    return (uint32_t)(((uint64_t)n * d.mul) >> d.shift);
}

__device__ __forceinline__ void chunk_box(const Geom& g, int64_t c, int64_t org[3], int64_t ext[3])
{
    const uint32_t cc = (uint32_t)c, q2 = div_by(cc, g.div[1]), q0 = div_by(q2, g.div[0]);
    const int64_t ci[3] = {q0, q2 - q0 * (uint32_t)g.grid[1], cc - q2 * (uint32_t)g.grid[2]};
#pragma unroll
    for (int i = 0; i < 3; i++) {
        org[i] = ci[i] * g.box[i];
        // in 32-bit compares, which the scalar unit has (it has no 64-bit ones)
        const uint64_t e = (uint64_t)(g.n[i] - org[i]);
        const uint32_t lo = (uint32_t)e, hi = (uint32_t)(e >> 32), box = (uint32_t)g.box[i];
        ext[i] = hi == 0u && lo < box ? lo : box;
    }
}

// The chunk of block b of n in kernels that read or write a field in place:
// runs of kXcdRun chunks, side by side along the contiguous axis, go to one
// XCD (blocks go round the 8 XCDs in turn), so that its L2 joins the lines that
// neighbouring chunks share, while the blocks in flight still cover one stretch
// of the field.  Measured, blocks in chunk order / runs of 8: 100x500x500
// decompression 33.7 / 31.8 us, the same in double with its compression 201 /
// 193 us, its field-global round trip 220 / 200 us (runs
// of 4: 207, one run per XCD: 213 and 2 to 4 % slower than chunk order at whole lines).
constexpr uint32_t kXcds = 8, kXcdRun = 8;
__device__ __forceinline__ int64_t xcd_order(uint32_t b, int64_t n)
{
    constexpr uint32_t window = kXcds * kXcdRun;
    if (b >= ((uint32_t)n & ~(window - 1))) return b;
    return (b & ~(window - 1)) + kXcdRun * (b & (kXcds - 1)) + ((b / kXcds) & (kXcdRun - 1));
}

// stored layers of a chunk whose extent along the step dimension is e
__device__ __forceinline__ int layers_of(int rank, int64_t e)
{
    const int64_t per = rank == 3 ? 4 : rank == 2 ? 8 : 8192;
    return (int)((e + per - 1) / per);
}

__device__ __forceinline__ int clampi(int64_t v, int lo, int hi)
{
    return v < lo ? lo : (v > hi ? hi : (int)v);
}

}  // namespace fz
