// fz_compress_dev.hpp -- device code of the compression pipeline, shared by
// the per-field kernels (fz_compress.hip) and the batched ones (fz_batch.hip).
//
// The path of one chunk: a workgroup of 4 waves, wave k on layer k (4 steps),
// one lane per 32-code patch.  Per step a lane prequantizes its 32 fp32 values
// (Sec. 2.3) and takes the Lorenzo difference on the integers (Sec. 2.3 / 3.2)
// along the sweep dimension against the previous step in its registers.  What
// follows runs packed, two 16-bit values per instruction: the rest of the
// difference (neighbours come from adjacent lanes), the sign-magnitude codes
// (Sec. 3.2) and the in-register bit transpose (the bitshuffle of Sec. 3.3).
// A lane keeps the plane words of its 4 steps: a brick (one bit plane of a
// patch over the layer) is 4 registers of one lane, so no exchange is needed.
// Ballots give the bit flags of the zero-block encoder (Sec. 3.4), and the
// nonzero bricks are compacted into LDS, which holds the chunk's whole
// payload.  One chunk later, when a look-back over the published chunk sizes
// (the device-wide prefix sum of Sec. 3.4) has given the chunk its offset, the
// payload is copied there.  A layer whose differences along the sweep do not
// fit the packed arithmetic is coded again out of line in 32 bits, where
// deltas that need escapes are logged.
//
// What bounds it: memory at large fields (512^3 ABS: 134 us, 4.6 TB/s of reads
// and stores where a copy reaches 5.1; 168 us in the form before, where each
// of 4 waves coded one layer with the plane words in LDS and the staged payload
// in a global slot), else the chain of one chunk through a workgroup.  256
// registers a lane (2 waves per SIMD) hold a layer's 64 plane words and the
// next step's loads; 8 waves of half a layer each at 128 registers measured
// 169 us with the same staging.
#pragma once
#include <hip/hip_runtime.h>

#include "fz_device.hpp"
#include "fz_format.hpp"
#include "fz_kernels.hpp"

namespace fz {

// ------------------------------------------------------------- workgroup
// A chunk's payload is staged in LDS up to this size (60 KB; the whole
// workgroup stays below half of a CU's 160 KB).  A larger one, more than 15
// bits per value, is placed at once.
constexpr uint32_t kPayUnits = 3840;

// Workgroup-shared state of a compression workgroup (one chunk at a time).
struct CompressLds {
    uint4 pay[kPayUnits];  // the staged chunk's payload: bricks, then escape pairs
    uint4 tile[kLayers][256];  // per wave: half a step on its way from rows to patches
    uint32_t arrived;  // waves whose layer of the current chunk is done
    // the workgroup's first ticket, in a word of its own: thread 0 leaves the
    // next one without a barrier after the other waves' read of this one
    uint64_t first;
    uint64_t ticket;   // the next ticket
    uint64_t excl;     // offset of the chunk being placed (16-B units), from the look-back
    // status bits, and bricks and escapes of each layer, by the chunk's parity:
    // a wave may be one chunk ahead of one that still reads them
    uint32_t err[2];
    uint32_t nnz[2][kLayers], nout[2][kLayers];
    // escapes (rare): pairs logged so far, and each step's block of them
    uint32_t esc_used;
    uint32_t esc_n[kSteps], esc_at[kSteps];
};
typedef __attribute__((address_space(3))) CompressLds LdsState;
// The workgroup's slot of the scratch, used by layers that are coded out of
// line: the words of their bricks (16 KB per layer; plane, step and lane, so that
// each store and load moves whole lines), then the chunk's escape pairs.
constexpr int kSlotPairs = kLayers * kPlanes * kPatches * 16;
static_assert(kSlotPairs + kChunkOutlierCap * 8 == kStageSlotBytes, "slot layout");

// ---------------------------------------------------------- one step's codes
// In the packed path the integers of the 2eb grid carry this bias (the bits of
// 1.5 * 2^23 as a float): rounding to the nearest integer is then one float
// add, whose result bits are bias + q, for products below 2^22 (larger ones
// are coded out of line).  The difference along the sweep dimension cancels it.
constexpr float kRoundMagic = 12582912.0f;
constexpr int kRoundBias = 0x4B400000;
constexpr float kRoundLimit = 4194304.0f;

// Largest difference along the sweep dimension whose codes the packed 16-bit
// arithmetic gets right: the rest of the predictor adds 4 such terms in 3-D
// and 2 in 2-D, and a code holds 32767.
template <int RANK>
__device__ __forceinline__ constexpr int packed_limit() { return RANK == 3 ? 8191 : RANK == 2 ? 16383 : 32767; }

template <int QM>
__device__ __forceinline__ constexpr int quant_bias() { return QM == kQuantGrid ? kRoundBias : 0; }

// prequantize 32 values; `facc` tracks max |p| with NaN propagating
// (v_maximum3_f32), so one compare finds NaN, Inf or an overflowing product.
// BIASED: the packed path's integers; else plain ones, for any product.
template <int QM, bool BIASED>
__device__ __forceinline__ void prequant32(const float (&v)[32], const Quant& z, float& facc, int (&q)[32])
{
    if constexpr (QM == kQuantInt) {  // the values are already the integers q (fp64 input)
#pragma unroll
        for (int i = 0; i < 32; i++) q[i] = __float_as_int(v[i]);
        return;
    }
    const float inv = z.inv;  // 0 in the point-wise mode: x * inv flags NaN/Inf there
#pragma unroll
    for (int i = 0; i < 32; i += 2) {
        const float p0 = v[i] * inv, p1 = v[i + 1] * inv;
        // one instruction per two values (from the nested form the compiler
        // builds a tree of half as many values per instruction)
        asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(facc) : "v"(p0), "v"(p1));
        if constexpr (QM == kQuantPw) {
            q[i] = pw_quant(v[i], z);
            q[i + 1] = pw_quant(v[i + 1], z);
        } else if constexpr (BIASED) {
            q[i] = __float_as_int(p0 + kRoundMagic);
            q[i + 1] = __float_as_int(p1 + kRoundMagic);
        } else {
            q[i] = (int)__builtin_rintf(p0);
            q[i + 1] = (int)__builtin_rintf(p1);
        }
    }
}

__device__ __forceinline__ bool escapes(int d) { return (uint32_t)d + 32767u > kEscapeLimit; }

// The escapes of a step (deltas that do not fit in 15 bits, of cells inside
// the field: keep): their (code index, delta) pairs go to a block of the
// slot's list, in code-index order (lane-major, then cell; past the chunk's
// allowance only counted), and the deltas are replaced by -32768, whose code
// is the escape 0x8000.  Returns their number.
__device__ __forceinline__ uint32_t log_escapes(int (&d)[32], uint32_t keep, int s, int lane, LdsState* S, uint2* pairs)
{
    uint32_t emask = 0;
#pragma unroll
    for (int i = 0; i < 32; i++) emask |= (escapes(d[i]) ? 1u : 0u) << i;
    emask &= keep;
    const int cnt = __popc(emask);
    const int incl = wave_incl_scan(cnt);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(incl, 63);
    uint32_t at = 0;
    if (lane == 0) {
        at = __hip_atomic_fetch_add(&S->esc_used, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        S->esc_at[s] = at;
        S->esc_n[s] = total;
    }
    uint32_t pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)(incl - cnt);
    const uint32_t n0 = (uint32_t)s * kStepCodes + (uint32_t)lane * kPatchCodes;
#pragma unroll
    for (int i = 0; i < 32; i++) {
        if ((emask >> i) & 1u) {
            if (pos < (uint32_t)kChunkOutlierCap) pairs[pos] = make_uint2(n0 + i, (uint32_t)d[i]);
            pos++;
            d[i] = -32768;
        }
    }
    return total;
}

// ------------------------------------------------------------------ loaders
// Loads go through a buffer resource whose base is the (uniform) first value
// of the step: lane offsets are 32-bit and the row offsets uniform, so no
// 64-bit per-lane address is held in registers.  The resource's range ends at
// the field's last value, so a load past it (its uniform offset counted)
// returns 0 without touching memory.  A chunk cut by the field's edge
// is loaded exactly like an interior one: its cells outside the field read 0
// (past the end) or values of other chunks (the rest of a row, the next
// rows), and their deltas are set to 0 afterwards (mask_outside), while the
// delta of a cell inside the field only looks at cells inside it.
// (on = false: a range of 0, every load returns 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t step_rsrc(const float* __restrict__ x, const Geom& g,
                                                           const float* base, bool on = true)
{
    // (uniform; in 32-bit compares, which the scalar unit has)
    const int64_t left = 4 * (g.n[0] * g.n[1] * g.n[2] - (base - x));
    const int hi = (int)(left >> 32);
    const int range = !on || hi < 0 ? 0 : hi > 0 ? -1 : (int)(uint32_t)left;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, range, kBufferFlags);
}

// CNT values from voff + soff; VEC4: in 16-byte loads, which need only 4-byte
// alignment and are range-checked per dword (the host's vec_loads); else one
// load per value.  NT: a nontemporal (streaming) load, for values this chunk
// reads only once.
template <int CNT, bool VEC4, bool NT = false>
__device__ __forceinline__ void load_run(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float* v)
{
    if (VEC4) {
#pragma unroll
        for (int j = 0; j < CNT / 4; j++) {
            const fz_u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 16u * j, soff, NT ? kCacheStream : 0);
            v[4 * j] = __uint_as_float(t.x); v[4 * j + 1] = __uint_as_float(t.y);
            v[4 * j + 2] = __uint_as_float(t.z); v[4 * j + 3] = __uint_as_float(t.w);
        }
    } else {
#pragma unroll
        for (int j = 0; j < CNT; j++)
            v[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff + 4u * j, soff, NT ? kCacheStream : 0));
    }
}

// Per-chunk, per-lane geometry.  step_base() is uniform (scalar); lane
// offsets inside a step are 32-bit.
struct Lane {
    int64_t org[3], ext[3];
    int live;      // steps of the chunk that hold cells of the field
    bool edge;
    uint32_t off;  // lane offset of its first value inside a step
};

template <int RANK>
__device__ __forceinline__ Lane lane_geo(const Geom& g, int64_t c, int lane)
{
    Lane l;
    chunk_box(g, c, l.org, l.ext);
    const int e0 = (int)l.ext[0];
    l.live = RANK == 3 ? e0 : RANK == 2 ? (e0 + 1) / 2 : (e0 + kStepCodes - 1) / kStepCodes;
    l.edge = false;
#pragma unroll
    for (int i = 0; i < 3; i++) l.edge |= l.ext[i] < g.box[i];
    if (RANK == 3) {
        const int py = lane & 7, px = lane >> 3;
        l.off = (uint32_t)(4 * py * g.n[2] + 8 * px);
    } else if (RANK == 2) {
        l.off = (uint32_t)(16 * lane);
    } else {
        l.off = (uint32_t)(kPatchCodes * lane);
    }
    return l;
}

// first value of step s (3-D: plane s; 2-D: row 2s; 1-D: value 2048 s) of the chunk
template <int RANK>
__device__ __forceinline__ const float* step_base(const float* __restrict__ x, const Geom& g, const Lane& l, int64_t s)
{
    if (RANK == 3) return x + ((l.org[0] + s) * g.n[1] + l.org[1]) * g.n[2] + l.org[2];
    if (RANK == 2) return x + (l.org[0] + 2 * s) * g.n[1] + l.org[1];
    return x + l.org[0] + (int64_t)kStepCodes * s;
}

// The lane's own 32 values of step s, patch by patch (the layers coded out of line).
template <int RANK, bool VEC4>
__device__ __forceinline__ void load_patch(const float* __restrict__ x, const Geom& g, const Lane& l, int64_t s, float (&v)[32])
{
    const __amdgpu_buffer_rsrc_t rs = step_rsrc(x, g, step_base<RANK>(x, g, l, s));
    if (RANK == 3) {
        const int64_t nx = g.n[2];
#pragma unroll
        for (int r = 0; r < 4; r++) load_run<8, VEC4>(rs, 4u * l.off, (uint32_t)(4 * r * nx), v + 8 * r);
    } else if (RANK == 2) {
        const int64_t nx = g.n[1];
#pragma unroll
        for (int r = 0; r < 2; r++) load_run<16, VEC4>(rs, 4u * l.off, (uint32_t)(4 * r * nx), v + 16 * r);
    } else {
        load_run<32, VEC4>(rs, 4u * l.off, 0u, v);
    }
}

// Step s as rows: each load covers whole lines of memory (a lane's own patch
// would give each load 16-byte pieces 32, 64 or 128 bytes apart, every line
// touched by several loads).  Loads 0 .. 3 and 4 .. 7 are two halves that
// rows_to_patches exchanges one after the other:
//   3-D: load j covers 4 rows of 64 values: rows 4 py + 0, 1 (first half) or
//   + 2, 3 of the patch rows py = 2j, 2j + 1, a row's 16 pieces exchanged by
//   XOR with py;
//   2-D: 256 columns of row 0 (first half) or 1;
//   1-D: the first or last 16 values of 16 patches.
template <int RANK, bool VEC4, bool NT>
__device__ __forceinline__ void load_rows_as(const float* __restrict__ x, const Geom& g, const Lane& l, int64_t s, bool on,
                                             int lane, float (&v)[32])
{
    const __amdgpu_buffer_rsrc_t rs = step_rsrc(x, g, step_base<RANK>(x, g, l, s), on);
    const uint32_t nx = (uint32_t)g.n[RANK - 1];  // (1-D: not used)
    if (RANK == 3) {
        const uint32_t row = 4u * (uint32_t)(lane >> 5) + (uint32_t)((lane >> 4) & 1);
        const uint32_t piece = (uint32_t)((lane & 15) ^ (lane >> 5));
#pragma unroll
        for (int j = 0; j < 8; j++)
            load_run<4, VEC4, NT>(rs, 4u * row * nx + 16u * (piece ^ (2u * (j & 3))), 4u * (8u * (j & 3) + 2u * (j >> 2)) * nx, v + 4 * j);
    } else if (RANK == 2) {
#pragma unroll
        for (int j = 0; j < 8; j++)
            load_run<4, VEC4, NT>(rs, 16u * (uint32_t)lane + 1024u * (j & 3), j < 4 ? 0u : 4u * nx, v + 4 * j);
    } else {
        const uint32_t at = 128u * (uint32_t)(lane >> 2) + 16u * (uint32_t)(lane & 3);
#pragma unroll
        for (int j = 0; j < 8; j++)
            load_run<4, VEC4, NT>(rs, at + 2048u * (j & 3) + 64u * (j >> 2), 0u, v + 4 * j);
    }
}

// A step's values from the rows that load_rows left in v to the lanes'
// patches, in place, through the wave's tile in two halves.  The tile's places
// are exchanged by XOR so that both directions spread over the banks.  One
// wave's LDS operations execute in order, so nothing is waited for in between;
// the compiler must only keep them in this order.
template <int RANK>
__device__ __forceinline__ void rows_to_patches(float (&v)[32], int lane, uint4* tile)
{
    const int py = lane & 7, px = lane >> 3;
#pragma unroll
    for (int hf = 0; hf < 2; hf++) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float* r = v + 16 * hf + 4 * i;
            tile[64 * i + (RANK == 3 ? lane : lane ^ (lane >> 4))] =
                make_uint4(__float_as_uint(r[0]), __float_as_uint(r[1]), __float_as_uint(r[2]), __float_as_uint(r[3]));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint4 t = tile[RANK == 3 ? 32 * py + 16 * (i >> 1) + ((2 * px + (i & 1)) ^ py)
                                           : 4 * lane + (i ^ ((lane >> 2) & 3))];
            float* w = v + 16 * hf + 4 * i;
            w[0] = __uint_as_float(t.x); w[1] = __uint_as_float(t.y);
            w[2] = __uint_as_float(t.z); w[3] = __uint_as_float(t.w);
        }
        asm volatile("" ::: "memory");
    }
}

// Step s as rows, nontemporal except for a step that is read again in the same
// iteration (cached: the top step of a layer, 3-D and 2-D, which is the next
// layer's halo) and must be found in the cache, and except in 1-D, where two
// loads share a line (measured, everything cached against this rule: 512^3
// ABS 135.2 -> 133.6 us, 112x512x512 44.6 -> 41.6 us, 8192^2 75.2 -> 73.9 us; 1-D of
// 2^26 values nontemporal 85.3, cached 78.8 us).
template <int RANK, bool VEC4>
__device__ __forceinline__ void load_rows(const float* __restrict__ x, const Geom& g, const Lane& l, int64_t s, bool on,
                                          bool cached, int lane, float (&v)[32])
{
    if (RANK == 1 || cached) load_rows_as<RANK, VEC4, false>(x, g, l, s, on, lane, v);
    else load_rows_as<RANK, VEC4, true>(x, g, l, s, on, lane, v);
}

// Whether layer k of a chunk is swept downwards (odd layers, 2-D and 3-D).
// An odd layer's halo is the top step of the layer below it, and an even
// layer's halo the top step of an odd layer; in this order each halo step is
// loaded in the same phase as by the wave that owns it, so the second load is
// served by the cache.
template <int RANK>
__device__ __forceinline__ bool swept_down(int k)
{
    return RANK >= 2 && (k & 1);
}

// Load the first two steps that layer k of a chunk uses ahead of time: the
// halo and the first step (upwards), or the top two steps (downwards).
// Branch-free: both loads are always issued, and one that has nothing to
// read (no next chunk: on; no layer k, the halo of layer 0 or of a 1-D layer) gets a range of 0
// and returns zeros.  A branch here would merge the loads' uniform row
// offsets at its join, where the compiler keeps them in vector registers and
// then has to build a loop around every later load that uses them.  The
// halo or top step is the one another wave reads again, the other one is
// streamed.
template <int RANK, bool VEC4>
__device__ __forceinline__ void prefetch(const float* __restrict__ x, const Geom& g, const Lane& l, int k,
                                         int lane, float (&h)[32], float (&v)[32], bool on = true)
{
    const bool live = on && 4 * k < l.live, dn = swept_down<RANK>(k);
    if (RANK == 1) {  // no halo step (a 1-D layer's halo is one value)
#pragma unroll
        for (int i = 0; i < 32; i++) h[i] = 0.0f;
    } else {
        load_rows<RANK, VEC4>(x, g, l, dn ? 4 * k + 3 : 4 * k - 1, live && (dn || k > 0), true, lane, h);
    }
    load_rows<RANK, VEC4>(x, g, l, dn ? 4 * k + 2 : 4 * k, live, false, lane, v);
}

// The lane's cells of step s inside the field, one bit per value of d (all
// set in a chunk not cut by the field's edge): 3-D, its rows r < ev and
// columns c < eh of a plane inside the field; 2-D, its columns c < eh of the
// step's rows inside the field; 1-D, its values inside the field.
template <int RANK>
__device__ __forceinline__ uint32_t keep_bits(const Lane& l, int64_t s, int lane)
{
    if (RANK == 3) {
        const int ev = clampi(l.ext[1] - 4 * (lane & 7), 0, 4), eh = clampi(l.ext[2] - 8 * (lane >> 3), 0, 8);
        const uint32_t cells = (uint32_t)((1ull << (8 * ev)) - 1ull) & (((1u << eh) - 1u) * 0x01010101u);
        return s < l.ext[0] ? cells : 0u;
    } else if (RANK == 2) {
        const uint32_t cols = (uint32_t)((1ull << clampi(l.ext[1] - 16 * lane, 0, 16)) - 1ull);
        return (2 * s < l.ext[0] ? cols : 0u) | (2 * s + 1 < l.ext[0] ? cols << 16 : 0u);
    } else {
        const int valid = clampi(l.ext[0] - ((int64_t)kStepCodes * s + l.off), 0, 32);
        return (uint32_t)((1ull << valid) - 1ull);
    }
}

// ------------------------------------------------------------ one layer
// In-plane part of the Lorenzo difference after the difference along the
// sweep dimension, on packed values: A[i] holds cells i (low half) and i + 16.
// 3-D: A[c] are rows 0 and 2, A[8 + c] rows 1 and 3; Dy, then Dx.
__device__ __forceinline__ fz_short2 as_short2(uint32_t v) { return __builtin_bit_cast(fz_short2, v); }
__device__ __forceinline__ uint32_t sub2(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, as_short2(a) - as_short2(b)); }
__device__ __forceinline__ void inplane3(uint32_t (&A)[16], int lane)
{
    const uint32_t below = (lane & 7) == 0 ? 0u : ~0u;  // whether a patch row comes before
    const int px = lane >> 3;
    uint32_t left[2];
#pragma unroll
    for (int c = 7; c >= 0; c--) {
        // rows 0 and 2 take row 3 of lane-1 (0 for py == 0; mask and shift are one instruction) and row 1
        const uint32_t up = shift_up1_zero(A[8 + c]) & below;
        const uint32_t prev = __builtin_amdgcn_alignbit(A[8 + c], up, 16);
        A[8 + c] = sub2(A[8 + c], A[c]);
        A[c] = sub2(A[c], prev);
        if (c == 7) {  // column 0 takes column 7 of lane-8 (0 for px == 0), asked for early
            left[0] = (uint32_t)lane_value((int)A[7], lane - 8);
            left[1] = (uint32_t)lane_value((int)A[15], lane - 8);
        }
    }
#pragma unroll
    for (int r = 0; r < 2; r++) {
#pragma unroll
        for (int c = 7; c > 0; c--) A[8 * r + c] = sub2(A[8 * r + c], A[8 * r + c - 1]);
        A[8 * r] = sub2(A[8 * r], px == 0 ? 0u : left[r]);
    }
}

// 2-D: A[c] holds column c of the step's two rows; Dx.
__device__ __forceinline__ void inplane2(uint32_t (&A)[16], int lane)
{
    const uint32_t left = shift_up1_zero(A[15]);  // column 0 takes column 15 of lane-1 (0 at lane 0)
#pragma unroll
    for (int c = 15; c > 0; c--) A[c] = sub2(A[c], A[c - 1]);
    A[0] = sub2(A[0], left);
}

// Whether some delta of a step may be an escape, from the differences along the
// sweep dimension in 256ths (H, packed, below 2^12 in magnitude; changed): the
// in-plane part of those is the delta in 256ths, off by less than 2.  keep: the
// cells that count.
template <int RANK>
__device__ __forceinline__ bool plane_escapes(uint32_t (&H)[16], bool edge, uint32_t keep, int lane)
{
    if (RANK == 3) inplane3(H, lane);
    else inplane2(H, lane);
    if (edge) {
#pragma unroll
        for (int i = 0; i < 16; i++)
            H[i] &= ((keep >> i) & 1u ? 0xFFFFu : 0u) | ((keep >> (i + 16)) & 1u ? 0xFFFF0000u : 0u);
    }
    fz_short2 mx = as_short2(H[0]), mn = mx;
#pragma unroll
    for (int i = 1; i < 16; i++) {
        mx = __builtin_elementwise_max(mx, as_short2(H[i]));
        mn = __builtin_elementwise_min(mn, as_short2(H[i]));
    }
    return __ballot(max(mx.x, mx.y) > 126 || min(mn.x, mn.y) < -126) != 0;
}

// One step: its difference along the sweep dimension (a; 1-D: its deltas) ->
// bit planes P.  keep: the cells inside the field (the codes of the others
// are cleared: bit i of each plane word is code i).  Returns whether some delta
// may be an escape.  The packed arithmetic is exact modulo 2^16, so its codes are
// right whenever none is; differences within packed_limit cannot give one, and
// on the 2eb grid with every |q| small (facc) none lies past it.  Otherwise the
// deltas are formed in 256ths and looked at (a field that varies by more than
// the limit within a plane, 320x192x192 ABS: 42.9 us with every such layer
// coded out of line, 28.2 so; 33.5 before any layer was packed).
// head: the step holds the chunk's first cell, whose delta is `first`.
template <int RANK, int QM>
__device__ __forceinline__ bool step_planes(const int (&a)[32], bool edge, uint32_t keep, float facc, int lane,
                                            bool head, int first, uint32_t (&P)[16])
{
    constexpr int lim = packed_limit<RANK>();
    bool wide = false;
    if (QM != kQuantGrid || __ballot(!(facc < (float)(lim / 2))) != 0) {
        int mn = 0, mx = 0;
#pragma unroll
        for (int i = 0; i < 32; i += 2) {
            mx = max(mx, max(a[i], a[i + 1]));
            mn = min(mn, min(a[i], a[i + 1]));
        }
        wide = __ballot(mx > lim || mn < -lim) != 0;
        if (RANK >= 2 && wide && __ballot(mx >= (1 << 20) || mn < -(1 << 20)) == 0) {
            uint32_t H[16];
#pragma unroll
            for (int i = 0; i < 16; i++) H[i] = __builtin_amdgcn_perm((uint32_t)a[i + 16], (uint32_t)a[i], 0x06050201u);
            wide = plane_escapes<RANK>(H, edge, keep, lane);
        }
    }
#pragma unroll
    for (int i = 0; i < 16; i++) P[i] = __builtin_amdgcn_perm((uint32_t)a[i + 16], (uint32_t)a[i], 0x05040100u);
    if (RANK == 3) inplane3(P, lane);
    else if (RANK == 2) inplane2(P, lane);
    if (head) {  // on lane 0 the cell's packed difference is 0 (see layer_fast); an escape's is -32768
        const uint32_t code = escapes(first) ? 0x8000u : (uint32_t)first & 0xFFFFu;
        P[0] |= lane == 0 ? code : 0u;
    }
    sign_magnitude(P);
    transpose16(P);
    if (edge) {
#pragma unroll
        for (int b = 0; b < 16; b++) P[b] &= keep;
    }
    return wide;
}

// Difference along the sweep dimension of a step with integers q against the
// step before it (qp).  3-D: the plane before; 2-D: row 1 of the step before,
// then row 0.
template <int RANK>
__device__ __forceinline__ void sweep_diff(const int (&q)[32], const int (&qp)[32], int (&a)[32])
{
#pragma unroll
    for (int i = 0; i < 32; i++) a[i] = q[i] - (RANK == 3 ? qp[i] : i < 16 ? qp[16 + i] : q[i - 16]);
}

// Layer k, its steps in order upwards or downwards (DOWN); `h` and `v` hold
// what prefetch loaded.  The differences of the chunk's first step are taken
// from its first cell's integer in place of the zeros before it: every other
// delta is the same (the constant cancels in it), and the first cell's, which
// is the integer itself, is put in afterwards.  So a field whose values lie far
// from 0 (|q| past the packed limit) does not send the first layer of each of
// its chunks out of line (256^3 point-wise, |q| about 60000, round trip: 85 us,
// now 70).  first: that integer (layer 0 only).  W[b][t]: the plane-b word of step 4k + t (the brick
// of this lane's patch).  Returns whether the layer has to be coded out of
// line.
template <int RANK, bool VEC4, int QM, bool DOWN>
__device__ __forceinline__ bool layer_fast(const float* __restrict__ x, const Geom& g, const Lane& l, int k, Quant inv,
                                           int lane, float (&h)[32], float (&v)[32], uint4* tile, uint32_t (&W)[kPlanes][4],
                                           float& facc, int& first)
{
    bool wide = false;
    int qp[32];     // UP: the step before the one coded; DOWN: the one coded
    int carry = 0;  // 1-D: the value before the step
    if constexpr (RANK == 1) {
        carry = QM == kQuantGrid ? kRoundBias : 0;
        if (k > 0) {
            uint32_t dummy = 0;
            const float xh = x[l.org[0] + (int64_t)kStepCodes * 4 * k - 1];
            if (QM == kQuantGrid) facc = __builtin_fabsf(xh * inv.inv);
            carry += QM == kQuantPw ? pw_quant(xh, inv) : QM == kQuantInt ? __float_as_int(xh) : prequant(xh, inv.inv, dummy);
        }
    } else if (DOWN || k > 0) {  // (layer 0 has no step before it: its first cell stands in, below)
        rows_to_patches<RANK>(h, lane, tile);
        prequant32<QM, true>(h, inv, facc, qp);
    }
#pragma unroll
    for (int it = 0; it < 4; it++) {
        const int t = DOWN ? 3 - it : it, s = 4 * k + t;
        float vn[32];
        const int sn = DOWN ? s - 2 : s + 1;  // DOWN: 4k - 1 at it = 2, the halo
        if (it < 3) load_rows<RANK, VEC4>(x, g, l, sn, true, (sn & 3) == 3, lane, vn);
        // keep the steps apart: the scheduler must not pull the next step's
        // arithmetic up to its loads, which would wait on them right away
        __builtin_amdgcn_sched_barrier(0);
        int q[32], a[32];
        rows_to_patches<RANK>(v, lane, tile);
        prequant32<QM, true>(v, inv, facc, q);
        const bool head = !DOWN && it == 0 && k == 0;
        if (head) {
            const int q0 = __builtin_amdgcn_readfirstlane(q[0]);
            first = q0 - quant_bias<QM>();
            if (RANK == 1) carry = q0;
            else {
#pragma unroll
                for (int i = RANK == 3 ? 0 : 16; i < 32; i++) qp[i] = q0;
            }
        }
        if constexpr (RANK == 1) {
            const int left = shift_up1_raw(q[31]);
            a[0] = q[0] - (lane == 0 ? carry : left);
#pragma unroll
            for (int m = 1; m < 32; m++) a[m] = q[m] - q[m - 1];
            carry = __builtin_amdgcn_readlane(q[31], 63);
        } else if constexpr (DOWN) {
            sweep_diff<RANK>(qp, q, a);
        } else {
            sweep_diff<RANK>(q, qp, a);
        }
        uint32_t P[16];
        wide |= step_planes<RANK, QM>(a, l.edge, l.edge ? keep_bits<RANK>(l, s, lane) : 0u, facc, lane, head, first, P);
#pragma unroll
        for (int b = 0; b < kPlanes; b++) W[b][t] = P[b];
#pragma unroll
        for (int i = 0; i < 32; i++) qp[i] = q[i];
        if (it < 3) {
#pragma unroll
            for (int i = 0; i < 32; i++) v[i] = vn[i];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    return wide || (QM == kQuantGrid && __ballot(!(facc < kRoundLimit)) != 0);
}

// In-plane part of the difference in 32 bits, in place (see inplane3, inplane2).
template <int RANK>
__device__ __forceinline__ void inplane_wide(int (&d)[32], int lane)
{
    if (RANK == 3) {
        const int py = lane & 7, px = lane >> 3;
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const int up = shift_up1_raw(d[24 + c]);
#pragma unroll
            for (int r = 3; r > 0; r--) d[8 * r + c] -= d[8 * (r - 1) + c];
            d[c] -= py == 0 ? 0 : up;
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int left = lane_value(d[8 * r + 7], lane - 8);
#pragma unroll
            for (int c = 7; c > 0; c--) d[8 * r + c] -= d[8 * r + c - 1];
            d[8 * r] -= px == 0 ? 0 : left;
        }
    } else if (RANK == 2) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const int left = shift_up1_raw(d[16 * r + 15]);
#pragma unroll
            for (int c = 15; c > 0; c--) d[16 * r + c] -= d[16 * r + c - 1];
            d[16 * r] -= lane == 0 ? 0 : left;
        }
    }
}

// Layer k of chunk c in 32-bit arithmetic, with escapes: its bricks go to the
// workgroup's slot, its escapes to the slot's list (log_escapes).  Returns
// their number.  It loads its own inputs and reads the geometry from its copy
// in the scratch, so that little crosses the call; a real call, as its
// registers would push the common path into spills.
template <int RANK, bool VEC4, int QM>
__device__ __noinline__ uint32_t layer_wide(const float* __restrict__ x, const uint8_t* scr, int64_t c, int k, Quant inv,
                                            int lane, uint8_t* slot, LdsState* S)
{
    const Geom g = *reinterpret_cast<const Geom*>(scr + kScratchGeomOff);
    const Lane l = lane_geo<RANK>(g, c, lane);
    uint2* pairs = reinterpret_cast<uint2*>(slot + kSlotPairs);
    uint32_t* word = reinterpret_cast<uint32_t*>(slot) + 4 * k * kPlanes * kPatches + lane;
    uint32_t total = 0;
    float facc = 0.0f, v[32];
    int qp[32], carry = 0;
#pragma unroll
    for (int i = 0; i < 32; i++) qp[i] = 0;
    if (k > 0) {
        if (RANK == 1) {
            uint32_t dummy = 0;
            const float xh = x[l.org[0] + (int64_t)kStepCodes * 4 * k - 1];
            carry = QM == kQuantPw ? pw_quant(xh, inv) : QM == kQuantInt ? __float_as_int(xh) : prequant(xh, inv.inv, dummy);
        } else {
            load_patch<RANK, VEC4>(x, g, l, 4 * k - 1, v);
            prequant32<QM, false>(v, inv, facc, qp);
        }
    }
#pragma unroll 1
    for (int t = 0; t < 4; t++) {
        const int s = 4 * k + t;
        load_patch<RANK, VEC4>(x, g, l, s, v);
        int q[32], d[32];
        prequant32<QM, false>(v, inv, facc, q);
        if (RANK == 1) {
            const int left = shift_up1_raw(q[31]);
            d[0] = q[0] - (lane == 0 ? carry : left);
#pragma unroll
            for (int m = 1; m < 32; m++) d[m] = q[m] - q[m - 1];
            carry = __builtin_amdgcn_readlane(q[31], 63);
        } else {
            sweep_diff<RANK == 1 ? 2 : RANK>(q, qp, d);
#pragma unroll
            for (int i = 0; i < 32; i++) qp[i] = q[i];
            inplane_wide<RANK>(d, lane);
        }
        const uint32_t keep = l.edge ? keep_bits<RANK>(l, s, lane) : ~0u;
        total += log_escapes(d, keep, s, lane, S, pairs);
        uint32_t P[16];
#pragma unroll
        for (int i = 0; i < 16; i++) P[i] = __builtin_amdgcn_perm((uint32_t)d[i + 16], (uint32_t)d[i], 0x05040100u);
        sign_magnitude(P);
        transpose16(P);
#pragma unroll
        for (int b = 0; b < 16; b++) word[64 * (4 * b + t)] = P[b] & keep;
    }
    return total;
}

// Rare path: a step saw NaN/Inf or |x*inv| >= 2^31.  Re-read the layer's
// cells and classify them the way the format defines the status bits
// (halo values belong to the layer below, which reports them).  A real call,
// with the geometry read from its copy in the scratch, so that nothing of it
// adds to the registers of the common path.
__device__ __noinline__ uint32_t classify_errors(const float* __restrict__ x, const uint8_t* scr, int64_t c, int wave,
                                                 float inv, int lane)
{
    const Geom g = *reinterpret_cast<const Geom*>(scr + kScratchGeomOff);
    int64_t o[3], e[3];
    chunk_box(g, c, o, e);
    uint32_t err = 0;
    for (int t = 0; t < 4; t++) {
        const int s = 4 * wave + t;
        for (int m = 0; m < 32; m++) {
            int64_t r0 = 0, r1 = 0, r2 = 0;
            if (g.rank == 3) { r0 = s; r1 = 4 * (lane % 8) + m / 8; r2 = 8 * (lane / 8) + m % 8; }
            else if (g.rank == 2) { r0 = 2 * s + m / 16; r1 = 16 * lane + m % 16; }
            else { r0 = (int64_t)kStepCodes * s + kPatchCodes * lane + m; }
            if (r0 >= e[0] || r1 >= e[1] || r2 >= e[2]) continue;
            const float v = x[((o[0] + r0) * g.n[1] + o[1] + r1) * g.n[2] + o[2] + r2];
            if (!__builtin_isfinite(v)) err |= kErrNonfinite;
            else if (!(__builtin_fabsf(v * inv) < 2147483648.0f)) err |= kErrEbRange;
        }
    }
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) err |= (uint32_t)__shfl_xor((int)err, sh);
    return err;
}

// ------------------------------------------------------------ one chunk
// Payload of the chunk whose layers' counts are in S (16-B units): its nonzero
// bricks, then its escape pairs padded to 16 bytes (none when the chunk holds
// more than kChunkOutlierCap escapes: the stream then carries the OUTLIER_CAP
// status).
struct ChunkSum {
    uint32_t bricks, esc, kept;
    uint32_t base;  // bricks of the layers before the wave's
};
__device__ __forceinline__ ChunkSum chunk_sum(const CompressLds& S, int par, int wave)
{
    ChunkSum c;
    uint32_t n[kLayers];
#pragma unroll
    for (int k = 0; k < kLayers; k++) n[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.nnz[par][k]);
    c.bricks = n[0] + n[1] + n[2] + n[3];
    c.base = (wave > 0 ? n[0] : 0u) + (wave > 1 ? n[1] : 0u) + (wave > 2 ? n[2] : 0u);
    c.esc = S.nout[par][0] + S.nout[par][1] + S.nout[par][2] + S.nout[par][3];  // each at most 8192: no overflow
    c.esc = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.esc);
    c.kept = c.esc > (uint32_t)kChunkOutlierCap ? 0u : c.esc;
    return c;
}
__device__ __forceinline__ uint32_t chunk_units(const ChunkSum& c) { return c.bricks + (c.kept + 1) / 2; }

// Chunk state words are read and written with agent-scope atomics: the
// workgroups that publish and read them run on different XCDs, whose L2
// caches are not coherent with one another.
__device__ __forceinline__ void publish_state(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t peek_state(const uint64_t* p)
{
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Flag words of a layer's bit planes (the lanes with a nonzero brick), the two
// halves of plane b's on lane b.
struct Flags {
    uint32_t lo, hi;
};

// Wave `wave`'s layer of chunk c: its bricks in W, its counts in S.  The
// chunk's last wave to get here publishes its size at once: a size published
// after the workgroup barrier would wait for this workgroup's look-back, and
// other look-backs for it in turn.
template <int RANK, bool VEC4, int QM = kQuantGrid>
__device__ __forceinline__ void chunk_layer(const float* __restrict__ x, const uint8_t* __restrict__ scr, const Geom& g,
                                            int64_t c, const Lane& l, int wave, int lane, int par, Quant inv,
                                            float (&h)[32], float (&v)[32], uint8_t* slot, CompressLds& S,
                                            uint32_t (&W)[kPlanes][4], Flags& F)
{
    uint32_t nout = 0;
    if (4 * wave < l.live) {
        float facc = 0.0f;
        bool wide;
        int first = 0;
        if (swept_down<RANK>(wave)) wide = layer_fast<RANK, VEC4, QM, RANK >= 2>(x, g, l, wave, inv, lane, h, v, S.tile[wave], W, facc, first);
        else wide = layer_fast<RANK, VEC4, QM, false>(x, g, l, wave, inv, lane, h, v, S.tile[wave], W, facc, first);
        if (wide) {
            nout = layer_wide<RANK, VEC4, QM>(x, scr, c, wave, inv, lane, slot, (LdsState*)&S);
            const uint32_t* word = reinterpret_cast<const uint32_t*>(slot) + 4 * wave * kPlanes * kPatches + lane;
#pragma unroll
            for (int b = 0; b < kPlanes; b++)
#pragma unroll
                for (int t = 0; t < 4; t++) W[b][t] = word[64 * (4 * b + t)];
        }
        else if (escapes(first)) {  // the chunk's first cell, the only escape of layer 0
            nout = 1;
            if (lane == 0) {
                const uint32_t at = __hip_atomic_fetch_add(&S.esc_used, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                S.esc_at[0] = at;
                S.esc_n[0] = 1;
                S.esc_n[1] = S.esc_n[2] = S.esc_n[3] = 0;
                if (at < (uint32_t)kChunkOutlierCap)
                    reinterpret_cast<uint2*>(slot + kSlotPairs)[at] = make_uint2(0u, (uint32_t)first);
            }
        }
        if (QM != kQuantInt && __ballot(!(facc < 2147483648.0f))) {  // NaN, Inf or |x*inv| >= 2^31 somewhere
            const uint32_t err = classify_errors(x, scr, c, wave, inv.inv, lane);
            if (lane == 0 && err) atomicOr(&S.err[par], err);
        }
    } else {
#pragma unroll
        for (int b = 0; b < kPlanes; b++) W[b][0] = W[b][1] = W[b][2] = W[b][3] = 0u;
    }
    uint32_t nnz = 0;
    F = Flags{0u, 0u};
#pragma unroll
    for (int b = 0; b < kPlanes; b++) {
        const uint64_t f = __ballot((W[b][0] | W[b][1] | W[b][2] | W[b][3]) != 0u);
        nnz += (uint32_t)__builtin_popcountll(f);
        set_lane(F.lo, b, (uint32_t)f);
        set_lane(F.hi, b, (uint32_t)(f >> 32));
    }
    if (lane == 0) {
        S.nnz[par][wave] = nnz;
        S.nout[par][wave] = nout;
        if (__hip_atomic_fetch_add(&S.arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == kLayers - 1) {
            S.arrived = 0;  // the next chunk's waves arrive after a barrier
            publish_state(reinterpret_cast<uint64_t*>(const_cast<uint8_t*>(scr) + kScratchStateOff) + c,
                          kFlagAgg | chunk_units(chunk_sum(S, par, 0)));
        }
    }
}

// polls of a look-back before it gives up (each poll sleeps about 64 cycles
// and waits for a load that bypasses the L2; far beyond any real wait)
constexpr int kLookbackSpins = 1 << 18;

// The states of the chunks before c, read ahead of a look-back (issued before
// the next chunk's layer, used after it): kAhead windows of 64.
constexpr int kAhead = 4;
struct StatesAhead {
    uint64_t v[kAhead];
};
__device__ __forceinline__ void states_ahead(const uint64_t* state, int64_t c, int lane, StatesAhead& a)
{
    // branch-free (chunk numbers stay below 2^31): before chunk 0, chunk 0's
    // state, which lookback takes for an inclusive prefix of 0
#pragma unroll
    for (int i = 0; i < kAhead; i++) a.v[i] = peek_state(state + max((int)c - 1 - 64 * i - lane, 0));
}

// Exclusive prefix of chunk c's payload size (Sec. 3.4: the offset of its
// data blocks), by one wave: the published states of chunks c-1, c-2, ... are
// taken 64 at a time (the first windows as read ahead) and summed back to the
// nearest chunk that published its inclusive prefix.  Chunks that have not
// published their size yet are polled until they do (every chunk before c was
// taken by a running workgroup, which publishes its size without waiting for
// anything).  Returns false if the polls ran out (the stream is then marked
// with an internal error).
__device__ __forceinline__ bool lookback(const uint64_t* state, int64_t c, int lane, const StatesAhead& a, uint64_t& excl)
{
    uint64_t sum = 0;
    // one window; 1: done (excl is set), 0: go on, -1: gave up
    auto window = [&](int hi, uint64_t v) -> int {
        const int i = hi - 1 - lane;  // lane 0 has the nearest chunk
        if (i < 0) v = kFlagIncl;     // before chunk 0: inclusive prefix 0
        for (int spin = 0;; spin++) {
            const uint32_t flag = (uint32_t)(v >> 62);
            const uint64_t incl = __ballot(flag == (uint32_t)(kFlagIncl >> 62));
            const int first = incl ? __builtin_ctzll(incl) : 64;
            const uint64_t below = first == 64 ? ~0ull : (1ull << first) - 1;
            const uint64_t miss = __ballot(flag == 0u) & below;
            if (!miss) {
                // sizes (below 2^13 each) summed over the lanes, then the prefix
                const int t = wave_incl_scan(lane < first ? (int)(uint32_t)v : 0);
                sum += (uint32_t)__builtin_amdgcn_readlane(t, 63);
                if (incl) {
                    const uint64_t p = v & kValueMask;
                    sum += (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(p >> 32), first) << 32 |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)p, first);
                }
                excl = sum;
                return incl ? 1 : 0;
            }
            if (spin >= kLookbackSpins) {
                excl = 0;
                return -1;
            }
            __builtin_amdgcn_s_sleep(1);
            if ((miss >> lane) & 1ull) v = peek_state(state + i);
        }
    };
    int hi = (int)c;
#pragma unroll
    for (int w = 0; w < kAhead; w++, hi -= 64) {
        const int r = window(hi, a.v[w]);
        if (r) return r > 0;
    }
    for (;; hi -= 64) {  // ends at the latest in the window of chunk 0
        const int r = window(hi, peek_state(state + max(hi - 1 - lane, 0)));
        if (r) return r > 0;
    }
}

typedef __attribute__((address_space(3))) fz_u32x4 LdsUnit;
__device__ __forceinline__ void put_pair(LdsUnit* units, uint32_t j, uint2 p)
{
    __attribute__((address_space(3))) uint32_t* w = (__attribute__((address_space(3))) uint32_t*)units + 2 * j;
    w[0] = p.x;
    w[1] = p.y;
}
__device__ __forceinline__ void put_pair(fz_u32x4* units, uint32_t j, uint2 p)
{
    reinterpret_cast<uint2*>(units)[j] = p;
}

// After a workgroup barrier that follows chunk_layer on all waves: the layer's
// flags go to the stream, the chunk's escape count to the table, and its
// payload to `dst`: nonzero bricks in (layer, plane, patch) order, then the
// escape pairs padded to 16 bytes.  dst: the LDS buffer, or the chunk's place
// in the stream (a payload past kPayUnits, whose look-back was not put off: 2^24
// values 1-D, 16.1 bits each 36.2 us, 15.1 bits and staged 33.2; 4096^2 36.8 / 34.8).
// A chunk may hold kChunkOutlierCap escapes wherever they fall; past that the
// stream carries the OUTLIER_CAP status and no pairs are written.  The flags
// come from the lanes they were counted into: formed again from W, the compiler
// kept 16 conditions in spilled scalar registers (1800x3600 REL 30.5 us, now
// 25.6 with the first chunk's loads issued before the range is folded).
template <typename Unit>  // uint4 in LDS or in global memory
__device__ __forceinline__ void store_chunk(uint8_t* __restrict__ out, const Geom& g, int64_t c, int wave, int lane, int par,
                                            const ChunkSum& m, const uint32_t (&W)[kPlanes][4], const Flags& F,
                                            const uint8_t* slot, CompressLds& S, Unit* dst)
{
    uint32_t base = m.base;
#pragma unroll
    for (int b = 0; b < kPlanes; b++) {
        const uint64_t f = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)F.hi, b) << 32 |
                           (uint32_t)__builtin_amdgcn_readlane((int)F.lo, b);
        const fz_u32x4 brick = {W[b][0], W[b][1], W[b][2], W[b][3]};
        if (__builtin_amdgcn_inverse_ballot_w64(f)) dst[base + mbcnt(f)] = brick;
        base += (uint32_t)__builtin_popcountll(f);
    }
    if (lane < kPlanes)
        reinterpret_cast<uint2*>(out + g.flags_off + (int64_t)kFlagBytesPerChunk * c + 128 * wave)[lane] = make_uint2(F.lo, F.hi);
    if (threadIdx.x == 0) {
        reinterpret_cast<uint32_t*>(out + g.table_off + 8 * c)[1] = m.kept;
        const uint32_t err = atomicExch(&S.err[par], 0u) | (m.esc > (uint32_t)kChunkOutlierCap ? kErrOutlierCap : 0u);
        if (err) atomicOr(reinterpret_cast<uint32_t*>(out + kOffStatus), err);
    }
    if (m.esc) {  // rare (the same on every wave)
        if (m.kept && S.nout[par][wave]) {  // this layer's pairs, behind those of the layers before
            uint32_t to = 0;
            for (int w = 0; w < wave; w++) to += S.nout[par][w];
            for (int s = 4 * wave; s < 4 * wave + 4; s++) {
                const uint32_t n = S.esc_n[s], at = S.esc_at[s];
                for (uint32_t j = (uint32_t)lane; j < n; j += 64) {
                    const uint2 pr = reinterpret_cast<const uint2*>(slot + kSlotPairs)[at + j];
                    put_pair(dst + m.bricks, to + j, pr);
                }
                to += n;
            }
        }
        if (threadIdx.x == 0) {
            if (m.kept & 1u) put_pair(dst + m.bricks, m.kept, make_uint2(0u, 0u));
            S.esc_used = 0;
        }
        __syncthreads();  // the list is written again by the next chunk's layers
    }
}

// A workgroup barrier for data in LDS only: it waits for this wave's LDS
// operations but leaves its loads and stores to memory in flight (the plain
// barrier waits for those too, here the next chunk's first loads).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Placement of chunk p, staged with `units` 16-B units of payload, in two
// parts.  place_lookback, by one wave (any time after the staging, before a
// barrier that precedes place_copy): the look-back finds the offset, thread 0 publishes the inclusive prefix, writes the offset to
// the table and, for the field's last chunk, the stream's total size to the
// header, and leaves the offset in S.excl.  A failed look-back marks the
// stream with an internal error and still publishes (as if at offset 0), so
// that no later chunk waits on this one; every offset stays inside the
// stream's bound.
__device__ __forceinline__ void place_lookback(uint8_t* __restrict__ out, uint8_t* __restrict__ scr, const Geom& g,
                                               int64_t p, uint32_t units, const StatesAhead& ahead, CompressLds& S, int lane)
{
    uint64_t* state = reinterpret_cast<uint64_t*>(scr + kScratchStateOff);
    uint64_t excl;
    const bool ok = lookback(state, p, lane, ahead, excl);
    if (lane == 0) {
        if (!ok) atomicOr(reinterpret_cast<uint32_t*>(out + kOffStatus), kErrInternal);
        const uint64_t at = ok ? excl : 0;
        S.excl = ok ? excl : ~0ull;
        publish_state(state + p, kFlagIncl | (at + units));
        reinterpret_cast<uint32_t*>(out + g.table_off)[2 * p] = (uint32_t)at;
        if (p == g.n_chunks - 1) *reinterpret_cast<uint64_t*>(out + kOffTotal) = (uint64_t)g.payload_off + 16 * (at + units);
    }
}

// place_copy, by the whole workgroup: the staged payload goes from LDS to its
// offset.
__device__ __forceinline__ void place_copy(uint8_t* __restrict__ out, const Geom& g, uint32_t units, const CompressLds& S)
{
    const uint64_t excl = S.excl;
    if (excl == ~0ull) return;
    uint4* dst = reinterpret_cast<uint4*>(out + g.payload_off) + excl;
    for (uint32_t i = threadIdx.x; i < units; i += 64 * kLayers) dst[i] = S.pay[i];
}

// A chunk whose payload does not fit the LDS buffer: looked up and stored at
// once, straight from the registers (after the barrier behind the previous
// chunk's place_copy; ends with a barrier).
__device__ __forceinline__ void place_now(uint8_t* __restrict__ out, uint8_t* __restrict__ scr, const Geom& g, int64_t c,
                                          int wave, int lane, int par, const ChunkSum& m, const uint32_t (&W)[kPlanes][4],
                                          const Flags& F, const uint8_t* slot, CompressLds& S)
{
    if (wave == 0) {
        StatesAhead ahead;
        states_ahead(reinterpret_cast<const uint64_t*>(scr + kScratchStateOff), c, lane, ahead);
        place_lookback(out, scr, g, c, chunk_units(m), ahead, S, lane);
    }
    __syncthreads();
    const uint64_t excl = S.excl;
    // a failed look-back marked the stream; its offset is 0, inside the bound
    store_chunk(out, g, c, wave, lane, par, m, W, F, slot, S, reinterpret_cast<fz_u32x4*>(out + g.payload_off) + (excl == ~0ull ? 0 : excl));
    lds_barrier();
}

// What a workgroup has stored of a field so far, added to the header's counts
// once (by thread 0): one atomic per workgroup, not per chunk.
struct Counts {
    uint64_t bricks = 0, pairs = 0;
    uint32_t chunks = 0;  // (batches: the field's chunks it has coded)
};
__device__ __forceinline__ void add_counts(uint8_t* __restrict__ out, Counts& n)
{
    if (threadIdx.x == 0) {
        if (n.bricks) atomicAdd(reinterpret_cast<unsigned long long*>(out + kOffNnz), (unsigned long long)n.bricks);
        if (n.pairs) atomicAdd(reinterpret_cast<unsigned long long*>(out + kOffNout), (unsigned long long)n.pairs);
    }
    n = Counts{};
}

// ------------------------------------------------- per-field pipeline steps
// These bodies run for one field; the per-field kernels call them with the
// whole grid, the batched kernels with the blocks given to that field.

// Header, table padding, scratch and chunk states of one field, by `nthreads`
// threads numbered `tid`.
__device__ __forceinline__ void init_field(uint8_t* __restrict__ out, uint8_t* __restrict__ scratch, const Geom& g,
                                           const HeaderImage& h, int64_t tid,
                                           int64_t nthreads)
{
    if (tid < kHeaderBytes / 4) reinterpret_cast<uint32_t*>(out)[tid] = h.w[tid];
    if (tid == 0 && (g.n_chunks & 1))  // the chunk table is padded to 16 bytes with zeros
        *reinterpret_cast<uint2*>(out + g.table_off + 8 * g.n_chunks) = make_uint2(0u, 0u);
    uint32_t* scr = reinterpret_cast<uint32_t*>(scratch);
    if (tid < kScratchGeomOff / 4) scr[tid] = 0u;
    static_assert(sizeof(Geom) % 4 == 0 && kScratchGeomOff + sizeof(Geom) <= kScratchStateOff, "scratch layout");
    if (tid < (int64_t)(sizeof(Geom) / 4))
        scr[kScratchGeomOff / 4 + tid] = reinterpret_cast<const uint32_t*>(&g)[tid];
    uint64_t* state = reinterpret_cast<uint64_t*>(scratch + kScratchStateOff);
    for (int64_t i = tid; i < g.n_chunks; i += nthreads) state[i] = 0;
}

// Partial value range of block `blk` of `nblk` (256 threads each) for the
// relative error bound: the blocks walk the field from its end so that its
// beginning, which compression reads first, is the most recently touched
// data.  The partial (min key, max key, non-finite) goes to the scratch.
__device__ __forceinline__ void minmax_block(const float* __restrict__ x, int64_t n, uint8_t* __restrict__ scr,
                                             const Geom& g, int64_t blk, int64_t nblk)
{
    __shared__ uint32_t s_red[3][4];
    // NaN-propagating minimum / maximum over the raw values: the range is only
    // used when every value is finite, and a NaN or an infinity shows up in
    // the result (the minimum is -Inf or NaN, or the maximum +Inf or NaN)
    float fmn = __builtin_inff(), fmx = -__builtin_inff();
    auto take4 = [&](const fz_f32x4& v) {
        fmn = __builtin_elementwise_minimum(__builtin_elementwise_minimum(fmn, v.x), v.y);
        fmx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fmx, v.x), v.y);
        fmn = __builtin_elementwise_minimum(__builtin_elementwise_minimum(fmn, v.z), v.w);
        fmx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fmx, v.z), v.w);
    };
    const int64_t stride = nblk * 256;
    const int64_t tid = blk * 256 + threadIdx.x;
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const int64_t n4 = vec ? n / 4 : 0;
    const fz_f32x4* x4 = reinterpret_cast<const fz_f32x4*>(x);
    // backwards, so that the front of the field, which the compression
    // kernel reads first, is the most recently read (one load per
    // iteration: unrolling by strided loads measured slower); streaming
    // loads, as no value is read twice here
    for (int64_t i = n4 - 1 - tid; i >= 0; i -= stride) take4(__builtin_nontemporal_load(x4 + i));
    for (int64_t k = 4 * n4 + tid; k < n; k += stride) {
        fmn = __builtin_elementwise_minimum(fmn, x[k]);
        fmx = __builtin_elementwise_maximum(fmx, x[k]);
    }
    const bool some = fmn <= fmx;  // false for a thread without values (and for NaN)
    uint32_t bad = (fmn >= -3.40282347e38f && fmx <= 3.40282347e38f) ? 0u : 1u;
    uint32_t lo = some ? float_key(fmn) : 0xFFFFFFFFu, hi = some ? float_key(fmx) : 0u;
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, sh));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, sh));
        bad |= (uint32_t)__shfl_xor((int)bad, sh);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { s_red[0][w] = lo; s_red[1][w] = hi; s_red[2][w] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t* part = reinterpret_cast<uint32_t*>(scr + g.scr_minmax) + 4 * blk;
        part[0] = min(min(s_red[0][0], s_red[0][1]), min(s_red[0][2], s_red[0][3]));
        part[1] = max(max(s_red[1][0], s_red[1][1]), max(s_red[1][2], s_red[1][3]));
        part[2] = s_red[2][0] | s_red[2][1] | s_red[2][2] | s_red[2][3];
    }
}

// The eb parameters of a REL compression, from the folded value range.
struct RelParams {
    uint32_t status;          // 0, kErrNonfinite or kErrEbRange
    float ebx2, inv, vmin, vmax;
};

// Fold the partial ranges of one field and derive the eb parameters, by one
// block of blockDim.x threads (a multiple of 64, at most 1024); every thread
// gets the result.  eb_abs = eb * (vmax - vmin) in double (a constant field
// uses eb * |vmax|, or eb if that is 0), ebx2 = fp32(2 eb_abs),
// inv = fp32(1 / (double)ebx2).
__device__ __forceinline__ RelParams fold_params(const uint8_t* __restrict__ scratch, const Geom& g, double eb,
                                                 int nparts)
{
    __shared__ uint32_t s_red[3][16];
    // the partials (16 B each) in 16-byte loads, 8 per thread in flight
    // together: every compression workgroup folds them before its first
    // chunk, and one load at a time cost a cache round trip per 256 partials
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(scratch + g.scr_minmax), (short)0, 16 * nparts, kBufferFlags);
    uint32_t lo = 0xFFFFFFFFu, hi = 0u, bad = 0u;
    for (int i0 = 0; i0 < nparts; i0 += 8 * (int)blockDim.x) {
        fz_u32x4 t[8];
#pragma unroll
        for (int k = 0; k < 8; k++)
            t[k] = __builtin_amdgcn_raw_buffer_load_b128(rp, 16u * (uint32_t)(i0 + k * blockDim.x + threadIdx.x), 0u, 0);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            if (i0 + k * (int)blockDim.x + (int)threadIdx.x < nparts) {
                lo = min(lo, t[k].x);
                hi = max(hi, t[k].y);
                bad |= t[k].z;
            }
        }
    }
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, sh));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, sh));
        bad |= (uint32_t)__shfl_xor((int)bad, sh);
    }
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) { s_red[0][w] = lo; s_red[1][w] = hi; s_red[2][w] = bad; }
    __syncthreads();
    lo = 0xFFFFFFFFu, hi = 0u, bad = 0u;
    for (int i = 0; i < nw; i++) {
        lo = min(lo, s_red[0][i]);
        hi = max(hi, s_red[1][i]);
        bad |= s_red[2][i];
    }
    // the same on every lane: kept scalar, so that a branch on the result is
    // uniform and nothing after it is treated as divergent
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    bad = __builtin_amdgcn_readfirstlane(bad);
    __syncthreads();  // s_red may be reused by the caller's next fold
    RelParams r{0u, 0.0f, 0.0f, 0.0f, 0.0f};
    if (bad) {
        r.status = kErrNonfinite;
    } else {
        r.vmin = key_float(lo);
        r.vmax = key_float(hi);
        const double range = (double)r.vmax - (double)r.vmin;
        double eb_abs;
        if (range > 0.0) eb_abs = eb * range;
        else {
            const double a = __builtin_fabs((double)r.vmax);
            eb_abs = eb * (a > 0.0 ? a : 1.0);
        }
        r.ebx2 = (float)(2.0 * eb_abs);
        r.inv = (float)(1.0 / (double)r.ebx2);
        if (!(r.ebx2 >= 1.17549435e-38f) || !__builtin_isfinite(r.ebx2) || !__builtin_isfinite(r.inv) || !(r.inv > 0.0f))
            r.status = kErrEbRange;
    }
    return r;
}

// The header's eb fields (and, on a failed range, its status and total) and
// the scratch's pre_status, by one thread.
__device__ __forceinline__ void write_params(uint8_t* __restrict__ out, uint8_t* __restrict__ scratch, const Geom& g,
                                             const RelParams& r)
{
    *reinterpret_cast<float*>(out + kOffEbx2) = r.ebx2;
    *reinterpret_cast<float*>(out + kOffInv) = r.inv;
    *reinterpret_cast<float*>(out + kOffVmin) = r.vmin;
    *reinterpret_cast<float*>(out + kOffVmax) = r.vmax;
    if (r.status) {
        *reinterpret_cast<uint32_t*>(out + kOffStatus) = r.status;
        *reinterpret_cast<uint64_t*>(out + kOffTotal) = (uint64_t)g.payload_off;
    }
    reinterpret_cast<Scratch*>(scratch)->pre_status = r.status;
}

// The eb parameters by a block of its own (the batch layer, the field-global
// predictor): fold, then thread 0 writes them.
__device__ __forceinline__ void params_field(uint8_t* __restrict__ out, uint8_t* __restrict__ scratch, const Geom& g,
                                             double eb, int nparts)
{
    const RelParams r = fold_params(scratch, g, eb, nparts);
    if (threadIdx.x == 0) write_params(out, scratch, g, r);
}

// End of one field's compression inside the kernel that codes it, by thread 0
// of a workgroup that adds its `part` (workgroups or chunks) of `all`: the last
// one settles the status word, so that no launch of its own is needed.  A
// failed prequantization anywhere (NaN/Inf, overflow) ends the pipeline before
// the encoder, so the escape-cap bit of chunks that went on counts only when no
// such bit is set.  The status word and the count are only touched with
// agent-scope atomics, which every XCD sees in one order (their L2 caches are
// not coherent with one another, so nothing here may rely on them).  Thread 0
// set its workgroup's status bits; an explicit wait for its outstanding memory
// operations (not an agent-scope release, which adds an L2 write-back at every
// workgroup's end: +9 us on 512^3) makes those atomics complete before the
// count is issued, and the last workgroup reads and clears the word only after
// its count has returned.  Workgroups that return because the range pass failed
// (pre_status) do not count; nothing is settled then.
__device__ __forceinline__ void finish_part(uint8_t* __restrict__ out, uint8_t* __restrict__ scratch, uint32_t part, uint32_t all)
{
    if (threadIdx.x != 0) return;
    Scratch* scr = reinterpret_cast<Scratch*>(scratch);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // no memory operation moves below this point
    __builtin_amdgcn_s_waitcnt(0);  // and every one of this thread's has completed (the fence alone emits no wait)
    if (__hip_atomic_fetch_add(&scr->done, part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != all - part) return;
    uint32_t* st = reinterpret_cast<uint32_t*>(out + kOffStatus);
    const uint32_t v = __hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v & (kErrNonfinite | kErrEbRange))
        __hip_atomic_fetch_and(st, ~kErrOutlierCap, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace fz
