// fz_global.hip -- the field-global Lorenzo predictor of libfzmi (gfx950).
//
// The classic Lorenzo predictor runs over the whole field (Sec. 2.3): a
// chunk's border cells are predicted from the neighbouring chunk's values.
// The stream stores the field-global deltas d chunk by chunk, exactly as the
// chunk-local stream stores its own, and header byte 15 says which.
//
// Compression reuses the chunk kernel unchanged.  That kernel takes the
// chunk-local Lorenzo difference of its input, so it is fed the integers p
// whose chunk-local difference is d: the inclusion-exclusion of q over the
// chunk's lower faces, p(c) = sum over subsets S of the axes of (-1)^|S|
// q(c with the axes in S moved to the plane just before the chunk), a
// neighbour outside the field counting 0.  k_face computes p from the input
// (prequantizing the few face values it needs on the fly) into the integer
// buffer behind the fp32 bound.
//
// Decompression runs the chunk kernel with integer output, which yields the
// chunk-local prefix sums p again, and then turns them into the field-global
// prefix sums q: per axis a small kernel computes the carries of every line's
// segments from the segment-end values (k_seg_carry), and one pass adds them
// all and dequantizes (k_seg_final).  Wrapping 32-bit integer arithmetic
// throughout.
#include <hip/hip_runtime.h>

#include "fz.h"
#include "fz_compress_dev.hpp"
#include "fz_decompress_dev.hpp"
#include "fz_kernels.hpp"

namespace fz {

constexpr int kGlobalThreads = 256;

// ------------------------------------------------- a chunk as runs of 4 values
// The passes over a field in place (k_face, k_seg_final) give a chunk to a
// workgroup of 16 waves, and a wave 8 runs; a lane's part of a run is 4 values,
// so every load and store moves whole lines.
//   3-D: plane `wave` of the chunk, a run is 4 of its rows;
//   2-D: 8 rows (8 (wave / 4) ..) of 256 columns (256 (wave mod 4) ..);
//   1-D: 2048 values, a run is 256.
// What a pass adds to a cell is the sum of a term per row, a term per column
// and in 3-D a term per row and column that is the same for every plane.
constexpr int kRuns = 8, kRunThreads = 1024;

struct Runs {
    int64_t org[3], ext[3];
    bool edge;
    uint32_t voff, step;  // byte offsets: the lane's first value in its wave's part, from run to run
};

template <int RANK>
__device__ __forceinline__ Runs runs_of(const Geom& g, int64_t c, int lane)
{
    Runs r;
    chunk_box(g, c, r.org, r.ext);
    r.edge = false;
#pragma unroll
    for (int i = 0; i < 3; i++) r.edge |= r.ext[i] < g.box[i];
    // below 2^32: at most 32 rows of a contiguous extent below 2^25
    const uint32_t nx = (uint32_t)g.n[RANK - 1];
    r.voff = RANK == 3 ? 4u * ((uint32_t)(lane >> 4) * nx + 4u * (uint32_t)(lane & 15)) : 16u * (uint32_t)lane;
    r.step = RANK == 3 ? 16u * nx : RANK == 2 ? 4u * nx : 1024u;
    return r;
}

// whether the wave's part of the chunk holds cells of the field, and its first cell
template <int RANK>
__device__ __forceinline__ bool part_live(const Runs& r, int wave)
{
    if (RANK == 3) return wave < r.ext[0];
    if (RANK == 2) return 8 * (wave >> 2) < r.ext[0] && 256 * (wave & 3) < r.ext[1];
    return 2048 * wave < r.ext[0];
}
template <int RANK>
__device__ __forceinline__ int64_t part_at(const Geom& g, const Runs& r, int wave)
{
    if (RANK == 3) return ((r.org[0] + wave) * g.n[1] + r.org[1]) * g.n[2] + r.org[2];
    if (RANK == 2) return (r.org[0] + 8 * (wave >> 2)) * g.n[1] + r.org[1] + 256 * (wave & 3);
    return r.org[0] + 2048 * wave;
}

// a resource from 4-byte word `at` of an array of n words to its end (on =
// false, or an `at` outside it: none; a load from it returns zeros)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const void* a, int64_t n, int64_t at, bool on = true)
{
    const int64_t left = 4 * (n - at);
    const int hi = (int)(left >> 32);
    const int range = !on || hi < 0 || at < 0 ? 0 : hi > 0 ? -1 : (int)(uint32_t)left;
    return __builtin_amdgcn_make_buffer_rsrc((uint32_t*)a + (on ? at : 0), (short)0, range, kBufferFlags);
}

__device__ __forceinline__ void load4(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, uint32_t* v)
{
    const fz_u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}

// how many of the lane's values of run j are cells of the chunk (any sign; the first ones)
template <int RANK>
__device__ __forceinline__ int run_cells(const Runs& r, int wave, int j, int lane)
{
    if (RANK == 3) return 4 * j + (lane >> 4) < r.ext[1] ? (int)r.ext[2] - 4 * (lane & 15) : 0;
    if (RANK == 2) return 8 * (wave >> 2) + j < r.ext[0] ? (int)r.ext[1] - 256 * (wave & 3) - 4 * lane : 0;
    return (int)r.ext[0] - (2048 * wave + 256 * j + 4 * lane);
}

template <int RANK, bool STREAM>
__device__ __forceinline__ void store_run(__amdgpu_buffer_rsrc_t rs, const Runs& r, int wave, int j, int lane,
                                          const uint32_t* v)
{
    const fz_u32x4 t = {v[0], v[1], v[2], v[3]};
    if (!r.edge) {
        __builtin_amdgcn_raw_buffer_store_b128(t, rs, r.voff, r.step * j, STREAM ? kCacheStream : 0);
        return;
    }
    const int n = run_cells<RANK>(r, wave, j, lane);
    if (n >= 4) __builtin_amdgcn_raw_buffer_store_b128(t, rs, r.voff, r.step * j, 0);
    else {
        if (n > 0) __builtin_amdgcn_raw_buffer_store_b32(t.x, rs, r.voff, r.step * j, 0);
        if (n > 1) __builtin_amdgcn_raw_buffer_store_b32(t.y, rs, r.voff + 4u, r.step * j, 0);
        if (n > 2) __builtin_amdgcn_raw_buffer_store_b32(t.z, rs, r.voff + 8u, r.step * j, 0);
    }
}

// lane l's value of a term per row is that of the chunk's row l (2-D, and 3-D
// within a plane; 1-D: one value on every lane): that of run j
template <int RANK>
__device__ __forceinline__ uint32_t row_term(uint32_t t, int wave, int j, int lane)
{
    if (RANK == 3) return (uint32_t)lane_value((int)t, 4 * j + (lane >> 4));
    if (RANK == 2) return (uint32_t)__builtin_amdgcn_readlane((int)t, 8 * (wave >> 2) + j);
    return t;
}

// -------------------------------------------------------------- compression
// N values through the stream's quantizer; facc tracks max |x * inv| with NaN
// propagating.  Values outside the field's faces (on = false) count 0.
template <int QM, int N>
__device__ __forceinline__ void quant_words(const uint32_t* v, const Quant& z, bool on, float& facc, uint32_t* q)
{
#pragma unroll
    for (int i = 0; i < N; i++) {
        const float x = __uint_as_float(v[i]), p = x * z.inv;
        facc = __builtin_elementwise_maximum(facc, __builtin_fabsf(p));
        const int k = QM == kQuantPw ? pw_quant(x, z) : (int)__builtin_rintf(p);
        q[i] = on ? (uint32_t)k : 0u;
    }
}

// The status bits of the chunk's own cells (a face's cells are reported by the
// chunk they belong to), by one wave; rare.
__device__ __noinline__ uint32_t face_errors(const float* __restrict__ x, const uint8_t* scr, int64_t c, float inv, int wave,
                                             int lane)
{
    uint32_t err = 0;
    for (int k = 0; k < 4; k++) err |= classify_errors(x, scr, c, (wave + k) & 3, inv, lane);
    return err;
}

// p of one chunk's cells: with the chunk's lower faces at Z, Y, X (the planes
// before it along the three axes), p(z, y, x) = r(z, y, x) - r(z, y, X),
// r(z, y, x) = q(z, y, x) - q(z, Y, x) - (q(Z, y, x) - q(Z, Y, x)).  The last
// difference is the same for every plane of the chunk; r(., X) is one value
// per row, quantized by one lane (and the corner (Y, X) by lane 32).  Bound by
// the reads of the field and the writes of p (both find the infinity cache for
// fields up to its size): 100x500x500 47 us, 4.3 TB/s; 227 us in the form
// before, a thread per cell that read and quantized all 8 corners.  Waves of
// several planes, which keep the common difference in registers, measured the
// same at 2 planes and 2 % slower at 4.
template <int RANK, int QM>
__global__ __launch_bounds__(kRunThreads) void k_face(const float* __restrict__ x, uint8_t* __restrict__ out, Geom g,
                                                      uint32_t first_block)
{
    uint8_t* scr = out + g.scratch_off;
    if (reinterpret_cast<const Scratch*>(scr)->pre_status) return;  // set before this launch (REL range pass): uniform
    const Quant z = quant_of(out);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n = g.n[0] * g.n[1] * g.n[2];
    const int64_t c = xcd_order(first_block + blockIdx.x, g.n_chunks);
    const Runs r = runs_of<RANK>(g, c, lane);
    if (!part_live<RANK>(r, wave)) return;  // (no barrier below)
    const bool inz = RANK == 3 && r.org[0] > 0;                    // 3-D: a plane Z
    const bool iny = RANK >= 2 && r.org[RANK == 3 ? 1 : 0] > 0;    // a row Y
    const bool inx = r.org[RANK - 1] > 0;                          // a column X
    float facc = 0.0f;
    uint32_t A[kRuns][4];  // 3-D: q(Z, y, x) - q(Z, Y, x) of the lane's cells; 2-D: A[0] = q(Y, x)
    uint32_t left = 0;     // 3-D: q(Z, y, X) per row; 2-D: r(y, X); 1-D: q(X)
    const int64_t nx = g.n[RANK - 1];
    // column X of the rows below cell `at`: row l on lane l < 32, row Y on lane 32
    auto column = [&](int64_t at, bool on) {
        const int64_t first = at - (iny ? nx : 0) - 1;  // row Y (or row 0), column X
        const __amdgpu_buffer_rsrc_t rs = words_rsrc(x, n, first, on && inx);
        const uint32_t row = lane < 32 ? (uint32_t)lane + (iny ? 1u : 0u) : 0u;
        uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(rs, 4u * row * (uint32_t)nx, 0, 0), q;
        quant_words<QM, 1>(&v, z, on && inx, facc, &q);
        return lane >= 32 && !iny ? 0u : q;
    };
    if constexpr (RANK == 3) {
        const int64_t at = part_at<3>(g, r, -1);  // plane Z
        uint32_t y[4];
        load4(words_rsrc(x, n, at - nx, inz && iny), 16u * (uint32_t)(lane & 15), 0, y);
        const __amdgpu_buffer_rsrc_t rs = words_rsrc(x, n, at, inz);
#pragma unroll
        for (int j = 0; j < kRuns; j++) load4(rs, r.voff, r.step * j, A[j]);
        quant_words<QM, 4>(y, z, inz && iny, facc, y);
        left = column(at, inz);
#pragma unroll
        for (int j = 0; j < kRuns; j++) {
            quant_words<QM, 4>(A[j], z, inz, facc, A[j]);
#pragma unroll
            for (int e = 0; e < 4; e++) A[j][e] -= y[e];
        }
    } else if constexpr (RANK == 2) {
        load4(words_rsrc(x, n, r.org[0] * nx + r.org[1] + 256 * (wave & 3) - nx, iny), r.voff, 0, A[0]);
        quant_words<QM, 4>(A[0], z, iny, facc, A[0]);
        left = column(r.org[0] * nx + r.org[1], true);
        left -= (uint32_t)__builtin_amdgcn_readlane((int)left, 32);
    } else {
        uint32_t v = inx ? __float_as_uint(x[r.org[0] - 1]) : 0u;
        quant_words<QM, 1>(&v, z, inx, facc, &left);
    }
    int32_t* p = reinterpret_cast<int32_t*>(out + g.q_off);
    const int64_t at = part_at<RANK>(g, r, wave);
    const __amdgpu_buffer_rsrc_t rs = words_rsrc(x, n, at);
    uint32_t v[kRuns][4], y[4];
    if (RANK == 3) load4(words_rsrc(x, n, at - nx, iny), 16u * (uint32_t)(lane & 15), 0, y);
#pragma unroll
    for (int j = 0; j < kRuns; j++) load4(rs, r.voff, r.step * j, v[j]);
    uint32_t t = left;
    if constexpr (RANK == 3) {
        t = column(at, true) - left;
        t -= (uint32_t)__builtin_amdgcn_readlane((int)t, 32);
        quant_words<QM, 4>(y, z, iny, facc, y);
    }
    const __amdgpu_buffer_rsrc_t ws = words_rsrc(p, n, at);
#pragma unroll
    for (int j = 0; j < kRuns; j++) {
        quant_words<QM, 4>(v[j], z, true, facc, v[j]);
        const uint32_t u = row_term<RANK>(t, wave, j, lane);
#pragma unroll
        for (int e = 0; e < 4; e++) v[j][e] -= (RANK == 3 ? y[e] + A[j][e] : RANK == 2 ? A[0][e] : 0u) + u;
        store_run<RANK, false>(ws, r, wave, j, lane, v[j]);
    }
    if (__ballot(!(facc < 2147483648.0f))) {  // NaN, Inf or |x * inv| >= 2^31 in the chunk or a face of it
        const uint32_t err = face_errors(x, scr, c, z.inv, wave, lane);
        if (lane == 0 && err) {
            atomicOr(reinterpret_cast<uint32_t*>(out + kOffStatus), err);
            *reinterpret_cast<uint64_t*>(out + kOffTotal) = (uint64_t)g.payload_off;
        }
    }
}

template <int RANK>
static hipError_t launch_face_rank(const float* x, uint8_t* out, const Geom& g, bool pw, hipStream_t st)
{
    return launch_chunks(g.n_chunks, [&](uint32_t first, dim3 blocks) {
        if (pw) hipLaunchKernelGGL((k_face<RANK, kQuantPw>), blocks, dim3(kRunThreads), 0, st, x, out, g, first);
        else hipLaunchKernelGGL((k_face<RANK, kQuantGrid>), blocks, dim3(kRunThreads), 0, st, x, out, g, first);
    });
}

hipError_t launch_face(const float* x, uint8_t* out, const Geom& g, bool pw, hipStream_t st)
{
    switch (g.rank) {
        case 3: return launch_face_rank<3>(x, out, g, pw, st);
        case 2: return launch_face_rank<2>(x, out, g, pw, st);
        default: return launch_face_rank<1>(x, out, g, pw, st);
    }
}

// ------------------------------------------------------------ decompression
template <int RANK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress_int(const uint8_t* __restrict__ s, uint64_t sb,
                                                           int32_t* __restrict__ y, Geom g, uint32_t* d_err, uint32_t first)
{
    __shared__ DecompressLds<8> S;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    decompress_chunk<RANK, int32_t, 8>(s, sb, y, STREAM, g, d_err, in_place_chunk<STREAM>(g, first + blockIdx.x), wave, threadIdx.x & 63, S);
}

// Carries of the field-global prefix sums.  Along axis ax the field splits
// into lines (every cell with the other coordinates fixed) and each line into
// segments of the chunk box's extent along ax (a power of two).  After the
// chunk kernel the field holds p, the chunk-local sums.  Taking the axes from
// the contiguous one to the slowest, the global sum along an axis of a value
// that already holds the earlier axes' carries is its local sum plus the
// totals of the line's earlier segments; those totals are the values at the
// segment ends, which are p plus the earlier axes' carries there.  So per axis
// one small kernel reads only the segment ends and writes the carries
// (carry[ax][j][line] = sum over the segments before j), and one final pass
// adds every axis's carry to p and dequantizes.  The sums commute, and all of
// it is wrapping 32-bit arithmetic.
struct Carries {
    // the field as a 3-D one, leading extents 1 below rank 3: axis a of the field is a + 3 - rank here
    int64_t n[3];
    int sh[3];          // log2 of the chunk box along each axis
    int64_t nlines[3];  // lines along each axis
    int64_t nseg[3];    // segments per line
    int64_t off[3];     // start of each axis's carries in the work buffer (u32 units)
    int64_t words;      // size of the work buffer
};

inline Carries carries_of(const Geom& g)
{
    Carries c;
    c.words = 0;
    const int first = 3 - g.rank;
    for (int a = 0; a < 3; a++) {
        c.n[a] = a < first ? 1 : g.n[a - first];
        c.sh[a] = a < first ? 0 : __builtin_ctz((unsigned)g.box[a - first]);
        c.nlines[a] = g.n[0] * g.n[1] * g.n[2] / c.n[a];
        c.nseg[a] = (c.n[a] + (1 << c.sh[a]) - 1) >> c.sh[a];
        c.off[a] = c.words;
        if (a >= first) c.words += c.nlines[a] * c.nseg[a];
    }
    return c;
}

// The carries of axis AX.  A block takes 2^lg lines and shares each out over
// 256 / 2^lg threads, two segments per thread at a time (a thread per line read
// its segment ends one after the other: 13 us per axis at 100x500x500, and all
// of a 1-D field by a single thread).
template <int AX>
__global__ __launch_bounds__(kGlobalThreads) void k_seg_carry(const uint32_t* __restrict__ p, uint32_t* __restrict__ w,
                                                              Carries k, int lg)
{
    constexpr int kEach = 2;
    __shared__ uint32_t s_sum[kGlobalThreads];
    const int lines = 1 << lg, parts = kGlobalThreads >> lg;
    const int l = threadIdx.x & (lines - 1), part = threadIdx.x >> lg;
    const int64_t nl = k.nlines[AX], nseg = k.nseg[AX];
    const int64_t along = AX == 2 ? 1 : AX == 1 ? k.n[2] : k.n[1] * k.n[2];
    for (int64_t tb = (int64_t)blockIdx.x << lg; tb < nl; tb += (int64_t)gridDim.x << lg) {
        const int64_t t = tb + l;
        // line t: along axis 2 row t; else column i of outer coordinate o (c0 or c1)
        const int64_t o = AX == 2 ? t : (t >> 31) ? t / k.n[2] : (int64_t)((uint32_t)t / (uint32_t)k.n[2]);
        const int64_t i = AX == 2 ? 0 : t - o * k.n[2];
        const int64_t cell = AX == 2 ? t * k.n[2] : AX == 1 ? o * k.n[1] * k.n[2] + i : t;
        uint32_t run = 0;
        for (int64_t j0 = 0; j0 < nseg; j0 += parts * kEach) {
            uint32_t v[kEach], sum = 0;
#pragma unroll
            for (int b = 0; b < kEach; b++) {
                const int64_t j = j0 + part * kEach + b, next = (j + 1) << k.sh[AX];
                const int64_t e = (next < k.n[AX] ? next : k.n[AX]) - 1;  // the segment's end
                v[b] = 0;
                if (t < nl && j < nseg) {
                    v[b] = p[cell + e * along];
                    if (AX <= 1) v[b] += w[k.off[2] + (i >> k.sh[2]) * k.nlines[2] + (AX == 1 ? o * k.n[1] + e : e * k.n[1] + o)];
                    if (AX == 0) v[b] += w[k.off[1] + (o >> k.sh[1]) * k.nlines[1] + e * k.n[2] + i];
                }
                sum += v[b];
            }
            // the sum of the line's parts before this one
            s_sum[threadIdx.x] = sum;
            __syncthreads();
            uint32_t upto = sum;
            for (int d = 1; d < parts; d <<= 1) {
                const uint32_t before = part >= d ? s_sum[threadIdx.x - (d << lg)] : 0u;
                __syncthreads();
                upto += before;
                s_sum[threadIdx.x] = upto;
                __syncthreads();
            }
            uint32_t c = run + upto - sum;
            run += s_sum[((parts - 1) << lg) + l];
#pragma unroll
            for (int b = 0; b < kEach; b++) {
                const int64_t j = j0 + part * kEach + b;
                if (t < nl && j < nseg) w[k.off[AX] + j * nl + t] = c;
                c += v[b];
            }
            __syncthreads();  // s_sum is written again
        }
    }
}

// q = p + the carries of every axis, dequantized (Sec. 2.3; the point-wise
// mode's inverse transform) and stored as fp32 in place.  Bound by reading and
// writing the field: 100x500x500 36 us, 5.6 TB/s (a thread per cell: 104 us).
template <int RANK, bool STREAM>
__global__ __launch_bounds__(kRunThreads) void k_seg_final(uint32_t* __restrict__ f, const uint32_t* __restrict__ w,
                                                              Carries k, Geom g, const uint8_t* __restrict__ s,
                                                              uint32_t first)
{
    const float ebx2 = *reinterpret_cast<const float*>(s + kOffEbx2);
    const bool pw = s[kOffEbMode] == 2;
    const uint32_t step = pw ? (uint32_t)ebx2 : 0u;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n = g.n[0] * g.n[1] * g.n[2];
    const int64_t c = xcd_order(first + blockIdx.x, g.n_chunks);
    const Runs r = runs_of<RANK>(g, c, lane);
    if (!part_live<RANK>(r, wave)) return;
    // the carries of this chunk's segment of each axis
    const int64_t cx = k.off[2] + (r.org[RANK - 1] >> k.sh[2]) * k.nlines[2];
    uint32_t A[kRuns][4], left = 0;
    if constexpr (RANK == 3) {
        const __amdgpu_buffer_rsrc_t rs =
            words_rsrc(w, k.words, k.off[0] + (r.org[0] >> k.sh[0]) * k.nlines[0] + r.org[1] * k.n[2] + r.org[2]);
#pragma unroll
        for (int j = 0; j < kRuns; j++) load4(rs, r.voff, r.step * j, A[j]);
    } else if constexpr (RANK == 2) {
        load4(words_rsrc(w, k.words, k.off[1] + (r.org[0] >> k.sh[1]) * k.nlines[1] + r.org[1] + 256 * (wave & 3)), r.voff, 0, A[0]);
        left = __builtin_amdgcn_raw_buffer_load_b32(words_rsrc(w, k.words, cx + r.org[0]), 4u * (uint32_t)(lane & 31), 0, 0);
    } else {
        left = w[cx];
    }
    const __amdgpu_buffer_rsrc_t rs = words_rsrc(f, n, part_at<RANK>(g, r, wave));
    uint32_t v[kRuns][4], y[4], t = left;
    if constexpr (RANK == 3) {
        const int64_t c0 = r.org[0] + wave;
        t = __builtin_amdgcn_raw_buffer_load_b32(words_rsrc(w, k.words, cx + c0 * k.n[1] + r.org[1]), 4u * (uint32_t)(lane & 31), 0, 0);
        load4(words_rsrc(w, k.words, k.off[1] + (r.org[1] >> k.sh[1]) * k.nlines[1] + c0 * k.n[2] + r.org[2]),
              16u * (uint32_t)(lane & 15), 0, y);
    }
#pragma unroll
    for (int j = 0; j < kRuns; j++) load4(rs, r.voff, r.step * j, v[j]);
#pragma unroll
    for (int j = 0; j < kRuns; j++) {
        const uint32_t u = row_term<RANK>(t, wave, j, lane);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int q = (int)(v[j][e] + (RANK == 3 ? y[e] + A[j][e] : RANK == 2 ? A[0][e] : 0u) + u);
            v[j][e] = __float_as_uint(pw ? pw_dequant(q, step) : (float)q * ebx2);
        }
        store_run<RANK, STREAM>(rs, r, wave, j, lane, v[j]);
    }
}

// A rejected stream (header or chunk check) sets d_err; the output is then
// unspecified (the carry passes run on whatever the chunk kernel left).
__global__ void k_clear_err_g(uint32_t* p)
{
    if (threadIdx.x == 0) *p = 0u;
}

template <int RANK, bool STREAM>
static hipError_t launch_rank_int(const uint8_t* s, uint64_t sb, int32_t* y, const Geom& g, uint32_t* d_err,
                                  hipStream_t st)
{
    return launch_chunks(g.n_chunks, [&](uint32_t first, dim3 blocks) {
        hipLaunchKernelGGL((k_decompress_int<RANK, STREAM>), blocks, dim3(512), 0, st, s, sb, y, g, d_err, first);
    });
}

template <int RANK>
static hipError_t launch_final(uint32_t* f, const uint32_t* w, const Carries& k, const Geom& g, const uint8_t* s,
                               bool stream, hipStream_t st)
{
    return launch_chunks(g.n_chunks, [&](uint32_t first, dim3 blocks) {
        if (stream) hipLaunchKernelGGL((k_seg_final<RANK, true>), blocks, dim3(kRunThreads), 0, st, f, w, k, g, s, first);
        else hipLaunchKernelGGL((k_seg_final<RANK, false>), blocks, dim3(kRunThreads), 0, st, f, w, k, g, s, first);
    });
}

// Threads per line: enough for one pass over its segments, but at least 16
// lines side by side where there are as many (the loads of neighbouring lines
// share cache lines).
template <int AX>
static hipError_t launch_carry(const uint32_t* f, uint32_t* w, const Carries& k, hipStream_t st)
{
    const int64_t nl = k.nlines[AX];
    int lg = 8;
    while (lg > 0 && 2 * (int64_t)(kGlobalThreads >> lg) < k.nseg[AX] && (lg > 4 || (nl >> (lg - 1)) < 1)) lg--;
    int64_t blocks = ((nl - 1) >> lg) + 1;
    if (blocks > (1 << 18)) blocks = 1 << 18;
    hipLaunchKernelGGL(k_seg_carry<AX>, dim3((unsigned)blocks), dim3(kGlobalThreads), 0, st, f, w, k, lg);
    return hipGetLastError();
}

size_t global_work_bytes(const Geom& g)
{
    return (size_t)(4 * carries_of(g).words);
}

hipError_t launch_decompress_global(const uint8_t* s, uint64_t sb, float* y, const Geom& g, uint32_t* d_err, void* work,
                                    hipStream_t st)
{
    hipError_t e;
    if (d_err) {
        hipLaunchKernelGGL(k_clear_err_g, dim3(1), dim3(64), 0, st, d_err);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    int32_t* yi = reinterpret_cast<int32_t*>(y);
    const bool stream = stream_stores(y, g, 4);
    switch (g.rank * 2 + (stream ? 1 : 0)) {
        case 7: e = launch_rank_int<3, true>(s, sb, yi, g, d_err, st); break;
        case 6: e = launch_rank_int<3, false>(s, sb, yi, g, d_err, st); break;
        case 5: e = launch_rank_int<2, true>(s, sb, yi, g, d_err, st); break;
        case 4: e = launch_rank_int<2, false>(s, sb, yi, g, d_err, st); break;
        case 3: e = launch_rank_int<1, true>(s, sb, yi, g, d_err, st); break;
        default: e = launch_rank_int<1, false>(s, sb, yi, g, d_err, st); break;
    }
    if (e != hipSuccess) return e;
    uint32_t* f = reinterpret_cast<uint32_t*>(y);
    uint32_t* w = static_cast<uint32_t*>(work);
    const Carries k = carries_of(g);
    // the contiguous axis first, then the middle, then the slowest
    if ((e = launch_carry<2>(f, w, k, st)) != hipSuccess) return e;
    if (g.rank >= 2 && (e = launch_carry<1>(f, w, k, st)) != hipSuccess) return e;
    if (g.rank == 3 && (e = launch_carry<0>(f, w, k, st)) != hipSuccess) return e;
    switch (g.rank) {
        case 3: return launch_final<3>(f, w, k, g, s, stream, st);
        case 2: return launch_final<2>(f, w, k, g, s, stream, st);
        default: return launch_final<1>(f, w, k, g, s, stream, st);
    }
}

}  // namespace fz
