// fz_decompress.hip -- per-field decompression kernels of libfzmi (gfx950):
// a workgroup of 8 waves per chunk, of 16 for fields with few chunks, or of 8
// that reads ahead for fields with many, running the device code of
// fz_decompress_dev.hpp.
#include <hip/hip_runtime.h>

#include "fz_decompress_dev.hpp"
#include "fz_kernels.hpp"

namespace fz {

// 128 registers (4 waves per SIMD) and 72 KB of LDS: two workgroups per CU.
template <int RANK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress(const uint8_t* __restrict__ s, uint64_t sb,
                                                       float* __restrict__ y, Geom g, uint32_t* d_err)
{
    __shared__ DecompressLds<8> S;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    decompress_chunk<RANK, float, 8>(s, sb, y, STREAM, g, d_err, in_place_chunk<STREAM>(g, blockIdx.x), wave, threadIdx.x & 63, S);
}

// the same with NW waves, one step each (fields with few chunks; launched
// with NW = 16)
template <int RANK, bool STREAM, int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_decompress_split(const uint8_t* __restrict__ s, uint64_t sb,
                                                                 float* __restrict__ y, Geom g, uint32_t* d_err)
{
    __shared__ DecompressLds<NW> S;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    decompress_chunk<RANK, float, NW>(s, sb, y, STREAM, g, d_err, blockIdx.x, wave, threadIdx.x & 63, S);
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
static ThinLayer thin_layer(const Geom& g, uint32_t at_once)
{
    const ThinLayer none{(uint32_t)g.n_chunks, 3};
    if (g.rank == 1) return none;
    const int64_t e = g.n[0] - (g.grid[0] - 1) * g.box[0], steps = g.rank == 3 ? e : (e + 1) / 2;
    if (steps > 8) return none;
    const ThinLayer t{(uint32_t)(g.n_chunks - g.grid[1] * g.grid[2]), steps > 4 ? 2 : steps > 2 ? 1 : 0};
    const uint32_t last = t.full % at_once, room = t.full && !last ? 0u : at_once - last;
    return none.full - t.full > room ? t : none;
}

// k_decompress for fields of more chunks than are at work at once (`ahead`): a
// workgroup reads ahead for the chunk that takes its place, chunks are taken in
// turned_chunk's order, and a thin last layer shares workgroups.  first: the
// launch's first block of the field (launch_chunks).
template <int RANK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress_ahead(const uint8_t* __restrict__ s, uint64_t sb,
                                                             float* __restrict__ y, Geom g, uint32_t* d_err, uint32_t first,
                                                             uint32_t ahead, ThinLayer thin)
{
    __shared__ DecompressLds<8> S;
    int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = 8, w0 = 0;
    const uint32_t b = first + blockIdx.x;
    int64_t c, next = -1;
    if (b < thin.full) {
        c = turned_chunk<RANK, STREAM>(g, b, thin.full);
        if (b + ahead < thin.full) next = turned_chunk<RANK, STREAM>(g, b + ahead, thin.full);
    } else {
        const int lg = thin.lg, per = 8 >> lg;
        c = (int64_t)thin.full + (int64_t)(b - thin.full) * per + (wave >> lg);
        if (c >= g.n_chunks) return;
        if (c + (int64_t)ahead * per < g.n_chunks) next = c + (int64_t)ahead * per;
        waves = 1 << lg;
        w0 = wave & ~(waves - 1);
        wave -= w0;
    }
    decompress_chunk<RANK, float, 8, true>(s, sb, y, STREAM, g, d_err, c, wave, threadIdx.x & 63,
                                           *reinterpret_cast<DecompressLds<8>*>(S.region[w0]), next, waves);
}

__global__ void k_set_u32(uint32_t* p, uint32_t v)
{
    if (threadIdx.x == 0) *p = v;
}

// Fields of at most this many chunks (one workgroup per CU) are decompressed
// with 16 waves per chunk: a lone workgroup of 8 waves leaves a SIMD with two
// waves to hide each other's latency, one of 16 with four (128x128x256, 128
// chunks: 11.0 us against 11.2-12.0 us a pass).  Beyond, two workgroups of 8
// waves share a CU (256^3, 512 chunks: 21 us against 30 us).  Fields of more
// chunks than that take k_decompress_ahead; without a chunk to read ahead for it
// is the slower one (96x100352, 294 chunks: 12.8 us, ahead 14.8; 48x512x512, 384:
// 15.5 and 17.0).
constexpr int64_t kSplitChunks = 256;

template <int RANK, bool STREAM>
static hipError_t launch_rank(const uint8_t* s, uint64_t sb, float* y, const Geom& g, uint32_t* d_err, hipStream_t st)
{
    const dim3 all((unsigned)g.n_chunks);  // (fits one launch where it is used)
    if (g.n_chunks <= kSplitChunks) {
        hipLaunchKernelGGL((k_decompress_split<RANK, STREAM, 16>), all, dim3(1024), 0, st, s, sb, y, g, d_err);
        return hipGetLastError();
    }
    const uint32_t at_once = 2u * (uint32_t)cu_count();
    if (g.n_chunks <= at_once) {
        hipLaunchKernelGGL((k_decompress<RANK, STREAM>), all, dim3(512), 0, st, s, sb, y, g, d_err);
        return hipGetLastError();
    }
    const ThinLayer thin = thin_layer(g, at_once);
    return launch_chunks(thin.blocks(g), [&](uint32_t first, dim3 blocks) {
        hipLaunchKernelGGL((k_decompress_ahead<RANK, STREAM>), blocks, dim3(512), 0, st, s, sb, y, g, d_err, first, at_once, thin);
    });
}

hipError_t launch_decompress(const uint8_t* s, uint64_t sb, float* y, const Geom& g, uint32_t* d_err, hipStream_t st)
{
    if (d_err) {
        hipLaunchKernelGGL(k_set_u32, dim3(1), dim3(64), 0, st, d_err, 0u);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool stream = stream_stores(y, g, 4);
    switch (g.rank * 2 + (stream ? 1 : 0)) {
        case 7: return launch_rank<3, true>(s, sb, y, g, d_err, st);
        case 6: return launch_rank<3, false>(s, sb, y, g, d_err, st);
        case 5: return launch_rank<2, true>(s, sb, y, g, d_err, st);
        case 4: return launch_rank<2, false>(s, sb, y, g, d_err, st);
        case 3: return launch_rank<1, true>(s, sb, y, g, d_err, st);
        default: return launch_rank<1, false>(s, sb, y, g, d_err, st);
    }
}

}  // namespace fz
