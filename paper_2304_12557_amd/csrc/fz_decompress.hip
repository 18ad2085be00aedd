// fz_decompress.hip -- per-field decompression kernels of libfzmi (gfx950):
// a workgroup of 8 waves per chunk, or for fields with few chunks one of 16
// waves, running the device code of fz_decompress_dev.hpp.
#include <hip/hip_runtime.h>

#include "fz_decompress_dev.hpp"
#include "fz_kernels.hpp"

namespace fz {

// 128 registers (4 waves per SIMD) and 9 KB of LDS a wave: two workgroups per
// CU, or more where they have fewer waves (chunk_waves), whose regions are the
// launch's dynamic LDS.  first: the launch's first block of the field
// (launch_chunks); ahead: how many blocks are at work at once.
template <int RANK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress(const uint8_t* __restrict__ s, uint64_t sb,
                                                       float* __restrict__ y, Geom g, uint32_t* d_err, uint32_t first,
                                                       uint32_t ahead)
{
    extern __shared__ uint4 lds[];
    DecompressLds<8>& S = *reinterpret_cast<DecompressLds<8>*>(lds);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b = first + blockIdx.x;
    decompress_chunk<RANK, float, 8, true>(s, sb, y, STREAM, g, d_err, in_place_chunk<STREAM>(g, b), wave, threadIdx.x & 63, S,
                                           b + ahead < (uint64_t)g.n_chunks ? in_place_chunk<STREAM>(g, b + ahead) : -1);
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

__global__ void k_set_u32(uint32_t* p, uint32_t v)
{
    if (threadIdx.x == 0) *p = v;
}

// Fields of at most this many chunks (one workgroup per CU) are decompressed
// with 16 waves per chunk: a lone workgroup of 8 waves leaves a SIMD with two
// waves to hide each other's latency, one of 16 with four (128x128x256, 128
// chunks: 11.0 us against 11.2-12.0 us a pass).  Beyond, two workgroups of 8
// waves share a CU (256^3, 512 chunks: 21 us against 30 us).
constexpr int64_t kSplitChunks = 256;

// Waves of a chunk's workgroup, two steps each.  In a field of one layer of
// chunks that is thinner than they are (2-D, 3-D), all chunks have the same few
// steps, and waves without one would only hold LDS and wave slots (1x2048x2048:
// 8 waves 19.8 us, 1 wave 11.0; 4x2048x2048: 27.4, 2 waves 16.5).  Five to seven
// waves leave room for two or three workgroups a CU only: 8 waves there
// (12x1024x2048: 6 waves 31.6 us, 8 waves 27.2).
static int chunk_waves(const Geom& g)
{
    if (g.rank == 1 || g.grid[0] > 1) return 8;
    const int64_t steps = g.rank == 3 ? g.n[0] : (g.n[0] + 1) / 2;
    return steps <= 8 ? (int)((steps + 1) / 2) : 8;
}

template <int RANK, bool STREAM>
static hipError_t launch_rank(const uint8_t* s, uint64_t sb, float* y, const Geom& g, uint32_t* d_err, hipStream_t st)
{
    const int waves = chunk_waves(g);
    const uint32_t ahead = (uint32_t)(cu_count() * (16 / waves));
    return launch_chunks(g.n_chunks, [&](uint32_t first, dim3 blocks) {
        if (g.n_chunks <= kSplitChunks)
            hipLaunchKernelGGL((k_decompress_split<RANK, STREAM, 16>), blocks, dim3(1024), 0, st, s, sb, y, g, d_err);
        else
            hipLaunchKernelGGL((k_decompress<RANK, STREAM>), blocks, dim3(64 * waves), waves * 4 * kRegionWords, st, s, sb, y,
                               g, d_err, first, ahead);
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
