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
    return launch_ahead<RANK, float, STREAM>(s, sb, y, g, d_err, at_once, st);
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
