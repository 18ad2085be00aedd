// fz_f64.hip -- the fp64-input front end and the fp64 decompression kernel
// of libfzmi (gfx950).
//
// fp64 fields are quantized in double precision (Sec. 2.3's quantizer with
// q = rint(x * inv), inv = 1 / (2 eb) as doubles) by a pass of their own,
// which writes the integers q (4 B per value) behind the fp32 bound of the
// output buffer; the compression kernel then reads q in place of fp32 values
// and the rest of the pipeline is unchanged.  REL mode first takes the value
// range in double (Sec. 4.1).  Decompression runs the fp32 kernel's device
// code with an fp64 dequantization and fp64 stores.
#include <hip/hip_runtime.h>

#include "fz.h"
#include "fz_compress_dev.hpp"
#include "fz_decompress_dev.hpp"
#include "fz_kernels.hpp"

namespace fz {

constexpr int kF64Threads = 256;

__device__ __forceinline__ bool finite64(double v) { return __builtin_fabs(v) <= 1.7976931348623157e308; }

// Partial range of block blk: min and max over the finite values (-0 as +0)
// and a flag for non-finite ones.  It also does k_init's work (a REL
// compression starts with it).
__global__ __launch_bounds__(kF64Threads) void k_minmax64(const double* __restrict__ x, int64_t n,
                                                         uint8_t* __restrict__ out, Geom g, HeaderImage h)
{
    __shared__ double s_lo[kF64Threads / 64], s_hi[kF64Threads / 64];
    __shared__ uint32_t s_bad[kF64Threads / 64];
    init_field(out, out + g.scratch_off, g, h, (int64_t)blockIdx.x * kF64Threads + threadIdx.x,
               (int64_t)gridDim.x * kF64Threads);
    double lo = __builtin_inf(), hi = -__builtin_inf();
    uint32_t bad = 0;
    auto take = [&](double v) {
        if (!finite64(v)) {
            bad = 1;
        } else {
            v = v == 0.0 ? 0.0 : v;
            lo = __builtin_fmin(lo, v);
            hi = __builtin_fmax(hi, v);
        }
    };
    const int64_t stride = (int64_t)gridDim.x * kF64Threads;
    const int64_t tid = (int64_t)blockIdx.x * kF64Threads + threadIdx.x;
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const int64_t n2 = vec ? n / 2 : 0;
    const fz_f64x2* x2 = reinterpret_cast<const fz_f64x2*>(x);
    for (int64_t i = tid; i < n2; i += stride) {
        const fz_f64x2 v = __builtin_nontemporal_load(x2 + i);
        take(v.x);
        take(v.y);
    }
    for (int64_t k = 2 * n2 + tid; k < n; k += stride) take(x[k]);
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
        lo = __builtin_fmin(lo, __shfl_xor(lo, sh));
        hi = __builtin_fmax(hi, __shfl_xor(hi, sh));
        bad |= (uint32_t)__shfl_xor((int)bad, sh);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { s_lo[w] = lo; s_hi[w] = hi; s_bad[w] = bad; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kF64Threads / 64; i++) {
            lo = __builtin_fmin(lo, s_lo[i]);
            hi = __builtin_fmax(hi, s_hi[i]);
            bad |= s_bad[i];
        }
        double* part = reinterpret_cast<double*>(out + g.part64_off);
        part[2 * blockIdx.x] = lo;
        part[2 * blockIdx.x + 1] = hi;
        reinterpret_cast<uint32_t*>(out + g.part64_off + 16 * kMinmaxBlocks)[blockIdx.x] = bad;
    }
}

// Fold the partials and derive 2 eb_abs and its reciprocal in double, by a whole
// block; the same result on every thread.
struct Params64 {
    uint32_t status;  // 0, kErrNonfinite or kErrEbRange
    double e2, inv, lo, hi;
};
__device__ __forceinline__ Params64 fold_params64(const uint8_t* __restrict__ out, const Geom& g, double eb, int nparts)
{
    __shared__ double s_lo[kF64Threads / 64], s_hi[kF64Threads / 64];
    __shared__ uint32_t s_bad[kF64Threads / 64];
    const double* part = reinterpret_cast<const double*>(out + g.part64_off);
    const uint32_t* pbad = reinterpret_cast<const uint32_t*>(out + g.part64_off + 16 * kMinmaxBlocks);
    double lo = __builtin_inf(), hi = -__builtin_inf();
    uint32_t bad = 0;
    for (int i = threadIdx.x; i < nparts; i += kF64Threads) {
        lo = __builtin_fmin(lo, part[2 * i]);
        hi = __builtin_fmax(hi, part[2 * i + 1]);
        bad |= pbad[i];
    }
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) {
        lo = __builtin_fmin(lo, __shfl_xor(lo, sh));
        hi = __builtin_fmax(hi, __shfl_xor(hi, sh));
        bad |= (uint32_t)__shfl_xor((int)bad, sh);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { s_lo[w] = lo; s_hi[w] = hi; s_bad[w] = bad; }
    __syncthreads();
    lo = s_lo[0], hi = s_hi[0], bad = s_bad[0];
    for (int i = 1; i < kF64Threads / 64; i++) {
        lo = __builtin_fmin(lo, s_lo[i]);
        hi = __builtin_fmax(hi, s_hi[i]);
        bad |= s_bad[i];
    }
    uint32_t status = 0;
    double e2 = 0.0, iv = 0.0;
    if (bad) {
        status = kErrNonfinite;
    } else {
        const double range = hi - lo;
        double eb_abs;
        if (range > 0.0) eb_abs = eb * range;
        else {
            const double a = __builtin_fabs(hi);
            eb_abs = eb * (a > 0.0 ? a : 1.0);
        }
        e2 = 2.0 * eb_abs;
        iv = 1.0 / e2;
        if (!(e2 >= 2.2250738585072014e-308) || !finite64(e2) || !finite64(iv) || !(iv > 0.0)) {
            status = kErrEbRange;
            e2 = 0.0;
            iv = 0.0;
        }
    }
    return Params64{status, e2, iv, lo, hi};
}

// The parameters (and their fp32 roundings, with the range's) to the header.  A
// non-finite value or an unusable bound ends the pipeline here: the status goes
// to the header, the stream to its header size.
__device__ __forceinline__ void write_params64(uint8_t* __restrict__ out, const Geom& g, const Params64& r)
{
    *reinterpret_cast<float*>(out + kOffEbx2) = (float)r.e2;
    *reinterpret_cast<float*>(out + kOffInv) = (float)r.inv;
    *reinterpret_cast<float*>(out + kOffVmin) = (float)r.lo;
    *reinterpret_cast<float*>(out + kOffVmax) = (float)r.hi;
    *reinterpret_cast<double*>(out + kOffEbx2F64) = r.e2;
    *reinterpret_cast<double*>(out + kOffInvF64) = r.inv;
    if (r.status) {
        *reinterpret_cast<uint32_t*>(out + kOffStatus) = r.status;
        *reinterpret_cast<uint64_t*>(out + kOffTotal) = (uint64_t)g.payload_off;
    }
}

// q = (int32) rint(x * inv) in double, round half to even, into the integer
// buffer; NaN/Inf and |x * inv| >= 2^31 set the status bits and end the
// pipeline (the compression kernel sees the status).  rel_eb > 0: a REL
// compression whose range pass left nparts partials; every block folds them
// itself and block 0 writes the parameters, so that no launch of its own sits
// between the two passes (4.8 us).
__global__ __launch_bounds__(kF64Threads) void k_prequant64(const double* __restrict__ x, int64_t n,
                                                           uint8_t* __restrict__ out, Geom g, double rel_eb, int nparts)
{
    __shared__ uint32_t s_err[kF64Threads / 64];
    double inv;
    if (rel_eb > 0.0) {
        const Params64 r = fold_params64(out, g, rel_eb, nparts);
        if (blockIdx.x == 0 && threadIdx.x == 0) write_params64(out, g, r);
        if (r.status) return;  // the same in every block
        inv = r.inv;
    } else {
        inv = *reinterpret_cast<const double*>(out + kOffInvF64);
    }
    int32_t* q = reinterpret_cast<int32_t*>(out + g.q_off);
    uint32_t err = 0;
    auto quant = [&](double v) -> int32_t {
        if (!finite64(v)) { err |= kErrNonfinite; return 0; }
        const double p = v * inv;
        if (!(__builtin_fabs(p) < 2147483648.0)) { err |= kErrEbRange; return 0; }
        return (int32_t)__builtin_rint(p);
    };
    const int64_t stride = (int64_t)gridDim.x * kF64Threads;
    const int64_t tid = (int64_t)blockIdx.x * kF64Threads + threadIdx.x;
    // 16-byte loads at any 8-byte alignment, which the hardware takes: with one
    // load a value where x is not 16-byte aligned, these few blocks do not keep
    // enough in flight (100x500x500 ABS, whole compression: 115 us, now 100;
    // aligned 97).  q's buffer is 256-aligned.
    typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));
    const int64_t n4 = n / 4;
    for (int64_t i = tid; i < n4; i += stride) {
        const f64x2 a = __builtin_nontemporal_load(reinterpret_cast<const f64x2*>(x) + 2 * i);
        const f64x2 b = __builtin_nontemporal_load(reinterpret_cast<const f64x2*>(x) + 2 * i + 1);
        *reinterpret_cast<int4*>(q + 4 * i) = make_int4(quant(a.x), quant(a.y), quant(b.x), quant(b.y));
    }
    for (int64_t k = 4 * n4 + tid; k < n; k += stride) q[k] = quant(x[k]);
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) err |= (uint32_t)__shfl_xor((int)err, sh);
    if ((threadIdx.x & 63) == 0) s_err[threadIdx.x >> 6] = err;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kF64Threads / 64; i++) err |= s_err[i];
        if (err) {
            atomicOr(reinterpret_cast<uint32_t*>(out + kOffStatus), err);
            // every failing block writes the same size: the header alone
            *reinterpret_cast<uint64_t*>(out + kOffTotal) = (uint64_t)g.payload_off;
        }
    }
}

hipError_t launch_f64_front(const double* x, uint8_t* out, const Geom& g, const HeaderImage& h, int mode, double eb,
                            hipStream_t st)
{
    const int64_t n = g.n[0] * g.n[1] * g.n[2];
    hipError_t e;
    int nparts = 0;
    if (mode == FZ_EB_REL) {
        int64_t blocks = (n / 2 + kF64Threads - 1) / kF64Threads;
        blocks = blocks < 1 ? 1 : blocks > kMinmaxBlocks ? kMinmaxBlocks : blocks;
        hipLaunchKernelGGL(k_minmax64, dim3((unsigned)blocks), dim3(kF64Threads), 0, st, x, n, out, g, h);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        nparts = (int)blocks;
    } else if ((e = launch_init(out, out + g.scratch_off, g, h, st)) != hipSuccess) {
        return e;
    }
    // blocks that stay resident, as each folds the range (100x500x500 REL round
    // trip: 4096 blocks 193.6 us, 2048 191.0, 1024 188.7)
    int64_t blocks = (n / 4 + kF64Threads - 1) / kF64Threads;
    blocks = blocks < 1 ? 1 : blocks > 1024 ? 1024 : blocks;
    hipLaunchKernelGGL(k_prequant64, dim3((unsigned)blocks), dim3(kF64Threads), 0, st, x, n, out, g, nparts ? eb : 0.0, nparts);
    return hipGetLastError();
}

// ------------------------------------------------------------ decompression
template <int RANK, bool STREAM>
__global__ __launch_bounds__(512, 4) void k_decompress64(const uint8_t* __restrict__ s, uint64_t sb, double* __restrict__ y,
                                                         Geom g, uint32_t* d_err)
{
    __shared__ DecompressLds<8> S;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    decompress_chunk<RANK, double, 8>(s, sb, y, STREAM, g, d_err, xcd_order(blockIdx.x, g.n_chunks), wave, threadIdx.x & 63, S);
}

__global__ void k_clear_err(uint32_t* p)
{
    if (threadIdx.x == 0) *p = 0u;
}

template <int RANK, bool STREAM>
static hipError_t launch_rank64(const uint8_t* s, uint64_t sb, double* y, const Geom& g, uint32_t* d_err, hipStream_t st)
{
    // (a small field does not ask for the device's size)
    const uint32_t at_once = g.n_chunks > 256 ? 2u * (uint32_t)cu_count() : 512u;
    if (g.n_chunks > at_once) return launch_ahead<RANK, double, STREAM>(s, sb, y, g, d_err, at_once, st);
    hipLaunchKernelGGL((k_decompress64<RANK, STREAM>), dim3((unsigned)g.n_chunks), dim3(512), 0, st, s, sb, y, g, d_err);
    return hipGetLastError();
}

hipError_t launch_decompress_f64(const uint8_t* s, uint64_t sb, double* y, const Geom& g, uint32_t* d_err,
                                 hipStream_t st)
{
    if (d_err) {
        hipLaunchKernelGGL(k_clear_err, dim3(1), dim3(64), 0, st, d_err);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool stream = stream_stores(y, g, 8);
    switch (g.rank * 2 + (stream ? 1 : 0)) {
        case 7: return launch_rank64<3, true>(s, sb, y, g, d_err, st);
        case 6: return launch_rank64<3, false>(s, sb, y, g, d_err, st);
        case 5: return launch_rank64<2, true>(s, sb, y, g, d_err, st);
        case 4: return launch_rank64<2, false>(s, sb, y, g, d_err, st);
        case 3: return launch_rank64<1, true>(s, sb, y, g, d_err, st);
        default: return launch_rank64<1, false>(s, sb, y, g, d_err, st);
    }
}

}  // namespace fz
