// gemvt.hip -- the launches of X~' r with the fused proximal epilogue (the
// phases themselves are in gemvt_dev.h).
#include "gemvt_dev.h"

namespace cox {
namespace {

using namespace gemvtdev;

constexpr int64_t kFewWorkgroups = 512;

template <int XT, int NB, bool VEC, int CPW>
__global__ __launch_bounds__(kGemvtThreads) void gemvt_sums_kernel(GemvtArgs a)
{
    __shared__ __attribute__((aligned(16))) float sr[NB * chunk_rows<NB>()];
    gemvt_sums_blk<XT, NB, VEC, CPW>(a, blockIdx.x, blockIdx.y, sr);
}

template <int CB>
__global__ __launch_bounds__(256) void gemvt_epilogue_kernel(GemvtArgs a)
{
    __shared__ int flag[CB];
    gemvt_epilogue_blk<CB>(a, blockIdx.x, flag);
}

template <int CB>
hipError_t launch_epilogue(const GemvtArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(gemvt_epilogue_kernel<CB>, dim3((unsigned)((a.x.p + CB - 1) / CB)), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int XT, int NB, int CPW>
hipError_t launch_cols(const GemvtArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)((a.x.p + 4 * CPW - 1) / (4 * CPW)), (unsigned)a.nsplit);
    if (a.x.vec16)
        hipLaunchKernelGGL((gemvt_sums_kernel<XT, NB, true, CPW>), grid, dim3(kGemvtThreads), 0, s, a);
    else
        hipLaunchKernelGGL((gemvt_sums_kernel<XT, NB, false, CPW>), grid, dim3(kGemvtThreads), 0, s, a);
    return hipGetLastError();
}

template <int XT, int NB>
hipError_t launch_t(const GemvtArgs& a, hipStream_t s)
{
    constexpr int CPW = cols_per_wave<XT, NB>();
    // fewer than two workgroups per compute unit: four columns a wavefront shorten each one's work
    const int64_t wgs = (a.x.p + 4 * CPW - 1) / (4 * CPW) * a.nsplit;
    if (CPW > 4 && wgs < kFewWorkgroups) return launch_cols<XT, NB, 4>(a, s);
    return launch_cols<XT, NB, CPW>(a, s);
}

template <int XT>
hipError_t launch_x(const GemvtArgs& a, hipStream_t s)
{
    if (a.nb <= 1) return launch_t<XT, 1>(a, s);
    if (a.nb <= 2) return launch_t<XT, 2>(a, s);
    if (a.nb <= 4) return launch_t<XT, 4>(a, s);
    return launch_t<XT, 8>(a, s);
}

}  // namespace

hipError_t launch_gemvt_epilogue(const GemvtArgs& a, hipStream_t s)
{
    if (a.nb < 1 || a.nsplit < 1) return hipErrorInvalidValue;
    // Up to 7 vectors: one thread per column.  More: 8 or 16 threads share a
    // column's vectors, so that few columns still fill the chip and many keep
    // more loads in flight (64 vectors: 701 columns 8.1 us with 16 threads per
    // column, 13.1 with 8, 73.7 with one; 62,500 columns 43.3, 36.4 and 103.5 us)
    if (a.nb < 8) return launch_epilogue<256>(a, s);
    return a.x.p < 32768 ? launch_epilogue<16>(a, s) : launch_epilogue<32>(a, s);
}

hipError_t launch_gemvt_sums(const GemvtArgs& a, hipStream_t s)
{
    if (a.nb < 1 || a.nb > 8 || a.nsplit < 1 || a.split_rows % kSplitRows != 0) return hipErrorInvalidValue;
    switch (a.x.xt) {
    case XT_F32: return launch_x<XT_F32>(a, s);
    case XT_FP8: return launch_x<XT_FP8>(a, s);
    default: return launch_x<XT_I8>(a, s);
    }
}

hipError_t launch_gemvt(const GemvtArgs& a, hipStream_t s)
{
    const hipError_t e = launch_gemvt_sums(a, s);
    if (e != hipSuccess) return e;
    return launch_gemvt_epilogue(a, s);
}

}  // namespace cox
