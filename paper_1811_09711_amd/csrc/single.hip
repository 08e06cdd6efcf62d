// Instantiations of the single-job sample kernel for one precision
// (MCV_SINGLE_FP32), dimension bucket (MCV_SINGLE_D) and generator
// (MCV_SINGLE_RNG: 0 Philox words, 1 MRG32k3a streams, Sec. 4.4, eq. mrg32k3a
// and eq. rngstream), with an exact-dimension variant where the problem's
// dimension is the bucket (no per-axis guards), and the trace instantiations
// of the same code path (lookup groups, skips, launch bounds) that write each
// call's f, g and w for a window of calls.  The build compiles this file once
// per combination, so that they compile in parallel.
#include <type_traits>

#include "sample_kernel.h"

#if !defined(MCV_SINGLE_FP32) || !defined(MCV_SINGLE_D) || !defined(MCV_SINGLE_RNG)
#error "single.hip is compiled with MCV_SINGLE_FP32, MCV_SINGLE_D and MCV_SINGLE_RNG defined"
#endif

namespace mcv {

namespace {
using ST = std::conditional_t<MCV_SINGLE_FP32 != 0, float, double>;
constexpr int kD = MCV_SINGLE_D, kR = MCV_SINGLE_RNG;
}  // namespace

Split MCV_SINGLE_NAME(launch, MCV_SINGLE_FP32, MCV_SINGLE_D, MCV_SINGLE_RNG)(
    const JobDev& j, int64_t n_points, hipStream_t s) {
  return j.d == kD ? launch_sample_t<ST, kD, true, kR>(j, n_points, s)
                   : launch_sample_t<ST, kD, false, kR>(j, n_points, s);
}

Split MCV_SINGLE_NAME(trace, MCV_SINGLE_FP32, MCV_SINGLE_D, MCV_SINGLE_RNG)(
    const JobDev& j, int64_t n_points, uint32_t tag, int64_t first, int64_t count, double* out,
    hipStream_t s) {
  return j.d == kD ? launch_sample_trace_t<ST, kD, true, kR>(j, n_points, tag, first, count, out, s)
                   : launch_sample_trace_t<ST, kD, false, kR>(j, n_points, tag, first, count, out, s);
}

}  // namespace mcv
