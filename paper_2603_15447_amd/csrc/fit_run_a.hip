// Many-step fitting kernels of degrees 1..5.
#include "fit_impl.h"

namespace bzi {
template int launch_fit_run_d<1>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<2>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<3>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<4>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<5>(int, const FitArgs &, const FitBias &, int, hipStream_t);
}  // namespace bzi
