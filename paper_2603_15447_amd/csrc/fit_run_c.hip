// Many-step fitting kernels of degrees 10..12.
#include "fit_impl.h"

namespace bzi {
template int launch_fit_run_d<10>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<11>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<12>(int, const FitArgs &, const FitBias &, int, hipStream_t);
}  // namespace bzi
