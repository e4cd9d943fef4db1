// Many-step fitting kernels of degrees 13..15.
#include "fit_impl.h"

namespace bzi {
template int launch_fit_run_d<13>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<14>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<15>(int, const FitArgs &, const FitBias &, int, hipStream_t);
}  // namespace bzi
