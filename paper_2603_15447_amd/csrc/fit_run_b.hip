// Many-step fitting kernels of degrees 6..9.
#include "fit_impl.h"

namespace bzi {
template int launch_fit_run_d<6>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<7>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<8>(int, const FitArgs &, const FitBias &, int, hipStream_t);
template int launch_fit_run_d<9>(int, const FitArgs &, const FitBias &, int, hipStream_t);
}  // namespace bzi
