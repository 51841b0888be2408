#include "slicer_launch_wg.hpp"

namespace slicer {
template <> hipError_t launch_wg<0, true>(const SmallArgs& sa, const WgLaunch& p, hipStream_t st) { return launch_wg_all<0, true>(sa, p, st); }
}  // namespace slicer
