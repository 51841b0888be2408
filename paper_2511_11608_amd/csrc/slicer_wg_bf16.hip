#include "slicer_launch_wg.hpp"

namespace slicer {
template <> hipError_t launch_wg<1, false>(const SmallArgs& sa, const WgLaunch& p, hipStream_t st) { return launch_wg_all<1, false>(sa, p, st); }
}  // namespace slicer
