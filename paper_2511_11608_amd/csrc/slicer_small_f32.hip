#include "slicer_launch_small.hpp"

namespace slicer {
template <> hipError_t launch_small<0, false, 7>(const SmallArgs& sa, const SmallLaunch& p, hipStream_t st) { return launch_small_all<0, false, 7>(sa, p, st); }
}  // namespace slicer
