#include "slicer_launch_small.hpp"

namespace slicer {
template <> hipError_t launch_small<1, true, 7>(const SmallArgs& sa, const SmallLaunch& p, hipStream_t st) { return launch_small_all<1, true, 7>(sa, p, st); }
}  // namespace slicer
