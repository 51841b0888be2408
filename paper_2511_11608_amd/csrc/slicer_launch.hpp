// Launchers of the two row-resident kernel families.  Each family is instantiated for many register
// layouts, so every element type, rule and kind of bitwidth set has a translation unit of its own (they compile in parallel).
#pragma once

#include "slicer_encode_small.hpp"

namespace slicer {

// elements per lane, LDS bytes, register slots of the list: see make_plan
struct SmallLaunch { int epl, lds_bytes, maxs; };
// wavefronts per row, 16-byte chunks per thread, LDS bytes
struct WgLaunch { int nw, chunks, lds_bytes; };

// NQ = 7: sets of seven bitwidths ({2..8} is the benchmarked one); NQ = 0: any other set
template <int DT, bool ASYM, int NQ> hipError_t launch_small(const SmallArgs& sa, const SmallLaunch& p, hipStream_t st);
template <int DT, bool ASYM> hipError_t launch_wg(const SmallArgs& sa, const WgLaunch& p, hipStream_t st);

}  // namespace slicer
