// Dispatch of the one-wavefront-per-row kernel over its register layouts (included by the translation
// units that instantiate it).
#pragma once

#include "slicer_launch.hpp"

namespace slicer {

template <int DT, int EPL, bool ASYM, int NQ>
void launch_small_epl(const SmallArgs& sa, const SmallLaunch& p, hipStream_t st)
{
    const dim3 g((unsigned)xcd_grid(sa.R)), b(kWave);
    const size_t lds = (size_t)p.lds_bytes;
    if (p.maxs == 4) hipLaunchKernelGGL((enc_small_kernel<DT, EPL, NQ, 4, ASYM>), g, b, lds, st, sa);
    else if (p.maxs == 10) hipLaunchKernelGGL((enc_small_kernel<DT, EPL, NQ, 10, ASYM>), g, b, lds, st, sa);
    else if (p.maxs == 20) hipLaunchKernelGGL((enc_small_kernel<DT, EPL, NQ, 20, ASYM>), g, b, lds, st, sa);
    else hipLaunchKernelGGL((enc_small_kernel<DT, EPL, NQ, 0, ASYM>), g, b, lds, st, sa);
}

template <int DT, bool ASYM, int NQ>
hipError_t launch_small_all(const SmallArgs& sa, const SmallLaunch& p, hipStream_t st)
{
    constexpr int E0 = DT == 0 ? 4 : 16;      // smallest instantiated elements-per-lane
    if constexpr (DT == 0) {
        if (p.epl == 12 || p.epl == 20) {
            if (p.epl == 12) launch_small_epl<0, 12, ASYM, NQ>(sa, p, st);
            else launch_small_epl<0, 20, ASYM, NQ>(sa, p, st);
            return hipGetLastError();
        }
    }
    if (p.epl <= E0) launch_small_epl<DT, E0, ASYM, NQ>(sa, p, st);
    else if (p.epl == E0 * 2) launch_small_epl<DT, E0 * 2, ASYM, NQ>(sa, p, st);
    else if (p.epl == E0 * 4) launch_small_epl<DT, E0 * 4, ASYM, NQ>(sa, p, st);
    else if (p.epl == E0 * 8 || DT != 0) launch_small_epl<DT, E0 * 8, ASYM, NQ>(sa, p, st);
    else launch_small_epl<DT, DT == 0 ? E0 * 16 : E0 * 8, ASYM, NQ>(sa, p, st);   // fp32 rows of 4096
    return hipGetLastError();
}

}  // namespace slicer
