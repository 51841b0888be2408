// Dispatch of the workgroup-per-row kernel (included by the translation units that instantiate it).
#pragma once

#include "slicer_launch.hpp"
#include "slicer_encode_wg.hpp"

namespace slicer {

// p.chunks: 16-byte chunks per thread (1..16; at most 64 chunk totals for the one-wavefront scan: 4 with 16 wavefronts)
template <int DT, int NQ, bool ASYM>
void launch_wg_nq(const SmallArgs& sa, const WgLaunch& p, hipStream_t st)
{
    constexpr int EPC = DT == 0 ? 4 : 8;
    const dim3 g((unsigned)sa.R), b((unsigned)(p.nw * kWave));
    const size_t lds = (size_t)p.lds_bytes;
    if (p.nw == 16) {
        if (p.chunks <= 1) hipLaunchKernelGGL((enc_wg_kernel<DT, 16, 1 * EPC, NQ, ASYM>), g, b, lds, st, sa);
        else if (p.chunks == 2) hipLaunchKernelGGL((enc_wg_kernel<DT, 16, 2 * EPC, NQ, ASYM>), g, b, lds, st, sa);
        else hipLaunchKernelGGL((enc_wg_kernel<DT, 16, 4 * EPC, NQ, ASYM>), g, b, lds, st, sa);
    } else {
        if (p.chunks <= 4) hipLaunchKernelGGL((enc_wg_kernel<DT, 4, 4 * EPC, NQ, ASYM>), g, b, lds, st, sa);
        else if (p.chunks == 8) hipLaunchKernelGGL((enc_wg_kernel<DT, 4, 8 * EPC, NQ, ASYM>), g, b, lds, st, sa);
        else hipLaunchKernelGGL((enc_wg_kernel<DT, 4, 16 * EPC, NQ, ASYM>), g, b, lds, st, sa);
    }
}

template <int DT, bool ASYM>
hipError_t launch_wg_all(const SmallArgs& sa, const WgLaunch& p, hipStream_t st)
{
    if (sa.nq == 7) launch_wg_nq<DT, 7, ASYM>(sa, p, st); else launch_wg_nq<DT, 0, ASYM>(sa, p, st);
    return hipGetLastError();
}

}  // namespace slicer
