// Launchers of the per-stage decode kernels (one launch per stage).
#include "decode_device.hpp"

namespace lr {

template <int MB>
static int launch_stage(const DStage& st, bool a_f32, int epi, hipStream_t s) {
    const dim3 grid((unsigned)st.total_tiles), block(256);
    constexpr int PF = 3, CPL = 4;
    if (epi == EPI_ATOMIC) {
        if (a_f32) hipLaunchKernelGGL((k_decode_stage<MB, CPL, true, EPI_ATOMIC, PF>), grid, block, 0, s, st);
        else       hipLaunchKernelGGL((k_decode_stage<MB, CPL, false, EPI_ATOMIC, PF>), grid, block, 0, s, st);
    } else if (epi == EPI_STORE) {
        if (a_f32) hipLaunchKernelGGL((k_decode_stage<MB, CPL, true, EPI_STORE, PF>), grid, block, 0, s, st);
        else       hipLaunchKernelGGL((k_decode_stage<MB, CPL, false, EPI_STORE, PF>), grid, block, 0, s, st);
    } else {
        if (!a_f32) { set_error("gate/up stage expects the fp32 rank-space input"); return LR_ERR_UNSUPPORTED; }
        hipLaunchKernelGGL((k_decode_stage<MB, CPL, true, EPI_GATEUP, PF>), grid, block, 0, s, st);
    }
    return launch_status("decode stage");
}

int decode_launch_stage(const DStage& st, bool a_f32, int epi, hipStream_t s) {
    if (st.total_tiles <= 0 || st.M <= 0) return LR_OK;
    return st.M <= 16 ? launch_stage<1>(st, a_f32, epi, s) : launch_stage<2>(st, a_f32, epi, s);
}

}  // namespace lr
