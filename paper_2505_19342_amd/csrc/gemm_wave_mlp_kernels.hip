// The wavefront-private product kernel's instantiations for the block around the attention layer (gemm_bf16_wave.h).
#include "gemm_bf16_wave.h"

namespace astra {

int launch_gemm_wave_mlp(int cfg, int epi, const GemmBatch& batch, int grid, hipStream_t s) {
    return with_wave_config(cfg, [&](auto mt, auto nt, auto st) {
        constexpr int MT = decltype(mt)::value, NT = decltype(nt)::value, ST = decltype(st)::value;
        switch (epi) {
            case kEpiResidualF32: return launch_wave_form<MT, NT, ST, false, false, kEpiResidualF32>(batch, grid, 0, s);
            case kEpiGeluTanh: return launch_wave_form<MT, NT, ST, false, false, kEpiGeluTanh>(batch, grid, 0, s);
            case kEpiGeluErf: return launch_wave_form<MT, NT, ST, false, false, kEpiGeluErf>(batch, grid, 0, s);
            case kEpiSwiGLU: return launch_wave_form<MT, NT, ST, false, false, kEpiSwiGLU>(batch, grid, 0, s);
            default: return (int)ASTRA_ERR_UNSUPPORTED;
        }
    });
}

}  // namespace astra
