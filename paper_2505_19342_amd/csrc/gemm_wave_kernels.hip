// The wavefront-private product kernel's instantiations for the attention layer's own launches (gemm_bf16_wave.h).
#include "gemm_bf16_wave.h"

namespace astra {

template <int MT, int NT, int ST>
static constexpr WaveConfig wave_config() {
    using S = WaveShape<MT, NT, ST>;
    return {S::BM, S::BN, S::kBytes, S::kBytes <= 80 * 1024 ? 2 : 1};
}
const WaveConfig kWaveTable[kWaveConfigs] = {wave_config<1, 1, 2>(), wave_config<2, 1, 2>(), wave_config<2, 2, 2>(),
                                             wave_config<2, 2, 1>(), wave_config<4, 2, 1>(), wave_config<4, 4, 1>()};

int launch_gemm_wave(int cfg, int epi, bool gather, const GemmBatch& batch, int grid, int code_lds, hipStream_t s) {
    if (epi != kEpiLayer) return batch.n_enc_wgs > 0 || gather ? ASTRA_ERR_UNSUPPORTED : launch_gemm_wave_mlp(cfg, epi, batch, grid, s);
    return with_wave_config(cfg, [&](auto mt, auto nt, auto st) {
        constexpr int MT = decltype(mt)::value, NT = decltype(nt)::value, ST = decltype(st)::value;
        if (batch.n_enc_wgs > 0)
            return gather ? launch_wave_form<MT, NT, ST, true, true, kEpiLayer>(batch, grid, code_lds, s)
                          : launch_wave_form<MT, NT, ST, false, true, kEpiLayer>(batch, grid, code_lds, s);
        return gather ? launch_wave_form<MT, NT, ST, true, false, kEpiLayer>(batch, grid, code_lds, s)
                      : launch_wave_form<MT, NT, ST, false, false, kEpiLayer>(batch, grid, code_lds, s);
    });
}

}  // namespace astra
