// The argmin over the scores of a wide group's encode, as a device function: a kernel of its own, or workgroups of the pass that looks up pre-projected codebooks.
#pragma once
#include "common.h"

namespace astra {

// codes[row] = argmin_k cnorm[g, k] - 2 scores[row, k], lowest k on ties; a wavefront per row (token, group), K a multiple of 4; 256 threads
template <typename CodeT>
__device__ __forceinline__ void vq_argmin_scores_rows(const float* __restrict__ scores, const float* __restrict__ cnorm, CodeT* __restrict__ codes,
                                                      int64_t n_rows, int G, int K, int block) {
    const int64_t row = ((int64_t)block * 256 + threadIdx.x) / kWave;             // (token, group)
    if (row >= n_rows) return;
    const int lane = lane_id();
    const int g = (int)(row % G);
    const float* __restrict__ sr = scores + row * K;
    const float* __restrict__ cn = cnorm + (int64_t)g * K;
    float best = INFINITY;
    int arg = 0x7fffffff;
    for (int k0 = 4 * lane; k0 < K; k0 += 4 * kWave) {                         // K is a multiple of 4
        const f32x4 sv = *reinterpret_cast<const f32x4*>(sr + k0);
        const f32x4 cv = *reinterpret_cast<const f32x4*>(cn + k0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d = fmaf(-2.f, sv[e], cv[e]);
            if (d < best) { best = d; arg = k0 + e; }
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best, off);
        const int oa = __shfl_xor(arg, off);
        if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
    }
    if (lane == 0) codes[row] = (CodeT)arg;
}

}  // namespace astra
