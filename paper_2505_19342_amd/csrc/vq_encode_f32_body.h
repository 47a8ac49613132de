// fp32 encode (paper Sec. 2 "Grouped VQ": nearest codeword per group, lowest index on ties), as a device function of one workgroup, so that it
// can run as a kernel of its own and as extra workgroups of the fp32 attention.
#pragma once
#include "vq_encode_body.h"

namespace astra {

// ------------------------------------------------------------------------------------------------
// A workgroup of 256 threads takes kEncF32Tokens tokens of one group; a thread takes every 256th codeword and forms its squared distances to all of
// them, sum (x - c)^2 in ascending order.  Bound by the round trip of the codeword loads: up to 64 values of a codeword are requested at once
// (16-byte loads where the slices allow it) and serve every token, whose values wait in LDS.  Values beyond the group are zeros on both sides: they
// add fma(0, 0, d) = d, and the work of a chunk has no branch.  64 tokens x 4 groups of 48, K = 256, back to back: 7.5 us with a wavefront per token and
// group, whose lanes took four codewords one after the other, 32 values and then 4 at a time; 4.4 now.
// ------------------------------------------------------------------------------------------------
constexpr int kEncF32Tokens = 4;
constexpr int kEncF32Threads = 256;
constexpr int kEncF32Staged = 512;         // values of a token's slice that LDS holds; longer slices are read from memory
struct EncF32Lds {
    f32x4 x[kEncF32Tokens][kEncF32Staged / 4];
    float best[kEncF32Threads / kWave][kEncF32Tokens];
    int arg[kEncF32Threads / kWave][kEncF32Tokens];
};

// item = group * token blocks + token block
__device__ __forceinline__ void vq_encode_f32_body(const EncodeJob& job, int64_t item, EncF32Lds& lds) {
    constexpr int NT = kEncF32Tokens, WAVES = kEncF32Threads / kWave;
    const int g = (int)(item / job.n_tb), t0 = (int)(item - (int64_t)g * job.n_tb) * NT;
    const int K = job.K, dg = job.dg, tid = threadIdx.x;
    const bool staged = dg % 4 == 0 && dg <= kEncF32Staged && (uintptr_t)job.codebook % 16 == 0;
    auto x_of = [&](int q) { return (const float*)job.x + (int64_t)min(t0 + q, job.n_tokens - 1) * job.ldx + (int64_t)g * dg; };
    if (staged) {
        const int padded = (dg + 15) & ~15;
        for (int i = tid; i < NT * padded; i += kEncF32Threads) {
            const int q = i / padded, j = i - q * padded;
            const float v = x_of(q)[min(j, dg - 1)];
            reinterpret_cast<float*>(lds.x[q])[j] = j < dg ? v : 0.f;
        }
        __syncthreads();
    }
    float best[NT];
    int arg[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) { best[q] = INFINITY; arg[q] = 0x7fffffff; }
    for (int k = tid; k < K; k += kEncF32Threads) {
        const float* __restrict__ e = (const float*)job.codebook + ((int64_t)g * K + k) * dg;
        float dist[NT] = {};
        if (staged) {
            auto chunk = [&](int j0, auto pieces) __attribute__((always_inline)) {
                constexpr int NP = decltype(pieces)::value;
                f32x4 ev[NP];
#pragma unroll
                for (int u = 0; u < NP; ++u) ev[u] = *reinterpret_cast<const f32x4*>(e + min(j0 + 4 * u, dg - 4));
#pragma unroll
                for (int u = 0; u < NP; ++u) {
                    if (u >= NP - 4) ev[u] = j0 + 4 * u < dg ? ev[u] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < NT; ++q) {
                        const f32x4 df = ev[u] - lds.x[q][j0 / 4 + u];
                        dist[q] = fmaf(df.x, df.x, dist[q]);
                        dist[q] = fmaf(df.y, df.y, dist[q]);
                        dist[q] = fmaf(df.z, df.z, dist[q]);
                        dist[q] = fmaf(df.w, df.w, dist[q]);
                    }
                }
            };
            for (int j0 = 0; j0 < dg; j0 += 64) {
                if (dg - j0 > 48) chunk(j0, std::integral_constant<int, 16>{});
                else if (dg - j0 > 32) chunk(j0, std::integral_constant<int, 12>{});
                else if (dg - j0 > 16) chunk(j0, std::integral_constant<int, 8>{});
                else chunk(j0, std::integral_constant<int, 4>{});
            }
        } else {
            for (int j = 0; j < dg; ++j) {
                const float ej = e[j];
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const float diff = ej - x_of(q)[j];
                    dist[q] = fmaf(diff, diff, dist[q]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < NT; ++q)
            if (dist[q] < best[q]) { best[q] = dist[q]; arg[q] = k; }
    }
    auto take = [](float& b, int& a, float ob, int oa) {          // the lower distance, the lower index on a tie
        const bool other = (ob < b) | ((ob == b) & (oa < a));
        b = other ? ob : b;
        a = other ? oa : a;
    };
    // four winners over 64 lanes: two steps that halve what a lane carries, then one token in each quarter of the lanes
    const int lane = lane_id();
    static_assert(NT == 4, "two halving steps");
#pragma unroll
    for (int n = 2; n > 0; n >>= 1) {
        const bool up = (lane & (16 * n)) != 0;
#pragma unroll
        for (int q = 0; q < n; ++q) {
            const float gb = __shfl_xor(up ? best[q] : best[q + n], 16 * n);
            const int ga = __shfl_xor(up ? arg[q] : arg[q + n], 16 * n);
            best[q] = up ? best[q + n] : best[q];
            arg[q] = up ? arg[q + n] : arg[q];
            take(best[q], arg[q], gb, ga);
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best[0], off);
        const int oa = __shfl_xor(arg[0], off);
        take(best[0], arg[0], ob, oa);
    }
    if ((lane & 15) == 0) {
        lds.best[tid / kWave][lane >> 4] = best[0];
        lds.arg[tid / kWave][lane >> 4] = arg[0];
    }
    __syncthreads();
    if (tid < NT && t0 + tid < job.n_tokens) {
        float b = lds.best[0][tid];
        int a = lds.arg[0][tid];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) take(b, a, lds.best[w][tid], lds.arg[w][tid]);
        const int64_t at = (int64_t)(t0 + tid) * job.G + g;
        if (job.code_bytes == 2) ((uint16_t*)job.codes)[at] = (uint16_t)a;
        else ((uint8_t*)job.codes)[at] = (uint8_t)a;
    }
}

}  // namespace astra
