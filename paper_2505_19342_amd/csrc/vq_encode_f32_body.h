// fp32 encode (paper Sec. 2 "Grouped VQ": nearest codeword per group, lowest index on ties), as a device function of one workgroup, so that it
// can run as a kernel of its own and as extra workgroups of the fp32 attention.
#pragma once
#include "vq_encode_body.h"

namespace astra {

// ------------------------------------------------------------------------------------------------
// A workgroup of 256 threads takes kEncF32Tokens tokens of one group; a lane forms squared distances sum (x - c)^2 in ascending order.  Bound by the round trip
// of the codeword loads: up to 64 values of a codeword are requested at once (16-byte loads where the slices allow it).  Values beyond the group are
// zeros on both sides: they add fma(0, 0, d) = d, and the work of a chunk has no branch.  Forms:
//   shared, long  a thread takes every 256th codeword and all four tokens, whose values wait in LDS (long: kEncF32Staged at a time).
//   few           small codebooks do not have a codeword for each of 256 threads: in a small launch a wavefront takes one of the tokens, again out of LDS.
//   solo          short slices, small codebooks: the same without LDS, barrier or another wavefront to wait for, and with half the registers.
// Shared / few, K = 16: 500 tokens x 2 groups of 384 (250 workgroups) 16.0 / 8.4 us, 2000 (1000 workgroups) 15.1 / 22.5; K = 64: 64 tokens x 1 group of 192
// 8.0 / 8.5, of 768 29 / 26, x 4 of 48 4.0 / 3.2.  Shared / solo: 2000 tokens x 4 groups of 12, K = 16 6.4 / 3.8, K = 100 6.5 / 5.1; of 16, K = 100
// 6.5 / 7.2.  A wavefront per token, 32 values of a codeword at a time / slices longer than 512 read value by value and small codebooks shared as well / this:
// 500 tokens x 1 group of 768, K = 16 17.0 / 67.3 / 14.2, K = 1024 417 / 438 / 91; 2000 x 4 groups of 1024 5333 / 6895 / 916; 500 x 2 groups of 384, K = 16
// 9.8 / 16.0 / 8.4; 64 x 4 groups of 48, K = 256 7.6 / 4.5 / 4.2.
// ------------------------------------------------------------------------------------------------
constexpr int kEncF32Tokens = 4;
constexpr int kEncF32Threads = 256;
constexpr int kEncF32Staged = 1024;        // values of a token's slice that LDS holds at a time
enum { kEncF32Shared = 0, kEncF32Long = 1, kEncF32Few = 2, kEncF32Solo = 3 };
struct EncF32Lds {
    f32x4 x[kEncF32Tokens][kEncF32Staged / 4];
    float best[kEncF32Threads / kWave][kEncF32Tokens];
    int arg[kEncF32Threads / kWave][kEncF32Tokens];
};

// values j .. end - 1 of codeword e (rows of dg) against those of NQ tokens: x(q, u) is token q's values j + 4u .. + 3, zeros from end on
template <bool VEC, int NQ, typename X>
__device__ __forceinline__ void vq_encode_f32_add(const float* __restrict__ e, int j, int end, int dg, float (&dist)[NQ], X x) {
    auto chunk = [&](auto pieces) __attribute__((always_inline)) {
        constexpr int NP = decltype(pieces)::value;
        f32x4 ev[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            if (VEC) ev[u] = *reinterpret_cast<const f32x4*>(e + min(j + 4 * u, dg - 4));
            else
#pragma unroll
                for (int i = 0; i < 4; ++i) ev[u][i] = e[min(j + 4 * u + i, dg - 1)];
        }
        __builtin_amdgcn_sched_barrier(0x104);     // all of them are on their way before the first is needed; reads of LDS may pass
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            if (u >= NP - 4)
#pragma unroll
                for (int i = 0; i < 4; ++i) ev[u][i] = j + 4 * u + (VEC ? 0 : i) < end ? ev[u][i] : 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const f32x4 df = ev[u] - x(q, u);
                dist[q] = fmaf(df.x, df.x, dist[q]);
                dist[q] = fmaf(df.y, df.y, dist[q]);
                dist[q] = fmaf(df.z, df.z, dist[q]);
                dist[q] = fmaf(df.w, df.w, dist[q]);
            }
        }
    };
    if (end - j > 48) chunk(std::integral_constant<int, 16>{});
    else if (end - j > 32) chunk(std::integral_constant<int, 12>{});
    else if (end - j > 16) chunk(std::integral_constant<int, 8>{});
    else if (VEC || end - j > 8) chunk(std::integral_constant<int, 4>{});
    else if (end - j > 4) chunk(std::integral_constant<int, 2>{});
    else chunk(std::integral_constant<int, 1>{});
}

__device__ __forceinline__ void vq_encode_f32_take(float& b, int& a, float ob, int oa) {          // the lower distance, the lower index on a tie
    const bool other = (ob < b) | ((ob == b) & (oa < a));
    b = other ? ob : b;
    a = other ? oa : a;
}
__device__ __forceinline__ void vq_encode_f32_store(const EncodeJob& job, int g, int t, int a) {
    const int64_t at = (int64_t)t * job.G + g;
    if (job.code_bytes == 2) ((uint16_t*)job.codes)[at] = (uint16_t)a;
    else ((uint8_t*)job.codes)[at] = (uint8_t)a;
}

// VEC: codewords and tokens come in whole 16-byte pieces
template <bool VEC>
__device__ __forceinline__ void vq_encode_f32_solo(const EncodeJob& job, int g, int t0) {
    const int K = job.K, dg = job.dg, lane = lane_id(), t = t0 + threadIdx.x / kWave;
    if (t >= job.n_tokens) return;
    const float* __restrict__ xs = (const float*)job.x + (int64_t)t * job.ldx + (int64_t)g * dg;
    float best = INFINITY;
    int arg = 0x7fffffff;
    for (int k = lane; k < K; k += kWave) {
        const float* __restrict__ e = (const float*)job.codebook + ((int64_t)g * K + k) * dg;
        float dist = 0.f;
        auto chunk = [&](int j, auto pieces) __attribute__((always_inline)) {
            constexpr int NP = decltype(pieces)::value;
            f32x4 ev[NP], xv[NP];
#pragma unroll
            for (int u = 0; u < NP; ++u)
                if (VEC) {
                    ev[u] = *reinterpret_cast<const f32x4*>(e + j + 4 * u);
                    xv[u] = *reinterpret_cast<const f32x4*>(xs + j + 4 * u);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        ev[u][i] = e[min(j + 4 * u + i, dg - 1)];
                        xv[u][i] = xs[min(j + 4 * u + i, dg - 1)];
                    }
                }
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                f32x4 df = ev[u] - xv[u];
                if (!VEC && u == NP - 1)
#pragma unroll
                    for (int i = 0; i < 4; ++i) df[i] = j + 4 * u + i < dg ? df[i] : 0.f;
                dist = fmaf(df.x, df.x, dist);
                dist = fmaf(df.y, df.y, dist);
                dist = fmaf(df.z, df.z, dist);
                dist = fmaf(df.w, df.w, dist);
            }
        };
        for (int j = 0; j < dg; j += 16) {
            if (dg - j > 12) chunk(j, std::integral_constant<int, 4>{});
            else if (dg - j > 8) chunk(j, std::integral_constant<int, 3>{});
            else if (dg - j > 4) chunk(j, std::integral_constant<int, 2>{});
            else chunk(j, std::integral_constant<int, 1>{});
        }
        if (dist < best) { best = dist; arg = k; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best, off);
        const int oa = __shfl_xor(arg, off);
        vq_encode_f32_take(best, arg, ob, oa);
    }
    if (lane == 0) vq_encode_f32_store(job, g, t, arg);
}

// NQ tokens per thread, 1 (a token per wavefront) or all; LONG: slices of several stages
template <bool VEC, int NQ, bool LONG>
__device__ __forceinline__ void vq_encode_f32_staged(const EncodeJob& job, int g, int t0, EncF32Lds& lds) {
    constexpr int NT = kEncF32Tokens, WAVES = kEncF32Threads / kWave, STEP = kEncF32Threads / NT * NQ;
    static_assert(NT == WAVES && (NQ == 1 || NQ == NT), "a token per wavefront, or all of them");
    const int K = job.K, dg = job.dg, tid = threadIdx.x, lane = lane_id();
    const int first = NQ == 1 ? __builtin_amdgcn_readfirstlane(tid / kWave) : 0, at = NQ == 1 ? lane : tid;
    auto row = [&](int q) __attribute__((always_inline)) { return (const float*)job.x + (int64_t)min(t0 + q, job.n_tokens - 1) * job.ldx + (int64_t)g * dg; };
    auto stage = [&](int s0) __attribute__((always_inline)) {          // values s0 .. of the four slices, zeros up to a multiple of 16
        const int n = min(dg - s0, kEncF32Staged), padded = (n + 15) & ~15;
        for (int i = tid; i < NT * padded; i += kEncF32Threads) {
            const int q = i / padded, j = i - q * padded;
            const float v = row(q)[min(s0 + j, dg - 1)];
            reinterpret_cast<float*>(lds.x[q])[j] = j < n ? v : 0.f;
        }
        __syncthreads();
    };
    float best[NQ];
    int arg[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) { best[q] = INFINITY; arg[q] = 0x7fffffff; }
    auto compare = [&](const float (&dist)[NQ], int k) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (dist[q] < best[q]) { best[q] = dist[q]; arg[q] = k; }
    };
    if (!VEC && !LONG && dg <= 8) {                                    // a few single values, straight from memory
        for (int k = at; k < K; k += STEP) {
            const float* __restrict__ e = (const float*)job.codebook + ((int64_t)g * K + k) * dg;
            float dist[NQ] = {};
            for (int j = 0; j < dg; ++j) {
                const float ej = e[j];
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const float diff = ej - row(first + q)[j];
                    dist[q] = fmaf(diff, diff, dist[q]);
                }
            }
            compare(dist, k);
        }
    } else if constexpr (LONG) {
        stage(0);
        for (int k0 = 0; k0 < K; k0 += STEP) {                         // the same rounds for every thread: the stages have barriers
            const float* __restrict__ e = (const float*)job.codebook + ((int64_t)g * K + min(k0 + at, K - 1)) * dg;
            float dist[NQ] = {};
            for (int s0 = 0; s0 < dg; s0 += kEncF32Staged) {
                if (s0 + k0 > 0 && dg > kEncF32Staged) {
                    __syncthreads();
                    stage(s0);
                }
                const int end = min(s0 + kEncF32Staged, dg);
                for (int j = s0; j < end; j += 64)
                    vq_encode_f32_add<VEC, NQ>(e, j, end, dg, dist, [&](int q, int u) __attribute__((always_inline)) { return lds.x[first + q][(j - s0) / 4 + u]; });
            }
            if (k0 + at < K) compare(dist, k0 + at);
        }
    } else {
        stage(0);
        for (int k = at; k < K; k += STEP) {
            const float* __restrict__ e = (const float*)job.codebook + ((int64_t)g * K + k) * dg;
            float dist[NQ] = {};
            for (int j = 0; j < dg; j += 64)
                vq_encode_f32_add<VEC, NQ>(e, j, dg, dg, dist, [&](int q, int u) __attribute__((always_inline)) { return lds.x[first + q][j / 4 + u]; });
            compare(dist, k);
        }
    }
    if constexpr (NQ == 1) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const float ob = __shfl_xor(best[0], off);
            const int oa = __shfl_xor(arg[0], off);
            vq_encode_f32_take(best[0], arg[0], ob, oa);
        }
        if (lane == 0 && t0 + first < job.n_tokens) vq_encode_f32_store(job, g, t0 + first, arg[0]);
        return;
    }
    // four winners over 64 lanes: two steps that halve what a lane carries, then one token in each quarter of the lanes
#pragma unroll
    for (int n = NQ / 2; n > 0; n >>= 1) {
        const bool up = (lane & (16 * n)) != 0;
#pragma unroll
        for (int q = 0; q < n; ++q) {
            const float gb = __shfl_xor(up ? best[q] : best[q + n], 16 * n);
            const int ga = __shfl_xor(up ? arg[q] : arg[q + n], 16 * n);
            best[q] = up ? best[q + n] : best[q];
            arg[q] = up ? arg[q + n] : arg[q];
            vq_encode_f32_take(best[q], arg[q], gb, ga);
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best[0], off);
        const int oa = __shfl_xor(arg[0], off);
        vq_encode_f32_take(best[0], arg[0], ob, oa);
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
        for (int w = 1; w < WAVES; ++w) vq_encode_f32_take(b, a, lds.best[w][tid], lds.arg[w][tid]);
        vq_encode_f32_store(job, g, t0 + tid, a);
    }
}

__host__ __device__ inline int vq_encode_f32_form(const EncodeJob& job) {
    const int K = job.K, dg = job.dg;
    const int64_t wgs = (int64_t)job.G * job.n_tb;
    if (K <= 64 ? dg <= 32 : K <= 128 && (dg <= 4 || dg == 8 || dg == 12)) return kEncF32Solo;
    if (K <= 16 ? wgs <= 512 : wgs <= 256 && (K <= 32 || (K <= 64 && (dg <= 48 || dg > 512)))) return kEncF32Few;
    return dg > kEncF32Staged ? kEncF32Long : kEncF32Shared;
}
__host__ __device__ inline bool vq_encode_f32_vec(const EncodeJob& job, int form) {
    return job.dg % 4 == 0 && (uintptr_t)job.codebook % 16 == 0 && (form != kEncF32Solo || (job.ldx % 4 == 0 && (uintptr_t)job.x % 16 == 0));
}

// item = group * token blocks + token block
template <int FORM, bool VEC>
__device__ __forceinline__ void vq_encode_f32_form_body(const EncodeJob& job, int64_t item, EncF32Lds& lds) {
    const int g = (int)(item / job.n_tb), t0 = (int)(item - (int64_t)g * job.n_tb) * kEncF32Tokens;
    if constexpr (FORM == kEncF32Solo) vq_encode_f32_solo<VEC>(job, g, t0);
    else vq_encode_f32_staged<VEC, FORM == kEncF32Few ? 1 : kEncF32Tokens, FORM != kEncF32Shared>(job, g, t0, lds);
}
// in another kernel's launch, whose registers leave nothing for solo to gain
__device__ __forceinline__ void vq_encode_f32_body(const EncodeJob& job, int64_t item, EncF32Lds& lds) {
    const int form = vq_encode_f32_form(job);
    const bool vec = vq_encode_f32_vec(job, kEncF32Few);
    auto run = [&](auto f) __attribute__((always_inline)) {
        constexpr int FORM = decltype(f)::value;
        if (vec) vq_encode_f32_form_body<FORM, true>(job, item, lds);
        else vq_encode_f32_form_body<FORM, false>(job, item, lds);
    };
    switch (form) {
        case kEncF32Shared: run(std::integral_constant<int, kEncF32Shared>{}); break;
        case kEncF32Long: run(std::integral_constant<int, kEncF32Long>{}); break;
        default: run(std::integral_constant<int, kEncF32Few>{}); break;
    }
}

}  // namespace astra
