// The parts of a Transformer block around the attention layer that are not matrix products (paper Sec. 3.1: each
// block normalises, attends with the mixed-precision layer, and runs its position-wise MLP locally): the row-wise
// normalisation of the fp32 residual stream into the layer's element type, and the gating of the fp32 MLP.
// Both are bound by HBM traffic: one read of the row, one write of the result.
#include "vq_decode_body.h"

namespace astra {

constexpr int kNormThreads = 256;
constexpr int kNormCache = 8;        // float4 values a thread keeps in registers: rows up to 256 * 8 * 4 = 8192 wide are read once

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
// sum over the workgroup; every thread gets the result.  `slot` alternates between calls so that a second reduction
// may start before every wavefront has read the first one's partial sums.
__device__ __forceinline__ float block_sum(float v, float (*part)[kNormThreads / kWave], int slot) {
    v = wave_sum(v);
    if (lane_id() == 0) part[slot][threadIdx.x / kWave] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kNormThreads / kWave; ++w) t += part[slot][w];
    return t;
}

template <typename OutT>
__device__ __forceinline__ void store_elem(OutT* o, float v);
template <>
__device__ __forceinline__ void store_elem<float>(float* o, float v) { *o = v; }
template <>
__device__ __forceinline__ void store_elem<uint16_t>(uint16_t* o, float v) { *o = f32_to_bf16_bits(v); }

// One workgroup per row, blockIdx.x.  kind 0: (x - mean) / sqrt(var + eps) * gain + bias, biased variance, computed as the mean of
// squared deviations (two passes over the registers, no cancellation); kind 1: x / sqrt(mean(x^2) + eps) * gain.
// VEC: D % 4 == 0 and D <= 8192, the row lives in registers; otherwise the row is re-read (from cache) per pass.
template <typename OutT, bool VEC>
__device__ __forceinline__ void norm_row(const float* __restrict__ x, int D, int kind, float eps, const float* __restrict__ gain,
                                         const float* __restrict__ bias, OutT* __restrict__ out) {
    __shared__ float part[2][kNormThreads / kWave];
    const int tid = threadIdx.x;
    const float* __restrict__ row = x + (int64_t)blockIdx.x * D;
    OutT* __restrict__ orow = out + (int64_t)blockIdx.x * D;
    const float inv_d = 1.f / (float)D;
    if (VEC) {
        const int n4 = D >> 2;
        f32x4 c[kNormCache];
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < kNormCache; ++j) {
            const int i = tid + j * kNormThreads;
            c[j] = i < n4 ? reinterpret_cast<const f32x4*>(row)[i] : f32x4{0.f, 0.f, 0.f, 0.f};
            s += (c[j].x + c[j].y) + (c[j].z + c[j].w);
        }
        const float mean = kind == 0 ? block_sum(s, part, 0) * inv_d : 0.f;
        float q = 0.f;
#pragma unroll
        for (int j = 0; j < kNormCache; ++j) {
            const int i = tid + j * kNormThreads;
            if (i < n4) {
                const f32x4 d = c[j] - mean;
                q += (d.x * d.x + d.y * d.y) + (d.z * d.z + d.w * d.w);
            }
        }
        const float inv = 1.f / sqrtf(block_sum(q, part, 1) * inv_d + eps);
#pragma unroll
        for (int j = 0; j < kNormCache; ++j) {
            const int i = tid + j * kNormThreads;
            if (i < n4) {
                f32x4 v = (c[j] - mean) * inv;
                if (gain) v *= reinterpret_cast<const f32x4*>(gain)[i];
                if (kind == 0 && bias) v += reinterpret_cast<const f32x4*>(bias)[i];
                if constexpr (sizeof(OutT) == 2) {
                    u32x2 w;
                    w.x = pack_bf16x2(v.x, v.y);
                    w.y = pack_bf16x2(v.z, v.w);
                    reinterpret_cast<u32x2*>(orow)[i] = w;
                } else {
                    reinterpret_cast<f32x4*>(orow)[i] = v;
                }
            }
        }
    } else {
        float s = 0.f;
        for (int i = tid; i < D; i += kNormThreads) s += row[i];
        const float mean = kind == 0 ? block_sum(s, part, 0) * inv_d : 0.f;
        float q = 0.f;
        for (int i = tid; i < D; i += kNormThreads) {
            const float d = row[i] - mean;
            q += d * d;
        }
        const float inv = 1.f / sqrtf(block_sum(q, part, 1) * inv_d + eps);
        for (int i = tid; i < D; i += kNormThreads) {
            float v = (row[i] - mean) * inv;
            if (gain) v *= gain[i];
            if (kind == 0 && bias) v += bias[i];
            store_elem<OutT>(orow + i, v);
        }
    }
}

// The same for rows of at most 1024 values with a wavefront per row: what four wavefronts hold and add above, one holds and adds here in the same order, so
// that the result is theirs bit for bit, without the two barriers.
constexpr int kNormWaveWidth = 1024;
template <typename OutT>
__device__ __forceinline__ void norm_row_wave(const float* __restrict__ x, int64_t r, int D, int kind, float eps, const float* __restrict__ gain,
                                              const float* __restrict__ bias, OutT* __restrict__ out) {
    constexpr int W = kNormThreads / kWave;
    const int lane = lane_id(), n4 = D >> 2;
    const f32x4* __restrict__ row = reinterpret_cast<const f32x4*>(x + r * D);
    const float inv_d = 1.f / (float)D;
    f32x4 c[W], g[W], b[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int i = min(lane + kWave * w, n4 - 1);
        c[w] = row[i];
        g[w] = gain ? reinterpret_cast<const f32x4*>(gain)[i] : f32x4{1.f, 1.f, 1.f, 1.f};
        b[w] = kind == 0 && bias ? reinterpret_cast<const f32x4*>(bias)[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto row_sum = [](const float(&p)[W]) __attribute__((always_inline)) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) t += wave_sum(p[w]);
        return t;
    };
    float p[W];
#pragma unroll
    for (int w = 0; w < W; ++w) p[w] = lane + kWave * w < n4 ? (c[w].x + c[w].y) + (c[w].z + c[w].w) : 0.f;
    const float mean = kind == 0 ? row_sum(p) * inv_d : 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const f32x4 d = c[w] - mean;
        p[w] = lane + kWave * w < n4 ? (d.x * d.x + d.y * d.y) + (d.z * d.z + d.w * d.w) : 0.f;
    }
    const float inv = 1.f / sqrtf(row_sum(p) * inv_d + eps);
    OutT* __restrict__ orow = out + r * D;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int i = lane + kWave * w;
        if (i < n4) {
            f32x4 v = (c[w] - mean) * inv;
            if (gain) v *= g[w];
            if (kind == 0 && bias) v += b[w];
            if constexpr (sizeof(OutT) == 2) {
                u32x2 o;
                o.x = pack_bf16x2(v.x, v.y);
                o.y = pack_bf16x2(v.z, v.w);
                reinterpret_cast<u32x2*>(orow)[i] = o;
            } else {
                reinterpret_cast<f32x4*>(orow)[i] = v;
            }
        }
    }
}
// A wavefront per workgroup (four rows to a workgroup: 12 GPT-2 blocks 608.7 us, 604 now, 614.5 with a workgroup of four wavefronts per row).
template <typename OutT>
__global__ __launch_bounds__(kWave) void norm_wave_kernel(const float* __restrict__ x, int D, int kind, float eps, const float* __restrict__ gain,
                                                          const float* __restrict__ bias, OutT* __restrict__ out) {
    norm_row_wave<OutT>(x, blockIdx.x, D, kind, eps, gain, bias, out);
}

// Eight wavefronts per SIMD: left to itself the compiler takes 68 registers for bf16 rows, which leaves seven (2000 rows of 8192: 17.2 us, 12000 of 1536: 21.9).
template <typename OutT, bool VEC>
__global__ __launch_bounds__(kNormThreads, 8) void norm_kernel(const float* __restrict__ x, int D, int kind, float eps,
                                                               const float* __restrict__ gain, const float* __restrict__ bias,
                                                               OutT* __restrict__ out) {
    norm_row<OutT, VEC>(x, D, kind, eps, gain, bias, out);
}

// The normalisation with the decode of the peers' codes behind its rows, where the projections need the rebuilt rows in memory (slices of no whole 16 bytes).
// The launch lasts what the longer of the two takes, both a few memory latencies for a small model: 6 blocks of 256 + 768 rows, 64 groups of 12, 334.6 us
// with a launch for the decode, 317.3 now; 512 + 1024 rows 522.8 / 501.0.
template <typename CodeT, bool WAVE>
__global__ __launch_bounds__(kNormThreads) void norm_decode_kernel(const float* __restrict__ x, int T, int D, int kind, float eps,
                                                                   const float* __restrict__ gain, const float* __restrict__ bias,
                                                                   uint16_t* __restrict__ out, const DecodeJob job) {
    static_assert(kNormThreads == kDecThreads, "one workgroup size for both");
    constexpr int ROWS = WAVE ? kNormThreads / kWave : 1;
    const int wgs = (T + ROWS - 1) / ROWS;
    if ((int)blockIdx.x >= wgs) {
        vq_decode_run<CodeT>(job, blockIdx.x - (uint32_t)wgs);
    } else if (WAVE) {
        const int r = (int)blockIdx.x * ROWS + (int)(threadIdx.x / kWave);
        if (r < T) norm_row_wave<uint16_t>(x, r, D, kind, eps, gain, bias, out);
    } else {
        norm_row<uint16_t, true>(x, D, kind, eps, gain, bias, out);
    }
}

static bool norm_by_wave(int D) { return D % 4 == 0 && D <= kNormWaveWidth; }
static bool norm_in_registers(int D) { return D % 4 == 0 && D <= kNormThreads * kNormCache * 4; }

bool norm_decode_ok(int64_t T, int D, const DecodeJob& job) { return T > 0 && norm_in_registers(D) && T + job.blocks <= 0x7fffffff; }

int launch_norm_decode(int kind, const float* x, int64_t T, int D, float eps, const float* gain, const float* bias, void* out, const DecodeJob& job,
                       hipStream_t s) {
    if (!norm_decode_ok(T, D, job) || (kind != 0 && kind != 1)) return ASTRA_ERR_SHAPE;
    const bool wave = norm_by_wave(D);
    const int n = (int)T, grid = (int)ceil_div(n, wave ? kNormThreads / kWave : 1) + job.blocks;
#define ASTRA_NORM_DECODE(CODE, WAVE) norm_decode_kernel<CODE, WAVE><<<grid, kNormThreads, 0, s>>>(x, n, D, kind, eps, gain, bias, (uint16_t*)out, job)
    if (job.code_bytes == 1) { if (wave) ASTRA_NORM_DECODE(uint8_t, true); else ASTRA_NORM_DECODE(uint8_t, false); }
    else { if (wave) ASTRA_NORM_DECODE(uint16_t, true); else ASTRA_NORM_DECODE(uint16_t, false); }
#undef ASTRA_NORM_DECODE
    return launch_status();
}

int launch_norm(int dtype, int kind, const float* x, int64_t T, int D, float eps, const float* gain, const float* bias, void* out,
                hipStream_t s) {
    if (T < 0 || D <= 0 || T > 0x7fffffff || (kind != 0 && kind != 1)) return ASTRA_ERR_SHAPE;
    if (T == 0) return ASTRA_OK;
    const bool vec = norm_in_registers(D);
    if (norm_by_wave(D)) {
        if (dtype == ASTRA_BF16) norm_wave_kernel<uint16_t><<<(int)T, kWave, 0, s>>>(x, D, kind, eps, gain, bias, (uint16_t*)out);
        else norm_wave_kernel<float><<<(int)T, kWave, 0, s>>>(x, D, kind, eps, gain, bias, (float*)out);
        return launch_status();
    }
    if (dtype == ASTRA_BF16) {
        if (vec) norm_kernel<uint16_t, true><<<(int)T, kNormThreads, 0, s>>>(x, D, kind, eps, gain, bias, (uint16_t*)out);
        else norm_kernel<uint16_t, false><<<(int)T, kNormThreads, 0, s>>>(x, D, kind, eps, gain, bias, (uint16_t*)out);
    } else {
        if (vec) norm_kernel<float, true><<<(int)T, kNormThreads, 0, s>>>(x, D, kind, eps, gain, bias, (float*)out);
        else norm_kernel<float, false><<<(int)T, kNormThreads, 0, s>>>(x, D, kind, eps, gain, bias, (float*)out);
    }
    return launch_status();
}

// fp32 MLP gate: out[t, f] = silu(a[t, f]) * a[t, F + f]  (the bf16 path does this in the epilogue of its first GEMM)
__global__ __launch_bounds__(256) void swiglu_f32_kernel(const float* __restrict__ a, int64_t n, int F, float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t t = i / F;
    const int f = (int)(i - t * F);
    const float g = a[t * 2 * F + f], u = a[t * 2 * F + F + f];
    out[i] = g / (1.f + expf(-g)) * u;
}

int launch_swiglu_f32(const float* a, int64_t T, int F, float* out, hipStream_t s) {
    if (T < 0 || F <= 0) return ASTRA_ERR_SHAPE;
    const int64_t n = T * F;
    if (n == 0) return ASTRA_OK;
    const int64_t blocks = ceil_div(n, 256);
    if (blocks > 0x7fffffff) return ASTRA_ERR_SHAPE;
    swiglu_f32_kernel<<<(int)blocks, 256, 0, s>>>(a, n, F, out);
    return launch_status();
}

// ---- optional rotary position embedding (not part of the paper; Su et al., "RoFormer", Eq. 34, interleaved pairs), in
// place on up to three [rows, n_heads * head_dim] matrices of the element type with row stride ld: pair i of every head's vector at
// position m is turned by m * base^(-2i / head_dim).  Row r has position r + add_lo when r < split and r + add_hi
// otherwise; rows below `skip` have no position and are left alone.  The angle is formed in fp64 and reduced to a
// fraction of a turn before it is rounded (positions reach 10^5, the cosine of an fp32 product would be off by 10^-3);
// the frequencies of a head are computed once per workgroup.  A thread turns the same PAIRS consecutive pairs of up to kRopeHeads
// heads of a row, which share their angles, with all of them requested before the angles are formed.
// What bounds it: memory, one read and one write.  32 + 8 heads of 128 on 1024 rows and 8 on 2048: a launch per matrix with angles for every head
// 7.9 + 4.9 + 5.5 us (and two gaps), together 8.4 - 10; four blocks 2124 -> 2103 us.
constexpr int kRopeThreads = 256;
constexpr int kRopeHeads = 8;

struct RopeBatch {
    RopeMat m[kMaxRopeMats];
    int32_t first_block[kMaxRopeMats + 1];
};

template <typename T, int PAIRS>
__global__ __launch_bounds__(kRopeThreads) void rope_kernel(const RopeBatch batch, int head_dim, float base) {
    extern __shared__ double theta[];                    // [head_dim / 2]
    int k = 0;
    while (k + 1 < kMaxRopeMats && (int)blockIdx.x >= batch.first_block[k + 1]) ++k;
    const RopeMat& M = batch.m[k];
    const int per_head = head_dim / (2 * PAIRS), groups = (M.n_heads + kRopeHeads - 1) / kRopeHeads;
    const int64_t id = (int64_t)((int)blockIdx.x - batch.first_block[k]) * kRopeThreads + threadIdx.x;
    const int per_row = per_head * groups;
    const int r = (int)min(id / per_row, (int64_t)M.rows - 1), c = (int)(id % per_row);
    const int h0 = c / per_head * kRopeHeads, c0 = c % per_head * 2 * PAIRS;       // first head and first column in a head of this thread
    const bool turns_row = id < (int64_t)M.rows * per_row && r >= M.skip;
    T* __restrict__ p = (T*)M.mat + (int64_t)r * M.ld + c0;
    constexpr bool VEC = sizeof(T) == 2 && PAIRS == 4;
    u32x4 w[VEC ? kRopeHeads : 1];
    if constexpr (VEC) {
#pragma unroll
        for (int j = 0; j < kRopeHeads; ++j) w[j] = *reinterpret_cast<const u32x4*>(p + min(h0 + j, M.n_heads - 1) * head_dim);
    }
    const int half = head_dim >> 1;
    for (int i = threadIdx.x; i < half; i += kRopeThreads) theta[i] = exp2(-2.0 * (double)i / (double)head_dim * log2((double)base));
    __syncthreads();
    if (!turns_row) return;
    const double m = (double)(r < M.split ? r + M.add_lo : r + M.add_hi);
    float cs[PAIRS], sn[PAIRS];
#pragma unroll
    for (int e = 0; e < PAIRS; ++e) {
        double turns = m * theta[(c0 >> 1) + e] * 0.15915494309189535;       // angle / 2 pi
        turns -= floor(turns);
        const float a = (float)(turns * 6.283185307179586);
        cs[e] = cosf(a);
        sn[e] = sinf(a);
    }
#pragma unroll
    for (int j = 0; j < kRopeHeads; ++j) {
        if (h0 + j >= M.n_heads) break;
        T* __restrict__ q = p + (h0 + j) * head_dim;
        if constexpr (VEC) {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = __uint_as_float(w[j][e] << 16), x1 = __uint_as_float(w[j][e] & 0xffff0000u);
                o[e] = pack_bf16x2(fmaf(x0, cs[e], -(x1 * sn[e])), fmaf(x1, cs[e], x0 * sn[e]));
            }
            *reinterpret_cast<u32x4*>(q) = o;
        } else {
#pragma unroll
            for (int e = 0; e < PAIRS; ++e) {
                float x0, x1;
                if constexpr (sizeof(T) == 2) {
                    x0 = bf16_bits_to_f32(q[2 * e]);
                    x1 = bf16_bits_to_f32(q[2 * e + 1]);
                } else {
                    x0 = q[2 * e];
                    x1 = q[2 * e + 1];
                }
                store_elem<T>(q + 2 * e, fmaf(x0, cs[e], -(x1 * sn[e])));
                store_elem<T>(q + 2 * e + 1, fmaf(x1, cs[e], x0 * sn[e]));
            }
        }
    }
}

int launch_rope(int dtype, const RopeMat* mats, int n_mats, int head_dim, float base, hipStream_t s) {
    if (n_mats < 0 || n_mats > kMaxRopeMats || head_dim <= 0 || head_dim % 2 != 0 || !(base > 0.f)) return ASTRA_ERR_SHAPE;
    bool vec = dtype == ASTRA_BF16 && head_dim % 8 == 0;
    for (int i = 0; i < n_mats; ++i) vec = vec && mats[i].ld % 8 == 0;
    RopeBatch batch{};
    int n = 0;
    int64_t blocks = 0;
    for (int i = 0; i < n_mats; ++i) {
        if (mats[i].rows <= 0) continue;
        batch.m[n] = mats[i];
        batch.first_block[n++] = (int32_t)blocks;
        blocks += ceil_div((int64_t)mats[i].rows * (head_dim / (vec ? 8 : 2)) * ceil_div(mats[i].n_heads, kRopeHeads), kRopeThreads);
        if (blocks > 0x7fffffff) return ASTRA_ERR_SHAPE;
    }
    if (n == 0) return ASTRA_OK;
    for (int i = n; i <= kMaxRopeMats; ++i) batch.first_block[i] = (int32_t)blocks;
    const size_t lds = (size_t)(head_dim / 2) * sizeof(double);
    if (vec) rope_kernel<uint16_t, 4><<<(int)blocks, kRopeThreads, lds, s>>>(batch, head_dim, base);
    else if (dtype == ASTRA_BF16) rope_kernel<uint16_t, 1><<<(int)blocks, kRopeThreads, lds, s>>>(batch, head_dim, base);
    else rope_kernel<float, 1><<<(int)blocks, kRopeThreads, lds, s>>>(batch, head_dim, base);
    return launch_status();
}

}  // namespace astra
