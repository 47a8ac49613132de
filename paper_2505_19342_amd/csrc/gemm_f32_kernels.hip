// fp32 products C[M,N] = A[M,K] . B[N,K]^T of the small fp32 configuration (paper: the projections named under Eq. 1, and the MLP of the block
// around the layer, Sec. 3.1).
#include "gemm_bf16_tile.h"

namespace astra {

// The problem of a tile.  With tiles of 64 its fields are read from the arguments where they are needed: a copy, in one trip, makes 266 registers of 242, one
// wavefront per SIMD instead of two (700 x 1536 outputs, K = 64: 13.9 us, 20.7 with the copy).  Smaller tiles have the registers for it.
struct ProblemInPlace {
    const GemmProblem& p;
    int tile, tiles_m;
};
template <int T, bool ONE>
__device__ __forceinline__ auto f32_problem(const GemmBatch& b, int tile) {
    if constexpr (T < 4) {
        return find_problem<ONE ? kOneProblem : kManyProblems>(b, tile);
    } else {
        int i = 0;
        while (i + 1 < b.n && tile >= b.tile_begin[i + 1]) ++i;
        return ProblemInPlace{b.p[i], tile - b.tile_begin[i], b.tiles_m[i]};
    }
}

// ------------------------------------------------------------------------------------------------
// fp32, matrix cores (16x16x4: fp32 products, fp32 sums).  A workgroup of four wavefronts owns a 16 T x 16 T output tile, and every wavefront
// computes all of it over every fourth slice of 16 of the contraction, straight from global memory: lane l holds row l % 16 of each operand, and since
// the order inside a slice is free, the four consecutive values of a 16-byte load of quarter l / 16 are that quarter's values of four MFMAs.  PD slices
// are requested at once, the next PD before these are multiplied; no LDS and no barrier before the partial tiles are added in wavefront order at
// the end.  What bounds it at the sizes it is for is the chain codes -> operands -> result, a memory latency each, and the fp32 rate of a unit
// (128 multiply-adds a clock: 2.6 us for 32 x 32 outputs at K = 768), hence the small tiles.
// As a vector-ALU kernel with two barriers and a latency per 64 of contraction, against now (back to back): 64 x 192 outputs, K = 192 / 768:
// 8.0 / 23.5 us, now 3.7 / 5.2; 1000 x 1000, K = 1000: 68.7, now 27.4.  Error against fp64 at K = 768: 4.9e-7 of the norm, now 2.5e-7.
// ------------------------------------------------------------------------------------------------
template <int T, bool ONE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmBatch batch) {
    constexpr int BT = 16 * T, WAVES = 4, PD = 4 / T, LDN = BT + 4;
    __shared__ __align__(16) float red[WAVES * BT * LDN];
    const auto tp = f32_problem<T, ONE>(batch, blockIdx.x);
    const GemmProblem& P = tp.p;
    const int tile = tp.tile, m0 = tile % tp.tiles_m * BT, n0 = tile / tp.tiles_m * BT;
    const int M = P.M, N = P.N, K = P.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, h = lane >> 4;
    const bool gather = P.codes != nullptr;
    const float* __restrict__ A = (const float*)(gather ? P.codebook : P.a);
    const float* __restrict__ B = (const float*)P.b;
    const int64_t ldb = P.ldb ? P.ldb : K;
    const int dg = gather ? P.dg : 1;
    const bool vec = K % 4 == 0 && ldb % 4 == 0 && (gather ? dg % 4 == 0 : P.lda % 4 == 0) &&
                     (reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) % 16 == 0;
    int64_t arow[T], brow[T];                 // first element of this lane's rows (gathered: of its codes); rows beyond the problem are its last one
#pragma unroll
    for (int t = 0; t < T; ++t) {
        arow[t] = (int64_t)min(m0 + 16 * t + i16, M - 1) * (gather ? P.G : P.lda);
        brow[t] = (int64_t)min(n0 + 16 * t + i16, N - 1) * ldb;
    }
    auto code_of = [&](int t, int g) {
        const int c = P.code_bytes == 1 ? (int)((const uint8_t*)P.codes)[arow[t] + g] : (int)((const uint16_t*)P.codes)[arow[t] + g];
        return c < P.Kc ? c : P.Kc - 1;
    };
    f32x4 fa[2][PD][T], fb[2][PD][T];
    // slices s, s + WAVES, ... (PD of them) into set `set`; values beyond the contraction are zeros on both sides
    auto fetch = [&](int set, int s) __attribute__((always_inline)) {
        if (vec) {
            int k[PD], code[PD][T];
#pragma unroll
            for (int d = 0; d < PD; ++d) k[d] = min((s + WAVES * d) * 16 + 4 * h, K - 4);
            if (gather)
#pragma unroll
                for (int d = 0; d < PD; ++d)
#pragma unroll
                    for (int t = 0; t < T; ++t) code[d][t] = code_of(t, k[d] / dg);
#pragma unroll
            for (int d = 0; d < PD; ++d)
#pragma unroll
                for (int t = 0; t < T; ++t) fb[set][d][t] = *reinterpret_cast<const f32x4*>(B + brow[t] + k[d]);
#pragma unroll
            for (int d = 0; d < PD; ++d) {
                const int g = gather ? k[d] / dg : 0;
#pragma unroll
                for (int t = 0; t < T; ++t)
                    fa[set][d][t] = *reinterpret_cast<const f32x4*>(A + (gather ? ((int64_t)g * P.Kc + code[d][t]) * dg + (k[d] - g * dg) : arow[t] + k[d]));
            }
            __builtin_amdgcn_sched_barrier(0);         // all of them are on their way before anything is multiplied
        } else {
#pragma unroll
            for (int d = 0; d < PD; ++d)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = min((s + WAVES * d) * 16 + 4 * h + e, K - 1);
                    const int g = gather ? k / dg : 0;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        fb[set][d][t][e] = B[brow[t] + k];
                        fa[set][d][t][e] = A[gather ? ((int64_t)g * P.Kc + code_of(t, g)) * dg + (k - g * dg) : arow[t] + k];
                    }
                }
        }
#pragma unroll
        for (int d = 0; d < PD; ++d)
            if ((s + WAVES * d) * 16 + 16 > K)          // the last slice, or none
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = (s + WAVES * d) * 16 + 4 * h + e < K;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        fb[set][d][t][e] = in ? fb[set][d][t][e] : 0.f;
                        fa[set][d][t][e] = in ? fa[set][d][t][e] : 0.f;
                    }
                }
    };
    f32x4 acc[T][T];
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int d = 0; d < PD; ++d)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < T; ++a)
#pragma unroll
                    for (int b = 0; b < T; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[set][d][b][e], fa[set][d][a][e], acc[a][b], 0, 0, 0);
    };
    const int slices = (K + 15) / 16;
    constexpr int STEP = WAVES * PD;
    if (wave < slices) {
        fetch(0, wave);
        for (int s = wave; s < slices; s += 2 * STEP) {          // the sets alternate, so each copy knows its own
            if (s + STEP < slices) fetch(1, s + STEP);
            multiply(0);
            if (s + STEP >= slices) break;
            if (s + 2 * STEP < slices) fetch(0, s + 2 * STEP);
            multiply(1);
        }
    }

    // ---- the partial tiles and the store.  acc[a][b][v] is C[16a + lane % 16, 16b + 4 (lane / 16) + v].
    float* C = (float*)P.c;                               // may be the residual itself: no restrict
    const float* __restrict__ bias = (const float*)P.bias;
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) *reinterpret_cast<f32x4*>(&red[(wave * BT + 16 * a + i16) * LDN + 16 * b + 4 * h]) = acc[a][b];
    __syncthreads();
#pragma unroll
    for (int e = tid; e < BT * BT; e += 256) {
        const int r = e / BT, c = e % BT, m = m0 + r, n = n0 + c;
        if (m >= M || n >= N) continue;
        float v = red[r * LDN + c];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v += red[(w * BT + r) * LDN + c];
        const int64_t at = (int64_t)m * P.ldc + n;
        v = apply_act<false>(v + (bias ? bias[n] : 0.f), P.act);
        C[at] = P.residual ? v + P.residual[at] : v;
    }
}

template <int T>
static void launch_f32_tiles(int tiles, const GemmBatch& batch, hipStream_t s) {
    if (T < 4 && batch.n == 1) gemm_f32_kernel<T, T < 4><<<tiles, 256, 0, s>>>(batch);
    else gemm_f32_kernel<T, false><<<tiles, 256, 0, s>>>(batch);
}

// the batch was filled for square tiles of 16, 32 or 64
int launch_gemm_f32(int tile, const GemmBatch& batch, hipStream_t s) {
    const int tiles = batch.tile_begin[batch.n];
    if (tiles == 0) return ASTRA_OK;
    if (tile == 64) launch_f32_tiles<4>(tiles, batch, s);
    else if (tile == 32) launch_f32_tiles<2>(tiles, batch, s);
    else launch_f32_tiles<1>(tiles, batch, s);
    return launch_status();
}

}  // namespace astra
