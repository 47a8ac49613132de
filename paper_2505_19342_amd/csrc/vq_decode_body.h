// Decode of codes into rows (paper Sec. 2: the rows a device rebuilds from its peers' codes) as extra workgroups of a block's first normalisation.
#pragma once
#include "common.h"

namespace astra {

// Slices of whole 8-byte pieces (with 16-byte pieces the projections fetch the codewords themselves).  A piece per thread and pass, kDecUnroll passes a
// whole grid of these workgroups apart; code reads, codeword reads and stores are three batches, as in vq_decode_kernel.
constexpr int kDecThreads = 256;
constexpr int kDecPieces = 4;

struct DecodeJob {
    const void* codes;
    const void* codebook;
    void* x_hat;
    uint32_t n_pieces, per_token, per_group, magic_token, magic_group;      // pieces; multiply-high divisors by per_token and per_group
    int32_t G, K;
    int32_t code_bytes;
    int32_t blocks;           // workgroups of kDecThreads
};

// false: other slices, or a call whose indices or divisions do not fit 32 bits
bool vq_decode_job(const astra_vq_desc& d, const void* codes, int64_t n_tokens, const void* codebook, void* x_hat, DecodeJob* job);

template <typename CodeT>
__device__ __forceinline__ void vq_decode_run(const DecodeJob& job, uint32_t block) {
    const CodeT* __restrict__ codes = (const CodeT*)job.codes;
    const u32x2* __restrict__ codebook = (const u32x2*)job.codebook;
    u32x2* __restrict__ x_hat = (u32x2*)job.x_hat;
    const uint32_t stride = (uint32_t)job.blocks * kDecThreads, first = block * kDecThreads + threadIdx.x;
    uint32_t src[kDecPieces];
    int code[kDecPieces];
#pragma unroll
    for (int u = 0; u < kDecPieces; ++u) {
        const uint32_t i = min(first + (uint32_t)u * stride, job.n_pieces - 1);       // clamped, not guarded: the store below is the only guard
        const uint32_t t = __umulhi(i, job.magic_token);
        const uint32_t c = i - t * job.per_token;
        const uint32_t g = __umulhi(c, job.magic_group);
        src[u] = g * (uint32_t)job.K * job.per_group + (c - g * job.per_group);
        code[u] = (int)codes[(uint64_t)t * (uint32_t)job.G + g];
    }
    u32x2 v[kDecPieces];
#pragma unroll
    for (int u = 0; u < kDecPieces; ++u) v[u] = codebook[(uint64_t)src[u] + (uint64_t)min(code[u], job.K - 1) * job.per_group];
#pragma unroll
    for (int u = 0; u < kDecPieces; ++u)
        if (first + (uint32_t)u * stride < job.n_pieces) x_hat[first + (uint32_t)u * stride] = v[u];
}

}  // namespace astra
