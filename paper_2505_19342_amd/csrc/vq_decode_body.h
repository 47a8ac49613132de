// Decode of codes into rows (paper Sec. 2: the rows a device rebuilds from its peers' codes), as a device function, so that it can run as a kernel of its
// own and as extra workgroups of a block's first normalisation.
#pragma once
#include "common.h"

namespace astra {

// ------------------------------------------------------------------------------------------------
// A pure gather.  One CHUNK-byte piece of one (token, group) row per thread and pass, kDecUnroll passes per
// thread a whole grid apart: consecutive threads write consecutive addresses of x_hat; the lanes of one group row read
// the same code (a broadcast) and consecutive pieces of one codeword.  The passes' code reads, codeword reads and stores
// are issued as three batches, so that every thread has kDecUnroll independent chains in flight (the step is bound by
// memory latency times bytes in flight, not by arithmetic); piece -> (token, group, offset) uses multiply-high divisions.
// ------------------------------------------------------------------------------------------------
constexpr int kDecUnroll = 4;
constexpr int kDecThreads = 256;

struct DecodeJob {
    const void* codes;
    const void* codebook;
    void* x_hat;
    uint32_t n_chunks, chunks_per_token, chunks_per_group, magic_token, magic_group;
    int32_t G, K;
    int32_t chunk_bytes, code_bytes;
    int32_t blocks;           // workgroups of kDecThreads
};

// false: the call's indices or divisions do not fit 32 bits
bool vq_decode_job(const astra_vq_desc& d, const void* codes, int64_t n_tokens, const void* codebook, void* x_hat, DecodeJob* job);

template <typename ChunkT, typename CodeT>
__device__ __forceinline__ void vq_decode_run(const DecodeJob& job, uint32_t block) {
    const CodeT* __restrict__ codes = (const CodeT*)job.codes;
    const ChunkT* __restrict__ codebook = (const ChunkT*)job.codebook;
    ChunkT* __restrict__ x_hat = (ChunkT*)job.x_hat;
    const uint32_t stride = (uint32_t)job.blocks * kDecThreads;
    const uint32_t first = block * kDecThreads + threadIdx.x;
    uint32_t idx[kDecUnroll], src[kDecUnroll];
    int code[kDecUnroll];
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
        idx[u] = first + (uint32_t)u * stride;
        const uint32_t i = idx[u] < job.n_chunks ? idx[u] : job.n_chunks - 1;       // clamped, not guarded: the store below is the only guard
        const uint32_t t = __umulhi(i, job.magic_token);
        const uint32_t c = i - t * job.chunks_per_token;
        const uint32_t g = __umulhi(c, job.magic_group);
        src[u] = g * (uint32_t)job.K * job.chunks_per_group + (c - g * job.chunks_per_group);
        code[u] = (int)codes[(uint64_t)t * (uint32_t)job.G + g];
    }
    ChunkT v[kDecUnroll];
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
        const int cd = code[u] < job.K ? code[u] : job.K - 1;
        v[u] = codebook[(uint64_t)src[u] + (uint64_t)cd * job.chunks_per_group];
    }
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u)
        if (idx[u] < job.n_chunks) x_hat[idx[u]] = v[u];
}

}  // namespace astra
