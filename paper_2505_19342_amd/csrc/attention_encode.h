// VQ encodes that ride in an attention launch.
#pragma once
#include "common.h"
#include "vq_encode_body.h"

namespace astra {

// The grid is the attention workgroups followed by n_enc_wgs workgroups that run VQ encodes nothing in this launch
// depends on (the layer that quantises K and V after projection sends their codes to its peers): they are dispatched as
// attention workgroups finish, i.e. into the tail that causal masking leaves on the units of the light query blocks.
struct AttnEncode {
    EncodeJob job[2];
    int32_t n_jobs, n_attn_wgs, n_enc_wgs;
};

// bf16, V transposed, a workgroup per 32 query rows; encodes ride on 128-wide heads only
int launch_attention_short(const AttnParams& p, int head_dim, const AttnEncode& e, const Prefetch* fetch, hipStream_t s);

// workgroup idx of those behind the attention's own; cb, cn: LDS for the encode's ring of codebook tiles and their norms
template <int THREADS>
__device__ __forceinline__ void attn_encode_wgs(const AttnEncode& e, int idx, u32x4* cb, f32x4* cn) {
    // the items of all jobs in one sequence, dealt in consecutive runs (consecutive items share the group)
    int n_total = 0;
    for (int j = 0; j < e.n_jobs; ++j) n_total += e.job[j].G * e.job[j].n_tb;
    const int chunk = (n_total + e.n_enc_wgs - 1) / e.n_enc_wgs;
    const int hi = min((idx + 1) * chunk, n_total);
    if (vq_encode_fast_needs_zero(e.job[0].dg)) {          // every job of a launch has the same group length
        vq_encode_fast_zero_lds<THREADS>(cb);
        __syncthreads();                           // zero fill done before any transfer lands
    }
    int first = 0;                                 // of job j in the sequence
    for (int j = 0; j < e.n_jobs; ++j) {
        const EncodeJob& job = e.job[j];
        const int n = job.G * job.n_tb, from = max(idx * chunk - first, 0), to = min(hi - first, n);
        if (from < to) {
            vq_encode_fast_run<THREADS, true>(job, from, to, cb, cn);
            __syncthreads();                       // all reads of this run's tiles done before the next run's transfers
        }
        first += n;
    }
}

}  // namespace astra
