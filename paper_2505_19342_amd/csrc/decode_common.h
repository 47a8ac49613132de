// The decode step's parameter block, shared by the kernels that carry it (decode_kernels.hip, decode_stream_kernels.hip).
#pragma once
#include "common.h"

namespace astra {

struct DecodeParams {
    const void* q;
    const void* k_loc;
    const void* v_loc;
    const void* codes_k;
    const void* codes_v;
    const unsigned long long* valid_bits;
    const void* cb_k;
    const void* cb_v;
    void* out;
    float* lse;
    float* lut;      // [H_kv][n_gh][K][H_q / H_kv]
    float* part;     // [n_chunks][H_q][dh + 2]: unnormalised o, then m, l
    int32_t Hq, Hkv, dh, n_local, n_nonlocal, G, K, dg, code16, n_gh, chunk_loc, chunk_nl, n_chunks_loc, n_chunks_nl;
    int32_t aux_floats;      // floats of the LDS region shared by the query floats, the table slice and the cross-phase sums
    float scale;
};

__device__ __forceinline__ int load_code(const void* codes, int code16, int64_t i, int K) {
    const int c = code16 ? (int)((const uint16_t*)codes)[i] : (int)((const uint8_t*)codes)[i];
    return c < K ? c : K - 1;
}

// How the matrix-core form of the step (decode_stream_kernels.hip) is launched for a shape
struct DecodeStreamPlan {
    bool applies;            // it has a kernel for the shape
    bool table;              // key scores of the index cache from a table of query-codeword products in LDS
    int wgs_loc, wgs_nl;     // workgroups per KV head for the local rows and for the index cache, one partial result each
    size_t lds;
};
DecodeStreamPlan plan_decode_stream(int dtype, int Hq, int Hkv, int dh, int n_local, int n_nonlocal, int K, int dg);
int launch_decode_stream(const DecodeParams& p, const DecodeStreamPlan& pl, hipStream_t s);

}  // namespace astra
