// The decode step (paper App. "Memory Cost Analysis", Sec. 3.1; see decode_kernels.hip) on the matrix cores: bf16, heads of 64 or
// 128, codewords of whole 16-byte pieces.
#include "decode_common.h"

#include <algorithm>
#include <type_traits>

namespace astra {

// ------------------------------------------------------------------------------------------------
// One new token's query heads against a cache.  Every wavefront walks tiles of 32 cached tokens of one KV head on its own, with
// its own running maximum: no barrier until the wavefronts of a workgroup merge at the end.
//
// Both contractions of a tile run on 16x16x32 MFMAs.  S^T = K . Q^T has tokens on the M side and the query heads that share the
// KV head on the N side, so a lane's scores all belong to one head and, rounded, already are the B operand of O^T += V^T . P^T:
// lane l (column l % 16, l / 16 = g) holds tokens 4g .. 4g+3 and 16+4g .. 16+4g+3, and any assignment of tokens to the
// contraction index serves as long as V uses the same one.  V^T's fragments are made in registers: a lane loads DH / 16 channels
// of each of its eight tokens (whole rows per instruction) and transposes the 8 x 8 block with byte permutes.
// fp32 probabilities keep their precision: p is cut into three bf16 parts that add up to it exactly (8 + 8 + 8 mantissa bits).  Every
// head has 16 / REP columns with the same scores; the first three of them take one part each, and their sums are added at the
// end (REP = 8: a head's two columns take two parts, the third goes through a second product).  A part that is zero would turn an
// infinite value into a NaN, so every part is the smallest normal number at least, those of rows past the end too (they repeat the last one);
// to a finite sum that adds 2^-126 of a value.  The sums are not normalised until the end and p may reach 2^kDsLazy: values
// beyond the largest float / (2^kDsLazy times the tokens of a wavefront) can overflow.
//
// Index cache: values are gathered from the codebook into the same registers, by codes that wait in LDS.  Key scores either the
// same way (gather and multiply), or (TABLE) as sums of entries of a table [group][codeword][head] of query-codeword products that
// the workgroup builds in LDS first; the columns of a head then look up one group each and add up.
//
// What bounds it: requests in flight per unit.  A unit brings in ~35 GB/s of local rows (16 KB per wavefront and tile, the next tile on
// its way while one is worked on) and ~43 GB/s of codeword pieces from the second-level cache, whichever other units do.  The whole step
// with the merge, against tables from a launch of their own and multiply-adds on the vector ALU: 32 769 + 98 304 rows of eight KV
// heads of 128 82.1 -> 52.3 us (2.9 TB/s of the bytes it needs), 1 025 + 3 072 rows 21.4 -> 13.2 us.
//
// NGH: groups of a head when they are whole groups of the head (1, 2 or 4 of DH / NGH channels); 0: any other cut into groups of whole
// 16-byte pieces (the codes are then read one by one).
// ------------------------------------------------------------------------------------------------
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
#define DS_INLINE __attribute__((always_inline))
constexpr int kDsTile = 32;
constexpr float kDsLazy = 8.f;       // base-2 units a score may exceed the running reference by before the sums are rescaled
constexpr int kDsCus = 256;          // compute units of the device the launch shapes are chosen for

__device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// the value of the lane whose number differs in bit 0 (X = 1) or bit 1 (X = 2)
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
    constexpr int kPerm = X == 1 ? 0xB1 : 0x4E;
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kPerm, 0xF, 0xF, true));
}

// Cache, codes and codebooks are read through pointers that are marked as global memory: behind the lambdas below the compiler no
// longer sees that they come from the kernel's arguments and would take the slower generic loads.
typedef const __attribute__((address_space(1))) char* gbytes;
// what a wavefront reads as one, by a scalar load: a vector load would be waited for behind all rows in flight (501 + 1505 rows, some lost: 10.26 us, 9.80 so)
typedef const __attribute__((address_space(4))) uint32_t* cwords;
template <typename V>
__device__ __forceinline__ V ld_global(gbytes at) { return *reinterpret_cast<const __attribute__((address_space(1))) V*>(at); }
__device__ __forceinline__ int ld_code(gbytes codes, int code16, int64_t i, int K) {
    const int c = code16 ? (int)ld_global<uint16_t>(codes + 2 * i) : (int)ld_global<uint8_t>(codes + i);
    return c < K ? c : K - 1;
}

template <int DH, int REP, int WAVES, int NGH, bool TABLE>
__global__ __launch_bounds__(64 * WAVES, 2) void decode_stream_kernel(const DecodeParams p) {
    constexpr int KC = DH / 32;       // contraction steps of a score
    constexpr int VCH = DH / 16;      // value channels per lane
    constexpr int P = 16 / REP;       // columns per head
    constexpr bool SPLIT2 = P == 2;
    using Piece = std::conditional_t<DH == 128, u32x4, u32x2>;
    struct Values {
        Piece t[8];                   // one piece of VCH channels per token
    };
    struct Keys {
        u32x4 t[2][KC];               // A operands of the two 16-token halves
    };
    extern __shared__ __align__(16) char ds_lds[];
    __shared__ float ml[WAVES][REP][2];
    __shared__ uint16_t stage[NGH > 0 ? WAVES : 1][2][2][32][4];      // codes of a tile: [slot][key | value][token][group]

    // the arguments arrive together; each branch asking for its own is another trip to them
    asm volatile("" ::"s"(p.q), "s"(p.k_loc), "s"(p.v_loc), "s"(p.codes_k), "s"(p.codes_v), "s"(p.valid_bits), "s"(p.cb_k), "s"(p.cb_v), "s"(p.part), "s"(p.Hq),
                 "s"(p.Hkv), "s"(p.n_local), "s"(p.n_nonlocal), "s"(p.G), "s"(p.K), "s"(p.dg), "s"(p.code16), "s"(p.n_chunks_loc), "s"(p.n_chunks_nl),
                 "s"(p.scale));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4;
    const int head = col / P, part = col % P;
    const int j = blockIdx.y, chunk = blockIdx.x;
    const int c_head = j * DH;
    const int K = p.K, dg = NGH > 0 ? DH / (NGH > 0 ? NGH : 1) : p.dg, G = p.G, code16 = p.code16;
    const gbytes codes_k = (gbytes)p.codes_k, codes_v = (gbytes)p.codes_v, cb_k = (gbytes)p.cb_k;
    const cwords bits = (cwords)p.valid_bits;

    // B operand of the scores
    bf16x8 qf[KC];
    {
        const gbytes q = (gbytes)p.q + ((int64_t)(j * REP + head) * DH + 8 * g) * 2;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) qf[kc] = __builtin_bit_cast(bf16x8, ld_global<u32x4>(q + 64 * kc));
    }
    const float sl2 = p.scale * 1.4426950408889634f;
    // what a column takes off p before the upper half of the rest is its part: nothing, the first, the first two parts
    const uint32_t off1 = part >= 1 ? 0xffff0000u : 0u, off2 = part >= 2 ? 0xffff0000u : 0u;

    f32x4 acc[VCH], acc_lo[SPLIT2 ? VCH : 1];
#pragma unroll
    for (int c = 0; c < VCH; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < (SPLIT2 ? VCH : 1); ++c) acc_lo[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    // scores of a tile (base-2 units, -inf = not attended) and its value pieces into the running sums.  A head's columns have the same
    // scores bit for bit: the parts they take belong to one p
    auto absorb = [&](const float (&s)[8], const Values& v) DS_INLINE {
        float mx = s[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) mx = fmaxf(mx, s[e]);
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kDsLazy) != 0) {
            mx = fmaxf(mx, __shfl_xor(mx, 16));              // the four lanes of a column share one reference
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx);
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < VCH; ++c) acc[c] *= alpha;
            if constexpr (SPLIT2)
#pragma unroll
                for (int c = 0; c < VCH; ++c) acc_lo[c] *= alpha;
            m_run = m_new;
        }
        const float m_ref = m_run == -INFINITY ? 0.f : m_run;
        uint32_t pa[8], pb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float pr = __builtin_amdgcn_exp2f(s[e] - m_ref);
            l_run += pr;
            // every difference is exact, and after two parts at most 8 mantissa bits are left
            const float r1 = pr - __uint_as_float(__float_as_uint(pr) & off1);
            pa[e] = __float_as_uint(SPLIT2 ? r1 : r1 - __uint_as_float(__float_as_uint(r1) & off2));
            if (SPLIT2) {
                const float q1 = pr - __uint_as_float(__float_as_uint(pr) & 0xffff0000u);
                pb[e] = __float_as_uint(q1 - __uint_as_float(__float_as_uint(q1) & 0xffff0000u));
            }
        }
        auto two = [&](uint32_t hi, uint32_t lo) DS_INLINE {      // their upper halves, 2^-126 at least (bits of numbers that are not negative compare as they do)
            const u16x2 parts = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(hi, lo, 0x07060302u)), tiny = {0x0080, 0x0080};
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(parts, tiny));
        };
        auto operand = [&](const uint32_t (&x)[8]) DS_INLINE {
            u32x4 w;
            w.x = two(x[1], x[0]);
            w.y = two(x[3], x[2]);
            w.z = two(x[5], x[4]);
            w.w = two(x[7], x[6]);
            return __builtin_bit_cast(bf16x8, w);
        };
        const bf16x8 pf = operand(pa);
        bf16x8 pf_lo = pf;
        if (SPLIT2) pf_lo = operand(pb);
#pragma unroll
        for (int c = 0; c < VCH; ++c) {
            const uint32_t sel = c & 1 ? 0x07060302u : 0x05040100u;      // channel c of two tokens side by side
            u32x4 w;
            w.x = __builtin_amdgcn_perm(v.t[1][c >> 1], v.t[0][c >> 1], sel);
            w.y = __builtin_amdgcn_perm(v.t[3][c >> 1], v.t[2][c >> 1], sel);
            w.z = __builtin_amdgcn_perm(v.t[5][c >> 1], v.t[4][c >> 1], sel);
            w.w = __builtin_amdgcn_perm(v.t[7][c >> 1], v.t[6][c >> 1], sel);
            const bf16x8 vf = __builtin_bit_cast(bf16x8, w);
            acc[c] = mfma_16x16x32(vf, pf, acc[c]);
            if constexpr (SPLIT2) acc_lo[c] = mfma_16x16x32(vf, pf_lo, acc_lo[c]);
        }
    };
    // token of score / value element e inside a tile
    auto tok = [&](int e) DS_INLINE { return (e < 4 ? 0 : 12) + 4 * g + e; };
    auto score = [&](const Keys& k, float (&s)[8]) DS_INLINE {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) d = mfma_16x16x32(__builtin_bit_cast(bf16x8, k.t[tt][kc]), qf[kc], d);
#pragma unroll
            for (int v = 0; v < 4; ++v) s[4 * tt + v] = d[v] * sl2;
        }
    };

    // the first workgroups of a head walk its local rows, the others its index cache
    const bool local = chunk < p.n_chunks_loc;
    const int n_waves = (local ? p.n_chunks_loc : p.n_chunks_nl) * WAVES;
    const int gw = (chunk - (local ? 0 : p.n_chunks_loc)) * WAVES + wave;
    const int tiles = ((local ? p.n_local : p.n_nonlocal) + kDsTile - 1) / kDsTile;

    if (TABLE && !local) {
        // table[(gi * K + k) * REP + h] = scale * log2(e) * q[h, slice gi] . codeword k: codewords on the M side, 16 at a time
        float* table = reinterpret_cast<float*>(ds_lds);
        constexpr int STEPS = KC / (NGH > 0 && NGH <= KC ? NGH : 1);        // contraction steps of a group
        const int kb = (K + 15) / 16, g0 = j * NGH;
        constexpr int U = 8 / STEPS;                 // tiles in flight per wavefront
#pragma unroll
        for (int gi = 0; gi < NGH; ++gi)
            for (int it0 = wave; it0 < kb; it0 += U * WAVES) {
                u32x4 w[U][STEPS];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const gbytes cw = cb_k + (((int64_t)(g0 + gi) * K + min((it0 + u * WAVES) * 16 + col, K - 1)) * dg + 8 * g) * 2;
#pragma unroll
                    for (int st = 0; st < STEPS; ++st) w[u][st] = ld_global<u32x4>(cw + 64 * st);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int st = 0; st < STEPS; ++st) d = mfma_16x16x32(__builtin_bit_cast(bf16x8, w[u][st]), qf[min(gi * STEPS + st, KC - 1)], d);
                    const int k = (it0 + u * WAVES) * 16 + 4 * g;
                    if (part == 0)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (k + v < K) table[(gi * K + k + v) * REP + head] = d[v] * sl2;
                }
            }
        __syncthreads();
    }

    // The next tile's rows are asked for as soon as their registers are free, and unconditionally (the last tile is a copy of the loop's
    // body), so that a wait covers only what it is for.
    // ---- local rows, streamed
    auto walk_local = [&]() DS_INLINE {
        const int row_b = p.Hkv * DH * 2;
        auto load_k = [&](int t, Keys& k) DS_INLINE {
            const int last = min(p.n_local - t * kDsTile, kDsTile) - 1;          // rows beyond the cache repeat its last one
            const gbytes kb = (gbytes)p.k_loc + ((int64_t)t * kDsTile * row_b + c_head * 2);
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const uint32_t off = (uint32_t)min(16 * tt + col, last) * (uint32_t)row_b + 16u * g;
#pragma unroll
                for (int kc = 0; kc < KC; ++kc) k.t[tt][kc] = ld_global<u32x4>(kb + off + 64 * kc);
            }
        };
        auto load_v = [&](int t, Values& v) DS_INLINE {
            const int last = min(p.n_local - t * kDsTile, kDsTile) - 1;
            const gbytes vb = (gbytes)p.v_loc + ((int64_t)t * kDsTile * row_b + c_head * 2);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v.t[e] = ld_global<Piece>(vb + ((uint32_t)min(tok(e), last) * (uint32_t)row_b + (uint32_t)(2 * VCH * col)));
        };
        auto compute = [&](int t, const Keys& k, const Values& v) DS_INLINE {
            float s[8];
            score(k, s);
            if (t * kDsTile + kDsTile > p.n_local)
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] = t * kDsTile + tok(e) < p.n_local ? s[e] : -INFINITY;
            absorb(s, v);
        };
        int t = gw;
        if (t >= tiles) return;
        Keys ka, kb;
        Values va, vb;
        load_k(t, ka);
        load_v(t, va);
        if constexpr (SPLIT2) {              // twice the accumulators: no registers for a second tile
            for (; t + n_waves < tiles; t += n_waves) {
                compute(t, ka, va);
                load_k(t + n_waves, ka);
                load_v(t + n_waves, va);
            }
            compute(t, ka, va);
            return;
        }
        for (;;) {
            if (t + n_waves >= tiles) { compute(t, ka, va); break; }
            load_k(t + n_waves, kb);
            load_v(t + n_waves, vb);
            compute(t, ka, va);
            t += n_waves;
            if (t + n_waves >= tiles) { compute(t, kb, vb); break; }
            load_k(t + n_waves, ka);
            load_v(t + n_waves, va);
            compute(t, kb, vb);
            t += n_waves;
        }
    };

    // ---- index cache
    const int cv = c_head + VCH * col, gv = cv / dg, off_v = cv - gv * dg;         // this lane's value channels: group, offset inside it
    const gbytes vcb = (gbytes)p.cb_v + ((int64_t)gv * K * dg + off_v) * 2;
    const uint32_t word_b = (uint32_t)dg * 2u;
    auto mask_index = [&](int t, float (&s)[8]) DS_INLINE {
        if (t * kDsTile + kDsTile > p.n_nonlocal || bits) {
            const uint32_t arrived = bits ? bits[t] : 0xffffffffu;      // tiles are half words
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] = t * kDsTile + tok(e) < p.n_nonlocal && ((arrived >> tok(e)) & 1u) ? s[e] : -INFINITY;
        }
    };
    // first piece of this lane's keys: group and byte offset inside a codeword, per contraction step
    int gk[KC];
    uint32_t off_k[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        const int ch = NGH > 0 && dg >= 32 ? 32 * kc : (NGH > 0 ? 0 : c_head) + 32 * kc + 8 * g;       // whole steps inside a group: the same for all lanes
        gk[kc] = ch / dg;
        off_k[kc] = (uint32_t)(ch - gk[kc] * dg) * 2u + (NGH > 0 && dg >= 32 ? 16u * g : 0u);
    }

    auto walk_index = [&]() DS_INLINE {
        // codes of a tile: lane l fetches those of token l % 32 (NGH of them, one aligned load), key codes (l < 32) or value codes,
        // and leaves them in LDS as 16-bit values: under TABLE key codes as byte offsets into a group's table
        const int g0 = j * NGH;
        const gbytes codes = lane < 32 ? codes_k : codes_v;
        const uint32_t mul = TABLE && lane < 32 ? (uint32_t)REP * 4u : 1u;
        auto fetch = [&](int t) DS_INLINE {
            const int64_t at = (int64_t)min(t * kDsTile + (lane & 31), p.n_nonlocal - 1) * G + g0;
            u32x2 raw = {0u, 0u};
            if (code16) {
                if constexpr (NGH == 4) raw = ld_global<u32x2>(codes + 2 * at);
                else if constexpr (NGH == 2) raw.x = ld_global<uint32_t>(codes + 2 * at);
                else raw.x = ld_global<uint16_t>(codes + 2 * at);
            } else {
                if constexpr (NGH == 4) raw.x = ld_global<uint32_t>(codes + at);
                else if constexpr (NGH == 2) raw.x = ld_global<uint16_t>(codes + at);
                else raw.x = ld_global<uint8_t>(codes + at);
            }
            return raw;
        };
        auto put = [&](int slot, const u32x2& raw) DS_INLINE {
            uint32_t c[4];
            c[0] = code16 ? raw.x & 0xffffu : raw.x & 0xffu;
            c[1] = code16 ? raw.x >> 16 : (raw.x >> 8) & 0xffu;
            c[2] = code16 ? raw.y & 0xffffu : (raw.x >> 16) & 0xffu;
            c[3] = code16 ? raw.y >> 16 : raw.x >> 24;
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) c[gi] = min(c[gi], (uint32_t)K - 1u) * mul;
            u32x2 w;
            w.x = c[0] | (c[1] << 16);
            w.y = c[2] | (c[3] << 16);
            *reinterpret_cast<u32x2*>(&stage[wave][slot][lane >> 5][lane & 31][0]) = w;
        };
        auto gather_v = [&](int slot, Values& v) DS_INLINE {
#pragma unroll
            for (int e = 0; e < 8; ++e) v.t[e] = ld_global<Piece>(vcb + (uint32_t)stage[wave][slot][1][tok(e)][gv - g0] * word_b);
        };
        auto gather_k = [&](int slot, Keys& k) DS_INLINE {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int kc = 0; kc < KC; ++kc)
                    k.t[tt][kc] = ld_global<u32x4>(cb_k + ((int64_t)(g0 + gk[kc]) * K * word_b + off_k[kc]) + (uint32_t)stage[wave][slot][0][16 * tt + col][gk[kc]] * word_b);
        };
        // table look-ups: column q of a head takes groups q, q + P, ...; the columns' sums are added pairwise, which gives all of them the same bits
        const int my_group = part % (NGH > 0 ? NGH : 1);
        const char* __restrict__ table = ds_lds + 4 * head + (uint32_t)my_group * ((uint32_t)K * (uint32_t)REP * 4u);
        auto look_up = [&](int slot, float (&s)[8]) DS_INLINE {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float a = *reinterpret_cast<const float*>(table + stage[wave][slot][0][tok(e)][my_group]);
#pragma unroll
                for (int gi = P; gi < NGH; gi += P)
                    a += *reinterpret_cast<const float*>(table + (uint32_t)gi * ((uint32_t)K * (uint32_t)REP * 4u) + stage[wave][slot][0][tok(e)][my_group + gi]);
                if (NGH >= 2) a += quad_xor<1>(a);
                if (NGH >= 4 && P >= 4) a += quad_xor<2>(a);
                s[e] = a;
            }
        };
        int t = gw, slot = 0;
        if (t >= tiles) return;
        u32x2 c = fetch(t);
        put(0, c);
        c = fetch(min(t + n_waves, tiles - 1));
        float s[8];
        if constexpr (TABLE) {
            auto compute = [&](const Values& v) DS_INLINE {
                look_up(slot, s);
                mask_index(t, s);
                absorb(s, v);
                t += n_waves;
                slot ^= 1;
            };
            auto next_codes = [&]() DS_INLINE {
                put(slot ^ 1, c);
                c = fetch(min(t + 2 * n_waves, tiles - 1));
            };
            Values va;
            gather_v(0, va);
            if constexpr (SPLIT2) {
                for (; t + n_waves < tiles;) {
                    next_codes();
                    compute(va);
                    gather_v(slot, va);
                }
                compute(va);
                return;
            }
            Values vb;
            for (;;) {
                if (t + n_waves >= tiles) { compute(va); break; }
                next_codes();
                gather_v(slot ^ 1, vb);
                compute(va);
                if (t + n_waves >= tiles) { compute(vb); break; }
                next_codes();
                gather_v(slot ^ 1, va);
                compute(vb);
            }
        } else {
            Keys k;
            Values v;
            gather_k(0, k);
            gather_v(0, v);
            for (; t + n_waves < tiles; t += n_waves, slot ^= 1) {
                put(slot ^ 1, c);
                c = fetch(min(t + 2 * n_waves, tiles - 1));
                score(k, s);
                mask_index(t, s);
                gather_k(slot ^ 1, k);
                absorb(s, v);
                gather_v(slot ^ 1, v);
            }
            score(k, s);
            mask_index(t, s);
            absorb(s, v);
        }
    };

    auto walk_index_any = [&]() DS_INLINE {
        struct Codes {
            int k[2][KC], v[8];
        };
        auto fetch = [&](int t, Codes& c) DS_INLINE {
            const int last = min(p.n_nonlocal - t * kDsTile, kDsTile) - 1;
            const int64_t row = (int64_t)t * kDsTile * G;
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int kc = 0; kc < KC; ++kc) c.k[tt][kc] = ld_code(codes_k, code16, row + min(16 * tt + col, last) * G + gk[kc], K);
#pragma unroll
            for (int e = 0; e < 8; ++e) c.v[e] = ld_code(codes_v, code16, row + min(tok(e), last) * G + gv, K);
        };
        auto gather_k = [&](const Codes& c, Keys& k) DS_INLINE {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int kc = 0; kc < KC; ++kc)
                    k.t[tt][kc] = ld_global<u32x4>(cb_k + (((int64_t)gk[kc] * K + c.k[tt][kc]) * word_b + off_k[kc]));
        };
        auto gather_v = [&](const Codes& c, Values& v) DS_INLINE {
#pragma unroll
            for (int e = 0; e < 8; ++e) v.t[e] = ld_global<Piece>(vcb + (uint64_t)c.v[e] * word_b);
        };
        int t = gw;
        if (t >= tiles) return;
        Codes c;
        Keys k;
        Values v;
        float s[8];
        fetch(t, c);
        gather_k(c, k);
        gather_v(c, v);
        for (; t + n_waves < tiles; t += n_waves) {
            fetch(t + n_waves, c);
            score(k, s);
            mask_index(t, s);
            gather_k(c, k);
            absorb(s, v);
            gather_v(c, v);
        }
        score(k, s);
        mask_index(t, s);
        absorb(s, v);
    };
    if (local) walk_local();
    else if constexpr (NGH > 0) walk_index();
    else walk_index_any();

    // ---- merge the wavefronts: the parts of a head side by side in its first column, then sums over the wavefronts in order
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (g == 0 && part == 0) {
        ml[wave][head][0] = m_run;
        ml[wave][head][1] = l_run;
    }
    if (TABLE && !local) __syncthreads();                // the table is no longer needed: its place takes the sums
    float* xs = reinterpret_cast<float*>(ds_lds);        // [wave][head][channel]
    constexpr int XS_LD = DH + 4;
#pragma unroll
    for (int c = 0; c < VCH; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float o = acc[c][v] + quad_xor<1>(acc[c][v]);
            if constexpr (SPLIT2) o += acc_lo[c][v];
            else o += quad_xor<2>(acc[c][v]);
            if (part == 0) xs[(wave * REP + head) * XS_LD + VCH * (4 * g + v) + c] = o;
        }
    __syncthreads();
    float* __restrict__ out = p.part + ((int64_t)chunk * p.Hq + (int64_t)j * REP) * (DH + 2);
    for (int i = tid; i < REP * DH; i += 64 * WAVES) {
        const int r = i / DH, d = i - r * DH;
        float M = ml[0][r][0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, ml[w][r][0]);
        const float m_ref = M == -INFINITY ? 0.f : M;
        float o = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float a = __builtin_amdgcn_exp2f(ml[w][r][0] - m_ref);
            o = fmaf(a, xs[(w * REP + r) * XS_LD + d], o);
            l = fmaf(a, ml[w][r][1], l);
        }
        out[r * (DH + 2) + d] = o;
        if (d == 0) {
            out[r * (DH + 2) + DH] = M;
            out[r * (DH + 2) + DH + 1] = l;
        }
    }
}

constexpr int kDsTableWaves = 8, kDsGatherWaves = 4;

DecodeStreamPlan plan_decode_stream(int dtype, int Hq, int Hkv, int dh, int n_local, int n_nonlocal, int K, int dg) {
    DecodeStreamPlan pl{};
    if (dtype != ASTRA_BF16 || (dh != 64 && dh != 128) || dg % 8 != 0) return pl;
    const int rep = Hq / Hkv;
    const int64_t t_loc = ceil_div(n_local, kDsTile), t_nl = ceil_div(n_nonlocal, kDsTile);
    pl.applies = true;
    if (t_loc + t_nl == 0) return pl;
    int wgs;
    // The table costs a workgroup one pass over the head's key codebook (K rows of the head), gathering keys one row per token, and the
    // look-ups are cheaper than the multiplications: it pays from K / 2 tokens per workgroup of a launch of one per unit (8 000 + 24 000
    // rows, K = 1024: 23.4 us against 27.9), but not for short caches, where twice the workgroups on half the wavefronts come first
    // (2 181 + 6 546 rows, K = 256: 16.6 us against 15.0).  Heads of 64 multiply half as much, and look-ups cost the same: a table pays only for one
    // group per head and a small codebook (12 KV heads, 10 000 + 30 000 rows: one group, K = 256 16.6 / 18.9 us; two groups, K = 1024 21.5 / 20.0).
    const int at_least = t_loc > 0 && t_nl > 0 ? 2 : 1;      // many KV heads: one workgroup per kind of tiles, and no partial results beyond those
    const int wgs_table = std::max(at_least, kDsCus / Hkv);
    const size_t table = (size_t)(dh / std::max(dg, 1)) * K * rep * sizeof(float);
    const size_t xs = (size_t)rep * (dh + 4) * sizeof(float);
    pl.table = (dg == dh || dg == dh / 2 || dg == dh / 4) && dg >= 32 && (int64_t)K * rep * 4 <= 65536 && table <= 140 * 1024 &&
               n_nonlocal / wgs_table > std::max(K / 2, 512) && (dh == 128 || (dg == dh && K <= 256));
    // Dealt to the two kinds of tiles in proportion to the time a unit takes for them: a tile of local rows (16 KB from memory) 1.5 times an
    // index tile's (8 KB from the second-level cache).  32 769 + 98 304 rows at ratios of 1 / 1.5 / 2 / 3: 63 / 52 / 55 / 58 us.  Heads of 64 without
    // a table take the same time for both (8 KB either way): 6 000 + 18 000 rows of 12 KV heads 16.4 us dealt evenly, 16.7 at 1.5.
    const bool even = dh == 64 && !pl.table;
    auto local_share = [&](int n) {
        if (t_loc == 0 || t_nl == 0) return t_loc == 0 ? 0 : n;
        const int64_t w_loc = (even ? 2 : 3) * t_loc, w_nl = 2 * t_nl;
        return std::min(std::max((int)((2 * w_loc * n + w_loc + w_nl) / (2 * (w_loc + w_nl))), 1), n - 1);
    };
    if (pl.table) {
        wgs = wgs_table;
        pl.lds = std::max(table, kDsTableWaves * xs);
    } else {
        // two workgroups per unit, or three on heads of 64 if a wavefront then walks fewer tiles (the same rows: 15.2 us; 4 832 + 4 832 rows, two
        // tiles either way: 10.2 with two per unit, 11.5 with three)
        const int most = (int)std::min<int64_t>(ceil_div(t_loc, kDsGatherWaves) + ceil_div(t_nl, kDsGatherWaves), 1 << 20);
        auto walk = [&](int n) {
            const int loc = local_share(n);
            return std::max(loc > 0 ? ceil_div(t_loc, (int64_t)loc * kDsGatherWaves) : 0, n > loc ? ceil_div(t_nl, (int64_t)(n - loc) * kDsGatherWaves) : 0);
        };
        wgs = std::min(std::max(at_least, 2 * kDsCus / Hkv), most);
        const int three = std::min(std::max(at_least, 3 * kDsCus / Hkv), most);
        if (even && at_least == 2 && walk(three) < walk(wgs)) wgs = three;
        pl.lds = kDsGatherWaves * xs;
    }
    pl.wgs_loc = local_share(wgs);
    pl.wgs_nl = wgs - pl.wgs_loc;
    return pl;
}

template <int DH, int REP, int WAVES, int NGH, bool TABLE>
static int launch_form(const DecodeParams& p, const DecodeStreamPlan& pl, hipStream_t s) {
    if (TABLE) {
        static std::atomic<uint64_t> allowed{0};
        const int rc = allow_dynamic_lds(allowed, (const void*)decode_stream_kernel<DH, REP, WAVES, NGH, TABLE>, 150 * 1024);
        if (rc) return rc;
    }
    decode_stream_kernel<DH, REP, WAVES, NGH, TABLE><<<dim3(pl.wgs_loc + pl.wgs_nl, p.Hkv), 64 * WAVES, pl.lds, s>>>(p);
    return ASTRA_OK;
}

template <int DH, int REP, int NGH>
static int launch_ngh(const DecodeParams& p, const DecodeStreamPlan& pl, hipStream_t s) {
    if constexpr (DH / NGH >= 32)
        if (pl.table) return launch_form<DH, REP, kDsTableWaves, NGH, true>(p, pl, s);
    return launch_form<DH, REP, kDsGatherWaves, NGH, false>(p, pl, s);
}

template <int DH, int REP>
static int launch_rep(const DecodeParams& p, const DecodeStreamPlan& pl, hipStream_t s) {
    if (p.dg == DH) return launch_ngh<DH, REP, 1>(p, pl, s);
    if (p.dg == DH / 2) return launch_ngh<DH, REP, 2>(p, pl, s);
    if (p.dg == DH / 4) return launch_ngh<DH, REP, 4>(p, pl, s);
    return launch_form<DH, REP, kDsGatherWaves, 0, false>(p, pl, s);
}

int launch_decode_stream(const DecodeParams& p, const DecodeStreamPlan& pl, hipStream_t s) {
    if (pl.wgs_loc + pl.wgs_nl == 0) return ASTRA_OK;
    switch (p.Hq / p.Hkv * 1000 + p.dh) {
        case 1064: return launch_rep<64, 1>(p, pl, s);
        case 2064: return launch_rep<64, 2>(p, pl, s);
        case 4064: return launch_rep<64, 4>(p, pl, s);
        case 8064: return launch_rep<64, 8>(p, pl, s);
        case 1128: return launch_rep<128, 1>(p, pl, s);
        case 2128: return launch_rep<128, 2>(p, pl, s);
        case 4128: return launch_rep<128, 4>(p, pl, s);
        case 8128: return launch_rep<128, 8>(p, pl, s);
        default: return ASTRA_ERR_UNSUPPORTED;
    }
}

}  // namespace astra
