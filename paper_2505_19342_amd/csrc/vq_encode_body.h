// Fast bf16 encode (paper Sec. 2 "Grouped VQ": nearest codeword per group, lowest index on ties), as a device
// function over caller-provided LDS, so that it can run as a kernel of its own and as extra workgroups of the
// projection launch.
#pragma once
#include <type_traits>

#include "common.h"

namespace astra {

constexpr int kEncCw = 128;       // codewords per LDS tile
constexpr int kEncKt = 64;        // contraction values per LDS tile
constexpr int kEncBufs = 4;       // LDS tile buffers of the fast path: transfers run three tiles ahead
constexpr int kEncCbSlots = kEncCw * 8;          // 16-byte slots of one codebook tile (16 KiB)
constexpr int kEncCnSlots = kEncCw / 4;          // 16-byte slots of one tile of norms (512 B)

__device__ __forceinline__ int enc_swz(int r) { return (r >> 1) & 7; }

// What the encode needs, as plain values (also travels inside the projection launch's argument block).
struct EncodeJob {
    const void* x;            // [n_tokens, ldx] bf16
    const void* codebook;     // [G, K, dg] bf16
    const float* cnorm;       // [G, K]
    void* codes;              // [n_tokens, G] uint8 / uint16
    int64_t ldx;
    int32_t n_tokens, G, K, dg;
    int32_t code_bytes;       // 1 or 2
    int32_t tb;               // 32-token blocks per wavefront, 1 or 2
    int32_t n_tb;             // token blocks per group (of THREADS/2 * tb tokens)
};

// ------------------------------------------------------------------------------------------------
// Groups of at most 64 values (dg a multiple of 8), and of 128 and 256 on tiles of 64 codewords.  An item is a group and a block of tokens; a workgroup of THREADS threads takes a run of items,
// 32 TB tokens per wavefront (on the N side of the 32x32x16 MFMA), and walks the group's codebook in tiles of 128 codewords (M side) for each.
//   - The score is kept as a distance, ||c||^2 - 2 x.c: the token fragments are loaded negated and doubled (exact in bf16).  The accumulation of up to four
//     steps starts from ||c||^2, so no vector-ALU work is spent on forming the score.  That of 8 or 16 steps rounds every partial sum at the size of ||c||^2,
//     about dg.  Codebooks of 2^17 elements and more, whose score products the body stands in for, are as accurate as those (ONCE): -2 x.c is summed by
//     itself and ||c||^2 added once, an addition per score.  Smaller ones start from ||c||^2, as in vq_encode_bf16_wide_kernel, which had them before (groups of
//     128, K = 256, 9901 tokens: 32.6 us, 37.2 with the addition), but for the single group of a layer, which has products whatever its codebook's size (128 wide,
//     K = 512, 8500 rows: layer 112.1 us from the norms, 113.3 now, 116.1 as products).
//   - Codebook tiles and their norms go from global memory straight into a ring of four LDS buffers, two to three tiles ahead, without a break
//     between items.  Pieces beyond dg are never transferred; the one such slot a contraction step can read (dg an odd multiple of 8) is
//     zeroed once by the caller (vq_encode_fast_zero_lds, when vq_encode_fast_needs_zero) and meets zero token values.
//   - A tile is UNITS units of two accumulators (two token blocks against 32 codewords, or one against 64; groups of 256: one against 32).  While a unit's MFMAs are issued, the
//     fragments of the next one are read and the scores of the one before are taken into the running argmin, so that the matrix core, the LDS and
//     the vector ALU work at the same time whatever the other wavefront of the SIMD does.
//   - The argmin goes by quads, four consecutive codewords in one lane: the minimum of the best so far and them (two instructions), and where that
//     is a new one, the quad's number and its first three scores are kept (a compare and four selects): seven instructions for four scores.  Which of the four it
//     was is worked out once per item.  Strict '<' and the first equal score keep the lowest index.
//   - With TB = 2 a codeword fragment and the norms are read from LDS once for 64 tokens.
// 16384 tokens x 64 groups of 64, K = 1024: 192 us as a kernel of one item of 128 tokens per workgroup with an argmin of a compare and two selects per
// score behind each tile's MFMAs, 150 now (185 with TB = 1); 4096 tokens 52 -> 40, 16384 x 16 groups of 48, K = 256 21 -> 15.  Of the
// 150, the MFMAs alone are about 70.
// cb_lds: kEncBufs * kEncCbSlots slots, cn_lds: kEncBufs * kEncCnSlots slots.  Ends with every wavefront past its last LDS read only after the
// caller's next barrier: callers that make several runs put a barrier between them.
// ------------------------------------------------------------------------------------------------
template <int THREADS>
__device__ __forceinline__ void vq_encode_fast_zero_lds(u32x4* cb_lds) {
    for (int i = threadIdx.x; i < kEncBufs * kEncCbSlots; i += THREADS) cb_lds[i] = u32x4{0u, 0u, 0u, 0u};
}
__device__ __forceinline__ bool vq_encode_fast_needs_zero(int dg) { return (dg & 8) != 0; }

// NKS = ceil(dg / 16) contraction steps; ONCE: the norm is added to the finished sum
template <int THREADS, int TB, int NKS, bool ONCE = false>
__device__ __forceinline__ void vq_encode_fast_run_nks(const EncodeJob& job, int lo, int hi, u32x4* cb_lds, f32x4* cn_lds) {
    constexpr int WAVES = THREADS / 64;
    constexpr int TOKENS = WAVES * 32 * TB;             // tokens per item
    // groups of 128 and 256 values: tiles of 64 codewords, and an item's tokens are asked for when the one before is done (no registers for two);
    // of 256, a unit is one accumulator, 32 codewords against 32 tokens (none for more either)
    constexpr bool WIDE = NKS > 4;
    static_assert(!WIDE || (TB == 2 && NKS == 8) || (TB == 1 && NKS == 16), "a tile of 64 codewords is two units of 32");
    static_assert(WIDE || !ONCE, "the norms of one block of codewords are held");
    constexpr int NB = NKS == 16 ? 1 : 2;               // accumulators of a unit
    constexpr int CW = WIDE ? kEncCw / 2 : kEncCw;      // codewords of a tile
    constexpr int PPR = WIDE ? 2 * NKS : 8;             // 16-byte slots of a codeword
    constexpr int CBS = CW * PPR;                       // slots of a tile
    constexpr int ITS = CBS / THREADS;                  // codebook transfers per thread per tile
    constexpr int NORM_LANES = CW / 4 / WAVES;          // lanes per wavefront that fetch 4 norms each
    constexpr int DMA = ITS + 1;                        // transfers of a wavefront per tile: "tile s has landed" is a fixed vmcnt threshold
    constexpr int NA = TB == 2 ? 1 : NB, UNITS = CW / (32 * NA);      // units of a tile, codeword blocks of 32 in one
    if (lo >= hi) return;
    const int K = job.K, dg = job.dg, n_tokens = job.n_tokens, n_tb = job.n_tb;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i32 = lane & 31, h = lane >> 5;
    const int n_pieces = dg >> 3;                       // valid 16-byte pieces per codeword
    const uint32_t row_b = (uint32_t)dg * 2u;
    const int n_tiles = (K + CW - 1) / CW, n_steps = (hi - lo) * n_tiles;

    // ---- transfers.  Slot c = tid + THREADS*it is (codeword c/PPR, physical piece c%PPR) and receives logical piece (c%PPR) ^ swz(c/PPR); swz has period 16
    // codewords and THREADS/PPR codewords separate two `it`.  Byte offsets past the group's last codeword are clamped to its row K-1.
    auto swz_of = [](int r) __attribute__((always_inline)) { return WIDE ? r & 15 : enc_swz(r); };
    const int cw_l = tid / PPR;
    const int piece = (tid % PPR) ^ swz_of(cw_l);
    const bool piece_ok = piece < n_pieces;
    uint32_t cb_off[ITS];
#pragma unroll
    for (int it = 0; it < ITS; ++it) cb_off[it] = (uint32_t)(cw_l + (THREADS / PPR) * it) * row_b + (uint32_t)piece * 16u;
    const uint32_t cb_off_max = (uint32_t)(K - 1) * row_b + (uint32_t)piece * 16u;
    const uint32_t cn_off = (uint32_t)(4 * NORM_LANES * wave + 4 * lane) * 4u, cn_off_max = (uint32_t)(K - 4) * 4u;
    int g = lo / n_tb, block = lo - g * n_tb;      // of the item that is worked on
    const char* s_cb = (const char*)job.codebook + (int64_t)g * K * row_b;                // the tile that is sent next
    const char* s_cn = (const char*)(job.cnorm + (int64_t)g * K);
    int s_block = block, s_tile = 0, s_step = 0;
    auto send_tile = [&]() __attribute__((always_inline)) {
        if (s_step >= n_steps) return;
        const int buf = s_step % kEncBufs;
        const uint32_t base = lds_byte_addr(cb_lds + buf * CBS);
        const uint32_t tile_b = (uint32_t)s_tile * (uint32_t)CW * row_b;
        if (piece_ok) {
#pragma unroll
            for (int it = 0; it < ITS; ++it)
                dma_global_to_lds_16(s_cb, min(cb_off[it] + tile_b, cb_off_max), base + (uint32_t)(64 * (wave + WAVES * it)) * 16u);
        }
        if (lane < NORM_LANES)                          // a tile's norms = WAVES x NORM_LANES lanes x 16 bytes
            dma_global_to_lds_16(s_cn, min(cn_off + (uint32_t)s_tile * (uint32_t)(CW * 4), cn_off_max),
                                 lds_byte_addr(cn_lds + buf * kEncCnSlots) + (uint32_t)wave * (16u * NORM_LANES));
        ++s_step;
        if (++s_tile == n_tiles) {
            s_tile = 0;
            if (++s_block == n_tb) {
                s_block = 0;
                s_cb += (int64_t)K * row_b;
                s_cn += (int64_t)K * 4;
            }
        }
    };

    // ---- tokens: raw values of an item, and as -2x
    u32x4 raw[TB][NKS];
    auto load_tokens = [&](int of_g, int of_block) __attribute__((always_inline)) {
        const int t0 = of_block * TOKENS + wave * (32 * TB) + i32;
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const uint16_t* xrow = (const uint16_t*)job.x + (int64_t)min(t0 + 32 * b, n_tokens - 1) * job.ldx + (int64_t)of_g * dg;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const int k = 16 * ks + 8 * h;
                raw[b][ks] = *reinterpret_cast<const u32x4*>(xrow + (k < dg ? k : 0));
            }
        }
    };
    bf16x8 xf[TB][NKS];
    auto take_tokens = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const bf16x8 xv = __builtin_bit_cast(bf16x8, raw[b][ks]);
                const bool in = 16 * ks + 8 * h < dg;
#pragma unroll
                for (int e = 0; e < 8; ++e) xf[b][ks][e] = (__bf16)(in ? -2.f * (float)xv[e] : 0.f);
            }
    };

    // ---- fragments of unit u of the tile in LDS buffer buf: rows 32 mb + lane % 32 (A), norms of rows 32 mb + 8q + 4h .. + 3
    constexpr int NR = NKS == 16 ? 8 : NKS;             // of groups of 256, half a unit's fragments are held
    bf16x8 fa[NR][NA];
    f32x16 cn[NA];
    auto block_of = [&](int u, int n) { return NA == 1 ? u : 2 * u + n; };
    auto read_a = [&](int buf, int u, int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NA; ++n)
            fa[ks % NR][n] = __builtin_bit_cast(bf16x8, cb_lds[buf * CBS + (block_of(u, n) * 32 + i32) * PPR + ((2 * ks + h) ^ swz_of(i32))]);
    };
    auto read_cn_quad = [&](int buf, int u, int n, int q) __attribute__((always_inline)) {
        const f32x4 v = cn_lds[buf * kEncCnSlots + block_of(u, n) * 8 + 2 * q + h];
#pragma unroll
        for (int e = 0; e < 4; ++e) cn[n][4 * q + e] = v[e];
    };
    auto read_cn = [&](int buf, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NA; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) read_cn_quad(buf, u, n, q);
    };
    // codewords past K (the last tile of a K that is no multiple of a tile's; lim: those of the tile and beyond) are infinitely far
    auto mask_cn = [&](int u, int lim) __attribute__((always_inline)) {
        if (lim >= CW) return;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
            const int left = lim - 32 * block_of(u, n) - 4 * h;
#pragma unroll
            for (int v = 0; v < 16; ++v) cn[n][v] = acc_row(v, 0) >= left ? INFINITY : cn[n][v];
        }
    };

    // ---- running argmin of this lane's tokens: quad grp (0..15) of tile til, and the quad's first three scores
    float best[TB], best_in[TB], k0[TB], k1[TB], k2[TB];
    int grp[TB], til[TB];
    f32x16 acc[2][NB];
    auto score = [&](int set, int j, int v) __attribute__((always_inline)) { return ONCE ? cn[0][v] + acc[set][j][v] : acc[set][j][v]; };
    auto take_quad = [&](int set, int u, int i) __attribute__((always_inline)) {         // i-th of a unit's 4 NB
        const int j = i >> 2, q = i & 3, b = TB == 2 ? j : 0;
        const float s0 = score(set, j, 4 * q), s1 = score(set, j, 4 * q + 1), s2 = score(set, j, 4 * q + 2), s3 = score(set, j, 4 * q + 3);
        const float m = fminf(fminf(fminf(fminf(best[b], s0), s1), s2), s3);
        const bool better = m < best[b];
        best[b] = m;
        grp[b] = better ? block_of(u, j) * 4 + q : grp[b];
        k0[b] = better ? s0 : k0[b];
        k1[b] = better ? s1 : k1[b];
        k2[b] = better ? s2 : k2[b];
    };
    auto close_tile = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            til[b] = best[b] < best_in[b] ? t : til[b];
            best_in[b] = best[b];
        }
    };

    // the first tiles are on their way before the token values are asked for: the two latencies overlap
#pragma unroll
    for (int t = 0; t < kEncBufs - 1; ++t) send_tile();
    load_tokens(g, block);
    take_tokens();
    wait_vmem_all();
    __syncthreads();
    if (!ONCE) read_cn(0, 0);
#pragma unroll
    for (int ks = 0; ks < NR; ++ks) read_a(0, 0, ks);

    int step = 0;
    for (int item = lo; item < hi; ++item) {
        const bool wraps = block + 1 == n_tb;                   // the next item is the next group's first
        const int next_g = wraps ? g + 1 : g, next_block = wraps ? 0 : block + 1;
        const int t_load = n_tiles > 3 ? n_tiles - 3 : 0;       // the next item's tokens are asked for two tiles before the end
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            best[b] = best_in[b] = k0[b] = k1[b] = k2[b] = INFINITY;
            grp[b] = til[b] = 0;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[1][j][v] = INFINITY;         // in the place of the unit before the first
        if (ONCE) cn[0] = f32x16{};
        for (int t = 0; t < n_tiles; ++t, ++step) {
            const int buf = step % kEncBufs, next_buf = (step + 1) % kEncBufs;
            const int lim = K - t * CW;                         // codewords of this tile and beyond
#pragma unroll
            for (int u = 0; u < UNITS; ++u) {
                if (u == UNITS - 1 && step + 1 < n_steps) {
                    // the next tile has landed (the one after it may be outstanding, and the tokens asked for a tile ago); every wavefront is done with
                    // the tile before this one, whose place takes the one three ahead
                    if (step + 2 < n_steps) {
                        if (!WIDE && t == t_load + 1 && item + 1 < hi) wait_vmem<DMA + TB * NKS>();
                        else wait_vmem<DMA>();
                    } else {
                        wait_vmem_all();
                    }
                    __syncthreads();
                    if (!WIDE && t == t_load && item + 1 < hi) load_tokens(next_g, next_block);
                    send_tile();
                }
                if (!ONCE) mask_cn(u, lim);
                const int set = u & 1, rb = u == UNITS - 1 ? next_buf : buf, ru = (u + 1) % UNITS, pu = (u + UNITS - 1) % UNITS;
#pragma unroll
                for (int i = 0; i < NB * NKS; ++i) {
                    const int ks = i / NB, j = i % NB;
                    acc[set][j] = mfma_32x32x16(fa[ks % NR][NA == 1 ? 0 : j], xf[TB == 2 ? j : 0][ks],
                                                ks > 0 ? acc[set][j] : ONCE ? f32x16{} : cn[NA == 1 ? 0 : j]);
                    if (!ONCE && i == 1) read_cn(rb, ru);
                    if (j == NB - 1) {
                        if (ks + NR < NKS) read_a(buf, u, ks + NR);
                        else read_a(rb, ru, ks + NR - NKS);
                    }
#pragma unroll
                    for (int x = i * 4 / NKS; x < (i + 1) * 4 / NKS; ++x) {
                        take_quad(set ^ 1, pu, x);
                        if (ONCE && (x >> 2) == NB - 1) read_cn_quad(buf, u, 0, x & 3);      // this unit's, in the place of the ones just used
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (u == 0) close_tile(t - 1);                  // the quads were those of the tile before
                // the argmin is worked out here: moved behind the branches that follow, it would keep the scores of several units alive
#pragma unroll
                for (int b = 0; b < TB; ++b) asm volatile("" : "+v"(best[b]), "+v"(grp[b]), "+v"(k0[b]), "+v"(k1[b]), "+v"(k2[b]), "+v"(til[b]));
                if (ONCE) mask_cn(u, lim);
            }
        }
#pragma unroll
        for (int x = 0; x < 4 * NB; ++x) take_quad(1, UNITS - 1, x);
        close_tile(n_tiles - 1);
        const int t0 = block * TOKENS + wave * (32 * TB) + i32;
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int e = k0[b] == best[b] ? 0 : k1[b] == best[b] ? 1 : k2[b] == best[b] ? 2 : 3;
            int arg = til[b] * CW + (grp[b] >> 2) * 32 + (grp[b] & 3) * 8 + 4 * h + e;
            // merge the two half-waves that hold the same token
            const float ob = __shfl_xor(best[b], 32);
            const int oa = __shfl_xor(arg, 32);
            if (ob < best[b] || (ob == best[b] && oa < arg)) arg = oa;
            if (h == 0 && t0 + 32 * b < n_tokens) {
                const int64_t at = (int64_t)(t0 + 32 * b) * job.G + g;
                if (job.code_bytes == 2) ((uint16_t*)job.codes)[at] = (uint16_t)arg;
                else ((uint8_t*)job.codes)[at] = (uint8_t)arg;
            }
        }
        if (WIDE && item + 1 < hi) load_tokens(next_g, next_block);
        if (item + 1 < hi) take_tokens();
        g = next_g;
        block = next_block;
    }
}

template <int THREADS, int TB>
__device__ __forceinline__ void vq_encode_fast_run_tb(const EncodeJob& job, int lo, int hi, u32x4* cb_lds, f32x4* cn_lds) {
    switch ((job.dg + 15) >> 4) {
        case 1: vq_encode_fast_run_nks<THREADS, TB, 1>(job, lo, hi, cb_lds, cn_lds); break;
        case 2: vq_encode_fast_run_nks<THREADS, TB, 2>(job, lo, hi, cb_lds, cn_lds); break;
        case 3: vq_encode_fast_run_nks<THREADS, TB, 3>(job, lo, hi, cb_lds, cn_lds); break;
        default: vq_encode_fast_run_nks<THREADS, TB, 4>(job, lo, hi, cb_lds, cn_lds); break;
    }
}

// items lo .. hi - 1 of the job; both: the job may have one or two blocks per wavefront, else it has one
template <int THREADS, bool BOTH>
__device__ __forceinline__ void vq_encode_fast_run(const EncodeJob& job, int lo, int hi, u32x4* cb_lds, f32x4* cn_lds) {
    if (BOTH && job.tb == 2) vq_encode_fast_run_tb<THREADS, 2>(job, lo, hi, cb_lds, cn_lds);
    else vq_encode_fast_run_tb<THREADS, 1>(job, lo, hi, cb_lds, cn_lds);
}

// Groups of 64 NCH values, few tokens: 32 tokens of a group per workgroup, whose eight wavefronts share its codewords, blocks of 32 dealt in turn.  Every
// wavefront streams its blocks in steps of 64 values through an LDS ring of its own (no barrier in the loop), four steps in flight, in transfers of whole
// 128-byte lines.  What bounds it: a unit's operand intake (64 B/clk) and the latency before it.  One round at K = 1024, 256 workgroups, against
// vq_encode_bf16_wide_kernel, which reads 16 bytes of 64 rows with an instruction: groups of 256 13.9 us, 23.8 before (37 as score products), of 128 9.8, 20.0.
constexpr int kStreamWaves = 8, kStreamRing = 4, kStreamTokens = 32;
constexpr int kStreamSlots = kStreamWaves * kStreamRing * 32 * 8, kStreamCnSlots = kStreamWaves * kStreamRing * 8;      // 16-byte slots of codewords, of norms
// item vid (group-major) of the job.  All kStreamWaves wavefronts come here.
template <int NCH>
__device__ __forceinline__ void vq_encode_stream_run(const EncodeJob& job, int vid, u32x4* cb_ring, f32x4* cn_ring, float (*m_val)[kStreamTokens],
                                                     int (*m_arg)[kStreamTokens]) {
    constexpr int PER = 5;                                          // transfers of a step: four of codewords, one of the block's norms
    auto cb_lds = reinterpret_cast<u32x4(*)[kStreamRing][32 * 8]>(cb_ring);     // a step: [32 codewords][8 pieces of 8 bf16], swizzled
    auto cn_lds = reinterpret_cast<f32x4(*)[kStreamRing][8]>(cn_ring);
    const int g = vid / job.n_tb, t0 = (vid - g * job.n_tb) * kStreamTokens;
    const int K = job.K, n_tokens = job.n_tokens;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i32 = lane & 31, h = lane >> 5;
    constexpr uint32_t row_b = 128u * NCH;
    const int n_blocks = (K + 31) >> 5, n_mine = (n_blocks - wave + kStreamWaves - 1) / kStreamWaves, n_steps = max(n_mine, 0) * NCH;
    const char* __restrict__ cb = (const char*)job.codebook + (int64_t)g * K * row_b;
    const char* __restrict__ cn = (const char*)(job.cnorm + (int64_t)g * K);

    // transfer i of a step: lane l fetches piece (l % 8) ^ (row % 8) of row 8 i + l / 8; rows past K are row K - 1
    int s_row = 32 * wave, s_ch = 0, s_step = 0;
    const int l_row = lane >> 3;
    const uint32_t l_piece = (uint32_t)((lane & 7) ^ l_row) * 16u;
    auto send = [&]() __attribute__((always_inline)) {
        if (s_step >= n_steps) return;
        const int ring = s_step % kStreamRing;
        const uint32_t base = lds_byte_addr(&cb_lds[wave][ring][0]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dma_global_to_lds_16(cb, (uint32_t)min(s_row + 8 * i + l_row, K - 1) * row_b + (uint32_t)s_ch * 128u + l_piece, base + 1024u * i);
        if (lane < 8) dma_global_to_lds_16(cn, (uint32_t)min(s_row + 4 * lane, K - 4) * 4u, lds_byte_addr(&cn_lds[wave][ring][0]));
        ++s_step;
        if (++s_ch == NCH) {
            s_ch = 0;
            s_row += 32 * kStreamWaves;
        }
    };
#pragma unroll
    for (int i = 0; i < kStreamRing; ++i) send();

    // the tokens as -2x (exact in bf16): the sums and the norms, added once at the end, are distances
    bf16x8 xf[4 * NCH];
    {
        const uint16_t* xrow = (const uint16_t*)job.x + (int64_t)min(t0 + i32, n_tokens - 1) * job.ldx + (int64_t)g * (64 * NCH) + 8 * h;
        u32x4 raw[4 * NCH];
#pragma unroll
        for (int ks = 0; ks < 4 * NCH; ++ks) raw[ks] = *reinterpret_cast<const u32x4*>(xrow + 16 * ks);
#pragma unroll
        for (int ks = 0; ks < 4 * NCH; ++ks) {
            const bf16x8 xv = __builtin_bit_cast(bf16x8, raw[ks]);
#pragma unroll
            for (int e = 0; e < 8; ++e) xf[ks][e] = (__bf16)(-2.f * (float)xv[e]);
        }
    }
    float best = INFINITY;
    int arg = 0, step = 0;
    for (int t = 0; t < n_mine; ++t) {
        f32x16 acc = {}, norm;
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch, ++step) {
            // this step has landed: the three sent after it may be outstanding
            if (step + kStreamRing <= n_steps) wait_vmem<PER * (kStreamRing - 1)>();
            else wait_vmem_all();
            const int ring = step % kStreamRing;
            bf16x8 fa[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) fa[ks] = __builtin_bit_cast(bf16x8, cb_lds[wave][ring][i32 * 8 + ((2 * ks + h) ^ (i32 & 7))]);
            if (ch == NCH - 1) {
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const f32x4 v = cn_lds[wave][ring][2 * p + h];
#pragma unroll
                    for (int e = 0; e < 4; ++e) norm[4 * p + e] = v[e];
                }
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt 0: the step is in registers, its place is free
            asm volatile("" ::: "memory");
            send();
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) acc = mfma_32x32x16(fa[ks], xf[4 * ch + ks], acc);
        }
        const int cw0 = 32 * (wave + kStreamWaves * t);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int cw = cw0 + acc_row(v, h);
            const float d = norm[v] + acc[v];
            const bool better = cw < K && d < best;
            best = better ? d : best;
            arg = better ? cw : arg;
        }
    }
    {
        const float ob = __shfl_xor(best, 32);
        const int oa = __shfl_xor(arg, 32);
        if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
    }
    if (h == 0) { m_val[wave][i32] = best; m_arg[wave][i32] = arg; }
    __syncthreads();
    if (tid < kStreamTokens && t0 + tid < n_tokens) {
        best = m_val[0][tid];
        arg = m_arg[0][tid];
#pragma unroll
        for (int w = 1; w < kStreamWaves; ++w) {
            const float ob = m_val[w][tid];
            const int oa = m_arg[w][tid];
            if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
        }
        const int64_t at = (int64_t)(t0 + tid) * job.G + g;
        if (job.code_bytes == 2) ((uint16_t*)job.codes)[at] = (uint16_t)arg;
        else ((uint8_t*)job.codes)[at] = (uint8_t)arg;
    }
}

// Token blocks per wavefront for an encode that `wgs` workgroups of 512 threads share.  Two take 1.6 times as long as one (16384 tokens x 64 groups, K = 1024:
// 150 us, 185 with one), so they pay where one block each makes more than 1.6 times the rounds.
inline int vq_encode_blocks(const EncodeJob& e, int64_t wgs) {
    const int64_t one = ceil_div(e.n_tokens, (int64_t)256) * e.G, two = ceil_div(e.n_tokens, (int64_t)512) * e.G;
    return 1.6 * (double)ceil_div(two, wgs) < (double)ceil_div(one, wgs) ? 2 : 1;
}

// Groups of 128, 192 and 256 values are taken by vq_encode_bf16_stream_kernel, 32 tokens per workgroup.  Of 256 values, codebooks of about a block of 32 codewords
// for each of the eight wavefronts stay with vq_encode_bf16_wide_kernel (wide / streamed, us, 16 groups and 64 tokens, the same within 1 % for 4 to 32 groups and
// up to 500 tokens: K = 136 6.9 / 6.6, 192 7.2 / 7.0, 224 7.6 / 7.5, 256 7.9 / 8.1, 288 9.0 / 8.3, 320 9.4 / 8.4; 17 tokens 7.6 / 6.9 at 256).
inline bool vq_encode_stream_fits(int K, int dg, int64_t ldx) {
    return dg > kEncKt && dg <= 256 && dg % 64 == 0 && K % 4 == 0 && ldx % 8 == 0 && (int64_t)K * dg * 2 < ((int64_t)1 << 31);
}
inline bool vq_encode_stream_ok(int K, int dg, int64_t ldx) { return vq_encode_stream_fits(K, dg, ldx) && (dg < 256 || K <= 224 || K > 256); }
// 16-byte transfers to LDS: arrays that start off such a boundary stay with the kernel for wide groups
inline bool vq_encode_on_16(const void* x, const void* codebook, const void* cnorm) {
    return ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(codebook) | reinterpret_cast<uintptr_t>(cnorm)) & 15) == 0;
}
// Beyond that kernel's second round groups of 128 and 256 go through the body in kernels of their own (64 and 32 tokens per wavefront); beyond its first where
// neither the walk nor the launch is long.  The body's items cost 21 and 30 us at K = 1024, the other's rounds 9.8 and 14.  Streamed / body: 512 tokens x 32 groups
// of 128 K = 16 6.6 / 7.1, 64 7.1 / 6.9, 256 10.5 / 10.0, 768 16.1 / 18.5, 1024 18.1 / 22.6, 700 tokens 25.6 / 23.1; 1000 x 16 groups of 256 K = 32 7.8 / 9.8,
// 256 15.8 / 13.9, 512 20.0 / 19.3, 768 23.3 / 24.9, 1024 26.1 / 29.8, 1531 tokens 38.5 / 30.8.
inline bool vq_encode_fast_wide(int64_t n_tokens, int G, int K, int dg, int64_t ldx) {
    const int64_t blocks = ceil_div(n_tokens, (int64_t)32) * G;
    return (dg == 128 || dg == 256) && K % 4 == 0 && ldx % 8 == 0 && (int64_t)K * dg * 2 < ((int64_t)1 << 31) &&
           (blocks > 512 || (blocks > 256 && K > 32 && K <= 512));
}
// Where such groups are better off without score products: of 128 where the products would be more than one launch, of 192 and 256 where they would be
// three or more, or two with more than 192 tokens (with / without scores: 16 groups of 256, K = 1024, 17 tokens 14.2 / 11.4 us, 128 19.7 / 13.0, 400 35.9 / 13.8; K = 4096 40 tokens 27.6 / 29.4,
// 250 45.5 / 31.7; 8 groups 100 tokens, K = 768 11.7 / 11.4, 4096 23.3 / 29.3, 500 39.8 / 30.4; 8 of 192, K = 2048 64 tokens 13.9 / 15.8, 500 29.8 / 16.7,
// K = 1024 2000 tokens 38.7 / 21.7, 16384 292 / 161);
// and with few groups once all units have a block, of 256 with up to 8 groups one and a half (4096 codewords, 2 groups: 4300 tokens 80 / 93, 8192 143 / 96).
inline bool vq_encode_without_scores(int64_t n_tokens, int G, int K, int dg, int64_t ldx) {
    if (dg == 128 && G > kMaxGemmProblems) return true;
    if (!vq_encode_stream_fits(K, dg, ldx)) return false;
    if (G > kMaxGemmProblems && n_tokens > 192) return true;
    if (G > 2 * kMaxGemmProblems && K <= 1024) return true;
    const int64_t blocks = ceil_div(n_tokens, (int64_t)32) * G;
    return dg == 128 ? blocks > 256 : dg == 256 && blocks > (G > 8 ? 256 : 384);
}

// true when the fast body handles this configuration
inline bool vq_encode_fast_ok(int K, int dg) {
    return dg <= kEncKt && dg % 8 == 0 && K % 4 == 0 && (int64_t)K * dg * 2 < ((int64_t)1 << 31);
}

}  // namespace astra
