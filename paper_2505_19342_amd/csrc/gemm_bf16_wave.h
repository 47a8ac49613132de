// The bf16 product C[M,N] = A[M,K] . B[N,K]^T for launches that a few large tiles cannot fill: short sequences, narrow outputs
// (paper: the projections named under Eq. 1, and the MLP of the block around the layer, Sec. 3.1).
#pragma once
#include "gemm_bf16_tile.h"

namespace astra {

// ------------------------------------------------------------------------------------------------
// A workgroup of four wavefronts owns a 32 MT x 32 NT output tile, and every wavefront computes ALL of it over a quarter of the
// contraction: the 64-deep slices w, w + 4, w + 8, ...  It brings its own operand slices into its own ring of ST stages in LDS by
// direct transfers (eight rows of 128 bytes per instruction, XOR-swizzled as in the tile kernel), so that nothing in the loop is
// shared between wavefronts and there is no barrier in it: a wavefront waits for its own transfers only, and all stages of the ring
// are in flight at once.  The four partial tiles are added through LDS in wavefront order at the end, by threads that own four
// consecutive columns of a row, whatever the store.  B is the MFMA's M side, so that a lane holds four consecutive columns.
//
// What bounds it: a compute unit's intake through its vector L1 (about 50 of the 64 B/clk are reached) and one memory latency at
// either end.  256 x 768 fp32 outputs on 192 tiles of 32 x 32: 3.3 us at K = 768 and 5.3 at K = 3072, where the tile kernel, with a
// barrier and a transfer round trip per 128 of contraction, took 6.1 and 12.8 us.  The larger tiles trade concurrency for fewer operand
// bytes per flop; with 128 x 128 and one stage the fragments of a whole stage sit in registers while the next one is transferred
// (1024 x 4096 fp32 outputs, K = 4096: 40.3 us; tile kernel on 128 x 128: 42.7).
//
// GATHER: problems with codes rebuild their A rows from the codebook; the tile's codes are copied to LDS first.  Rows beyond M are copies of
// row M - 1 there too: a transposed store writes them into its padding, which attention multiplies by zero.
// ------------------------------------------------------------------------------------------------
constexpr int kWaveThreads = 256;
constexpr int kWaveWaves = kWaveThreads / kWave;

template <int MT, int NT, int ST>
struct WaveShape {
    static constexpr int BM = 32 * MT, BN = 32 * NT, R = BM + BN;
    static constexpr int kStage = R * 128;                                   // bytes of one stage of one wavefront
    static constexpr int kRing = kWaveWaves * ST * kStage;
    static constexpr int LDN = BN + 4;                                       // floats per row of a partial tile
    static constexpr int kRedRows = kWaveWaves * 32 * LDN * 4;               // bytes of 32 rows of the four partial tiles
    static constexpr int MP = kRing / kRedRows >= MT ? MT : (kRing / kRedRows > 0 ? kRing / kRedRows : 1);     // 32-row groups per reduction pass
    static constexpr int kBytes = kRing > MP * kRedRows ? kRing : MP * kRedRows;
};
constexpr int kWaveEncBytes = kEncBufs * (kEncCbSlots + kEncCnSlots) * 16;    // the encode's tiles and norms

template <int MT, int NT, int ST, bool GATHER, bool ENC, int EPI>
__global__ __launch_bounds__(kWaveThreads) void gemm_wave_kernel(const GemmBatch batch) {
    using S = WaveShape<MT, NT, ST>;
    constexpr int BM = S::BM, BN = S::BN, R = S::R, LDN = S::LDN, MP = S::MP;
    constexpr int DA = BM / 8, DB = BN / 8, DM = DA + DB;                     // transfers per stage: A rows, B rows
    constexpr bool HALVES = MT == 4 && NT == 4 && ST == 1;
    extern __shared__ __align__(16) char wv_lds[];

    int vt;
    if (ENC) {
        // workgroups behind the tiles encode the local rows (nothing in the products depends on the codes or the other way round)
        const FusedId id = fused_id(blockIdx.x, gridDim.x - batch.n_enc_wgs, batch.n_enc_wgs);
        if (id.enc) {
            u32x4* cb = reinterpret_cast<u32x4*>(wv_lds);
            f32x4* cn = reinterpret_cast<f32x4*>(wv_lds + kEncBufs * kEncCbSlots * 16);
            const EncodeJob& job = batch.enc;
            if (vq_encode_fast_needs_zero(job.dg)) {
                vq_encode_fast_zero_lds<kWaveThreads>(cb);
                __syncthreads();                           // zero fill done before any transfer lands
            }
            const int n_items = job.G * job.n_tb;
            const int chunk = (n_items + batch.n_enc_wgs - 1) / batch.n_enc_wgs;     // consecutive items share the group
            const int hi = min((id.idx + 1) * chunk, n_items);
            vq_encode_fast_run<kWaveThreads, false>(job, id.idx * chunk, hi, cb, cn);
            return;
        }
        vt = id.idx;
    } else {
        vt = xcd_remap(blockIdx.x, gridDim.x);
    }
    const TileProblem tp = find_problem<EPI != kEpiLayer ? kOneProblem : GATHER || ENC ? kManyProblems : kMaybeOneProblem>(batch, vt);
    const GemmProblem& P = tp.p;
    const int tile = tp.tile, tiles_m = tp.tiles_m;
    const int m0 = (tile % tiles_m) * BM, tn = tile / tiles_m, n0 = tn * BN;
    const int M = P.M, N = P.N, K = P.K;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i32 = lane & 31, h = lane >> 5;
    const bool gather = GATHER && P.codes != nullptr;

    // transfer j of a stage fills rows 8j + lane / 8 of the stage (A rows, then B rows); a lane's piece depends on j's parity only
    const int r8 = lane >> 3;
    const int piece[2] = {(lane & 7) ^ (r8 >> 1), (lane & 7) ^ (4 + (r8 >> 1))};
    const int m_codes = min(m0, M - 1), n_codes = min(BM, M - m_codes);      // rows whose codes the tile holds (one when all of it is padding)
    uint32_t off[DM];
#pragma unroll
    for (int j = 0; j < DM; ++j) {
        if (j < DA) {
            off[j] = (uint32_t)min(m0 + 8 * j + r8, M - 1) * (uint32_t)P.lda * 2u + 16u * piece[j & 1];
        } else {
            int rb = n0 + 8 * (j - DA) + r8;
            if (EPI == kEpiSwiGLU) {                       // the tile's first half of rows: gate rows, second half: up rows of the same columns
                const int rr = 8 * (j - DA) + r8, Fh = N >> 1;
                rb = (rr >= BN / 2 ? Fh : 0) + min(n0 / 2 + rr % (BN / 2), Fh - 1);
            }
            off[j] = (uint32_t)min(rb, N - 1) * (uint32_t)(P.ldb ? P.ldb : K) * 2u + 16u * piece[j & 1];
        }
    }
    char* const ring = wv_lds + wave * (ST * S::kStage);
    const uint32_t ring_a = lds_byte_addr(ring);
    const char* __restrict__ a_base = (const char*)P.a + 128 * wave;
    const char* __restrict__ b_base = (const char*)P.b + 128 * wave;
    const int steps = K / kBK;
    const int n = (steps - wave + kWaveWaves - 1) / kWaveWaves;          // slices of this wavefront

    // gathered rows: the tile's codes, copied to LDS as they lie in memory (rows are contiguous)
    const int G = gather ? P.G : 0, Kc = gather ? P.Kc : 1, dg = gather ? P.dg : 1;
    const uint32_t magic = gather ? (uint32_t)(0x100000000ull / (uint32_t)dg) + 1u : 0u;
    const bool code16 = gather && P.code_bytes == 2;
    const char* const codes_lds = wv_lds + S::kBytes;
    int k_next = wave * kBK;                               // contraction index of the slice whose transfers are issued next
    auto issue_b = [&](int slot) __attribute__((always_inline)) {
        const uint32_t dst = ring_a + (uint32_t)(slot * S::kStage);
#pragma unroll
        for (int j = DA; j < DM; ++j) dma_global_to_lds_16(b_base, off[j], dst + (uint32_t)(j * 1024));
        if (!HALVES) b_base += 128 * kWaveWaves;
    };
    // gathered rows: transfers from .. to - 1 of the slice at contraction index k0
    auto gather_a = [&](int k0, int from, int to, uint32_t dst) __attribute__((always_inline)) {
        uint32_t g_[2], at[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t k = (uint32_t)(k0 + 8 * piece[q]);
            g_[q] = __umulhi(k, magic);
            at[q] = g_[q] * (uint32_t)Kc;
            at[q] = at[q] * (uint32_t)dg + (k - g_[q] * (uint32_t)dg);
        }
#pragma unroll
        for (int j = from; j < to; ++j) {
            const uint32_t x = (uint32_t)min(8 * j + r8, n_codes - 1) * (uint32_t)G + g_[j & 1];
            const uint32_t code = code16 ? (uint32_t)reinterpret_cast<const uint16_t*>(codes_lds)[x] : (uint32_t)reinterpret_cast<const uint8_t*>(codes_lds)[x];
            const uint32_t go = (at[j & 1] + min(code, (uint32_t)Kc - 1u) * (uint32_t)dg) * 2u;
            dma_global_to_lds_16(P.codebook, go, dst + (uint32_t)(j * 1024));
        }
    };
    auto issue_a = [&](int slot) __attribute__((always_inline)) {
        const uint32_t dst = ring_a + (uint32_t)(slot * S::kStage);
        if (GATHER && gather) {
            gather_a(k_next, 0, DA, dst);
        } else {
#pragma unroll
            for (int j = 0; j < DA; ++j) dma_global_to_lds_16(a_base, off[j], dst + (uint32_t)(j * 1024));
            a_base += 128 * kWaveWaves;
        }
        k_next += kBK * kWaveWaves;
    };
    // the first stages: all of their B rows before the codes are copied, which only A rows need
#pragma unroll
    for (int u = 0; u < ST; ++u)
        if (u < n) issue_b(u);
    if (GATHER && gather) {
        const int row_b = G * P.code_bytes;
        const int total = n_codes * row_b;
        const char* __restrict__ src = (const char*)P.codes + (int64_t)m_codes * row_b;
        char* dst = wv_lds + S::kBytes;
        for (int o = tid * 16; o < total; o += kWaveThreads * 16) {
            if (o + 16 <= total) *reinterpret_cast<u32x4*>(dst + o) = *reinterpret_cast<const u32x4*>(src + o);
            else for (int b = o; b < total; ++b) dst[b] = src[b];
        }
        __syncthreads();
    }


    f32x16 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    if constexpr (HALVES) {
        // ---- the slice in halves: rows A0, A1 and columns B0, B1 of 64 each, multiplied as A0 B0, A0 B1, A1 B1, A1 B0.  While one product runs, the half that
        // the next one needs is read into the registers of the half whose last product is over (B1 and the next slice's B0 take each other's), and
        // the same half of the next slice is sent to its place as soon as it is read: three of four halves are always on their way, where a
        // slice read whole left none of them while it was waited for and read.
        bf16x8 ha[2][4][MT / 2], hb[2][4][NT / 2];
        const u32x4* rows = reinterpret_cast<const u32x4*>(ring);
        auto read_a = [&](int half, int ks, int a) __attribute__((always_inline)) {
            ha[half][ks][a] = __builtin_bit_cast(bf16x8, rows[(16 * MT * half + 32 * a + i32) * 8 + ((2 * ks + h) ^ swz(i32))]);
        };
        auto read_b = [&](int half, int slot, int ks, int b) __attribute__((always_inline)) {
            hb[slot][ks][b] = __builtin_bit_cast(bf16x8, rows[(BM + 16 * NT * half + 32 * b + i32) * 8 + ((2 * ks + h) ^ swz(i32))]);
        };
        constexpr int DH = 2 * MT;                           // transfers of a half
        // Gathered rows: the codes of the half sent next are read together with the fragments, so that no transfer waits for its code between the MFMAs
        // (read one by one in front of each transfer, launches of 224 workgroups with K = 4096, layers of 387 + 387 rows: 94.7 us, 83.3 now; 91.6 before slices were halved).
        uint32_t code_q[DH], at_q[2];
        auto read_codes = [&](int half, int slice) __attribute__((always_inline)) {
            uint32_t g_[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t k = (uint32_t)((slice * kWaveWaves + wave) * kBK + 8 * piece[q]);
                g_[q] = __umulhi(k, magic);
                at_q[q] = g_[q] * (uint32_t)Kc * (uint32_t)dg + (k - g_[q] * (uint32_t)dg);
            }
            if (code16) {
#pragma unroll
                for (int j = 0; j < DH; ++j)
                    code_q[j] = reinterpret_cast<const uint16_t*>(codes_lds)[__umul24(min(8 * (half * DH + j) + r8, n_codes - 1), G) + g_[j & 1]];
            } else {
#pragma unroll
                for (int j = 0; j < DH; ++j)
                    code_q[j] = reinterpret_cast<const uint8_t*>(codes_lds)[__umul24(min(8 * (half * DH + j) + r8, n_codes - 1), G) + g_[j & 1]];
            }
        };
        auto send_a = [&](int half, int j, int slice) __attribute__((always_inline)) {
            const uint32_t dst = ring_a + (uint32_t)((half * DH + j) * 1024);
            if (GATHER && gather) dma_global_to_lds_16(P.codebook, (at_q[j & 1] + __umul24(min(code_q[j], (uint32_t)Kc - 1u), dg)) * 2u, dst);
            else dma_global_to_lds_16(a_base + (int64_t)slice * (128 * kWaveWaves), off[half * DH + j], dst);
        };
        auto send_b = [&](int half, int j, int slice) __attribute__((always_inline)) {
            dma_global_to_lds_16(b_base + (int64_t)slice * (128 * kWaveWaves), off[DA + half * DH + j], ring_a + (uint32_t)((DA + half * DH + j) * 1024));
        };
        auto reads_done = [&]() __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt 0: the half is in registers, its place is free
            asm volatile("" ::: "memory");
        };
        // product Q of slice i, whose B0 is in register slot S0; FULL: slice i + 2 exists
        auto product = [&](auto q_tag, auto s_tag, auto full_tag, int i) __attribute__((always_inline)) {
            constexpr int Q = decltype(q_tag)::value, S0 = decltype(s_tag)::value, S1 = S0 ^ 1;
            constexpr bool FULL = decltype(full_tag)::value;
            constexpr int HA = Q >= 2, HB = Q == 1 || Q == 2, SB = HB ? S1 : S0;
            const bool reads = FULL || Q < 2 || i + 1 < n, sends = FULL || i + (Q < 2 ? 1 : 2) < n;
            if (FULL) wait_vmem<3 * DH>();                   // the half read here has landed: the three sent after it may be outstanding
            else if (reads) wait_vmem_all();
            constexpr int NM = 4 * (MT / 2) * (NT / 2);
            if ((Q == 1 || Q == 2) && sends && GATHER && gather) read_codes(Q == 1, i + (Q < 2 ? 1 : 2));
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int ks = m / (NM / 4), a = m / (NT / 2) % (MT / 2), b = m % (NT / 2);
                acc[HA * (MT / 2) + a][HB * (NT / 2) + b] = mfma_32x32x16(hb[SB][ks][b], ha[HA][ks][a], acc[HA * (MT / 2) + a][HB * (NT / 2) + b]);
                if (reads && m < 8) {
                    if (Q == 0) read_b(1, S1, m / 2, m % 2);
                    else if (Q == 1) read_a(1, m / 2, m % 2);
                    else if (Q == 2) read_a(0, m / 2, m % 2);
                    else read_b(0, S1, m / 2, m % 2);
                }
                if (sends && m == 9) reads_done();
                if (sends && m >= 10)
#pragma unroll
                    for (int j = (m - 10) * DH / (NM - 10); j < (m - 9) * DH / (NM - 10); ++j) {
                        if (Q == 0) send_b(1, j, i + 1);
                        else if (Q == 1) send_a(1, j, i + 1);
                        else if (Q == 2) send_a(0, j, i + 2);
                        else send_b(0, j, i + 2);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto slice = [&](auto s_tag, auto full_tag, int i) __attribute__((always_inline)) {
            product(std::integral_constant<int, 0>{}, s_tag, full_tag, i);
            product(std::integral_constant<int, 1>{}, s_tag, full_tag, i);
            product(std::integral_constant<int, 2>{}, s_tag, full_tag, i);
            product(std::integral_constant<int, 3>{}, s_tag, full_tag, i);
        };
        if (n > 0) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {                            // behind the slice's B rows
                if (GATHER && gather) read_codes(half, 0);
#pragma unroll
                for (int j = 0; j < DH; ++j) send_a(half, j, 0);
            }
            wait_vmem<DH>();
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    read_a(0, ks, t);
                    read_b(0, 0, ks, t);
                }
            reads_done();
            if (n > 1) {
                if (GATHER && gather) read_codes(0, 1);
#pragma unroll
                for (int j = 0; j < DH; ++j) send_a(0, j, 1);
#pragma unroll
                for (int j = 0; j < DH; ++j) send_b(0, j, 1);
            }
            int i = 0;
            for (; i + 3 < n; i += 2) {
                slice(std::integral_constant<int, 0>{}, std::true_type{}, i);
                slice(std::integral_constant<int, 1>{}, std::true_type{}, i + 1);
            }
            for (; i < n; i += 2) {
                slice(std::integral_constant<int, 0>{}, std::false_type{}, i);
                if (i + 1 < n) slice(std::integral_constant<int, 1>{}, std::false_type{}, i + 1);
            }
        }
    } else {
    bf16x8 fa[4][MT], fb[4][NT];
    auto read = [&](int slot) __attribute__((always_inline)) {
        const u32x4* s = reinterpret_cast<const u32x4*>(ring + slot * S::kStage);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
            for (int b = 0; b < NT; ++b) fb[ks][b] = __builtin_bit_cast(bf16x8, s[(BM + 32 * b + i32) * 8 + ((2 * ks + h) ^ swz(i32))]);
#pragma unroll
            for (int a = 0; a < MT; ++a) fa[ks][a] = __builtin_bit_cast(bf16x8, s[(32 * a + i32) * 8 + ((2 * ks + h) ^ swz(i32))]);
        }
    };
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b) acc[a][b] = mfma_32x32x16(fb[ks][b], fa[ks][a], acc[a][b]);
    };
    static_assert(ST <= 2, "thresholds of the last stages are written out below");
#pragma unroll
    for (int u = 0; u < ST; ++u)
        if (u < n) issue_a(u);
    if (ST == 2 && n > 1) wait_vmem<DA>();           // the first stage has landed: younger than its A rows are those of the second only
    int i = 0, slot = 0;
    for (; i + ST < n; ++i) {
        wait_vmem<(ST - 1) * DM>();                  // the oldest stage has landed
        read(slot);
        __builtin_amdgcn_s_waitcnt(0xC07F);          // its fragments are in registers (lgkmcnt 0): the slot is free
        asm volatile("" ::: "memory");
        issue_b(slot);
        issue_a(slot);
        multiply();
        slot = slot + 1 == ST ? 0 : slot + 1;
    }
#pragma unroll
    for (int u = ST - 1; u >= 0; --u)
        if (n > u) {                                 // u younger stages are outstanding
            if (u == 1) wait_vmem<DM>();
            else wait_vmem<0>();
            read(slot);
            multiply();
            slot = slot + 1 == ST ? 0 : slot + 1;
        }

    }

    // ---- the four partial tiles, 32 MP rows at a time, and the store
    const uint16_t* __restrict__ bias = (const uint16_t*)P.bias;
    float* red = reinterpret_cast<float*>(wv_lds);
    constexpr int PS = 32 * MP * LDN;                // floats of one wavefront's part
    auto bias4 = [&](int c) __attribute__((always_inline)) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (bias) {
            const u32x2 w = *reinterpret_cast<const u32x2*>(bias + c);
            v = f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
        }
        return v;
    };
    auto sum4 = [&](int r, int c) __attribute__((always_inline)) {
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[r * LDN + c]);
#pragma unroll
        for (int w = 1; w < kWaveWaves; ++w) s += *reinterpret_cast<const f32x4*>(&red[w * PS + r * LDN + c]);
        return s;
    };
#pragma unroll
    for (int p0 = 0; p0 < MT; p0 += MP) {
        __syncthreads();                             // every wavefront is done with the ring / with the previous rows
#pragma unroll
        for (int a = 0; a < MP; ++a)
            if (p0 + a < MT)
#pragma unroll
                for (int b = 0; b < NT; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<f32x4*>(&red[wave * PS + (32 * a + i32) * LDN + 32 * b + 8 * q + 4 * h]) =
                            f32x4{acc[p0 + a][b][4 * q], acc[p0 + a][b][4 * q + 1], acc[p0 + a][b][4 * q + 2], acc[p0 + a][b][4 * q + 3]};
        __syncthreads();
        const int mp = m0 + 32 * p0;
        const int rows = min(32 * MP, BM - 32 * p0);
        if (EPI == kEpiLayer && P.c_mode == kCTransposedV) {
            // C^T with tokens permuted inside 16-token blocks (vt_pos); P.ldc is the padded token count.  Rows beyond M of the last tile
            // are finite copies of row M - 1 and are written too, so that the padding never holds uninitialised bits.
            uint16_t* __restrict__ C = (uint16_t*)P.c;
            for (int e = tid; e < rows / 8 * BN; e += kWaveThreads) {
                const int q = e % (rows / 8), c = e / (rows / 8);
                const int r = 16 * (q >> 1) + 4 * (q & 1), nn = n0 + c;
                if (nn >= N || mp + 16 * (q >> 1) >= P.ldc) continue;
                const float bv = bias ? bf16_bits_to_f32(bias[nn]) : 0.f;
                float x[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int rr = r + (t & 3) + 8 * (t >> 2);
                    x[t] = red[rr * LDN + c];
#pragma unroll
                    for (int w = 1; w < kWaveWaves; ++w) x[t] += red[w * PS + rr * LDN + c];
                    x[t] += bv;
                }
                u32x4 w;
                w.x = pack_bf16x2(x[0], x[1]);
                w.y = pack_bf16x2(x[2], x[3]);
                w.z = pack_bf16x2(x[4], x[5]);
                w.w = pack_bf16x2(x[6], x[7]);
                *reinterpret_cast<u32x4*>(C + (int64_t)nn * P.ldc + mp + 8 * q) = w;
            }
        } else if (EPI == kEpiSwiGLU) {
            uint16_t* __restrict__ C = (uint16_t*)P.c;
            const int Fh = N >> 1;
            for (int e = tid; e < rows * (BN / 8); e += kWaveThreads) {
                const int r = e / (BN / 8), c = e % (BN / 8) * 4, nn = n0 / 2 + c;
                if (mp + r >= M || nn >= Fh) continue;
                const f32x4 gt = sum4(r, c) + bias4(nn), up = sum4(r, c + BN / 2) + bias4(Fh + nn);
                u32x2 w;
                w.x = pack_bf16x2(silu<true>(gt.x) * up.x, silu<true>(gt.y) * up.y);
                w.y = pack_bf16x2(silu<true>(gt.z) * up.z, silu<true>(gt.w) * up.w);
                *reinterpret_cast<u32x2*>(C + (int64_t)(mp + r) * P.ldc + nn) = w;
            }
        } else {
            for (int e = tid; e < rows * (BN / 4); e += kWaveThreads) {
                const int r = e / (BN / 4), c = e % (BN / 4) * 4, nn = n0 + c;
                if (mp + r >= M || nn >= N) continue;
                const int64_t at = (int64_t)(mp + r) * P.ldc + nn;
                f32x4 s = sum4(r, c) + bias4(nn);
                if (EPI == kEpiResidualF32 || (EPI == kEpiLayer && P.c_mode == kCF32)) {
                    if (EPI == kEpiResidualF32 && P.residual) s += *reinterpret_cast<const f32x4*>(P.residual + at);
                    *reinterpret_cast<f32x4*>((float*)P.c + at) = s;
                } else {
                    constexpr int ACT = EPI == kEpiGeluTanh ? kActGeluTanh : EPI == kEpiGeluErf ? kActGeluErf : kActNone;
                    u32x2 w;
                    w.x = pack_bf16x2(apply_act<true>(s.x, ACT), apply_act<true>(s.y, ACT));
                    w.y = pack_bf16x2(apply_act<true>(s.z, ACT), apply_act<true>(s.w, ACT));
                    *reinterpret_cast<u32x2*>((uint16_t*)P.c + at) = w;
                }
            }
        }
    }
}

// the tile shapes built, in the order of WaveConfig::index
struct WaveConfig {
    int bm, bn, lds, per_cu;          // tile, LDS bytes without codes, workgroups that fit a compute unit
};
constexpr int kWaveConfigs = 6;
extern const WaveConfig kWaveTable[kWaveConfigs];

int launch_gemm_wave(int cfg, int epi, bool gather, const GemmBatch& batch, int grid, int code_lds, hipStream_t s);
int launch_gemm_wave_mlp(int cfg, int epi, const GemmBatch& batch, int grid, hipStream_t s);

template <int MT, int NT, int ST, bool GATHER, bool ENC, int EPI>
static int launch_wave_form(const GemmBatch& batch, int grid, int code_lds, hipStream_t s) {
    auto* kernel = gemm_wave_kernel<MT, NT, ST, GATHER, ENC, EPI>;
    const int lds = (ENC && kWaveEncBytes > WaveShape<MT, NT, ST>::kBytes ? kWaveEncBytes : WaveShape<MT, NT, ST>::kBytes) + code_lds;
    static std::atomic<uint64_t> allowed{0};
    const int rc = allow_dynamic_lds(allowed, (const void*)kernel, 160 * 1024);
    if (rc) return rc;
    kernel<<<grid, kWaveThreads, lds, s>>>(batch);
    return launch_status();
}

// F: a generic lambda called with (MT, NT, ST) as integral constants
template <typename F>
static int with_wave_config(int cfg, F&& f) {
    auto call = [&](auto mt, auto nt, auto st) { return f(mt, nt, st); };
#define ASTRA_WAVE(I, MT, NT, ST) case I: return call(std::integral_constant<int, MT>{}, std::integral_constant<int, NT>{}, std::integral_constant<int, ST>{});
    switch (cfg) {
        ASTRA_WAVE(0, 1, 1, 2)
        ASTRA_WAVE(1, 2, 1, 2)
        ASTRA_WAVE(2, 2, 2, 2)
        ASTRA_WAVE(3, 2, 2, 1)
        ASTRA_WAVE(4, 4, 2, 1)
        ASTRA_WAVE(5, 4, 4, 1)
        default: return ASTRA_ERR_UNSUPPORTED;
    }
#undef ASTRA_WAVE
}

}  // namespace astra
