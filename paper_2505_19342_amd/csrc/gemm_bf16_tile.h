// The bf16 matrix-core GEMM tile kernel C[M,N] = A[M,K] . B[N,K]^T shared by the attention layer's projection launches
// (paper: the projections named under Eq. 1) and by the MLP of the block around the layer (Sec. 3.1).
#pragma once
#include "common.h"
#include "vq_encode_body.h"

#include <type_traits>

namespace astra {

struct GemmBatch {
    int32_t n;
    int32_t tile_begin[kMaxGemmProblems + 1];
    int32_t tiles_m[kMaxGemmProblems];     // tiles along M of each problem (tile index = tn * tiles_m + tm)
    GemmProblem p[kMaxGemmProblems];
    int32_t n_enc_wgs;                     // fused launch: workgroups beyond the GEMM tiles that run the VQ encode
    EncodeJob enc;
    int32_t n_split, k_split;              // split contraction (one problem): the grid is n_split copies of the tiles, copy s
                                           // contracts k in [s * k_split, (s + 1) * k_split) into slice s of an fp32 buffer
};

// The problem a tile belongs to, with the tile's number in it.  The arguments are a memory latency away, and the fields of a problem whose number has to be
// found first are another: with ONE (launches of one problem) nothing is found, and launches that may be of one (MAYBE_ONE) ask for the first problem's
// together with the number of problems.  12 GPT-2 blocks, 36 launches of one problem with an epilogue of the MLP: 603.5 us, 583.1 now.
enum { kOneProblem, kMaybeOneProblem, kManyProblems };
struct TileProblem {
    GemmProblem p;
    int tile, tiles_m;
};
template <int MODE>
__device__ __forceinline__ TileProblem find_problem(const GemmBatch& b, int tile) {
    if (MODE == kMaybeOneProblem)
        asm volatile("" ::"s"(b.n), "s"(b.tiles_m[0]), "s"(b.p[0].a), "s"(b.p[0].b), "s"(b.p[0].bias), "s"(b.p[0].c), "s"(b.p[0].M), "s"(b.p[0].N), "s"(b.p[0].K),
                     "s"(b.p[0].lda), "s"(b.p[0].ldc), "s"(b.p[0].ldb), "s"(b.p[0].c_mode));
    if (MODE == kOneProblem || (MODE == kMaybeOneProblem && b.n == 1)) return {b.p[0], tile, b.tiles_m[0]};
    int i = 0;
    while (i + 1 < b.n && tile >= b.tile_begin[i + 1]) ++i;
    return {b.p[i], tile - b.tile_begin[i], b.tiles_m[i]};
}

// ------------------------------------------------------------------------------------------------
// bf16, matrix cores.  A workgroup of WM x WN wavefronts owns a BM x BN output tile; each wavefront
// owns a (BM/WM) x (BN/WN) sub-tile made of 32x32x16 MFMA tiles.  The contraction runs in steps of 64
// through double-buffered LDS.  Operand tiles travel from memory straight into LDS (one wavefront instruction
// fills 64 consecutive 16-byte slots, nothing passes through registers), two tiles ahead of the matrix cores; there are two
// forms of the loop, by halves of a tile and by whole tiles.  LDS tiles are
// [rows][8 pieces of 8 bf16]; piece p of row r sits at p ^ ((r >> 1) & 7): rows are 128 bytes, the
// LDS has 64 four-byte banks, so the 16-byte fragment reads of 16 consecutive rows touch every bank once.
//
// Workgroup -> tile mapping: hardware hands consecutive workgroup ids to the 8 XCDs round-robin, each
// with its own L2.  Ids are remapped so that every XCD gets one contiguous range of tiles, walked with
// the M index fastest: the tiles an XCD runs at the same time share their weight (B) panel and draw
// their A panels from a few rows, so most operand traffic is served by that XCD's L2.
// ------------------------------------------------------------------------------------------------
constexpr int kBK = 64;
constexpr int kXcds = 8;
constexpr int kCus = 256;         // compute units of the device the launch shapes are chosen for

__device__ __forceinline__ int xcd_remap(int wg, int total) {
    const int q = total / kXcds, r = total % kXcds;
    const int xcd = wg % kXcds, slot = wg / kXcds;
    return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Activations of the position-wise MLP that follows the attention layer inside a block (paper Sec. 3.1), applied in
// the epilogue.  x * sigmoid(2u) is 0.5 x (1 + tanh u).  FAST uses the hardware exponential (results are rounded to bf16 afterwards);
// otherwise the library routines.  The quotient is a division, not the hardware reciprocal: that one returns zero where 1 / (1 + e^-v)
// is below the smallest normal number, while v times it (-5e-37 at v = -88) is well inside bf16's range.
template <bool FAST>
__device__ __forceinline__ float silu(float v) { return v / (1.f + (FAST ? __expf(-v) : expf(-v))); }
template <bool FAST>
__device__ __forceinline__ float apply_act(float v, int act) {
    if (act == kActGeluTanh) {
        const float u = 0.7978845608028654f * (v + 0.044715f * v * v * v);
        return FAST ? v / (1.f + __expf(-2.f * u)) : 0.5f * v * (1.f + tanhf(u));
    }
    if (act == kActGeluErf) return 0.5f * v * (1.f + erff(v * 0.7071067811865476f));
    return v;
}

// Fused launch of T GEMM tiles and E encode workgroups (E a multiple of 8): every XCD gets a contiguous range of
// tiles, as with xcd_remap, followed by E/8 encode workgroups, so both kinds of work are spread over all XCDs.
struct FusedId {
    bool enc;
    int idx;
};
__device__ __forceinline__ FusedId fused_id(int wg, int T, int E) {
    const int xcd = wg % kXcds, slot = wg / kXcds;
    const int tq = T / kXcds, tr = T % kXcds;
    const int t_x = tq + (xcd < tr ? 1 : 0);
    if (slot < t_x) return {false, xcd * tq + (xcd < tr ? xcd : tr) + slot};
    return {true, xcd * (E / kXcds) + slot - t_x};
}

// position of token offset o (0..15) inside a 16-token block of the transposed-V layout: the 8 tokens
// one half-wave holds of an MFMA accumulator column ({4h..4h+3} and {8+4h..8+4h+3}) become contiguous,
// which is also the order the attention kernel's P^T operand keeps its 16 keys in.
__device__ __forceinline__ int vt_pos(int o) { return 8 * ((o >> 2) & 1) + (o & 3) + 4 * (o >> 3); }

int launch_gemm_f32(int tile, const GemmBatch& batch, hipStream_t s);
int launch_gemm_mlp(int epi, bool big, const GemmBatch& batch, int grid, hipStream_t s);
int launch_split_reduce(const float* part, int n_split, const GemmProblem& p, hipStream_t s);
int gemm_split_factor(int dtype, int64_t M, int64_t N, int64_t K);

// EPI selects the epilogue at compile time.  kEpiLayer is the attention layer's: the store follows the problem's c_mode
// (bf16, fp32, transposed V).  The others belong to the block around the layer (one plain-A problem per launch) and each
// carries exactly one form, so that the tail of a launch that runs as a single round of workgroups stays short:
//   kEpiResidualF32  fp32 store of A.B^T + bias, accumulation started from `residual` when it is set
//   kEpiSplit        the contraction slice batch.k_split of copy blockIdx / tiles, raw fp32 partial sums
//   kEpiGeluTanh / kEpiGeluErf   bf16 store of gelu(A.B^T + bias)
//   kEpiSwiGLU       bf16 store of silu(A.gate^T + b_g) * (A.up^T + b_u)
enum { kEpiLayer = 0, kEpiResidualF32 = 1, kEpiSplit = 2, kEpiGeluTanh = 3, kEpiGeluErf = 4, kEpiSwiGLU = 5 };

template <int B, int W>
constexpr bool halves() { return B % (64 * W) == 0; }
// row of the tile that LDS row r holds, for W wavefronts along a side of B
template <int B, int W, bool QUAD>
__device__ __forceinline__ int tile_row(int r) {
    constexpr int P = B / 2 / W;                               // rows of half a wavefront tile
    return QUAD ? (r % (B / 2)) / P * 2 * P + r / (B / 2) * P + r % P : r;
}

template <int BM, int BN, int WM, int WN, bool CODE16, bool ENC = false, int EPI = kEpiLayer>
__global__ __launch_bounds__(64 * WM * WN) void gemm_nt_bf16_kernel(const GemmBatch batch) {
    constexpr int THREADS = 64 * WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;        // MFMA tiles per wavefront
    constexpr int RPP = THREADS / 8;                           // rows staged per pass
    constexpr int PA = BM / RPP, PB = BN / RPP;                // staging passes per thread
    static_assert(RPP % 16 == 0, "direct transfers: the row swizzle has to be periodic in the pass stride");
    // Every wavefront's rows and columns come in two halves of whole 32s: the loop in quadrants (below).  In LDS the first halves of all wavefronts then
    // precede the second ones.
    constexpr bool QUAD = halves<BM, WM>() && halves<BN, WN>();
    constexpr bool GATHER = EPI == kEpiLayer;                  // only the layer's launches have problems with codes
    constexpr int PAH = QUAD ? PA / 2 : 1;                     // staging passes of half of the A rows
    __shared__ u32x4 lds_a[2][BM * kBK / 8];
    __shared__ u32x4 lds_b[2][BN * kBK / 8];
    __shared__ uint32_t lds_code[QUAD && GATHER ? 4 * PAH * THREADS : 1];

    int vt;
    if (ENC) {
        // The grid is the GEMM tiles plus batch.n_enc_wgs workgroups that encode the local rows (nothing in the
        // projections depends on the codes or the other way round): they fill compute units the tiles leave idle.
        // The encode reuses the operand buffers: its ring of codebook tiles is exactly the one of 256 rows, the norms sit in the other.
        constexpr size_t kRing = sizeof(u32x4) * kEncBufs * kEncCbSlots, kNorms = sizeof(f32x4) * kEncBufs * kEncCnSlots;
        constexpr bool RING_IN_A = sizeof(lds_a) == kRing;
        static_assert(!ENC || (RING_IN_A && sizeof(lds_b) >= kNorms) || (sizeof(lds_b) == kRing && sizeof(lds_a) >= kNorms),
                      "encode ring must be one of the operand buffers");
        const FusedId id = fused_id(blockIdx.x, gridDim.x - batch.n_enc_wgs, batch.n_enc_wgs);
        if (id.enc) {
            u32x4* cb = RING_IN_A ? &lds_a[0][0] : &lds_b[0][0];
            f32x4* cn = reinterpret_cast<f32x4*>(RING_IN_A ? &lds_b[0][0] : &lds_a[0][0]);
            const EncodeJob& job = batch.enc;
            if (vq_encode_fast_needs_zero(job.dg)) {
                vq_encode_fast_zero_lds<THREADS>(cb);
                __syncthreads();                           // zero fill done before any transfer lands
            }
            const int n_items = job.G * job.n_tb;
            const int chunk = (n_items + batch.n_enc_wgs - 1) / batch.n_enc_wgs;     // consecutive items share the group
            const int hi = min((id.idx + 1) * chunk, n_items);
            vq_encode_fast_run<THREADS, true>(job, id.idx * chunk, hi, cb, cn);
            return;
        }
        vt = id.idx;
    } else {
        vt = xcd_remap(blockIdx.x, gridDim.x);
    }
    int split = 0;
    if (EPI == kEpiSplit) {
        const int tiles = batch.tile_begin[batch.n];
        split = vt / tiles;
        vt -= split * tiles;
    }
    const TileProblem tp = find_problem<EPI != kEpiLayer ? kOneProblem : ENC ? kManyProblems : kMaybeOneProblem>(batch, vt);
    const GemmProblem& P = tp.p;
    const int tile = tp.tile, tiles_m = tp.tiles_m;
    const int tm = tile % tiles_m, tn = tile / tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;
    const int M = P.M, N = P.N, K = P.K;

    const int tid = (int)threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int i32 = lane & 31, h = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int r0 = tid >> 3;                    // staging: 16-byte piece kc of rows r0 + RPP * it
    // With direct global -> LDS transfers a lane's LDS slot is fixed by its lane number (slot tid & 7 of its row), so the
    // swizzle moves to the global side: the lane fetches the piece that belongs into its slot.
    const int kc = (tid & 7) ^ swz(r0);

    // One straight-line loader serves plain and gathered A rows.  For gathered rows the piece at
    // contraction index k lies in group g = k / dg at offset j = k - g*dg of codeword codes[row, g];
    // for plain rows the code load is a harmless read of the first bytes of A and the gathered offset is
    // discarded by a select.  k / dg is a multiply-high by ceil(2^32 / dg), exact for k, dg < 2^16.
    // Addresses are a wave-uniform base (scalar registers, advanced once per tile) plus a 32-bit byte
    // offset per thread, which keeps the per-row state to one register.
    const bool gather = P.codes != nullptr;
    const int dg = gather ? P.dg : 1, Kc = gather ? P.Kc : 1, G = gather ? P.G : 0;
    const uint32_t magic = gather ? (uint32_t)(0x100000000ull / (uint32_t)dg) + 1u : 0u;
    const char* __restrict__ a_base = (const char*)(gather ? P.codebook : P.a);   // plain A advances 128 bytes per tile
    const int a_step = gather ? 0 : kBK * 2;
    const uint32_t gmask = gather ? 0xffffffffu : 0u;                           // keeps the gathered offset, or zeroes it
    const char* __restrict__ b_base = (const char*)P.b;
    if (EPI == kEpiSplit) {                    // plain A only: both operands start at this copy's slice of the contraction
        a_base += (int64_t)split * batch.k_split * 2;
        b_base += (int64_t)split * batch.k_split * 2;
    }
    const char* __restrict__ c_base = (const char*)(gather ? P.codes : P.a);
    uint32_t aoff[PA], coff[PA], boff[PB];
#pragma unroll
    for (int it = 0; it < PA; ++it) {
        int ra = m0 + tile_row<BM, WM, QUAD>(r0 + RPP * it);
        ra = ra < M ? ra : M - 1;
        aoff[it] = gather ? 0u : ((uint32_t)ra * (uint32_t)P.lda + kc * 8) * 2u;
        coff[it] = (uint32_t)ra * (uint32_t)G * (CODE16 ? 2u : 1u);
    }
#pragma unroll
    for (int it = 0; it < PB; ++it) {
        int rb = n0 + tile_row<BN, WN, QUAD>(r0 + RPP * it);
        rb = rb < N ? rb : N - 1;
        if (EPI == kEpiSwiGLU) {
            // tile row r of B -> weight row such that, in every wavefront, MFMA column tiles b < TN/2 hold gate rows and
            // tiles b + TN/2 the up rows of the same BN/WN/2 output columns: both factors of an output meet in one lane
            const int rr = tile_row<BN, WN, QUAD>(r0 + RPP * it), Fh = N >> 1;
            const int wn_r = rr / (32 * TN), b_r = (rr % (32 * TN)) / 32, i_r = rr % 32;
            int col = n0 / 2 + wn_r * (16 * TN) + (b_r % (TN / 2)) * 32 + i_r;
            col = col < Fh ? col : Fh - 1;
            rb = (b_r >= TN / 2 ? Fh : 0) + col;
        }
        boff[it] = ((uint32_t)rb * (uint32_t)(P.ldb ? P.ldb : K) + kc * 8) * 2u;
    }
    int k_code = kc * 8; // contraction index of this thread's piece in the tile whose codes are fetched next
    int k_use = kc * 8;  // ... in the tile whose operand pieces are fetched next
    int code[PA];

    auto load_codes = [&]() {
        const uint32_t g_ = __umulhi((uint32_t)k_code, magic) * (CODE16 ? 2u : 1u);
#pragma unroll
        for (int it = 0; it < PA; ++it) {
            if (CODE16) code[it] = *reinterpret_cast<const uint16_t*>(c_base + (coff[it] + g_));
            else code[it] = *reinterpret_cast<const uint8_t*>(c_base + (coff[it] + g_));
        }
        k_code += kBK;
    };
    // direct transfer of the tile at k_use into LDS buffer buf_: the lanes of a wavefront fill 64 consecutive slots
    // (8 rows of 8 pieces), nothing passes through registers; pass it_ of the A rows, then of the B rows
    const uint32_t wave_rows = (uint32_t)__builtin_amdgcn_readfirstlane(8 * (tid >> 6));
    auto dma_piece = [&](int buf_, int j_it) {
        if (j_it < PA) {
            const int it = j_it;
            const uint32_t g_ = __umulhi((uint32_t)k_use, magic);
            const uint32_t j_ = (uint32_t)k_use - g_ * (uint32_t)dg;
            int code_here = code[it];
            asm volatile("" : "+v"(code_here));      // the code is first touched here: an earlier use would wait for the transfers issued before its load
            const uint32_t c_ = (uint32_t)(code_here < Kc ? code_here : Kc - 1);
            const uint32_t goff_ = ((g_ * (uint32_t)Kc + c_) * (uint32_t)dg + j_) * 2u;
            dma_global_to_lds_16(a_base, (goff_ & gmask) + aoff[it], lds_byte_addr(&lds_a[buf_][(wave_rows + RPP * it) * 8]));
        } else {
            const int it = j_it - PA;
            dma_global_to_lds_16(b_base, boff[it], lds_byte_addr(&lds_b[buf_][(wave_rows + RPP * it) * 8]));
        }
    };
    auto dma_advance = [&]() {
        a_base += a_step;
        b_base += kBK * 2;
        k_use += kBK;
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    if (EPI == kEpiResidualF32 && P.residual != nullptr) {
        // The residual is where the accumulation starts: its loads are issued here, all at once, and land while the first
        // operand tiles are fetched.  (Added in the epilogue, every load would be a round trip to memory in front of a store.)
        // Rows and columns beyond the problem are clamped: those accumulators are never stored.
        const char* __restrict__ R = (const char*)P.residual;
        const uint32_t ldc = (uint32_t)P.ldc;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int n = min(n0 + wn * (BN / WN) + b * 32 + i32, N - 1);
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = min(m0 + wm * (BM / WM) + a * 32 + acc_row(v, h), M - 1);
                    acc[a][b][v] = *reinterpret_cast<const float*>(R + ((uint32_t)m * ldc + (uint32_t)n) * 4u);
                }
        }
    }

    const int n_kt = (EPI == kEpiSplit ? batch.k_split : K) / kBK;
    if constexpr (QUAD) {
        // ---- main loop in quadrants.  A wavefront's rows are two halves, A0 and A1, its columns likewise, B0 and B1.  A tile of 64 along the
        // contraction is four products A0 B0, A0 B1, A1 B1, A1 B0, each over the whole 64, so that every fragment is read from LDS once and takes the
        // registers of one that has just been used for the last time: A1 those of A0, B0 of the next tile those of B1, and so on (64 registers of
        // fragments next to 128 of accumulators on 256 x 256).  Half a tile's rows in LDS are therefore free long before the tile is done.  Two barriers
        // per tile, in the middle of A0 B0 and of A1 B1, cut the loop into half steps of 8 NQ MFMAs; in each of them the fragments of one half (A1, B1 of
        // this tile; A0, B0 of the next) are read, and the same half of the tile after the next is sent to the place of the one read a half step ago.
        // A transfer has two to three half steps to land, one to one and a half tiles' time, and they are spread evenly over the loop.  The loop below
        // sends whole tiles in the last quarter of the tile before and gives them three quarters of one to land; that, not the matrix cores or the LDS, was
        // what held it up.  With it, back to back: 256 x 256 tiles, 4096 x 4096 fp32 outputs, K = 256 / 1024 / 4096: 21.8 / 40.3 / 116 us, now
        // 21.2 / 38.5 / 110; 192 of them at K = 4096 99.8, now 90.9; gate and up rows of 1024 x 14336, K = 4096: 219, now 190.  128 x 256 tiles,
        // 1024 x 5120, K = 1024 / 4096: 22.2 / 59.7, now 20.1 / 47.9.  Four wavefronts of 128 x 128 read a third less from LDS and take the same time;
        // transfers behind a branch each (one copy of the loop instead of a tail of its own) take 3 % longer.  128 x 128 tiles have no such
        // halves on eight wavefronts, and on four they are 1 - 2 us slower than the loop below over short contractions and level over long ones.
        // The codes of gathered rows come by transfers too, four half steps ahead of the ones that use them: every wavefront sends those of its own rows
        // to its own part of LDS.  The compiler sees none of it, so nothing but the waits written here holds up the transfers.
        constexpr int TMH = TM / 2, TNH = TN / 2, PBH = PB / 2, NQ = TMH * TNH;
        constexpr int DPH = PAH + PBH + (GATHER ? PAH : 0);              // transfers of a half step
        constexpr int NM = 8 * NQ;                                       // MFMAs of a half step
        static_assert(!QUAD || NQ % TNH == 0, "a B fragment is replaced no earlier than after its last use");
        bf16x8 fa[4][TMH], fb[2][4][TNH];
        const int at_a = (wm * (BM / 2 / WM) + i32) * 8, at_b = (wn * (BN / 2 / WN) + i32) * 8;
        auto read_a = [&](int buf, int half, int ks, int a) {
            fa[ks][a] = __builtin_bit_cast(bf16x8, lds_a[buf][at_a + ((2 * ks + h) ^ swz(i32)) + (half * (BM / 2) + a * 32) * 8]);
        };
        auto read_b = [&](int buf, int half, int slot, int ks, int b) {
            fb[slot][ks][b] = __builtin_bit_cast(bf16x8, lds_b[buf][at_b + ((2 * ks + h) ^ swz(i32)) + (half * (BN / 2) + b * 32) * 8]);
        };
        int kt_code = 2;                                  // tile whose codes are sent next
        uint32_t code_q[PAH];
        auto send_b = [&](int buf, int half, int it) {
            dma_global_to_lds_16(b_base, boff[half * PBH + it], lds_byte_addr(&lds_b[buf][(wave_rows + RPP * (half * PBH + it)) * 8]));
        };
        auto send_a = [&](int buf, int half, int it, uint32_t c_raw) {
            const uint32_t dst = lds_byte_addr(&lds_a[buf][(wave_rows + RPP * (half * PAH + it)) * 8]);
            if (GATHER) {
                const uint32_t g_ = __umulhi((uint32_t)k_use, magic);
                const uint32_t j_ = (uint32_t)k_use - g_ * (uint32_t)dg;
                const uint32_t c_ = min(c_raw, (uint32_t)Kc - 1u);
                dma_global_to_lds_16(a_base, ((((g_ * (uint32_t)Kc + c_) * (uint32_t)dg + j_) * 2u) & gmask) + aoff[half * PAH + it], dst);
            } else {
                dma_global_to_lds_16(a_base, aoff[half * PAH + it], dst);
            }
        };
        // codes of half `half` of tile kt_code (or of the last tile: sent for nothing) into ring slot `slot`
        auto send_code = [&](int slot, int half, int it) {
            const uint32_t g_ = __umulhi((uint32_t)(kc * 8 + kBK * min(kt_code, n_kt - 1)), magic) * (CODE16 ? 2u : 1u);
            dma_code_to_lds<CODE16>(c_base, coff[half * PAH + it] + g_, lds_byte_addr(&lds_code[(slot * PAH + it) * THREADS]) + wave_rows * 32u);
        };
        // Half step TAG of four (tile kt even: 0, 1, odd: 2, 3).  nx: tile kt + 1 exists; FULL or fetch: tile kt + 2 exists
        auto half_step = [&](auto tag, auto full_tag, bool nx_, bool fetch_) {
            constexpr int TAG = decltype(tag)::value, BUF = TAG >> 1, HALF = TAG & 1;
            constexpr bool FULL = decltype(full_tag)::value;
            const bool nx = FULL || nx_, fetch = FULL || fetch_;
            constexpr int S0 = BUF, S1 = BUF ^ 1;                        // where B0 and B1 of tile kt are
            if (GATHER && fetch) {
#pragma unroll
                for (int it = 0; it < PAH; ++it) code_q[it] = lds_code[(TAG * PAH + it) * THREADS + tid];
            }
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int st = m / NQ, a = m % NQ / TNH, b = m % TNH;    // step of 16: two of the first product, four, two of the third
                const int ks = st < 2 ? st + 2 : st < 6 ? st - 2 : st - 6;
                const int qa = st < 6 ? HALF : HALF ^ 1, qb = st < 2 ? HALF : st < 6 ? HALF ^ 1 : HALF ^ 1;
                // B slot of the product: B0, B1, B1; in the second half step B1, B0, and B0 of the next tile (read into the place of B1)
                const int slot = HALF == 0 ? (st < 2 ? S0 : S1) : (st < 2 ? S1 : st < 6 ? S0 : S1);
                if (HALF == 0 || st < 6 || nx) acc[qa * TMH + a][qb * TNH + b] = mfma_32x32x16(fa[ks][a], fb[slot][ks][b], acc[qa * TMH + a][qb * TNH + b]);
                // fragments into the registers of those used for the last time: B steps 0 and 1 during step 0, 2 and 3 after it
                if (st < 2) {
#pragma unroll
                    for (int j = m * 2 * TNH / NQ; j < (m + 1) * 2 * TNH / NQ; ++j) {
                        if (HALF == 0) read_b(BUF, 1, S1, j / TNH, j % TNH);
                        else if (nx) read_b(BUF ^ 1, 0, S1, j / TNH, j % TNH);
                    }
                } else if (st < 6 && b == TNH - 1) {
                    if (HALF == 0) read_a(BUF, 1, ks, a);
                    else if (nx) read_a(BUF ^ 1, 0, ks, a);
                }
                if (fetch) {
#pragma unroll
                    for (int j = m * DPH / NM; j < (m + 1) * DPH / NM; ++j) {
                        if (j < PBH) send_b(BUF, HALF, j);
                        else if (j < PBH + PAH) send_a(BUF, HALF, j - PBH, GATHER ? code_q[j - PBH] : 0u);
                        else send_code(TAG, HALF, j - PBH - PAH);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (HALF == 1 && fetch) {
                dma_advance();
                ++kt_code;
            }
            if (HALF == 0 || nx) {
                // the half that is read from here on has landed: at most the transfers of the last two half steps are outstanding
                if (FULL || fetch) wait_vmem<2 * DPH>();
                else wait_vmem_all();
                __syncthreads();
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // prologue: tiles 0 and 1, and the codes of tiles 2 and 3
        const bool two = n_kt > 1;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int it = 0; it < PBH; ++it) send_b(0, j, it);
        uint32_t code_0[PA], code_1[PA];
        if (GATHER) {
            const uint32_t g0_ = __umulhi((uint32_t)(kc * 8), magic), g1_ = __umulhi((uint32_t)(kc * 8 + (two ? kBK : 0)), magic);
#pragma unroll
            for (int it = 0; it < PA; ++it) {
                if (CODE16) {
                    code_0[it] = *reinterpret_cast<const uint16_t*>(c_base + (coff[it] + g0_ * 2u));
                    code_1[it] = *reinterpret_cast<const uint16_t*>(c_base + (coff[it] + g1_ * 2u));
                } else {
                    code_0[it] = *reinterpret_cast<const uint8_t*>(c_base + (coff[it] + g0_));
                    code_1[it] = *reinterpret_cast<const uint8_t*>(c_base + (coff[it] + g1_));
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int it = 0; it < PAH; ++it) send_a(0, j, it, GATHER ? code_0[j * PAH + it] : 0u);
            if (GATHER && two)
#pragma unroll
                for (int it = 0; it < PAH; ++it) send_code(j, j, it);
        }
        dma_advance();
        ++kt_code;
        if (two) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int it = 0; it < PBH; ++it) send_b(1, j, it);
#pragma unroll
                for (int it = 0; it < PAH; ++it) send_a(1, j, it, GATHER ? code_1[j * PAH + it] : 0u);
                if (GATHER)
#pragma unroll
                    for (int it = 0; it < PAH; ++it) send_code(2 + j, j, it);
            }
            dma_advance();
            ++kt_code;
            wait_vmem<2 * DPH + (GATHER ? 3 : 1) * PAH>();          // A0 and all of B of tile 0
        } else {
            wait_vmem_all();
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
            for (int b = 0; b < TNH; ++b) read_b(0, 0, 0, ks, b);
#pragma unroll
            for (int a = 0; a < TMH; ++a) read_a(0, 0, ks, a);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int a = 0; a < TMH; ++a)
#pragma unroll
                for (int b = 0; b < TNH; ++b) acc[a][b] = mfma_32x32x16(fa[ks][a], fb[0][ks][b], acc[a][b]);
        if (two) wait_vmem<2 * DPH>();
        else wait_vmem_all();
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        using T = std::true_type;
        using F = std::false_type;
        int kt = 0;
        for (; kt + 3 < n_kt; kt += 2) {
            half_step(std::integral_constant<int, 0>{}, T{}, true, true);
            half_step(std::integral_constant<int, 1>{}, T{}, true, true);
            half_step(std::integral_constant<int, 2>{}, T{}, true, true);
            half_step(std::integral_constant<int, 3>{}, T{}, true, true);
        }
        // the last one to three tiles; only the first of three fetches
        auto tail = [&](auto even, auto odd) {
            half_step(even, F{}, kt + 1 < n_kt, kt + 2 < n_kt);
            half_step(odd, F{}, kt + 1 < n_kt, kt + 2 < n_kt);
            ++kt;
        };
        tail(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        if (kt < n_kt) tail(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
        if (kt < n_kt) tail(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
    } else {
        // ---- main loop by whole tiles.
        // fragment rows
        int arow[TM], brow[TN];
    #pragma unroll
        for (int a = 0; a < TM; ++a) arow[a] = wm * (BM / WM) + a * 32 + i32;
    #pragma unroll
        for (int b = 0; b < TN; ++b) brow[b] = wn * (BN / WN) + b * 32 + i32;

        // One tile of 64 along the contraction is four MFMA steps of 16.  Per step a wavefront
        // issues TM*TN MFMAs on fragments it requested from LDS one step earlier (two fragment slots), and between those
        // MFMAs, in program order, the "side jobs" of the step: the TM+TN fragment reads of the next step and, in step 3,
        // the transfers of tile kt+2.  LDS and global latencies are covered by the MFMAs issued meanwhile.  The workgroup
        // barrier follows step 2, after which step 3 may read the first fragments of tile kt+1 from the other buffer, and
        // the buffer of tile kt (all of whose fragments were requested before the barrier) is free for the transfers.
        bf16x8 fa[2][TM], fb[2][TN];
        auto read_frag = [&](int buf_, int ks, int slot, int j) {
            if (j < TM) fa[slot][j] = __builtin_bit_cast(bf16x8, lds_a[buf_][arow[j] * 8 + ((2 * ks + h) ^ swz(arow[j]))]);
            else fb[slot][j - TM] = __builtin_bit_cast(bf16x8, lds_b[buf_][brow[j - TM] * 8 + ((2 * ks + h) ^ swz(brow[j - TM]))]);
        };
        constexpr int NR = TM + TN, NM = TM * TN;
        {
            // Tiles go from memory straight into LDS.  Buffer kt & 1 is free once every wavefront has passed the barrier of
            // iteration kt (all reads of tile kt were requested and awaited before it): tile kt + 2 is sent there during step 3
            // of iteration kt and has until the wait in front of the barrier of iteration kt + 1 to land.
            // buf_tag: std::integral_constant<int, kt & 1> makes the buffer static (LDS addresses become immediates; steady
            // state, where tiles kt + 1, kt + 2 and the codes of kt + 3 all exist), std::integral_constant<int, -1> reads it from kt
            // (the last few tiles, with the run-time guards)
            auto tile_steps_dma = [&](int kt, auto buf_tag) {
                constexpr bool FULL = decltype(buf_tag)::value >= 0;
                const int buf = FULL ? decltype(buf_tag)::value : (kt & 1);
                const bool nx = FULL || kt + 1 < n_kt, nx2 = FULL || kt + 2 < n_kt;
    #pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int cur = ks & 1, nxt = cur ^ 1;
                    const int nd = ks == 3 ? PA + PB : 0;
                    const int nj = NR + nd;
                    const bool rd = ks < 3 || nx;
    #pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        const int a = m / TN, b = m % TN;
                        acc[a][b] = mfma_32x32x16(fa[cur][a], fb[cur][b], acc[a][b]);
    #pragma unroll
                        for (int j = m * nj / NM; j < (m + 1) * nj / NM; ++j) {
                            if (j < NR) {
                                if (rd) read_frag(ks < 3 ? buf : buf ^ 1, (ks + 1) & 3, nxt, j);
                            } else if (nx2) {
                                dma_piece(buf, j - NR);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (ks == 2) {
                        wait_vmem_all();          // this wavefront's transfers of tile kt + 1 have landed
                        __syncthreads();
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (nx2) dma_advance();
                if (FULL || kt + 3 < n_kt) load_codes();
            };
            load_codes();                 // codes of tile 0
    #pragma unroll
            for (int j = 0; j < PA + PB; ++j) dma_piece(0, j);
            dma_advance();
            if (n_kt > 1) {
                load_codes();             // codes of tile 1
    #pragma unroll
                for (int j = 0; j < PA + PB; ++j) dma_piece(1, j);
                dma_advance();
            }
            if (n_kt > 2) load_codes();   // codes of tile 2
            wait_vmem_all();
            __syncthreads();
    #pragma unroll
            for (int j = 0; j < NR; ++j) read_frag(0, 0, 0, j);
            int kt = 0;
            for (; kt + 4 < n_kt; kt += 2) {
                tile_steps_dma(kt, std::integral_constant<int, 0>{});
                tile_steps_dma(kt + 1, std::integral_constant<int, 1>{});
            }
            for (; kt < n_kt; ++kt) tile_steps_dma(kt, std::integral_constant<int, -1>{});
        }
    }

    // epilogue.  acc[a][b][v] is C[m, n] with m = wave row base + 32a + acc_row(v, h), n = wave column base + 32b + lane % 32.
    const uint16_t* __restrict__ bias = (const uint16_t*)P.bias;
    if constexpr (EPI == kEpiSplit) {
        // partial sums: slice `split` of the fp32 buffer, [M, N] dense; bias and residual are added by the reduction
        float* __restrict__ C = (float*)P.c + (int64_t)split * M * N;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int n = n0 + wn * (BN / WN) + b * 32 + i32;
            if (n >= N) continue;
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + wm * (BM / WM) + a * 32 + acc_row(v, h);
                    if (m < M) C[(int64_t)m * N + n] = acc[a][b][v];
                }
        }
    } else if constexpr (EPI == kEpiSwiGLU) {
        static_assert(EPI != kEpiSwiGLU || TN % 2 == 0, "gate and up tiles pair up inside a wavefront");
        const int Fh = N >> 1;
        uint16_t* __restrict__ C = (uint16_t*)P.c;
#pragma unroll
        for (int b = 0; b < TN / 2; ++b) {
            const int col = n0 / 2 + wn * (16 * TN) + b * 32 + i32;
            if (col >= Fh) continue;
            const float bg = bias ? bf16_bits_to_f32(bias[col]) : 0.f, bu = bias ? bf16_bits_to_f32(bias[Fh + col]) : 0.f;
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + wm * (BM / WM) + a * 32 + acc_row(v, h);
                    if (m < M) C[(int64_t)m * P.ldc + col] = f32_to_bf16_bits(silu<true>(acc[a][b][v] + bg) * (acc[a][b + TN / 2][v] + bu));
                }
        }
    } else {
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int n = n0 + wn * (BN / WN) + b * 32 + i32;
            if (n >= N) continue;
            const float bv = bias ? bf16_bits_to_f32(bias[n]) : 0.f;
            if (EPI == kEpiLayer && P.c_mode == kCTransposedV) {
                // C^T with tokens permuted inside 16-token blocks; P.ldc is the padded token count.  Rows
                // m >= M of the last tile are finite copies of row M-1 (clamped loads) and are written too,
                // so the padding never holds uninitialised bits.
                uint16_t* __restrict__ C = (uint16_t*)P.c + (int64_t)n * P.ldc;
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int blk = 0; blk < 2; ++blk) {
                        const int mb = m0 + wm * (BM / WM) + a * 32 + 16 * blk;
                        if (mb < P.ldc) {
                            u32x4 w;
                            w.x = pack_bf16x2(acc[a][b][8 * blk + 0] + bv, acc[a][b][8 * blk + 1] + bv);
                            w.y = pack_bf16x2(acc[a][b][8 * blk + 2] + bv, acc[a][b][8 * blk + 3] + bv);
                            w.z = pack_bf16x2(acc[a][b][8 * blk + 4] + bv, acc[a][b][8 * blk + 5] + bv);
                            w.w = pack_bf16x2(acc[a][b][8 * blk + 6] + bv, acc[a][b][8 * blk + 7] + bv);
                            *reinterpret_cast<u32x4*>(C + mb + 8 * h) = w;
                        }
                    }
            } else if (EPI == kEpiResidualF32 || (EPI == kEpiLayer && P.c_mode == kCF32)) {
                float* C = (float*)P.c;                       // may be the residual itself (already inside acc): no restrict
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = m0 + wm * (BM / WM) + a * 32 + acc_row(v, h);
                        if (m < M) C[(int64_t)m * P.ldc + n] = acc[a][b][v] + bv;
                    }
            } else {
                constexpr int ACT = EPI == kEpiGeluTanh ? kActGeluTanh : EPI == kEpiGeluErf ? kActGeluErf : kActNone;
                uint16_t* __restrict__ C = (uint16_t*)P.c;
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int m = m0 + wm * (BM / WM) + a * 32 + acc_row(v, h);
                        if (m < M) C[(int64_t)m * P.ldc + n] = f32_to_bf16_bits(apply_act<true>(acc[a][b][v] + bv, ACT));
                    }
            }
        }
    }
}

}  // namespace astra
