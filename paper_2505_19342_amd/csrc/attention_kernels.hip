// Mixed-precision attention of one device (paper Sec. 3.2, Eq. 1): local queries attend to the
// full-precision local keys/values and to keys/values projected from the tokens rebuilt from codes.
// The two key/value sources are never concatenated in memory: the kernels walk the visible
// non-local rows first and the local rows after them (softmax does not depend on key order).
#include "attention_encode.h"
#include "vq_encode_f32_body.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace astra {

// ------------------------------------------------------------------------------------------------
// bf16, matrix cores, flash style (online softmax, nothing of size T_q x T_k is ever stored).
//
// Scores are computed transposed, S^T = K_tile . Q^T (keys on the M side, queries on the N side of the
// 32x32x16 MFMA), so the 16 accumulator values of a lane all belong to ONE query: the running max / sum
// of the online softmax are per-lane scalars, and the probabilities, rounded to bf16 in place, already
// have the register layout of the B operand of O^T += V^T . P^T.
//
// A workgroup of 8 wavefronts owns 128 query rows of one head.  Wavefront w owns the 32 rows of query
// group w & 3 and walks only the key/value tiles of parity w >> 2; the two wavefronts that share a query
// group merge their (max, sum, O) triples through LDS at the end.  The two wavefronts of a SIMD have
// different parities and are kept in opposite phases (see the schedule below): one runs its softmax on
// the vector ALU while the other occupies the matrix core.  (NPAR = 4, for short sequences with 64-wide heads: 64 query
// rows per workgroup, two query groups, and the tiles dealt to four wavefronts per group: twice the workgroups, half the
// iterations; wavefronts 0..3 still run one phase ahead of wavefronts 4..7.)  A wavefront's whole state (O^T 64, S^T 32,
// Q 32, P 16 registers) stays in ordinary vector registers.  Tiles of 64 keys are double-buffered in LDS
// with XOR-swizzled 16-byte pieces and arrive by direct global->LDS transfers, issued one iteration ahead
// by the four wavefronts that will read them.
//
// V is consumed as V^T.  With VT = true it arrives already transposed ([H_kv*dh, T_pad], tokens permuted
// inside blocks of 16 as the projection kernel writes them) and fragments are plain 16-byte LDS reads;
// with VT = false it arrives row-major [T, H_kv, dh] and is transposed by the 64-bit transposing LDS read.
//
// Workgroup order: ids are remapped so that each XCD (own L2) gets a contiguous run of heads, i.e. the
// query heads of as few KV heads as possible, and inside a head the later (heavier under causal
// masking) query blocks come first.
// ------------------------------------------------------------------------------------------------
constexpr int kAttQ = 128;       // query rows per workgroup (64 with four tile parities)
constexpr int kAttKV = 64;       // key/value rows per tile
constexpr int kAttThreads = 512;
constexpr int kXcdsA = 8;
constexpr int kAttCus = 256;     // compute units of the device the launch shapes are chosen for
constexpr float kLazy = 8.f;     // base-2 units
constexpr int kPartFloats = kAttQ * 128 + 2 * kAttQ;     // partial result of a part of a walk: O of 128 rows, their maxima, their sums
constexpr int kMaxParts = 8;

__device__ __forceinline__ int xcd_remap_attn(int wg, int total) {
    const int q = total / kXcdsA, r = total % kXcdsA;
    const int xcd = wg % kXcdsA, slot = wg / kXcdsA;
    return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

template <int DH>
__device__ __forceinline__ int swz_k(int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); }
// row-major V tile read by the transposing load: 4 consecutive rows x 64 bytes must hit distinct banks
template <int DH>
__device__ __forceinline__ int swz_v(int r) { return DH == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); }
// transposed V tile: rows of 64 keys = 128 bytes, same rule as the GEMM operand tiles
__device__ __forceinline__ int swz_vt(int r) { return (r >> 1) & 7; }

// LOST: the caller passed a validity bit per non-local token (an instantiation of its own, so that the code for it does
// not disturb the register allocation and schedule of the kernel that runs without)
// ENC: VQ encodes ride in the launch (AttnEncode)
// CUT: the blocks of all heads of an XCD side by side, walks possibly cut between workgroups (AttnParams::n_whole, n_cut); a part leaves its unnormalised result, on the
// scale of its own maxima, in AttnParams::part (error against 64 bits, 300 + 2565 / 512 + 3584 / 1280 + 3840 rows: 1.81e-3, 1.87e-3, 1.96e-3 of the norm cut,
// 1.82e-3, 1.87e-3, 1.96e-3 whole).  Few query blocks leave
// units idle, and a few more than a round of them leave most units idle for a second whole walk.  A part costs 6 us before its first tile and after its
// last, and its 64 KiB.  Layers 4096 wide, every walk whole / cut (us): 20 + 4096 rows 132.1 / 123.5, 300 + 2565 157.8 / 151.1, 512 + 3584 185.6 / 175.9,
// 1030 + 2565 261.1 / 251.0, 1400 + 4096 383.6 / 366.2; with K and V quantised after projection 300 + 2100 104.3 / 100.9, 1280 + 3840 276.1 / 261.9.
template <int DH, bool VT, bool LOST, int NPAR, bool ENC, bool CUT>
__device__ __forceinline__ void attn_bf16_body(const AttnParams& p, const AttnEncode& e) {
    static_assert(NPAR == 2 || NPAR == 4, "two or four tile parities");
    constexpr int NQG = 8 / NPAR;              // query groups of 32 rows (wavefronts per parity)
    constexpr int kQRows = 32 * NQG;           // query rows per workgroup
    constexpr int CPR = DH / 8;                // 16-byte pieces per K (and row-major V) row
    constexpr int NKS = DH / 16;               // contraction steps of Q.K
    constexpr int NDB = DH / 32;               // 32-wide blocks of the head dimension
    constexpr int PIECES = kAttKV * CPR;       // pieces per tile
    constexpr int kParThreads = kAttThreads / NPAR;        // threads of one key parity
    constexpr int LPT = PIECES / kParThreads;  // transfers per thread per tile
    // [buffer][parity] tiles
    __shared__ u32x4 lds_k[2][NPAR][PIECES];
    __shared__ u32x4 lds_v[2][NPAR][PIECES];
    static_assert(sizeof(lds_k) + sizeof(lds_v) <= 128 * 1024, "tile buffers");
    if constexpr (ENC) {
        static_assert(!ENC || (sizeof(lds_k) >= sizeof(u32x4) * kEncBufs * kEncCbSlots && sizeof(lds_v) >= sizeof(f32x4) * kEncBufs * kEncCnSlots),
                      "the encode's ring of codebook tiles fits the key buffers, its norms the value buffers");
        if ((int)blockIdx.x >= e.n_attn_wgs) {
            u32x4* cb = &lds_k[0][0][0];
            f32x4* cn = reinterpret_cast<f32x4*>(&lds_v[0][0][0]);
            attn_encode_wgs<kAttThreads>(e, (int)blockIdx.x - e.n_attn_wgs, cb, cn);
            return;
        }
    }

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: keeps the tile bookkeeping in scalar registers
    const int i32 = lane & 31, h = lane >> 5;
    // wavefronts w and w + 4 share a SIMD and run in opposite phases; the NQG wavefronts of a parity are consecutive
    const int phase = wave >> 2;
    const int qg = wave & (NQG - 1), par = 2 * ((wave & 3) / NQG) + phase;
    const int ptid = tid & (kParThreads - 1);

    const int n_qb = (p.Tq + kQRows - 1) / kQRows;
    int head, qb, part = 0;
    bool cut = false;
    if (CUT) {
        // one block of every head of the XCD after the other, the whole walks first: the long pieces start first and the short ones fill the end
        int piece;
        if (p.Hq % kXcdsA == 0) {
            const int per_xcd = p.Hq / kXcdsA, slot = blockIdx.x / kXcdsA;
            head = (int)blockIdx.x % kXcdsA * per_xcd + slot % per_xcd;
            piece = slot / per_xcd;
        } else {
            head = (int)blockIdx.x % p.Hq;
            piece = (int)blockIdx.x / p.Hq;
        }
        cut = piece >= p.n_whole;
        qb = cut ? n_qb - 1 - (piece - p.n_whole) / p.n_cut : p.n_whole - 1 - piece;
        part = cut ? (piece - p.n_whole) % p.n_cut : 0;
    } else {
        const int vt_id = xcd_remap_attn(blockIdx.x, ENC ? e.n_attn_wgs : (int)gridDim.x);
        head = vt_id / n_qb;
        qb = n_qb - 1 - (vt_id % n_qb);
    }
    const int hk = head / (p.Hq / p.Hkv);
    const int q0 = qb * kQRows;
    const int Tq = p.Tq;
    const int64_t q_ld = (int64_t)p.Hq * DH, kv_ld = (int64_t)p.Hkv * DH;

    // this lane's query (N side)
    const int qrow = q0 + 32 * qg + i32;
    bf16x8 qf[NKS];
    {
        const int r = qrow < Tq ? qrow : Tq - 1;
        const uint16_t* __restrict__ Q = (const uint16_t*)p.q + (int64_t)r * q_ld + (int64_t)head * DH;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Q + 16 * ks + 8 * h));
    }

    f32x16 acc_o[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[db][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float sl2 = p.scale * 1.4426950408889634f;       // logits in base-2 units

    const int n_hat_tiles = (p.Tn_vis + kAttKV - 1) / kAttKV;
    const int loc_rows = p.causal ? min(q0 + kQRows, Tq) : Tq;    // local keys any row of this block may see
    int n_tiles = n_hat_tiles + (loc_rows + kAttKV - 1) / kAttKV;     // the walk ends before this tile ...
    int n_pairs = (n_tiles + NPAR - 1) / NPAR;
    int t_first = 0;                                                  // ... and begins at this one
    if (CUT && cut) {                                                 // every part has a pair: the launcher sees to it
        const int from = n_pairs * part / p.n_cut, to = n_pairs * (part + 1) / p.n_cut;
        t_first = NPAR * from;
        n_tiles = min(NPAR * to, n_tiles);
        n_pairs = to - from;
    }
    const int wave_q_lo = q0 + 32 * qg;

    // ---- tiles of this wavefront's parity: own iteration i works on tile t_first + NPAR * i + par of the walk (visible
    // non-local tiles first, local tiles after them).  An index past the end (odd tile count) is the last
    // tile again with every key masked, so all wavefronts run the same number of iterations.
    struct Tile {
        bool is_loc;
        int row0, count;
    };
    auto tile_of = [&](int i) {
        const int t_in = t_first + NPAR * i + par;
        const int t = t_in < n_tiles ? t_in : n_tiles - 1;
        Tile tl;
        tl.is_loc = t >= n_hat_tiles;
        tl.row0 = (tl.is_loc ? t - n_hat_tiles : t) * kAttKV;
        tl.count = t_in >= n_tiles ? 0 : (tl.is_loc ? Tq : p.Tn_vis);
        return tl;
    };

    // ---- staging: global -> LDS without passing through registers, by the four wavefronts of the parity that
    // consumes the tile.  One wavefront instruction moves 64 consecutive 16-byte LDS slots; the XOR swizzle is
    // applied on the global side (the lane that owns slot (row, piece) fetches piece ^ swizzle(row) of that row).
    // Slot c = ptid + 256*it of a K tile is (row c / CPR, piece c % CPR); both swizzles are periodic in the row
    // step between two `it`, so the piece a lane fetches is the same for every `it` and only the row changes.
    constexpr int ROW_STEP = kParThreads / CPR;               // K rows between consecutive `it`
    const int kr0 = ptid / CPR, kph = ptid % CPR;
    const uint32_t kcol = (uint32_t)((kph ^ swz_k<DH>(kr0)) * 16);                 // bytes
    const uint32_t vcol = VT ? (uint32_t)(((ptid & 7) ^ swz_vt(ptid >> 3)) * 16)    // V^T: row ptid/8 + 32*it, piece ptid%8
                             : (uint32_t)((kph ^ swz_v<DH>(kr0)) * 16);
    const uint32_t kv_ld_b = (uint32_t)kv_ld * 2u;
    const uint32_t wave_slot = (uint32_t)(64 * qg) * 16u;                      // this wavefront's 64 slots inside a pass of its parity
    constexpr uint32_t kPassBytes = (uint32_t)kParThreads * 16u;
    // byte offset of row kr0 inside a tile; the rows of pass `it` lie ROW_STEP rows further (a scalar product), and a
    // row beyond the source's last one is replaced by that last row by clamping the offset: no per-lane multiply
    const uint32_t krow_b = (uint32_t)kr0 * kv_ld_b;
    auto dma_k = [&](const Tile& tl, int buf, int it) {
        const char* __restrict__ Kb = (const char*)(tl.is_loc ? p.k_loc : p.k_hat) + ((int64_t)tl.row0 * kv_ld + (int64_t)hk * DH) * 2;
        const int lim = (tl.is_loc ? Tq : p.Tn_vis) - 1 - tl.row0;                 // last valid row of the tile
        const uint32_t off = min(krow_b + (uint32_t)(ROW_STEP * it) * kv_ld_b, (uint32_t)min(lim, kAttKV - 1) * kv_ld_b);
        dma_global_to_lds_16(Kb, off + kcol, lds_byte_addr(&lds_k[buf][par][0]) + wave_slot + (uint32_t)it * kPassBytes);
    };
    auto dma_v = [&](const Tile& tl, int buf, int it) {
        const uint32_t dst = lds_byte_addr(&lds_v[buf][par][0]) + wave_slot + (uint32_t)it * kPassBytes;
        if (VT) {
            const uint32_t v_ld_b = (uint32_t)(tl.is_loc ? p.ldv_loc : p.ldv_hat) * 2u;
            const char* __restrict__ Vb = (const char*)(tl.is_loc ? p.v_loc : p.v_hat) + ((int64_t)hk * DH * v_ld_b + (int64_t)tl.row0 * 2);
            // row ptid / 8 + (kParThreads / 8) * it of the transposed tile: one per-lane product per tile source, the pass adds a scalar
            dma_global_to_lds_16(Vb, (uint32_t)(ptid >> 3) * v_ld_b + (uint32_t)((kParThreads / 8) * it) * v_ld_b + vcol, dst);
        } else {
            const char* __restrict__ Vb = (const char*)(tl.is_loc ? p.v_loc : p.v_hat) + ((int64_t)tl.row0 * kv_ld + (int64_t)hk * DH) * 2;
            const int lim = (tl.is_loc ? Tq : p.Tn_vis) - 1 - tl.row0;
            const uint32_t off = min(krow_b + (uint32_t)(ROW_STEP * it) * kv_ld_b, (uint32_t)min(lim, kAttKV - 1) * kv_ld_b);
            dma_global_to_lds_16(Vb, off + vcol, dst);
        }
    };

    // ---- matrix-core phase of iteration i: O^T += V^T(i-1) . P^T(i-1) (PV, 16 MFMAs for dh = 128), then
    // S^T(i) = K(i) . Q^T (QK, 16 MFMAs), in units of NDB / 4 MFMAs.  The fragments of unit u+1 are requested from
    // LDS before the MFMAs of unit u are issued, and the transfers of the tiles needed one iteration later (K(i+1),
    // V(i)) are issued one per unit between the MFMAs, so that no wavefront stalls on the memory pipeline's queue.
    f32x16 acc_s[2];
    bf16x8 pf[4];
    constexpr int QK_UNITS = NKS / 2;
    auto mm_phase = [&](int i, auto parity_tag) {
        constexpr int IB = decltype(parity_tag)::value;          // = i & 1, static: the buffer addresses become immediates
        constexpr int NPV = 4, NU = NPV + QK_UNITS;
        constexpr int NDMA = 2 * LPT;
        const u32x4* __restrict__ Kt = lds_k[IB][par];
        const u32x4* __restrict__ Vt = lds_v[IB ^ 1][par];
        const Tile t_k = tile_of(i + 1), t_v = tile_of(i);
        auto load_unit = [&](int u, bf16x8(&f)[4]) {
            if (u < NPV) {
                const int kstep = u;
#pragma unroll
                for (int db = 0; db < NDB; ++db) {
                    if (VT) {
                        const int d = db * 32 + i32;
                        f[db] = __builtin_bit_cast(bf16x8, Vt[d * 8 + ((2 * kstep + h) ^ swz_vt(d))]);
                    } else {
                        const int s16 = lane & 15, q4 = lane >> 4;
                        const int c = db * 4 + 2 * (q4 & 1) + ((s16 & 3) >> 1);
                        const int r_lo = 16 * kstep + 4 * h + (s16 >> 2);
                        const int r_hi = r_lo + 8;
                        const char* base = reinterpret_cast<const char*>(Vt);
                        const s16x4 lo = lds_read_tr16_b64(base + (r_lo * CPR + (c ^ swz_v<DH>(r_lo))) * 16 + 8 * (s16 & 1));
                        const s16x4 hi = lds_read_tr16_b64(base + (r_hi * CPR + (c ^ swz_v<DH>(r_hi))) * 16 + 8 * (s16 & 1));
                        u32x4 packed;
                        packed.x = (uint16_t)lo[0] | ((uint32_t)(uint16_t)lo[1] << 16);
                        packed.y = (uint16_t)lo[2] | ((uint32_t)(uint16_t)lo[3] << 16);
                        packed.z = (uint16_t)hi[0] | ((uint32_t)(uint16_t)hi[1] << 16);
                        packed.w = (uint16_t)hi[2] | ((uint32_t)(uint16_t)hi[3] << 16);
                        f[db] = __builtin_bit_cast(bf16x8, packed);
                    }
                }
            } else {
                const int g = u - NPV;
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) {
                        const int r = mb * 32 + i32, ks = 2 * g + j;
                        f[j * 2 + mb] = __builtin_bit_cast(bf16x8, Kt[r * CPR + ((2 * ks + h) ^ swz_k<DH>(r))]);
                    }
            }
        };
        auto compute_unit = [&](int u, const bf16x8(&f)[4]) {
            if (u < NPV) {
#pragma unroll
                for (int db = 0; db < NDB; ++db) acc_o[db] = mfma_32x32x16(f[db], pf[u], acc_o[db]);
            } else {
                const int g = u - NPV;
                if (g == 0) {
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc_s[mb][v] = 0.f;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) acc_s[mb] = mfma_32x32x16(f[j * 2 + mb], qf[2 * g + j], acc_s[mb]);
            }
        };
        bf16x8 fa[4], fb[4];
        load_unit(0, fa);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (u + 1 < NU) load_unit(u + 1, (u & 1) ? fa : fb);
            // spread the NDMA transfers over the NU units
#pragma unroll
            for (int x = u * NDMA / NU; x < (u + 1) * NDMA / NU; ++x) {
                if (x < LPT) dma_k(t_k, IB ^ 1, x);
                else dma_v(t_v, IB, x - LPT);
            }
            compute_unit(u, (u & 1) ? fb : fa);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- vector-ALU phase of iteration i: masking and online softmax of S^T(i), in base-2 units, leaving the
    // probabilities as the bf16 B operand of the next PV.  The reference maximum m_run is only raised when a score
    // exceeds it by more than kLazy (2^kLazy fits bf16 and fp32 easily): after the first tiles the accumulators are
    // almost never rescaled.
    auto softmax_phase = [&](int i) {
        const Tile tl = tile_of(i);
        const bool diag = tl.is_loc && p.causal && (tl.row0 + kAttKV - 1 > wave_q_lo);     // some pair of this wave is hidden
        // non-local keys of this tile whose codes never arrived (bit = key index inside the tile; tiles start at
        // multiples of 64 keys, one word of the caller's bit array each; a wave-uniform scalar load)
        unsigned long long lost = 0ull;
        if (LOST && !tl.is_loc && tl.count > 0) lost = ~load_uniform_u64(p.valid_bits + (tl.row0 >> 6));
        // masking (lost codes; ragged source tail, causal diagonal): wave-uniform passes of their own
        // (one pass for a tile that has both holds a word of bits per lane next to the keys' numbers, and on row-major values of 128 spilled in the loop: 32 heads, 300 + 300 rows
        // 21.8 us, 19.0 as two; of 64 12.7 / 11.6)
        if (LOST && lost != 0ull) {
            // Key index inside the tile = 32*mb + 4*h + c(v) with c(v) = acc_row(v, 0): the 32 lanes of
            // a half-wave look at the same key, so the lanes to drop are one scalar word per score, built on the scalar
            // unit from two bits of the tile's word, and each score costs a single select.
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int k0 = 32 * mb + acc_row(v, 0);
                    const unsigned long long lanes = (((lost >> k0) & 1ull) ? 0x00000000ffffffffull : 0ull) |
                                                     (((lost >> (k0 + 4)) & 1ull) ? 0xffffffff00000000ull : 0ull);
                    acc_s[mb][v] = __builtin_amdgcn_inverse_ballot_w64(lanes) ? -INFINITY : acc_s[mb][v];
                }
        }
        if (diag || tl.row0 + kAttKV > tl.count) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = tl.row0 + mb * 32 + acc_row(v, h);
                    const bool drop = (key >= tl.count) | (diag & (key > qrow));
                    acc_s[mb][v] = drop ? -INFINITY : acc_s[mb][v];
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc_s[mb][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * sl2;
        float alpha = 1.f;
        const bool rescale = mx > m_run + kLazy;          // also true for the first visible key (m_run = -inf)
        if (rescale) {
            alpha = __builtin_amdgcn_exp2f(m_run - mx);
            m_run = mx;
        }
        const float m_ref = m_run == -INFINITY ? 0.f : m_run;
        float lsum = 0.f;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float e = __builtin_amdgcn_exp2f(fmaf(acc_s[mb][v], sl2, -m_ref));
                lsum += e;
                pf[mb * 2 + (v >> 3)][v & 7] = (__bf16)e;
            }
        l_run = l_run * alpha + lsum;
        if (__builtin_amdgcn_ballot_w64(rescale) != 0) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc_o[db][v] *= alpha;
        }
    };

    // ---- schedule.  The two wavefronts of a SIMD have different parities; parity 1 runs one phase behind parity 0,
    // and a workgroup barrier closes every phase, so while one wavefront of a SIMD occupies the matrix core the
    // other runs its softmax on the vector ALU:
    //   parity 0:  QK(0) | sm(0) | PV(0) QK(1) | sm(1) | ... | sm(n-1) | PV(n-1) |
    //   parity 1:        | QK(0) | sm(0) | PV(0) QK(1) | ... | PV(n-2) QK(n-1) | sm(n-1) | PV(n-1)
    // A tile's buffer is rewritten (by transfers issued in a matrix-core phase) one barrier-closed iteration after
    // its last reader, and every wavefront waits for its own transfers at the end of its softmax phase, before the
    // barrier that precedes the phase which reads them.
    // The loop body is the same for every iteration: the first PV multiplies zero probabilities with a zeroed V
    // buffer and the last QK (on a finite copy of the last tile) is discarded, 32 of about 1000 MFMAs.
    const int n_it = n_pairs;
    {
        const Tile t0 = tile_of(0);
#pragma unroll
        for (int it = 0; it < LPT; ++it) dma_k(t0, 0, it);
        u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int it = 0; it < LPT; ++it) lds_v[1][par][ptid + kParThreads * it] = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) pf[j] = __builtin_bit_cast(bf16x8, zero);
    }
    wait_vmem_all();
    __syncthreads();
    if (phase == 1) __syncthreads();
    for (int i = 0;; i += 2) {          // two iterations per trip: the tile buffers alternate, so each copy knows its own
        __builtin_amdgcn_s_setprio(2);      // the matrix-core phase goes first when both wavefronts of the SIMD can issue
        mm_phase(i, std::integral_constant<int, 0>{});
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        if (i == n_it) break;
        softmax_phase(i);
        wait_vmem_all();
        __syncthreads();
        __builtin_amdgcn_s_setprio(2);
        mm_phase(i + 1, std::integral_constant<int, 1>{});
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        if (i + 1 == n_it) break;
        softmax_phase(i + 1);
        wait_vmem_all();
        __syncthreads();
    }
    wait_vmem_all();          // transfers issued by the last matrix-core phase land in buffers the merge reuses
    if (phase == 0) __syncthreads();
    __syncthreads();

    // ---- merge the parities of each query group through LDS (the tile buffers are free now): parities 1.. hand their
    // triples to parity 0, which adds them in ascending parity
    float* xch = reinterpret_cast<float*>(&lds_k[0][0][0]);        // NDB*16*64 floats per (query group, parity > 0)
    float* xml = reinterpret_cast<float*>(&lds_v[0][0][0]);        // m, l per (query group, parity > 0, lane)
    static_assert(sizeof(lds_k) >= sizeof(float) * NQG * (NPAR - 1) * NDB * 16 * 64, "the exchange fits the key tiles");
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (par > 0) {
        const int sl = qg * (NPAR - 1) + par - 1;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) xch[((sl * NDB + db) * 16 + v) * 64 + lane] = acc_o[db][v];
        xml[(sl * 2 + 0) * 64 + lane] = m_run;
        xml[(sl * 2 + 1) * 64 + lane] = l_tot;
    }
    __syncthreads();
    if (par == 0) {
        float mo[NPAR - 1], lo[NPAR - 1];
        float m = m_run;
#pragma unroll
        for (int q = 0; q < NPAR - 1; ++q) {
            mo[q] = xml[((qg * (NPAR - 1) + q) * 2 + 0) * 64 + lane];
            lo[q] = xml[((qg * (NPAR - 1) + q) * 2 + 1) * 64 + lane];
            m = fmaxf(m, mo[q]);
        }
        const float m_safe = m == -INFINITY ? 0.f : m;
        const float a0 = __builtin_amdgcn_exp2f(m_run - m_safe);
        float ao[NPAR - 1];
        float l = l_tot * a0;
#pragma unroll
        for (int q = 0; q < NPAR - 1; ++q) {
            ao[q] = __builtin_amdgcn_exp2f(mo[q] - m_safe);
            l += lo[q] * ao[q];
        }
        if (CUT && cut) {
            if (wave_q_lo >= Tq) return;                  // a group without rows
            // a part of a walk: unnormalised, in the register order of the lanes (1 KiB per store), with its maximum and sum per row
            const int slot = (head * (n_qb - p.n_whole) + n_qb - 1 - qb) * p.n_cut + part;
            float* __restrict__ P = p.part + (int64_t)slot * kPartFloats;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    f32x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * vq + e;
                        o[e] = acc_o[db][v] * a0;
#pragma unroll
                        for (int q = 0; q < NPAR - 1; ++q)
                            o[e] += xch[(((qg * (NPAR - 1) + q) * NDB + db) * 16 + v) * 64 + lane] * ao[q];
                    }
                    *reinterpret_cast<f32x4*>(P + (((qg * NDB + db) * 4 + vq) * 64 + lane) * 4) = o;
                }
            if (h == 0) {
                P[kAttQ * DH + 32 * qg + i32] = m;
                P[kAttQ * DH + kAttQ + 32 * qg + i32] = l;
            }
            return;
        }
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const float c0 = a0 * inv;
        float co[NPAR - 1];
#pragma unroll
        for (int q = 0; q < NPAR - 1; ++q) co[q] = ao[q] * inv;
        if (qrow < Tq) {
            uint16_t* __restrict__ O = (uint16_t*)p.out + (int64_t)qrow * q_ld + (int64_t)head * DH;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = 4 * vq + e;
                        o[e] = acc_o[db][v] * c0;
#pragma unroll
                        for (int q = 0; q < NPAR - 1; ++q)
                            o[e] += xch[(((qg * (NPAR - 1) + q) * NDB + db) * 16 + v) * 64 + lane] * co[q];
                    }
                    u32x2 w;
                    w.x = pack_bf16x2(o[0], o[1]);
                    w.y = pack_bf16x2(o[2], o[3]);
                    *reinterpret_cast<u32x2*>(O + db * 32 + 8 * vq + 4 * h) = w;
                }
            if (p.lse && h == 0) p.lse[(int64_t)head * Tq + qrow] = (m + log2f(l)) * 0.6931471805599453f;
        }
    }
}

template <int DH, bool VT, bool LOST = false, int NPAR = 2, bool ENC = false>
__global__ __launch_bounds__(kAttThreads) void attn_bf16_kernel(const AttnParams p, const AttnEncode e) {
    attn_bf16_body<DH, VT, LOST, NPAR, ENC, false>(p, e);
}

template <bool LOST, bool ENC>
__global__ __launch_bounds__(kAttThreads) void attn_cut_kernel(const AttnParams p, const AttnEncode e) {
    attn_bf16_body<128, true, LOST, 2, ENC, true>(p, e);
}

// ------------------------------------------------------------------------------------------------
// The parts of the walks that were cut: O = sum_i 2^(m_i - m) O_i / sum_i 2^(m_i - m) l_i, parts in ascending order.  A wavefront owns 32 rows x 32
// channels of a block, in the lanes' order of the accumulators that wrote them; all parts are requested before the first is needed.  Bound by memory: 16.8 MB, 256 parts, in 5.5 us.
// ------------------------------------------------------------------------------------------------
template <int PARTS>
__global__ __launch_bounds__(256) void attn_merge_kernel(const AttnParams p) {
    constexpr int DH = 128;
    const int n_qb = (p.Tq + kAttQ - 1) / kAttQ;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i32 = lane & 31, h = lane >> 5;
    const int blk = blockIdx.x >> 2, qg = blockIdx.x & 3, db = wave;      // the cut blocks of a head one after the other, the last first
    const int head = blk / (n_qb - p.n_whole), qb = n_qb - 1 - blk % (n_qb - p.n_whole);
    if (qb * kAttQ + 32 * qg >= p.Tq) return;
    const float* __restrict__ P = p.part + (int64_t)blk * PARTS * kPartFloats;
    f32x4 o[PARTS][4];
    float m_i[PARTS], l_i[PARTS];
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
        m_i[i] = P[(int64_t)i * kPartFloats + kAttQ * DH + 32 * qg + i32];
        l_i[i] = P[(int64_t)i * kPartFloats + kAttQ * DH + kAttQ + 32 * qg + i32];
    }
#pragma unroll
    for (int i = 0; i < PARTS; ++i)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
            o[i][vq] = *reinterpret_cast<const f32x4*>(P + (int64_t)i * kPartFloats + (((qg * 4 + db) * 4 + vq) * 64 + lane) * 4);
    float m = m_i[0];
#pragma unroll
    for (int i = 1; i < PARTS; ++i) m = fmaxf(m, m_i[i]);
    const float m_safe = m == -INFINITY ? 0.f : m;
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
        m_i[i] = __builtin_amdgcn_exp2f(m_i[i] - m_safe);
        l += l_i[i] * m_i[i];
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const int row = qb * kAttQ + 32 * qg + i32;
    if (row >= p.Tq) return;
    uint16_t* __restrict__ O = (uint16_t*)p.out + (int64_t)row * p.Hq * DH + (int64_t)head * DH + 32 * db + 4 * h;
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
        f32x4 r = o[0][vq] * (m_i[0] * inv);
#pragma unroll
        for (int i = 1; i < PARTS; ++i) r += o[i][vq] * (m_i[i] * inv);
        u32x2 w;
        w.x = pack_bf16x2(r.x, r.y);
        w.y = pack_bf16x2(r.z, r.w);
        *reinterpret_cast<u32x2*>(O + 8 * vq) = w;
    }
}

static int launch_attn_merge(const AttnParams& p, hipStream_t s) {
    const int blocks = (int)(ceil_div(p.Tq, kAttQ) - p.n_whole) * p.Hq * 4;
    switch (p.n_cut) {
        case 2: attn_merge_kernel<2><<<blocks, 256, 0, s>>>(p); break;
        case 3: attn_merge_kernel<3><<<blocks, 256, 0, s>>>(p); break;
        case 4: attn_merge_kernel<4><<<blocks, 256, 0, s>>>(p); break;
        case 5: attn_merge_kernel<5><<<blocks, 256, 0, s>>>(p); break;
        case 6: attn_merge_kernel<6><<<blocks, 256, 0, s>>>(p); break;
        case 7: attn_merge_kernel<7><<<blocks, 256, 0, s>>>(p); break;
        case 8: attn_merge_kernel<8><<<blocks, 256, 0, s>>>(p); break;
        default: return ASTRA_ERR_UNSUPPORTED;
    }
    return launch_status();
}

// ------------------------------------------------------------------------------------------------
// fp32, vector ALU: one workgroup of four wavefronts per (query row, head).  The keys ([K-hat | K], 64 at a time) are dealt to the wavefronts chunk by
// chunk, each wavefront runs an online softmax over its chunks, and the four partial results are merged through LDS in wavefront order.
//
// In a chunk 16 lanes hold a row, four values (16 bytes) each and 64 further ones per U = ceil(dh / 64), and a load covers four rows; a lane's sixteen
// partial dots (rows 4j + lane / 16) are added over the 16 lanes so that lane (r, c) of the wavefront ends with the logit of row 4c + r.  Bound by the
// latency of the chain keys -> logits -> values, so by the loads in flight on a unit: a wavefront's (JB U at a time, batches beyond a ragged chunk
// left out; the first batch of values lands behind the softmax) times its wavefronts.  Heads of up to 64 take a chunk in one batch, wider ones in batches of eight
// loads, which leaves room for three to four wavefronts per SIMD.  A key per lane and a cache line per lane and load / keys and values of a chunk at once (176 registers
// and more, one or two wavefronts) / this: 64 rows x 3 heads of 64 over 256 keys 7.8 / 4.3 / 4.1 us; 12 heads, 257 rows over 1025 keys: heads of 64
// 146 / 78 / 62, of 128 257 / 131 / 113, of 256 489 / 361 / 225; 100 causal rows, heads of 64 9.1 / 9.1 / 6.5, of 128 12.4 / 11.9 / 8.0, of 256
// 19.2 / 25.6 / 12.5.  (Heads of 64 in two batches of eight: 4.9 for the last of 64, but 0.4 to 0.8 us more for layers whose keys are not in the second-level cache:
// 82 rows over 328 keys 15.6, now 15.0.)  Error against fp64 3.1e-7 of the norm, now 1.5e-7.
// VEC = false: head dimensions or addresses that 16-byte pieces do not fit; a key per lane, 16 of its values at a time (one by one: 3 heads of 50, 64 rows over 256 keys
// 13.0 us, now 10.3; 12 heads of 130, 257 rows over 1025 keys 1766, now 850).
//
// ENC: the workgroups behind the attention's encode the local rows (fp32 codes; nothing here depends on them or the other way round).
// ------------------------------------------------------------------------------------------------
template <int U, bool VEC, bool ENC>
__global__ __launch_bounds__(256) void attn_f32_kernel(const AttnParams p, int dh, const AttnEncode e) {
    constexpr int kWaves = 4;
    constexpr int JB = U == 1 ? 16 : U == 2 ? 4 : 2;       // loads of a batch, 4 rows each, per 64 values of a row
    __shared__ __align__(16) float part[kWaves][U * kWave + 4];
    if constexpr (ENC) {
        __shared__ EncF32Lds enc_lds;
        if ((int)blockIdx.x >= e.n_attn_wgs) {
            int item = (int)blockIdx.x - e.n_attn_wgs;
            const int j = item >= e.job[0].G * e.job[0].n_tb ? 1 : 0;
            if (j) item -= e.job[0].G * e.job[0].n_tb;
            vq_encode_f32_body(e.job[j], item, enc_lds);
            return;
        }
    }
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int head = blockIdx.x / p.Tq, row = blockIdx.x % p.Tq;
    const int hk = head / (p.Hq / p.Hkv);
    const int64_t q_ld = (int64_t)p.Hq * dh, kv_ld = (int64_t)p.Hkv * dh;
    const float* __restrict__ q = (const float*)p.q + (int64_t)row * q_ld + (int64_t)head * dh;
    const int sub = lane & 15, rg = lane >> 4;
    const uint32_t ld_b = (uint32_t)kv_ld * 4u;

    const int n_hat = p.Tn_vis;
    const int n_loc = p.causal ? row + 1 : p.Tq;
    const int chunks_hat = (n_hat + kWave - 1) / kWave, chunks = chunks_hat + (n_loc + kWave - 1) / kWave;
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[U];                     // VEC: values 64u + 4 sub .. + 3 of the rows 4j + rg; else o[u].x is value 64u + lane of all rows
    f32x4 qv[U];
    int col[U];                     // first value of this lane's pieces, clamped into the row; those beyond it count as zeros
#pragma unroll
    for (int u = 0; u < U; ++u) {
        o[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        col[u] = min(64 * u + 4 * sub, dh - 4);
        if (VEC) qv[u] = *reinterpret_cast<const f32x4*>(q + col[u]);
    }

    for (int c = wave; c < chunks; c += kWaves) {
        const int src = c < chunks_hat ? 0 : 1;
        const int base = (src == 0 ? c : c - chunks_hat) * kWave;
        const int cnt = min(kWave, (src == 0 ? n_hat : n_loc) - base);          // rows of the chunk
        const float* __restrict__ Kp = (const float*)(src == 0 ? p.k_hat : p.k_loc) + (int64_t)base * kv_ld + (int64_t)hk * dh;
        const float* __restrict__ Vp = (const float*)(src == 0 ? p.v_hat : p.v_loc) + (int64_t)base * kv_ld + (int64_t)hk * dh;
        const int key = VEC ? 4 * sub + rg : lane;                              // this lane's row in the chunk
        const unsigned long long bits = src != 0 || p.valid_bits == nullptr ? ~0ull : p.valid_bits[base >> 6];
        const bool arrived = key < cnt && ((bits >> key) & 1ull);
        // VEC: values of rows beyond the chunk are zeros (an infinity times a weight of zero is none), their logits are dropped.  Up to 64 values a row the rows are
        // out of a buffer's range, which costs nothing (a layer of 28 rows over 81 keys 11.5 -> 11.3 us); on wider heads, where the buffers' addresses
        // take a wavefront's room (heads of 256 12.6 -> 16.2), they repeat the last row and its values are replaced.
        constexpr bool BUFFERS = U == 1;
        const int range = (int)((uint32_t)(cnt - 1) * ld_b + 4u * (uint32_t)dh);
        const auto k_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Kp, 0, range, 0x00020000), v_buf = __builtin_amdgcn_make_buffer_rsrc((void*)Vp, 0, range, 0x00020000);
        auto piece = [&](const float* base_, __amdgpu_buffer_rsrc_t buf, int j, int u) __attribute__((always_inline)) {
            const uint32_t at = (uint32_t)(BUFFERS ? 4 * j + rg : min(4 * j + rg, cnt - 1)) * ld_b + (uint32_t)col[u] * 4u;
            if (BUFFERS) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)at, 0, 0));
            return *reinterpret_cast<const f32x4*>((const char*)base_ + at);
        };
        constexpr int kRows = VEC ? 1 : U <= 2 ? 16 : 8;        // not VEC: value rows in flight, the first of them on narrow heads sent before the keys
        constexpr bool EARLY = U <= 2;
        float x[kRows][U];
        auto load_rows = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < kRows; ++b)
#pragma unroll
                for (int u = 0; u < U; ++u) x[b][u] = Vp[(int64_t)min(r0 + b, cnt - 1) * kv_ld + min(lane + 64 * u, dh - 1)];
        };
        f32x4 vv[JB][U];                                   // VEC: a batch of values
        auto load_values = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u) vv[j][u] = piece(Vp, v_buf, b + j, u);
        };
        float s;
        if (VEC) {
            float dot[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) dot[j] = 0.f;
#pragma unroll
            for (int b = 0; b < 16; b += JB) {
                if (b > 0 && 4 * b >= cnt) break;
                f32x4 kk[JB][U];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int j = 0; j < JB; ++j) kk[j][u] = piece(Kp, k_buf, b + j, u);
                __builtin_amdgcn_sched_barrier(0);         // all of them are on their way before the first is waited for
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool in = 64 * u + 4 * sub < dh;
#pragma unroll
                    for (int j = 0; j < JB; ++j) {
                        float d = dot[b + j];
                        d = fmaf(qv[u].x, kk[j][u].x, d);
                        d = fmaf(qv[u].y, kk[j][u].y, d);
                        d = fmaf(qv[u].z, kk[j][u].z, d);
                        d = fmaf(qv[u].w, kk[j][u].w, d);
                        dot[b + j] = in ? d : dot[b + j];
                    }
                }
                // worked out here: moved behind the branches that follow, the sums would keep the keys of all batches alive
#pragma unroll
                for (int j = 0; j < JB; ++j) asm volatile("" : "+v"(dot[b + j]));
                __builtin_amdgcn_sched_barrier(0);
            }
            load_values(0);                                // lands behind the softmax
            __builtin_amdgcn_sched_barrier(0);
            // sixteen sums over sixteen lanes: every step halves the sums a lane still carries
            auto halve = [&](auto n) __attribute__((always_inline)) {
                constexpr int W = decltype(n)::value;
                const bool up = (sub & W) != 0;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    const float keep = up ? dot[j + W] : dot[j], give = up ? dot[j] : dot[j + W];
                    dot[j] = keep + __shfl_xor(give, W);
                }
            };
            halve(std::integral_constant<int, 8>{});
            halve(std::integral_constant<int, 4>{});
            halve(std::integral_constant<int, 2>{});
            halve(std::integral_constant<int, 1>{});
            s = dot[0] * p.scale;
        } else {
            if (EARLY) load_rows(0);
            const float* kr = Kp + (int64_t)key * kv_ld;
            float d = 0.f;
            // a row per lane (none for the keys that are not there), 16 values at a time and the rest at once
            auto take = [&](int i, auto n) __attribute__((always_inline)) {
                constexpr int N = decltype(n)::value;
                float kk[N];
#pragma unroll
                for (int t = 0; t < N; ++t) kk[t] = kr[min(i + t, dh - 1)];
#pragma unroll
                for (int t = 0; t < N; ++t) d = i + t < dh ? fmaf(q[min(i + t, dh - 1)], kk[t], d) : d;
            };
            if (arrived) {
                int i = 0;
                for (; i + 16 <= dh; i += 16) take(i, std::integral_constant<int, 16>{});
                if (dh - i > 12) take(i, std::integral_constant<int, 16>{});
                else if (dh - i > 8) take(i, std::integral_constant<int, 12>{});
                else if (dh - i > 4) take(i, std::integral_constant<int, 8>{});
                else if (dh - i > 0) take(i, std::integral_constant<int, 4>{});
            }
            s = d * p.scale;
        }
        if (!arrived) s = -INFINITY;
        float mx = s;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        const float m_new = fmaxf(m_run, mx);          // -inf only while every key so far was lost
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = expf(m_run - m_safe);
        const float w = arrived ? expf(s - m_safe) : 0.f;
        float sum = w;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        l_run = l_run * alpha + sum;
        m_run = m_new;
        if (VEC) {
            float wj[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) wj[j] = __shfl(w, (lane & 48) | j);      // weight of row 4j + rg
#pragma unroll
            for (int u = 0; u < U; ++u) o[u] *= alpha;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < 16; b += JB) {
                if (b > 0 && 4 * b >= cnt) break;
                if (b > 0) load_values(b);
                if (!BUFFERS && 4 * (b + JB) > cnt)
#pragma unroll
                    for (int j = 0; j < JB; ++j)
#pragma unroll
                        for (int u = 0; u < U; ++u) vv[j][u] = 4 * (b + j) + rg < cnt ? vv[j][u] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < JB; ++j)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        o[u].x = fmaf(wj[b + j], vv[j][u].x, o[u].x);
                        o[u].y = fmaf(wj[b + j], vv[j][u].y, o[u].y);
                        o[u].z = fmaf(wj[b + j], vv[j][u].z, o[u].z);
                        o[u].w = fmaf(wj[b + j], vv[j][u].w, o[u].w);
                    }
#pragma unroll
                for (int u = 0; u < U; ++u) asm volatile("" : "+v"(o[u]));
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) o[u].x *= alpha;
            for (int r0 = 0; r0 < cnt; r0 += kRows) {
                if (!EARLY || r0 > 0) load_rows(r0);
#pragma unroll
                for (int b = 0; b < kRows; ++b) {
                    const float wr = __shfl(w, r0 + b);
#pragma unroll
                    for (int u = 0; u < U; ++u) o[u].x = r0 + b < cnt ? fmaf(wr, x[b][u], o[u].x) : o[u].x;
                }
            }
        }
    }
    // merge: wavefront w leaves (o, m, l); the first wavefront adds the four in order
    if (VEC) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int off = 16; off < 64; off <<= 1)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[u][i] += __shfl_xor(o[u][i], off);
            if (rg == 0) *reinterpret_cast<f32x4*>(&part[wave][64 * u + 4 * sub]) = o[u];
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) part[wave][u * kWave + lane] = o[u].x;
    }
    if (lane == 0) {
        part[wave][U * kWave] = m_run;
        part[wave][U * kWave + 1] = l_run;
    }
    __syncthreads();
    if (wave != 0) return;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, part[w][U * kWave]);
    const float m_safe = M == -INFINITY ? 0.f : M;
    float L = 0.f;
    float r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const float wgt = expf(part[w][U * kWave] - m_safe);       // exp(-inf) = 0 for a wavefront without keys
        L = fmaf(wgt, part[w][U * kWave + 1], L);
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = fmaf(wgt, part[w][u * kWave + lane], r[u]);
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    float* __restrict__ out = (float*)p.out + (int64_t)row * q_ld + (int64_t)head * dh;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int d = lane + 64 * u;
        if (d < dh) out[d] = r[u] * inv;
    }
    if (p.lse && lane == 0) p.lse[(int64_t)head * p.Tq + row] = M + logf(L);
}

template <int U>
static void launch_attn_f32(int blocks, const AttnParams& p, int head_dim, const AttnEncode& e, hipStream_t s) {
    const bool vec = head_dim % 4 == 0 && (int64_t)p.Hkv * head_dim * 4 * kWave < (1ll << 32) &&       // offsets in a chunk are 32 bits wide
                     ((uintptr_t)p.q | (uintptr_t)p.k_loc | (uintptr_t)p.k_hat | (uintptr_t)p.v_loc | (uintptr_t)p.v_hat) % 16 == 0;
    if (e.n_enc_wgs > 0) {
        if (vec) attn_f32_kernel<U, true, true><<<blocks, 256, 0, s>>>(p, head_dim, e);
        else attn_f32_kernel<U, false, true><<<blocks, 256, 0, s>>>(p, head_dim, e);
    } else {
        if (vec) attn_f32_kernel<U, true, false><<<blocks, 256, 0, s>>>(p, head_dim, e);
        else attn_f32_kernel<U, false, false><<<blocks, 256, 0, s>>>(p, head_dim, e);
    }
}

// 16.5 us and its start at K = 1024, dg = 64, beside other work.  (By quads an item of one block per wavefront takes what it took before: 1000 tokens x 64 groups, K = 1024
// as a kernel of its own 13.9 us, 13.7; K = 256 6.6, 6.2.)
static double encode_item_us(const EncodeJob& e) { return 256.0 * e.K * e.dg / 1048576.0 + 2.5; }

// About how long an attention launch lasts with `items` workgroups of encodes behind its own, by either kernel, every block walked whole (us).
static double attention_us(const AttnParams& p, bool few, int64_t items, double item) {
    const int64_t total = ceil_div(p.Tq, few ? 32 : kAttQ) * p.Hq, rounds = ceil_div(total, (int64_t)kAttCus);
    const int64_t more = ceil_div(total + items, (int64_t)kAttCus) - rounds;
    const double tiles = (double)(p.Tn_vis + p.Tq) / kAttKV;                // a workgroup walks them all
    const double walk = few ? 5.0 + 0.8 * tiles : 6.0 + 1.1 * tiles;
    return walk * rounds + (items == 0 ? 0.0 : more > 0 ? more * item : std::max(0.0, item - walk));
}

struct AttnCut {
    int n_whole, n_cut;      // n_cut 0: every block is walked whole
    double us;
};

// Tiles that a query block of a head walks
struct Walks {
    int n_qb, hat, loc;
    bool causal;
    explicit Walks(const AttnParams& p)
        : n_qb((int)ceil_div(p.Tq, kAttQ)), hat((int)ceil_div(p.Tn_vis, kAttKV)), loc((int)ceil_div(p.Tq, kAttKV)), causal(p.causal != 0) {}
    int tiles(int qb) const { return hat + (causal ? std::min(kAttQ / kAttKV * (qb + 1), loc) : loc); }
    int64_t all() const {      // of all blocks; only the last one may be short of its two tiles
        return (int64_t)n_qb * hat + (causal ? (int64_t)(n_qb - 1) * n_qb * (kAttQ / kAttKV) / 2 + loc : (int64_t)n_qb * loc);
    }
};

// About how long the launch lasts with the first `w` blocks of a head walked whole and the others in `c` parts (us): the units' mean load, or what the
// number of pieces leaves of it, and the partial results on their way out and back in.  A tile takes the longer the more units are at it (0.73 us on 32 of
// them, 0.81 on 96, 1.01 on 256: the clock and the second-level caches are everyone's); 6 us go before the first and after the last.
// `best` or more where the mean load alone says so: the rest, whose cost grows with the rounds, is for the few that are left.
static double cut_us(const AttnParams& p, const Walks& walks, int w, int c, int64_t items, double item, double best) {
    const int n_qb = walks.n_qb, per_head = w + (n_qb - w) * c;
    const int64_t pieces = (int64_t)per_head * p.Hq;
    const double tile = 0.69 + 0.00125 * std::min<int64_t>(pieces + items, kAttCus);
    auto piece_us = [&](int k) { return 6.0 + tile * walks.tiles(k < w ? w - 1 - k : n_qb - 1 - (k - w) / c) / (k < w ? 1 : c); };
    // 16.8 MB of partial results behind a single round: 12 us; behind whole walks they leave while others still run
    const double behind = (items > 0 ? 0.25 * item : 0.0) +
                          (w == n_qb ? 0.0 : (w > 0 ? 5.0 : 4.0) + (w > 0 ? 1.0 : 2.0) * (p.Tq - w * kAttQ) * c * p.Hq * 520.0 / 4.0e6);
    double us = ((6.0 * per_head + tile * walks.all()) * p.Hq + items * item) / kAttCus;
    if (us + behind >= best) return us + behind;
    for (int64_t j = 0; j * kAttCus < pieces; ++j) us = std::max(us, (j + 1) * piece_us((int)(j * kAttCus / p.Hq)));
    if (pieces <= kAttCus && pieces + items > kAttCus) us = std::max(us, item + (pieces < kAttCus ? std::min(item, piece_us(per_head - 1)) : piece_us(per_head - 1)));
    return us + behind;
}

static size_t cut_bytes(const AttnParams& p, int w, int c) { return (size_t)(ceil_div(p.Tq, kAttQ) - w) * c * p.Hq * kPartFloats * sizeof(float); }

static AttnCut attention_cut(const AttnParams& p, int head_dim, int64_t items, double item, size_t part_bytes) {
    AttnCut best = {0, 0, 0.0};
    const Walks walks(p);
    const int n_qb = walks.n_qb;
    if (head_dim != 128 || !p.v_transposed || p.lse || (int64_t)n_qb * p.Hq > 4 * kAttCus) return best;
    best.us = cut_us(p, walks, n_qb, 1, items, item, INFINITY);
    for (int j = 0; j * kAttCus / p.Hq < n_qb; ++j) {
        const int w = j * kAttCus / p.Hq;
        const int pairs = (int)ceil_div(walks.tiles(w), 2);      // of the shortest one cut
        // Encodes aboard are work for units that whole walks leave idle, and the estimate of a cut knows little of that: parts of walks of fewer than 16 tiles have to
        // promise 3 us (17 and 40 + 588 rows, 16 groups, K and V quantised after projection: whole 38.2, 41.5 us, cut 38.8, 42.4 with 1 - 2 promised; 8 heads,
        // not causal, 20 + 627: 24.5 / 29.1 with 3).
        const double margin = items > 0 && walks.tiles(n_qb - 1) < 16 ? 3.0 : 0.0;
        for (int c = 2; c <= kMaxParts && c <= pairs; ++c) {
            if (cut_bytes(p, w, c) > part_bytes) break;
            const double us = cut_us(p, walks, w, c, items, item, best.us - margin) + margin;
            if (us < best.us) best = {w, c, us};
        }
    }
    return best;
}

// A workgroup per 32 query rows (attention_short_kernels.hip) where those make a single round of the units, and where encodes in the launch do not
// lose the units that fewer workgroups would leave them.  Whole layers, there / on the kernel above:
// 12 heads of 64, 256 + 768 / 256 + 8000 rows 23.7 / 27.4, 64.7 / 79.0 us; 700 + 700 rows (264 workgroups) 37.4 / 38.0, 700 + 3000 56.6 / 50.3.
// 32 heads of 128 over 8 KV heads, 17 + 51 rows 29.8 / 32.8, 128 + 384 47.2 / 53.0, 256 + 768 71 / 78, 256 + 4096 130 / 149; 384 + 1152 rows (two rounds)
// 94.4 / 93.7, 512 + 4096 174 / 168.  With the encodes of K and V, 1024 codewords each, in the launch: 100 + 300 rows 40.6 / 44.3, but 256 + 768, whose
// workgroups take every unit, 66.5 / 64.2.
static bool attention_short(const AttnParams& p, int head_dim, int64_t items, double item) {
    if ((head_dim != 64 && head_dim != 128) || !p.v_transposed || ceil_div(p.Tq, 32) * p.Hq > kAttCus) return false;
    return items == 0 || attention_us(p, true, items, item) < attention_us(p, false, items, item);
}

// The kernel of a launch and where its walks are cut.  The short form gives way where its walk takes longer than parts of one on the kernel above do.  Encodes
// take turns on the units without a query block; those that are not done within the walk slow all of it a little and end it, at the latest an encode later.
// Had they to wait for the walk, it would give way too early: layers 4096 wide with the encodes of K and V aboard, 1024 codewords, 84 + 588 rows, 32 groups
// 45.5 us cut, 41.1 short; 16 groups 40 + 1000 43.5 / 39.2, 200 + 1000 65.0 / 58.8; with one encode, 64 groups, 128 + 1000 77.6 / 73.0.
static AttnCut attention_form(const AttnParams& p, int head_dim, int64_t items, double item, size_t part_bytes, bool* few) {
    *few = attention_short(p, head_dim, items, item);
    const AttnCut cut = attention_cut(p, head_dim, items, item, part_bytes);
    if (!*few || cut.n_cut == 0) return cut;
    const int64_t units = ceil_div(p.Tq, 32) * p.Hq, idle = kAttCus - units;
    const double tiles = (double)(p.Tn_vis + p.Tq) / kAttKV, crowd = 0.56 * units / kAttCus;
    double us = 5.0 + std::max(0.37, crowd) * tiles;
    if ((double)idle * std::floor(us / std::max(item, 1.0)) < (double)items) {
        const double beside = 5.0 + std::max(0.43, crowd) * tiles, waiting = us + item;
        us = idle > 0 ? std::min(waiting, std::max(beside, (double)ceil_div(items, idle) * item)) : waiting;
    }
    *few = us < cut.us + 1.0;
    return *few ? AttnCut{0, 0, 0.0} : cut;
}

double attention_encode_us(const AttnParams& p, int head_dim, const EncodeJob& e) {
    if (head_dim != 128 || !p.v_transposed || e.n_tokens <= 0 || !vq_encode_fast_ok(e.K, e.dg)) return -1.0;
    const int64_t items = ceil_div(e.n_tokens, kAttThreads / 2) * e.G;
    const double item = encode_item_us(e);
    const double with = attention_us(p, attention_short(p, head_dim, items, item), items, item);
    return std::max(0.0, with - attention_us(p, attention_short(p, head_dim, 0, 0.0), 0, 0.0));
}

// Work items of the encodes that the general kernels' launch carries behind its own workgroups (128-wide heads on transposed V: the instantiations built);
// 0: it does not carry them.
static int64_t carried_items(const AttnParams& p, int head_dim, const EncodeJob* enc, int n_enc) {
    if (!enc || n_enc < 1 || n_enc > 2 || head_dim != 128 || !p.v_transposed || ceil_div(p.Tq, kAttQ) * p.Hq + kAttCus > 0x7fffffff) return 0;
    int64_t items = 0;
    for (int j = 0; j < n_enc; ++j) {
        const int64_t n_tb = ceil_div(enc[j].n_tokens, kAttThreads / 2);
        if (enc[j].n_tokens <= 0 || !vq_encode_fast_ok(enc[j].K, enc[j].dg) || n_tb * enc[j].G > 0x3fffffff || enc[j].dg != enc[0].dg) return 0;
        items += n_tb * enc[j].G;
    }
    return items;
}

size_t attention_part_bytes(int dtype, const AttnParams& p, int head_dim, const EncodeJob* enc, int n_enc) {
    if (dtype != ASTRA_BF16 || p.Tq == 0) return 0;
    const int64_t items = carried_items(p, head_dim, enc, n_enc);
    bool few = false;
    const AttnCut cut = attention_form(p, head_dim, items, items > 0 ? encode_item_us(enc[0]) : 0.0, SIZE_MAX, &few);
    return cut.n_cut > 1 ? cut_bytes(p, cut.n_whole, cut.n_cut) : 0;
}

int launch_attention(int dtype, const AttnParams& p_in, int head_dim, hipStream_t s, bool plan_only, const EncodeJob* enc, int n_enc,
                     bool* enc_fused, const Prefetch* fetch) {
    AttnParams p = p_in;
    if (enc_fused) *enc_fused = false;
    if (p.Tq == 0) return ASTRA_OK;
    AttnEncode ae{};
    if (dtype == ASTRA_BF16) {
        int64_t total = (int64_t)ceil_div(p.Tq, kAttQ) * p.Hq;
        if (total > 0x7fffffff) return ASTRA_ERR_SHAPE;
        const bool vt = p.v_transposed != 0;
        const bool lost = p.valid_bits != nullptr;
        if (head_dim != 64 && head_dim != 128) return ASTRA_ERR_UNSUPPORTED;
        // the kernel forms byte offsets inside one head's tile source in 32 bits: rows of the transposed V buffers
        // (head_dim of them, ldv tokens each) and 64 key rows of H_kv * head_dim elements
        if (vt && (int64_t)max(p.ldv_loc, p.ldv_hat) * 2 * head_dim >= (1ll << 32)) return ASTRA_ERR_UNSUPPORTED;
        if ((int64_t)p.Hkv * head_dim * 2 * kAttKV >= (1ll << 32)) return ASTRA_ERR_UNSUPPORTED;
        int64_t items = enc_fused ? carried_items(p, head_dim, enc, n_enc) : 0;      // encodes offered by the caller ride in the launch's tail
        // 64-wide heads otherwise: when 128-row query blocks would leave half of the compute units without a
        // workgroup, 64-row blocks whose tiles are dealt to four wavefronts per query group (half the iterations each)
        if (plan_only) return ASTRA_OK;
        bool few = false;
        const AttnCut cut = attention_form(p, head_dim, items, items > 0 ? encode_item_us(enc[0]) : 0.0, p.part ? p.part_bytes : 0, &few);
        p.n_whole = cut.n_whole;
        p.n_cut = cut.n_cut;
        // Whole walks of unequal length in more than a round: the longest of all heads first, so that the short ones are what the last round is made of.  A
        // head after the other, the last head's longest blocks start when most are done (us, a head after the other / longest first): layers 4096 wide of
        // 1531 + 2565 rows 282 / 273, 1531 + 900 226 / 218, 1400 + 4096 344 / 337, with K and V quantised after projection 1531 + 2565 259 / 253.
        if (p.n_cut == 0 && !few && head_dim == 128 && vt && p.causal && total > kAttCus && p.Hq % kXcdsA == 0 && !p.lse) {
            p.n_whole = (int)ceil_div(p.Tq, kAttQ);
            p.n_cut = 1;
        }
        const bool four = !few && head_dim == 64 && total <= kAttCus / 2;
        if (few || four) total = (int64_t)ceil_div(p.Tq, few ? 32 : kAttQ / 2) * p.Hq;
        if (p.n_cut > 1) total = (p.n_whole + (ceil_div(p.Tq, kAttQ) - p.n_whole) * p.n_cut) * p.Hq;
        if (items > 0) {
            const int tb = vq_encode_blocks(enc[0], kAttCus / n_enc);
            items = 0;
            for (int j = 0; j < n_enc; ++j) {
                ae.job[j] = enc[j];
                ae.job[j].tb = tb;
                ae.job[j].n_tb = (int)ceil_div(enc[j].n_tokens, kAttThreads / 2 * tb);
                items += (int64_t)ae.job[j].n_tb * enc[j].G;
            }
            ae.n_jobs = n_enc;
            ae.n_attn_wgs = (int)total;
            ae.n_enc_wgs = (int)std::min<int64_t>(items, kAttCus);
            *enc_fused = true;
        }
        // An encode of wide groups rides beside the short form on units without a query block.  Layers 4096 wide, encode as a launch
        // of its own / beside: 40 + 120 rows, 16 groups 53.6 / 45.7 us, 32 groups 49.2 / 42.0, 100 + 300 70.2 / 61.1, 66.0 / 57.7.
        if (items == 0 && few && enc && enc_fused && n_enc == 1 && head_dim == 128 && enc[0].n_tokens > 0 &&
            vq_encode_stream_fits(enc[0].K, enc[0].dg, enc[0].ldx) && vq_encode_on_16(enc[0].x, enc[0].codebook, enc[0].cnorm)) {
            const int64_t n_tb = ceil_div(enc[0].n_tokens, kStreamTokens), wgs = n_tb * enc[0].G;
            if (total + wgs <= kAttCus) {
                ae.job[0] = enc[0];
                ae.job[0].n_tb = (int)n_tb;
                ae.n_jobs = 1;
                ae.n_attn_wgs = (int)total;
                ae.n_enc_wgs = (int)wgs;
                *enc_fused = true;
            }
        }
        if (few) return launch_attention_short(p, head_dim, ae, fetch, s);
        if (p.n_cut > 0) {
            const int grid = (int)total + ae.n_enc_wgs;
            if (ae.n_enc_wgs > 0 && lost) attn_cut_kernel<true, true><<<grid, kAttThreads, 0, s>>>(p, ae);
            else if (ae.n_enc_wgs > 0) attn_cut_kernel<false, true><<<grid, kAttThreads, 0, s>>>(p, ae);
            else if (lost) attn_cut_kernel<true, false><<<grid, kAttThreads, 0, s>>>(p, ae);
            else attn_cut_kernel<false, false><<<grid, kAttThreads, 0, s>>>(p, ae);
            const int rc = launch_status();
            return rc || p.n_cut == 1 ? rc : launch_attn_merge(p, s);
        }
        if (ae.n_enc_wgs > 0) {
            if (lost) attn_bf16_kernel<128, true, true, 2, true><<<(int)total + ae.n_enc_wgs, kAttThreads, 0, s>>>(p, ae);
            else attn_bf16_kernel<128, true, false, 2, true><<<(int)total + ae.n_enc_wgs, kAttThreads, 0, s>>>(p, ae);
        } else if (head_dim == 128) {
            if (vt && lost) attn_bf16_kernel<128, true, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (vt) attn_bf16_kernel<128, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (lost) attn_bf16_kernel<128, false, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else attn_bf16_kernel<128, false><<<(int)total, kAttThreads, 0, s>>>(p, ae);
        } else if (four) {
            if (vt && lost) attn_bf16_kernel<64, true, true, 4><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (vt) attn_bf16_kernel<64, true, false, 4><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (lost) attn_bf16_kernel<64, false, true, 4><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else attn_bf16_kernel<64, false, false, 4><<<(int)total, kAttThreads, 0, s>>>(p, ae);
        } else if (head_dim == 64) {
            if (vt && lost) attn_bf16_kernel<64, true, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (vt) attn_bf16_kernel<64, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else if (lost) attn_bf16_kernel<64, false, true><<<(int)total, kAttThreads, 0, s>>>(p, ae);
            else attn_bf16_kernel<64, false><<<(int)total, kAttThreads, 0, s>>>(p, ae);
        } else {
            return ASTRA_ERR_UNSUPPORTED;
        }
    } else {
        if (head_dim > 256 || p.v_transposed) return ASTRA_ERR_UNSUPPORTED;
        const int64_t blocks = (int64_t)p.Hq * p.Tq;
        if (blocks > 0x7fffffff) return ASTRA_ERR_SHAPE;
        int64_t items = 0;
        for (int j = 0; j < (enc && enc_fused && n_enc <= 2 ? n_enc : 0); ++j) {
            ae.job[j] = enc[j];
            ae.job[j].n_tb = (int)ceil_div(enc[j].n_tokens, kEncF32Tokens);
            items += (int64_t)ae.job[j].n_tb * enc[j].G;
        }
        if (items > 0 && blocks + items <= 0x7fffffff) {
            ae.n_jobs = n_enc;
            ae.n_attn_wgs = (int)blocks;
            ae.n_enc_wgs = (int)items;
            *enc_fused = true;
        }
        if (plan_only) return ASTRA_OK;
        const int grid = (int)blocks + ae.n_enc_wgs;
        switch ((head_dim + 63) / 64) {
            case 1: launch_attn_f32<1>(grid, p, head_dim, ae, s); break;
            case 2: launch_attn_f32<2>(grid, p, head_dim, ae, s); break;
            case 3: launch_attn_f32<3>(grid, p, head_dim, ae, s); break;
            default: launch_attn_f32<4>(grid, p, head_dim, ae, s); break;
        }
    }
    return launch_status();
}

}  // namespace astra
