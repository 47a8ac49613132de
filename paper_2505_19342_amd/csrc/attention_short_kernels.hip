// Mixed-precision attention of one device (paper Sec. 3.2, Eq. 1) for launches that a few large workgroups cannot fill: short sequences, few heads.
#include "attention_encode.h"
#include "prefetch.h"

#include <algorithm>
#include <type_traits>

namespace astra {

// ------------------------------------------------------------------------------------------------
// bf16, matrix cores, flash style, V transposed (the layout of the projection kernel's kCTransposedV).  The arithmetic is attn_bf16_kernel's: scores
// S^T = K . Q^T with the keys on the M side of the 32x32x16 MFMA, a lane's scores all of one query, probabilities already in the layout of the B operand
// of O^T += V^T . P^T, a reference maximum that is raised lazily.
//
// A workgroup of eight wavefronts owns 32 query rows of one head; wavefront w walks the tiles w, w + 8, ... of 4096 / DH keys (64 or 32; visible
// non-local ones first) for itself: direct transfers bring its keys and values into LDS of its own (8 KiB each, XOR-swizzled pieces), so that the loop has
// no barrier and no other wavefront to wait for.  A tile's fragments are read into registers whole, and its place takes the wavefront's next tile at once.  The
// reference maxima start from the ones attn_bf16_kernel would have (its wavefronts' first tiles: a quarter of the 64-key tiles each on 64-wide heads, half on
// 128-wide ones), exchanged once through LDS: probabilities are then rounded to bf16 on the same scale and a row's output does not depend on which of
// the two took it but for the order of fp32 sums (layers' outputs then differ by 2e-5 of the norm instead of 2e-3, for 0.5 us of a ViT layer's 23.9); where
// that kernel cuts its walks, every part has maxima of its own, and the outputs differ by 2e-3.  The
// eight (max, sum, O) triples meet in LDS, and every thread adds four of the workgroup's outputs in wavefront order.
//
// What bounds it: a launch, a memory latency at either end, and what the second-level caches give all units together (4 DH bytes a key for every 32
// queries: 32 heads of 128, 256 + 4096 rows are 570 MB in about 50 us; with the fragments loaded straight into registers, 32 rows a load, a short launch
// took several times as long).
// 12 heads, causal, whole layer on attn_bf16_kernel (64 query rows per workgroup, tiles shared by two wavefronts) and here: 17 rows 16.3 -> 13.8 us,
// 256 + 768 rows 26.0 -> 23.1, 512 + 1024 35.2 -> 31.4.  32 heads of 128 (128 query rows per workgroup before): 17 rows 27.4 -> 24.2, 128 + 384
// 53.0 -> 47.2, 256 + 4096 149 -> 130.
//
// ENC: VQ encodes ride in the launch (AttnEncode).  Units that are left read ahead (prefetch.h).
// Longer walks and more rows are better off sharing tiles through LDS (launch_attention).
// ------------------------------------------------------------------------------------------------
constexpr int kShortThreads = 512;
constexpr int kShortWaves = kShortThreads / kWave;
constexpr float kLazyShort = 8.f;     // base-2 units
constexpr int kShortUnits = 256;      // compute units of the device

// WIDTH: the head's, and in its lowest bit that the encode aboard is one of wide groups (job 0, a workgroup per item), which wants another body.  (The walk as a
// function shared by two kernels compiled to 60 more instructions, 0.7 % of a layer of 40 rows.)
constexpr int kStreamed = 1;
template <int WIDTH, bool LOST, bool ENC>
__global__ __launch_bounds__(kShortThreads) void attn_short_kernel(const AttnParams p, const AttnEncode e, const Prefetch f) {
    constexpr int DH = WIDTH & ~kStreamed;
    constexpr int TK = 4096 / DH, NMB = TK / 32, NKS = DH / 16, NDB = DH / 32, NPV = TK / 16, LDP = DH + 4;
    constexpr int KP = DH / 8, VP = TK / 8;    // 16-byte pieces of a row of keys, of values
    constexpr int NT = 8, KR = 64 / KP, VR = 64 / VP;      // transfers of a tile of keys or of values, and their rows
    constexpr int kTile = TK * KP;             // pieces of a tile: keys [TK keys][DH values], values [DH values][TK keys]
    constexpr int kPart = kShortWaves * 32 * LDP / 4;      // the partial outputs, once every wavefront is done with its tiles
    __shared__ __align__(16) u32x4 ring[kPart > kShortWaves * 2 * kTile ? kPart : kShortWaves * 2 * kTile];
    __shared__ float part_m[kShortWaves][32], part_l[kShortWaves][32];
    auto part = reinterpret_cast<float(*)[32][LDP]>(&ring[0]);
    if constexpr (ENC && (WIDTH & kStreamed)) {
        static_assert(sizeof(ring) >= sizeof(u32x4) * (kStreamSlots + kStreamCnSlots) && kStreamWaves == kShortWaves && kStreamTokens == 32, "the streamed encode's rings fit");
        const int item = (int)blockIdx.x - e.n_attn_wgs;
        if (item >= 0 && item < e.n_enc_wgs) {
            f32x4* cn = reinterpret_cast<f32x4*>(ring + kStreamSlots);
            auto arg = reinterpret_cast<int(*)[32]>(&part_l[0]);
            if (e.job[0].dg == 128) vq_encode_stream_run<2>(e.job[0], item, ring, cn, part_m, arg);
            else if (e.job[0].dg == 192) vq_encode_stream_run<3>(e.job[0], item, ring, cn, part_m, arg);
            else vq_encode_stream_run<4>(e.job[0], item, ring, cn, part_m, arg);
            return;
        }
    } else if constexpr (ENC) {
        static_assert(sizeof(ring) >= sizeof(u32x4) * kEncBufs * (kEncCbSlots + kEncCnSlots), "the encode's codebook tiles and norms fit");
        if ((int)blockIdx.x >= e.n_attn_wgs && (int)blockIdx.x < e.n_attn_wgs + e.n_enc_wgs) {
            attn_encode_wgs<kShortThreads>(e, (int)blockIdx.x - e.n_attn_wgs, ring, reinterpret_cast<f32x4*>(ring + kEncBufs * kEncCbSlots));
            return;
        }
    }

    // the arguments arrive together, before the branch on one of them
    asm volatile("" ::"s"(e.n_attn_wgs), "s"(p.q), "s"(p.k_loc), "s"(p.v_loc), "s"(p.k_hat), "s"(p.v_hat), "s"(p.out), "s"(p.Hq), "s"(p.Hkv), "s"(p.Tq),
                 "s"(p.Tn_vis), "s"(p.causal), "s"(p.ldv_loc), "s"(p.ldv_hat), "s"(p.scale));
    if ((int)blockIdx.x >= e.n_attn_wgs) {
        prefetch_wgs<kShortThreads>(f, blockIdx.x - (uint32_t)(e.n_attn_wgs + e.n_enc_wgs));
        return;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i32 = lane & 31, h = lane >> 5;
    const int Tq = p.Tq, n_qb = (Tq + 31) / 32;
    // contiguous runs of heads per XCD, so that a KV head's keys and values stay in one L2; later (longer) query blocks first
    const int total = e.n_attn_wgs, xq = total / 8, xr = total % 8, xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int vid = xcd < xr ? xcd * (xq + 1) + slot : xr * (xq + 1) + (xcd - xr) * xq + slot;
    const int head = vid / n_qb, q0 = (n_qb - 1 - vid % n_qb) * 32;
    const int hk = head / (p.Hq / p.Hkv);
    const int64_t q_ld = (int64_t)p.Hq * DH;
    const uint32_t kv_ld_b = (uint32_t)p.Hkv * DH * 2u;

    const int qrow = q0 + i32;
    bf16x8 qf[NKS];
    {
        const uint16_t* __restrict__ Q = (const uint16_t*)p.q + (int64_t)min(qrow, Tq - 1) * q_ld + (int64_t)head * DH;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Q + 16 * ks + 8 * h));
    }
    const int n_hat_tiles = (p.Tn_vis + TK - 1) / TK;
    const int loc_rows = p.causal ? min(q0 + 32, Tq) : Tq;        // local keys any row of this block may see
    const int n_tiles = n_hat_tiles + (loc_rows + TK - 1) / TK;

    struct Tile {
        bool is_loc;
        int row0, count;
    };
    auto tile_of = [&](int t) {
        Tile tl;
        tl.is_loc = t >= n_hat_tiles;
        tl.row0 = (tl.is_loc ? t - n_hat_tiles : t) * TK;
        tl.count = tl.is_loc ? Tq : p.Tn_vis;
        return tl;
    };
    // Slot c of row r of a tile holds piece c ^ swizzle(r), by which the rows a fragment read takes at a time lie in different banks.
    // Transfer j of a tile fills rows KR j + lane / KP of keys, VR j + lane / VP of values.  Rows beyond the source's last one are copies of it;
    // their scores are dropped.
    auto swz_keys = [](int r) __attribute__((always_inline)) { return DH == 128 ? r & 15 : (r >> 1) & 7; };
    auto swz_vals = [](int r) __attribute__((always_inline)) { return DH == 128 ? (r >> 2) & 3 : (r >> 1) & 7; };
    const int rk = lane / KP, rv = lane / VP;
    u32x4* const tiles = &ring[wave * 2 * kTile];
    const uint32_t lds_k = lds_byte_addr(tiles), lds_v = lds_byte_addr(tiles + kTile);
    auto send_k = [&](const Tile& tl) __attribute__((always_inline)) {
        const char* __restrict__ base = (const char*)(tl.is_loc ? p.k_loc : p.k_hat) + ((int64_t)tl.row0 * kv_ld_b + (int64_t)hk * (DH * 2));
        const uint32_t lim = (uint32_t)min(tl.count - 1 - tl.row0, TK - 1) * kv_ld_b;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const uint32_t piece = 16u * ((lane % KP) ^ swz_keys(KR * j + rk));
            dma_global_to_lds_16(base, min((uint32_t)rk * kv_ld_b + (uint32_t)(KR * j) * kv_ld_b, lim) + piece, lds_k + 1024u * j);
        }
    };
    auto send_v = [&](const Tile& tl) __attribute__((always_inline)) {
        const uint32_t v_ld_b = (uint32_t)(tl.is_loc ? p.ldv_loc : p.ldv_hat) * 2u;
        const char* __restrict__ base = (const char*)(tl.is_loc ? p.v_loc : p.v_hat) + ((int64_t)hk * DH * v_ld_b + (int64_t)tl.row0 * 2);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const uint32_t piece = 16u * ((lane % VP) ^ swz_vals(VR * j + rv));
            dma_global_to_lds_16(base, (uint32_t)rv * v_ld_b + (uint32_t)(VR * j) * v_ld_b + piece, lds_v + 1024u * j);
        }
    };
    // fragment (row block, step) of a tile in LDS: lane holds row 32 block + lane % 32, piece 2 step + lane / 32
    auto frag_k = [&](int block, int step) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, tiles[(32 * block + i32) * KP + ((2 * step + h) ^ swz_keys(i32))]);
    };
    auto frag_v = [&](int block, int step) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, tiles[kTile + (32 * block + i32) * VP + ((2 * step + h) ^ swz_vals(i32))]);
    };
    auto reads_done = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xC07F);      // the fragments are in registers (lgkmcnt 0): their place is free
        asm volatile("" ::: "memory");
    };

    f32x16 acc_o[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[db][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float sl2 = p.scale * 1.4426950408889634f;       // logits in base-2 units

    if (wave < n_tiles) {
        send_k(tile_of(wave));
        send_v(tile_of(wave));
    } else {
        if (h == 0) part_m[wave][i32] = -INFINITY;
        __syncthreads();                         // the others' meeting over their first tiles
    }
    for (int t = wave; t < n_tiles; t += kShortWaves) {
        const Tile tl = tile_of(t), next = tile_of(min(t + kShortWaves, n_tiles - 1));
        const bool more = t + kShortWaves < n_tiles;
        bf16x8 kf[NMB][NKS], vf[NDB][NPV];
        wait_vmem<NT>();                         // the keys have landed, their values may be outstanding
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) kf[mb][ks] = frag_k(mb, ks);
        reads_done();
        if (more) send_k(next);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc_s[NMB];
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_s[mb][v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) acc_s[mb] = mfma_32x32x16(kf[mb][ks], qf[ks], acc_s[mb]);

        const bool diag = tl.is_loc && p.causal && (tl.row0 + TK - 1 > q0);          // some pair of this tile is hidden
        unsigned long long lost = 0ull;                                              // non-local keys whose codes never arrived
        if (LOST && !tl.is_loc) {                                                    // bit = key of the tile
            lost = ~load_uniform_u64(p.valid_bits + (tl.row0 >> 6)) >> (tl.row0 & 63);
        }
        if (diag || tl.row0 + TK > tl.count || lost != 0ull) {
            const uint32_t lost_w[2] = {(uint32_t)(lost >> (4 * h)), (uint32_t)(lost >> (32 + 4 * h))};
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int key = tl.row0 + mb * 32 + acc_row(v, h);
                    const bool drop = (key >= tl.count) | (diag & (key > qrow)) | (((lost_w[mb] >> acc_row(v, 0)) & 1u) != 0u);
                    acc_s[mb][v] = drop ? -INFINITY : acc_s[mb][v];
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc_s[mb][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * sl2;
        if (t == wave) {
            if (h == 0) part_m[wave][i32] = mx;
            __syncthreads();
            m_run = DH == 64 ? part_m[wave & 3][i32] : fmaxf(part_m[wave & 2][i32], part_m[(wave & 2) | 1][i32]);
        }
        float alpha = 1.f;
        const bool rescale = mx > m_run + kLazyShort;          // also true for the first visible key (m_run = -inf)
        if (rescale) {
            alpha = __builtin_amdgcn_exp2f(m_run - mx);
            m_run = mx;
        }
        const float m_ref = m_run == -INFINITY ? 0.f : m_run;
        float lsum = 0.f;
        bf16x8 pf[NPV];
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb)
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
        if (more) wait_vmem<NT>();               // the values have landed, the next keys may be outstanding
        else wait_vmem_all();
#pragma unroll
        for (int u = 0; u < NPV; ++u)
#pragma unroll
            for (int db = 0; db < NDB; ++db) vf[db][u] = frag_v(db, u);
        reads_done();
        if (more) send_v(next);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NPV; ++u)
#pragma unroll
            for (int db = 0; db < NDB; ++db) acc_o[db] = mfma_32x32x16(vf[db][u], pf[u], acc_o[db]);
    }

    // ---- merge: lane (query i32, half h) holds O^T rows 32 db + 8 vq + 4h .. + 3 in values 4 vq .. 4 vq + 3
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    __syncthreads();
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
            *reinterpret_cast<f32x4*>(&part[wave][i32][db * 32 + 8 * vq + 4 * h]) =
                f32x4{acc_o[db][4 * vq], acc_o[db][4 * vq + 1], acc_o[db][4 * vq + 2], acc_o[db][4 * vq + 3]};
    if (h == 0) {
        part_m[wave][i32] = m_run;
        part_l[wave][i32] = l_tot;
    }
    __syncthreads();
    constexpr int PER_ROW = DH / 4;
#pragma unroll
    for (int i = tid; i < 32 * PER_ROW; i += kShortThreads) {
        const int r = i / PER_ROW, d = i % PER_ROW * 4;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) m = fmaxf(m, part_m[w][r]);
        const float m_safe = m == -INFINITY ? 0.f : m;
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kShortWaves; ++w) {
            const float a = __builtin_amdgcn_exp2f(part_m[w][r] - m_safe);             // 0 for a wavefront without keys
            l += part_l[w][r] * a;
            o += *reinterpret_cast<const f32x4*>(&part[w][r][d]) * a;
        }
        const float inv = l > 0.f ? 1.f / l : 0.f;
        if (q0 + r < Tq) {
            u32x2 w;
            w.x = pack_bf16x2(o.x * inv, o.y * inv);
            w.y = pack_bf16x2(o.z * inv, o.w * inv);
            *reinterpret_cast<u32x2*>((uint16_t*)p.out + (int64_t)(q0 + r) * q_ld + (int64_t)head * DH + d) = w;
            if (p.lse && d == 0) p.lse[(int64_t)head * Tq + q0 + r] = (m + log2f(l)) * 0.6931471805599453f;
        }
    }
}

int launch_attention_short(const AttnParams& p, int head_dim, const AttnEncode& e_in, const Prefetch* fetch, hipStream_t s) {
    AttnEncode e = e_in;
    e.n_attn_wgs = (int)(ceil_div(p.Tq, 32) * p.Hq);
    Prefetch f{};
    if (fetch) f = fetch->on(kShortUnits - e.n_attn_wgs - e.n_enc_wgs, kShortThreads);
    const int grid = e.n_attn_wgs + e.n_enc_wgs + f.n_wgs;
    const bool lost = p.valid_bits != nullptr;
    if (head_dim == 64) {
        if (lost) attn_short_kernel<64, true, false><<<grid, kShortThreads, 0, s>>>(p, e, f);
        else attn_short_kernel<64, false, false><<<grid, kShortThreads, 0, s>>>(p, e, f);
    } else if (e.n_enc_wgs > 0 && e.job[0].dg > kEncKt) {
        if (lost) attn_short_kernel<128 | kStreamed, true, true><<<grid, kShortThreads, 0, s>>>(p, e, f);
        else attn_short_kernel<128 | kStreamed, false, true><<<grid, kShortThreads, 0, s>>>(p, e, f);
    } else if (e.n_enc_wgs > 0) {
        if (lost) attn_short_kernel<128, true, true><<<grid, kShortThreads, 0, s>>>(p, e, f);
        else attn_short_kernel<128, false, true><<<grid, kShortThreads, 0, s>>>(p, e, f);
    } else {
        if (lost) attn_short_kernel<128, true, false><<<grid, kShortThreads, 0, s>>>(p, e, f);
        else attn_short_kernel<128, false, false><<<grid, kShortThreads, 0, s>>>(p, e, f);
    }
    return launch_status();
}

}  // namespace astra
