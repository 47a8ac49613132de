// Linear projections C[M,N] = A[M,K] . B[N,K]^T (+ bias) for the attention layer (the projections
// named under Eq. 1 of the paper): Q, K, V of the local rows, K-hat, V-hat of the rows rebuilt from
// codes, and the output projection.  Several problems run in one grouped launch; a problem may take
// its A rows straight from the codebook through the token codes (decode fused into the operand load).
// This file holds the layer's instantiations of the bf16 tile kernel and the launcher; the instantiations for the MLP of the
// surrounding block are compiled in gemm_mlp_kernels.hip, the fp32 kernel in gemm_f32_kernels.hip.
#include "gemm_bf16_tile.h"
#include "gemm_bf16_wave.h"

#include <algorithm>
#include <cmath>

namespace astra {

// row tiles of a problem; a transposed store covers the padded rows too
static int64_t tile_rows(const GemmProblem& p, int bm) {
    return ceil_div(p.c_mode == kCTransposedV && p.ldc > p.M ? p.ldc : p.M, bm);
}

static int fill_batch(GemmBatch& batch, int dtype, const GemmProblem* problems, int n_problems, int bm, int bn, int* total_out) {
    int total = 0, n = 0;
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = problems[i];
        if (p.M <= 0 || p.N <= 0) continue;
        if (p.K <= 0) return ASTRA_ERR_SHAPE;
        if (dtype == ASTRA_BF16) {
            const int64_t lim = (int64_t)1 << 31;
            // whole 64-wide contraction tiles; 16-byte operand pieces must not straddle rows or codewords
            if (p.K % kBK != 0 || (!p.codes && p.lda % 8 != 0) || (p.codes && p.dg % 8 != 0)) return ASTRA_ERR_UNSUPPORTED;
            if (p.c_mode == kCTransposedV && (p.ldc % 64 != 0 || p.ldc < p.M)) return ASTRA_ERR_SHAPE;
            if (p.c_mode == kCSwiGLU && (p.N % 2 != 0 || p.ldc < p.N / 2)) return ASTRA_ERR_SHAPE;
            if (p.residual && (p.c_mode != kCF32 || p.act != kActNone || (int64_t)p.M * p.ldc * 4 >= lim)) return ASTRA_ERR_UNSUPPORTED;
            if ((p.c_mode == kCTransposedV || p.c_mode == kCSwiGLU) && p.act != kActNone) return ASTRA_ERR_UNSUPPORTED;
            // operands are addressed with 32-bit byte offsets from their base
            if (p.ldb != 0 && (p.ldb < p.K || p.ldb % 8 != 0)) return ASTRA_ERR_UNSUPPORTED;
            if ((int64_t)p.M * p.lda * 2 >= lim || (int64_t)p.N * (p.ldb ? p.ldb : p.K) * 2 >= lim) return ASTRA_ERR_UNSUPPORTED;
            if (p.codes && ((int64_t)p.G * p.Kc * p.dg * 2 >= lim || (int64_t)p.M * p.G * 2 >= lim)) return ASTRA_ERR_UNSUPPORTED;
        } else if (p.c_mode != kCF32) {
            return ASTRA_ERR_UNSUPPORTED;
        }
        const int64_t tm = tile_rows(p, bm), tn = ceil_div(p.N, bn);
        const int64_t nt = tm * tn;
        if (nt + total > 0x7fffffff) return ASTRA_ERR_SHAPE;
        batch.p[n] = p;
        batch.tile_begin[n] = total;
        batch.tiles_m[n] = (int)tm;
        total += (int)nt;
        ++n;
    }
    batch.n = n;
    for (int i = n; i <= kMaxGemmProblems; ++i) batch.tile_begin[i] = total;
    *total_out = total;
    return ASTRA_OK;
}

// Tiles of a set of problems at a tile shape (0 when a problem is rejected: the caller's own pass reports the error).
static int64_t count_tiles(const GemmProblem* problems, int n_problems, int bm, int bn) {
    int64_t t = 0;
    for (int i = 0; i < n_problems; ++i)
        if (problems[i].M > 0 && problems[i].N > 0) t += tile_rows(problems[i], bm) * ceil_div(problems[i].N, bn);
    return t;
}

// ---- durations (us) by which a launch's form is chosen, fitted to 4819 products of 4 - 6000 rows, 64 - 8192 columns and contractions of
// 64 - 14336, every form timed on each (20 launches back to back).  In 99 of 100 the form chosen is within 3.4 % of the fastest the product
// has had, with the forms there are or with the two-contraction-group tiles they took the place of; 14 % off at most but for a few of more than
// 4000 rows over 2000 - 5000 (30 %).  Gathered rows: 1087 layers of 17 - 1500 rows at three widths, every form of their projection launch timed,
// within 4 % in 99 of 100.

constexpr double kLaunchUs = 4.0;             // a dependent launch that does next to nothing

struct FormTimes {
    double first, first_k;        // the first workgroup of a unit, and its part per 1000 of contraction
    double next, next_k;          // one more, where that makes the number of workgroups on the unit even ...
    double pair, pair_k;          // ... and two more (two fit a unit at a time, or this is twice the line above)
    double store;                 // TB/s at which results leave: a round's stores are all issued at its end
    double fetch;                 // TB/s at which operands come in at best
    double codes = 0, codes_k = 0, codes_next = 0, codes_next_k = 0;      // gathered rows, on top of what they add to the tile kernel: the codes are
                                  // copied to LDS before a workgroup fetches anything, which two on a unit hide from each other; ... per further round
    double from_memory = 1.0;     // factor where the weights are too large for the second-level caches
};
// 2000 x 4096 outputs over K = 64: 16.4 us on 64 x 64 tiles (a workgroup's start, reduction and stores come again in every round), 25.6 on 32 x 32,
// 10.8 on 128 x 256.  6 x 718 x 1024 over K = 128 in one launch after another: 89.8 on 64 x 64, 79.3 on 128 x 128 of the tile kernel.
// 64 x 1024 over K = 1024: 3.7 on 32 x 32, 11.5 on 128 x 128.
constexpr FormTimes kWaveTimes[kWaveConfigs] = {
    {2.8, 0.91, 0.0, 1.6, 0.75, 2.6, 5.0, 6.0, 2.0, -1.5, 0.4, -0.1},      // 32 x 32
    {3.1, 1.55, 0.9, 2.6, 1.8, 5.2, 2.65, 6.0, 2.8, -1.2, 0.3, 1.1},       // 64 x 32
    {3.3, 2.45, 1.1, 3.2, 2.2, 6.4, 3.3, 6.0, 2.5, -0.7, 1.4, 0.4},        // 64 x 64, two stages
    {3.4, 2.9, 0.0, 2.3, 0.4, 5.9, 3.8, 6.0, 2.2, -1.1, 0.6, -0.2, 1.04},  // 64 x 64, one stage
    {4.5, 4.6, 1.2, 5.9, 2.4, 11.8, 2.9, 6.0, 3.0, 0.1, 1.9, 1.1},         // 128 x 64
    {6.5, 6.05, 1.2, 8.2, 2.4, 16.4, 2.9, 6.0, 3.3, 0.9, 3.4, 2.1}};       // 128 x 128
constexpr FormTimes kTile256 = {8.6, 18.9, 4.4, 22.0, 8.8, 44.0, 8.4, 4.2};       // 256 x 256
constexpr FormTimes kTile128x256 = {5.5, 10.3, 5.5, 10.3, 11.0, 20.6, 6.7, 4.2};  // a single round
// 128 x 128 on eight wavefronts.  Its two stages do not cover a round trip to memory: a Llama block of 335 rows took 337 us with its projections on
// these tiles and 317 with them on the wavefront-private ones, which are level when the same layer is repeated and the weights stay in the caches
// (2543 products with weights of 15 - 300 MB that change with every launch: 1.6 times the time below, 1.1 - 1.4 for the other forms).
constexpr FormTimes kTile128 = {3.7, 8.35, 1.0, 2.0, 4.0, 10.0, 4.5, 4.2, 0, 0, 0, 0, 1.25};
constexpr double kCachedWeights = 16e6;       // bytes; half of the second-level caches

static bool plain_layer(const GemmProblem* problems, int n_problems) {
    for (int i = 0; i < n_problems; ++i)
        if (problems[i].c_mode == kCSwiGLU || problems[i].act != kActNone || problems[i].residual) return false;
    return true;
}

static double form_us(const FormTimes& f, const GemmProblem* problems, int n_problems, int64_t tiles) {
    double k = 0.0, operands = 0.0, weights = 0.0, results = 0.0;
    bool gather = false;
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = problems[i];
        if (p.M <= 0 || p.N <= 0) continue;
        k = std::max(k, p.K * 1e-3);
        gather = gather || p.codes;
        weights += (double)p.N * p.K * 2.0;
        if (!p.codes) operands += (double)p.M * p.K * 2.0;
        results += (double)p.M * p.N * (p.c_mode == kCF32 ? 4.0 : p.c_mode == kCSwiGLU ? 1.0 : 2.0);
    }
    const double more = (double)(std::max<int64_t>(ceil_div(tiles, (int64_t)kCus), 1) - 1), pairs = std::floor(more / 2.0), odd = more - 2.0 * pairs;
    const double compute = f.first + f.first_k * k + odd * (f.next + f.next_k * k) + pairs * (f.pair + f.pair_k * k);
    // Rows from a codebook in the caches come in sooner than others, which is no gain in a launch of few rounds, or of the smallest tiles, that waits for
    // its weights.  A layer 4096 wide of 87 + 43 rows: 54.2 us with its projections on 64 x 64 in two stages, 58.5 in one, which the bound below keeps
    // from being 1.4 us ahead here; over the layers above, the form chosen is 0.18 % slower than the fastest on average, 0.26 without the bound.
    double codes = gather ? f.codes + f.codes_k * k + more * (f.codes_next + f.codes_next_k * k) : 0.0;
    if (gather && (more <= 1.0 || &f == &kWaveTimes[0])) codes = std::max(codes, -0.5);
    const double us = codes + std::max(compute, 3.0 + (operands + weights) / (f.fetch * 1e6)) + results / (f.store * 1e6);
    return weights > kCachedWeights ? us * f.from_memory : us;
}

// the tile kernel's form for a set of problems, in the order launch_gemm_batch picks it
static const FormTimes& tile_form(const GemmProblem* problems, int n_problems, int64_t* tiles) {
    const int64_t big = count_tiles(problems, n_problems, 256, 256);
    if (plain_layer(problems, n_problems) && big <= 128) {
        *tiles = count_tiles(problems, n_problems, 128, 256);
        if (*tiles > kCus / 2 && *tiles <= kCus) return kTile128x256;
    }
    *tiles = big >= 128 ? big : count_tiles(problems, n_problems, 128, 128);
    return big >= 128 ? kTile256 : kTile128;
}

static double tile_launch_us(const GemmProblem* problems, int n_problems, bool can_split) {
    int64_t tiles = 0;
    const FormTimes& f = tile_form(problems, n_problems, &tiles);
    const GemmProblem& p0 = problems[0];
    const int ns = can_split && &f == &kTile128 && n_problems == 1 && !plain_layer(problems, 1) && p0.c_mode == kCF32 && p0.ldc % 4 == 0
                       ? gemm_split_factor(ASTRA_BF16, p0.M, p0.N, p0.K) : 1;
    if (ns > 1) {
        // the sliced contraction and its reduction.  The other forms' times fall short by a fifth over contractions as long as these
        // (1024 x 4096 outputs, K = 14336: 130 us sliced and 135 on 128 x 128 tiles; 2048 x 2048, K = 8192: 83 and 72)
        GemmProblem slice = p0;
        slice.K = p0.K / ns;
        const double mn = (double)p0.M * p0.N * 4.0;
        return 0.8 * (form_us(kTile256, &slice, 1, count_tiles(problems, 1, 256, 256) * ns) + (ns - 1.0) * mn / (kTile256.store * 1e6) + 4.5 +
                      (ns + 2.0) * mn / 5.0e6);
    }
    return form_us(f, problems, n_problems, tiles);
}

// LDS bytes for a tile's codes (the largest of the problems); -1: they do not fit beside the ring
static int wave_code_bytes(const GemmProblem* problems, int n_problems, int cfg) {
    int64_t need = 0;
    for (int i = 0; i < n_problems; ++i)
        if (problems[i].codes && problems[i].M > 0) need = std::max<int64_t>(need, (int64_t)kWaveTable[cfg].bm * problems[i].G * problems[i].code_bytes);
    need = (int64_t)align_up((size_t)need, 16);
    return kWaveTable[cfg].lds + need <= 156 * 1024 ? (int)need : -1;
}

// ---- the encode of the local rows, offered to a projection launch.  An item is 128 tokens of one group on four wavefronts, or 256 on eight.
static double encode_item_us(const EncodeJob& e) { return 256.0 * e.K * e.dg / 1048576.0; }      // its codewords; 2.5 us before the first of them
// otherwise: in a later launch, or as one of its own (two items share a unit in 0.9 of their time)
static double encode_later_us(const EncodeJob& e, double later_us) {
    if (later_us >= 0.0) return later_us;
    const double items = (double)ceil_div(e.n_tokens, (int64_t)kWaveThreads / 2) * e.G;
    return kLaunchUs + 2.5 + encode_item_us(e) * std::max(1.0, 0.45 * items / kCus);
}

// Workgroups for it in a launch of `tiles` 256 x 256 or 128 x 256 tiles; 0: it does not ride.  It takes units that the last round leaves idle, and
// must not outlast the tiles by more than it costs later (16.5 us measured for an item at K = 1024, dg = 64).
static int tile_encode_wgs(const EncodeJob& e, int64_t tiles, bool mid, int k_max) {
    const int rem = (int)(tiles % kCus), E = rem == 0 ? 0 : (kCus - rem) & ~7;
    const int64_t items = ceil_div(e.n_tokens, 256) * e.G;
    const double tile_us = (mid ? 70.0 : 105.0) * k_max / 4096.0;      // 52 and 92 measured, and what a launch of its own would add
    return E >= 8 && E <= kCus / 2 && items <= 0x7fffffff && (double)ceil_div(items, (int64_t)E) * encode_item_us(e) <= 1.05 * tile_us ? E : 0;
}

// The same in a launch of the wavefront-private kernel that lasts `us` without it; *extra_us: what the encode adds, riding or later.  It rides
// in what room the last round leaves, from when that round begins, if it outlasts the products by less than it costs later.
static int wave_encode_wgs(const EncodeJob& e, const WaveConfig& wc, int64_t tiles, double us, double later_us, double* extra_us) {
    const int64_t items = ceil_div(e.n_tokens, (int64_t)kWaveThreads / 2) * e.G, slots = (int64_t)kCus * wc.per_cu;
    const int64_t room = (ceil_div(tiles, slots) * slots - tiles) & ~(int64_t)7;
    const int64_t E = std::min<int64_t>(align_up((size_t)items, 8), room > 0 ? std::min<int64_t>(room, kCus) : kCus);
    const double ride = (double)ceil_div(items, E) * (encode_item_us(e) + 2.5), later = encode_later_us(e, later_us);
    const double begins = room > 0 ? us * (1.0 - 1.0 / (double)std::max<int64_t>(ceil_div(tiles, slots), 1)) : us;
    const double over = std::max(0.0, begins + ride - us);
    *extra_us = std::min(over, later);
    return items <= 0x7fffffff && over < later ? (int)E : 0;
}

struct WaveChoice {
    int cfg;                 // -1: none applies
    int enc_wgs;             // workgroups for the encode
    double us;               // with the encode, riding or later
};

// the fastest wavefront-private form of a set of problems; enc: the encode it is offered (nullable)
static WaveChoice best_wave(const GemmProblem* problems, int n_problems, const EncodeJob* enc, double enc_later_us) {
    WaveChoice best = {-1, 0, 0.0};
    for (int i = 0; i < n_problems; ++i) {
        const GemmProblem& p = problems[i];
        if (p.M > 0 && (p.N % 8 != 0 || p.ldc % 4 != 0)) return best;          // four consecutive columns per thread
    }
    for (int cfg = 0; cfg < kWaveConfigs; ++cfg) {
        if (wave_code_bytes(problems, n_problems, cfg) < 0) continue;
        const int64_t tiles = count_tiles(problems, n_problems, kWaveTable[cfg].bm, kWaveTable[cfg].bn);
        const double t = form_us(kWaveTimes[cfg], problems, n_problems, tiles);
        double extra = 0.0;
        const int E = enc ? wave_encode_wgs(*enc, kWaveTable[cfg], tiles, t, enc_later_us, &extra) : 0;
        if (best.cfg < 0 || t + extra < best.us) best = {cfg, E, t + extra};
    }
    return best;
}

static double launch_us(const GemmProblem* problems, int n_problems) {
    const double t = tile_launch_us(problems, n_problems, false);
    const WaveChoice w = best_wave(problems, n_problems, nullptr, -1.0);
    return w.cfg >= 0 && w.us < t ? w.us : t;
}

int launch_gemm_batch(int dtype, const GemmProblem* problems, int n_problems, hipStream_t s, const EncodeJob* enc, bool* enc_fused,
                      bool plan_only, void* split_ws, size_t split_ws_bytes, bool may_cut, double enc_later_us) {
    if (enc_fused) *enc_fused = false;
    if (n_problems > kMaxGemmProblems) return ASTRA_ERR_UNSUPPORTED;
    // A launch whose last round of 256 x 256 tiles is nearly empty lasts a whole tile longer for a few tiles.  When the
    // problems can be dealt into two launches that are shorter together (say one that fills its rounds and a small one
    // on smaller tiles), run those: the launches are independent and follow each other on the stream.
    if (dtype == ASTRA_BF16 && may_cut && n_problems >= 2) {
        const int64_t big = count_tiles(problems, n_problems, 256, 256);
        if (plain_layer(problems, n_problems) && big > kCus && big % kCus != 0 && big % kCus <= 3 * kCus / 8) {
            const double whole = launch_us(problems, n_problems);
            double best = whole - 10.0;        // a second launch has to pay for itself with some margin
            unsigned best_mask = 0;
            GemmProblem a[kMaxGemmProblems], b[kMaxGemmProblems];
            for (unsigned mask = 1; mask + 1 < (1u << n_problems); ++mask) {
                int na = 0, nb = 0;
                for (int i = 0; i < n_problems; ++i) ((mask >> i) & 1u ? a[na++] : b[nb++]) = problems[i];
                const double t = launch_us(a, na) + launch_us(b, nb);
                if (t < best) { best = t; best_mask = mask; }
            }
            if (best_mask != 0) {
                int na = 0, nb = 0;
                for (int i = 0; i < n_problems; ++i) ((best_mask >> i) & 1u ? a[na++] : b[nb++]) = problems[i];
                bool fused_a = false, fused_b = false;
                int rc;
                if (!plan_only) {               // every problem is checked before the first of the two launches
                    rc = launch_gemm_batch(dtype, a, na, s, nullptr, nullptr, true, nullptr, 0, false);
                    if (rc) return rc;
                    rc = launch_gemm_batch(dtype, b, nb, s, nullptr, nullptr, true, nullptr, 0, false);
                    if (rc) return rc;
                }
                rc = launch_gemm_batch(dtype, a, na, s, enc, enc ? &fused_a : nullptr, plan_only, nullptr, 0, false, enc_later_us);
                if (rc) return rc;
                rc = launch_gemm_batch(dtype, b, nb, s, fused_a ? nullptr : enc, enc && !fused_a ? &fused_b : nullptr, plan_only,
                                       nullptr, 0, false, enc_later_us);
                if (enc_fused) *enc_fused = fused_a || fused_b;
                return rc;
            }
        }
    }
    GemmBatch batch{};
    int total = 0;
    if (dtype != ASTRA_BF16) {
        // the largest tile that still gives three quarters of the units one: 257 x 576 outputs, K = 192: 10.0 / 5.8 / 5.4 us on tiles of 64 / 32 / 16;
        // 500 x 768, K = 768: 21.2 / 15.8 / 18.5; 1000 x 1000, K = 1000: 27.4 on 64, 37.2 on 32
        int tile = 128;
        do {
            tile /= 2;
            const int rc = fill_batch(batch, dtype, problems, n_problems, tile, tile, &total);
            if (rc) return rc;
        } while (tile > 16 && total > 0 && total < 3 * kCus / 4);
        return plan_only ? ASTRA_OK : launch_gemm_f32(tile, batch, s);
    }
    bool code16 = false, mlp = false;
    for (int i = 0; i < n_problems; ++i) {
        if (problems[i].codes && problems[i].code_bytes == 2) code16 = true;
        if (problems[i].c_mode == kCSwiGLU || problems[i].act != kActNone || problems[i].residual) mlp = true;
    }
    int epi = kEpiLayer;
    if (mlp) {
        // the MLP's GEMMs and the residual-adding output projection of a block: plain A rows, one problem per launch
        if (n_problems != 1 || problems[0].codes) return ASTRA_ERR_UNSUPPORTED;
        const GemmProblem& p0 = problems[0];
        if (p0.c_mode == kCSwiGLU) epi = kEpiSwiGLU;
        else if (p0.c_mode == kCBf16 && p0.act == kActGeluTanh) epi = kEpiGeluTanh;
        else if (p0.c_mode == kCBf16 && p0.act == kActGeluErf) epi = kEpiGeluErf;
        else if (p0.c_mode == kCF32 && p0.act == kActNone) epi = kEpiResidualF32;
        else return ASTRA_ERR_UNSUPPORTED;
    }
    const EncodeJob* offered = enc && enc_fused && epi == kEpiLayer && enc->n_tokens > 0 && vq_encode_fast_ok(enc->K, enc->dg) ? enc : nullptr;
    const WaveChoice wave = best_wave(problems, n_problems, offered, enc_later_us);
    double tile_us = tile_launch_us(problems, n_problems, plan_only || split_ws != nullptr);
    int k_max = 0;
    for (int i = 0; i < n_problems; ++i) k_max = std::max(k_max, problems[i].K);
    if (offered) {
        int64_t tiles = 0;
        const FormTimes& f = tile_form(problems, n_problems, &tiles);
        if (&f == &kTile128 || tile_encode_wgs(*enc, tiles, &f == &kTile128x256, k_max) == 0) tile_us += encode_later_us(*enc, enc_later_us);
    }
    if (wave.cfg >= 0 && wave.us < tile_us) {
        const WaveConfig& wc = kWaveTable[wave.cfg];
        int rc = fill_batch(batch, dtype, problems, n_problems, wc.bm, wc.bn, &total);
        if (rc) return rc;
        if (total == 0) return ASTRA_OK;
        bool gather = false;
        for (int i = 0; i < batch.n; ++i) gather = gather || batch.p[i].codes != nullptr;
        if (wave.enc_wgs > 0) {
            batch.n_enc_wgs = wave.enc_wgs;
            batch.enc = *enc;
            batch.enc.tb = 1;
            batch.enc.n_tb = (int)ceil_div(enc->n_tokens, kWaveThreads / 2);
            *enc_fused = true;
        }
        if (plan_only) return ASTRA_OK;
        return launch_gemm_wave(wave.cfg, epi, gather, batch, total + batch.n_enc_wgs, wave_code_bytes(problems, n_problems, wave.cfg), s);
    }
    if (mlp) {
        const GemmProblem& p0 = problems[0];
        int rc = fill_batch(batch, dtype, problems, n_problems, 256, 256, &total);
        if (rc) return rc;
        if (total == 0) return ASTRA_OK;
        if (total >= 128) return plan_only ? ASTRA_OK : launch_gemm_mlp(epi, true, batch, total, s);
        const int ns = epi == kEpiResidualF32 && p0.ldc % 4 == 0 ? gemm_split_factor(dtype, p0.M, p0.N, p0.K) : 1;
        if (ns > 1 && split_ws && split_ws_bytes >= (size_t)ns * p0.M * p0.N * sizeof(float)) {
            if (plan_only) return ASTRA_OK;
            batch.n_split = ns;
            batch.k_split = p0.K / ns;
            batch.p[0].c = split_ws;
            rc = launch_gemm_mlp(kEpiSplit, true, batch, total * ns, s);
            if (rc) return rc;
            return launch_split_reduce((const float*)split_ws, ns, p0, s);
        }
        rc = fill_batch(batch, dtype, problems, n_problems, 128, 128, &total);
        if (rc) return rc;
        if (plan_only) return ASTRA_OK;
        return launch_gemm_mlp(epi, false, batch, total, s);
    }
    // Large tiles quarter the operand traffic per flop; use them once they still fill most of the chip.  What is left after the choice above
    // are launches of many tiles, short contractions with large outputs, outputs that are no multiple of eight columns wide, and cuts into groups
    // whose codes do not fit the wavefront-private kernel's LDS.
    int rc = fill_batch(batch, dtype, problems, n_problems, 256, 256, &total);
    if (rc) return rc;
    bool big = total >= 128;
    // In between, 128 x 256 tiles: when they run as a single round of workgroups that fills more than half of the chip,
    // the launch lasts one such tile (about two thirds of a 256 x 256 one), where 256 x 256 tiles would leave half of
    // the units idle and 128 x 128 tiles would need a second workgroup per unit at a lower rate each.
    bool mid = false;
    if (total <= 128) {
        GemmBatch mb{};
        int mt = 0;
        rc = fill_batch(mb, dtype, problems, n_problems, 128, 256, &mt);
        if (rc) return rc;
        if (mt > kCus / 2 && mt <= kCus) {
            mid = true;
            big = false;
            batch = mb;
            total = mt;
        }
    }
    // Fuse the encode into the launch when the tiles leave a good part of the last round of compute units idle.
    if ((big || mid) && offered) {
        const int E = tile_encode_wgs(*enc, total, mid, k_max);
        if (E > 0) {
            batch.n_enc_wgs = E;
            batch.enc = *enc;
            batch.enc.tb = vq_encode_blocks(*enc, E);
            batch.enc.n_tb = (int)ceil_div(enc->n_tokens, 256 * batch.enc.tb);
            *enc_fused = true;
            if (plan_only) return ASTRA_OK;
            if (mid) {
                if (code16) gemm_nt_bf16_kernel<128, 256, 2, 4, true, true><<<total + E, 512, 0, s>>>(batch);
                else gemm_nt_bf16_kernel<128, 256, 2, 4, false, true><<<total + E, 512, 0, s>>>(batch);
            } else {
                if (code16) gemm_nt_bf16_kernel<256, 256, 2, 4, true, true><<<total + E, 512, 0, s>>>(batch);
                else gemm_nt_bf16_kernel<256, 256, 2, 4, false, true><<<total + E, 512, 0, s>>>(batch);
            }
            return launch_status();
        }
    }
    if (mid) {
        if (plan_only) return ASTRA_OK;
        if (code16) gemm_nt_bf16_kernel<128, 256, 2, 4, true><<<total, 512, 0, s>>>(batch);
        else gemm_nt_bf16_kernel<128, 256, 2, 4, false><<<total, 512, 0, s>>>(batch);
        return launch_status();
    }
    if (big) {
        if (total == 0 || plan_only) return ASTRA_OK;
        if (code16) gemm_nt_bf16_kernel<256, 256, 2, 4, true><<<total, 512, 0, s>>>(batch);
        else gemm_nt_bf16_kernel<256, 256, 2, 4, false><<<total, 512, 0, s>>>(batch);
        return launch_status();
    }
    rc = fill_batch(batch, dtype, problems, n_problems, 128, 128, &total);
    if (rc) return rc;
    if (total == 0) return ASTRA_OK;
    if (plan_only) return ASTRA_OK;
    if (code16) gemm_nt_bf16_kernel<128, 128, 4, 2, true><<<total, 512, 0, s>>>(batch);
    else gemm_nt_bf16_kernel<128, 128, 4, 2, false><<<total, 512, 0, s>>>(batch);
    return launch_status();
}

}  // namespace astra
