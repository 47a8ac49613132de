// Reading ahead: weights of the launches that follow, brought into the last-level cache by workgroups of a launch that leaves units idle.
#pragma once
#include "common.h"

namespace astra {

// A launch of a small model is a few microseconds of which its weights' way from memory is a good part, while the attention of such a model runs on a
// third of the units.  One byte of every 128-byte line is read; nothing is kept but the caches' contents.
// Passes over weights that come from memory (as those of a model or of models of more than 256 MB do), without / with (us): 12 GPT-2 blocks of 256 + 768 rows
// 660 / 620, of 64 + 192 529 / 490, 8 of 512 + 1024 560 / 530, 12 ViT blocks of 257 + 768 648 / 616; over weights that are in the cache anyway
// 589 / 585, 453 / 454, 504 / 503, 584 / 581.
struct Prefetch {
    static constexpr int kMax = 3;
    // 10.6 MB beside 24 or 96 workgroups of attention: one or two lines a thread, on 166 or 83 units, take the same (490 and 620 us), four on 42 units are
    // too slow beside 24 (517).  Beside 192, on all that is left, four lines 530, two (half of the weights) 545, one 557.
    static constexpr int kLines = 2, kMostLines = 4;
    const void* at[kMax];
    uint32_t lines[kMax];          // in the order in which they are needed
    int32_t n, n_wgs;

    void add(const void* p, size_t bytes) {
        if (!p || n == kMax || bytes < 128) return;
        at[n] = p;
        lines[n++] = (uint32_t)((bytes < ((size_t)1 << 31) ? bytes : (size_t)1 << 31) >> 7);
    }
    // for at most `wgs` workgroups of `threads`: kLines lines a thread, or up to kMostLines where there are too few of them
    Prefetch on(int wgs, int threads) const {
        Prefetch f = *this;
        int64_t left = wgs > 0 ? (int64_t)wgs * threads * kMostLines : 0, all = 0;
        for (int i = 0; i < n; ++i) {
            f.lines[i] = (uint32_t)(lines[i] < left ? lines[i] : left);
            left -= f.lines[i];
            all += f.lines[i];
        }
        const int64_t want = ceil_div(all, (int64_t)threads * kLines);
        f.n_wgs = (int)(want < wgs ? want : wgs > 0 ? wgs : 0);
        return f;
    }
};

// Workgroup idx of those that read ahead, in passes of kMostLines lines per thread
template <int THREADS>
__device__ __forceinline__ void prefetch_wgs(const Prefetch& f, uint32_t idx) {
    const uint32_t first = idx * THREADS + threadIdx.x, step = (uint32_t)f.n_wgs * THREADS;
    for (int k = 0; k < f.n; ++k) {
        const char* __restrict__ at = (const char*)f.at[k];
        const uint32_t lines = f.lines[k];
        for (uint32_t l = first; l < lines; l += Prefetch::kMostLines * step) {
            uint32_t got = 0;
#pragma unroll
            for (uint32_t u = 0; u < Prefetch::kMostLines; ++u) got ^= *reinterpret_cast<const uint8_t*>(at + (uint64_t)min(l + u * step, lines - 1) * 128u);
            asm volatile("" ::"v"(got));           // the loads are for the caches
        }
    }
}

}  // namespace astra
