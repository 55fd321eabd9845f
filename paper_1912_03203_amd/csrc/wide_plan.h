// wide_plan.h -- host-side plan of the channel-parallel patch kernel (wide.h):
// the cut of an image into patches, the kernel instantiation for a block, and
// its LDS.  Host code only, free of HIP, so that a CPU test can sweep it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "dynconv.h"

namespace dynconv {

constexpr int kWideWaves = 8;
constexpr int kWideThreads = kWideWaves * 64;
constexpr int kWideOwn = 64;                   // own positions of a patch: 4 tiles
constexpr int kWideSlots = 128;                // region slots of a patch: two ballot words
constexpr int kMaxWideC = 192;                 // the B fragments of x stay in registers
constexpr int kWideMaxCols = 40;               // Wu

// Patch geometry and the multipliers that replace the divisions by its sizes
// (div20).
struct WideGeom {
    int R, Wu, nph, npw;
    int slots;                 // (R + 2) * (Wu + 2)
    int tiles;                 // tiles of 16 needed slots that the kernel has to hold
    int m_wp, m_wu, m_pieces;  // by the region row, the own row and the 8-element pieces of an x row
};

inline int div20_mul(int d) { return ((1 << 20) + d - 1) / d; }

// The most positions of one patch whose expansion its depthwise reads: the
// patch and, where the image goes on, the ring around it.
inline int wide_need(const WideGeom &g) {
    return (g.R + std::min(g.nph - 1, 2)) * (g.Wu + std::min(g.npw - 1, 2));
}

// The cut into nph x npw patches with the least estimated time.  A patch costs
// a fixed part (staging, lists, the barriers and latencies of its chunks) plus
// its tiles of 16 needed and own positions; patches beyond one per compute unit
// queue up.  The search tries the 16 smallest numbers of columns and the 8
// smallest of rows; R = 0: none of them stays within max_patches and max_need.
inline WideGeom wide_geom_of(dynconv_shape s, int64_t max_patches, int max_need) {
    WideGeom best{};
    double best_cost = 0.0;
    const int w0 = (s.w + kWideMaxCols - 1) / kWideMaxCols;
    int last_wu = 0;
    for (int npw_t = w0; npw_t <= s.w && npw_t < w0 + 16; ++npw_t) {
        const int wu = (s.w + npw_t - 1) / npw_t;
        if (wu == last_wu) continue;
        last_wu = wu;
        const int npw = (s.w + wu - 1) / wu;
        const int rmax = std::min({s.h, kWideOwn / wu, kWideSlots / (wu + 2) - 2});
        if (rmax < 1) continue;
        int last_r = 0;
        const int h0 = (s.h + rmax - 1) / rmax;
        for (int nph_t = h0; nph_t <= s.h && nph_t < h0 + 8; ++nph_t) {
            const int r = (s.h + nph_t - 1) / nph_t;
            if (r == last_r) continue;
            last_r = r;
            WideGeom g{};
            g.R = r;
            g.Wu = wu;
            g.nph = (s.h + r - 1) / r;
            g.npw = npw;
            const int64_t patches = static_cast<int64_t>(s.n) * g.nph * npw;
            if (patches > max_patches) continue;
            const int need = wide_need(g);
            if (need > max_need) continue;
            const double load = std::max(1.0, static_cast<double>(patches) / 256.0);
            const double cost = load * (8 + (need + 15) / 16 + (r * wu + 15) / 16);
            if (best.R == 0 || cost < best_cost - 1e-9) {
                best_cost = cost;
                best = g;
            }
        }
    }
    if (best.R == 0) return best;
    best.slots = (best.R + 2) * (best.Wu + 2);
    best.m_wp = div20_mul(best.Wu + 2);
    best.m_wu = div20_mul(best.Wu);
    return best;
}

// The x fragments of 8 needed tiles (128 positions) fit the registers up to 96
// channels.  Above that the patches are kept to 4 tiles; up to 128 channels
// there is a form with 8 tiles and smaller chunks for the maps on which the
// search finds no such cut (from about 100 positions a side, or wide strips).
// Above 128 channels no form holds 8 tiles, and such maps get no cut (R = 0).
inline WideGeom wide_geom(dynconv_shape s, int64_t max_patches) {
    WideGeom g = wide_geom_of(s, max_patches, s.c <= 96 ? 128 : 64);
    if (g.R == 0 && s.c > 96 && s.c <= 128) g = wide_geom_of(s, max_patches, 128);
    if (g.R == 0) return g;
    const int need = wide_need(g);
    g.tiles = need <= 32 ? 2 : need <= 64 ? 4 : 8;
    return g;
}

// A kernel instantiation: steps of 32 input channels, hidden channels per
// chunk, tiles of 16 needed positions held, whether one chunk is all there is.
struct WideForm {
    int ks, ec, nt;
    bool one;
};
#define DC_WIDE_FORMS_32(X) X(1, 64, 4, false) X(1, 64, 8, false) X(2, 64, 4, false) X(2, 64, 8, false)
#define DC_WIDE_FORMS_16(X)                                                                            \
    X(1, 128, 8, false) X(2, 64, 8, true) X(2, 128, 8, true) X(2, 128, 4, false) X(2, 128, 8, false)   \
    X(3, 128, 4, false) X(3, 128, 8, false) X(4, 128, 4, true) X(4, 128, 4, false) X(4, 64, 8, false)  \
    X(5, 128, 2, false) X(5, 64, 4, false) X(6, 64, 4, false)

// The instantiation for the element size, the channels, the hidden width and
// the patches' needed tiles.  128 hidden channels per chunk halve the barriers
// and load each weight once per workgroup; 64 where the registers or (fp32) the
// LDS don't hold 128, and where 64 are all there are.
inline WideForm wide_form(size_t elem, int c, int e, int tiles) {
    const bool t8 = tiles == 8;
    if (elem == 4) return {c <= 32 ? 1 : 2, 64, t8 ? 8 : 4, false};
    if (c <= 32) return {1, 128, 8, false};
    if (c <= 64) return e <= 64 ? WideForm{2, 64, 8, true} : e <= 128 ? WideForm{2, 128, 8, true}
                                                                      : WideForm{2, 128, t8 ? 8 : 4, false};
    if (c <= 96) return {3, 128, t8 ? 8 : 4, false};
    if (c <= 128) return t8 ? WideForm{4, 64, 8, false} : WideForm{4, 128, 4, e <= 128};
    if (c <= 160) return tiles == 2 ? WideForm{5, 128, 2, false} : WideForm{5, 64, 4, false};
    return {6, 64, 4, false};
}

// Dynamic LDS of a form at C channels: rows of EC + 8 hidden channels.
inline size_t wide_lds_bytes(size_t elem, const WideForm &f, int C, int slots) {
    const size_t nbuf = f.one ? 1 : 2, row = static_cast<size_t>(f.ec) + 8;
    return 256 /* words */ + 2 * (kWideSlots + kWideOwn)              // lists
           + nbuf * (9 * static_cast<size_t>(f.ec) * elem + 4 * f.ec)  // depthwise weights, biases
           + static_cast<size_t>(slots) * (C + 8) * elem               // x
           + nbuf * static_cast<size_t>(slots + 1) * row * elem        // H1
           + nbuf * static_cast<size_t>(kWideOwn) * row * elem;        // H2
}

// The hidden channels of a stack's blocks and their chunks of 128.
struct WideWork {
    int64_t blocks, hidden, chunks;
    int most;  // the widest block's
    void add(int e) {
        ++blocks;
        hidden += e;
        chunks += (e + 127) / 128;
        most = std::max(most, e);
    }
};

// Up to how many patches of its own a stack that k_block_fused also runs (up to
// 64 channels, fp32 32) takes the channel-parallel kernel: the larger patches of
// k_block_fused amortise their fixed part better once a compute unit has many.
// The time goes in rounds of 256 patches (one workgroup per compute unit) by
// chunks of 128 hidden channels, that of k_block_fused in rounds of 512 patches by
// slices of 32, so the line depends on how full the chunks are.  Measured per
// block, k_block_fused / this kernel, us, fp16 or bf16 unless noted:
//   one chunk, 64 channels: hidden 64, 64 x 28x28 (896 patches) 14.0 / 12.6 dense,
//     64 x 56x56 47.7 / 32.1: no line
//   full chunks (over 0.9), 64 channels: hidden 384, 128 x 14x14 (512 patches) dense
//     31 / 23, 192 x 14x14 (768) 36 / 34, 64 x 28x28 (896) 35 / 46 and at 0.2 active
//     36 / 39; hidden 256, 128 x 14x14 23 / 19, 96 x 17x20 (576) dense 26 / 29, at
//     0.2 26 / 24
//   0.7 to 0.9: 48 channels, hidden 288, dense: 128 x 14x14 24 / 23, 96 x 17x20 27 / 34
//   below: 40 channels, hidden 160, dense: 64 x 14x14 (256) 15 / 11, 24 x 28x28 (336)
//     16 / 20
//   up to 32 channels, fp32: 1 x 32x32x32 (128 patches) 17.1 / 11.2, 16 x 48x48x32
//     (576) 30 / 39
// A map that k_block_fused cuts into more than 512 patches costs it a second
// round, which moves the line to twice as many, and to 1,024 at most: bf16
// 80 x 26x26 (960 patches, 560 of k_block_fused) at 0.5 active and dense: 64
// channels, hidden 384 65 / 52 and 65 / 55, hidden 256 49 / 42 and 48 / 43; 40
// channels, hidden 240 47 / 40 and 47 / 42, hidden 160 (line 512) 35 / 39 and 34 / 39.
// Wider blocks have no other one-launch kernel (64 x 14x14x96 42 / 17.5, when
// k_block_fused took up to 128 channels; fp32 16 x 48x48x64 144 / 91).
inline int64_t wide_most_patches(int c, const WideWork &w, bool dense, int64_t fused_patches) {
    if (c <= 32) return 256;
    if (w.most <= 128) return INT64_MAX;
    const double fill = static_cast<double>(w.hidden) / static_cast<double>(std::max<int64_t>(w.chunks, 1) * 128);
    const int64_t most = fill > 0.9 ? (dense && w.hidden < 384 * w.blocks ? 512 : 768) : fill > 0.7 ? 512 : 256;
    return fused_patches > 512 ? std::min<int64_t>(2 * most, 1024) : most;
}

}  // namespace dynconv
