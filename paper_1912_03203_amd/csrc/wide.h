// wide.h -- one-launch gated block on small patches, channel-parallel (gfx950).
//
// k_block_wide runs a whole spatially gated block (Sec. 3.2) for one patch of
// at most 64 positions per workgroup of 8 waves, with the arithmetic and the
// summation orders of k_block_fused and of the kernel chain:
//   1. x of the patch's region (the patch and a one-position ring) goes to
//      LDS; the hard mask of the region (read, or computed from the staged x)
//      becomes two ballot words; active set, needed set (the in-image slots
//      next to an active one) and their raster-ordered lists follow by shifts
//      and popcount ranks;
//   2. the hidden channels pass in chunks of EC.  A wave owns a 16-channel
//      tile of the chunk's expansion (its x fragments stay in registers for
//      all chunks), a 32-channel slice of the depthwise on position tiles of
//      16 active positions, and output tiles of the projection.  Weights of
//      the products go straight from the L2 to registers, requested a chunk
//      ahead; only the depthwise's few go through LDS.  H1 and H2 are double
//      buffered, so that one interval holds the depthwise of chunk s, the
//      projection of chunk s - 1 and the expansion of chunk s + 1, with one
//      barrier;
//   3. y = x + F at the active positions in the staged rows, a coalesced
//      store, and the next block's mask unit on the stored values.
//
// Why: at MobileNetV2's 64- to 160-channel maps there is about one patch per
// compute unit, so the time is one patch's chain of latencies.  k_block_fused
// pays two barriers and an LDS round trip of all weights per 32 channels with
// one wave per SIMD; the kernel chain pays six launches.  Per-phase clocks of
// 64 x 14x14x96, hidden 576, fp16, density 0.4 (256 patches of 7 x 7, k cycles):
// 8.4 to the first expansion, 5 intervals of 3.5, 3 for the epilogue.  An
// interval is bound by the weights' way through the L1 (48 KB at 64 B per
// clock) and the two waves per SIMD that share the depthwise's vector issue.
// Measured per block: 17.5 us (k_block_fused 42); 64 x 7x7x160, hidden 960:
// 24 us (kernel chain 75); a ShuffleNetV2 unit, batch 64, bf16: 28x28x116 18 us
// (25), 14x14x232 14 us (27).
#pragma once

#include "fused.h"
#include "kernels.h"
#include "wide_plan.h"

namespace dynconv {

// i / d == (i * m) >> 20 for i * d < 2^20, m = div20_mul(d).
__device__ __forceinline__ int div20(int i, int m) {
    return static_cast<int>((static_cast<unsigned>(i) * static_cast<unsigned>(m)) >> 20);
}

// One bit per region slot, the same in every lane.
template <int NW> struct Bits {
    uint64_t w[NW];
    __device__ __forceinline__ Bits operator|(const Bits &o) const {
        Bits v;
#pragma unroll
        for (int i = 0; i < NW; ++i) v.w[i] = w[i] | o.w[i];
        return v;
    }
    __device__ __forceinline__ Bits operator&(const Bits &o) const {
        Bits v;
#pragma unroll
        for (int i = 0; i < NW; ++i) v.w[i] = w[i] & o.w[i];
        return v;
    }
    // 1 <= k <= 63
    __device__ __forceinline__ Bits up(int k) const {
        Bits v;
#pragma unroll
        for (int i = 0; i < NW; ++i) v.w[i] = (w[i] << k) | (i ? w[i - 1] >> (64 - k) : 0ull);
        return v;
    }
    __device__ __forceinline__ Bits down(int k) const {
        Bits v;
#pragma unroll
        for (int i = 0; i < NW; ++i) v.w[i] = (w[i] >> k) | (i + 1 < NW ? w[i + 1] << (64 - k) : 0ull);
        return v;
    }
    // the slots next to a set one, itself included (rows of wp slots)
    __device__ __forceinline__ Bits dilate(int wp) const {
        const Bits v = *this | up(wp) | down(wp);
        return v | v.up(1) | v.down(1);
    }
    __device__ __forceinline__ int count() const {
        int c = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) c += __popcll(w[i]);
        return c;
    }
};
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

template <typename T>
__device__ __forceinline__ void store8(T *p, const float v[8]) {
    *reinterpret_cast<typename mma<T>::frag *>(p) = mma<T>::pack(v);
}
template <>
__device__ __forceinline__ void store8<float>(float *p, const float v[8]) {
    io<float>::store4(p, v);
    io<float>::store4(p + 4, v + 4);
}
template <typename T>
__device__ __forceinline__ void store8(T *p, const typename io<T>::vec8 &v) {
    *reinterpret_cast<typename io<T>::vec8 *>(p) = v;
}
template <>
__device__ __forceinline__ void store8<float>(float *p, const io<float>::vec8 &v) {
    store8(p, v.v);
}

// 8 channels of a half row of a ShuffleNetV2 unit (4-byte aligned), `left` of
// them inside the half (whole 4-byte words); the others come out as zeros and
// are not read.
template <typename T>
__device__ __forceinline__ typename io<T>::vec8 half_piece(const T *base, uint32_t off, int left) {
    typedef typename io<T>::vec8 V;
    if constexpr (sizeof(T) == 4) {
        V r;
        const T *f = base + off;
#pragma unroll
        for (int u = 0; u < 8; ++u) r.v[u] = u < left ? f[u] : 0.0f;
        return r;
    } else {
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        struct __attribute__((packed, aligned(4))) piece {
            u4 v;
        };
        const char *p = reinterpret_cast<const char *>(base) + static_cast<uint32_t>(off * sizeof(T));
        if (left >= 8) return __builtin_bit_cast(V, reinterpret_cast<const piece *>(p)->v);
        const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
        u4 v = {0u, 0u, 0u, 0u};
        if (left >= 2) v[0] = q[0];
        if (left >= 4) v[1] = q[1];
        if (left >= 6) v[2] = q[2];
        return __builtin_bit_cast(V, v);
    }
}

// (a[k], b[k]) pairs of the first min(left, 8) channels, 8-byte aligned.
template <typename T>
__device__ __forceinline__ void store_pairs(T *dst, typename io<T>::vec8 a, typename io<T>::vec8 b, int left) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < left) *reinterpret_cast<float2 *>(dst + 2 * k) = make_float2(a[k], b[k]);
        return;
    }
    typedef T quad_t __attribute__((ext_vector_type(4)));
    quad_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k][0] = a[2 * k];
        v[k][1] = b[2 * k];
        v[k][2] = a[2 * k + 1];
        v[k][3] = b[2 * k + 1];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (2 * k < left) *reinterpret_cast<quad_t *>(dst + 4 * k) = v[k];
}

// Barrier for data in LDS: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Element `off` (32 bits) past a uniform base: one address register per lane.
template <typename V, typename T>
__device__ __forceinline__ V ld_at(const T *base, uint32_t off) {
    return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + static_cast<uint32_t>(off * sizeof(T)));
}
// the 8 elements there
template <typename T>
__device__ __forceinline__ typename io<T>::vec8 ld8_at(const T *base, uint32_t off) {
    return io<T>::raw8(reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + static_cast<uint32_t>(off * sizeof(T))));
}
template <typename T>
__device__ __forceinline__ typename mma<T>::frag ldf_at(const T *base, uint32_t off) {
    return mma<T>::load(reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + static_cast<uint32_t>(off * sizeof(T))));
}

// The mask unit (Eq. 2, Eq. 8 at zero noise) on a row staged in LDS: the fp32
// multiply-add chain of k_mask, channels ascending from +0, then the bias,
// strict threshold.  32 channels at a time: their loads overlap.
template <typename T>
__device__ __forceinline__ bool mask_of_row(const T *row, int C, const float *wm, float bm, int mode) {
    typedef const __attribute__((address_space(4))) float *cfptr;
    cfptr w = (cfptr)(wm);
    float a = 0.0f;
    for (int c0 = 0; c0 + 32 <= C; c0 += 32) {
        typename io<T>::vec8 v[4];
        float wc[32];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = io<T>::raw8(row + c0 + 8 * q);
#pragma unroll
        for (int u = 0; u < 32; ++u) wc[u] = w[c0 + u];
#pragma unroll
        for (int u = 0; u < 32; ++u) a = __builtin_fmaf(wc[u], static_cast<float>(v[u / 8][u % 8]), a);
    }
    for (int c0 = C & ~31; c0 < C; c0 += 8) {
        const typename io<T>::vec8 v = io<T>::raw8(row + c0);
#pragma unroll
        for (int u = 0; u < 8; ++u) a = __builtin_fmaf(w[c0 + u], static_cast<float>(v[u]), a);
    }
    return mask_decision(a + bm, mode);
}

template <typename T, bool DENSE, int KS, bool SHUF, int EC, int NT, bool ONE>
__global__ void __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(EC == 64 && KS == 2 && sizeof(T) == 2 ? 4 : 2)))
k_block_wide(const T *__restrict__ xin, T *__restrict__ yout, int N, int H, int W, int C, int E, WideGeom G,
             int cb, const uint8_t *__restrict__ mask_in, const float *__restrict__ wm_self, float bm_self,
             uint8_t *__restrict__ mask_self, const T *__restrict__ w1, const float *__restrict__ b1, int act1,
             const T *__restrict__ w2, const float *__restrict__ b2, int act2, const T *__restrict__ w3,
             const float *__restrict__ b3, int act3, const float *__restrict__ wm_next, float bm_next,
             uint8_t *__restrict__ mask_next, uint16_t *__restrict__ band_counts, int mask_mode) {
    typedef mma<T> M;
    typedef typename M::frag Frag;
    typedef typename io<T>::vec8 V;
    constexpr int TP = kWideOwn / 16, NWD = kWideSlots / 64;
    constexpr int kPitch = EC + 8;
    constexpr int MW = EC / 16, SH = kWideWaves / MW;  // hidden tiles of a chunk, waves per hidden tile
    constexpr int TW = NT / SH;                        // needed tiles per wave
    constexpr int KP = EC / 32;                        // 32-channel slices of a chunk
    constexpr int DS = kWideWaves / KP;                // position tiles of the depthwise at a time
    constexpr int MS = kWideWaves / SH;                // output tiles at a time
    constexpr int JM = (2 * KS + MS - 1) / MS;         // output tiles per wave
    constexpr int NP = TP / SH;                        // position tiles per wave in the projection
    constexpr int TS = (9 * EC + kWideThreads - 1) / kWideThreads;  // staged depthwise weights per thread
    static_assert(TW % 2 == 0 && NP % 2 == 0, "tiles are taken in pairs");
    extern __shared__ __align__(16) unsigned char wd_lds[];
    uint64_t *words = reinterpret_cast<uint64_t *>(wd_lds);  // [3][NWD]: mask, own, in-image
    int16_t *need = reinterpret_cast<int16_t *>(wd_lds + 256);
    int16_t *act = need + kWideSlots;
    const int XP = C + 8;
    const int nbuf = ONE ? 1 : 2;
    T *w2t = reinterpret_cast<T *>(act + kWideOwn);                    // [nbuf][9][EC]
    float *b2s = reinterpret_cast<float *>(w2t + nbuf * 9 * EC);   // [nbuf][EC]
    T *xs = reinterpret_cast<T *>(b2s + nbuf * EC);
    T *h1s = xs + G.slots * XP;
    const int h1_elems = (G.slots + 1) * kPitch;
    constexpr int h2_elems = kWideOwn * kPitch;
    T *h2s = h1s + nbuf * h1_elems;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    const int r = lane % 16, g = lane / 16;
    const int npatch = N * G.nph * G.npw;
    // XCD-aware: workgroup i runs on XCD i % 8, so consecutive patches
    // (which share ring rows and columns) go to the same XCD.
    const int per_xcd = (npatch + 7) / 8;
    const int bid = block_xy();
    const int patch = (bid % 8) * per_xcd + bid / 8;
    if (bid / 8 >= per_xcd || patch >= npatch) return;  // uniform per workgroup
    const int pimg = G.nph * G.npw;
    const int n = patch / pimg, prem = patch - n * pimg;
    const int pr = prem / G.npw;
    const int h0 = pr * G.R, w0 = (prem - pr * G.npw) * G.Wu;
    const int rows_out = min(G.R, H - h0), cols_out = min(G.Wu, W - w0);
    const int WP = G.Wu + 2;
    const int nslots = G.slots;
    const int nchunks = ONE ? 1 : (E + EC - 1) / EC;
    // in-image region rows and columns
    const int r_lo = h0 == 0 ? 1 : 0, c_lo = w0 == 0 ? 1 : 0;
    const unsigned r_n = min(G.R + 2, H - h0 + 1) - r_lo, c_n = min(WP, W - w0 + 1) - c_lo;
    // the region's first position (may lie before the tensor: only in-image
    // positions are accessed), and 32-bit offsets from there
    const int64_t pos0 = (static_cast<int64_t>(n) * H + h0 - 1) * W + (w0 - 1);
    const int CX = SHUF ? 2 * cb : C;
    const T *xb = xin + pos0 * CX;
    T *yb = yout + pos0 * CX;
    const uint8_t *mb = mask_in + pos0;
    const float lo1 = act_lo(act1), hi1 = act_hi(act1);
    const float lo2 = act_lo(act2), hi2 = act_hi(act2);
    const float lo3 = act_lo(act3), hi3 = act_hi(act3);

    // this thread's region slot (threads 0 .. kWideSlots - 1)
    const int srow = div20(tid, G.m_wp), scol = tid - srow * WP;
    const bool s_img = tid < nslots && static_cast<unsigned>(srow - r_lo) < r_n && static_cast<unsigned>(scol - c_lo) < c_n;
    const bool s_own = s_img && static_cast<unsigned>(srow - 1) < static_cast<unsigned>(rows_out) &&
                       static_cast<unsigned>(scol - 1) < static_cast<unsigned>(cols_out);
    uint8_t mbyte = 0;
    if (!DENSE && !wm_self && s_img) mbyte = mb[static_cast<uint32_t>(srow * W + scol)];

    // ---- x of the region: 8-element pieces of the in-image positions
    const int pieces = C / 8;
    const int total = nslots * pieces;
    constexpr int kB = SHUF ? 2 : 4;
    for (int i0 = tid; i0 < total; i0 += kB * kWideThreads) {
        V v[kB];
        int d[kB];
#pragma unroll
        for (int q = 0; q < kB; ++q) {
            const int i = i0 + q * kWideThreads;
            const int slot = div20(i, G.m_pieces), pc = i - slot * pieces;
            const int rr = div20(slot, G.m_wp), cc = slot - rr * WP;
            const bool in = i < total && static_cast<unsigned>(rr - r_lo) < r_n && static_cast<unsigned>(cc - c_lo) < c_n;
            d[q] = in ? slot * XP + pc * 8 : -1;
            if (in) {
                const uint32_t off = (rr * W + cc) * CX + pc * 8;
                if (!SHUF) v[q] = ld8_at(xb, off);
                else v[q] = half_piece(xb + cb, off, cb - pc * 8);
            }
        }
#pragma unroll
        for (int q = 0; q < kB; ++q)
            if (d[q] >= 0) store8(xs + d[q], v[q]);
    }
    // weights of the matrix products, requested an interval ahead: the
    // expansion's hidden tile m of a chunk and the projection's output tiles
    // mt0 + MS j.  Channels past C: their x fragments are zero, and so
    // are these (c_tail).  Output rows past C read row 0 and are not stored.
    const int m = wave % MW, half = wave / MW;
    const int phalf = wave % SH, mt0 = wave / SH;
    const bool c_tail = C != KS * 32;
    const bool last_in = (KS - 1) * 32 + 8 * g < C;
    const uint32_t a1_off = (m * 16 + r) * C + 8 * g;
    const uint32_t a1_last = (m * 16 + r) * C + (last_in ? (KS - 1) * 32 + 8 * g : 0);
    const uint32_t b1_off = m * 16 + 4 * g;
    uint32_t a3_off[JM];
#pragma unroll
    for (int j = 0; j < JM; ++j) {
        const int c = (mt0 + MS * j) * 16 + r;
        a3_off[j] = (c < C ? c : 0) * E;
    }
    Frag a1[KS], a3[JM][KP];
    floatx4 bi1 = {0.0f, 0.0f, 0.0f, 0.0f};
    // No branch around these loads: what is in flight is then known at every
    // wait.  Past the last chunk or channel they read valid weights again,
    // which expand and project don't use.
    auto load_a1 = [&](int ch) {
        const int ea = min(ch * EC, E - 16 - m * 16);  // so that tile m ends within E
        const T *wb = w1 + ea * C;
#pragma unroll
        for (int ks = 0; ks + 1 < KS; ++ks) a1[ks] = ldf_at(wb, a1_off + ks * 32);
        a1[KS - 1] = ldf_at(wb, a1_last);
        bi1 = ld_at<floatx4>(b1 + ea, b1_off);
    };
    auto load_a3 = [&](int ch) {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int e = min(ch * EC + 32 * k + 8 * g, E - 8);
#pragma unroll
            for (int j = 0; j < JM; ++j) a3[j][k] = ldf_at(w3, a3_off[j] + e);
        }
    };
    // depthwise weights of a chunk: requested an interval before they go to
    // LDS (transposed), an interval before their use
    T w2v[TS];
    float b2v;
    auto load_w2 = [&](int ch) {
        const T *wb = w2 + ch * (EC * 9);
        const int n = (E - ch * EC) * 9 - 1;  // past E: the last weight again, never used
#pragma unroll
        for (int q = 0; q < TS; ++q) w2v[q] = ld_at<T>(wb, min(tid + q * kWideThreads, n));
        b2v = ld_at<float>(b2, min(ch * EC + tid, E - 1));
    };
    auto store_w2 = [&](int ch) {
        T *wt = w2t + (ch & 1) * (9 * EC);
#pragma unroll
        for (int q = 0; q < TS; ++q) {
            const int j = tid + q * kWideThreads;
            const int e = div20(j, (1 << 20) / 9 + 1), k = j - 9 * e;
            if (j < 9 * EC) wt[k * EC + e] = w2v[q];
        }
        if (tid < EC) b2s[(ch & 1) * EC + tid] = b2v;
    };
    load_w2(0);
    load_a1(0);
    load_a3(0);
    // projection bias
    floatx4 acc[JM][NP];
#pragma unroll
    for (int j = 0; j < JM; ++j) {
        const int c0 = (mt0 + MS * j) * 16 + 4 * g;
        acc[j][0] = ld_at<floatx4>(b3, c0 < C ? c0 : 0);
    }
    // the pass-through half of this thread's output pieces (SHUF)
    constexpr int XO = SHUF ? (kWideOwn * 4 * KS + kWideThreads - 1) / kWideThreads : 1;
    V x1v[XO];
    if (SHUF) {
#pragma unroll
        for (int q = 0; q < XO; ++q) {
            const int i = tid + q * kWideThreads;
            const int p = div20(i, G.m_pieces), pc = i - p * pieces;
            const int rr = div20(p, G.m_wu), cc = p - rr * G.Wu;
            if (rr < rows_out && cc < cols_out && pc * 8 < cb)
                x1v[q] = half_piece(xb, ((rr + 1) * W + cc + 1) * CX + pc * 8, cb - pc * 8);
        }
    }
    // zero regions: slots outside the image are never written again
    if (static_cast<int>(r_n) < G.R + 2 || static_cast<int>(c_n) < WP) {
        uint4 *z = reinterpret_cast<uint4 *>(h1s);
        const int nz = nbuf * h1_elems * static_cast<int>(sizeof(T)) / 16;
        for (int i = tid; i < nz; i += kWideThreads) z[i] = make_uint4(0, 0, 0, 0);
    }
    // ---- mask words, dilation, lists
    bool bit = DENSE ? s_img : mbyte != 0;
    if (!DENSE && wm_self) {
        lds_barrier();  // the region's x, for the block's own mask unit
        if (s_img) {
            bit = mask_of_row<T>(xs + tid * XP, C, wm_self, bm_self, mask_mode);
            if (mask_self && s_own) (mask_self + pos0)[static_cast<uint32_t>(srow * W + scol)] = bit ? 1 : 0;
        }
    }
    if (wave < NWD) {
        const uint64_t bg = __ballot(bit), bo = __ballot(s_own), bi = __ballot(s_img);
        if (lane == 0) {
            words[wave] = bg;
            words[NWD + wave] = bo;
            words[2 * NWD + wave] = bi;
        }
    }
    store_w2(0);
    lds_barrier();
    Bits<NWD> mg, mo, mi;
#pragma unroll
    for (int i = 0; i < NWD; ++i) {
        mg.w[i] = uniform64(words[i]);
        mo.w[i] = uniform64(words[NWD + i]);
        mi.w[i] = uniform64(words[2 * NWD + i]);
    }
    const Bits<NWD> ma = mg & mo, mn = ma.dilate(WP) & mi;
    const int n_act = ma.count(), n_need = mn.count();
    if (!DENSE && band_counts && tid == 0)
        band_counts[patch] = static_cast<uint16_t>(n_act | ((mg.dilate(WP) & mo).count() << 8));
#pragma unroll
    for (int i = 0, bn = 0, ba = 0; i < NWD; ++i) {
        if (wave == i) {
            const uint64_t lt = lanemask_lt(lane);
            if ((mn.w[i] >> lane) & 1ull) need[bn + __popcll(mn.w[i] & lt)] = static_cast<int16_t>(tid);
            if ((ma.w[i] >> lane) & 1ull) act[ba + __popcll(ma.w[i] & lt)] = static_cast<int16_t>(tid);
        }
        bn += __popcll(mn.w[i]);
        ba += __popcll(ma.w[i]);
    }
    lds_barrier();

    if (n_act > 0) {
        // expansion: every SH-th tile of 16 needed slots, whose B fragments
        // stay in registers
        int nq[TW];
        Frag bx[TW][KS];
#pragma unroll
        for (int j = 0; j < TW; ++j) {
            const int i = (half + SH * j) * 16 + r;
            const int q = (i < n_need) ? static_cast<int>(need[i]) : -1;
            nq[j] = ((q >= 0) ? q : nslots) * kPitch + m * 16 + 4 * g;  // past the list: the spare row
            const T *row = xs + ((q >= 0) ? q : WP + 1) * XP + 8 * g;  // else an own slot; its column is never read
#pragma unroll
            for (int ks = 0; ks + 1 < KS; ++ks) bx[j][ks] = M::load(row + ks * 32);
            bx[j][KS - 1] = last_in ? M::load(row + (KS - 1) * 32) : M::zero();
        }
        // depthwise: slice wave % KP of a chunk, position tiles wave / KP + DS i;
        // lane (r, g): position r of the tile, channels 8 g .. 8 g + 7 of the slice
        const int dsl = wave % KP, dt0 = wave / KP;
        int aq[TP / DS];
#pragma unroll
        for (int i = 0; i < TP / DS; ++i) {
            const int p = (dt0 + DS * i) * 16 + r;
            aq[i] = ((p < n_act) ? static_cast<int>(act[p]) : WP + 1) * kPitch + 32 * dsl + 8 * g;
        }
        const int row_e = WP * kPitch;
        // projection: position tiles phalf + SH p
#pragma unroll
        for (int j = 0; j < JM; ++j)
#pragma unroll
            for (int p = 1; p < NP; ++p) acc[j][p] = acc[j][0];
        // interval s: depthwise of chunk s, projection of chunk s - 1,
        // expansion of chunk s + 1; one barrier per interval
        auto expand = [&](int ch) {
            if (ch * EC + m * 16 >= E) return;
            T *hb = h1s + (ch & 1) * h1_elems;
            if (c_tail && !last_in) a1[KS - 1] = M::zero();
#pragma unroll
            for (int jp = 0; jp < TW; jp += 2) {
                if ((half + SH * jp) * 16 < n_need) {
                    floatx4 d[2] = {bi1, bi1};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int j = 0; j < 2; ++j) d[j] = M::run(a1[ks], bx[jp + j][ks], d[j]);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        float o[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) o[v] = clamp_act(d[j][v], lo1, hi1);
                        io<T>::store4(hb + nq[jp + j], o);
                    }
                }
            }
        };
        auto project = [&](int ch) {
            if (phalf * 16 >= n_act) return;
            if ((ch + 1) * EC > E) {  // the last chunk of a hidden width that is no multiple of 64
#pragma unroll
                for (int k = 0; k < KP; ++k)
                    if (ch * EC + 32 * k + 8 * g >= E)
#pragma unroll
                        for (int j = 0; j < JM; ++j) a3[j][k] = M::zero();
            }
            const T *hb = h2s + (ch & 1) * h2_elems + r * kPitch + 8 * g;
            // two position tiles at a time, skipped past the active list
#pragma unroll
            for (int pp = 0; pp < NP; pp += 2) {
                if ((phalf + SH * pp) * 16 < n_act) {
                    Frag bf[2][KP];
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int k = 0; k < KP; ++k)
                            bf[p][k] = M::load(hb + (phalf + SH * (pp + p)) * 16 * kPitch + 32 * k);
#pragma unroll
                    for (int k = 0; k < KP; ++k)
#pragma unroll
                        for (int j = 0; j < JM; ++j)
#pragma unroll
                            for (int p = 0; p < 2; ++p) acc[j][pp + p] = M::run(a3[j][k], bf[p][k], acc[j][pp + p]);
                }
            }
        };
        auto depthwise = [&](int ch) {
            const int cg = 32 * dsl + 8 * g;  // within the chunk
            // past E: zeros, by clamping to [0, 0]
            const bool ein = ch * EC + cg < E;
            const float lo = ein ? lo2 : 0.0f, hi = ein ? hi2 : 0.0f;
            const T *wt = w2t + (ch & 1) * (9 * EC) + cg;
            const float *bs = b2s + (ch & 1) * EC + cg;
            const T *hb = h1s + (ch & 1) * h1_elems;
            T *db = h2s + (ch & 1) * h2_elems + r * kPitch + cg;
#pragma unroll
            for (int i = 0; i < TP / DS; ++i) {
                if ((dt0 + DS * i) * 16 < n_act) {
                    const T *own = hb + aq[i];
                    __asm__ volatile("" ::: "memory");  // the weights are read again per tile
                    float sum[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) sum[u] = bs[u];
                    // a kernel row of taps and weights at a time, the next row in flight
                    V tv[2][3], wv[2][3];
                    auto load_row = [&](int kr) {
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            tv[kr & 1][q] = io<T>::raw8(own + (kr - 1) * row_e + (q - 1) * kPitch);
                            wv[kr & 1][q] = io<T>::raw8(wt + (3 * kr + q) * EC);
                        }
                    };
                    constexpr bool kAhead = EC > 64;  // registers for two rows
                    if constexpr (kAhead) load_row(0);
#pragma unroll
                    for (int kr = 0; kr < 3; ++kr) {
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (!kAhead) load_row(kr);
                        else if (kr < 2) load_row(kr + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int q = 0; q < 3; ++q)
#pragma unroll
                            for (int u = 0; u < 8; ++u)
                                sum[u] = __builtin_fmaf(static_cast<float>(wv[kr & 1][q][u]),
                                                        static_cast<float>(tv[kr & 1][q][u]), sum[u]);
                    }
                    float hv[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) hv[u] = clamp_act(sum[u], lo, hi);
                    store8(db + (dt0 + DS * i) * 16 * kPitch, hv);
                }
            }
        };
        expand(0);
        if constexpr (!ONE) {
            load_a1(1);
            load_w2(min(1, nchunks - 1));
        }
        lds_barrier();
        if constexpr (ONE) {
            depthwise(0);
            lds_barrier();
        } else {
            for (int s = 0; s < nchunks; ++s) {
                // each product's next weights are requested behind it; the
                // four waves of each half start at different ends, so that a
                // SIMD's two waves use the matrix cores and the VALU in turn
                if (wave < 4) depthwise(s);
                if (s + 1 < nchunks) expand(s + 1);
                load_a1(s + 2);
                store_w2(s + 1);
                load_w2(min(s + 2, nchunks - 1));
                __builtin_amdgcn_sched_barrier(0);
                if (s >= 1) project(s - 1);
                load_a3(s);
                __builtin_amdgcn_sched_barrier(0);
                if (wave >= 4) depthwise(s);
                lds_barrier();
            }
        }
        project(nchunks - 1);
        // ---- residual sum at the active positions, in place in xs
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = (phalf + SH * p) * 16 + r;
            if (i < n_act) {
                T *row = xs + static_cast<int>(act[i]) * XP;
#pragma unroll
                for (int j = 0; j < JM; ++j) {
                    const int c0 = (mt0 + MS * j) * 16 + 4 * g;
                    if (c0 < C) {
                        float xv[4], o[4];
                        io<T>::load4(row + c0, xv);
#pragma unroll
                        for (int v = 0; v < 4; ++v) o[v] = xv[v] + clamp_act(acc[j][p][v], lo3, hi3);
                        io<T>::store4(row + c0, o);
                    }
                }
            }
        }
        lds_barrier();
    }
    // ---- store the patch (inactive positions: x unchanged); items are the
    // 8-element pieces of the own positions
    const int own_total = G.R * G.Wu * pieces;
    if (SHUF) {
        // output rows: (first input half, block output) interleaved
#pragma unroll
        for (int q = 0; q < XO; ++q) {
            const int i = tid + q * kWideThreads;
            const int p = div20(i, G.m_pieces), pc = i - p * pieces;
            const int rr = div20(p, G.m_wu), cc = p - rr * G.Wu;
            const int left = cb - pc * 8;  // channels of this piece and beyond
            if (i < own_total && rr < rows_out && cc < cols_out && left > 0)
                store_pairs(yb + static_cast<uint32_t>(((rr + 1) * W + cc + 1) * CX + 2 * pc * 8), x1v[q],
                            io<T>::raw8(xs + ((rr + 1) * WP + cc + 1) * XP + pc * 8), left);
        }
    } else {
        for (int i = tid; i < own_total; i += kWideThreads) {
            const int p = div20(i, G.m_pieces), pc = i - p * pieces;
            const int rr = div20(p, G.m_wu), cc = p - rr * G.Wu;
            if (rr < rows_out && cc < cols_out)
                store8(reinterpret_cast<T *>(reinterpret_cast<char *>(yb) +
                                             static_cast<uint32_t>((((rr + 1) * W + cc + 1) * C + pc * 8) * sizeof(T))),
                       io<T>::raw8(xs + ((rr + 1) * WP + cc + 1) * XP + pc * 8));
        }
    }
    // ---- the next block's mask unit on the stored values
    if (!SHUF && mask_next && s_own)
        (mask_next + pos0)[static_cast<uint32_t>(srow * W + scol)] =
            mask_of_row<T>(xs + tid * XP, C, wm_next, bm_next, mask_mode) ? 1 : 0;
}

}  // namespace dynconv
