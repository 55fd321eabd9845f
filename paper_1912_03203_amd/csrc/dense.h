// dense.h -- the dense layers of a whole MobileNetV2 feature extractor
// (gfx950).  The paper gates only the stride-1 residual blocks; the stem, the
// strided and width-changing blocks and the final 1x1 convolution run on
// every position (Sec. 4.1.2).  All tensors are NHWC, dense, channels
// fastest.
//
//   k_conv1x1    pointwise convolution as a matrix-core contraction:
//                y[p][o] = act(sum_c w[o][c] x[p][c] + b[o]) (+ r[p][o])
//   k_dwconv3x3  depthwise 3x3, stride 1 or 2, zero padding 1, + bias + act
//   k_conv3x3    full 3x3 convolution (the stem: few input channels),
//                stride 1 or 2, zero padding 1, + bias + act
// Output size of the 3x3 layers: (H - 1) / stride + 1.
#pragma once

#include "kernels.h"

namespace dynconv {

// ------------------------------------------------------------ pointwise
// A work item is a tile of 64 positions (16 per wave) and a range of OT
// 16-row output tiles.  Outputs run along M (rows of w), positions along N:
// lane (r, g) supplies 8 consecutive channels of position r (B) and of output
// row r (A).  The contraction runs in chunks of KB 32-channel steps: the
// wave issues the chunk's KB x loads at once, the workgroup stages the
// chunk's weights for its output range in LDS (rows padded by 8 elements),
// then every wave runs KB x OT matrix-core steps from there.  With one chunk
// (C <= 32 KB) the weights are staged once per workgroup: a workgroup keeps
// its output range and walks position tiles, requesting the next tile's x
// before it contracts the current one.  The accumulation starts from
// the bias and takes c in ascending steps of 32, zero past C.  Every MFMA is
// issued unconditionally (zero fragments out of range).
// Workgroup b runs on XCD b % 8 and takes output range (b / 8) % nor; the
// nor workgroups of one position tile run on the same XCD, so its x rows
// are read from HBM once.
constexpr int kPwPos = 64;

template <typename T, int OT, int KB>
__host__ __device__ constexpr size_t pw_lds_bytes() {
    return static_cast<size_t>(OT) * 16 * (KB * 32 + 8) * sizeof(T);
}

// MULTI: more than one chunk; the next chunk's weights and x are in flight
// while the current one is contracted (their registers would cost the one-chunk
// form a third of its waves: 14x14, batch 64, 96 -> 576 15.0 -> 18.2 us).
template <typename T, int OT, int KB, bool MULTI>
__global__ void __launch_bounds__(kBlock)
k_conv1x1(const T *__restrict__ x, int64_t P, int C, const T *__restrict__ w, const float *__restrict__ b,
          int O, int act, const T *__restrict__ res, T *__restrict__ y, int nor) {
    typedef mma<T> M;
    typedef typename M::frag Frag;
    constexpr int ROWS = OT * 16;
    constexpr int LD = KB * 32 + 8;  // LDS row pitch in elements
    constexpr int PIECES = KB * 4;   // 8-element pieces per staged row
    extern __shared__ __align__(16) unsigned char pw_lds[];
    T *ws = reinterpret_cast<T *>(pw_lds);  // [ROWS][LD]
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r = lane % 16, g = lane / 16;
    const int xcd = blockIdx.x % 8;
    const int orng = static_cast<int>((blockIdx.x / 8) % nor);
    const int64_t slot = (blockIdx.x / 8) / nor, nslot = gridDim.x / 8 / nor;
    const int o_base = orng * ROWS;
    const int64_t ptiles = (P + kPwPos - 1) / kPwPos;
    const int nch = (C + KB * 32 - 1) / (KB * 32);
    const float lo = act_lo(act), hi = act_hi(act);
    // weights of output rows o_base .. o_base+ROWS-1, channels c_base .. c_base+32KB-1
    auto stage = [&](int c_base) {
        for (int i = threadIdx.x; i < ROWS * PIECES; i += kBlock) {
            const int row = i / PIECES, c = c_base + (i % PIECES) * 8;
            const int o = o_base + row;
            const Frag v = (o < O && c < C) ? M::load(w + static_cast<int64_t>(o) * C + c) : M::zero();
            *reinterpret_cast<Frag *>(ws + row * LD + (c - c_base)) = v;
        }
    };
    auto init = [&](floatx4 (&acc)[OT]) {
#pragma unroll
        for (int mt = 0; mt < OT; ++mt) {
            const int o0 = o_base + mt * 16 + 4 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[mt][v] = (o0 + v < O) ? b[o0 + v] : 0.0f;
        }
    };
    auto load_x = [&](Frag (&bx)[KB], int64_t p, int c_base) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int c = c_base + kb * 32 + 8 * g;
            bx[kb] = (p < P && c < C) ? M::load(x + p * C + c) : M::zero();
        }
    };
    auto contract = [&](floatx4 (&acc)[OT], const Frag (&bx)[KB]) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int mt = 0; mt < OT; ++mt) {
                const Frag a = *reinterpret_cast<const Frag *>(ws + (mt * 16 + r) * LD + kb * 32 + 8 * g);
                acc[mt] = M::run(a, bx[kb], acc[mt]);
            }
        }
    };
    auto finish = [&](const floatx4 (&acc)[OT], int64_t p) {
#pragma unroll
        for (int mt = 0; mt < OT; ++mt) {
            const int o0 = o_base + mt * 16 + 4 * g;
            if (p < P && o0 < O) {  // O is a multiple of 8: all four outputs exist
                float out[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = clamp_act(acc[mt][v], lo, hi);
                if (res) {
                    float rv[4];
                    io<T>::load4(res + p * O + o0, rv);
#pragma unroll
                    for (int v = 0; v < 4; ++v) out[v] += rv[v];
                }
                io<T>::store4(y + p * O + o0, out);
            }
        }
    };
    const int64_t step = nslot * 8;
    const int64_t lane_p = wave * 16 + r;  // this lane's position within a tile (B column)
    if constexpr (!MULTI) {
        // weights staged once; the next tile's x is requested before the
        // current tile is contracted
        stage(0);
        __syncthreads();
        int64_t pt = slot * 8 + xcd;
        Frag bn[KB];
        load_x(bn, pt * kPwPos + lane_p, 0);
        for (; pt < ptiles; pt += step) {
            // small weight ranges stay in registers across tiles; larger ones
            // are re-read from LDS per tile (a compiler barrier keeps them
            // from being hoisted out of the loop)
            if constexpr (OT * KB * sizeof(Frag) > 128) __asm__ volatile("" ::: "memory");
            Frag bx[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) bx[kb] = bn[kb];
            if (pt + step < ptiles) load_x(bn, (pt + step) * kPwPos + lane_p, 0);
            floatx4 acc[OT];
            init(acc);
            contract(acc, bx);
            finish(acc, pt * kPwPos + lane_p);
        }
    } else if constexpr (sizeof(Frag) * KB > 128) {
        // fp32 chunks of 256 channels: two of them in flight spill into fewer waves
        // (64 x 7x7, 320 -> 1280 63.1 us, now 59.1; 64 x 14x14, 384 -> 96 25.0, now 22.6)
        for (int64_t pt = slot * 8 + xcd; pt < ptiles; pt += step) {
            const int64_t p = pt * kPwPos + lane_p;
            floatx4 acc[OT];
            init(acc);
            for (int ch = 0; ch < nch; ++ch) {
                Frag bx[KB];
                load_x(bx, p, ch * KB * 32);
                __syncthreads();  // every wave is done with the previous chunk
                stage(ch * KB * 32);
                __syncthreads();
                contract(acc, bx);
            }
            finish(acc, p);
        }
    } else {
        constexpr int WP = (ROWS * PIECES + kBlock - 1) / kBlock;
        Frag wv[WP], bn[KB];
        auto load_w = [&](int c_base) {
#pragma unroll
            for (int q = 0; q < WP; ++q) {
                const int i = threadIdx.x + q * kBlock;
                const int row = i / PIECES, c = c_base + (i % PIECES) * 8;
                const int o = o_base + row;
                const bool in = i < ROWS * PIECES && o < O && c < C;
                wv[q] = M::load(w + (in ? static_cast<int64_t>(o) * C + c : 0));
                if (!in) wv[q] = M::zero();
            }
        };
        auto store_w = [&]() {
#pragma unroll
            for (int q = 0; q < WP; ++q) {
                const int i = threadIdx.x + q * kBlock;
                if (i < ROWS * PIECES) *reinterpret_cast<Frag *>(ws + (i / PIECES) * LD + (i % PIECES) * 8) = wv[q];
            }
        };
        for (int64_t pt = slot * 8 + xcd; pt < ptiles; pt += step) {
            const int64_t p = pt * kPwPos + lane_p;
            load_w(0);
            load_x(bn, p, 0);
            floatx4 acc[OT];
            init(acc);
            for (int ch = 0; ch < nch; ++ch) {
                Frag bx[KB];
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) bx[kb] = bn[kb];
                __syncthreads();  // every wave is done with the previous chunk
                store_w();
                __syncthreads();
                if (ch + 1 < nch) {
                    load_w((ch + 1) * KB * 32);
                    load_x(bn, p, (ch + 1) * KB * 32);
                }
                contract(acc, bx);
            }
            finish(acc, p);
        }
    }
}

// ---------------------------------------------- pointwise, few positions
// The same contraction where a tile of 16 outputs x 16 positions per wave is all
// there is (single images): every wave on its own, both operands straight from
// the caches into a ring of D steps of 32 channels, without LDS, barriers or
// branches around the loads (what is in flight is known at every wait).
// Accumulation as in k_conv1x1 (bias first, steps of 32 channels ascending), so
// the outputs are the same.  Bound by the latency of the first loads; k_conv1x1
// pays two barriers and a memory latency per 256 channels there.  One image, us
// per launch in a graph, k_conv1x1 / this one: 7x7 960 -> 320 9.3 / 9.0, 320 -> 1280
// 6.8 / 5.4, 56x56 144 -> 24 3.9 / 3.0; fp32 7x7 320 -> 1280 15.4 / 7.6.
// The four waves of a workgroup take neighbouring output tiles of the same
// positions.
template <typename T, int D>
__global__ void __launch_bounds__(kBlock)
k_conv1x1_tile(const T *__restrict__ x, int P, int C, const T *__restrict__ w, const float *__restrict__ b, int O,
               int act, const T *__restrict__ res, T *__restrict__ y, int nog) {
    typedef mma<T> M;
    typedef typename M::frag Frag;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int r = lane % 16, g = lane / 16;
    const int og = blockIdx.x % nog, p0 = (blockIdx.x / nog) * 16;
    const int o0 = (og * kWavesPerBlock + wave) * 16;
    if (o0 >= O) return;  // uniform per wave, no barrier below
    const int nks = (C + 31) / 32;
    // rows past P or O read the last one; their products are not stored
    const T *xr = x + static_cast<int64_t>(min(p0 + r, P - 1)) * C;
    const T *wr = w + static_cast<int64_t>(min(o0 + r, O - 1)) * C;
    Frag a[D], v[D];
    auto load = [&](int ks, int d) {
        const int c = min(ks * 32 + 8 * g, C - 8);  // past C: zeroed before use
        a[d] = M::load(wr + c);
        v[d] = M::load(xr + c);
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d) load(d, d);
    const int o = o0 + 4 * g;
    floatx4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = b[min(o + q, O - 1)];
    auto step = [&](int ks, int d) {
        if (ks * 32 + 8 * g >= C) {  // the contraction's tail
            a[d] = M::zero();
            v[d] = M::zero();
        }
        acc = M::run(a[d], v[d], acc);
    };
    int ks = 0;
    for (; ks + D <= nks; ks += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            load(ks + d + D - 1, (d + D - 1) % D);
            step(ks + d, d);
        }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (ks + d < nks) step(ks + d, d);
    const float lo = act_lo(act), hi = act_hi(act);
    const int p = p0 + r;
    if (p < P && o < O) {  // O is a multiple of 8: all four outputs exist
        const int64_t at = static_cast<int64_t>(p) * O + o;
        float out[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = clamp_act(acc[q], lo, hi);
        if (res) {
            float rv[4];
            io<T>::load4(res + at, rv);
#pragma unroll
            for (int q = 0; q < 4; ++q) out[q] += rv[q];
        }
        io<T>::store4(y + at, out);
    }
}

// ------------------------------------------------------------ depthwise
// A work item is (image, block of R output rows, 256 consecutive (column,
// 8-channel group) tasks, groups fastest).  A lane's task walks the input
// rows of its R output rows once: each input row's three taps (16-byte
// loads, zeros past the left and right edges) feed every output row that
// uses it, so a lane issues (S (R - 1) + 3) x 3 tap loads for R outputs
// instead of 9 R.  The 72 weights of the lane's 8 channels are contiguous in
// memory ([C][9]): each lane reads them itself, with the taps of the first
// rows in flight behind them, or (LDSW, few channels) the workgroup stages all
// of them in LDS first.  Each output accumulates in fp32 from the bias,
// taps in (kh, kw) order; rows outside the image are skipped.
// Bound by the latency of these loads: few work items take small R, so that
// more waves are in flight (launch_dwconv_s).  Staging 9 C weights per
// workgroup (two-byte loads, a division each, and a barrier) took 8.2 us for
// 14x14x576 -> 7x7 of one image, lanes reading their own 4.1; at 64 x 112x112x32,
// where it is one weight per lane, LDS is the faster (launch_dwconv_r).
template <typename T>
struct DwWeights {  // [8][9]
    struct __attribute__((packed, aligned(2))) raw_t {
        uint32_t v[36];
    };
    raw_t w;
    __device__ __forceinline__ void load(const T *p) { w = *reinterpret_cast<const raw_t *>(p); }
    __device__ __forceinline__ float at(int u, int k) const {
        const int i = u * 9 + k;
        typedef T pair_t __attribute__((ext_vector_type(2)));
        return static_cast<float>(__builtin_bit_cast(pair_t, w.v[i / 2])[i % 2]);
    }
};
template <>
struct DwWeights<float> {
    float w[72];
    __device__ __forceinline__ void load(const float *p) {
#pragma unroll
        for (int i = 0; i < 72; ++i) w[i] = p[i];
    }
    __device__ __forceinline__ float at(int u, int k) const { return w[u * 9 + k]; }
};

// The weights of 8 channels out of LDS, transposed [9][C].
template <typename T>
struct DwWeightsLds {
    typename io<T>::vec8 w[9];
    __device__ __forceinline__ void load(const T *p, int C) {
#pragma unroll
        for (int k = 0; k < 9; ++k) w[k] = io<T>::raw8(p + k * C);
    }
    __device__ __forceinline__ float at(int u, int k) const { return static_cast<float>(w[k][u]); }
};

template <typename T, int S, int R, bool LDSW>
__global__ void __launch_bounds__(kBlock)
k_dwconv3x3(const T *__restrict__ x, int N, int H, int W, int C, const T *__restrict__ w,
            const float *__restrict__ b, int act, T *__restrict__ y, int Ho, int Wo) {
    typedef typename io<T>::vec8 V;
    constexpr int ROWS = S * (R - 1) + 3;  // input rows of R output rows
    extern __shared__ __align__(16) unsigned char dw_smem[];
    T *wt = reinterpret_cast<T *>(dw_smem);  // LDSW: [9][C]
    if constexpr (LDSW) {
        for (int i = threadIdx.x; i < 9 * C; i += kBlock) {
            const int ch = i / 9, k = i % 9;
            wt[k * C + ch] = w[i];
        }
        __syncthreads();
    }
    const float lo = act_lo(act), hi = act_hi(act);
    const uint32_t cgs = C / 8;
    const uint32_t tasks = Wo * cgs;
    const uint32_t chunks = (tasks + kBlock - 1) / kBlock;
    const uint32_t rbs = (Ho + R - 1) / R;
    const uint32_t items = N * rbs * chunks;  // fits: fewer than the outputs' 8-channel groups
    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        const uint32_t nr = it / chunks, chunk = it - nr * chunks;
        const uint32_t n = nr / rbs;
        const int i0 = (nr - n * rbs) * R;  // first output row
        const uint32_t task = chunk * kBlock + threadIdx.x;
        if (task >= tasks) continue;
        const int j = task / cgs, c = (task - j * cgs) * 8;
        std::conditional_t<LDSW, DwWeightsLds<T>, DwWeights<T>> wk;
        if constexpr (LDSW) wk.load(wt + c, C);
        else wk.load(w + c * 9);
        float acc[R][8];
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[q][u] = b[c + u];
        const T *img = x + static_cast<int64_t>(n) * H * W * C;
#pragma unroll
        for (int t = 0; t < ROWS; ++t) {
            const int hh = S * i0 - 1 + t;
            if (hh < 0 || hh >= H) continue;
            V v[3];
#pragma unroll
            for (int dw = 0; dw < 3; ++dw) {
                const int ww = S * j - 1 + dw;
                if (ww >= 0 && ww < W) {
                    v[dw] = io<T>::raw8(img + (static_cast<int64_t>(hh) * W + ww) * C + c);
                } else {
                    v[dw] = V{};
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int dh = t - S * q;  // compile-time after unrolling
                if (dh < 0 || dh > 2) continue;
#pragma unroll
                for (int dw = 0; dw < 3; ++dw)
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        acc[q][u] = __builtin_fmaf(wk.at(u, dh * 3 + dw), static_cast<float>(v[dw][u]), acc[q][u]);
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            if (i0 + q >= Ho) break;
            float o[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = clamp_act(acc[q][u], lo, hi);
            T *dst = y + ((static_cast<int64_t>(n) * Ho + i0 + q) * Wo + j) * C + c;
            io<T>::store4(dst, o);
            io<T>::store4(dst + 4, o + 4);
        }
    }
}

// ------------------------------------------------------ expansion + depthwise
// An ungated block's 1x1 expansion and depthwise 3x3 in one launch, so that
// the expanded tensor never goes to HBM.  A work item is a tile of 8 x 8
// depthwise outputs of one image; its input region, (S*7+3)^2 positions, is
// staged in LDS (rows of C + 8 elements, zeros outside the image).  The
// workgroups are persistent: each stages all weights in LDS once (expansion
// rows of C + 8, depthwise taps transposed to [9][E]) and walks items,
// loading the next item's region into registers while it computes the
// current one.  Per 32-channel slice of the hidden layer: each wave expands
// 16-position tiles of the region on the matrix cores (operands as in
// k_conv1x1: bias first, 32-channel steps ascending), applies the activation
// and stores the slice into a region array (zeros at positions outside the
// image: the depthwise's zero padding); then lane (o, cg) computes the
// depthwise of output o for 8 hidden channels from 9 fixed slots of that
// array, fp32 from the bias, taps in (kh, kw) order, and writes it to
// h2 [Ho*Wo][E].
constexpr int kEdTile = 8;  // depthwise outputs per tile side

template <int S>
__host__ __device__ constexpr int ed_region_side() { return S * (kEdTile - 1) + 3; }
template <int S>
__host__ __device__ constexpr int ed_region_tiles() {
    return (ed_region_side<S>() * ed_region_side<S>() + 15) / 16;
}
template <typename T, int S>
__host__ __device__ constexpr size_t ed_lds_bytes(int C, int E) {
    return static_cast<size_t>(ed_region_tiles<S>()) * 16 * ((C + 8) + 40) * sizeof(T)  // xs + h1
           + static_cast<size_t>(E) * (C + 8) * sizeof(T) + 9 * static_cast<size_t>(E) * sizeof(T)  // w1, w2t
           + 8 * static_cast<size_t>(E);                                                            // b1, b2
}

template <typename T, int S, int KS>
__global__ void __launch_bounds__(kBlock)
k_expand_dw(const T *__restrict__ x, int N, int H, int W, int C, const T *__restrict__ w1,
            const float *__restrict__ b1, int act1, int E, const T *__restrict__ w2, const float *__restrict__ b2,
            int act2, T *__restrict__ h2, int Ho, int Wo) {
    typedef mma<T> M;
    typedef typename M::frag Frag;
    typedef typename io<T>::vec8 V;
    constexpr int RS = ed_region_side<S>();
    constexpr int RP = RS * RS;
    constexpr int NT = ed_region_tiles<S>();
    constexpr int TPW = (NT + kWavesPerBlock - 1) / kWavesPerBlock;  // tiles per wave
    constexpr int HP = 40;                                          // h1 row pitch (32 + 8)
    constexpr int XP = (NT * 16 * KS * 4 + kBlock - 1) / kBlock;     // x pieces per thread (<= 32)
    static_assert(XP <= 32, "x pieces per thread exceed the validity mask");
    extern __shared__ __align__(16) unsigned char ed_smem[];
    const int PX = C + 8;  // row pitch of x and of the expansion weights
    T *xs = reinterpret_cast<T *>(ed_smem);  // [NT*16][PX]
    T *h1 = xs + NT * 16 * PX;               // [NT*16][HP]
    T *w1s = h1 + NT * 16 * HP;              // [E][PX]
    T *w2t = w1s + E * PX;                   // [9][E]
    float *b1s = reinterpret_cast<float *>(w2t + 9 * E);  // [E]
    float *b2s = b1s + E;                                 // [E]
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int r = lane % 16, g = lane / 16;
    const float lo1 = act_lo(act1), hi1 = act_hi(act1), lo2 = act_lo(act2), hi2 = act_hi(act2);
    const int tr = (Ho + kEdTile - 1) / kEdTile, tc = (Wo + kEdTile - 1) / kEdTile;
    const int64_t items = static_cast<int64_t>(N) * tr * tc;
    const int nsl = (E + 31) / 32;
    const int pieces = C / 8;  // 16-byte pieces of an x row
    if (static_cast<int64_t>(blockIdx.x) >= items) return;
    // all weights, once
    for (int i = tid; i < E * pieces; i += kBlock) {
        const int e = i / pieces, pc = (i % pieces) * 8;
        *reinterpret_cast<V *>(w1s + e * PX + pc) = io<T>::raw8(w1 + static_cast<int64_t>(e) * C + pc);
    }
    for (int i = tid; i < 9 * E; i += kBlock) {
        const int e = i / 9, k = i % 9;
        w2t[k * E + e] = w2[i];
    }
    for (int e = tid; e < E; e += kBlock) {
        b1s[e] = b1[e];
        b2s[e] = b2[e];
    }
    // the item's region origin; one thread's x pieces of it, into registers
    auto origin = [&](int64_t it, int &n, int &i0, int &j0) {
        n = static_cast<int>(it / (tr * tc));
        const int rem = static_cast<int>(it % (tr * tc));
        i0 = (rem / tc) * kEdTile;
        j0 = (rem % tc) * kEdTile;
    };
    // Loads are issued unconditionally (pieces outside the image read the
    // tensor's first piece) and replaced by zeros only when stored, so no
    // wait for them is needed before the current item's slices.
    auto load_x = [&](int64_t it, V (&xr)[XP], uint32_t &ok) {
        int n, i0, j0;
        origin(it, n, i0, j0);
        const int hb = S * i0 - 1, wb = S * j0 - 1;
        const T *img = x + static_cast<int64_t>(n) * H * W * C;
        ok = 0;
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            const int i = tid + q * kBlock;
            const int slot = i / pieces, pc = (i % pieces) * 8;
            const int hh = hb + slot / RS, ww = wb + slot % RS;
            const bool in = i < NT * 16 * pieces && slot < RP && hh >= 0 && hh < H && ww >= 0 && ww < W;
            xr[q] = io<T>::raw8(in ? img + (static_cast<int64_t>(hh) * W + ww) * C + pc : x);
            ok |= static_cast<uint32_t>(in) << q;
        }
    };
    auto store_x = [&](const V (&xr)[XP], uint32_t ok) {
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            const int i = tid + q * kBlock;
            if (i < NT * 16 * pieces)
                *reinterpret_cast<V *>(xs + (i / pieces) * PX + (i % pieces) * 8) = ((ok >> q) & 1u) ? xr[q] : V{};
        }
    };
    V xr[XP];
    uint32_t xok;
    int64_t it = blockIdx.x;
    load_x(it, xr, xok);
    store_x(xr, xok);
    __syncthreads();
    for (;;) {
        const int64_t next = it + gridDim.x;
        if (next < items) load_x(next, xr, xok);
        int n, i0, j0;
        origin(it, n, i0, j0);
        const int hb = S * i0 - 1, wb = S * j0 - 1;
        // the item's B fragments (region x) and activation bounds, kept for
        // every slice (kBounds; a select per value and slice instead: 49.3 us for
        // 64 x 112x112x16 -> 56x56x96, now 47.2, but with stride 1 and one
        // contraction step the bounds' registers cost more: 64 x 56x56x24, hidden 144,
        // with its projection 62.1 us by selects, 66.4 so); waves past the last tile
        // repeat it (same values), so every wave issues the same MFMAs
        constexpr bool kBounds = S == 2 || KS == 2;
        uint32_t inside = 0;
        Frag bx[TPW][KS];
        float lo_t[TPW], hi_t[TPW];
#pragma unroll
        for (int jt = 0; jt < TPW; ++jt) {
            const int t = wave + kWavesPerBlock * jt;
            const int slot = (t < NT ? t : NT - 1) * 16 + r;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int c = ks * 32 + 8 * g;
                bx[jt][ks] = (c < C) ? *reinterpret_cast<const Frag *>(xs + slot * PX + c) : M::zero();
            }
            const int hh = hb + slot / RS, ww = wb + slot % RS;
            // zeros outside the image, by clamping to [0, 0]
            const bool in = slot < RP && hh >= 0 && hh < H && ww >= 0 && ww < W;
            lo_t[jt] = in ? lo1 : 0.0f;
            hi_t[jt] = in ? hi1 : 0.0f;
            inside |= static_cast<uint32_t>(in) << jt;
        }
        for (int sl = 0; sl < nsl; ++sl) {
            const int e0 = sl * 32;
            // the slice's expansion rows (A) and biases, once per slice
            Frag a1[2][KS];
            floatx4 binit[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int er = e0 + m * 16 + r;  // A row: hidden channel
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int c = ks * 32 + 8 * g;
                    a1[m][ks] = (er < E && c < C) ? *reinterpret_cast<const Frag *>(w1s + er * PX + c) : M::zero();
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int e = e0 + m * 16 + 4 * g + v;
                    binit[m][v] = (e < E) ? b1s[e] : 0.0f;
                }
            }
            // D[e][slot]: rows are hidden channels, columns region slots
#pragma unroll
            for (int jt = 0; jt < TPW; ++jt) {
                const int t = wave + kWavesPerBlock * jt;
                const int slot = (t < NT ? t : NT - 1) * 16 + r;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    floatx4 d = binit[m];
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) d = M::run(a1[m][ks], bx[jt][ks], d);
                    if (t < NT) {
                        float o[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            o[v] = kBounds                 ? clamp_act(d[v], lo_t[jt], hi_t[jt])
                                   : (inside >> jt) & 1u ? clamp_act(d[v], lo1, hi1)
                                                           : 0.0f;
                        io<T>::store4(h1 + slot * HP + m * 16 + 4 * g, o);
                    }
                }
            }
            __syncthreads();
            // depthwise: lane (o, cg), output o of the tile, channels 8cg..8cg+7
            {
                const int o = tid / 4, cg = tid % 4;
                const int oi = o / kEdTile, oj = o % kEdTile;
                const int e8 = e0 + 8 * cg;
                const int i = i0 + oi, j = j0 + oj;
                if (e8 < E) {
                    float acc[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc[u] = b2s[e8 + u];
#pragma unroll
                    for (int k = 0; k < 9; ++k) {
                        const int slot = (S * oi + k / 3) * RS + S * oj + k % 3;
                        const V v = io<T>::raw8(h1 + slot * HP + 8 * cg);
                        const V wk = io<T>::raw8(w2t + k * E + e8);
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            acc[u] = __builtin_fmaf(static_cast<float>(wk[u]), static_cast<float>(v[u]), acc[u]);
                    }
                    if (i < Ho && j < Wo) {
                        float out[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) out[u] = clamp_act(acc[u], lo2, hi2);
                        T *dst = h2 + ((static_cast<int64_t>(n) * Ho + i) * Wo + j) * E + e8;
                        io<T>::store4(dst, out);
                        io<T>::store4(dst + 4, out + 4);
                    }
                }
            }
            __syncthreads();  // h1 is rewritten by the next slice, xs by the next item
        }
        if (next >= items) break;
        store_x(xr, xok);
        __syncthreads();
        it = next;
    }
}

// ------------------------------------------------------------ full 3x3
// One lane per output position computing 32 outputs at a time; weights
// [O][Ci][3][3] and biases staged in LDS as fp32, reordered to [k][ci][o] so
// that the 32 weights of one tap and input channel are 8 broadcast 16-byte
// reads.  Ci is small (the stem's 3 input channels): a lane reads each of its
// 9 Ci input values once per 32 outputs.  Accumulation in fp32 from the
// bias, taps in (kh, kw) order, input channels ascending (dynamic shared
// memory: 9*Ci*O + O floats).
template <typename T>
__global__ void __launch_bounds__(kBlock)
k_conv3x3(const T *__restrict__ x, int N, int H, int W, int Ci, int stride, const T *__restrict__ w,
          const float *__restrict__ b, int O, int act, T *__restrict__ y, int Ho, int Wo) {
    extern __shared__ __align__(16) unsigned char cv_smem[];
    float *ws = reinterpret_cast<float *>(cv_smem);  // [9][Ci][O]
    float *bs = ws + 9 * Ci * O;
    for (int i = threadIdx.x; i < 9 * Ci * O; i += kBlock) {
        const int o = i / (9 * Ci), c = (i / 9) % Ci, k = i % 9;  // w[o][c][k]
        ws[(k * Ci + c) * O + o] = static_cast<float>(w[i]);
    }
    for (int o = threadIdx.x; o < O; o += kBlock) bs[o] = b[o];
    __syncthreads();
    const float lo = act_lo(act), hi = act_hi(act);
    const int64_t total = static_cast<int64_t>(N) * Ho * Wo;
    for (int64_t q = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; q < total;
         q += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int64_t ni = q / Wo;
        const int j = static_cast<int>(q - ni * Wo);
        const int n = static_cast<int>(ni / Ho), i = static_cast<int>(ni - static_cast<int64_t>(n) * Ho);
        const T *img = x + static_cast<int64_t>(n) * H * W * Ci;
        for (int o0 = 0; o0 < O; o0 += 32) {
            const int ng = min(4, (O - o0) / 8);  // 8-output groups in this pass
            float s[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) s[u] = (u / 8 < ng) ? bs[o0 + u] : 0.0f;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int hh = stride * i + k / 3 - 1, ww = stride * j + k % 3 - 1;
                if (hh < 0 || hh >= H || ww < 0 || ww >= W) continue;
                const T *px = img + (static_cast<int64_t>(hh) * W + ww) * Ci;
                for (int c = 0; c < Ci; ++c) {
                    const float v = static_cast<float>(px[c]);
                    const float *wr = ws + (k * Ci + c) * O + o0;
#pragma unroll
                    for (int gq = 0; gq < 4; ++gq) {
                        if (gq >= ng) break;
                        const float4 wa = *reinterpret_cast<const float4 *>(wr + 8 * gq);
                        const float4 wb = *reinterpret_cast<const float4 *>(wr + 8 * gq + 4);
                        const float wk[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
                        for (int u = 0; u < 8; ++u) s[8 * gq + u] = __builtin_fmaf(wk[u], v, s[8 * gq + u]);
                    }
                }
            }
            T *dst = y + q * O + o0;
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                if (gq >= ng) break;
                float o[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) o[u] = clamp_act(s[8 * gq + u], lo, hi);
                io<T>::store4(dst + 8 * gq, o);
                io<T>::store4(dst + 8 * gq + 4, o + 4);
            }
        }
    }
}

// ------------------------------------------------ full 3x3 on the matrix cores
// The same convolution as an implicit-im2col contraction for 16-bit
// storage: the contraction index runs over (tap, input channel) pairs,
// kk = k * Ci + c with tap k = 3 kh + kw, zero-padded to KS steps of 32.
// Outputs run along M, output positions along N: lane (r, g) gathers the 8
// input values kk = 32 ks + 8 g .. +7 of its position r (zeros outside the
// image and past 9 Ci) straight into its B fragment, the weights sit in LDS
// as [O][32 KS + 8] rows in kk order, and the wave walks the outputs in
// ranges of OT tiles of 16.  Accumulation from the bias in kk order (32 at a
// time on the matrix core); the taps' (dh, dw, c) per kk come from a small
// LDS table.  Dynamic shared memory: O (32 KS + 8) elements + 32 KS ints, at
// least 384 bytes (the masks of WIN).
// A wave takes tiles of 16 consecutive output positions, which may cross rows
// and images: no width leaves lanes idle.
//
// WIN (3 input channels, the stem): the 8 values of a fragment lie in at most
// two kernel rows, 9 consecutive elements each in memory, so a lane reads two
// 16-byte windows, placed so that value u of either is kk = 8 g + u of its row,
// and picks by masks.  Waves with a position at the border narrow the masks and
// move windows that would reach outside the tensor (shifted back in registers).
// 8 two-byte loads with their LDS table reads and bounds took 40.2 us for
// 64 x 224x224x3 -> 112x112x32 (70 MB), the windows 25.7.  With tiles of 16 columns
// of one row and a gather beside the windows at borders, narrow maps were slower
// than that: 64 x 224x33 -> 112x17x32 10.2 (gather), 13.2, now 8.5; one 224x224 image
// 4.8, 5.5, now 4.6.
struct __attribute__((packed, aligned(2))) half8_bits {
    uint32_t v[4];
};

// q / d for q < 2^28: (q * m) >> (32 + s), or q itself for d = 1
struct Div28 {
    uint32_t m, s, one;
};
inline Div28 div28(uint32_t d) {
    if (d == 1) return {0, 0, 0xffffffffu};
    uint32_t l = 1;
    while ((uint64_t{1} << l) < d) ++l;
    const uint32_t k = l <= 4 ? 32 : 28 + l;  // 2^28 d <= 2^k, and m below 2^32
    return {static_cast<uint32_t>(((uint64_t{1} << k) + d - 1) / d), k - 32, 0};
}
__device__ __forceinline__ uint32_t quotient(uint32_t q, Div28 d) { return (__umulhi(q, d.m) >> d.s) + (q & d.one); }

// w moved by d elements, zeros moving in: value u of the result is value u - d of w
__device__ __forceinline__ half8_bits moved(half8_bits w, int d) {
    half8_bits out;
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
        uint32_t pair = 0;
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            uint32_t h = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (u + z - d == k) h = (w.v[k / 2] >> (16 * (k % 2))) & 0xffffu;
            pair |= h << (16 * z);
        }
        out.v[u / 2] = pair;
    }
    return out;
}

template <typename T, int KS, int OT, bool WIN>
__global__ void __launch_bounds__(kBlock)
k_conv3x3_mfma(const T *__restrict__ x, int N, int H, int W, int Ci, int stride, const T *__restrict__ w,
               const float *__restrict__ b, int O, int act, T *__restrict__ y, int Ho, int Wo, Div28 dHo, Div28 dWo) {
    typedef mma<T> M;
    typedef typename M::frag Frag;
    constexpr int KP = KS * 32 + 8;  // LDS row pitch of the weights
    extern __shared__ __align__(16) unsigned char c3_smem[];
    T *ws = reinterpret_cast<T *>(c3_smem);         // [O][KP]
    int *tap = reinterpret_cast<int *>(ws + O * KP);  // [32 KS]: (dh+1) | (dw+1) << 2 | c << 4, -1 past 9 Ci
    const int K = 9 * Ci;
    for (int i = threadIdx.x; i < O * KP; i += kBlock) {
        const int o = i / KP, kk = i % KP;
        ws[i] = (kk < K) ? w[(o * Ci + kk % Ci) * 9 + kk / Ci] : static_cast<T>(0.0f);
    }
    // WIN: the fragment's values of lanes with this g that the window of its first
    // and of its second kernel row hold, of those the ones in the row's first and
    // in its last column: masks [g][3][2]
    uint4 *masks = reinterpret_cast<uint4 *>(tap);
    if constexpr (WIN) {
        if (threadIdx.x < 24) {
            const int mg = threadIdx.x / 6, col = threadIdx.x / 2 % 3, second = threadIdx.x % 2;
            uint32_t bits[4] = {0, 0, 0, 0};
            for (int u = 0; u < 8; ++u) {
                const int kk = 8 * mg + u, at = kk % 9 / 3;  // column of the kernel row
                if (kk < 27 && (kk / 9 != 8 * mg / 9) == (second == 1) && (col == 0 || at == (col == 1 ? 0 : 2)))
                    bits[u / 2] |= 0xffffu << (16 * (u % 2));
            }
            masks[threadIdx.x] = make_uint4(bits[0], bits[1], bits[2], bits[3]);
        }
    } else {
        for (int kk = threadIdx.x; kk < 32 * KS; kk += kBlock) {
            const int k = kk / Ci, c = kk % Ci;
            tap[kk] = (kk < K) ? ((k / 3) | ((k % 3) << 2) | (c << 4)) : -1;
        }
    }
    __syncthreads();
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r = lane % 16, g = lane / 16;
    const float lo = act_lo(act), hi = act_hi(act);
    const int nmt = (O + 15) / 16;
    const uint32_t total = static_cast<uint32_t>(N) * Ho * Wo, tiles = (total + 15) / 16;  // positions fit 28 bits
    // WIN: element offsets of this lane's two windows from the position's first tap
    // (32 bits: the tensor has at most 3 2^28 elements); without a second one
    // the first again
    const int kk0 = 8 * g, kh0 = kk0 / 9, off0 = kk0 - kh0 * 9, n0 = 9 - off0;
    const bool two = n0 < 8 && kh0 < 2;
    const int run0 = kh0 * W * 3 + off0, run1 = two ? (kh0 + 1) * W * 3 - n0 : run0;
    uint4 m0, m1;
    if constexpr (WIN) {
        m0 = masks[6 * g];
        m1 = masks[6 * g + 1];
    }
    const uint32_t wave0 = __builtin_amdgcn_readfirstlane(blockIdx.x * kWavesPerBlock + wave);
    for (uint32_t t = wave0; t < tiles; t += gridDim.x * kWavesPerBlock) {
        const bool qin = t * 16 + r < total;
        const uint32_t q = min(t * 16 + r, total - 1);
        const uint32_t row = quotient(q, dWo), n = quotient(row, dHo);
        const int i = row - n * Ho, j = q - row * Wo;
        const int h0 = stride * i - 1, w0 = stride * j - 1;
        Frag bx[KS];
        if constexpr (WIN) {
            const int size = N * H * W * 3, first = ((static_cast<int>(n) * H + h0) * W + w0) * 3;
            const int at0 = first + run0, at1 = first + run1;
            const int from0 = min(max(at0, 0), size - 8), from1 = min(max(at1, 0), size - 8);
            half8_bits a = *reinterpret_cast<const half8_bits *>(x + from0);
            half8_bits c = *reinterpret_cast<const half8_bits *>(x + from1);
            uint4 s0 = m0, s1 = m1;
            const bool left = w0 < 0, right = w0 + 3 > W, top = h0 < 0, bottom = h0 + 3 > H;
            if (__any(left | right | top | bottom)) {
                const bool in0 = h0 + kh0 >= 0 && h0 + kh0 < H, in1 = h0 + kh0 + 1 < H;
                const uint4 zero = make_uint4(0, 0, 0, 0);
                auto narrow = [&](uint4 m, bool in, int second) {
                    const uint4 l = left ? masks[6 * g + 2 + second] : zero, e = right ? masks[6 * g + 4 + second] : zero;
                    return in ? make_uint4(m.x & ~(l.x | e.x), m.y & ~(l.y | e.y), m.z & ~(l.z | e.z), m.w & ~(l.w | e.w)) : zero;
                };
                s0 = narrow(m0, in0, 0);
                s1 = narrow(m1, in1, 1);
            }
            // windows that would reach outside the tensor were read where it ends
            if (__any(from0 != at0 || from1 != at1)) {
                a = moved(a, from0 - at0);
                c = moved(c, from1 - at1);
            }
            half8_bits v;
            const uint32_t k0[4] = {s0.x, s0.y, s0.z, s0.w}, k1[4] = {s1.x, s1.y, s1.z, s1.w};
#pragma unroll
            for (int z = 0; z < 4; ++z) v.v[z] = (a.v[z] & k0[z]) | (c.v[z] & k1[z]);
            bx[0] = __builtin_bit_cast(Frag, v);
        } else {
            const T *img = x + static_cast<int64_t>(n) * H * W * Ci;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = tap[ks * 32 + 8 * g + u];
                    const int hh = h0 + (e & 3), ww = w0 + ((e >> 2) & 3), c = e >> 4;
                    v[u] = (qin && e >= 0 && hh >= 0 && hh < H && ww >= 0 && ww < W)
                               ? static_cast<float>(img[(static_cast<int64_t>(hh) * W + ww) * Ci + c])
                               : 0.0f;
                }
                bx[ks] = M::pack(v);
            }
        }
        for (int ob = 0; ob < nmt; ob += OT) {
            floatx4 acc[OT];
#pragma unroll
            for (int mt = 0; mt < OT; ++mt) {
                const int o0 = (ob + mt) * 16 + 4 * g;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[mt][v] = (o0 + v < O) ? b[o0 + v] : 0.0f;
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int mt = 0; mt < OT; ++mt) {
                    const int o = (ob + mt) * 16 + r;
                    const Frag a = (o < O) ? *reinterpret_cast<const Frag *>(ws + o * KP + ks * 32 + 8 * g)
                                           : M::zero();
                    acc[mt] = M::run(a, bx[ks], acc[mt]);
                }
            }
#pragma unroll
            for (int mt = 0; mt < OT; ++mt) {
                const int o0 = (ob + mt) * 16 + 4 * g;
                if (qin && o0 < O) {  // O is a multiple of 8: all four outputs exist
                    float out[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) out[v] = clamp_act(acc[mt][v], lo, hi);
                    io<T>::store4(y + static_cast<int64_t>(q) * O + o0, out);
                }
            }
        }
    }
}

}  // namespace dynconv
