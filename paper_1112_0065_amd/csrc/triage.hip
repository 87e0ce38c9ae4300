// Triage network kernels: candidate tiles, a 4-layer bfloat16 CNN forward and
// backward pass, and Adam.
//
// The paper's section 2.1 names radio-frequency interference as the main
// source of false events.  This network scores (DM, time) candidate tiles so
// that interference can be rejected; the plain S/N detector remains the
// fallback.  Layout: activations NHWC bfloat16 (channels innermost, 64 bytes
// per pixel), float32 accumulation.  Every layer's ReLU and 2x2 max-pool
// follow its convolution in registers: only pooled maps and the winners' places
// (2 bits) are stored, and the backward pass keeps one gradient per window.
// The 32->32 convolutions (forward and input gradient) are implicit GEMMs on
// the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, gfx950's double-K form: M =
// pixels, N = 32 output channels, K = 9 taps x 32 input channels = 288, one
// tap per step); the weight gradients are GEMMs over pixels (K = 32 pixels per
// step) on the same instruction, reduced across blocks in a fixed order (no
// float atomics: training is reproducible bit for bit).  The 1->32 first layer
// (K = 9) runs on VALU.
#include <algorithm>
#include <cstdint>

#include "triage_kernels.hpp"

namespace tk {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest even (finite inputs)
    return static_cast<uint16_t>(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// ---------------------------------------------------------------------------
// Candidate tiles: one block of 256 threads per (event, row), 64 columns per
// wave.  A row's 256 columns are adjacent windows of w samples, so a row reads
// 256 w consecutive samples once: the kernel is bound by those reads (up to
// 256 KiB a row, from the last-level cache where candidates overlap).  A
// thread per column read 2 bytes per load at a stride of 2 w bytes: 1957 us
// for 217 candidates at widths 1..512, 0.4 TB/s.  Groups of lanes that share a
// column and read it in consecutive 16-byte pieces take 112 us (6.5 TB/s).  Widths
// that are no multiple of 8 read pieces as well (300 tiles at width 9: a thread per
// column 35 us, groups that read single samples 64, pieces KK9; width 33: 332, 346,
// KK33); below 8 a thread per column is left.
// ---------------------------------------------------------------------------

// Eight consecutive samples at any (2-byte aligned) address.
struct __attribute__((packed, aligned(2))) Piece {
    uint32_t w[4];
};
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Sum of a piece's samples from `skip` (0 .. 7; a multiple of 8 if not RAGGED) on.
template <bool RAGGED>
__device__ __forceinline__ uint32_t piece_sum(const Piece& p, int skip) {
    const u16x2 one = {1, 1};
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t keep = !RAGGED || skip <= 2 * i ? 0xFFFFFFFFu : skip == 2 * i + 1 ? 0xFFFF0000u : 0u;
        s = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, p.w[i] & keep), one, s, false);
    }
    return s;
}

// Sums of the wave's 64 adjacent windows of w >= 8 samples from `row` on, window
// l in lane l; the first `ncol` (>= 1) windows lie inside the series, the
// others repeat the last one.  A window is read in 16-byte pieces; RAGGED (w not a
// multiple of 8): the last one is read so that it ends with the window, and what it
// shares with the one before does not count.  G = 2^LG lanes, enough for the
// pieces or 64, share a window, so 64 / G windows are read at a time; up to 8
// such rounds are in flight at once.  Lanes without a piece read a valid one
// and count 0, so the loads carry no branch.
template <bool RAGGED, int LG>
__device__ __forceinline__ uint32_t window_sums(const uint16_t* __restrict__ row, int w, int pieces,
                                                int ncol, int lane) {
    constexpr int G = 1 << LG, C = 64 >> LG;
    constexpr int kRounds = G < 8 ? G : 8;
    const int c = lane >> LG, p = lane & (G - 1);
    uint32_t mine = 0;
    for (int it0 = 0; it0 < G; it0 += kRounds) {
        uint32_t s[kRounds];
#pragma unroll
        for (int k = 0; k < kRounds; ++k) s[k] = 0;
        for (int q0 = 0; q0 < pieces; q0 += G) {
            const bool has = q0 + p < pieces;
            const int q = has ? q0 + p : 0;
            const int at = RAGGED ? min(8 * q, w - 8) : 8 * q;
            uint32_t x[kRounds];
#pragma unroll
            for (int k = 0; k < kRounds; ++k) {
                const uint16_t* src = row + static_cast<int64_t>(min((it0 + k) * C + c, ncol - 1)) * w;
                x[k] = piece_sum<RAGGED>(*reinterpret_cast<const Piece*>(src + at), 8 * q - at);
            }
#pragma unroll
            for (int k = 0; k < kRounds; ++k) s[k] += has ? x[k] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kRounds; ++k) {
#pragma unroll
            for (int o = G >> 1; o >= 1; o >>= 1)
                s[k] += static_cast<uint32_t>(__shfl_xor(static_cast<int>(s[k]), o, 64));
            // lanes [C (it0 + k), C (it0 + k + 1)) keep this round's windows
            const uint32_t v = static_cast<uint32_t>(__shfl(static_cast<int>(s[k]), (lane & (C - 1)) << LG, 64));
            if (lane / C == it0 + k) mine = v;
        }
    }
    return mine;
}

template <bool RAGGED>
__device__ __forceinline__ uint32_t window_sums_w(const uint16_t* __restrict__ row, int w, int ncol, int lane) {
    const int pieces = (w + 7) >> 3;
    if (pieces > 32) return window_sums<RAGGED, 6>(row, w, pieces, ncol, lane);
    if (pieces > 16) return window_sums<RAGGED, 5>(row, w, pieces, ncol, lane);
    if (pieces > 8) return window_sums<RAGGED, 4>(row, w, pieces, ncol, lane);
    if (pieces > 4) return window_sums<RAGGED, 3>(row, w, pieces, ncol, lane);
    if (pieces > 2) return window_sums<RAGGED, 2>(row, w, pieces, ncol, lane);
    if (RAGGED || pieces > 1) return window_sums<RAGGED, 1>(row, w, pieces, ncol, lane);
    return window_sums<RAGGED, 0>(row, w, pieces, ncol, lane);
}

// Windows of fewer than 8 samples: one lane each, neighbouring ones.
__device__ __forceinline__ uint32_t window_sums_short(const uint16_t* __restrict__ row, int w, int ncol, int lane) {
    const uint16_t* src = row + min(lane, ncol - 1) * w;
    uint32_t s = 0;
    for (int k = 0; k < w; ++k) s += src[k];
    return s;
}

__global__ __launch_bounds__(256) void tiles_kernel(const uint16_t* __restrict__ series, int ndm,
                                                    int64_t nout, int64_t nbx, TileWidths W,
                                                    const dedisp_event* __restrict__ events,
                                                    const uint64_t* __restrict__ s1,
                                                    const double* __restrict__ sqrt_d,
                                                    uint16_t* __restrict__ tiles) {
    const int e = blockIdx.x;
    const int r = blockIdx.y;
    const int j = threadIdx.x;
    const int lane = j & 63;
    const int j0 = __builtin_amdgcn_readfirstlane(j & ~63);
    const dedisp_event ev = events[e];
    const int w = W.w[ev.width_idx];
    int d0 = ev.dm_idx - 32;
    d0 = min(max(d0, 0), max(ndm - 64, 0));
    int64_t t0 = ev.t_peak - 128 * static_cast<int64_t>(w);
    t0 = min(max(t0, int64_t(0)), max(nbx - 255 * static_cast<int64_t>(w) - 1, int64_t(0)));
    const int d = d0 + r;
    float v = 0.0f;
    // the wave's columns: t = tw + w l; those below nbx are inside the series
    // with their whole window
    const int64_t tw = t0 + static_cast<int64_t>(j0) * w;
    const int ncol = __popcll(__ballot(tw + static_cast<int64_t>(lane) * w < nbx));
    if (d < ndm && ncol > 0) {
        const int sidx = ev.width_idx * ndm + d;
        const double sq = sqrt_d[sidx];
        if (sq > 0.0) {
            const uint16_t* row = series + static_cast<int64_t>(d) * nout + tw;
            const uint32_t b = w < 8          ? window_sums_short(row, w, ncol, lane)
                               : (w & 7) == 0 ? window_sums_w<false>(row, w, ncol, lane)
                                              : window_sums_w<true>(row, w, ncol, lane);
            const int64_t lval = nbx * static_cast<int64_t>(b) - static_cast<int64_t>(s1[sidx]);
            if (lane < ncol) v = static_cast<float>(static_cast<double>(lval) / sq);
        }
    }
    tiles[(static_cast<int64_t>(e) * 64 + r) * 256 + j] = f2bf(v);
}

// ---------------------------------------------------------------------------
// Packing helpers.
// ---------------------------------------------------------------------------
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two floats rounded to bfloat16 (nearest even), a in the low half.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Two consecutive values; the caller's tiles may start at any 2-byte boundary.
__device__ __forceinline__ uint32_t load_pair(const uint16_t* p, bool aligned) {
    return aligned ? *reinterpret_cast<const uint32_t*>(p) : p[0] | (static_cast<uint32_t>(p[1]) << 16);
}

// The value held by the neighbouring lane (lane ^ 1).
__device__ __forceinline__ uint32_t neighbour(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xF, 0xF, false));
}

// 2x2 max-pool of four values rounded to bfloat16, ReLU included: max(x, 0) of
// a NaN of either sign is 0, as fmaxf gives it.  A value's key is its bits, 0x7F
// above them modulo 2^16, over 3 - k: the signed maximum is then the largest
// value, of equal ones the first in raster order.  0 has 0x7F and infinity
// 0x7FFF; negative values and NaNs with a clear sign are negative, NaNs with a
// set sign below 0x7F, so all of these lose to 0, whose winner nobody asks for
// (a pooled 0 passes no gradient).  Returns the pooled value in bits 16-31 and
// 3 - winner in bits 0-1.
__device__ __forceinline__ uint32_t pool_key(uint32_t v01, uint32_t v23) {
    const u16x2 above = {0x7F, 0x7F};
    const uint32_t a = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, v01) + above);
    const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, v23) + above);
    const int k0 = static_cast<int>((a << 16) | 3u);
    const int k1 = static_cast<int>((a & 0xFFFF0000u) | 2u);
    const int k2 = static_cast<int>((b << 16) | 1u);
    const int k3 = static_cast<int>(b & 0xFFFF0000u);
    return static_cast<uint32_t>(max(max(max(k0, k1), max(k2, k3)), 0x7F0000)) - 0x7F0000u;
}

// ---------------------------------------------------------------------------
// Layer 1 (1 -> 32 channels, 3x3, pad 1, + bias, ReLU) and its 2x2 max-pool;
// VALU.  One thread per pooled pixel: the 4 x 4 patch once, then 32 channels
// of four outputs.  The full-resolution map (64 bytes per pixel) is never
// written: the backward pass needs the pooled value and the winner only.
// Bound by VALU (4 x 9 multiply-adds per channel and pooled pixel); the
// weights and biases come through the constant address space, so they are
// scalar operands.  With the map written and pooled by a kernel of its own,
// 256 tiles took 127 + 68 us; 65 us in one.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void conv1_pool_kernel(const uint16_t* __restrict__ x,
                                                         const uint16_t* __restrict__ w1b,
                                                         const float* __restrict__ b1,
                                                         uint16_t* __restrict__ p, uint2* __restrict__ idx) {
    typedef const __attribute__((address_space(4))) uint16_t* cw_t;
    typedef const __attribute__((address_space(4))) float* cb_t;
    const cw_t wc = (cw_t)w1b;
    const cb_t bc = (cb_t)b1;
    // two pooled rows of 128 pixels per block
    const int64_t row = static_cast<int64_t>(blockIdx.x) * 2 + (threadIdx.x >> 7);   // n * 32 + y2
    const int x2 = threadIdx.x & 127;
    const int y2 = static_cast<int>(row & 31);
    const uint16_t* img = x + (row >> 5) * (64 * 256);
    const bool aligned = (reinterpret_cast<uintptr_t>(x) & 3) == 0;
    float in[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int y = 2 * y2 - 1 + i;
        const uint16_t* r = img + min(max(y, 0), 63) * 256;
        const bool ok = y >= 0 && y < 64;
        const uint32_t mid = load_pair(r + 2 * x2, aligned);
        const uint16_t l = r[max(2 * x2 - 1, 0)], e = r[min(2 * x2 + 2, 255)];
        in[i][0] = ok && x2 > 0 ? bf2f(l) : 0.0f;
        in[i][1] = ok ? bf2f(static_cast<uint16_t>(mid)) : 0.0f;
        in[i][2] = ok ? bf2f(static_cast<uint16_t>(mid >> 16)) : 0.0f;
        in[i][3] = ok && x2 < 127 ? bf2f(e) : 0.0f;
    }
    uint32_t packed[kCH / 2];
    uint32_t lo = 0, hi = 0;   // bits 0 and 1 of 3 - winner, channel c at bit c in the end
#pragma unroll
    for (int c = 0; c < kCH; c += 2) {
        uint32_t key[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float z[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) z[k] = bc[c + h];
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const float w = bf2f(wc[(c + h) * 9 + t]);
#pragma unroll
                for (int k = 0; k < 4; ++k) z[k] += w * in[(k >> 1) + t / 3][(k & 1) + t % 3];
            }
            key[h] = pool_key(pack2(z[0], z[1]), pack2(z[2], z[3]));
            lo = __builtin_amdgcn_alignbit(key[h], lo, 1);
            hi = __builtin_amdgcn_alignbit(key[h] >> 1, hi, 1);
        }
        packed[c / 2] = __builtin_amdgcn_perm(key[1], key[0], 0x07060302u);
    }
    const int64_t o = row * 128 + x2;
    uint4* dst = reinterpret_cast<uint4*>(p + o * kCH);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        dst[q] = make_uint4(packed[4 * q], packed[4 * q + 1], packed[4 * q + 2], packed[4 * q + 3]);
    idx[o] = make_uint2(~lo, ~hi);
}

// ---------------------------------------------------------------------------
// Gradients of the pre-activations are kept compact: of a 2x2 window only the
// winner's gradient is not zero, so a layer stores, per pooled pixel and
// channel, that one value (bfloat16, zero where the pooled value is 0: ReLU)
// and reads the winner's place from idx.  expand8 gives the values of 8
// channels at window place k: v where the winner is k, else 0.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 expand8(uint4 v, uint32_t b0, uint32_t b1, int k) {
    // winner's bits of the 8 channels, in the low byte
    const uint32_t sel = ((k & 1) ? b0 : ~b0) & ((k & 2) ? b1 : ~b1);
    uint32_t m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(sel), 2 * j, 1));
        const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_sbfe(static_cast<int>(sel), 2 * j + 1, 1));
        m[j] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    }
    return make_uint4(v.x & m[0], v.y & m[1], v.z & m[2], v.w & m[3]);
}

// ---------------------------------------------------------------------------
// 32 -> 32 convolution as an implicit GEMM on MFMA.  A block takes a tile of
// 4 RPW image rows x 32 pixels: its input (with a halo of one pixel) and the
// weights are staged in LDS; a wave takes RPW rows x 32 pixels x 32 output
// channels (2 x 2 tiles of 16 x 16 per row), K = 288 in 9 steps of 32 (one
// tap, all 32 input channels).  An input fragment serves the taps of up to
// three output rows, the wave's 18 weight fragments stay in registers: 54
// fragments read per 144 matrix instructions at RPW = 4 (fragments read from
// global memory for every tap, 36 per 36, ran at the L1's rate: 83 us for
// layer 2 of 256 tiles, 233 TFLOP/s, and its pooling 15 us more; 42 us, 463
// TFLOP/s, for both).  What is left is mostly a block's staging, which only the
// CU's other block overlaps.
//
// FORWARD: x is the layer's input map; bias, ReLU and the 2x2 max-pool follow
// in registers (a lane holds both rows and four neighbouring pixels), p and
// idx are the pooled output.  Otherwise the input gradient: x and idx are the
// layer's compact gradient, wt the flipped and transposed kernel, and p (read
// through pin) the pooled map below: its compact gradient is written to `p`.
// ---------------------------------------------------------------------------
template <int RPW>
struct ConvTile {
    static constexpr int kRows = 4 * RPW;
    static constexpr int kPx = 34;
    uint4 in[(kRows + 2) * kPx * 4];
    uint4 w[9 * kCH * 4];
};

template <int RPW, bool FORWARD>
__global__ __launch_bounds__(256, 2) void conv32_kernel(const uint16_t* __restrict__ x,
                                                        uint2* __restrict__ idx, int H, int W,
                                                        const uint16_t* __restrict__ wt,
                                                        const float* __restrict__ bias,
                                                        const uint16_t* __restrict__ pin,
                                                        uint16_t* __restrict__ p) {
    using Tile = ConvTile<RPW>;
    __shared__ Tile t;
    const int tid = threadIdx.x;
    const int segs = W / 32;
    const int blk = blockIdx.x;
    const int xs = (blk % segs) * 32;
    const int groups = H / Tile::kRows;
    const int y0 = (blk / segs) % groups * Tile::kRows;
    const int64_t n = blk / (segs * groups);
    // 1. stage: the weights as [tap][co][ci], the input with its halo (zeros
    //    outside the image)
    for (int i = tid; i < 9 * kCH * 4; i += 256)
        t.w[i] = *reinterpret_cast<const uint4*>(wt + (((i >> 2) & 31) * 9 + (i >> 7)) * kCH + 8 * (i & 3));
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    if (FORWARD) {
        constexpr int kChunks = (Tile::kRows + 2) * Tile::kPx * 4;
#pragma unroll
        for (int i0 = 0; i0 < kChunks; i0 += 256) {
            const int i = i0 + tid;
            const int r = i / (Tile::kPx * 4), c = i % (Tile::kPx * 4);
            const int y = y0 - 1 + r, xx = xs - 1 + (c >> 2);
            if (i < kChunks)
                t.in[i] = y >= 0 && y < H && xx >= 0 && xx < W
                              ? *reinterpret_cast<const uint4*>(x + ((n * H + y) * W + xx) * kCH + 8 * (c & 3))
                              : zero;
        }
    } else {
        // pooled pixels (y0 / 2 - 1 + r, xs / 2 - 1 + c): each covers tile
        // rows 2 r - 1, 2 r and pixels 2 c - 1, 2 c of the tile
        constexpr int kChunks = (Tile::kRows / 2 + 2) * 18 * 4;
        const int Hp = H / 2, Wp = W / 2;
#pragma unroll
        for (int i0 = 0; i0 < kChunks; i0 += 256) {
            const int i = i0 + tid;
            if (i >= kChunks) break;
            const int q = i & 3, c = (i >> 2) % 18, r = (i >> 2) / 18;
            const int yp = y0 / 2 - 1 + r, xp = xs / 2 - 1 + c;
            uint4 v = zero;
            uint2 b = make_uint2(0u, 0u);
            if (yp >= 0 && yp < Hp && xp >= 0 && xp < Wp) {
                const int64_t o = (n * Hp + yp) * Wp + xp;
                v = *reinterpret_cast<const uint4*>(x + o * kCH + 8 * q);
                b = idx[o];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int tr = 2 * r - 1 + (k >> 1), tp = 2 * c - 1 + (k & 1);
                if (tr >= 0 && tr < Tile::kRows + 2 && tp >= 0 && tp < Tile::kPx)
                    t.in[(tr * Tile::kPx + tp) * 4 + q] = expand8(v, b.x >> (8 * q), b.y >> (8 * q), k);
            }
        }
    }
    __syncthreads();
    // 2. the wave's products
    const int lane = tid & 63;
    const int rb = __builtin_amdgcn_readfirstlane(tid >> 6) * RPW;   // first row of the wave in the tile
    const int row = lane & 15;       // A row (pixel) / B column (channel) within a tile
    const int kq = lane >> 4;        // which 8-channel K slice
    bf16x8 bfr[9][2];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
            bfr[tap][ct] = __builtin_bit_cast(bf16x8, t.w[(tap * kCH + 16 * ct + row) * 4 + kq]);
    f32x4 acc[RPW][2][2];
#pragma unroll
    for (int r = 0; r < RPW; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[r][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // input row i serves output row i - ky: every accumulator takes its taps
    // in raster order
    const uint4* in = t.in + (rb * Tile::kPx + row) * 4 + kq;
#pragma unroll
    for (int i = 0; i < RPW + 2; ++i)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            bf16x8 afr[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
                afr[rt] = __builtin_bit_cast(bf16x8, in[(i * Tile::kPx + 16 * rt + kx) * 4]);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                const int r = i - ky;
                if (r < 0 || r >= RPW) continue;
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct)
                        acc[r][rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr[rt], bfr[3 * ky + kx][ct],
                                                                                 acc[r][rt][ct], 0, 0, 0);
            }
        }
    // 3. D[i][c]: lane holds pixels 16 rt + 4 kq + j (j = 0..3) of channel
    //    16 ct + row.  Neighbouring lanes hold neighbouring channels: of a
    //    pair of pixels the even lane stores the first, the odd lane the
    //    second, two channels in one word.
    const bool odd = lane & 1;
    if (FORWARD) {
        const int Hp = H / 2, Wp = W / 2;
#pragma unroll
        for (int r = 0; r < RPW; r += 2) {
            const int64_t prow = (n * Hp + (y0 + rb + r) / 2) * Wp;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                const int64_t o = prow + xs / 2 + 8 * rt + 2 * kq;   // pixels o, o + 1
                uint32_t key[2][2];   // [ct][pixel]
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    const float bs = bias[16 * ct + row];
                    const f32x4 u = acc[r][rt][ct], v = acc[r + 1][rt][ct];
                    key[ct][0] = pool_key(pack2(u[0] + bs, u[1] + bs), pack2(v[0] + bs, v[1] + bs));
                    key[ct][1] = pool_key(pack2(u[2] + bs, u[3] + bs), pack2(v[2] + bs, v[3] + bs));
                    const uint32_t got = neighbour(odd ? key[ct][0] : key[ct][1]);
                    const uint32_t word = odd ? __builtin_amdgcn_perm(key[ct][1], got, 0x07060302u)
                                              : __builtin_amdgcn_perm(got, key[ct][0], 0x07060302u);
                    *reinterpret_cast<uint32_t*>(p + (o + odd) * kCH + 16 * ct + (row & ~1)) = word;
                }
                // winners: a ballot holds 16 channels of four pixels (kq)
#pragma unroll
                for (int px = 0; px < 2; ++px) {
                    uint32_t bits[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const uint64_t m0 = __ballot((key[0][px] >> b) & 1), m1 = __ballot((key[1][px] >> b) & 1);
                        bits[b] = static_cast<uint32_t>((m0 >> (16 * kq)) & 0xFFFFu) |
                                  (static_cast<uint32_t>((m1 >> (16 * kq)) & 0xFFFFu) << 16);
                    }
                    if (row == 0) idx[o + px] = make_uint2(~bits[0], ~bits[1]);
                }
            }
        }
    } else {
        typedef unsigned short u16x2v __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                    for (int j = 0; j < 4; j += 2) {
                        const f32x4 u = acc[r][rt][ct];
                        const float got = __uint_as_float(neighbour(__float_as_uint(odd ? u[j] : u[j + 1])));
                        const uint32_t word = odd ? pack2(got, u[j + 1]) : pack2(u[j], got);
                        const int64_t o = ((n * H + y0 + rb + r) * W + xs + 16 * rt + 4 * kq + j + odd) * kCH +
                                          16 * ct + (row & ~1);
                        // 0xFFFF where the pooled value is not 0
                        const u16x2v one = {1, 1}, none = {0, 0};
                        const u16x2v a = __builtin_bit_cast(u16x2v, *reinterpret_cast<const uint32_t*>(pin + o));
                        const uint32_t m = __builtin_bit_cast(uint32_t, none - __builtin_elementwise_min(a, one));
                        *reinterpret_cast<uint32_t*>(p + o) = word & m;
                    }
    }
}

// Global average over the 4x16 map, then the 32 -> 1 linear layer: one block
// of 64 threads per tile, thread (half, channel) summing 32 of the 64
// positions (consecutive channels: coalesced), then the halves and the
// channels' products in a fixed order.  logits_out and scores (the sigmoid)
// may be null.
__global__ __launch_bounds__(64) void gap_fc_fwd_kernel(const uint16_t* __restrict__ p4, int N,
                                                        const float* __restrict__ wf,
                                                        const float* __restrict__ bf, float* __restrict__ g,
                                                        float* __restrict__ logits,
                                                        float* __restrict__ logits_out,
                                                        float* __restrict__ scores) {
    __shared__ float hs[2][kCH];
    __shared__ float prod[kCH];
    const int n = blockIdx.x;
    if (n >= N) return;
    const int c = threadIdx.x & (kCH - 1), h = threadIdx.x >> 5;
    float s = 0.0f;
#pragma unroll 8
    for (int q = 32 * h; q < 32 * h + 32; ++q) s += bf2f(p4[(static_cast<int64_t>(n) * 64 + q) * kCH + c]);
    hs[h][c] = s;
    __syncthreads();
    if (threadIdx.x < kCH) {
        const float gc = (hs[0][c] + hs[1][c]) * (1.0f / 64.0f);
        g[n * kCH + c] = gc;
        prod[c] = gc * wf[c];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float lg = bf[0];
        for (int k = 0; k < kCH; ++k) lg += prod[k];
        logits[n] = lg;
        if (logits_out) logits_out[n] = lg;
        if (scores) scores[n] = 1.0f / (1.0f + expf(-lg));
    }
}

// Loss (mean binary cross-entropy with logits), d loss / d logit, and the
// gradients of the linear layer; one block.  For the latter thread (slice,
// channel) sums the tiles of its slice (every 8th), the 33rd column being the
// bias, then the 8 slices in order.
__global__ __launch_bounds__(512) void head_bwd_kernel(const float* __restrict__ logits,
                                                       const float* __restrict__ labels, int N,
                                                       const float* __restrict__ g, float* dlogit,
                                                       float* __restrict__ loss, float* __restrict__ gwf,
                                                       float* __restrict__ gbf) {
    __shared__ float part[256];
    __shared__ float sl[8][kCH + 1];
    const int tid = threadIdx.x;
    if (tid < 256) {
        float s = 0.0f;
        for (int n = tid; n < N; n += 256) {
            const float z = logits[n], y = labels[n];
            s += fmaxf(z, 0.0f) - z * y + log1pf(expf(-fabsf(z)));
            dlogit[n] = (1.0f / (1.0f + expf(-z)) - y) / static_cast<float>(N);
        }
        part[tid] = s;
    }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) part[tid] += part[tid + o];
        __syncthreads();
    }
    if (tid == 0) *loss = part[0] / static_cast<float>(N);
    const int c = tid % 64, q = tid / 64;   // c < 33 used
    if (c <= kCH) {
        float s = 0.0f;
        for (int n = q; n < N; n += 8) s += dlogit[n] * (c < kCH ? g[n * kCH + c] : 1.0f);
        sl[q][c] = s;
    }
    __syncthreads();
    if (tid <= kCH) {
        float s = 0.0f;
        for (int k = 0; k < 8; ++k) s += sl[k][tid];
        if (tid < kCH)
            gwf[tid] = s;
        else
            gbf[0] = s;
    }
}

// Compact gradient of the last layer: the average's gradient where the pooled
// value is not 0.
__global__ void head_grad_kernel(const float* __restrict__ dlogit, const float* __restrict__ wf, int N,
                                 const uint16_t* __restrict__ p4, uint16_t* __restrict__ zc) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= static_cast<int64_t>(N) * 64 * kCH) return;
    const int c = static_cast<int>(i % kCH);
    const int64_t n = i / (64 * kCH);
    zc[i] = p4[i] ? f2bf(dlogit[n] * wf[c] * (1.0f / 64.0f)) : uint16_t(0);
}

// ---------------------------------------------------------------------------
// Weight gradients: GEMMs over pixels (M = output channel, K = pixels, 32 per
// step).  Both operands lie in LDS as [pixel][channel] rows of 64 bytes;
// ds_read_b64_tr_b16 reads them as 16-lane transposes (lane l of 16 gives the
// address of pixel l / 4, channels 4 (l % 4) .. + 3, and gets channel l of
// the four pixels), so any pixel shift is an address.  The two 32-byte halves
// of a row swap places every 8 pixels: the lanes of two K slices then hit
// different banks.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int px_half(int px, int half) { return px * 64 + (((half ^ (px >> 3)) & 1) << 5); }

// Fragment of 16 channels (half) x 32 pixels from px0 on: lane (16 kq + l)
// holds pixels 8 kq .. 8 kq + 7 of channel 16 half + l.
__device__ __forceinline__ bf16x8 pixel_frag(const char* base, int px0, int half, int lane) {
    typedef __attribute__((address_space(3))) bf16x4* lds4;
    const int px = px0 + 8 * (lane >> 4) + ((lane & 15) >> 2);
    const int ch = 8 * (lane & 3);
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(base + px_half(px, half) + ch));
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(base + px_half(px + 4, half) + ch));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const s16x8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// The contiguous range of work units of a block.
__device__ __forceinline__ void unit_range(int units, int* u0, int* u1) {
    *u0 = static_cast<int>(static_cast<int64_t>(units) * blockIdx.x / gridDim.x);
    *u1 = static_cast<int>(static_cast<int64_t>(units) * (blockIdx.x + 1) / gridDim.x);
}

// Layers 2-4: dW[tap][co][ci] = sum over pixels of dz[p][co] x[p + tap][ci],
// and the bias gradient (the sum of the compact gradient).  A unit is a strip
// of 8 rows x 32 pixels; wave (a, b) takes co half a x ci half b for all 9
// taps, and keeps the three input rows a row of dz needs in registers: 4
// fragments read per 9 matrix instructions.  part[blk] = [tap][co][ci], then
// the bias.  (A wave per tap that gathered both operands 2 bytes at a time:
// 151 us for layer 2 of 256 tiles, its bias 33 us; 57 us for both.)
__global__ __launch_bounds__(256, 2) void wgrad32_kernel(const uint16_t* __restrict__ x,
                                                         const uint16_t* __restrict__ zc,
                                                         const uint2* __restrict__ idx, int H, int W,
                                                         int units, float* __restrict__ part) {
    __shared__ uint4 xt[10 * 34 * 4];
    __shared__ uint4 dz[8 * 32 * 4];
    char* xb = reinterpret_cast<char*>(xt);
    char* zb = reinterpret_cast<char*>(dz);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int a = wave >> 1, b = wave & 1;
    const int segs = W / 32, groups = H / 8;
    f32x4 acc[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int u0, u1;
    unit_range(units, &u0, &u1);
    for (int u = u0; u < u1; ++u) {
        const int xs = (u % segs) * 32, y0 = (u / segs) % groups * 8;
        const int64_t n = u / (segs * groups);
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
        constexpr int kChunks = 10 * 34 * 4;
        uint4 v[(kChunks + 255) / 256];
#pragma unroll
        for (int k = 0; k < (kChunks + 255) / 256; ++k) {
            const int i = k * 256 + tid;
            const int y = y0 - 1 + i / 136, xx = xs - 1 + (i % 136) / 4;
            v[k] = i < kChunks && y >= 0 && y < H && xx >= 0 && xx < W
                       ? *reinterpret_cast<const uint4*>(x + ((n * H + y) * W + xx) * kCH + 8 * (i & 3))
                       : zero;
        }
        // one pooled pixel x 8 channels per thread: 4 x 16 x 4
        const int q = tid & 3, c = (tid >> 2) & 15, r = tid >> 6;
        const int64_t o = (n * (H / 2) + y0 / 2 + r) * (W / 2) + xs / 2 + c;
        const uint4 zv = *reinterpret_cast<const uint4*>(zc + o * kCH + 8 * q);
        const uint2 zi = idx[o];
        __syncthreads();   // the last unit's reads are done
#pragma unroll
        for (int k = 0; k < (kChunks + 255) / 256; ++k) {
            const int i = k * 256 + tid;
            const int row = i / 136, px = (i % 136) / 4, h = i & 3;
            if (i < kChunks)
                *reinterpret_cast<uint4*>(xb + row * (34 * 64) + px_half(px, h >> 1) + 16 * (h & 1)) = v[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<uint4*>(zb + (2 * r + (k >> 1)) * (32 * 64) + px_half(2 * c + (k & 1), q >> 1) +
                                      16 * (q & 1)) = expand8(zv, zi.x >> (8 * q), zi.y >> (8 * q), k);
        const uint32_t zw[4] = {zv.x, zv.y, zv.z, zv.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) bsum[j] += bf2f(static_cast<uint16_t>(zw[j >> 1] >> (16 * (j & 1))));
        __syncthreads();
        bf16x8 bfr[3][3];   // [input row mod 3][kx]
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) bfr[i][kx] = pixel_frag(xb + i * (34 * 64), kx, b, lane);
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            const bf16x8 afr = pixel_frag(zb + y * (32 * 64), 0, a, lane);
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
                bfr[(y + 2) % 3][kx] = pixel_frag(xb + (y + 2) * (34 * 64), kx, b, lane);
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
                acc[tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr, bfr[(y + tap / 3) % 3][tap % 3], acc[tap],
                                                                   0, 0, 0);
        }
    }
    float* dst = part + static_cast<int64_t>(blockIdx.x) * kPart32;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            dst[(tap * kCH + 16 * a + 4 * (lane >> 4) + j) * kCH + 16 * b + (lane & 15)] = acc[tap][j];
    // bias: thread (q, pixel) holds 8 channels; the 64 pixels in order
    __syncthreads();
    float* bs = reinterpret_cast<float*>(xt);
#pragma unroll
    for (int j = 0; j < 8; ++j) bs[(tid >> 2) * kCH + 8 * (tid & 3) + j] = bsum[j];
    __syncthreads();
    if (tid < kCH) {
        float s = 0.0f;
        for (int k = 0; k < 64; ++k) s += bs[k * kCH + tid];
        dst[9 * kCH * kCH + tid] = s;
    }
}

// Layer 1 (one input channel): N = the 9 taps and a column of ones, which
// gives the bias gradient (columns 10-15 are zero).  A unit is a pooled row:
// two image rows of 256 pixels, 16 steps of 32 pixels over the four waves.
// part[blk] = [co][tap], then the bias.  (From the full-resolution gradient,
// written and read again: 126 + 88 us for 256 tiles; 31 us.)
__global__ __launch_bounds__(256, 2) void wgrad1_kernel(const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ zc,
                                                        const uint2* __restrict__ idx, int units,
                                                        float* __restrict__ part) {
    constexpr int kXRow = 264;   // uint16 per staged input row: pixel x at x + 2
    __shared__ uint4 dz[2 * 256 * 4];
    __shared__ uint32_t xt[4 * kXRow / 2];
    char* zb = reinterpret_cast<char*>(dz);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const int tap = min(col, 8);
    for (int i = tid; i < 4 * kXRow / 2; i += 256) xt[i] = 0u;   // the pixels outside a row stay 0
    f32x4 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    int u0, u1;
    unit_range(units, &u0, &u1);
    for (int u = u0; u < u1; ++u) {
        const int yp = u & 31;
        const uint16_t* img = x + static_cast<int64_t>(u >> 5) * (64 * 256);
        const bool aligned = (reinterpret_cast<uintptr_t>(x) & 3) == 0;
        const int64_t o0 = static_cast<int64_t>(u) * 128;
        uint32_t xv[2];
        uint4 zv[2];
        uint2 zi[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = k * 256 + tid;            // word i % 128 of input row i / 128
            const int y = 2 * yp - 1 + (i >> 7);
            xv[k] = y >= 0 && y < 64 ? load_pair(img + y * 256 + 2 * (i & 127), aligned) : 0u;
            const int64_t o = o0 + (i >> 2);        // pooled pixel i / 4, channels 8 (i % 4) .. + 7
            zv[k] = *reinterpret_cast<const uint4*>(zc + o * kCH + 8 * (i & 3));
            zi[k] = idx[o];
        }
        __syncthreads();   // the last unit's reads (and the clearing) are done
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = k * 256 + tid;
            xt[(i >> 7) * (kXRow / 2) + 1 + (i & 127)] = xv[k];
            const int q = i & 3, xp = i >> 2;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                *reinterpret_cast<uint4*>(zb + (w >> 1) * (256 * 64) + px_half(2 * xp + (w & 1), q >> 1) +
                                          16 * (q & 1)) = expand8(zv[k], zi[k].x >> (8 * q), zi[k].y >> (8 * q), w);
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int dy = wave >> 1, px0 = 32 * (4 * (wave & 1) + s);
            // B: pixels px0 + 8 kq + kx - 1 .. of input row dy + ky
            const int e = px0 + 8 * kq + tap % 3 + 1;
            const uint32_t* src = xt + (dy + tap / 3) * (kXRow / 2) + (e >> 1);
            uint32_t w[5];
#pragma unroll
            for (int j = 0; j < 5; ++j) w[j] = src[j];
            uint32_t bw[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t v = __builtin_amdgcn_alignbit(w[j + 1], w[j], (e & 1) * 16);
                bw[j] = col < 9 ? v : col == 9 ? 0x3F803F80u : 0u;   // bf16 ones
            }
            const bf16x8 bfr = __builtin_bit_cast(bf16x8, make_uint4(bw[0], bw[1], bw[2], bw[3]));
#pragma unroll
            for (int h = 0; h < 2; ++h)
                acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pixel_frag(zb + dy * (256 * 64), px0, h, lane), bfr,
                                                                 acc[h], 0, 0, 0);
        }
    }
    // D[co][col]: lane holds co = 16 h + 4 kq + j, column col; the waves' sums
    // in order
    __syncthreads();
    float* red = reinterpret_cast<float*>(dz);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[(wave * kCH + 16 * h + 4 * kq + j) * 16 + col] = acc[h][j];
    __syncthreads();
    float* dst = part + static_cast<int64_t>(blockIdx.x) * kPart1;
    for (int i = tid; i < kCH * 10; i += 256) {
        const int co = i / 10, cc = i % 10;
        float s = 0.0f;
        for (int w = 0; w < 4; ++w) s += red[(w * kCH + co) * 16 + cc];
        dst[cc < 9 ? co * 9 + cc : 288 + co] = s;
    }
}

// Sums of the blocks' partials of every layer, in a fixed order: slice s of
// kRedSlices adds its contiguous range of parts in order, then the slices are
// added in order and go to their place in the gradient.  Index i of all
// layers: layer 1's kPart1 values, then kPart32 per further layer.
__global__ __launch_bounds__(256) void reduce_slices_kernel(GradParts gp, float* __restrict__ red) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int sl = blockIdx.y;
    if (i >= kPartAll) return;
    const int l = i < kPart1 ? 0 : 1 + (i - kPart1) / kPart32;
    const int r = l == 0 ? i : (i - kPart1) % kPart32;
    const int stride = l == 0 ? kPart1 : kPart32;
    const int nparts = gp.n[l];
    const float* part = gp.part[l] + r;
    const int b0 = static_cast<int>(static_cast<int64_t>(nparts) * sl / kRedSlices);
    const int b1 = static_cast<int>(static_cast<int64_t>(nparts) * (sl + 1) / kRedSlices);
    float s = 0.0f;
#pragma unroll 4
    for (int b = b0; b < b1; ++b) s += part[static_cast<int64_t>(b) * stride];
    red[static_cast<int64_t>(sl) * kPartAll + i] = s;
}

__global__ __launch_bounds__(256) void reduce_final_kernel(const float* __restrict__ red, Offsets off,
                                                           float* __restrict__ grad) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kPartAll) return;
    float s = 0.0f;
#pragma unroll 8
    for (int k = 0; k < kRedSlices; ++k) s += red[static_cast<int64_t>(k) * kPartAll + i];
    if (i < kPart1) {
        grad[i < 288 ? off.w[0] + i : off.b[0] + i - 288] = s;
        return;
    }
    const int l = 1 + (i - kPart1) / kPart32, r = (i - kPart1) % kPart32;
    if (r >= 9 * kCH * kCH) {
        grad[off.b[l] + r - 9 * kCH * kCH] = s;
    } else {
        const int tap = r / (kCH * kCH), co = (r / kCH) % kCH, ci = r % kCH;
        grad[off.w[l] + (co * kCH + ci) * 9 + tap] = s;
    }
}

// Adam on float32 master weights.
__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int n, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// bf16 copies of the convolution weights in the kernels' layouts.
__global__ void derive_weights_kernel(const float* __restrict__ master, Offsets off,
                                      uint16_t* __restrict__ w1b, uint16_t* __restrict__ wfwd,
                                      uint16_t* __restrict__ wdg) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kCH * 9) w1b[i] = f2bf(master[off.w[0] + i]);   // [co][tap]
    const int per = kCH * 9 * kCH;
    if (i >= 3 * per) return;
    const int l = i / per;          // layers 2..4 -> 0..2
    const int r = i % per;          // master index within [co][ci][ky][kx]
    const int tap = r % 9, ci = (r / 9) % kCH, co = r / (9 * kCH);
    const uint16_t b = f2bf(master[off.w[l + 1] + r]);
    wfwd[l * per + (co * 9 + tap) * kCH + ci] = b;            // [co][tap][ci]
    wdg[l * per + (ci * 9 + (8 - tap)) * kCH + co] = b;       // [ci][flipped tap][co]
}

__global__ void finite_check_kernel(const float* __restrict__ a, int n, int* __restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !isfinite(a[i])) atomicAdd(bad, 1);
}

// ---------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------

static inline unsigned blocks(int64_t n, int t) { return static_cast<unsigned>((n + t - 1) / t); }

hipError_t launch_tiles(const uint16_t* series, int ndm, int64_t nout, int64_t nbx, const TileWidths& W,
                        const dedisp_event* events, int nev, const uint64_t* s1, const double* sqrt_d,
                        uint16_t* tiles, hipStream_t s) {
    if (nev <= 0) return hipSuccess;
    hipLaunchKernelGGL(tiles_kernel, dim3(nev, 64), dim3(256), 0, s, series, ndm, nout, nbx, W, events,
                       s1, sqrt_d, tiles);
    return hipGetLastError();
}

hipError_t launch_derive(const float* master, const Offsets& off, uint16_t* w1b, uint16_t* wfwd,
                         uint16_t* wdg, hipStream_t s) {
    hipLaunchKernelGGL(derive_weights_kernel, dim3(blocks(3 * kCH * 9 * kCH, 256)), dim3(256), 0, s, master,
                       off, w1b, wfwd, wdg);
    return hipGetLastError();
}

// Rows per wave of the convolution at image height H.
template <bool FORWARD>
static void launch_conv32(const uint16_t* x, uint2* idx, int N, int H, int W, const uint16_t* wt, const float* bias,
                          const uint16_t* pin, uint16_t* p, hipStream_t s) {
    if (H % 16 == 0)
        hipLaunchKernelGGL((conv32_kernel<4, FORWARD>), dim3(static_cast<unsigned>(N * (H / 16) * (W / 32))),
                           dim3(256), 0, s, x, idx, H, W, wt, bias, pin, p);
    else
        hipLaunchKernelGGL((conv32_kernel<2, FORWARD>), dim3(static_cast<unsigned>(N * (H / 8) * (W / 32))),
                           dim3(256), 0, s, x, idx, H, W, wt, bias, pin, p);
}

hipError_t launch_forward(const Net& net, const uint16_t* tiles, int N, float* logits, float* scores,
                          hipStream_t s) {
    hipLaunchKernelGGL(conv1_pool_kernel, dim3(static_cast<unsigned>(N) * 16), dim3(256), 0, s, tiles, net.w1b,
                       net.master + net.off.b[0], net.p[0], net.idx[0]);
    for (int l = 1; l < 4; ++l)
        launch_conv32<true>(net.p[l - 1], net.idx[l], N, 64 >> l, 256 >> l, net.wfwd + (l - 1) * kCH * 9 * kCH,
                            net.master + net.off.b[l], nullptr, net.p[l], s);
    hipLaunchKernelGGL(gap_fc_fwd_kernel, dim3(N), dim3(64), 0, s, net.p[3], N, net.master + net.off.wf,
                       net.master + net.off.bf, net.g, net.logits, logits, scores);
    return hipGetLastError();
}

hipError_t launch_backward(const Net& net, const uint16_t* tiles, const float* labels, int N,
                           hipStream_t s) {
    hipLaunchKernelGGL(head_bwd_kernel, dim3(1), dim3(512), 0, s, net.logits, labels, N, net.g, net.dlogit, net.loss,
                       net.grad + net.off.wf, net.grad + net.off.bf);
    hipLaunchKernelGGL(head_grad_kernel, dim3(blocks(static_cast<int64_t>(N) * 64 * kCH, 256)), dim3(256), 0, s,
                       net.dlogit, net.master + net.off.wf, N, net.p[3], net.zc[3]);
    GradParts gp{};
    int64_t at = 0;
    for (int l = 0; l < 4; ++l) {
        const int H = 64 >> l, W = 256 >> l;
        const int units = l == 0 ? N * 32 : N * (H / 8) * (W / 32);
        gp.n[l] = std::min(units, kMaxParts[l]);
        gp.part[l] = net.part + at;
        at += static_cast<int64_t>(kMaxParts[l]) * (l == 0 ? kPart1 : kPart32);
    }
    for (int l = 3; l >= 1; --l) {
        const int H = 64 >> l, W = 256 >> l;
        hipLaunchKernelGGL(wgrad32_kernel, dim3(gp.n[l]), dim3(256), 0, s, net.p[l - 1], net.zc[l], net.idx[l], H, W,
                           N * (H / 8) * (W / 32), gp.part[l]);
        launch_conv32<false>(net.zc[l], net.idx[l], N, H, W, net.wdg + (l - 1) * kCH * 9 * kCH, nullptr,
                             net.p[l - 1], net.zc[l - 1], s);
    }
    hipLaunchKernelGGL(wgrad1_kernel, dim3(gp.n[0]), dim3(256), 0, s, tiles, net.zc[0], net.idx[0], N * 32,
                       gp.part[0]);
    hipLaunchKernelGGL(reduce_slices_kernel, dim3(blocks(kPartAll, 256), kRedSlices), dim3(256), 0, s, gp, net.red);
    hipLaunchKernelGGL(reduce_final_kernel, dim3(blocks(kPartAll, 256)), dim3(256), 0, s, net.red, net.off, net.grad);
    return hipGetLastError();
}

hipError_t launch_adam(const Net& net, float lr, int step, hipStream_t s) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.0f - powf(b1, static_cast<float>(step));
    const float c2 = 1.0f - powf(b2, static_cast<float>(step));
    hipLaunchKernelGGL(adam_kernel, dim3(blocks(kNumParams, 256)), dim3(256), 0, s, net.master, net.grad, net.m,
                       net.v, kNumParams, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_finite_check(const float* a, int n, int* bad, hipStream_t s) {
    hipLaunchKernelGGL(finite_check_kernel, dim3(blocks(n, 256)), dim3(256), 0, s, a, n, bad);
    return hipGetLastError();
}

}  // namespace tk
