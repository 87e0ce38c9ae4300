// Boxcar matched filter, exact sigma-cut and peak finding (paper section 2.3).
//
// Boxcars come from a running sum: B_w[t] = P[t+w] - P[t] with P the prefix
// sum of a dedispersed series (the leading window; every width shares the
// valid length n_bx = nout - w_max + 1).  A block owns one (DM, segment of
// L start positions); it scans its window of the series in LDS with a
// wave-shuffle prefix sum -- only differences of P are used, so a segment
// needs no carry from the segments before it -- and evaluates every width
// from that one scan.  All boxcar arithmetic is uint32 modular (exact, since
// each B_w < 2^31).
//
// The sigma-cut is decided in integers: per (width, DM) series the exact sums
// S1 = sum B and S2 = sum B^2 give D = n S2 - S1^2, and a sample is above the
// cut iff B >= B_thr = ceil((S1 + isqrt(floor(k^2 D)) + 1) / n), k being the
// exact binary value of the float threshold (128/256-bit integer helpers).
//
// Events (section 2.3: each maximal run of above-cut samples of one series
// is one event) are compacted deterministically: count run starts per
// (width, DM, segment) and per series, exclusive scan over the series, then
// write each event at its series' slot plus the counts of the segments before
// (a series of many segments: at the scan of all counts) -- the output order is (width, DM, t_start) without any sort.  Only the
// (DM, segment)s whose largest boxcar reaches the cut are counted, and only
// those with events are written: both passes work through lists of them.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dedisp_internal.hpp"
#include "intmath.hpp"
#include "search_internal.hpp"

namespace {

constexpr int kThreads = 256;
// Threads per block of the list-driven count and write passes (see list_threads).
constexpr int kFewThreads = 1024, kMidThreads = 512;
// ----------------------------------------------------------------------------
// Block-level helpers.
// ----------------------------------------------------------------------------

// Exclusive prefix of one value per thread over the block (uint32, modular).
template <int NT = kThreads>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wave_tot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    uint32_t base = 0;
    if (NT <= 256) {
        for (int i = 0; i < wave; ++i) base += wave_tot[i];
    } else {
        // the totals of the waves before this one, one per lane
        uint32_t t = lane < wave ? wave_tot[lane] : 0u;
#pragma unroll
        for (int o = 1; o < NT / 64; o <<= 1) t += static_cast<uint32_t>(__shfl_xor(static_cast<int>(t), o, NT / 64));
        base = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(t)));
    }
    __syncthreads();
    return base + x - v;
}

// Fill pl[0..n) with the running sum of the series values s[first + i]
// (values outside [0, nout) count as 0): pl[i] = sum_{k<i} s[first+k].
// Loads and LDS reads are issued in batches of kBatch per thread so that
// their latencies overlap.
constexpr int kBatch = 12;
// Word 3 of a raw (unstrided) buffer resource on gfx9-family GPUs: 32-bit
// data format, no swizzle; loads are range-checked against the byte count.
constexpr int kRowRsrcWord3 = 0x00020000;

// One sample of a series row through a buffer resource whose range is the
// row: offsets outside it (negative ones wrap to huge) read as 0.
__device__ __forceinline__ uint32_t row_load(__amdgpu_buffer_rsrc_t rs, int byte_off, uint16_t*) {
    return __builtin_amdgcn_raw_buffer_load_b16(rs, byte_off, 0, 0);
}
__device__ __forceinline__ uint32_t row_load(__amdgpu_buffer_rsrc_t rs, int byte_off, int32_t*) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, byte_off, 0, 0);
}

template <int NT = kThreads, typename T>
__device__ void load_prefix(const T* __restrict__ row, int64_t nout, int64_t first, int n,
                            uint32_t* pl, uint32_t* wave_tot, uint32_t* vmax = nullptr) {
    // coalesced load of the raw values into pl[1..n); the launchers keep a
    // row (and first + n) below 2^31 bytes
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(row), 0, static_cast<int>(nout * static_cast<int64_t>(sizeof(T))), kRowRsrcWord3);
    const int off0 = static_cast<int>(first) * static_cast<int>(sizeof(T));
    uint32_t m = 0;
    // full batches (every index below n - 1) store without checks; the last,
    // partial one checks each index
    int base = threadIdx.x;
    for (; base + (kBatch - 1) * NT < n - 1; base += kBatch * NT) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            v[k] = row_load(rs, off0 + (base + k * NT) * static_cast<int>(sizeof(T)),
                            static_cast<T*>(nullptr));
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            pl[base + k * NT + 1] = v[k];
            m = max(m, v[k]);
        }
    }
    if (base < n - 1) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = base + k * NT;
            v[k] = row_load(rs, off0 + i * static_cast<int>(sizeof(T)), static_cast<T*>(nullptr));
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = base + k * NT;
            if (i < n - 1) {
                pl[i + 1] = v[k];
                m = max(m, v[k]);
            }
        }
    }
    if (vmax) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m = max(m, static_cast<uint32_t>(__shfl_xor(m, o, 64)));
    }
    __syncthreads();
    // after the barrier, which orders them after the caller's clearing of
    // *vmax; the barrier at the end orders them before its readers
    if (vmax && (threadIdx.x & 63) == 0) atomicMax(vmax, m);
    // each thread scans a contiguous chunk (odd chunk stride: no bank conflicts)
    const int chunk = (((n - 1) + NT - 1) / NT) | 1;
    const int lo = 1 + threadIdx.x * chunk;
    const int hi = min(n, lo + chunk);
    // full batches without checks, then one checked remainder batch
    const int full_end = lo + ((max(hi - lo, 0)) / kBatch) * kBatch;
    uint32_t sum = 0;
    for (int i0 = lo; i0 < full_end; i0 += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = pl[i0 + k];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) sum += v[k];
    }
    if (full_end < hi) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = full_end + k < hi ? pl[full_end + k] : 0u;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) sum += v[k];
    }
    const uint32_t scan_base = block_exclusive_scan<NT>(sum, wave_tot);
    uint32_t run = scan_base;
    for (int i0 = lo; i0 < full_end; i0 += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = pl[i0 + k];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            run += v[k];
            pl[i0 + k] = run;
        }
    }
    if (full_end < hi) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = full_end + k < hi ? pl[full_end + k] : 0u;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            run += v[k];
            if (full_end + k < hi) pl[full_end + k] = run;
        }
    }
    if (threadIdx.x == 0) pl[0] = 0u;
    __syncthreads();
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ----------------------------------------------------------------------------
// Kernels.
// ----------------------------------------------------------------------------

// Materialised boxcars for a DM sub-range (tests and inspection).
template <typename T>
__global__ __launch_bounds__(kThreads) void boxcar_kernel(const T* __restrict__ in, int64_t nout,
                                                          int64_t nbx, dd::Widths W, int dm_first,
                                                          int L, int32_t* __restrict__ out,
                                                          int dm_count) {
    extern __shared__ uint32_t pl[];
    __shared__ uint32_t wave_tot[kThreads / 64];
    const int d = dm_first + blockIdx.y;
    const int64_t s0 = static_cast<int64_t>(blockIdx.x) * L;
    const int n = L + W.w[W.n - 1] + 1;
    load_prefix(in + static_cast<int64_t>(d) * nout, nout, s0 - 1, n, pl, wave_tot);
    for (int i = threadIdx.x; i < L; i += kThreads) {
        const int64_t t = s0 + i;
        if (t >= nbx) break;
        const uint32_t p0 = pl[i + 1];
        for (int wi = 0; wi < W.n; ++wi)
            out[(static_cast<int64_t>(wi) * dm_count + blockIdx.y) * nbx + t] =
                static_cast<int32_t>(pl[i + 1 + W.w[wi]] - p0);
    }
}

// Baseline (red-noise) removal by a running mean (section 2.3, first
// paragraph), streamed: out[t] = s[t + R] - floor(W(t) / (2R + 1)) + offset,
// W(t) = sum_{j=t}^{t+2R} s[j], integer and exact.  One wave walks kBlSeg
// outputs of one row in steps of `bl_rows` rows of 256, a lane taking 4
// consecutive outputs of each.  The window slides: W(t + 1) - W(t) =
// s[t + 2R + 1] - s[t], so W(t) is W(t0) plus an exclusive wave prefix (DPP
// scan) of those differences, one scan per 256 outputs; every sample comes once
// through the front cursor and again, from cache, through the middle and back
// ones.  Integers modulo 2^32 are exact as every window sum is below 2^31; the
// division is a high multiply and a shift.
// Bound by memory: the back cursor's samples have to outlast 2R + 1 others of
// every stream in an XCD's 4 MB, so the outputs go past it (non-temporal stores,
// from 128-byte boundaries of the output on, as a part of a line that leaves
// early costs a second write), and long steps keep fewer waves on wider
// accesses.  Survey series (1200 x 503812 samples of 16 bits, R = 2048), us: one
// output per lane, 1024 per step 733; 4 per lane, steps of 1024 / 2048 / 4096
// outputs 706 / 688 / 660; of 4096 with non-temporal stores 621, and aligned
// 599 (R = 30 at 1000 x 333333: 364 before, 372 and 324).  32-bit samples: steps
// of 2048, the same bytes in registers (1000 x 333333, R = 2048: 817 before, 661).
constexpr int kBlSeg = 16384;       // outputs per wave
template <typename T>
constexpr int bl_rows() {
    return sizeof(T) == 2 ? 16 : 8;   // rows of 256 outputs per step
}
constexpr int kBlShortRows = 4;     // of the shorter steps that follow
constexpr int kBlTailRows = 16;     // rows of 64 outputs per step at a row's end
// Rows with fewer outputs take the steps of a row's end alone, without the outputs
// before a line and the long steps, and read past the row's end, which a buffer
// load answers with 0, in place of clamping every index.  65535 rows of 300 outputs,
// us: 80 with the long form, 45; 20000 of 1000 32 and 24, of 1500 41 and 34, of 2200
// 52 and 48 (16-bit samples; 50 and 50 at R = 500), 32-bit samples 38 and 37 of
// 1300, 49 and 60 of 1800.
template <typename T>
constexpr int64_t bl_brief() {
    return sizeof(T) == 2 ? 2048 : 1600;
}

// Inclusive prefix sum over the 64 lanes of a wave: shifts within each row
// of 16 lanes, then the row totals carried across rows.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x111, 0xF, 0xF, true));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x112, 0xF, 0xF, true));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x114, 0xF, 0xF, true));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x118, 0xF, 0xF, true));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x142, 0xA, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x143, 0xC, 0xF, false));
    return x;
}

// Two uint16 values packed in a 32-bit word.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// c + the two 16-bit halves of v (one v_dot2_u32_u16 with the vector (1, 1)).
__device__ __forceinline__ uint32_t add_halves(uint32_t v, uint32_t c) {
    const u16x2 one = {1, 1};
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, v), one, c, false);
}

// The same running sums of a uint16 series window, for rows of a multiple of
// 4 samples from an 8-byte aligned series, without the LDS passes of the
// scan.  The window is read from a = first rounded down to a multiple of 4
// (and not below 0) in kRounds rounds of 1024 samples; in round i thread t
// takes samples a + 4(256 i + t) .. + 3 with one 8-byte load (every load lies
// wholly inside the row or wholly past its end, where it reads 0).  The
// thread sums its four (two packed 16-bit dot products), a DPP scan per
// round gives the wave's prefix, one DPP scan of the 36 wave totals in
// (round, wave) order gives the block's, and each group of four running
// sums goes to LDS with one 16-byte store.  The samples
// between a and first and past the window enter the sums too: only
// differences of the running sums are used, and the largest value only gates
// the fast path, so both stay exact.  lds needs kRunWords words.
// Returns ps with ps[i] - ps[j] = the sum of s[first + j .. first + i).
constexpr int kRounds = 9;
constexpr int kRunWords = 4 + 4 * kThreads * kRounds;

__device__ __forceinline__ const uint32_t* load_prefix_runs(const uint16_t* __restrict__ row,
                                                            int64_t nout, int64_t first, uint32_t* lds,
                                                            uint32_t* round_tot, uint32_t* vmax) {
    // first >= -1; the window of the first segment (first = -1) starts at 0
    // with shift -1 (its sample -1 counts as 0)
    const int64_t a = first < 0 ? 0 : first - (first & 3);
    const int shift = static_cast<int>(first - a);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(row), 0, static_cast<int>(nout * 2), kRowRsrcWord3);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int off0 = static_cast<int>(a) * 2 + static_cast<int>(threadIdx.x) * 8;
    uint32_t v[2 * kRounds];
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(rs, off0 + i * (8 * kThreads), 0, 0);
        v[2 * i] = x[0];
        v[2 * i + 1] = x[1];
    }
    u16x2 m2 = {0, 0};
    uint32_t excl[kRounds];
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        m2 = __builtin_elementwise_max(m2, __builtin_elementwise_max(__builtin_bit_cast(u16x2, v[2 * i]),
                                                                     __builtin_bit_cast(u16x2, v[2 * i + 1])));
        const uint32_t c = add_halves(v[2 * i + 1], add_halves(v[2 * i], 0u));
        const uint32_t incl = wave_incl_scan(c);
        excl[i] = incl - c;
        if (lane == 63) round_tot[i * (kThreads / 64) + wave] = incl;
    }
    uint32_t m = max(static_cast<uint32_t>(m2.x), static_cast<uint32_t>(m2.y));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = max(m, static_cast<uint32_t>(__shfl_xor(m, o, 64)));
    __syncthreads();
    // after the barrier (ordered after the caller's clearing of *vmax) and
    // before the final one (ordered before its readers)
    if (lane == 0) atomicMax(vmax, m);
    // The block's prefix before (round i, wave w) is the exclusive scan of
    // the wave totals in (round, wave) order: lane 4 i + w of every wave
    // scans them, and each wave reads its rounds' entries.
    const uint32_t tv = lane < kRounds * (kThreads / 64) ? round_tot[lane] : 0u;
    const uint32_t tin = wave_incl_scan(tv);
    const uint32_t tex = tin - tv;
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const uint32_t pre = static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(tex), i * (kThreads / 64) + wave));
        const uint32_t run = pre + excl[i];
        // lds[3 + k] = sum of s[a .. a + k): sample a + 4g + j ends at 4 + 4g + j
        const uint32_t w0 = run + (v[2 * i] & 0xFFFFu);
        const uint32_t w1 = add_halves(v[2 * i], run);
        const uint32_t w2 = w1 + (v[2 * i + 1] & 0xFFFFu);
        const uint32_t w3 = add_halves(v[2 * i + 1], w1);
        *reinterpret_cast<uint4*>(lds + 4 + 4 * (i * kThreads + threadIdx.x)) = make_uint4(w0, w1, w2, w3);
    }
    if (threadIdx.x == 0) {
        lds[2] = 0u;
        lds[3] = 0u;
    }
    __syncthreads();
    return lds + 3 + shift;
}

// Four consecutive samples at any element boundary, one 8- or 16-byte access.
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Four {
    T v[4];
};

// Writes o[0 .. 3], past the caches.
template <typename U>
__device__ __forceinline__ void bl_store(U* o, const int (&r)[4]) {
    typedef U V4 __attribute__((ext_vector_type(4), aligned(sizeof(U))));
    const V4 q = {static_cast<U>(r[0]), static_cast<U>(r[1]), static_cast<U>(r[2]), static_cast<U>(r[3])};
    __builtin_nontemporal_store(q, reinterpret_cast<V4*>(o));
}

template <typename T, typename U, bool SHORT>
__global__ __launch_bounds__(kThreads) void baseline_kernel(const T* __restrict__ in, int ndm,
                                                            int64_t nout, int64_t nres, int radius,
                                                            int offset, int64_t nseg, uint32_t magic,
                                                            int shift, U* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    // the wave's item, in scalar registers (so is everything derived from it)
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t item = static_cast<int64_t>(blockIdx.x) * (kThreads / 64) + wave;
    if (item >= static_cast<int64_t>(ndm) * nseg) return;   // whole waves
    const int d = static_cast<int>(item / nseg);
    const T* row = in + static_cast<int64_t>(d) * nout;
    U* o = out + static_cast<int64_t>(d) * nres;
    // outputs before the row's first 128-byte line of 64-element pieces; the
    // row's first wave takes them, and every segment starts on such a boundary
    const int head = SHORT ? 0 : static_cast<int>(min<int64_t>(
        -static_cast<int64_t>(reinterpret_cast<uintptr_t>(o) / sizeof(U)) & 63, nres));
    const int64_t seg = item % nseg;
    const int64_t t0 = seg == 0 ? 0 : seg * kBlSeg + head;
    const int64_t t1 = min<int64_t>((seg + 1) * kBlSeg + head, nres);
    if (t0 >= t1) return;
    const int win = 2 * radius + 1;
    // floor(sum / win), exact for sum < 2^31 (see the launcher)
    auto mean = [&](uint32_t sum) {
        return static_cast<int>(win == 1 ? sum : __umulhi(sum, magic) >> shift);
    };
    // W(t0): the sum of s[t0 .. t0 + 2R]
    uint32_t acc = 0;
    {
        const T* p = row + t0;
        int i = 0;
        for (; i + 1024 <= win; i += 1024) {
            Four<T> f[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = *reinterpret_cast<const Four<T>*>(p + i + 256 * k + 4 * lane);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc += static_cast<uint32_t>(f[k].v[j]);
        }
        uint32_t v[16];   // up to 1023 left: all the loads at once
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = static_cast<uint32_t>(p[min(i + 64 * k + lane, win - 1)]);
#pragma unroll
        for (int k = 0; k < 16; ++k) acc += i + 64 * k + lane < win ? v[k] : 0u;
    }
    uint32_t wcur = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wave_incl_scan(acc)), 63));
    int64_t tc = t0;
    if (!SHORT && seg == 0 && head > 0) {
        const int t = min(lane, head - 1);
        const uint32_t bk = static_cast<uint32_t>(row[t]);
        const uint32_t fr = static_cast<uint32_t>(row[min<int64_t>(t + win, nout - 1)]);
        const int md = static_cast<int>(row[t + radius]);
        const uint32_t delta = lane < head ? fr - bk : 0u;
        const uint32_t incl = wave_incl_scan(delta);
        if (lane < head) o[lane] = static_cast<U>(md - mean(wcur + incl - delta) + offset);
        wcur += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
        tc = head;
    }
    // whole steps, every sample they touch inside the row
    auto walk = [&](auto rows_c) {
        constexpr int rows = decltype(rows_c)::value, step = 256 * rows;
        for (; tc + step <= t1 && tc + step + win <= nout; tc += step) {
            const T* p = row + tc + 4 * lane;
            Four<T> b[rows], f[rows], m[rows];
#pragma unroll
            for (int i = 0; i < rows; ++i) {
                b[i] = *reinterpret_cast<const Four<T>*>(p + 256 * i);
                f[i] = *reinterpret_cast<const Four<T>*>(p + 256 * i + win);
                m[i] = *reinterpret_cast<const Four<T>*>(p + 256 * i + radius);
            }
#pragma unroll
            for (int i = 0; i < rows; ++i) {
                uint32_t w[5];   // W(t + j) - W(first of the row)
                w[0] = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    w[j + 1] = w[j] + static_cast<uint32_t>(f[i].v[j]) - static_cast<uint32_t>(b[i].v[j]);
                const uint32_t incl = wave_incl_scan(w[4]);
                const uint32_t first = wcur + incl - w[4];
                int r[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    r[j] = static_cast<int>(m[i].v[j]) - mean(first + w[j]) + offset;
                bl_store(o + tc + 256 * i + 4 * lane, r);
                wcur += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
            }
        }
    };
    if (!SHORT) {
        walk(std::integral_constant<int, bl_rows<T>()>{});
        walk(std::integral_constant<int, kBlShortRows>{});
    }
    // the rest, one output per lane and row.  Indices are clamped to the row;
    // the sample that enters after the row's last output lies past its end and
    // reaches no output.
    struct Tail {
        uint32_t bk[kBlTailRows], fr[kBlTailRows];
        int md[kBlTailRows];
    };
    auto load = [&](Tail& q, int64_t at) {
        if constexpr (SHORT) {
            // loads at one offset per lane and cursor; past the row's end they read 0
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<T*>(row), 0, static_cast<int>(nout * static_cast<int64_t>(sizeof(T))), kRowRsrcWord3);
            constexpr int sz = static_cast<int>(sizeof(T));
            const int base = (static_cast<int>(at) + lane) * sz;
#pragma unroll
            for (int i = 0; i < kBlTailRows; ++i) {
                q.bk[i] = row_load(rs, base + 64 * i * sz, static_cast<T*>(nullptr));
                q.fr[i] = row_load(rs, base + win * sz + 64 * i * sz, static_cast<T*>(nullptr));
                q.md[i] = static_cast<int>(row_load(rs, base + radius * sz + 64 * i * sz, static_cast<T*>(nullptr)));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < kBlTailRows; ++i) {
            const int64_t t = min<int64_t>(at + 64 * i + lane, t1 - 1);
            q.bk[i] = static_cast<uint32_t>(row[t]);
            q.fr[i] = static_cast<uint32_t>(row[min<int64_t>(t + win, nout - 1)]);
            q.md[i] = static_cast<int>(row[t + radius]);
        }
    };
    if (tc >= t1) return;
    Tail cur, nxt;
    load(cur, tc);
    for (;;) {
        const int64_t next = tc + 64 * kBlTailRows;
        if (next < t1) load(nxt, next);   // in flight while this one is computed
#pragma unroll
        for (int i = 0; i < kBlTailRows; ++i) {
            if (SHORT && tc + 64 * i >= t1) break;
            const int64_t t = tc + 64 * i + lane;
            const uint32_t delta = cur.fr[i] - cur.bk[i];
            const uint32_t incl = wave_incl_scan(delta);
            if (t < t1) o[t] = static_cast<U>(cur.md[i] - mean(wcur + incl - delta) + offset);
            wcur += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
        }
        if (next >= t1) break;
        tc = next;
        cur = nxt;
    }
}

// Pass 1: per (width, DM, segment) partial sums of B and B^2 and the largest B.
// Per thread and width at most L/256 <= 32 positions are summed in registers.
// When every B of the block's window is below 2^26 (the largest raw value
// times w_max says so) a 64-bit square sum cannot overflow even after the
// 64-lane reduction; otherwise the sums are carried as 128-bit values.
template <bool SMALL>
__device__ __forceinline__ void wave_totals(uint64_t s1, uint64_t lo, uint64_t hi, uint32_t mx, uint64_t* s1_out,
                                            u128* s2_out, uint32_t* mx_out) {
    s1 = wave_sum_u64(s1);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = max(mx, static_cast<uint32_t>(__shfl_xor(mx, o, 64)));
    if (SMALL) {
        *s2_out = wave_sum_u64(lo);
    } else {
        const uint64_t a = wave_sum_u64(lo & 0xFFFFFFFFull);
        const uint64_t b = wave_sum_u64(lo >> 32);
        const uint64_t c = wave_sum_u64(hi);
        *s2_out = static_cast<u128>(a) + (static_cast<u128>(b) << 32) + (static_cast<u128>(c) << 64);
    }
    *s1_out = s1;
    *mx_out = mx;
}

template <bool SMALL>
__device__ __forceinline__ void width_sums(const uint32_t* pl, int npos, int w, uint64_t* s1_out,
                                           u128* s2_out, uint32_t* mx_out) {
    uint64_t s1 = 0, lo = 0, hi = 0;
    uint32_t mx = 0;
    for (int i = threadIdx.x; i < npos; i += kThreads) {
        const uint32_t b = pl[i + 1 + w] - pl[i + 1];
        s1 += b;
        const uint64_t sq = static_cast<uint64_t>(b) * b;   // one v_mad_u64_u32 when SMALL
        lo += sq;
        if (!SMALL) hi += lo < sq ? 1u : 0u;
        mx = max(mx, b);
    }
    wave_totals<SMALL>(s1, lo, hi, mx, s1_out, s2_out, mx_out);
}

// Positions per thread in the fast path of a full segment.
constexpr int kPerThread = 32;

// Row stride, in values, of the per-width rows in the fast path's block
// reductions through LDS: the 16 lanes of one width read 16 consecutive
// values, and the next width's lanes start 16 banks further on for 4-byte
// values (32 for 8-byte ones).
constexpr int kRedStride = kThreads + 16;

// Sum / maximum over the 16 lanes of a DPP row (every lane gets it): swaps
// of neighbours and of pairs within each quad, then rotations by 4 and 8.
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x, int ctrl_sel) {
    switch (ctrl_sel) {
        case 0: return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xF, 0xF, false));
        case 1: return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x4E, 0xF, 0xF, false));
        case 2: return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x124, 0xF, 0xF, false));
        default: return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x128, 0xF, 0xF, false));
    }
}
__device__ __forceinline__ uint64_t row_sum_u64(uint64_t v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint64_t o = (static_cast<uint64_t>(dpp_u32(static_cast<uint32_t>(v >> 32), c)) << 32) |
                           dpp_u32(static_cast<uint32_t>(v), c);
        v += o;
    }
    return v;
}
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) v = max(v, dpp_u32(v, c));
    return v;
}

// Fast path of a full segment with small values and NW (compile-time)
// widths: positions outer, widths inner, every partial sum in registers, then
// one block reduction through LDS (which the running sums no longer need).
template <int NW>
__device__ __forceinline__ void stats_full_nw(const uint32_t* ps, uint32_t* pl, const dd::Widths& W,
                                              const dd::PeaksWs& ws, int64_t idx0, int64_t stride) {
    uint64_t s2[NW];
    uint32_t mx[NW];
    int woff[NW];
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) {
        mx[wi] = 0;
        s2[wi] = 0;
        woff[wi] = W.w[wi];
    }
    const uint32_t* base = ps + 1 + threadIdx.x;
#pragma unroll 8
    for (int j = 0; j < kPerThread; ++j) {
        const uint32_t p0 = base[j * kThreads];
#pragma unroll
        for (int wi = 0; wi < NW; ++wi) {
            const uint32_t b = base[j * kThreads + woff[wi]] - p0;
            s2[wi] += static_cast<uint64_t>(b) * b;
            mx[wi] = max(mx[wi], b);
        }
    }
    // Sum of the segment's boxcars by telescoping: with P the running sums,
    //   sum_{j<L} (P[j+1+w] - P[j+1]) = sum_{k=1..w} (P[L+k] - P[k]),
    // each term D(k) a sum of L samples (below 2^32 by the caller's check).
    // (After the main loop, so that its registers are free there.)  Lane l
    // of a wave takes k = k0 + l, 64 consecutive values, and a DPP scan of
    // D's two 16-bit halves (each below 2^22 over 64 lanes) gives their
    // inclusive prefix.  Lane wi < NW keeps width wi's sum: it takes the
    // prefix at lane w - k0, clamped to 63 (every k of the wave when
    // k0 + 63 <= w), and nothing when w < k0.
    constexpr int L = kPerThread * kThreads;
    const int lane = threadIdx.x & 63;
    int myw = 0;   // this lane's width (lanes >= NW: none)
#pragma unroll
    for (int wi = 0; wi < NW; ++wi)
        if (lane == wi) myw = woff[wi];
    uint64_t s1 = 0;
    for (int k0 = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) & ~63) + 1;
         k0 <= woff[NW - 1]; k0 += kThreads) {
        const int k = k0 + lane;
        const int kc = min(k, woff[NW - 1]);   // k past the widest width reads in range, counts 0
        const uint32_t dk = k <= woff[NW - 1] ? ps[L + kc] - ps[kc] : 0u;
        const uint32_t lo = wave_incl_scan(dk & 0xFFFFu);
        const uint32_t hi = wave_incl_scan(dk >> 16);
        const int l = myw - k0;
        const int src = min(max(l, 0), 63);
        const uint32_t glo = static_cast<uint32_t>(__shfl(static_cast<int>(lo), src, 64));
        const uint32_t ghi = static_cast<uint32_t>(__shfl(static_cast<int>(hi), src, 64));
        if (l >= 0) s1 += static_cast<uint64_t>(glo) + (static_cast<uint64_t>(ghi) << 16);
    }
    __syncthreads();   // the running sums are no longer needed: reuse pl
    // Per width, thread (wi, l) = 16 wi + l takes partials l, l+16, ..., of
    // width wi (rows of kRedStride values: the next width's 16 lanes start
    // on other banks), then the 16 lanes of the width, one DPP row, sum
    // their values; lane 16 wi ends with width wi's total.
    const int t = threadIdx.x;
    uint64_t* r = reinterpret_cast<uint64_t*>(pl);
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) r[wi * kRedStride + t] = s2[wi];
    __syncthreads();
    uint64_t acc = 0;
    if (t < NW * 16) {
        const uint64_t* q = r + (t / 16) * kRedStride + (t % 16);
#pragma unroll
        for (int k = 0; k < 16; ++k) acc += q[16 * k];
    }
    acc = row_sum_u64(acc);
    __syncthreads();
    // maxima, and the sums (one per wave and width)
    uint32_t* rm = pl + 2 * NW * kRedStride;
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) rm[wi * kRedStride + t] = mx[wi];
    if (lane < NW) r[(t >> 6) * NW + lane] = s1;
    __syncthreads();
    uint64_t a1 = 0;
    uint32_t am = 0;
    if (t < NW * 16) {
        const uint32_t* qm = rm + (t / 16) * kRedStride + (t % 16);
#pragma unroll
        for (int k = 0; k < 16; ++k) am = max(am, qm[16 * k]);
        if ((t & 15) == 0) {
#pragma unroll
            for (int v = 0; v < kThreads / 64; ++v) a1 += r[v * NW + (t >> 4)];
        }
    }
    am = row_max_u32(am);
    // every global write after the last barrier (a barrier would wait for
    // them)
    if (t < NW * 16 && (t & 15) == 0) {
        const int64_t i = idx0 + (t >> 4) * stride;
        ws.part_s2lo[i] = acc;
        ws.part_s2hi[i] = 0u;   // below 2^63 (see the caller)
        ws.part_s1[i] = a1;
        ws.part_max[i] = am;
    }
}

template <typename T, int NW>
__global__ __launch_bounds__(kThreads) void boxcar_stats_kernel(const T* __restrict__ in,
                                                                int64_t nout, int64_t nbx,
                                                                dd::Widths W, int L, int nseg,
                                                                int runs, dd::PeaksWs ws) {
    // the dynamic LDS as 16-byte elements, so that its base is 16-byte
    // aligned (16-byte LDS accesses in the window loads)
    extern __shared__ uint4 pl16[];
    uint32_t* pl = reinterpret_cast<uint32_t*>(pl16);
    __shared__ uint32_t wave_tot[kThreads / 64];
    __shared__ __attribute__((aligned(16))) uint32_t round_tot[kRounds * (kThreads / 64)];
    __shared__ uint64_t red1[kThreads / 64][dd::kMaxWidths];
    __shared__ u128 red2[kThreads / 64][dd::kMaxWidths];
    __shared__ uint32_t redm[kThreads / 64][dd::kMaxWidths];
    __shared__ uint32_t vmax;
    const int d = blockIdx.y;
    const int seg = blockIdx.x;
    const int64_t s0 = static_cast<int64_t>(seg) * L;
    const int w_max = W.w[W.n - 1];
    const int n = L + w_max + 1;
    if (threadIdx.x == 0) vmax = 0;
    // the window's running sums: ps[i] - ps[j] = sum of s[s0 - 1 + j .. s0 - 1 + i)
    const uint32_t* ps = pl;
    if constexpr (std::is_same<T, uint16_t>::value) {
        if (runs)
            ps = load_prefix_runs(in + static_cast<int64_t>(d) * nout, nout, s0 - 1, pl, round_tot, &vmax);
        else
            load_prefix(in + static_cast<int64_t>(d) * nout, nout, s0 - 1, n, pl, wave_tot, &vmax);
    } else {
        load_prefix(in + static_cast<int64_t>(d) * nout, nout, s0 - 1, n, pl, wave_tot, &vmax);
    }
    const int npos = static_cast<int>(min<int64_t>(L, nbx - s0));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t bmax = static_cast<uint64_t>(vmax) * static_cast<uint64_t>(w_max);
    // every boxcar below 2^26: a wave's 64-bit square sum (at most 64 x 32
    // squares below 2^52) cannot overflow
    const bool small = bmax < (uint64_t(1) << 26);
    // full fast path: a whole segment whose square sum, over all its
    // kPerThread * 256 = 2^13 positions, stays below 2^13 * 2^50 = 2^63 (every
    // boxcar below 2^25), and every sum of L consecutive samples below 2^32
    // (for the telescoped S1)
    const bool full = bmax < (uint64_t(1) << 25) && npos == kPerThread * kThreads &&
                      vmax < (1u << 19) && L == kPerThread * kThreads;
    constexpr int NWS = NW > 0 ? NW : 1;
    if (NW > 0 && full) {
        // partial of width wi at idx0 + wi * stride
        stats_full_nw<NWS>(ps, pl, W, ws, static_cast<int64_t>(d) * nseg + seg,
                           static_cast<int64_t>(gridDim.y) * nseg);
        return;
    }
    for (int wi = 0; wi < W.n; ++wi) {
        uint64_t s1;
        u128 s2;
        uint32_t mx;
        if (small)
            width_sums<true>(ps, npos, W.w[wi], &s1, &s2, &mx);
        else
            width_sums<false>(ps, npos, W.w[wi], &s1, &s2, &mx);
        if (lane == 0) {
            red1[wave][wi] = s1;
            red2[wave][wi] = s2;
            redm[wave][wi] = mx;
        }
    }
    __syncthreads();
    if (threadIdx.x < W.n) {
        const int wi = threadIdx.x;
        uint64_t s1 = 0;
        u128 s2 = 0;
        uint32_t mx = 0;
        for (int v = 0; v < kThreads / 64; ++v) {
            s1 += red1[v][wi];
            s2 += red2[v][wi];
            mx = max(mx, redm[v][wi]);
        }
        const int64_t idx = (static_cast<int64_t>(wi) * gridDim.y + d) * nseg + seg;
        ws.part_s1[idx] = s1;
        ws.part_s2lo[idx] = static_cast<uint64_t>(s2);
        ws.part_s2hi[idx] = static_cast<uint64_t>(s2 >> 64);
        ws.part_max[idx] = mx;
    }
}

// ----------------------------------------------------------------------------
// Pass 1 on 16-bit running sums.
//
// With c near the window's mean sample, P'(k) = P(k) - c k stays close to 0: the
// running sum of a noise series of sigma 30 wanders about 5000 over a window of
// 9216 samples.  While P' spans at most 2^14 - 1 over the window, every centred
// boxcar B' = P'(p + w) - P'(p) = B - c w does too, so two positions share a
// word: one packed subtraction, one v_dot2_i32_i16 for the squares and one
// packed maximum per two positions and width, instead of a subtraction, a
// 64-bit multiply-add and half a three-way maximum each.  The sums of B follow
// exactly: S1 = S1' + n c w, S2 = S2' + 2 c w S1' + n (c w)^2.  The running sums
// take half the LDS as well (20 KiB a block), and rows of any alignment load in
// aligned quads.  Bound by VALU issue as before, with less to issue: find_peaks
// on the survey series 1029 -> 851 us (10 widths), on 301 int32 rows of odd
// length 164 -> 133.  Eight steps unrolled (four: 952 us).  Five waves per SIMD
// for uint16, four for int32 (whose quads take twice the registers): one more
// spills the sums of the wide form and gains nothing.
//
// Windows that span more (bright pulses, a drifting baseline) put the same sums
// into LDS with 32 bits, half the segment at a time, from the samples that the
// block still holds: as many instructions as the running sums of the general
// kernel, but no second load.  A drift shows in the values between the waves'
// runs, before anything is spent on 16 bits.  find_peaks on a survey series that
// all drifts 814 us (877 in the general kernel; 927 when every window was tried on
// 16 bits first), 11 widths to 1000 892 (949), 1200 rows of 5000 samples with pulses
// 60 (98), int32 samples of 2^17 to 2^18 79 (125).  Samples from 2^19 on, or with a
// widest boxcar from 2^25 on, take P itself, width by width: 160 (174) and 257 (270).
// ----------------------------------------------------------------------------
constexpr int kSegLen = 8192;                       // positions per segment
constexpr int kHalfLen = kSegLen / 2;
constexpr int kWinSamples = 4 * kThreads * kRounds;     // samples a block loads
constexpr int kMaxSpan16 = (1 << 14) - 1;
// widest boxcar: 3 samples of misalignment, the last position and the window
// of the widest boxcar inside the running sums P(0 .. kWinSamples - 1)
constexpr int kMaxWidth16 = kWinSamples - 3 - kSegLen;
// LDS words: the 16-bit running sums (up to 3 places on), or half a window's
// 32-bit ones, or a value of 8 bytes per pair of lanes and width (16 widths)
constexpr int kPairStride = kThreads / 2 + 16;
constexpr int kHalfRounds = kRounds - 4;            // rounds that half a segment's window takes
constexpr int kLds16Words = 4 * kThreads * kHalfRounds;
static_assert(kHalfLen == 4 * 4 * kThreads, "a half starts at a round");
static_assert(kLds16Words >= kHalfLen + kMaxWidth16 + 3, "half a window fits");
static_assert(kLds16Words * 2 >= kWinSamples + 4, "16-bit sums fit");
static_assert(kLds16Words >= 2 * 16 * kPairStride, "reductions fit");

typedef short i16x2 __attribute__((ext_vector_type(2)));

// Minimum and maximum over the wave (in lane 63).
__device__ __forceinline__ int dpp_i32(int x, int ctrl) {
    switch (ctrl) {
        case 0: return __builtin_amdgcn_update_dpp(x, x, 0x111, 0xF, 0xF, false);
        case 1: return __builtin_amdgcn_update_dpp(x, x, 0x112, 0xF, 0xF, false);
        case 2: return __builtin_amdgcn_update_dpp(x, x, 0x114, 0xF, 0xF, false);
        case 3: return __builtin_amdgcn_update_dpp(x, x, 0x118, 0xF, 0xF, false);
        case 4: return __builtin_amdgcn_update_dpp(x, x, 0x142, 0xA, 0xF, false);
        default: return __builtin_amdgcn_update_dpp(x, x, 0x143, 0xC, 0xF, false);
    }
}
__device__ __forceinline__ int wave_max_i32(int x) {
#pragma unroll
    for (int c = 0; c < 6; ++c) x = max(x, dpp_i32(x, c));
    return x;
}

// The block's totals of NW widths from every thread's sum of squares and
// maximum (as int), and every wave's sums (lane wi: width wi).  Lane 16 wi of
// the block returns true with width wi's totals.  lds: 2 NW kPairStride words,
// free on entry for every thread (the caller's barrier).
template <int NW>
__device__ __forceinline__ bool stats_reduce(const uint64_t (&s2)[NW], const int (&mx)[NW], int64_t s1,
                                             uint32_t* lds, uint64_t* s2_out, int* mx_out, int64_t* s1_out) {
    const int t = threadIdx.x, lane = t & 63;
    uint64_t* r = reinterpret_cast<uint64_t*>(lds);
    // pairs of lanes first, then rows of 128 values per width: lane 16 wi + l
    // takes l, l + 16, ... and the 16 lanes of a DPP row their sum
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) {
        const uint64_t o = (static_cast<uint64_t>(dpp_u32(static_cast<uint32_t>(s2[wi] >> 32), 0)) << 32) |
                           dpp_u32(static_cast<uint32_t>(s2[wi]), 0);
        if (!(t & 1)) r[wi * kPairStride + (t >> 1)] = s2[wi] + o;
    }
    __syncthreads();
    uint64_t acc = 0;
    if (t < NW * 16) {
        const uint64_t* q = r + (t >> 4) * kPairStride + (t & 15);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += q[16 * k];
    }
    acc = row_sum_u64(acc);
    __syncthreads();
    int* rm = reinterpret_cast<int*>(lds) + 2 * 16 * (kThreads / 64);
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) {
        const int o = max(mx[wi], static_cast<int>(dpp_u32(static_cast<uint32_t>(mx[wi]), 0)));
        if (!(t & 1)) rm[wi * kPairStride + (t >> 1)] = o;
    }
    int64_t* rs = reinterpret_cast<int64_t*>(lds);
    if (lane < NW) rs[(t >> 6) * NW + lane] = s1;
    __syncthreads();
    int am = INT32_MIN;
    int64_t a1 = 0;
    if (t < NW * 16) {
        const int* q = rm + (t >> 4) * kPairStride + (t & 15);
#pragma unroll
        for (int k = 0; k < 8; ++k) am = max(am, q[16 * k]);
        if ((t & 15) == 0) {
#pragma unroll
            for (int v = 0; v < kThreads / 64; ++v) a1 += rs[v * NW + (t >> 4)];
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) am = max(am, static_cast<int>(dpp_u32(static_cast<uint32_t>(am), c)));
    *s2_out = acc;
    *mx_out = am;
    *s1_out = a1;
    return t < NW * 16 && (t & 15) == 0;
}

// This lane's width (lane wi < NW) and the wave's share of its sum of boxcars
// over n positions, by telescoping: sum_p (P(p + w) - P(p)) = sum_{i < w}
// (P(n + i) - P(i)).  diff(i, k) gives the i-th term, the thread's k-th; a DPP
// scan gives the prefix, lane wi fetches the one at w - 1.  Terms up to kMaxSpan16
// are scanned as they are; WIDE ones, any int, by 16-bit halves.
constexpr int kTerms = (kMaxWidth16 + kThreads - 1) / kThreads;   // of a thread
template <int NW, bool WIDE, typename F>
__device__ __forceinline__ int64_t telescoped(const int (&w)[NW], F diff) {
    static_assert(64 * static_cast<int64_t>(kMaxSpan16) < (int64_t(1) << 31), "the sum of a wave's terms is an int");
    const int lane = threadIdx.x & 63;
    int myw = 0;
#pragma unroll
    for (int wi = 0; wi < NW; ++wi)
        if (lane == wi) myw = w[wi];
    const int wave0 = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) & ~63);
    int64_t s1 = 0;
#pragma unroll
    for (int k = 0; k < kTerms; ++k) {
        const int i0 = wave0 + k * kThreads;
        if (i0 >= w[NW - 1]) break;
        const int i = i0 + lane;
        const int d = i < w[NW - 1] ? diff(i, k) : 0;
        const int l = myw - 1 - i0;
        const int src = min(max(l, 0), 63);
        int64_t got = __shfl(static_cast<int>(wave_incl_scan(static_cast<uint32_t>(WIDE ? d & 0xFFFF : d))), src, 64);
        if (WIDE)
            got += int64_t(65536) *
                   __shfl(static_cast<int>(wave_incl_scan(static_cast<uint32_t>(d >> 16))), src, 64);
        if (l >= 0) s1 += got;
    }
    return s1;
}

// Four consecutive samples, as loaded (one aligned 8- or 16-byte load).
template <typename T>
struct Quad;
template <>
struct Quad<uint16_t> {
    uint32_t v[2];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int off) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
        v[0] = x[0];
        v[1] = x[1];
    }
    __device__ __forceinline__ uint32_t get(int j) const { return (v[j >> 1] >> (16 * (j & 1))) & 0xFFFFu; }
    __device__ __forceinline__ void set(int j, uint32_t s) {
        v[j >> 1] = (v[j >> 1] & (j & 1 ? 0xFFFFu : 0xFFFF0000u)) | (s << (16 * (j & 1)));
    }
    __device__ __forceinline__ uint32_t sum() const { return add_halves(v[1], add_halves(v[0], 0u)); }
    // P(0 .. 2) of the quad on top of base
    __device__ __forceinline__ uint32_t s1(uint32_t base) const { return base + (v[0] & 0xFFFFu); }
    __device__ __forceinline__ uint32_t s2(uint32_t base) const { return add_halves(v[0], base); }
    __device__ __forceinline__ uint32_t s3(uint32_t base) const { return s2(base) + (v[1] & 0xFFFFu); }
    // m, vmax: two maxima in one word
    __device__ __forceinline__ uint32_t vmax(uint32_t m) const {
        const u16x2 a = __builtin_bit_cast(u16x2, v[0]), b = __builtin_bit_cast(u16x2, v[1]);
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m),
                                                                      __builtin_elementwise_max(a, b)));
    }
};
template <>
struct Quad<int32_t> {
    uint32_t v[4];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int off) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = x[j];
    }
    __device__ __forceinline__ uint32_t get(int j) const { return v[j]; }
    __device__ __forceinline__ void set(int j, uint32_t s) { v[j] = s; }
    __device__ __forceinline__ uint32_t sum() const { return v[0] + v[1] + v[2] + v[3]; }
    __device__ __forceinline__ uint32_t s1(uint32_t base) const { return base + v[0]; }
    __device__ __forceinline__ uint32_t s2(uint32_t base) const { return base + v[0] + v[1]; }
    __device__ __forceinline__ uint32_t s3(uint32_t base) const { return base + v[0] + v[1] + v[2]; }
    __device__ __forceinline__ uint32_t vmax(uint32_t m) const { return max(max(max(m, v[0]), max(v[1], v[2])), v[3]); }
};

// One (DM, segment) per block.  `in` is aligned to four samples; w_max <=
// kMaxWidth16; every width even, but for the first one when ODD1.
template <typename T, int NW, bool ODD1>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? 5 : 4)))
void boxcar_stats16_kernel(const T* __restrict__ in, int64_t nout, int64_t nbx, dd::Widths W, int nseg,
                           dd::PeaksWs ws) {
    __shared__ uint4 lds16[(kLds16Words + 3) / 4];
    __shared__ uint32_t round_tot[kRounds * (kThreads / 64)];
    __shared__ int span[2][kThreads / 64];      // per wave: largest P' and largest -P'
    __shared__ uint32_t vmax_w[kThreads / 64];
    constexpr bool kU16 = std::is_same<T, uint16_t>::value;
    uint32_t* lds = reinterpret_cast<uint32_t*>(lds16);
    const int d = blockIdx.y, seg = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t s0 = static_cast<int64_t>(seg) * kSegLen;
    const int npos = static_cast<int>(min<int64_t>(kSegLen, nbx - s0));
    int w[NW];
#pragma unroll
    for (int wi = 0; wi < NW; ++wi) w[wi] = W.w[wi];
    const int w_max = w[NW - 1];
    // The window: kWinSamples samples from the four-sample boundary at or before
    // the segment's first one (k0 samples on), loaded in kRounds rounds of one
    // aligned quad per thread, up to the end of the array; what lies past the
    // segment's last window (the next row) enters no difference that is used.
    const int64_t first = static_cast<int64_t>(d) * nout + s0;
    const int k0 = static_cast<int>(first & 3);
    const int64_t left = static_cast<int64_t>(gridDim.y) * nout - (first - k0);
    const int num = static_cast<int>(min<int64_t>(left, kWinSamples));
    const T* win = in + (first - k0);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(win), 0, (num & ~3) * static_cast<int>(sizeof(T)), kRowRsrcWord3);
    Quad<T> v[kRounds];
#pragma unroll
    for (int i = 0; i < kRounds; ++i) v[i].load(rs, 4 * (i * kThreads + t) * static_cast<int>(sizeof(T)));
    if (num & 3) {   // the array ends inside a quad: its samples one by one
        uint32_t tail[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) tail[j] = j < (num & 3) ? static_cast<uint32_t>(win[(num & ~3) + j]) : 0u;
#pragma unroll
        for (int i = 0; i < kRounds; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) v[i].set(j, i * kThreads + t == num >> 2 ? tail[j] : v[i].get(j));
    }
    uint32_t excl[kRounds];
    uint32_t vm = 0;
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const uint32_t c = v[i].sum();
        const uint32_t incl = wave_incl_scan(c);
        excl[i] = incl - c;
        if (lane == 63) round_tot[i * (kThreads / 64) + wave] = incl;
        if (!kU16) vm = v[i].vmax(vm);   // below 2^16 anyway
    }
    if (!kU16) {
        vm = static_cast<uint32_t>(wave_max_i32(static_cast<int>(min(vm, 0x7FFFFFFFu))));
        if (lane == 63) vmax_w[wave] = vm;
    }
    __syncthreads();
    const uint32_t tv = lane < kRounds * (kThreads / 64) ? round_tot[lane] : 0u;
    const uint32_t tin = wave_incl_scan(tv);
    const uint32_t tex = tin - tv;
    // a sample near the mean, the same in every lane (int32 samples up to 2^19 sum
    // beyond 2^32: their half sums)
    const uint32_t sum = static_cast<uint32_t>(
        __builtin_amdgcn_readlane(static_cast<int>(kU16 ? tin : wave_incl_scan(tv >> 1)), 63));
    const float mean = static_cast<float>(sum) * (kU16 ? 1.0f : 2.0f) * __builtin_amdgcn_rcpf(static_cast<float>(num));
    const int c = __builtin_amdgcn_readfirstlane(static_cast<int>(fminf(mean, 1e9f) + 0.5f));
    // The places of P' that are used are k0 .. kneed.  Where it spans too much, mostly
    // its values between the waves' runs of 256 samples, which every wave has, show it.
    const int kneed = k0 + npos - 1 + w_max;
    const int at256 = static_cast<int>(tex - static_cast<uint32_t>(c) * 256u * static_cast<uint32_t>(lane));
    const bool far = lane < kRounds * (kThreads / 64) && 256 * lane <= kneed &&
                     (at256 > kMaxSpan16 || at256 < -kMaxSpan16);
    // excl[i] = P'(4 g), g the thread's quad of round i, from here on
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        const uint32_t pre = static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(tex), i * (kThreads / 64) + wave));
        excl[i] += pre - static_cast<uint32_t>(c) * 4u * static_cast<uint32_t>(i * kThreads + t);
    }
    uint32_t vmax = 0xFFFFu;
    if (!kU16) {
        vmax = vmax_w[0];
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) vmax = max(vmax, vmax_w[k]);
    }
    const int64_t idx0 = static_cast<int64_t>(d) * nseg + seg;
    const int64_t stride = static_cast<int64_t>(gridDim.y) * nseg;
    // width t / 16's totals of B from those of B' = B - c w (lane 16 wi)
    auto store = [&](uint64_t a2, int am, int64_t a1) {
        const int64_t cw = static_cast<int64_t>(c) * W.w[t >> 4];
        const int64_t i = idx0 + (t >> 4) * stride;
        ws.part_s1[i] = static_cast<uint64_t>(a1 + npos * cw);
        ws.part_s2lo[i] = a2 + static_cast<uint64_t>(2 * cw) * static_cast<uint64_t>(a1) +
                          static_cast<uint64_t>(npos * cw * cw);   // below 2^64, modulo which it is formed
        ws.part_s2hi[i] = 0u;
        ws.part_max[i] = static_cast<uint32_t>(am + static_cast<int>(cw));
    };
    int smax = INT32_MAX, smin = INT32_MAX;   // largest P' and -P'
    if (!__ballot(far)) {
        const int off = k0 & 1 ? 4 - k0 : 0;   // k0 + off is even: pairs of positions are words
        int hi = 0, lo = 0;
        uint32_t word[kRounds][2];
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            const uint32_t base = excl[i];
            const int p0 = static_cast<int>(base);
            const int p1 = static_cast<int>(v[i].s1(base) - c);
            const int p2 = static_cast<int>(v[i].s2(base) - 2 * c);
            const int p3 = static_cast<int>(v[i].s3(base) - 3 * c);
            const bool need = 4 * (i * kThreads + t) <= kneed;
            const int h4 = max(max(max(hi, p0), max(p1, p2)), p3), l4 = min(min(min(lo, p0), min(p1, p2)), p3);
            hi = need ? h4 : hi;
            lo = need ? l4 : lo;
            word[i][0] = __builtin_amdgcn_perm(static_cast<uint32_t>(p1), static_cast<uint32_t>(p0), 0x05040100u);
            word[i][1] = __builtin_amdgcn_perm(static_cast<uint32_t>(p3), static_cast<uint32_t>(p2), 0x05040100u);
        }
        hi = wave_max_i32(hi);
        lo = wave_max_i32(-lo);
        if (lane == 63) {
            span[0][wave] = hi;
            span[1][wave] = lo;
        }
        // half-word h = k + off holds P'(k)
        uint16_t* half = reinterpret_cast<uint16_t*>(lds);
        if (off == 0) {
#pragma unroll
            for (int i = 0; i < kRounds; ++i)
                *reinterpret_cast<uint2*>(lds + 2 * (i * kThreads + t)) = make_uint2(word[i][0], word[i][1]);
        } else {
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {   // odd off: a half, a word, a half
                const int h = 4 * (i * kThreads + t) + off;
                half[h] = static_cast<uint16_t>(word[i][0]);
                *reinterpret_cast<uint32_t*>(half + h + 1) = __builtin_amdgcn_alignbit(word[i][1], word[i][0], 16);
                half[h + 3] = static_cast<uint16_t>(word[i][1] >> 16);
            }
        }
        __syncthreads();
        smax = smin = 0;
#pragma unroll
        for (int k = 0; k < kThreads / 64; ++k) {
            smax = max(smax, span[0][k]);
            smin = max(smin, span[1][k]);
        }
        // P' did not wrap (see below), the span, and every square sum below 2^13 x 2^50
        const bool narrow = vmax < (1u << 17) && smax <= kMaxSpan16 - smin && smin <= kMaxSpan16 &&
                            static_cast<int64_t>(c) * w_max + (1 << 14) < (1 << 25);
        if (narrow) {
            uint32_t sq[2][NW];   // at most 16 squares below 2^28 each
            i16x2 mx[NW];
#pragma unroll
            for (int wi = 0; wi < NW; ++wi) {
                sq[0][wi] = sq[1][wi] = 0u;
                mx[wi] = i16x2{INT16_MIN, INT16_MIN};
            }
            const uint32_t* base = lds + (k0 + off) / 2 + t;
            auto pair = [&](const uint32_t* q, int wi) -> uint32_t {
                return ODD1 && wi == 0 ? __builtin_amdgcn_alignbit(q[(w[0] + 1) / 2], q[(w[0] - 1) / 2], 16)
                                       : q[w[wi] / 2];
            };
            if (npos == kSegLen) {
#pragma unroll
                for (int hf = 0; hf < 2; ++hf)
#pragma unroll 8
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t* q = base + (8 * hf + j) * kThreads;
                        const i16x2 p = __builtin_bit_cast(i16x2, q[0]);
#pragma unroll
                        for (int wi = 0; wi < NW; ++wi) {
                            const i16x2 b = __builtin_bit_cast(i16x2, pair(q, wi)) - p;
                            sq[hf][wi] = static_cast<uint32_t>(
                                __builtin_amdgcn_sdot2(b, b, static_cast<int>(sq[hf][wi]), false));
                            mx[wi] = __builtin_elementwise_max(mx[wi], b);
                        }
                    }
            } else {
                for (int j = 0; j < 16 && 2 * j * kThreads < npos; ++j) {
                    const uint32_t* q = base + j * kThreads;
                    const int at = 2 * (j * kThreads + t);
                    const uint32_t m = at + 1 < npos ? 0xFFFFFFFFu : at < npos ? 0xFFFFu : 0u;
                    const i16x2 p = __builtin_bit_cast(i16x2, q[0]);
#pragma unroll
                    for (int wi = 0; wi < NW; ++wi) {
                        const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, pair(q, wi)) - p);
                        const i16x2 bs = __builtin_bit_cast(i16x2, b & m);
                        const uint32_t dot = static_cast<uint32_t>(
                            __builtin_amdgcn_sdot2(bs, bs, static_cast<int>(j < 8 ? sq[0][wi] : sq[1][wi]), false));
                        if (j < 8) sq[0][wi] = dot;
                        else sq[1][wi] = dot;
                        mx[wi] = __builtin_elementwise_max(
                            mx[wi], __builtin_bit_cast(i16x2, (b & m) | (0x80008000u & ~m)));
                    }
                }
            }
            const int16_t* ph = reinterpret_cast<const int16_t*>(half) + k0 + off;
            const int64_t s1 =
                telescoped<NW, false>(w, [&](int i, int) { return static_cast<int>(ph[npos + i]) - ph[i]; });
            uint64_t s2[NW];
            int m32[NW];
#pragma unroll
            for (int wi = 0; wi < NW; ++wi) {
                s2[wi] = static_cast<uint64_t>(sq[0][wi]) + sq[1][wi];
                m32[wi] = max(static_cast<int>(mx[wi].x), static_cast<int>(mx[wi].y));
            }
            __syncthreads();   // the running sums are no longer needed
            uint64_t a2;
            int am;
            int64_t a1;
            if (stats_reduce<NW>(s2, m32, s1, lds, &a2, &am, &a1)) store(a2, am, a1);
            return;
        }
    }
    // 32-bit running sums, half the segment at a time, from the loaded samples.
    // Position p of half hf is ps[p]; base(i) is P or P' at quad i.
    const int* ps = reinterpret_cast<const int*>(lds) + k0;
    auto fill_half = [&](int hf, int cc, auto base) {
        __syncthreads();   // what the LDS held is no longer needed
#pragma unroll
        for (int r = 0; r < kHalfRounds; ++r) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {   // constant indices keep the quads in registers
                const int i = 4 * h + r;
                if (h != hf) continue;
                const uint32_t b = base(i);
                lds16[r * kThreads + t] = make_uint4(b, v[i].s1(b) - cc, v[i].s2(b) - 2 * cc, v[i].s3(b) - 3 * cc);
            }
        }
        __syncthreads();
    };
    if (kU16 && w_max > 512) {   // (otherwise the largest 16-bit value passes below)
        vm = 0;
#pragma unroll
        for (int i = 0; i < kRounds; ++i) vm = v[i].vmax(vm);
        vm = static_cast<uint32_t>(wave_max_i32(static_cast<int>(max(vm & 0xFFFFu, vm >> 16))));
        if (lane == 63) vmax_w[wave] = vm;
        __syncthreads();
        vmax = vmax_w[0];
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) vmax = max(vmax, vmax_w[k]);
    }
    // Samples below 2^19: with c within 1 of their mean, P' of N samples spans at
    // most N 2^19 / 4 (it returns to 0 at the window's end) < 2^31.  Boxcars and
    // centred boxcars below 2^25 by the largest sample, or |B'| < 2^24 by the span
    // and c w < 2^24: every square sum below 2^13 x 2^50.
    const int64_t vw = static_cast<int64_t>(max(vmax, static_cast<uint32_t>(c))) * w_max;
    if (vmax < (1u << 19) &&
        (vw < (1 << 25) || (smax < (1 << 23) && smin < (1 << 23) && static_cast<int64_t>(c) * w_max < (1 << 24)))) {
        uint64_t s2[NW];
        int mx[NW];
        int64_t s1 = 0;
        int first[kTerms];   // P'(i) of the thread's terms
#pragma unroll
        for (int wi = 0; wi < NW; ++wi) {
            s2[wi] = 0;
            mx[wi] = INT32_MIN;
        }
        constexpr int kUnroll = NW > 10 ? 2 : 4;   // (four spill with 11 widths: 1089 us, 948)
        const int* base = ps + t;
        auto add = [&](const int* q) {
            const int p0 = q[0];
#pragma unroll
            for (int wi = 0; wi < NW; ++wi) {
                const int b = q[w[wi]] - p0;
                s2[wi] += static_cast<uint64_t>(static_cast<int64_t>(b) * b);
                mx[wi] = max(mx[wi], b);
            }
        };
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int n = min(kHalfLen, npos - hf * kHalfLen);
            if (n <= 0) break;
            fill_half(hf, c, [&](int i) { return excl[i]; });
            if (hf == 0) {
#pragma unroll
                for (int k = 0; k < kTerms; ++k) first[k] = base[k * kThreads];
            }
            if (n == kHalfLen) {
#pragma unroll kUnroll
                for (int j = 0; j < kHalfLen / kThreads; ++j) add(base + j * kThreads);
            } else {
                for (int i = t; i < n; i += kThreads) add(ps + i);
            }
            if (hf == 1 || npos <= kHalfLen)
                s1 = telescoped<NW, true>(w, [&](int i, int k) { return ps[n + i] - first[k]; });
        }
        __syncthreads();
        uint64_t a2;
        int am;
        int64_t a1;
        if (stats_reduce<NW>(s2, mx, s1, lds, &a2, &am, &a1)) store(a2, am, a1);
        return;
    }
    // any values: P itself, one width after the other; 64-bit square sums for
    // boxcars below 2^26 (see width_sums), else 128-bit ones
    __shared__ uint64_t red1[kThreads / 64][NW];
    __shared__ u128 red2[kThreads / 64][NW];
    __shared__ uint32_t redm[kThreads / 64][NW];
    const bool small = static_cast<uint64_t>(vmax) * static_cast<uint64_t>(w_max) < (uint64_t(1) << 26);
#pragma unroll 1
    for (int wi = 0; wi < NW; ++wi) {
        const int ww = W.w[wi];
        uint64_t s1 = 0, lo = 0, hi = 0;
        uint32_t mx = 0;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int n = min(kHalfLen, npos - hf * kHalfLen);
            if (n <= 0) break;
            fill_half(hf, 0, [&](int i) {
                return excl[i] + static_cast<uint32_t>(c) * 4u * static_cast<uint32_t>(i * kThreads + t);
            });
            for (int i = t; i < n; i += kThreads) {
                const uint32_t b = static_cast<uint32_t>(ps[i + ww]) - static_cast<uint32_t>(ps[i]);
                const uint64_t sq = static_cast<uint64_t>(b) * b;
                s1 += b;
                lo += sq;
                hi += lo < sq ? 1u : 0u;
                mx = max(mx, b);
            }
        }
        uint64_t a1;
        u128 a2;
        uint32_t am;
        if (small)
            wave_totals<true>(s1, lo, hi, mx, &a1, &a2, &am);
        else
            wave_totals<false>(s1, lo, hi, mx, &a1, &a2, &am);
        if (lane == 0) {
            red1[wave][wi] = a1;
            red2[wave][wi] = a2;
            redm[wave][wi] = am;
        }
    }
    __syncthreads();
    if (t < NW) {
        uint64_t a1 = 0;
        u128 a2 = 0;
        uint32_t am = 0;
        for (int k = 0; k < kThreads / 64; ++k) {
            a1 += red1[k][t];
            a2 += red2[k][t];
            am = max(am, redm[k][t]);
        }
        const int64_t i = idx0 + t * stride;
        ws.part_s1[i] = a1;
        ws.part_s2lo[i] = static_cast<uint64_t>(a2);
        ws.part_s2hi[i] = static_cast<uint64_t>(a2 >> 64);
        ws.part_max[i] = am;
    }
}

// Pass 2: exact sums, D and B_thr per (width, DM) series, kSerPerBlock
// series per block.  A series' partials are contiguous (series-major), so the
// block stages a chunk of segments of all its series in LDS with loads that
// every thread issues at once (one memory round trip per chunk); thread t then
// adds series t's entries.  The sums are exact integers: their order is free.
constexpr int kSerPerBlock = 64;
constexpr int kSerChunk = 32;   // segments per staged chunk: 3 x 64 x 32 x 8 B = 48 KiB
__global__ __launch_bounds__(kThreads) void series_threshold_kernel(int nseries, int nseg,
                                                                    int64_t nbx, uint32_t kmant,
                                                                    int kexp2, dd::PeaksWs ws) {
    __shared__ uint64_t st1[kSerPerBlock * kSerChunk];
    __shared__ uint64_t st2lo[kSerPerBlock * kSerChunk];
    __shared__ uint64_t st2hi[kSerPerBlock * kSerChunk];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ws.nlist[0] = 0u;   // the mark and count passes append to the work lists
        ws.nlist[1] = 0u;
    }
    const int s0 = blockIdx.x * kSerPerBlock;
    const int ns = min(kSerPerBlock, nseries - s0);
    const int t = threadIdx.x;
    uint64_t s1 = 0;
    u128 s2 = 0;
    for (int c0 = 0; c0 < nseg; c0 += kSerChunk) {
        const int nc = min(kSerChunk, nseg - c0);
        const int n = ns * nc;
        constexpr int kPer = kSerPerBlock * kSerChunk / kThreads;
        uint64_t v1[kPer], vlo[kPer], vhi[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = t + k * kThreads;
            const int64_t idx = static_cast<int64_t>(s0 + i / nc) * nseg + c0 + i % nc;
            const bool in = i < n;
            v1[k] = in ? ws.part_s1[idx] : 0;
            vlo[k] = in ? ws.part_s2lo[idx] : 0;
            vhi[k] = in ? ws.part_s2hi[idx] : 0;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = t + k * kThreads;
            if (i < n) {
                st1[i] = v1[k];
                st2lo[i] = vlo[k];
                st2hi[i] = vhi[k];
            }
        }
        __syncthreads();
        if (t < ns) {
            for (int k = 0; k < nc; ++k) {
                const int i = t * nc + k;
                s1 += st1[i];
                s2 += static_cast<u128>(st2lo[i]) | (static_cast<u128>(st2hi[i]) << 64);
            }
        }
        __syncthreads();   // the next chunk overwrites the staging arrays
    }
    if (t >= ns) return;
    const int s = s0 + t;
    ws.tot[s] = 0u;     // the count pass adds the segments' run starts
    ws.s1[s] = s1;
    ws.s2lo[s] = static_cast<uint64_t>(s2);
    ws.s2hi[s] = static_cast<uint64_t>(s2 >> 64);
    u128 d = 0;
    const int64_t thr = cut_level(static_cast<uint64_t>(nbx), s1, s2, kmant, kexp2, &d);
    if (thr < 0) {
        ws.thr[s] = -1;
        ws.thr32[s] = 0xFFFFFFFFu;
        ws.sqrt_d[s] = 0.0;
        return;
    }
    ws.thr[s] = thr;
    ws.thr32[s] = thr > 0xFFFFFFFFll ? 0xFFFFFFFFu : static_cast<uint32_t>(thr);
    ws.sqrt_d[s] = sqrt(u128_to_double(d));
}

// Pass 3a: one thread per (DM, segment).  A segment where, for some width,
// the largest boxcar reaches the series' cut goes on the count work list;
// every other segment gets zero run starts for all widths here.
__global__ __launch_bounds__(kThreads) void mark_kernel(int ndm, int nseg, int nw, dd::PeaksWs ws) {
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (idx >= static_cast<int64_t>(ndm) * nseg) return;
    const int d = static_cast<int>(idx / nseg);
    bool any = false;
#pragma unroll 4
    for (int wi = 0; wi < nw; ++wi)
        any |= ws.part_max[static_cast<int64_t>(wi) * ndm * nseg + idx] >= ws.thr32[wi * ndm + d];
    if (any) {
        ws.list[atomicAdd(&ws.nlist[0], 1u)] = static_cast<uint32_t>(idx);
    } else {
        for (int wi = 0; wi < nw; ++wi) ws.counts[static_cast<int64_t>(wi) * ndm * nseg + idx] = 0;
    }
}

// Pass 3b: number of run starts per (width, DM, segment) of the listed
// segments (a fixed grid of blocks works through the list).  Segments with
// any start go on the write list.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void peaks_count_kernel(const T* __restrict__ in, int ndm,
                                                               int64_t nout, int64_t nbx,
                                                               dd::Widths W, int L, int nseg,
                                                               dd::PeaksWs ws) {
    extern __shared__ uint32_t pl[];
    __shared__ uint32_t wave_tot[NT / 64];
    __shared__ uint32_t cnt[dd::kMaxWidths];
    const uint32_t nitems = ws.nlist[0];
    const int lane = threadIdx.x & 63;
    for (uint32_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int64_t idx = ws.list[item];
        const int d = static_cast<int>(idx / nseg);
        const int seg = static_cast<int>(idx % nseg);
        const int64_t s0 = static_cast<int64_t>(seg) * L;
        const int n = L + W.w[W.n - 1] + 1;
        if (threadIdx.x < dd::kMaxWidths) cnt[threadIdx.x] = 0;
        load_prefix<NT>(in + static_cast<int64_t>(d) * nout, nout, s0 - 1, n, pl, wave_tot);
        const int npos = static_cast<int>(min<int64_t>(L, nbx - s0));
        for (int wi = 0; wi < W.n; ++wi) {
            const uint32_t thr = ws.thr32[wi * ndm + d];
            if (ws.part_max[(static_cast<int64_t>(wi) * ndm + d) * nseg + seg] < thr) continue;
            const int w = W.w[wi];
            uint32_t c = 0;
            for (int i0 = threadIdx.x; i0 < npos; i0 += 4 * NT) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = i0 + k * NT;
                    if (i < npos) {
                        const bool above = pl[i + 1 + w] - pl[i + 1] >= thr;
                        const bool prev = (s0 + i > 0) && (pl[i + w] - pl[i] >= thr);
                        c += (above && !prev) ? 1u : 0u;
                    }
                }
            }
            if (!__ballot(c != 0)) continue;   // most waves of the larger blocks
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
            if (lane == 0) atomicAdd(&cnt[wi], c);
        }
        __syncthreads();
        if (threadIdx.x < W.n) {
            const int64_t series = static_cast<int64_t>(threadIdx.x) * ndm + d;
            ws.counts[series * nseg + seg] = cnt[threadIdx.x];
            // (a series of one segment: its count is its total)
            if (nseg > 1 && !ws.offs && cnt[threadIdx.x]) atomicAdd(&ws.tot[series], cnt[threadIdx.x]);
        }
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int wi = 0; wi < W.n; ++wi) tot += cnt[wi];
            if (tot) ws.list2[atomicAdd(&ws.nlist[1], 1u)] = static_cast<uint32_t>(idx);
        }
        __syncthreads();   // pl and cnt are reused by the next item
    }
}

// Exclusive scan of counts (uint32) into offsets (int64): three small kernels.
constexpr int kScanChunk = 4096;

__global__ __launch_bounds__(kThreads) void scan_chunks_kernel(const uint32_t* __restrict__ counts,
                                                               int64_t n, int64_t* __restrict__ offs,
                                                               int64_t* __restrict__ chunk_tot) {
    __shared__ uint32_t wave_tot[kThreads / 64];
    __shared__ int64_t carry;
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kScanChunk;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < kScanChunk; base += kThreads) {
        const int64_t i = c0 + base + threadIdx.x;
        const uint32_t v = i < n ? counts[i] : 0u;
        const uint32_t ex = block_exclusive_scan(v, wave_tot);
        const int64_t cur = carry;
        if (i < n) offs[i] = cur + ex;
        __syncthreads();
        if (threadIdx.x == kThreads - 1) carry = cur + ex + v;
        __syncthreads();
    }
    if (threadIdx.x == 0) chunk_tot[blockIdx.x] = carry;
}

// Exclusive scan of the chunk totals in place (one block; 64-bit sums).
__global__ __launch_bounds__(kThreads) void scan_totals_kernel(int64_t* __restrict__ chunk_tot,
                                                               int nchunks,
                                                               int64_t* __restrict__ total) {
    __shared__ int64_t wave_tot[kThreads / 64];
    __shared__ int64_t carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nchunks; base += kThreads) {
        const int i = base + static_cast<int>(threadIdx.x);
        const int64_t v = i < nchunks ? chunk_tot[i] : 0;
        int64_t x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wave_tot[wave] = x;
        __syncthreads();
        int64_t before = carry;
        for (int w = 0; w < wave; ++w) before += wave_tot[w];
        if (i < nchunks) chunk_tot[i] = before + x - v;
        __syncthreads();
        if (threadIdx.x == kThreads - 1) carry = before + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kThreads) void scan_add_kernel(int64_t* __restrict__ offs, int64_t n,
                                                            const int64_t* __restrict__ chunk_tot) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i < n) offs[i] += chunk_tot[i / kScanChunk];
}

// Exclusive scan of the series' event counts into their first slots, and the
// total, by one block: kSeriesScan series per step, four per thread (64-bit
// sums).
constexpr int kScanThreads = 1024;
constexpr int kSeriesScan = 4 * kScanThreads;
__global__ __launch_bounds__(kScanThreads) void scan_series_kernel(const uint32_t* __restrict__ tot,
                                                                   int n, int64_t* __restrict__ soff,
                                                                   int64_t* __restrict__ total) {
    __shared__ int64_t wave_tot[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t carry = 0;
    for (int base = 0; base < n; base += kSeriesScan) {
        const int i = base + 4 * static_cast<int>(threadIdx.x);
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = i + k < n ? tot[i + k] : 0u;
        const int64_t own = static_cast<int64_t>(v[0]) + v[1] + v[2] + v[3];
        int64_t x = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wave_tot[wave] = x;
        __syncthreads();
        int64_t ex = carry + x - own;
#pragma unroll
        for (int w = 0; w < kScanThreads / 64; ++w) {
            const int64_t t = wave_tot[w];
            if (w < wave) ex += t;
            carry += t;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (i + k < n) soff[i + k] = ex;
            ex += v[k];
        }
        __syncthreads();   // the next step rewrites wave_tot
    }
    if (threadIdx.x == 0) *total = carry;
}

// Walk the run that starts at t with boxcar value b and write its event
// record.  Positions whose boxcar the block's running sums cover (local index
// below `lim`, running sums pl relative to s0) are read from LDS, kWalk at a
// time (the reads do not depend on each other); a run that goes on past them
// continues on the series in global memory with the sliding-window update,
// again loading kWalk positions' samples at once.
constexpr int kWalk = 16;

template <typename T>
__device__ __forceinline__ void write_event(const T* __restrict__ row, int64_t nbx, int w, int wi, int d,
                                            int64_t t, uint32_t b, uint32_t thr, uint64_t s1, double sqrt_d,
                                            dedisp_event* __restrict__ out, const uint32_t* pl,
                                            int64_t s0, int lim) {
    int64_t te = t, tp = t;
    uint32_t cur = b, best = b;
    bool open = true;                       // the run has not ended yet
    int64_t u = t;                          // last position of the run so far
    while (open && u + 1 < nbx && u + 1 - s0 < lim) {
        uint32_t bb[kWalk];
#pragma unroll
        for (int k = 0; k < kWalk; ++k) {
            const int64_t j = u + 1 + k - s0;
            bb[k] = (j < lim && u + 1 + k < nbx) ? pl[j + 1 + w] - pl[j + 1] : 0u;
        }
        int k = 0;
        for (; k < kWalk; ++k) {
            const int64_t v = u + 1 + k;
            if (v >= nbx || v - s0 >= lim) break;   // leave the LDS window: continue below
            if (bb[k] < thr) {
                open = false;
                break;
            }
            cur = bb[k];
            te = v;
            if (cur > best) {
                best = cur;
                tp = v;
            }
        }
        u += k;
    }
    while (open && u + 1 < nbx) {
        uint32_t add[kWalk], sub[kWalk];
#pragma unroll
        for (int k = 0; k < kWalk; ++k) {
            const bool in = u + 1 + k < nbx;    // then u + k + w <= nout - 1
            add[k] = in ? static_cast<uint32_t>(row[u + k + w]) : 0u;
            sub[k] = in ? static_cast<uint32_t>(row[u + k]) : 0u;
        }
        int k = 0;
        for (; k < kWalk; ++k) {
            if (u + 1 + k >= nbx) break;
            const uint32_t nb = cur + add[k] - sub[k];
            if (nb < thr) {
                open = false;
                break;
            }
            cur = nb;
            te = u + 1 + k;
            if (nb > best) {
                best = nb;
                tp = te;
            }
        }
        u += k;
        if (k < kWalk) break;
    }
    const int64_t lval = static_cast<int64_t>(nbx) * best - static_cast<int64_t>(s1);
    dedisp_event ev;
    ev.width_idx = wi;
    ev.dm_idx = d;
    ev.t_start = t;
    ev.t_end = te;
    ev.t_peak = tp;
    ev.b_peak = static_cast<int32_t>(best);
    ev.snr = static_cast<float>(static_cast<double>(lval) / sqrt_d);
    *out = ev;
}

// The same walk done by a whole wave, 64 consecutive positions per step.
// Inside the LDS window a lane takes its position's boxcar from the running
// sums; beyond it, the boxcars follow from the last one by a wave prefix sum
// of the add/subtract pairs.  The run goes on through the lanes before the
// first one whose boxcar is below the cut (a ballot); the peak is the largest
// boxcar, the earliest on ties, as in the walk above, so both give the same
// event.  Arguments are uniform over the wave; lane 0 writes the event.
template <typename T>
__device__ __forceinline__ void write_event_wave(const T* __restrict__ row, int64_t nbx, int w, int wi,
                                                 int d, int64_t t, uint32_t b, uint32_t thr, uint64_t s1,
                                                 double sqrt_d, dedisp_event* __restrict__ out,
                                                 const uint32_t* pl, int64_t s0, int lim, int lane) {
    int64_t te = t, tp = t;
    uint32_t cur = b, best = b;
    bool open = true;
    int64_t u = t;   // last position of the run so far
    while (open && u + 1 < nbx) {
        const int64_t v = u + 1 + lane;
        bool valid;
        uint32_t bb = 0u;
        if (u + 1 - s0 < lim) {
            // validity falls from true to false at most once along the lanes
            valid = v < nbx && v - s0 < lim;
            if (valid) {
                const int j = static_cast<int>(v - s0);
                bb = pl[j + 1 + w] - pl[j + 1];
            }
        } else {
            valid = v < nbx;   // then u + lane + w <= nout - 1
            const uint32_t delta =
                valid ? static_cast<uint32_t>(row[u + lane + w]) - static_cast<uint32_t>(row[u + lane]) : 0u;
            bb = cur + wave_incl_scan(delta);
        }
        const uint64_t below = __ballot(valid && bb < thr);
        const uint64_t stop = below | __ballot(!valid);
        const int nlive = stop ? __builtin_ctzll(stop) : 64;
        if (nlive > 0) {
            uint32_t m = lane < nlive ? bb : 0u;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) m = max(m, static_cast<uint32_t>(__shfl_xor(m, o, 64)));
            if (m > best) {
                best = m;
                tp = u + 1 + __builtin_ctzll(__ballot(lane < nlive && bb == m));
            }
            cur = static_cast<uint32_t>(__shfl(bb, nlive - 1, 64));
            te = u + nlive;
        }
        // the run ends at a position below the cut; leaving the window or the
        // data does not end it
        if (nlive < 64 && ((below >> nlive) & 1u)) open = false;
        u += nlive;
    }
    if (lane == 0) {
        const int64_t lval = static_cast<int64_t>(nbx) * best - static_cast<int64_t>(s1);
        dedisp_event ev;
        ev.width_idx = wi;
        ev.dm_idx = d;
        ev.t_start = t;
        ev.t_end = te;
        ev.t_peak = tp;
        ev.b_peak = static_cast<int32_t>(best);
        ev.snr = static_cast<float>(static_cast<double>(lval) / sqrt_d);
        *out = ev;
    }
}

// Pass 4: write the events of segments that have any.  The run starts of a
// (width, DM, segment) are collected in LDS (any order), ranked by position
// (they are few), and each is expanded by one thread at offset + rank;
// segments with very many starts use block-wide scans in position order.
constexpr int kMaxStarts = 1024;

// The events of one listed (DM, segment).
template <int NT, typename T>
__device__ __forceinline__ void write_segment(const T* __restrict__ in, int ndm, int64_t nout, int64_t nbx,
                              const dd::Widths& W, int L, int nseg, const dd::PeaksWs& ws,
                              dedisp_event* __restrict__ events, int64_t capacity, int d, int seg,
                              uint32_t* pl, uint32_t* wave_tot, int* starts, int* nstart_p,
                              uint32_t* slab_total_p) {
    int& nstart = *nstart_p;
    uint32_t& slab_total = *slab_total_p;
    const int64_t s0 = static_cast<int64_t>(seg) * L;
    const int n = L + W.w[W.n - 1] + 1;
    const T* row = in + static_cast<int64_t>(d) * nout;
    load_prefix<NT>(row, nout, s0 - 1, n, pl, wave_tot);
    const int npos = static_cast<int>(min<int64_t>(L, nbx - s0));

    // Every width at once when all the segment's run starts fit the list:
    // width wi's starts fill starts[base[wi] .. base[wi] + count[wi]) (the
    // counts are known from the count pass), one pass over the positions
    // finds them, and then all runs of all widths are walked concurrently.
    __shared__ uint32_t wb[dd::kMaxWidths + 1], wc[dd::kMaxWidths], wfill[dd::kMaxWidths];
    __shared__ uint32_t wthr[dd::kMaxWidths];
    __shared__ int64_t woff[dd::kMaxWidths];   // slot of the segment's first event of each width
    if (ws.offs) {
        if (threadIdx.x < W.n) woff[threadIdx.x] = ws.offs[(static_cast<int64_t>(threadIdx.x) * ndm + d) * nseg + seg];
    } else {
        // the series' first slot, then the events of its segments before this one:
        // 16 widths at a time
        constexpr int kG = NT / 16;
        const int l = threadIdx.x % kG;
        for (int wi = threadIdx.x / kG; wi < W.n; wi += 16) {
            const int64_t series = static_cast<int64_t>(wi) * ndm + d;
            int64_t before = l == 0 ? ws.soff[series] : 0;
            for (int k = l; k < seg; k += kG) before += ws.counts[series * nseg + k];
#pragma unroll
            for (int o = kG / 2; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
            if (l == 0) woff[wi] = before;
        }
    }
    if (threadIdx.x < W.n) {
        const int wi = threadIdx.x;
        wc[wi] = ws.counts[(static_cast<int64_t>(wi) * ndm + d) * nseg + seg];
        wthr[wi] = ws.thr32[wi * ndm + d];
        wfill[wi] = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t b = 0;
        for (int wi = 0; wi < W.n; ++wi) {
            wb[wi] = b;
            b += wc[wi];
        }
        wb[W.n] = b;
    }
    __syncthreads();
    const uint32_t total = wb[W.n];
    if (total <= static_cast<uint32_t>(kMaxStarts)) {
        // width outer (uniform), four positions per step: as in the count pass
        for (int wi = 0; wi < W.n; ++wi) {
            if (wc[wi] == 0) continue;
            const int w = W.w[wi];
            const uint32_t thr = wthr[wi];
            for (int i0 = threadIdx.x; i0 < npos; i0 += 4 * NT) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + q * NT;
                    if (i < npos) {
                        const bool above = pl[i + 1 + w] - pl[i + 1] >= thr;
                        const bool prev = (s0 + i > 0) && (pl[i + w] - pl[i] >= thr);
                        if (above && !prev) {
                            const uint32_t k = atomicAdd(&wfill[wi], 1u);
                            if (k < wc[wi]) starts[wb[wi] + k] = i;
                        }
                    }
                }
            }
        }
        __syncthreads();
        // one run per wave: its rank among its width's starts, then its walk
        const int lane = threadIdx.x & 63;
        for (uint32_t k = threadIdx.x >> 6; k < total; k += NT / 64) {
            int wi = 0;
            while (wb[wi + 1] <= k) ++wi;
            const int i = starts[k];
            uint32_t rank = 0;
            for (uint32_t q = wb[wi] + lane; q < wb[wi + 1]; q += 64) rank += starts[q] < i;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) rank += __shfl_xor(rank, o, 64);
            const int64_t e = woff[wi] + rank;
            const int w = W.w[wi];
            const int sidx = wi * ndm + d;
            if (e < capacity)
                write_event_wave(row, nbx, w, wi, d, s0 + i, pl[i + 1 + w] - pl[i + 1], wthr[wi],
                                 ws.s1[sidx], ws.sqrt_d[sidx], &events[e], pl, s0, n - 1 - w, lane);
        }
        return;
    }

    for (int wi = 0; wi < W.n; ++wi) {
        const uint32_t cnt = wc[wi];
        if (cnt == 0) continue;
        const int sidx = wi * ndm + d;
        const uint32_t thr = ws.thr32[sidx];
        const int w = W.w[wi];
        const int64_t off = woff[wi];
        const uint64_t s1 = ws.s1[sidx];
        const double sq = ws.sqrt_d[sidx];
        const int lim = n - 1 - w;   // local positions whose boxcar the running sums cover
        if (cnt <= kMaxStarts) {
            if (threadIdx.x == 0) nstart = 0;
            __syncthreads();
            for (int i = threadIdx.x; i < npos; i += NT) {
                const uint32_t b = pl[i + 1 + w] - pl[i + 1];
                const bool prev = (s0 + i > 0) && (pl[i + w] - pl[i] >= thr);
                if (b >= thr && !prev) {
                    const int k = atomicAdd(&nstart, 1);
                    if (k < kMaxStarts) starts[k] = i;
                }
            }
            __syncthreads();
            const int m = min(nstart, kMaxStarts);
            for (int k = threadIdx.x; k < m; k += NT) {
                const int i = starts[k];
                int rank = 0;
                for (int q = 0; q < m; ++q) rank += starts[q] < i;
                const int64_t e = off + rank;
                if (e < capacity)
                    write_event(row, nbx, w, wi, d, s0 + i, pl[i + 1 + w] - pl[i + 1], thr, s1, sq, &events[e],
                                pl, s0, lim);
            }
            __syncthreads();
        } else {
            int64_t rank = off;
            for (int base = 0; base < npos; base += NT) {
                const int i = base + threadIdx.x;
                bool start = false;
                uint32_t b = 0;
                if (i < npos) {
                    b = pl[i + 1 + w] - pl[i + 1];
                    const bool prev = (s0 + i > 0) && (pl[i + w] - pl[i] >= thr);
                    start = b >= thr && !prev;
                }
                const uint32_t ex = block_exclusive_scan<NT>(start ? 1u : 0u, wave_tot);
                if (start && rank + ex < capacity)
                    write_event(row, nbx, w, wi, d, s0 + i, b, thr, s1, sq, &events[rank + ex], pl, s0,
                                lim);
                if (threadIdx.x == NT - 1) slab_total = ex + (start ? 1u : 0u);
                __syncthreads();
                rank += slab_total;
                __syncthreads();
            }
        }
    }
}

// (128 registers, four waves per SIMD: with one more the many events of 74 400
// segments at 4 sigma took 1460 us in place of 1150.)
template <typename T, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
void peaks_write_kernel(const T* __restrict__ in, int ndm, int64_t nout, int64_t nbx, dd::Widths W, int L,
                        int nseg, dd::PeaksWs ws, dedisp_event* __restrict__ events, int64_t capacity) {
    extern __shared__ uint32_t pl[];
    __shared__ uint32_t wave_tot[NT / 64];
    __shared__ int starts[kMaxStarts];
    __shared__ int nstart;
    __shared__ uint32_t slab_total;
    const uint32_t nitems = ws.nlist[1];
    for (uint32_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int64_t idx = ws.list2[item];
        write_segment<NT>(in, ndm, nout, nbx, W, L, nseg, ws, events, capacity,
                      static_cast<int>(idx / nseg), static_cast<int>(idx % nseg), pl, wave_tot,
                      starts, &nstart, &slab_total);
        __syncthreads();   // LDS is reused by the next item
    }
}

}  // namespace

namespace dd {

int segment_length(int w_max) {
    // LDS holds L + w_max + 1 running sums.
    int L = 8192;
    while (L > 256 && static_cast<int64_t>(L + w_max + 1) * 4 > 60 * 1024) L >>= 1;
    return L;
}

// Blocks of the count and write passes.  They work through lists whose lengths only
// the device knows: a few per cent of the (DM, segment)s in a clean search, most of
// them at a low cut or with interference.  Larger blocks finish a listed segment
// sooner, smaller ones keep more of them in flight (a block of 1024 write threads
// fills a CU).  So the number of all segments decides, and of those that noise alone
// lists; us for count + write with 1024, 512 and 256 threads, clean and all listed:
//      108 segments    48   65  105       52   68  113
//      800             44   54   86       98   87  118
//     1960            101   83  110      210  158  190
//     3913             75   69  110      312  253  246
//    12400            216  155  176      969  754  722
// (1960: more pulses than in the others' clean series.)  Up to 4096 what the largest
// blocks lose with interference is less than the rest of the search has gained, and a
// list of fewer segments than CUs, 12 us shorter with them (16 800 segments with 95
// events: 38 and 50 us), is common and the call short.  Where noise lists more than
// 512 (S/N cuts below 4.7 at 4096 segments of 10 widths) they lose outright (64 x
// 500000 at 4 sigma: find_peaks 464 us, 352 with 512 threads).  Beyond 32768 the
// larger blocks only lose (the survey series, 74 400: 192 us with 256 threads, 247
// with 1024).
constexpr int64_t kFewSegments = 4096, kMidSegments = 32768;
constexpr double kFewNoise = 512;
int list_threads(int64_t segments, int L, int nw, uint32_t kmant, int kexp2) {
    if (segments > kMidSegments) return kThreads;
    const double k = std::ldexp(static_cast<double>(kmant), kexp2);
    const double noise = segments * std::min(1.0, 0.5 * std::erfc(k * M_SQRT1_2) * L * nw);
    return segments <= kFewSegments && noise <= kFewNoise ? kFewThreads : kMidThreads;
}
// Waves of the list-driven passes' blocks: 32 per CU.
constexpr int64_t kListWaves = 8192;

// Series that one block scans (a step of 4096 takes about 3 us: 12 000 series
// 9.6 us, where scanning the counts of all their segments with three kernels
// took 25); more take the three-kernel scan.
constexpr int64_t kOneBlockScan = 16 * kSeriesScan;

// Most segments of a series whose counts every listed segment of it adds up by
// itself; the events' slots of longer series come from a scan of all counts with
// three kernels.  find_peaks on 4 series of uint16 with every segment listed, us,
// without and with the scan: 512 segments each 280 and 303, 1024 499 and 516, 2048
// 920 and 918, 4096 1798 and 1708; one series of 32768 segments 7315 and 5024.
constexpr int kSeriesSegments = 2048;

size_t peaks_lds_bytes(int L, int w_max) { return static_cast<size_t>(L + w_max + 1) * 4; }

hipError_t set_lds_limit(const void* fn, size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
}

hipError_t launch_boxcar(const void* in, int in_u16, int ndm, int64_t nout, const Widths& W,
                         int dm_first, int dm_count, int32_t* out, hipStream_t s) {
    (void)ndm;
    const int w_max = W.w[W.n - 1];
    const int64_t nbx = nout - w_max + 1;
    const int L = segment_length(w_max);
    const size_t lds = peaks_lds_bytes(L, w_max);
    const dim3 grid(static_cast<unsigned>((nbx + L - 1) / L), static_cast<unsigned>(dm_count));
    if (in_u16) {
        set_lds_limit(reinterpret_cast<const void*>(boxcar_kernel<uint16_t>), lds);
        hipLaunchKernelGGL(boxcar_kernel<uint16_t>, grid, dim3(kThreads), lds, s,
                           static_cast<const uint16_t*>(in), nout, nbx, W, dm_first, L, out, dm_count);
    } else {
        set_lds_limit(reinterpret_cast<const void*>(boxcar_kernel<int32_t>), lds);
        hipLaunchKernelGGL(boxcar_kernel<int32_t>, grid, dim3(kThreads), lds, s,
                           static_cast<const int32_t*>(in), nout, nbx, W, dm_first, L, out, dm_count);
    }
    return hipGetLastError();
}

hipError_t launch_baseline(const void* in, int in_u16, int ndm, int64_t nout, int radius,
                           int offset, void* out, int out_u16, hipStream_t s) {
    const int64_t nres = nout - 2 * static_cast<int64_t>(radius);
    // floor(n / w) = (n * M) >> k with k = 31 + ceil(log2 w), M = ceil(2^k / w):
    // writing M w = 2^k + e (0 <= e < w), n M / 2^k = n / w + n e / (w 2^k), and
    // n e < 2^31 * 2^ceil(log2 w) = 2^k for n < 2^31, so the extra term stays
    // below 1/w and cannot carry past the next integer; n M < 2^63.
    const uint32_t win = 2u * static_cast<uint32_t>(radius) + 1u;
    int lg = 0;
    while ((1u << lg) < win) ++lg;
    // k >= 32 and M < 2^32 but for win = 1 (no division): the high half of the
    // product, then a shift by k - 32.
    const int k = 31 + lg;
    const uint32_t magic = static_cast<uint32_t>(((uint64_t(1) << k) + win - 1) / win);
    const int shift = std::max(k - 32, 0);
    const int64_t nseg = (nres + kBlSeg - 1) / kBlSeg;
    const int64_t waves = static_cast<int64_t>(ndm) * nseg;
    const dim3 grid(static_cast<unsigned>((waves + kThreads / 64 - 1) / (kThreads / 64)));
#define DD_BL(T, U)                                                                            \
    hipLaunchKernelGGL((nres < bl_brief<T>() ? baseline_kernel<T, U, true> : baseline_kernel<T, U, false>), \
                       grid, dim3(kThreads), 0, s, static_cast<const T*>(in), ndm, nout, nres, radius, \
                       offset, nseg, magic, shift, static_cast<U*>(out));
    if (in_u16 && out_u16) DD_BL(uint16_t, uint16_t)
    else if (in_u16) DD_BL(uint16_t, int32_t)
    else if (out_u16) DD_BL(int32_t, uint16_t)
    else DD_BL(int32_t, int32_t)
#undef DD_BL
    return hipGetLastError();
}

template <typename T, int NW>
hipError_t launch_stats_t(const void* in, int64_t nout, const Widths& W, const PeaksLayout& lay,
                          const PeaksWs& ws, dim3 grid, size_t lds, hipStream_t s) {
    // contiguous-run window loads (uint16 only): rows of a multiple of 4
    // samples from an 8-byte aligned series, and a window that the runs cover
    const int w_max = W.w[W.n - 1];
    const int runs = std::is_same<T, uint16_t>::value && nout % 4 == 0 &&
                     reinterpret_cast<uintptr_t>(in) % 8 == 0 && lay.L + w_max + 1 + 3 <= 4 * kThreads * kRounds;
    if (runs) lds = std::max(lds, static_cast<size_t>(kRunWords) * 4);
    auto kern = boxcar_stats_kernel<T, NW>;
    hipError_t e = set_lds_limit(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, s, static_cast<const T*>(in), nout, lay.nbx,
                       W, lay.L, lay.nseg, runs, ws);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_stats_w(const void* in, int64_t nout, const Widths& W, const PeaksLayout& lay,
                          const PeaksWs& ws, dim3 grid, size_t lds, hipStream_t s) {
    // the register fast path reuses the running-sum area (L + w_max + 1 words)
    // for its reduction (3 * NW * kRedStride words)
    const int w_max = W.w[W.n - 1];
    const int nw = (lay.L == kPerThread * kThreads && W.n <= 16 &&
                    3 * W.n * kRedStride <= lay.L + w_max + 1) ? W.n : 0;
    switch (nw) {
#define DD_NW(N) case N: return launch_stats_t<T, N>(in, nout, W, lay, ws, grid, lds, s);
        DD_NW(1) DD_NW(2) DD_NW(3) DD_NW(4) DD_NW(5) DD_NW(6) DD_NW(7) DD_NW(8)
        DD_NW(9) DD_NW(10) DD_NW(11) DD_NW(12) DD_NW(13) DD_NW(14) DD_NW(15) DD_NW(16)
#undef DD_NW
        default: return launch_stats_t<T, 0>(in, nout, W, lay, ws, grid, lds, s);
    }
}

// The 16-bit form's rule: whole segments of kSegLen, a series that starts on a
// four-sample boundary (rows need not), widths that fit its window, all even but
// the first (two positions share a word, so an odd width costs a shift per word and
// width).  4 to 12 widths are compiled, no more for the lists that searches use;
// shorter and longer lists would gain too (600 x 200004 samples of 16 bits, 3 widths
// 131 us in the general kernel, 118 so; 13 widths 632 and 199).
template <typename T>
bool stats16_fits(const void* in, const Widths& W, const PeaksLayout& lay) {
    if (lay.L != kSegLen || W.n < 4 || W.n > 12 || W.w[W.n - 1] > kMaxWidth16 ||
        reinterpret_cast<uintptr_t>(in) % (4 * sizeof(T)))
        return false;
    for (int i = 1; i < W.n; ++i)
        if (W.w[i] & 1) return false;
    return true;
}

template <typename T, int NW>
hipError_t launch_stats16_nw(const T* in, int64_t nout, const Widths& W, const PeaksLayout& lay,
                             const PeaksWs& ws, dim3 grid, hipStream_t s) {
    if (W.w[0] & 1)
        hipLaunchKernelGGL((boxcar_stats16_kernel<T, NW, true>), grid, dim3(kThreads), 0, s, in, nout, lay.nbx, W,
                           lay.nseg, ws);
    else
        hipLaunchKernelGGL((boxcar_stats16_kernel<T, NW, false>), grid, dim3(kThreads), 0, s, in, nout, lay.nbx, W,
                           lay.nseg, ws);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_stats16(const void* in, int64_t nout, const Widths& W, const PeaksLayout& lay,
                          const PeaksWs& ws, dim3 grid, hipStream_t s) {
    switch (W.n) {
#define DD_NW(N) case N: return launch_stats16_nw<T, N>(static_cast<const T*>(in), nout, W, lay, ws, grid, s);
        DD_NW(4) DD_NW(5) DD_NW(6) DD_NW(7) DD_NW(8) DD_NW(9) DD_NW(10) DD_NW(11) DD_NW(12)
#undef DD_NW
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_stats(const void* in, int in_u16, int64_t nout, const Widths& W,
                        const PeaksLayout& lay, const PeaksWs& ws, dim3 grid, size_t lds,
                        hipStream_t s) {
    if (in_u16 && stats16_fits<uint16_t>(in, W, lay)) return launch_stats16<uint16_t>(in, nout, W, lay, ws, grid, s);
    if (!in_u16 && stats16_fits<int32_t>(in, W, lay)) return launch_stats16<int32_t>(in, nout, W, lay, ws, grid, s);
    return in_u16 ? launch_stats_w<uint16_t>(in, nout, W, lay, ws, grid, lds, s)
                  : launch_stats_w<int32_t>(in, nout, W, lay, ws, grid, lds, s);
}

PeaksLayout peaks_layout(int ndm, int64_t nout, const Widths& W) {
    PeaksLayout lay{};
    const int w_max = W.w[W.n - 1];
    lay.nbx = nout - w_max + 1;
    lay.L = segment_length(w_max);
    lay.nseg = static_cast<int>((lay.nbx + lay.L - 1) / lay.L);
    lay.nseries = static_cast<int64_t>(W.n) * ndm;
    lay.ncounts = lay.nseries * lay.nseg;
    lay.nchunks = static_cast<int>((lay.ncounts + kScanChunk - 1) / kScanChunk);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~size_t(255);
        return o;
    };
    lay.o_part_s1 = take(lay.ncounts * 8);
    lay.o_part_s2lo = take(lay.ncounts * 8);
    lay.o_part_s2hi = take(lay.ncounts * 8);
    lay.o_part_max = take(lay.ncounts * 4);
    lay.o_s1 = take(lay.nseries * 8);
    lay.o_s2lo = take(lay.nseries * 8);
    lay.o_s2hi = take(lay.nseries * 8);
    lay.o_thr = take(lay.nseries * 8);
    lay.o_thr32 = take(lay.nseries * 4);
    lay.o_sqrt_d = take(lay.nseries * 8);
    lay.o_counts = take(lay.ncounts * 4);
    lay.o_offs = take(lay.ncounts * 8);
    lay.o_chunk = take(static_cast<size_t>(lay.nchunks) * 8);
    lay.o_total = take(8);
    lay.o_list = take(static_cast<size_t>(ndm) * lay.nseg * 4);
    lay.o_list2 = take(static_cast<size_t>(ndm) * lay.nseg * 4);
    lay.o_nlist = take(8);
    lay.bytes = off;
    return lay;
}

PeaksWs peaks_ws(void* base, const PeaksLayout& lay) {
    char* b = static_cast<char*>(base);
    PeaksWs ws;
    ws.part_s1 = reinterpret_cast<uint64_t*>(b + lay.o_part_s1);
    ws.part_s2lo = reinterpret_cast<uint64_t*>(b + lay.o_part_s2lo);
    ws.part_s2hi = reinterpret_cast<uint64_t*>(b + lay.o_part_s2hi);
    ws.part_max = reinterpret_cast<uint32_t*>(b + lay.o_part_max);
    ws.s1 = reinterpret_cast<uint64_t*>(b + lay.o_s1);
    ws.s2lo = reinterpret_cast<uint64_t*>(b + lay.o_s2lo);
    ws.s2hi = reinterpret_cast<uint64_t*>(b + lay.o_s2hi);
    ws.thr = reinterpret_cast<int64_t*>(b + lay.o_thr);
    ws.thr32 = reinterpret_cast<uint32_t*>(b + lay.o_thr32);
    ws.sqrt_d = reinterpret_cast<double*>(b + lay.o_sqrt_d);
    ws.counts = reinterpret_cast<uint32_t*>(b + lay.o_counts);
    ws.soff = reinterpret_cast<int64_t*>(b + lay.o_offs);
    ws.offs = lay.nseg > kSeriesSegments ? ws.soff : nullptr;
    ws.tot = lay.nseg > 1 ? reinterpret_cast<uint32_t*>(ws.soff + lay.nseries) : ws.counts;
    ws.chunk_tot = reinterpret_cast<int64_t*>(b + lay.o_chunk);
    ws.total = reinterpret_cast<int64_t*>(b + lay.o_total);
    ws.list = reinterpret_cast<uint32_t*>(b + lay.o_list);
    ws.list2 = reinterpret_cast<uint32_t*>(b + lay.o_list2);
    ws.nlist = reinterpret_cast<uint32_t*>(b + lay.o_nlist);
    return ws;
}

hipError_t launch_scan_u32(const uint32_t* counts, int64_t n, int64_t* offs, int64_t* chunk_tot,
                           int64_t* total, hipStream_t s) {
    const int nchunks = static_cast<int>((n + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(scan_chunks_kernel, dim3(nchunks), dim3(kThreads), 0, s, counts, n, offs,
                       chunk_tot);
    hipLaunchKernelGGL(scan_totals_kernel, dim3(1), dim3(kThreads), 0, s, chunk_tot, nchunks, total);
    hipLaunchKernelGGL(scan_add_kernel, dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, offs, n, chunk_tot);
    return hipGetLastError();
}

int64_t scan_chunk_count(int64_t n) { return (n + kScanChunk - 1) / kScanChunk; }

template <typename T, int NT>
void launch_count_nt(const T* in, int ndm, int64_t nout, const Widths& W, const PeaksLayout& lay,
                     const PeaksWs& ws, size_t lds, hipStream_t s) {
    const int64_t nblk = std::min<int64_t>(static_cast<int64_t>(ndm) * lay.nseg, kListWaves * 64 / NT);
    set_lds_limit(reinterpret_cast<const void*>(peaks_count_kernel<T, NT>), lds);
    hipLaunchKernelGGL((peaks_count_kernel<T, NT>), dim3(static_cast<unsigned>(nblk)), dim3(NT), lds, s, in,
                       ndm, nout, lay.nbx, W, lay.L, lay.nseg, ws);
}

// launch(block size) of a list-driven pass (see list_threads).
template <typename F>
void launch_list(int threads, F launch) {
    if (threads == kFewThreads)
        launch(std::integral_constant<int, kFewThreads>{});
    else if (threads == kMidThreads)
        launch(std::integral_constant<int, kMidThreads>{});
    else
        launch(std::integral_constant<int, kThreads>{});
}

template <typename T>
void launch_count(const T* in, int ndm, int64_t nout, const Widths& W, const PeaksLayout& lay,
                  const PeaksWs& ws, size_t lds, int threads, hipStream_t s) {
    launch_list(threads, [&](auto nt) {
        launch_count_nt<T, decltype(nt)::value>(in, ndm, nout, W, lay, ws, lds, s);
    });
}

template <typename T, int NT>
void launch_write_nt(const T* in, int ndm, int64_t nout, const Widths& W, const PeaksLayout& lay,
                     const PeaksWs& ws, dedisp_event* events, int64_t capacity, size_t lds, hipStream_t s) {
    const int64_t nblk = std::min<int64_t>(static_cast<int64_t>(ndm) * lay.nseg, kListWaves * 64 / NT);
    set_lds_limit(reinterpret_cast<const void*>(peaks_write_kernel<T, NT>), lds);
    hipLaunchKernelGGL((peaks_write_kernel<T, NT>), dim3(static_cast<unsigned>(nblk)), dim3(NT), lds, s, in,
                       ndm, nout, lay.nbx, W, lay.L, lay.nseg, ws, events, capacity);
}

template <typename T>
void launch_write(const T* in, int ndm, int64_t nout, const Widths& W, const PeaksLayout& lay,
                  const PeaksWs& ws, dedisp_event* events, int64_t capacity, size_t lds, int threads,
                  hipStream_t s) {
    launch_list(threads, [&](auto nt) {
        launch_write_nt<T, decltype(nt)::value>(in, ndm, nout, W, lay, ws, events, capacity, lds, s);
    });
}

hipError_t launch_peaks_count(const void* in, int in_u16, int ndm, int64_t nout, const Widths& W,
                              const PeaksLayout& lay, const PeaksWs& ws, uint32_t kmant, int kexp2,
                              hipStream_t s) {
    const int w_max = W.w[W.n - 1];
    const size_t lds = peaks_lds_bytes(lay.L, w_max);
    const dim3 grid(static_cast<unsigned>(lay.nseg), static_cast<unsigned>(ndm));
    hipError_t e = launch_stats(in, in_u16, nout, W, lay, ws, grid, lds, s);
    if (e != hipSuccess) return e;
    const int nser = static_cast<int>(lay.nseries);
    hipLaunchKernelGGL(series_threshold_kernel, dim3((nser + kSerPerBlock - 1) / kSerPerBlock), dim3(kThreads),
                       0, s, nser, lay.nseg, lay.nbx, kmant, kexp2, ws);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nblk = static_cast<int64_t>(ndm) * lay.nseg;
    hipLaunchKernelGGL(mark_kernel, dim3(static_cast<unsigned>((nblk + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, ndm, lay.nseg, W.n, ws);
    const int threads = list_threads(nblk, lay.L, W.n, kmant, kexp2);
    if (in_u16)
        launch_count(static_cast<const uint16_t*>(in), ndm, nout, W, lay, ws, lds, threads, s);
    else
        launch_count(static_cast<const int32_t*>(in), ndm, nout, W, lay, ws, lds, threads, s);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ws.offs) return launch_scan_u32(ws.counts, lay.ncounts, ws.offs, ws.chunk_tot, ws.total, s);
    if (lay.nseries <= kOneBlockScan) {
        hipLaunchKernelGGL(scan_series_kernel, dim3(1), dim3(kScanThreads), 0, s, ws.tot, nser, ws.soff, ws.total);
        return hipGetLastError();
    }
    return launch_scan_u32(ws.tot, lay.nseries, ws.soff, ws.chunk_tot, ws.total, s);
}

hipError_t launch_peaks_write(const void* in, int in_u16, int ndm, int64_t nout, const Widths& W,
                              const PeaksLayout& lay, const PeaksWs& ws, dedisp_event* events,
                              int64_t capacity, uint32_t kmant, int kexp2, hipStream_t s) {
    const int w_max = W.w[W.n - 1];
    const size_t lds = peaks_lds_bytes(lay.L, w_max);
    const int threads = list_threads(static_cast<int64_t>(ndm) * lay.nseg, lay.L, W.n, kmant, kexp2);
    if (in_u16)
        launch_write(static_cast<const uint16_t*>(in), ndm, nout, W, lay, ws, events, capacity, lds, threads, s);
    else
        launch_write(static_cast<const int32_t*>(in), ndm, nout, W, lay, ws, events, capacity, lds, threads, s);
    return hipGetLastError();
}

}  // namespace dd
