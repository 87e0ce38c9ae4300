// Brute-force incoherent dedispersion (paper section 2.2):
//     out[d][t] = sum_c x[c][t + delay[d][c]],   0 <= t < nout.
//
// Design for gfx950 (integer gather-sum, no contraction, so no MFMA):
//   * input is the channel-major bit-plane copy made by repack.hip: 32
//     samples of one channel per {lo, hi} word pair;
//   * a block owns a tile of `ND` consecutive DM trials x T = 2048*G output
//     samples; its four waves each own ND/4 trials, every lane owns G
//     32-sample groups (lane-strided, so LDS reads are conflict-free);
//   * channels are streamed in stages of CS channels: the block copies, per
//     channel, the skewed window of words all its trials need into LDS
//     (one coalesced load shared by the ND trials), as 16-byte quads that
//     each hold two consecutive words (every word is stored twice);
//   * per (trial, channel) a lane reads one aligned quad per group (one
//     ds_read_b128, which moves about 1.5x the bytes per clock of the two
//     8-byte reads of unaligned word pairs) at an LDS offset taken from the
//     plan's per-tile-shape offset table (one scalar load per channel; the
//     table also carries the shift within the word), aligns the two words
//     to the trial's delay with one funnel shift per plane, and adds the 32
//     2-bit samples into a bit-sliced counter with carry-save adder trees:
//     8 channels at a time into a 5-level low counter (2 bit-operations per
//     input plane, see gen_csa.py), whose carry-out plane waits for the next
//     8 channels' so that the two ripple through the upper levels once;
//   * after the last stage the counter planes are transposed to integers in
//     registers and written once (int32 or uint16), through LDS.
// The result is exact; its order of additions is irrelevant (integers).
#include <algorithm>

#include "bitslice.hpp"
#include "dedisp_internal.hpp"

namespace {

// Waves per block when the work items fill the chip (and always in the
// persistent kernel); grids with few items use up to 16 (see few_shape).
constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kFewTrials = 16;   // trials of a DM block there
// L2 bytes of LDS-offset rows that one group of DM blocks may occupy: a
// quarter of an XCD's 4 MiB L2, the rest holding the input windows and the
// blocks' delay rows (one row per block).
constexpr int64_t kItemGroupBytes = int64_t(1) << 20;
constexpr int64_t kLdsBytes = 160 * 1024;   // LDS of a CU
constexpr int kFewStages = 8;               // few-items kernel: stages per buffer, at most

// Read-only tables (delays, skews, beam descriptors) are read through the
// constant address space: the loads stay scalar even after the output stores
// of an earlier work item, which would otherwise force them onto the vector
// memory path in the persistent kernel.
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
    return (cptr<T>)p;
}

// Word-wise copy of a descriptor out of the constant address space.
__device__ __forceinline__ dd::BeamArgs load_beam(cptr<dd::BeamArgs> p) {
    static_assert(sizeof(dd::BeamArgs) % 4 == 0, "descriptor size");
    constexpr int n = sizeof(dd::BeamArgs) / 4;
    const cptr<uint32_t> w = (cptr<uint32_t>)p;
    uint32_t tmp[n];
#pragma unroll
    for (int i = 0; i < n; ++i) tmp[i] = w[i];
    dd::BeamArgs a;
    __builtin_memcpy(&a, tmp, sizeof a);
    return a;
}

template <int NL, int N>
__device__ __forceinline__ void csa_add(uint32_t (&a)[NL], const uint32_t (&lo)[N],
                                        const uint32_t (&hi)[N]);

#define DD_CSA_SPEC(NL_, N_)                                                                   \
    template <>                                                                                \
    __device__ __forceinline__ void csa_add<NL_, N_>(uint32_t (&a)[NL_], const uint32_t (&lo)[N_], \
                                                     const uint32_t (&hi)[N_]) {               \
        csa_add_##N_##_##NL_(a, lo, hi);                                                       \
    }
DD_CSA_SPEC(12, 4) DD_CSA_SPEC(12, 8) DD_CSA_SPEC(12, 16) DD_CSA_SPEC(12, 32)
DD_CSA_SPEC(16, 4) DD_CSA_SPEC(16, 8) DD_CSA_SPEC(16, 16) DD_CSA_SPEC(16, 32)
#undef DD_CSA_SPEC

// Low counter of 5 levels per chunk (see gen_csa.py): the chunk's carry-out
// plane of weight 32 waits in `pend` for the next chunk's, and the two enter
// the upper levels together -- one ripple per two chunks instead of one per
// chunk.
template <int NL, int N>
__device__ __forceinline__ uint32_t csa_low(uint32_t (&a)[NL], const uint32_t (&lo)[N],
                                            const uint32_t (&hi)[N]) {
    if constexpr (N == 8)
        return csa5_add_8<NL>(a, lo, hi);
    else
        return csa5_add_4<NL>(a, lo, hi);
}

// Accumulate channels [c, c+N) of the current stage for one trial into the
// counters of its G groups.
// The trial's offset-table row gives, per channel, the LDS byte offset of the
// channel's first needed quad (bits 5 and up) and the funnel shift (bits 0-4,
// which is all the shift instruction reads).  A quad is a 16-byte aligned
// copy of two consecutive words, so each (trial, channel, group) is one
// aligned 16-byte LDS read.
template <int NL, int G, int N, bool ODD>
__device__ __forceinline__ void accumulate_chunk(uint32_t (&acc)[G][NL], uint32_t (&pend)[G],
                                                 const char* lds_lane, cptr<uint32_t> trow, int c) {
    uint32_t e[N];
#pragma unroll
    for (int k = 0; k < N; ++k) e[k] = trow[c + k];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        // all N reads first, then the shifts: the reads' latencies overlap
        uint4 w[N];
#pragma unroll
        for (int k = 0; k < N; ++k)
            w[k] = *reinterpret_cast<const uint4*>(lds_lane + (e[k] >> 5) + 1024 * g);
        uint32_t lo[N], hi[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            lo[k] = bs::funnel(w[k].z, w[k].x, e[k]);
            hi[k] = bs::funnel(w[k].w, w[k].y, e[k]);
        }
        const uint32_t cy = csa_low<NL, N>(acc[g], lo, hi);
        if (ODD)
            bs::carry_in2<NL, 5>(acc[g], pend[g], cy);
        else
            pend[g] = cy;
    }
}

// One chunk, completing a pair of carry-outs when it is the second of two.
template <int NL, int G, int N>
__device__ __forceinline__ void chunk(uint32_t (&acc)[G][NL], uint32_t (&pend)[G], int k,
                                      const char* lds_lane, cptr<uint32_t> trow, int c) {
    if (k & 1)
        accumulate_chunk<NL, G, N, true>(acc, pend, lds_lane, trow, c);
    else
        accumulate_chunk<NL, G, N, false>(acc, pend, lds_lane, trow, c);
}

// Asynchronous copy of one channel's row of an LDS stage (a.pitch quads of 16
// bytes).  Quad j of the row holds the words j and j + 1 of the window that
// starts at word w_base + (dlo >> 5), dlo the delay of the DM block's first
// trial: stride - 1 quads cover the `stride` words, cut at the end of the
// channel's words (what lies beyond only feeds output samples past nout, which
// are never stored).  Each lane copies one quad, global -> LDS directly (16
// bytes from an 8-byte aligned word address); the copies complete
// asynchronously: the caller waits for them before the barrier that publishes
// the stage.
__device__ __forceinline__ void fill_row(const dd::BeamArgs& a, int dlo, int64_t w_base, int stride, int c,
                                         char* __restrict__ dst, int lane) {
    const int64_t w0 = w_base + (dlo >> 5);
    // words of the row from w0 on: > 0 (w0 < nsamps / 32 + 1 < nwords) and
    // below 2^31, so the bound is 32-bit scalar arithmetic (a 64-bit
    // signed compare would go through vector registers)
    const int avail = static_cast<int>(a.nwords - w0);
    const int nq = min(avail, stride) - 1;
    // uniform source row; each lane adds its own 8-byte word offset
    const uint2* src = a.words + static_cast<int64_t>(c) * a.nwords + w0;
    // full batches of 64 quads need no per-lane check; only the last,
    // partial one (if any) compares lanes
    int i = 0;
    for (; i + 64 <= nq; i += 64)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i + lane),
                                         (__attribute__((address_space(3))) void*)(dst + 16 * i), 16, 0, 0);
    if (i < nq && lane < nq - i)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i + lane),
                                         (__attribute__((address_space(3))) void*)(dst + 16 * i), 16, 0, 0);
}

// Copy of channels [c0, c0 + cs), channel c0 + r into row r; cs is a multiple
// of BATCH.  The waves take BATCH consecutive rows at a time, whose delay
// entries come from one scalar load: a load per row put its latency before
// every row's copies (survey beam 4865 -> 4804 us with batches of 2).
template <int NWV, int BATCH>
__device__ __forceinline__ void fill_stage(const dd::BeamArgs& a, cptr<int32_t> dlo_row,
                                           int64_t w_base, int stride, int c0, int cs,
                                           char* __restrict__ lds, int lane, int wave) {
    for (int r0 = wave * BATCH; r0 < cs; r0 += NWV * BATCH) {
        int dlo[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) dlo[k] = dlo_row[c0 + r0 + k];
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
            fill_row(a, dlo[k], w_base, stride, c0 + r0 + k, lds + (r0 + k) * a.pitch * 16, lane);
    }
}

// One stage: start the copy of the next stage into `nxt` (if any), then add
// this stage's channels from `cur`.  The two buffers are passed as restrict
// pointers so the compiler knows the LDS reads do not wait on the copy.
template <int NL, int NDW, int G, int NWV>
__device__ __forceinline__ void run_stage(const dd::BeamArgs& a, uint32_t (&acc)[NDW][G][NL],
                                          uint32_t (&pend)[NDW][G], int kbase,
                                          cptr<int32_t> dlo_row, int64_t w_base, int stride,
                                          int c0, int stage_chans, int d_lo,
                                          const char* __restrict__ cur, char* __restrict__ nxt,
                                          bool more, int lane, int wave) {
    const int cs = min(stage_chans, a.nchans - c0);
    if (more)
        fill_stage<NWV, 1>(a, dlo_row, w_base, stride, c0 + stage_chans,
                        min(stage_chans, a.nchans - c0 - stage_chans), nxt, lane, wave);
#pragma unroll
    for (int i = 0; i < NDW; ++i) {
        const int d = d_lo + wave + NWV * i;
        if (d < a.ndm) {
            const cptr<uint32_t> trow = as_const(a.offs) + static_cast<int64_t>(d) * a.nchans;
            int cl = 0, k = kbase;
            // 8-channel steps: fewer live registers than 16, more resident waves
#pragma unroll 1
            for (; cl + 8 <= cs; cl += 8, ++k)
                chunk<NL, G, 8>(acc[i], pend[i], k, cur + 16 * lane, trow, c0 + cl);
            if (cl + 4 <= cs) chunk<NL, G, 4>(acc[i], pend[i], k, cur + 16 * lane, trow, c0 + cl);
        }
    }
}

// One stage of exactly 8 channels: start the copy of the next stage, then add
// this stage's 8-channel chunk for every trial.  SECOND: the chunk is the
// second of a pair (its carry-out joins the first one's).
template <int NL, int NDW, int G, int NWV, bool SECOND>
__device__ __forceinline__ void stage8(const dd::BeamArgs& a, uint32_t (&acc)[NDW][G][NL],
                                       uint32_t (&pend)[NDW][G], cptr<int32_t> dlo_row,
                                       int64_t w_base, int stride, int c0, int d_lo,
                                       const char* __restrict__ cur, char* __restrict__ nxt,
                                       bool more, int lane, int wave) {
    if (more) fill_stage<NWV, 8 / NWV>(a, dlo_row, w_base, stride, c0 + 8, 8, nxt, lane, wave);
#pragma unroll
    for (int i = 0; i < NDW; ++i) {
        // a trial past the last one (a short last DM block) repeats the last
        // trial's offsets, so the code has no branch; its sums are never stored
        const int d = min(d_lo + wave + NWV * i, a.ndm - 1);
        const cptr<uint32_t> trow = as_const(a.offs) + static_cast<int64_t>(d) * a.nchans;
        accumulate_chunk<NL, G, 8, SECOND>(acc[i], pend[i], cur + 16 * lane, trow, c0);
        // The trial's sums must exist here (an empty statement that reads and
        // writes them): the compiler may not sink the adds past the next
        // stage's barrier, where every trial's quads would be live at once.
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int l = 0; l < NL; ++l) asm volatile("" : "+v"(acc[i][g][l]));
            asm volatile("" : "+v"(pend[i][g]));
        }
    }
}

// The n stages of 8 channels of one LDS buffer (first channel c0), for a wave
// that owns one trial: the quads of a step are read, and its successor's
// table entries loaded, before the adds of the step before it.  A wave's chain
// (table entry -> LDS read -> adds) then overlaps itself, where few waves per
// SIMD leave nothing else to hide it (2 to 7% over reads just before the adds).
struct Step {
    uint32_t e[8];
    uint4 w[8];
};

__device__ __forceinline__ void step_entries(Step& s, cptr<uint32_t> trow, int c) {
#pragma unroll
    for (int k = 0; k < 8; ++k) s.e[k] = trow[c + k];
}

__device__ __forceinline__ void step_quads(Step& s, const char* lds_lane) {
#pragma unroll
    for (int k = 0; k < 8; ++k) s.w[k] = *reinterpret_cast<const uint4*>(lds_lane + (s.e[k] >> 5));
}

template <int NL, bool SECOND>
__device__ __forceinline__ void step_adds(const Step& s, uint32_t (&acc)[NL], uint32_t& pend) {
    uint32_t lo[8], hi[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        lo[k] = bs::funnel(s.w[k].z, s.w[k].x, s.e[k]);
        hi[k] = bs::funnel(s.w[k].w, s.w[k].y, s.e[k]);
    }
    const uint32_t cy = csa_low<NL, 8>(acc, lo, hi);
    if (SECOND)
        bs::carry_in2<NL, 5>(acc, pend, cy);
    else
        pend = cy;
}

template <int NL>
__device__ __forceinline__ void deep_stages(uint32_t (&acc)[NL], uint32_t& pend, cptr<uint32_t> trow,
                                            int c0, int n, const char* lds_lane, int64_t sub) {
    Step a, b;
    step_entries(a, trow, c0);
    step_quads(a, lds_lane);
    step_entries(b, trow, c0 + 8 * min(1, n - 1));
    int q = 0;
#pragma unroll 1
    for (; q + 1 < n; q += 2) {   // past the last stage the last one is read again
        Step a2, b2;
        step_quads(b, lds_lane + (q + 1) * sub);
        step_entries(a2, trow, c0 + 8 * min(q + 2, n - 1));
        __builtin_amdgcn_sched_barrier(0);
        step_adds<NL, false>(a, acc, pend);
        __builtin_amdgcn_sched_barrier(0);
        step_quads(a2, lds_lane + min(q + 2, n - 1) * sub);
        step_entries(b2, trow, c0 + 8 * min(q + 3, n - 1));
        __builtin_amdgcn_sched_barrier(0);
        step_adds<NL, true>(b, acc, pend);
        __builtin_amdgcn_sched_barrier(0);
        a = a2;
        b = b2;
    }
    if (q < n) step_adds<NL, false>(a, acc, pend);   // the last stage of an odd number
}

// Bytes of LDS a wave stages its output in: 2048 samples of 16 bits.
constexpr int kStoreBytes = 4096;

// Four words at any element boundary (2 bytes), one 16-byte store.
struct __attribute__((packed, aligned(2))) Words4 {
    uint32_t w[4];
};

// Store a wave's 2048 consecutive outputs, lane l holding samples 32 l + b as
// r[b & 15]'s half b >> 4, at element `at` of the series; the first n are
// inside the row.  A lane's own 32 samples are 64 or 128 consecutive bytes, so
// stores straight from the registers touched 64 lines each, four bytes apiece
// (and two bytes at a time where a row of odd length put them off alignment).
// The tile goes through LDS instead (16-byte chunk k of lane l at chunk
// k ^ (l >> 2 & 3): no bank conflicts) and out in stores of 1 KiB.  It shows
// where few channels are added per output: the 16 x 8 subband plan of the
// survey beam, 64 channels per stage-1 output, 3.49 -> 2.67 ms; the direct sum
// of its 1024 channels 4.80 -> 4.74.
template <bool OUT16>
__device__ __forceinline__ void store_tile(const uint32_t (&r)[16], void* out, int64_t at, int n,
                                           char* buf, int lane) {
    // chunk k: samples 32 l + 8 k .. + 7
    uint4* own = reinterpret_cast<uint4*>(buf) + 4 * lane;
    const int sw = (lane >> 2) & 3;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = r[(8 * k + 2 * j) & 15], y = r[(8 * k + 2 * j + 1) & 15];
            v[j] = k < 2 ? __builtin_amdgcn_perm(y, x, 0x05040100u) : __builtin_amdgcn_perm(y, x, 0x07060302u);
        }
        own[k ^ sw] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    // the wave's lanes exchange through the buffer
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (OUT16) {
        // 16-byte chunk 64 i + lane (of lane l' = 16 i + lane / 4)
        const uint4* src = reinterpret_cast<const uint4*>(buf) + (lane ^ ((lane >> 4) & 3));
        uint16_t* o = static_cast<uint16_t*>(out) + at + 8 * lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = src[64 * i];
            const int left = n - 8 * (64 * i + lane);   // samples of the row from this chunk on
            if (left >= 8) {
                *reinterpret_cast<Words4*>(o + 512 * i) = Words4{{v.x, v.y, v.z, v.w}};
            } else if (left > 0) {
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int b = 0; b < 7; ++b)
                    if (b < left) o[512 * i + b] = static_cast<uint16_t>(w[b >> 1] >> (16 * (b & 1)));
            }
        }
    } else {
        // 8-byte half chunk 64 i + lane (of lane l' = 8 i + lane / 8)
        int32_t* o = static_cast<int32_t*>(out) + at + 4 * lane;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = (lane >> 1) ^ (((lane >> 5) & 1) | (2 * (i & 1)));
            const uint2 v = reinterpret_cast<const uint2*>(buf)[64 * i + 2 * c + (lane & 1)];
            const uint32_t w[4] = {v.x & 0xFFFFu, v.x >> 16, v.y & 0xFFFFu, v.y >> 16};
            const int left = n - 4 * (64 * i + lane);
            if (left >= 4) {
                *reinterpret_cast<Words4*>(o + 256 * i) = Words4{{w[0], w[1], w[2], w[3]}};
            } else {
#pragma unroll
                for (int b = 0; b < 3; ++b)
                    if (b < left) o[256 * i + b] = static_cast<int32_t>(w[b]);
            }
        }
    }
    // the next tile overwrites the buffer
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One work item: DM block `dblk` x time tile `tile` of one beam.
//
// The LDS holds two stage buffers of `stage_chans` rows each; stage s lives in
// buffer s & 1, channel c in row c mod stage_chans of it -- the row the offset
// table assumes.  While the waves work on stage s, the copy of
// stage s + 1 into the other buffer is in flight.  With DEEP (S8 only) a
// buffer holds `nsub` stages of 8 channels, copied and published together:
// stage q of the buffer takes rows 8 q .. 8 q + 7.
template <int NL, int NDW, int G, bool OUT16, bool S8, int NWV = kWaves, bool DEEP = false,
          int ND = NDW * NWV>
__device__ __forceinline__ void process_item(const dd::BeamArgs& a, int tile, int dblk,
                                             int stage_chans, char* lds, int lane, int wave,
                                             int nsub = 1, int d_sub = 0) {
    // the block takes NDW * NWV of the DM block's ND trials, from d_sub on
    constexpr int T = 2048 * G;
    const int64_t T0 = static_cast<int64_t>(tile) * T;
    const int d_blk = dblk * ND;
    const int d_lo = d_blk + d_sub;
    // words this block needs per channel row (<= a.pitch + 1)
    const int stride = a.tile_words + as_const(a.skew)[dblk];
    const int64_t w_base = T0 >> 5;
    const cptr<int32_t> dlo_row = as_const(a.delays) + static_cast<int64_t>(d_blk) * a.nchans;
    const int nst = (a.nchans + stage_chans - 1) / stage_chans;

    uint32_t acc[NDW][G][NL];
    uint32_t pend[NDW][G];
#pragma unroll
    for (int i = 0; i < NDW; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            pend[i][g] = 0u;
#pragma unroll
            for (int l = 0; l < NL; ++l) acc[i][g][l] = 0u;
        }
    int kbase = 0;   // chunks added so far (the same for every trial)

    // rows per wave: 4 at a time of a deep buffer, an 8-channel stage's 8 / NWV
    constexpr int kFill = DEEP ? 4 : S8 ? 8 / NWV : 1;
    fill_stage<NWV, kFill>(a, dlo_row, w_base, stride, 0, min(stage_chans * nsub, a.nchans), lds, lane, wave);
    const int64_t half = static_cast<int64_t>(stage_chans) * nsub * a.pitch * 16;   // bytes
    if constexpr (DEEP) {
        const int64_t sub = static_cast<int64_t>(8) * a.pitch * 16;   // bytes of one stage
        char* cur = lds;
        char* nxt = lds + half;
#pragma unroll 1
        for (int s0 = 0; s0 < nst; s0 += nsub) {   // nsub is even: pairs never cross buffers
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (s0 + nsub < nst)
                fill_stage<NWV, kFill>(a, dlo_row, w_base, stride, 8 * (s0 + nsub),
                                       8 * min(nsub, nst - s0 - nsub), nxt, lane, wave);
            const int d = min(d_lo + wave, a.ndm - 1);
            deep_stages<NL>(acc[0][0], pend[0][0], as_const(a.offs) + static_cast<int64_t>(d) * a.nchans,
                            8 * s0, min(nsub, nst - s0), cur + 16 * lane, sub);
            char* t = cur;
            cur = nxt;
            nxt = t;
        }
        kbase = nst;
    } else if constexpr (S8) {
        // stages of 8 channels, every one full: pairs of stages, the first in
        // buffer 0 and the second in buffer 1, so the pairing of carry-outs
        // and the buffers are fixed in the code
        int st = 0;
#pragma unroll 1
        for (; st + 1 < nst; st += 2) {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            stage8<NL, NDW, G, NWV, false>(a, acc, pend, dlo_row, w_base, stride, 8 * st, d_lo, lds,
                                      lds + half, true, lane, wave);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            stage8<NL, NDW, G, NWV, true>(a, acc, pend, dlo_row, w_base, stride, 8 * st + 8, d_lo,
                                     lds + half, lds, st + 2 < nst, lane, wave);
        }
        kbase = st;
        if (st < nst) {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            stage8<NL, NDW, G, NWV, false>(a, acc, pend, dlo_row, w_base, stride, 8 * st, d_lo, lds,
                                      lds + half, false, lane, wave);
            kbase = nst;
        }
    }
#pragma unroll 1
    for (int st = 0; st < (S8 || DEEP ? 0 : nst); ++st) {
        const int c0 = st * stage_chans;
        // this wave's copies of stage st are done; after the barrier every
        // wave's are, and every wave has finished stage st - 1, whose buffer
        // the copy of stage st + 1 now overwrites
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        run_stage<NL, NDW, G, NWV>(a, acc, pend, kbase, dlo_row, w_base, stride, c0, stage_chans, d_lo,
                              (st & 1) ? lds + half : lds, (st & 1) ? lds : lds + half,
                              st + 1 < nst, lane, wave);
        const int cs = min(stage_chans, a.nchans - c0);
        kbase += cs / 8 + ((cs & 4) ? 1 : 0);
    }
    // an odd number of chunks leaves one carry-out waiting
    if (kbase & 1) {
#pragma unroll
        for (int i = 0; i < NDW; ++i)
#pragma unroll
            for (int g = 0; g < G; ++g) bs::carry_in1<NL, 5>(acc[i][g], pend[i][g]);
    }

    // Write: counters -> integers.  Every wave has left the stage buffers
    // (kStoreBytes per wave of them hold its output tile now).
    __syncthreads();
    char* tile_buf = lds + wave * kStoreBytes;
#pragma unroll
    for (int i = 0; i < NDW; ++i) {
        const int d = d_lo + wave + NWV * i;
        if (d >= a.ndm) continue;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t t0 = T0 + 2048 * g;
            if (t0 >= a.nout) continue;
            // one tile after the other: their transposes at once would take
            // the kernel's registers
#pragma unroll
            for (int l = 0; l < NL; ++l) asm volatile("" : "+v"(acc[i][g][l]) : : "memory");
            uint32_t r[16];
            bs::planes_to_pairs<NL>(acc[i][g], r);
            store_tile<OUT16>(r, a.out, static_cast<int64_t>(d) * a.nout + t0,
                              static_cast<int>(min<int64_t>(2048, a.nout - t0)), tile_buf, lane);
        }
    }
}

// Work items go in groups of a.dm_group DM blocks: inside a group the DM
// block varies fastest, then the time tile.  The group's offset rows then stay
// in L2 while its time tiles go by, and the DM blocks of one time tile, whose
// input windows overlap, run together.
__device__ __forceinline__ void item_coords(const dd::BeamArgs& a, int64_t item, int* tile,
                                            int* dblk) {
    const int64_t n_tt = a.n_items / a.n_dm_blocks;
    const int64_t per_group = static_cast<int64_t>(a.dm_group) * n_tt;
    const int g = static_cast<int>(item / per_group);
    const int64_t rem = item - g * per_group;
    const int gs = min(a.dm_group, a.n_dm_blocks - g * a.dm_group);
    *tile = static_cast<int>(rem / gs);
    *dblk = g * a.dm_group + static_cast<int>(rem % gs);
}

// The 12-level, 16-trial, one-group shape (the survey's) asks for 5 waves
// per SIMD: the int32 stores, and the item queue's extra scalars in the
// persistent kernel, would otherwise take a few registers more and leave 4
// (the compiler then spills per-item values to scratch instead).
template <int NL, int NDW, int G>
constexpr int min_waves() {
    return (NL == 12 && NDW == 4 && G == 1) ? 5 : 1;
}

template <int NL, int NDW, int G, bool OUT16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(min_waves<NL, NDW, G>())))
void dedisperse_kernel(dd::BeamArgs a, int stage_chans,
                                                              int n_items) {
    extern __shared__ uint4 lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // XCD-aware order: hardware deals consecutive blocks round-robin to the 8
    // XCDs; give each XCD a contiguous run of (time tile, DM block) items with
    // the DM block fastest, so blocks resident on one XCD share input words in
    // its L2.
    const int per_xcd = gridDim.x / 8;
    const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (item >= n_items) return;
    int tile, dblk;
    item_coords(a, item, &tile, &dblk);
    if (stage_chans == 8 && (a.nchans & 7) == 0)
        process_item<NL, NDW, G, OUT16, true>(a, tile, dblk, 8, reinterpret_cast<char*>(lds), lane,
                                              wave);
    else
        process_item<NL, NDW, G, OUT16, false>(a, tile, dblk, stage_chans,
                                               reinterpret_cast<char*>(lds), lane, wave);
}

// The same over the items of several inputs (the subbands of a two-stage plan),
// whose launches one by one each start and drain the chip.  The whole two-stage
// call, us, with a launch per subband and with one: survey beam 16 x 8 2446 and
// 2340, 1024 channels x 2^16, 13 coarse trials, 16
// subbands 271 and 160 (32 items each), 256 x 2^15, 25 x 8 84 and 49.
struct ManyArgs {
    dd::BeamArgs b[dd::kMaxMany];
};
static_assert(sizeof(ManyArgs) <= 4000, "kernel arguments");

template <int NL, int NDW, int G, bool OUT16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(min_waves<NL, NDW, G>())))
void dedisperse_many_kernel(ManyArgs m, int n, int stage_chans, int n_items) {
    extern __shared__ uint4 lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = gridDim.x / 8;
    const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (item >= n_items) return;
    int b = 0;
    while (b + 1 < n && item >= m.b[b + 1].item_begin) ++b;
    const dd::BeamArgs a = m.b[b];
    int tile, dblk;
    item_coords(a, item - a.item_begin, &tile, &dblk);
    if (stage_chans == 8 && (a.nchans & 7) == 0)
        process_item<NL, NDW, G, OUT16, true>(a, tile, dblk, 8, reinterpret_cast<char*>(lds), lane,
                                              wave);
    else
        process_item<NL, NDW, G, OUT16, false>(a, tile, dblk, stage_chans,
                                               reinterpret_cast<char*>(lds), lane, wave);
}

// Form for grids with too few items to fill the chip: an item's kFewTrials
// trials go to kFewTrials / NWV blocks of NWV waves, one trial per wave, on
// the ordinary kernel's tile and tables, with nsub stages per buffer (see
// few_shape).
template <int NL, int NWV, bool OUT16>
__global__ __launch_bounds__(64 * NWV) void dedisperse_few_kernel(dd::BeamArgs a, int n_items, int nsub) {
    extern __shared__ uint4 lds[];
    constexpr int kSplit = kFewTrials / NWV;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_xcd = gridDim.x / 8;
    const int b = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const int item = b / kSplit;
    if (item >= n_items) return;
    int tile, dblk;
    item_coords(a, item, &tile, &dblk);
    const int d_sub = (b % kSplit) * NWV;
    if (dblk * kFewTrials + d_sub >= a.ndm) return;
    process_item<NL, 1, 1, OUT16, true, NWV, true, kFewTrials>(
        a, tile, dblk, 8, reinterpret_cast<char*>(lds), lane, wave, nsub, d_sub);
}

// Persistent form over the work items of several beams: blocks pop items
// from `nq` queues (block b serves queue b % nq; queue q owns the contiguous
// item range [q*total/nq, (q+1)*total/nq)), so that the blocks of one XCD work
// through neighbouring (beam, time tile, DM block) items.  Every block leaves
// once its queue is drained.
template <int NL, int NDW, int G, bool OUT16>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(min_waves<NL, NDW, G>())))
void dedisperse_persistent_kernel(
    const dd::BeamArgs* __restrict__ beams, int nbeams, int64_t total, int stage_chans,
    unsigned long long* __restrict__ counters, int nq) {
    extern __shared__ uint4 lds[];
    __shared__ long long item_sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = blockIdx.x % nq;
    const int64_t q_lo = total * q / nq;
    const int64_t q_hi = total * (q + 1) / nq;
    for (;;) {
        if (threadIdx.x == 0) item_sh = static_cast<long long>(q_lo + atomicAdd(&counters[q], 1ull));
        __syncthreads();
        // The popped item is uniform over the block: keep it (and all that is
        // derived from it: beam, delay rows, skew) in scalar registers.
        const unsigned long long raw = static_cast<unsigned long long>(item_sh);
        const int64_t item = static_cast<int64_t>(
            (static_cast<unsigned long long>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(raw >> 32))) << 32) |
            static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(raw))));
        __syncthreads();
        if (item >= q_hi) break;
        const cptr<dd::BeamArgs> cb = as_const(beams);
        int b = 0;
        while (b + 1 < nbeams && item >= cb[b + 1].item_begin) ++b;
        const dd::BeamArgs a = load_beam(cb + b);
        const int64_t local = item - a.item_begin;
        int tile, dblk;
        item_coords(a, local, &tile, &dblk);
        if (stage_chans == 8 && (a.nchans & 7) == 0)
            process_item<NL, NDW, G, OUT16, true>(a, tile, dblk, 8, reinterpret_cast<char*>(lds),
                                                  lane, wave);
        else
            process_item<NL, NDW, G, OUT16, false>(a, tile, dblk, stage_chans,
                                                   reinterpret_cast<char*>(lds), lane, wave);
    }
}

__global__ void zero_counters_kernel(unsigned long long* c, int n) {
    if (static_cast<int>(threadIdx.x) < n) c[threadIdx.x] = 0ull;
}

template <int NL, int NDW, int G, bool OUT16>
hipError_t launch_cfg(const dd::BeamArgs& a, int stage_chans, size_t lds, hipStream_t s) {
    auto kern = dedisperse_kernel<NL, NDW, G, OUT16>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    if (a.n_items > (int64_t(1) << 30)) return hipErrorInvalidValue;
    const int64_t nblocks = 8 * ((a.n_items + 7) / 8);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(nblocks)), dim3(kThreads), lds, s, a,
                       stage_chans, static_cast<int>(a.n_items));
    return hipGetLastError();
}

template <int NL, int NDW, int G>
hipError_t launch_many_cfg(const ManyArgs& m, int n, int64_t total, int stage_chans, size_t lds, hipStream_t s) {
    auto kern = dedisperse_many_kernel<NL, NDW, G, true>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    const int64_t nblocks = 8 * ((total + 7) / 8);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(nblocks)), dim3(kThreads), lds, s, m, n, stage_chans,
                       static_cast<int>(total));
    return hipGetLastError();
}

// Launch shape of a grid with few items (waves == 0: the ordinary kernel).
//
// The ordinary kernel gives an item four waves of four trials, 16 channels in
// flight: with at most two items per CU the chip waits for each block's chain
// of stages (1024 channels: 195 us with 0.16, 260 us with 1.75 items per CU).
// One trial per wave makes that chain a quarter as long, and a CU's whole LDS
// holds 8 stages per buffer, so the copies' latency and the barrier are paid
// once per 64 channels.  16 waves per block fill a CU by themselves: 89-100 us
// up to one item per CU, 190 us up to two (1024 channels; 4096: 960 -> 370 and
// 960 -> 730 us).  Up to half an item per CU, halving the trials per block
// uses twice the CUs: 70-79 us.  Above two items per CU the ordinary kernel's
// more adds per table entry and copy win (2.5: 295 against 296 us, 3.5: 345
// against 381).  A plan with a tuned tile takes this form as well, but for just
// above one item per CU, where a second pass runs nearly empty: of the other tiles
// the best takes 174 us at 1.09 items per CU of 1024 channels, this form 187; 142
// and 95 at 0.88, 209 and 187 at 1.75.
struct FewShape {
    int waves, nsub;
};

// `a` at the default tile; `tuned`: the plan has another.
FewShape few_shape(const dd::BeamArgs& a, bool tuned, int device) {
    constexpr FewShape kNone = {0, 0};
    static_assert(dd::kDefaultTile.dms_per_block == kFewTrials && dd::kDefaultTile.groups == 1 &&
                  dd::kDefaultTile.stage_chans == 8, "the form's tile");
    if (a.nchans & 7) return kNone;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1)
        return kNone;
    if (a.n_items > 2 * static_cast<int64_t>(cus)) return kNone;
    if (tuned && a.n_items > cus && 4 * a.n_items <= 5 * static_cast<int64_t>(cus)) return kNone;
    // pairs of stages that both buffers hold in a CU's LDS (one block per CU)
    const int64_t pair = 2 * int64_t(16) * a.pitch * 16;
    const int64_t n = std::min<int64_t>({kLdsBytes / pair, kFewStages / 2, (a.nchans / 8 + 1) / 2});
    if (n < 1) return kNone;
    return {2 * a.n_items <= cus ? 8 : 16, static_cast<int>(2 * n)};
}

template <int NL, int NWV, bool OUT16>
hipError_t launch_few(const dd::BeamArgs& a, int nsub, hipStream_t s) {
    auto kern = dedisperse_few_kernel<NL, NWV, OUT16>;
    const size_t lds = std::max(static_cast<size_t>(nsub) * 2 * 8 * a.pitch * 16,
                                static_cast<size_t>(NWV) * kStoreBytes);
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    const int64_t nblocks = 8 * ((a.n_items * (kFewTrials / NWV) + 7) / 8);
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(nblocks)), dim3(64 * NWV), lds, s, a,
                       static_cast<int>(a.n_items), nsub);
    return hipGetLastError();
}

template <int NL, bool OUT16>
hipError_t launch_few_shape(const dd::BeamArgs& a, const FewShape& f, hipStream_t s) {
    return f.waves == 16 ? launch_few<NL, 16, OUT16>(a, f.nsub, s) : launch_few<NL, 8, OUT16>(a, f.nsub, s);
}

template <int NL, int NDW, int G, bool OUT16>
hipError_t launch_persistent_cfg(const dd::BeamArgs* beams, int nbeams, int64_t total,
                                 int stage_chans, size_t lds, unsigned long long* counters, int nq,
                                 int grid, hipStream_t s) {
    auto kern = dedisperse_persistent_kernel<NL, NDW, G, OUT16>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, s, counters, nq);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, beams, nbeams, total, stage_chans,
                       counters, nq);
    return hipGetLastError();
}

template <int NL, int NDW, int G, bool OUT16>
int occupancy_cfg(size_t lds) {
    auto kern = dedisperse_persistent_kernel<NL, NDW, G, OUT16>;
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess)
        return 0;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, kThreads, lds) != hipSuccess) return 0;
    return n;
}

}  // namespace

namespace dd {


int tile_pitch(const dedisp_plan_s* p, const TileConfig& cfg) {
    // quads per LDS row: one fewer than the words a row covers
    const int k = dm_block_index(cfg.dms_per_block);
    return k < 0 ? 0 : 2048 * cfg.groups / 32 + p->skew_max[k];
}

size_t tile_lds_bytes(const dedisp_plan_s* p, const TileConfig& cfg) {
    // two stage buffers of stage_chans rows of 16-byte quads, the waves'
    // output tiles in their place at the end
    return std::max(2 * static_cast<size_t>(cfg.stage_chans) * tile_pitch(p, cfg) * sizeof(uint4),
                    static_cast<size_t>(kWaves) * kStoreBytes);
}

BeamArgs beam_args(const dedisp_plan_s* p, const uint2* words, int64_t nwords, int64_t nout,
                   void* out, const TileConfig& cfg) {
    const int k = dm_block_index(cfg.dms_per_block);
    BeamArgs a{};
    a.words = words;
    a.nwords = nwords;
    a.nchans = p->nchans;
    a.ndm = p->ndm;
    a.nout = nout;
    a.delays = p->d_delays;
    a.offs = offset_table(p, cfg, false);
    a.skew = k >= 0 ? p->d_skew[k] : nullptr;
    a.out = out;
    a.n_dm_blocks = (p->ndm + cfg.dms_per_block - 1) / cfg.dms_per_block;
    // groups whose LDS-offset rows (4 bytes per trial and channel) fill about
    // kItemGroupBytes of L2
    const int64_t rows = static_cast<int64_t>(cfg.dms_per_block) * p->nchans * 4;
    a.dm_group = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(a.n_dm_blocks, kItemGroupBytes / rows)));
    const int64_t T = 2048 * cfg.groups;
    a.tile_words = static_cast<int>(T / 32 + 1);
    a.pitch = tile_pitch(p, cfg);
    a.item_begin = 0;
    a.n_items = ((nout + T - 1) / T) * a.n_dm_blocks;
    return a;
}

#define DD_SHAPES(X)                                                                   \
    X(12, 1, 1) X(12, 2, 1) X(12, 4, 1) X(12, 8, 1) X(12, 1, 2) X(12, 2, 2) X(12, 4, 2)   \
    X(16, 1, 1) X(16, 2, 1) X(16, 4, 1) X(16, 8, 1) X(16, 1, 2) X(16, 2, 2) X(16, 4, 2)

dedisp_status launch_dedisperse(const dedisp_plan_s* p, const uint2* words, int64_t nwords,
                                int64_t nout, void* out, int out_u16, const TileConfig& cfg,
                                Form form, hipStream_t s) {
    const int k = dm_block_index(cfg.dms_per_block);
    if (k < 0 || cfg.stage_chans < 4 || cfg.stage_chans % 4 || cfg.groups < 1 || cfg.groups > 2)
        return fail(DEDISP_ERR_INVALID_ARG, "unsupported tile configuration");
    const size_t lds = tile_lds_bytes(p, cfg);
    if (lds > 160 * 1024)
        return fail(DEDISP_ERR_UNSUPPORTED,
                    "DM block of %d trials spans %d words of skew: LDS tile of %zu bytes too large",
                    cfg.dms_per_block, p->skew_max[k], lds);
    const int nl = levels_for(p->nchans);
    dedisp_status st = DEDISP_OK;
    if (!offset_table(p, cfg, true, &st)) return st;
    const BeamArgs a = beam_args(p, words, nwords, nout, out, cfg);
    hipError_t e = hipErrorInvalidValue;
    const bool own = same_tile(cfg, kDefaultTile);
    if (form == Form::kPlan || (form == Form::kTile && own)) {
        const BeamArgs b = own ? a : beam_args(p, words, nwords, nout, out, kDefaultTile);
        const FewShape few = b.offs ? few_shape(b, !own, p->device) : FewShape{0, 0};
        if (few.waves) {
            e = nl == 12 ? (out_u16 ? launch_few_shape<12, true>(b, few, s) : launch_few_shape<12, false>(b, few, s))
                         : (out_u16 ? launch_few_shape<16, true>(b, few, s) : launch_few_shape<16, false>(b, few, s));
            if (e != hipSuccess)
                return fail(DEDISP_ERR_HIP, "dedispersion launch failed: %s", hipGetErrorString(e));
            return DEDISP_OK;
        }
    }
#define DD_DISPATCH(NL_, NDW_, G_)                                                    \
    if (nl == NL_ && cfg.dms_per_block == NDW_ * kWaves && cfg.groups == G_)          \
        e = out_u16 ? launch_cfg<NL_, NDW_, G_, true>(a, cfg.stage_chans, lds, s)     \
                    : launch_cfg<NL_, NDW_, G_, false>(a, cfg.stage_chans, lds, s);
    DD_SHAPES(DD_DISPATCH)
#undef DD_DISPATCH
    if (e != hipSuccess)
        return fail(e == hipErrorInvalidValue ? DEDISP_ERR_UNSUPPORTED : DEDISP_ERR_HIP,
                    "dedispersion launch failed: %s", hipGetErrorString(e));
    return DEDISP_OK;
}

dedisp_status launch_dedisperse_many(const ManyItem* items, int n, const TileConfig& cfg, hipStream_t s) {
    const int k = dm_block_index(cfg.dms_per_block);
    ManyArgs m{};
    int64_t total = 0;
    size_t lds = 0;
    bool one_by_one = n == 1 || n > kMaxMany || k < 0 || cfg.stage_chans < 4 || cfg.stage_chans % 4 ||
                      cfg.groups < 1 || cfg.groups > 2;
    for (int i = 0; i < n && !one_by_one; ++i) {
        const ManyItem& it = items[i];
        dedisp_status st = DEDISP_OK;
        if (tile_lds_bytes(it.plan, cfg) > 160 * 1024) {
            one_by_one = true;
            break;
        }
        if (!offset_table(it.plan, cfg, true, &st)) return st;
        m.b[i] = beam_args(it.plan, it.words, it.nwords, it.nout, it.out, cfg);
        m.b[i].item_begin = total;
        total += m.b[i].n_items;
        lds = std::max(lds, tile_lds_bytes(it.plan, cfg));
    }
    // One launch each reports what cannot be launched.
    if (one_by_one || total > (int64_t(1) << 30)) {
        for (int i = 0; i < n; ++i) {
            const ManyItem& it = items[i];
            const dedisp_status st = launch_dedisperse(it.plan, it.words, it.nwords, it.nout, it.out, 1, cfg, Form::kPlan, s);
            if (st != DEDISP_OK) return st;
        }
        return DEDISP_OK;
    }
    const int nl = levels_for(items[0].plan->nchans);
    hipError_t e = hipErrorInvalidValue;
#define DD_DISPATCH(NL_, NDW_, G_)                                                    \
    if (nl == NL_ && cfg.dms_per_block == NDW_ * kWaves && cfg.groups == G_)          \
        e = launch_many_cfg<NL_, NDW_, G_>(m, n, total, cfg.stage_chans, lds, s);
    DD_SHAPES(DD_DISPATCH)
#undef DD_DISPATCH
    if (e != hipSuccess)
        return fail(e == hipErrorInvalidValue ? DEDISP_ERR_UNSUPPORTED : DEDISP_ERR_HIP,
                    "dedispersion launch failed: %s", hipGetErrorString(e));
    return DEDISP_OK;
}

hipError_t launch_dedisperse_persistent(const BeamArgs* d_beams, int nbeams, int64_t total,
                                        int nl, int out_u16, const TileConfig& cfg, size_t lds,
                                        unsigned long long* d_counters, int nq, int grid,
                                        hipStream_t s) {
    hipError_t e = hipErrorInvalidValue;
#define DD_DISPATCH(NL_, NDW_, G_)                                                              \
    if (nl == NL_ && cfg.dms_per_block == NDW_ * kWaves && cfg.groups == G_)                    \
        e = out_u16 ? launch_persistent_cfg<NL_, NDW_, G_, true>(d_beams, nbeams, total,        \
                          cfg.stage_chans, lds, d_counters, nq, grid, s)                        \
                    : launch_persistent_cfg<NL_, NDW_, G_, false>(d_beams, nbeams, total,       \
                          cfg.stage_chans, lds, d_counters, nq, grid, s);
    DD_SHAPES(DD_DISPATCH)
#undef DD_DISPATCH
    return e;
}

int persistent_blocks_per_cu(int nl, int out_u16, const TileConfig& cfg, size_t lds) {
    int n = 0;
#define DD_DISPATCH(NL_, NDW_, G_)                                                   \
    if (nl == NL_ && cfg.dms_per_block == NDW_ * kWaves && cfg.groups == G_)         \
        n = out_u16 ? occupancy_cfg<NL_, NDW_, G_, true>(lds) : occupancy_cfg<NL_, NDW_, G_, false>(lds);
    DD_SHAPES(DD_DISPATCH)
#undef DD_DISPATCH
    return n;
}

}  // namespace dd
