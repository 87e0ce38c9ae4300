// Multibeam coincidence RFI mask (paper section 2.1).
//
// Interference is not localised on the sky: the 13 beams of the multibeam
// receiver serve as reference antennas for one another.  The paper's method is
// a transform of the multibeam time series: for each sample the beams are
// tested against a signal-to-noise threshold and the sample is flagged as
// interference when enough of them exceed it (its example: 3 sigma in 4 or
// more of the 13 beams), giving a boolean mask.
//
// Readings taken here: the per-beam series is the zero-DM series z_b[t] =
// sum_c x_b[c][t] of the beam's 2-bit samples over the common sample range;
// mean and sigma are the population statistics of z_b over that range, from
// exact integer sums; exceeding k sigma means the strict S/N > k, decided exactly
// as in the sigma-cut (z >= ceil((S1 + isqrt(floor(k^2 D)) + 1) / n)).
//
// Kernels: zero-DM sums of all beams straight from the packed bytes (popcounts
// of the two bit-planes of each 32-bit word) with their partial sums, one wave
// per beam for the exact cut level, and four samples per thread for the vote.
// All of it is bound by the one read of the packed input.
#include <algorithm>
#include <type_traits>

#include "dedisp_internal.hpp"
#include "intmath.hpp"
#include "search_internal.hpp"

namespace {

constexpr int kCThreads = 256;
constexpr int kStatBlock = 8192;   // samples per partial-sum block

// Level sum of the sixteen 2-bit fields of a word: bit 0s count once, bit 1s twice.
__device__ __forceinline__ uint32_t level_sum(uint32_t w) {
    return static_cast<uint32_t>(__builtin_popcount(w & 0x55555555u)) +
           2u * static_cast<uint32_t>(__builtin_popcount(w & 0xAAAAAAAAu));
}

struct BeamsIn {
    const uint8_t* p[64];
};

// Sixteen bytes of a sample at any address, one load.
struct __attribute__((packed, aligned(1))) Piece {
    uint32_t w[4];
};

__global__ __launch_bounds__(kCThreads) void zero_dm_clear_kernel(int n, uint64_t* __restrict__ p1,
                                                                  uint64_t* __restrict__ p2) {
    const int i = blockIdx.x * kCThreads + threadIdx.x;
    if (i < n) p1[i] = p2[i] = 0ull;
}

// Adds a block's partial sums into those of its kStatBlock samples.  The sums
// are integers: the order in which blocks add them does not matter.
// z <= 3*nchans < 2^16, so S2 of up to 2^31 samples fits 64 bits.
__device__ __forceinline__ void add_stats(uint64_t a1, uint64_t a2, uint64_t* p1, uint64_t* p2) {
    __shared__ uint64_t r1[kCThreads / 64], r2[kCThreads / 64];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        a1 += __shfl_xor(a1, o, 64);
        a2 += __shfl_xor(a2, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        r1[threadIdx.x >> 6] = a1;
        r2[threadIdx.x >> 6] = a2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s1 = 0, s2 = 0;
        for (int w = 0; w < kCThreads / 64; ++w) {
            s1 += r1[w];
            s2 += r2[w];
        }
        atomicAdd(reinterpret_cast<unsigned long long*>(p1), static_cast<unsigned long long>(s1));
        atomicAdd(reinterpret_cast<unsigned long long*>(p2), static_cast<unsigned long long>(s2));
    }
}

// Sum over groups of G lanes, left in all of them.
template <int G>
__device__ __forceinline__ uint32_t group_sum(uint32_t s) {
    auto dpp = [&](auto ctrl) {
        s += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(s), decltype(ctrl)::value,
                                                               0xF, 0xF, true));
    };
    if constexpr (G >= 2) dpp(std::integral_constant<int, 0xB1>{});     // lane ^ 1
    if constexpr (G >= 4) dpp(std::integral_constant<int, 0x4E>{});     // lane ^ 2
    if constexpr (G >= 8) dpp(std::integral_constant<int, 0x141>{});    // mirror of 8 lanes
    if constexpr (G >= 16) dpp(std::integral_constant<int, 0x140>{});   // mirror of 16 lanes
    if constexpr (G >= 32) s += __shfl_xor(s, 16, 64);
    if constexpr (G >= 64) s += __shfl_xor(s, 32, 64);
    return s;
}

// Samples of 16 bytes or more: G lanes per sample, a 16-byte piece each (the
// last piece is read so that it ends with the sample, and the bytes that it
// shares with the one before are masked out), kZUnroll loads in flight per lane.
// Grid: (blocks of `iters` * 4 waves * kZUnroll * 64 / G samples, beams); a
// block lies inside one block of partial sums.  Bound by the read.  The whole mask
// of 13 beams, us, with one launch per beam and separate partial sums (and, but
// for 1024 channels, one thread per sample), and now: 1024 channels x 2^19
// samples 398 -> 358 (the read alone 356 at a copy's rate), x 2^17 173 -> 122;
// 256 x 2^18 210 -> 75; 1000 x 2^18 2740 -> 210; 2048 x 2^17 919 -> 199.
constexpr int kZUnroll = 8;

template <int G>
__global__ __launch_bounds__(kCThreads) void zero_dm_kernel(BeamsIn in, int64_t nsamps, int bps,
                                                            int iters, int nblk,
                                                            int32_t* __restrict__ z,
                                                            uint64_t* __restrict__ p1,
                                                            uint64_t* __restrict__ p2) {
    constexpr int kPer = 64 / G;                 // samples per load of a wave
    constexpr int kStep = kPer * kZUnroll;       // and per step
    constexpr int kPick = G < kZUnroll ? G : kZUnroll;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int sub = lane / G, part = lane % G;
    const uint8_t* beam = in.p[blockIdx.y];
    int32_t* zb = z + static_cast<int64_t>(blockIdx.y) * nsamps;
    const int pieces = (bps + 15) / 16;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * (kCThreads / 64) * kStep * iters;
    uint64_t a1 = 0, a2 = 0;
    for (int it = 0; it < iters; ++it) {
        const int64_t tb = first + (static_cast<int64_t>(it) * (kCThreads / 64) + wave) * kStep;
        if (tb >= nsamps) break;                 // whole waves
        uint32_t s[kZUnroll] = {};
        for (int c0 = 0; c0 < pieces; c0 += G) {
            const int c = min(c0 + part, pieces - 1);
            const int off = min(16 * c, bps - 16);
            // bytes of this piece that the one before has, or all of them
            const int skip = c0 + part < pieces ? 16 * c - off : 16;
            uint32_t keep[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int n = min(max(skip - 4 * k, 0), 4);
                keep[k] = n == 4 ? 0u : 0xFFFFFFFFu << (8 * n);
            }
            Piece v[kZUnroll];
#pragma unroll
            for (int u = 0; u < kZUnroll; ++u) {
                const int64_t t = min<int64_t>(tb + u * kPer + sub, nsamps - 1);
                v[u] = *reinterpret_cast<const Piece*>(beam + t * bps + off);
            }
#pragma unroll
            for (int u = 0; u < kZUnroll; ++u)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[u] += level_sum(v[u].w[k] & keep[k]);
        }
#pragma unroll
        for (int u = 0; u < kZUnroll; ++u) s[u] = group_sum<G>(s[u]);
        // lane `part` of a group writes the group's sample of load u0 + part
#pragma unroll
        for (int u0 = 0; u0 < kZUnroll; u0 += kPick) {
            uint32_t x = s[u0];
#pragma unroll
            for (int j = 1; j < kPick; ++j) x = part == j ? s[u0 + j] : x;
            const int64_t t = tb + (u0 + part) * kPer + sub;
            if (part < kPick && t < nsamps) {
                zb[t] = static_cast<int32_t>(x);
                a1 += x;
                a2 += static_cast<uint64_t>(x) * x;
            }
        }
    }
    const int64_t g = static_cast<int64_t>(blockIdx.y) * nblk + first / kStatBlock;
    add_stats(a1, a2, p1 + g, p2 + g);
}

// Samples of fewer than 16 bytes: one thread per sample, whole words then the
// remaining bytes.
__global__ __launch_bounds__(kCThreads) void zero_dm_narrow_kernel(BeamsIn in, int64_t nsamps, int bps,
                                                                   int nblk, int32_t* __restrict__ z,
                                                                   uint64_t* __restrict__ p1,
                                                                   uint64_t* __restrict__ p2) {
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kCThreads;
    const int64_t t = first + threadIdx.x;
    uint32_t s = 0;
    if (t < nsamps) {
        const uint8_t* p = in.p[blockIdx.y] + t * bps;
        int i = 0;
        if ((reinterpret_cast<uintptr_t>(p) & 3) == 0)
            for (; i + 4 <= bps; i += 4) s += level_sum(*reinterpret_cast<const uint32_t*>(p + i));
        for (; i < bps; ++i) s += level_sum(p[i]);
        z[static_cast<int64_t>(blockIdx.y) * nsamps + t] = static_cast<int32_t>(s);
    }
    const int64_t g = static_cast<int64_t>(blockIdx.y) * nblk + first / kStatBlock;
    add_stats(s, static_cast<uint64_t>(s) * s, p1 + g, p2 + g);
}

// One wave per beam: exact sums and the cut level (thr[b] = -1: D == 0,
// the beam never votes).  The first also clears the masked-sample counter.
__global__ __launch_bounds__(64) void zero_dm_threshold_kernel(
    int nblk, int64_t nsamps, uint32_t kmant, int kexp2, const uint64_t* __restrict__ p1,
    const uint64_t* __restrict__ p2, int64_t* __restrict__ thr,
    unsigned long long* __restrict__ count) {
    const int64_t b = blockIdx.x;
    uint64_t s1 = 0, s2 = 0;
    for (int g = threadIdx.x; g < nblk; g += 64) {
        s1 += p1[b * nblk + g];
        s2 += p2[b * nblk + g];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        s1 += __shfl_xor(s1, o, 64);
        s2 += __shfl_xor(s2, o, 64);
    }
    if (threadIdx.x != 0) return;
    if (b == 0) *count = 0ull;
    thr[b] = cut_level(static_cast<uint64_t>(nsamps), s1, s2, kmant, kexp2, nullptr);
}

// Four samples per thread: votes of the beams and the mask bytes.
constexpr int kVote = 4;

__global__ __launch_bounds__(kCThreads) void coincidence_vote_kernel(
    const int32_t* __restrict__ z, int64_t nsamps, int nbeams, int min_beams,
    const int64_t* __restrict__ thr, uint8_t* __restrict__ mask,
    unsigned long long* __restrict__ count) {
    struct __attribute__((packed, aligned(4))) Levels {
        int32_t v[kVote];
    };
    struct __attribute__((packed, aligned(1))) Flags {
        uint8_t m[kVote];
    };
    __shared__ unsigned int bc;
    if (threadIdx.x == 0) bc = 0u;
    __syncthreads();
    const int64_t t = (static_cast<int64_t>(blockIdx.x) * kCThreads + threadIdx.x) * kVote;
    unsigned int n = 0;
    if (t < nsamps) {
        const int64_t t4 = min<int64_t>(t, nsamps - kVote);   // the last four of the row
        int votes[kVote] = {};
        auto add = [&](int j, int64_t th, int32_t level) {
            votes[j] += th >= 0 && static_cast<int64_t>(level) >= th ? 1 : 0;
        };
        if (t4 >= 0) {
            for (int b = 0; b < nbeams; ++b) {
                const Levels q = *reinterpret_cast<const Levels*>(z + static_cast<int64_t>(b) * nsamps + t4);
                const int64_t th = thr[b];
#pragma unroll
                for (int j = 0; j < kVote; ++j) add(j, th, q.v[j]);
            }
            Flags f;
#pragma unroll
            for (int j = 0; j < kVote; ++j) {
                f.m[j] = votes[j] >= min_beams ? 1 : 0;
                n += t4 + j >= t ? f.m[j] : 0u;
            }
            *reinterpret_cast<Flags*>(mask + t4) = f;
        } else {   // fewer than four samples
            for (int64_t i = t; i < nsamps; ++i) {
                votes[0] = 0;
                for (int b = 0; b < nbeams; ++b) add(0, thr[b], z[static_cast<int64_t>(b) * nsamps + i]);
                const bool m = votes[0] >= min_beams;
                mask[i] = m ? 1 : 0;
                n += m ? 1u : 0u;
            }
        }
    }
    if (n) atomicAdd(&bc, n);
    __syncthreads();
    if (threadIdx.x == 0 && bc) atomicAdd(count, static_cast<unsigned long long>(bc));
}

struct CoincLayout {
    size_t o_z, o_p1, o_p2, o_thr, o_count, bytes;
    int nblk;
};

CoincLayout coinc_layout(int nbeams, int64_t nsamps) {
    CoincLayout l{};
    l.nblk = static_cast<int>((nsamps + kStatBlock - 1) / kStatBlock);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~size_t(255);
        return o;
    };
    l.o_z = take(static_cast<size_t>(nbeams) * nsamps * 4);
    l.o_p1 = take(static_cast<size_t>(nbeams) * l.nblk * 8);
    l.o_p2 = take(static_cast<size_t>(nbeams) * l.nblk * 8);
    l.o_thr = take(static_cast<size_t>(nbeams) * 8);
    l.o_count = take(8);
    l.bytes = off;
    return l;
}

bool coinc_args_ok(int32_t nbeams, int32_t nchans, int64_t nsamps) {
    return nbeams >= 1 && nbeams <= 64 && nchans >= 4 && nchans % 4 == 0 && nchans <= 21844 &&
           nsamps >= 1 && nsamps < (int64_t(1) << 31);
}

}  // namespace

namespace {

// Masked samples take the mean level 1.5 in every channel: levels 1 and 2 in
// alternate channels (byte 0x99: channels 4k and 4k + 2 at level 1, 4k + 1
// and 4k + 3 at level 2).  One thread per (beam, sample); flagged samples are
// rare, so the write is a short loop over the sample's bytes.
struct BeamPtrs {
    uint8_t* p[64];
};

__global__ __launch_bounds__(kCThreads) void rfi_apply_kernel(BeamPtrs beams, int nbeams,
                                                              int64_t nsamps, int bytes_per_sample,
                                                              const uint8_t* __restrict__ mask) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kCThreads + threadIdx.x;
    if (i >= nsamps * nbeams) return;
    const int b = static_cast<int>(i / nsamps);
    const int64_t t = i - static_cast<int64_t>(b) * nsamps;
    if (!mask[t]) return;
    uint8_t* row = beams.p[b] + t * bytes_per_sample;
    if ((bytes_per_sample & 15) == 0 && (reinterpret_cast<uintptr_t>(row) & 15) == 0) {
        const uint4 v = make_uint4(0x99999999u, 0x99999999u, 0x99999999u, 0x99999999u);
        for (int k = 0; k < bytes_per_sample / 16; ++k) reinterpret_cast<uint4*>(row)[k] = v;
    } else {
        for (int k = 0; k < bytes_per_sample; ++k) row[k] = 0x99;
    }
}

}  // namespace

namespace dd {

size_t rfi_mask_ws_bytes(int nbeams, int64_t nsamps) { return coinc_layout(nbeams, nsamps).bytes; }

hipError_t launch_rfi_mask(const uint8_t* const* ins, int nbeams, int nchans, int64_t nsamps,
                           uint32_t kmant, int kexp2, int min_beams, uint8_t* mask, void* workspace,
                           hipStream_t stream) {
    const CoincLayout l = coinc_layout(nbeams, nsamps);
    char* w = static_cast<char*>(workspace);
    int32_t* z = reinterpret_cast<int32_t*>(w + l.o_z);
    uint64_t* p1 = reinterpret_cast<uint64_t*>(w + l.o_p1);
    uint64_t* p2 = reinterpret_cast<uint64_t*>(w + l.o_p2);
    int64_t* thr = reinterpret_cast<int64_t*>(w + l.o_thr);
    unsigned long long* count = reinterpret_cast<unsigned long long*>(w + l.o_count);
    const int bps = nchans / 4;
    BeamsIn beams{};
    for (int b = 0; b < nbeams; ++b) beams.p[b] = ins[b];
    const int parts = nbeams * l.nblk;
    hipLaunchKernelGGL(zero_dm_clear_kernel, dim3((parts + kCThreads - 1) / kCThreads), dim3(kCThreads), 0,
                       stream, parts, p1, p2);
    if (bps < 16) {
        hipLaunchKernelGGL(zero_dm_narrow_kernel,
                           dim3(static_cast<unsigned>((nsamps + kCThreads - 1) / kCThreads), nbeams),
                           dim3(kCThreads), 0, stream, beams, nsamps, bps, l.nblk, z, p1, p2);
    } else {
        auto launch = [&](auto g) {
            constexpr int G = decltype(g)::value;
            // four steps per block, one where that leaves CUs without a block
            constexpr int64_t step = int64_t(kCThreads / 64) * kZUnroll * (64 / G);
            const int iters = (nsamps + 4 * step - 1) / (4 * step) * nbeams >= 1024 ? 4 : 1;
            static_assert(kStatBlock % (4 * step) == 0, "a block lies inside one block of sums");
            hipLaunchKernelGGL((zero_dm_kernel<G>),
                               dim3(static_cast<unsigned>((nsamps + iters * step - 1) / (iters * step)), nbeams),
                               dim3(kCThreads), 0, stream, beams, nsamps, bps, iters, l.nblk, z, p1, p2);
        };
        const int pieces = (bps + 15) / 16;
        if (pieces <= 1) launch(std::integral_constant<int, 1>{});
        else if (pieces <= 2) launch(std::integral_constant<int, 2>{});
        else if (pieces <= 4) launch(std::integral_constant<int, 4>{});
        else if (pieces <= 8) launch(std::integral_constant<int, 8>{});
        else if (pieces <= 16) launch(std::integral_constant<int, 16>{});
        else if (pieces <= 32) launch(std::integral_constant<int, 32>{});
        else launch(std::integral_constant<int, 64>{});
    }
    hipLaunchKernelGGL(zero_dm_threshold_kernel, dim3(nbeams), dim3(64), 0, stream, l.nblk, nsamps, kmant,
                       kexp2, p1, p2, thr, count);
    hipLaunchKernelGGL(coincidence_vote_kernel,
                       dim3(static_cast<unsigned>((nsamps + kCThreads * kVote - 1) / (kCThreads * kVote))),
                       dim3(kCThreads), 0, stream, z, nsamps, nbeams, min_beams, thr, mask, count);
    return hipGetLastError();
}

const unsigned long long* rfi_mask_count(const void* workspace, int nbeams, int64_t nsamps) {
    return reinterpret_cast<const unsigned long long*>(static_cast<const char*>(workspace) +
                                                       coinc_layout(nbeams, nsamps).o_count);
}

hipError_t launch_rfi_apply(uint8_t* const* beams, int nbeams, int nchans, int64_t nsamps,
                            const uint8_t* mask, hipStream_t stream) {
    if (nbeams < 1 || nbeams > 64) return hipErrorInvalidValue;
    BeamPtrs ptrs{};
    for (int b = 0; b < nbeams; ++b) ptrs.p[b] = beams[b];
    const int64_t n = nsamps * nbeams;
    hipLaunchKernelGGL(rfi_apply_kernel, dim3(static_cast<unsigned>((n + kCThreads - 1) / kCThreads)),
                       dim3(kCThreads), 0, stream, ptrs, nbeams, nsamps, nchans / 4, mask);
    return hipGetLastError();
}

}  // namespace dd

extern "C" size_t dedisp_rfi_mask_workspace_bytes(int32_t nbeams, int64_t nsamps) {
    if (nbeams < 1 || nbeams > 64 || nsamps < 1 || nsamps >= (int64_t(1) << 31)) return 0;
    return coinc_layout(nbeams, nsamps).bytes;
}

extern "C" dedisp_status dedisp_rfi_mask(const uint8_t* const* in_2bit, int32_t nbeams,
                                         int32_t nchans, int64_t nsamps, float k_sigma,
                                         int32_t min_beams, uint8_t* mask, int64_t* n_masked,
                                         void* workspace, dedisp_stream stream) {
    using dd::fail;
    if (!in_2bit || !mask || !n_masked || !workspace)
        return fail(DEDISP_ERR_INVALID_ARG, "NULL argument");
    if (!coinc_args_ok(nbeams, nchans, nsamps))
        return fail(DEDISP_ERR_INVALID_ARG,
                    "need 1 <= nbeams <= 64, nchans a multiple of 4 in [4, 21844], 1 <= nsamps < 2^31");
    if (min_beams < 1) return fail(DEDISP_ERR_INVALID_ARG, "min_beams must be >= 1");
    if (reinterpret_cast<uintptr_t>(workspace) % 256)
        return fail(DEDISP_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    for (int b = 0; b < nbeams; ++b)
        if (!in_2bit[b]) return fail(DEDISP_ERR_INVALID_ARG, "beam %d input is NULL", b);
    uint32_t kmant = 0;
    int kexp2 = 0;
    dedisp_status st = dd::split_threshold_public(k_sigma, &kmant, &kexp2);
    if (st != DEDISP_OK) return st;
    DD_HIP(dd::launch_rfi_mask(in_2bit, nbeams, nchans, nsamps, kmant, kexp2, min_beams, mask,
                               workspace, stream));
    unsigned long long total = 0;
    DD_HIP(hipMemcpyAsync(&total, dd::rfi_mask_count(workspace, nbeams, nsamps), sizeof total,
                          hipMemcpyDeviceToHost, stream));
    DD_HIP(hipStreamSynchronize(stream));
    *n_masked = static_cast<int64_t>(total);
    dd::clear_error();
    return DEDISP_OK;
}

extern "C" dedisp_status dedisp_rfi_mask_read_stats(const void* workspace, int32_t nbeams,
                                                    int64_t nsamps, int32_t* zero_dm,
                                                    int64_t* thr, dedisp_stream stream) {
    using dd::fail;
    if (!workspace || nbeams < 1 || nbeams > 64 || nsamps < 1 || nsamps >= (int64_t(1) << 31))
        return fail(DEDISP_ERR_INVALID_ARG, "bad arguments");
    const CoincLayout l = coinc_layout(nbeams, nsamps);
    const char* w = static_cast<const char*>(workspace);
    if (zero_dm)
        DD_HIP(hipMemcpyAsync(zero_dm, w + l.o_z, static_cast<size_t>(nbeams) * nsamps * 4,
                              hipMemcpyDeviceToHost, stream));
    if (thr)
        DD_HIP(hipMemcpyAsync(thr, w + l.o_thr, static_cast<size_t>(nbeams) * 8,
                              hipMemcpyDeviceToHost, stream));
    DD_HIP(hipStreamSynchronize(stream));
    return DEDISP_OK;
}

extern "C" dedisp_status dedisp_rfi_apply(uint8_t* const* beams_2bit, int32_t nbeams,
                                          int32_t nchans, int64_t nsamps, const uint8_t* mask,
                                          dedisp_stream stream) {
    using dd::fail;
    if (!beams_2bit || !mask) return fail(DEDISP_ERR_INVALID_ARG, "NULL argument");
    if (!coinc_args_ok(nbeams, nchans, nsamps))
        return fail(DEDISP_ERR_INVALID_ARG,
                    "need 1 <= nbeams <= 64, nchans a multiple of 4 in [4, 21844], 1 <= nsamps < 2^31");
    for (int b = 0; b < nbeams; ++b)
        if (!beams_2bit[b]) return fail(DEDISP_ERR_INVALID_ARG, "beam %d is NULL", b);
    DD_HIP(dd::launch_rfi_apply(beams_2bit, nbeams, nchans, nsamps, mask, stream));
    dd::clear_error();
    return DEDISP_OK;
}
