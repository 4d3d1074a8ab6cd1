// Kernels for what the tiled kernels do not take: reductions of regular segments whose length is no power
// of two (long ones; short ones run on the fixed tiles of tcr_irregular.hpp), the shortest segments and the
// moments.  The paper handles such sizes by zero padding
// or by masking (Section 4, "Support for arbitrary segment sizes ...").  Padding in place is not possible
// behind this interface, so:
//   masked_*        one to 16 wavefronts per segment (or per piece of a long one) walk the 512-element
//                   tiles of the ARRAY (aligned to the array, not to the segment) that the segment
//                   touches; elements of a tile outside the segment count as zero -- the paper's
//                   zero padding, applied to the operand registers -- and the matrix-core products,
//                   the running sums through the accumulator and the 128-bit loads of the tuned
//                   kernels apply unchanged.
//   generic_*       one thread per segment: 16-bit loads, binary32 adds.
// They are correct for every seg_len >= 1; none of them is tuned.
#pragma once
#include "tcr_device.hpp"
#include "tcr_scan.hpp"
#include "tcr_irregular.hpp"
#include "tcr_reduce.hpp"

namespace tcr {

constexpr int kGenericThreads = 256;

// One thread per segment (short segments).
__device__ __forceinline__ void put(void* out, uint64_t i, float v, bool f16) {
    if (f16) static_cast<_Float16*>(out)[i] = (_Float16)v;
    else static_cast<float*>(out)[i] = v;
}

// exclusive: each output leaves out its own element; f16: outputs rounded to binary16.
template <bool SCAN>
__global__ __launch_bounds__(kGenericThreads) void generic_thread_kernel(const _Float16* __restrict__ in,
                                                                         void* __restrict__ out, uint64_t nseg,
                                                                         uint64_t seg_len, bool exclusive, bool f16) {
    const uint64_t s = (uint64_t)blockIdx.x * kGenericThreads + threadIdx.x;
    if (s >= nseg) return;
    const _Float16* p = in + s * seg_len;
    float acc = 0.0f;
    for (uint64_t k = 0; k < seg_len; ++k) {
        const float v = (float)p[k];
        if (SCAN) put(out, s * seg_len + k, exclusive ? acc : acc + v, f16);
        acc += v;
    }
    if (!SCAN) put(out, s, acc, f16);
}

// Segments of 1, 2, 4 or 8 elements: a lane adds up the whole segments inside its 8 consecutive elements and
// stores the 8 >> LOG2L results side by side (seg_len 1 is the conversion to binary32, also the inclusive scan).
template <int LOG2L>
__global__ __launch_bounds__(kGenericThreads) void tiny_reduce_kernel(const _Float16* __restrict__ in,
                                                                      float* __restrict__ out, uint64_t n) {
    static_assert(LOG2L >= 0 && LOG2L <= 3, "");
    constexpr int kResults = 8 >> LOG2L;
    const uint64_t g = ((uint64_t)blockIdx.x * kGenericThreads + threadIdx.x) * 8;
    if (g >= n) return;
    const half8 x = load8_guarded<true>(in, g, n);
    float r[kResults];
#pragma unroll
    for (int i = 0; i < kResults; ++i) {
        float acc = 0.0f;
#pragma unroll
        for (int e = 0; e < (1 << LOG2L); ++e) acc += (float)x[(i << LOG2L) + e];
        r[i] = acc;
    }
    float* dst = out + (g >> LOG2L);
    if (g + 8 <= n) {
        if constexpr (kResults == 8) {
            store4(dst, 0, (float4v){r[0], r[1], r[2], r[3]});
            store4(dst, 4, (float4v){r[4], r[5], r[6], r[7]});
        } else if constexpr (kResults == 4) {
            store4(dst, 0, (float4v){r[0], r[1], r[2], r[3]});
        } else {
#pragma unroll
            for (int i = 0; i < kResults; ++i) dst[i] = r[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kResults; ++i)
            if (g + (uint64_t)((i + 1) << LOG2L) <= n) dst[i] = r[i];
    }
}

// Both moments of segments of 4 or 8 elements, whole inside a lane's 8, U groups of 8 per lane.  Added in binary64, which is free here and
// rounds once (in binary32, two elements per v_dot2_f32_f16: squares of 8 elements 3.4e-8 off, one rounding 2.5e-8, the packed rows 2.6e-8).
// Bound: memory (64 * 2^20 elements in segments of 4, 268 MB, 43 us).
template <int LOG2L, int U>
__global__ __launch_bounds__(kGenericThreads) void tiny_moments_kernel(const _Float16* __restrict__ in, float* __restrict__ sum,
                                                                       float* __restrict__ sumsq, uint64_t n) {
    static_assert(LOG2L == 2 || LOG2L == 3, "");
    constexpr int kResults = 8 >> LOG2L;
    const uint64_t first = ((uint64_t)blockIdx.x * U * kGenericThreads + threadIdx.x) * 8;
    half8 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = load8_guarded<true>(in, first + (uint64_t)(u * 8 * kGenericThreads), n);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t g = first + (uint64_t)(u * 8 * kGenericThreads);
        float a[kResults], q[kResults];
#pragma unroll
        for (int i = 0; i < kResults; ++i) {
            double sum64 = 0.0, squares64 = 0.0;
#pragma unroll
            for (int e = 0; e < (1 << LOG2L); ++e) {
                const double v = (double)(float)x[u][(i << LOG2L) + e];
                sum64 += v;
                squares64 = __builtin_fma(v, v, squares64);
            }
            a[i] = (float)sum64;
            q[i] = (float)squares64;
        }
        if (g + 8 <= n) {
            if constexpr (kResults == 2) {
                typedef float pair __attribute__((ext_vector_type(2), aligned(4)));       // (results are aligned to their size only)
                *reinterpret_cast<pair*>(sum + (g >> LOG2L)) = (pair){a[0], a[1]};
                *reinterpret_cast<pair*>(sumsq + (g >> LOG2L)) = (pair){q[0], q[1]};
            } else {
                sum[g >> LOG2L] = a[0];
                sumsq[g >> LOG2L] = q[0];
            }
        } else if (kResults == 2 && g + 4 <= n) {
            sum[g >> LOG2L] = a[0];
            sumsq[g >> LOG2L] = q[0];
        }
    }
}

// The inclusive scan of segments of 1, 2, 4 or 8 elements: running sums inside a lane's 8 elements, restarted
// every 1 << LOG2L of them (seg_len 1: the conversion again).
template <int LOG2L>
__global__ __launch_bounds__(kGenericThreads) void tiny_scan_kernel(const _Float16* __restrict__ in,
                                                                    float* __restrict__ out, uint64_t n) {
    static_assert(LOG2L >= 0 && LOG2L <= 3, "");
    const uint64_t g = ((uint64_t)blockIdx.x * kGenericThreads + threadIdx.x) * 8;
    if (g >= n) return;
    const half8 x = load8_guarded(in, g, n);
    float r[8];
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if ((e & ((1 << LOG2L) - 1)) == 0) acc = 0.0f;
        acc += (float)x[e];
        r[e] = acc;
    }
    store4_guarded(out, g, n, (float4v){r[0], r[1], r[2], r[3]});
    store4_guarded(out, g + 4, n, (float4v){r[4], r[5], r[6], r[7]});
}

// ---------------------------------------------------------------------------------------- masked tiles
// What one wavefront -- number `part` of the W that share the work -- adds up of the elements [begin, end): the sum,
// and for kBoth the sum of squares (uniform).  `in` is 16-byte aligned, end <= n, end - begin < 2^30.
// The sum is Reduction_256N (V <- ones . X^T + V).  The sum of squares takes the data as BOTH operands: entry (i, j) of
// X . X^T is the inner product of data rows i and j, so the DIAGONAL of W <- X . X^T + W accumulates the sums of
// squares of the 16 rows (the other entries are not used); a product of two binary16 values is exact in the binary32
// accumulator.
// The tiles of the ARRAY from the one that holds `begin` on, U of them per step and wavefront, all U loads on their way
// at once: a buffer resource that ends with the group of 8 that holds the last element keeps them free of branches (a
// branch around a load makes the compiler wait where the paths rejoin: 10 % at segments of 4096 elements), and what the
// first and the last tile hold of neighbours is masked in the registers afterwards.
template <int KIND, int U, int W>
__device__ __forceinline__ void masked_part_sums(const _Float16* __restrict__ in, uint64_t n, uint64_t begin, uint64_t end,
                                                 int part, const LaneId& id, float& sum, float& sumsq) {
    const uint64_t first = begin & ~(uint64_t)(kTile - 1);
    const uint32_t lead = (uint32_t)(begin - first), len = (uint32_t)(end - first);      // the range, counted from `first`
    // whole groups of 8 inside the array; the one that the end of the array cuts is read element by element
    const bool cut = ((end + 7) & ~7ull) > n;
    const __amdgpu_buffer_rsrc_t src = make_rsrc(in + first, (cut ? len & ~7u : (len + 7u) & ~7u) * 2u);
    const uint32_t lane_off = (uint32_t)(kRow * id.j + 8 * id.g);
    float4v acc = splat(0.0f), sq = splat(0.0f);
    for (uint32_t t = (uint32_t)part * (uint32_t)(kTile * U); t < len; t += (uint32_t)(kTile * U * W)) {
        half8 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = buffer_load8<true>(src, (t + (uint32_t)(kTile * u) + lane_off) * 2u);
        if (t < lead) x[0] = drop_leading(x[0], (int)lead - (int)lane_off);              // (t == 0: the first tile)
        if ((len & 7u) != 0u && len - t <= (uint32_t)(kTile * U)) {                      // the step that holds the last tile
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t at = t + (uint32_t)(kTile * u) + lane_off;
                if (cut && at < len && at + 8u > len) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[u][e] = at + (uint32_t)e >= lead && at + (uint32_t)e < len ? in[first + at + (uint32_t)e] : (_Float16)0.0f;
                }
                x[u] = keep_leading(x[u], (int)len - (int)at);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = mfma(const_ones(), x[u], acc);
            if constexpr (KIND == kBoth) sq = mfma(x[u], x[u], sq);
        }
    }
    sum = read_lane(row_sum_to_last<16>(acc[0]), 15);
    if constexpr (KIND == kBoth) {
        // lane (j, g) holds rows 4g .. 4g+3 of column j: the diagonal entry of column j sits in lane (j, j / 4), register j % 4
        const int r = id.j & 3;
        const float d = r == 0 ? sq[0] : (r == 1 ? sq[1] : (r == 2 ? sq[2] : sq[3]));
        sumsq = wave_sum(id.g == (id.j >> 2) ? d : 0.0f);
    }
}

// Piece w % per of segment w / per (pieces of `span` elements counted from the segment's start, the last one shorter;
// per == 1: whole segments) -> dst[w], dst2[w].  W == 1: a wavefront per piece, kMaskedWaves of them in a workgroup.
// W > 1: a workgroup of W wavefronts per piece, their sums added through LDS in wavefront order; with fin.counter the
// workgroup that finishes last adds up the pieces too (dst2 follows dst's nseg * per).
// Bound by memory.  One wavefront per segment leaves the chip idle when there are few segments (16 KiB in flight per
// wavefront, and 256 compute units): the launch picks W and the span so that about 4096 wavefronts share the array.
constexpr int kMaskedWaves = 4;
template <int W>
constexpr int masked_group_waves() { return W == 1 ? kMaskedWaves : W; }
template <int KIND, int U, int W, bool PIECES>
__device__ __forceinline__ void masked_piece(const _Float16* __restrict__ in, float* __restrict__ dst, float* __restrict__ dst2,
                                             uint64_t nseg, uint64_t seg_len, uint64_t span, uint64_t per, const ReduceFinish& fin) {
    const LaneId id;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t w = W == 1 ? (uint64_t)blockIdx.x * kMaskedWaves + (uint64_t)wave : (uint64_t)blockIdx.x;
    if (w >= (PIECES ? nseg * per : nseg)) return;       // (W > 1: the whole workgroup alike)
    const uint64_t s = PIECES ? w / per : w;
    const uint64_t seg_end = (s + 1) * seg_len;
    uint64_t begin = s * seg_len, end = seg_end;
    if constexpr (PIECES) {
        begin += (w - s * per) * span;
        if (begin + span < seg_end) end = begin + span;
    }
    float a = 0.0f, q = 0.0f;
    masked_part_sums<KIND, U, W>(in, nseg * seg_len, begin, end, W == 1 ? 0 : wave, id, a, q);
    if constexpr (W > 1) {
        __shared__ float s_part[2][W];
        if (id.lane == 0) {
            s_part[0][wave] = a;
            s_part[1][wave] = q;
        }
        __syncthreads();
        const bool finish = PIECES && fin.counter != nullptr;
        if (threadIdx.x != 0 && !finish) return;
        a = pairwise_sum(s_part[0]);
        q = pairwise_sum(s_part[1]);
        if constexpr (PIECES) {
            if (finish) {
                if (threadIdx.x == 0) {
                    __hip_atomic_store(&dst[w], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if constexpr (KIND == kBoth) __hip_atomic_store(&dst2[w], q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                finish_partials<W>(dst, fin, wave, id.lane);
                return;
            }
        }
    }
    if (id.lane == 0) {
        dst[w] = a;
        if constexpr (KIND == kBoth) dst2[w] = q;
    }
}

// Whole segments; pieces of long ones (reduce_final_kernel adds them); both moments of either -- the statistics of a
// normalisation layer, which the paper's conclusion names as the next use of reductions on matrix cores.
template <int U, int W>
__global__ __launch_bounds__(masked_group_waves<W>() * kWave) void masked_wave_reduce_kernel(const _Float16* __restrict__ in,
                                                                                             float* __restrict__ out,
                                                                                             uint64_t nseg, uint64_t seg_len) {
    masked_piece<kSum, U, W, false>(in, out, nullptr, nseg, seg_len, seg_len, 1, ReduceFinish{});
}
template <int W>
__global__ __launch_bounds__(masked_group_waves<W>() * kWave) void masked_span_reduce_kernel(const _Float16* __restrict__ in,
                                                                                             float* __restrict__ dst, uint64_t nseg,
                                                                                             uint64_t seg_len, uint64_t span,
                                                                                             uint64_t per, ReduceFinish fin) {
    masked_piece<kSum, 8, W, true>(in, dst, nullptr, nseg, seg_len, span, per, fin);
}
template <int U, int W, bool PIECES>
__global__ __launch_bounds__(masked_group_waves<W>() * kWave) void masked_moments_kernel(const _Float16* __restrict__ in,
                                                                                         float* __restrict__ sum,
                                                                                         float* __restrict__ sumsq, uint64_t nseg,
                                                                                         uint64_t seg_len, uint64_t span, uint64_t per,
                                                                                         ReduceFinish fin) {
    masked_piece<kBoth, U, W, PIECES>(in, sum, sumsq, nseg, seg_len, span, per, fin);
}

// Short segments: one thread per segment, binary32 adds and fused multiply-adds.
__global__ __launch_bounds__(kGenericThreads) void generic_moments_kernel(const _Float16* __restrict__ in,
                                                                          float* __restrict__ sum,
                                                                          float* __restrict__ sumsq, uint64_t nseg,
                                                                          uint64_t seg_len) {
    const uint64_t s = (uint64_t)blockIdx.x * kGenericThreads + threadIdx.x;
    if (s >= nseg) return;
    const _Float16* p = in + s * seg_len;
    float a = 0.0f, q = 0.0f;
    for (uint64_t k = 0; k < seg_len; ++k) {
        const float v = (float)p[k];
        a += v;
        q = __builtin_fmaf(v, v, q);
    }
    sum[s] = a;
    sumsq[s] = q;
}

}  // namespace tcr
