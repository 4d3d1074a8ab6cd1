// Long sums in one launch.
//
// As reduce_span_kernel with a span per wavefront, and the wavefronts' sums added up by the last workgroup of each segment: they
// are published in a table of descriptors (tcr_scan.hpp), tagged with the launch, so nothing is counted and no workgroup but that
// one waits.  A sum that is not there after `patience` looks is added up again from the elements, to the same bits, and
// published by the one who waits; every wait therefore ends, whatever else the device runs.
// Bound: memory; at the end one write and one read on the far side of the caches.  Four wavefronts, each with 4
// descriptors per lane asked for at once: four rounds for 4096 partials (16 at once, or values held from one look to the next, cost
// the whole kernel its registers: 140 and three wavefronts per SIMD, 2^28 elements 98.9 us).
// Against reduce_span_kernel with reduce_final_kernel behind, us back to back, full reduction of 2^20 * 8.5 / 10 / 12 / 16 elements:
// 9.2 / 9.1 / 8.9 / 9.0 -> 5.9 / 6.1 / 6.5 / 8.1; segments of 2^18 / 2^20 / 2^22, 2^24 in all: 9.2 / 8.8 / 8.9 -> 8.1 / 7.9 / 7.5.
#pragma once

#include "tcr_scan.hpp"

namespace tcr {

constexpr int kGatherWaves = 4, kGatherLoads = 4, kGatherTiles = 8;
struct ReduceGather {
    const _Float16* in;
    float* out;
    uint64_t n, span;
    uint32_t per, nspans;        // wavefronts per segment (several segments: a multiple of kGatherWaves) and in all
    uint32_t patience;
};

// Elements [begin, end) (whole wavefront).  STEP: tiles asked for at once, U (a divisor of U that is even gives the same bits: the
// additions and their order do not depend on it).
template <int FORM, int U, int STEP>
__device__ __forceinline__ float gather_span_sum(const _Float16* __restrict__ in, uint64_t begin, uint64_t end, const LaneId& id) {
    static_assert(U % STEP == 0 && STEP % 2 == 0, "");
    const int lane_off = (FORM == kMfma) ? (kRow * id.j + 8 * id.g) : (8 * id.lane);
    float4v acc = splat(0.0f);
    float s0 = 0.0f, s1 = 0.0f;
    uint64_t t = begin;
    const uint64_t whole = begin + (end - begin) / (uint64_t)(kTile * U) * (uint64_t)(kTile * U);
#pragma unroll 1
    for (; t < whole; t += (uint64_t)(kTile * STEP)) {
        half8 x[STEP];
#pragma unroll
        for (int u = 0; u < STEP; ++u) x[u] = load8<true>(in, t + (uint64_t)(kTile * u + lane_off));
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            if constexpr (FORM == kMfma) acc = mfma(const_ones(), x[u], acc);
            else if (u & 1) s1 += sum8(x[u]);
            else s0 += sum8(x[u]);
        }
    }
    if (t < end) {                       // (as in reduce_span_kernel)
        const uint32_t left = (uint32_t)(end - t);
        const __amdgpu_buffer_rsrc_t src = make_rsrc(in + t, (left & ~7u) * 2u);
#pragma unroll 1
        for (uint32_t from = 0; from < left; from += (uint32_t)(kTile * STEP)) {
            half8 x[STEP];
#pragma unroll
            for (int u = 0; u < STEP; ++u) x[u] = buffer_load8<true>(src, (from + (uint32_t)(kTile * u + lane_off)) * 2u);
            if (left & 7u) {
#pragma unroll
                for (int u = 0; u < STEP; ++u) {
                    const uint32_t at = from + (uint32_t)(kTile * u + lane_off);
                    if (at == (left & ~7u)) x[u] = load8_guarded<true>(in, t + at, end);
                }
            }
#pragma unroll
            for (int u = 0; u < STEP; ++u) {
                if constexpr (FORM == kMfma) acc = mfma(const_ones(), x[u], acc);
                else s0 += sum8(x[u]);
            }
        }
    }
    if constexpr (FORM == kMfma) return read_lane(row_sum_to_last<16>(acc[0]), 15);
    else return read_lane(lanes_sum_to_last<64>(s0 + s1), 63);
}

template <int FORM>
__global__ __launch_bounds__(kGatherWaves * kWave) void reduce_gather_kernel(const ReduceGather a, const ScanWorkspace ws_arg) {
    __shared__ float s_total[kGatherWaves];
    const ScanWorkspace ws = resolve_workspace(ws_arg);
    const LaneId id;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t w = blockIdx.x * kGatherWaves + (uint32_t)wave;
    const auto span_end = [&a](uint64_t begin) { return begin + a.span < a.n ? begin + a.span : a.n; };
    if (w < a.nspans) {
        const uint64_t begin = (uint64_t)w * a.span;
        const float total = gather_span_sum<FORM, kGatherTiles, kGatherTiles>(a.in, begin, span_end(begin), id);
        if (id.lane == 0) {
            if (w == 0 && ws.state != nullptr && !ws.device_managed) ws.state[0] = ws.epoch;
            __hip_atomic_store(&ws.desc[w], pack_desc(ws.epoch, kStatusAggregate, total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    const uint32_t groups = (a.per + kGatherWaves - 1u) / kGatherWaves;          // workgroups of a segment
    const uint32_t seg = blockIdx.x / groups;
    if (blockIdx.x - seg * groups != groups - 1u) return;
    const uint32_t first = seg * a.per, want = ws.epoch * 4u + kStatusAggregate;
    float acc = 0.0f;
    constexpr uint32_t kRound = kGatherWaves * kWave * kGatherLoads;
    for (uint32_t base = 0; base < a.per; base += kRound) {
        const uint32_t mine = base + threadIdx.x;
        uint32_t polls = 0;
        float sum = 0.0f;
        while (true) {
            unsigned long long d[kGatherLoads];
#pragma unroll
            for (int k = 0; k < kGatherLoads; ++k) {
                const uint32_t i = mine + (uint32_t)(k * kGatherWaves * kWave);
                d[k] = load_descriptor(&ws.desc[first + (i < a.per ? i : a.per - 1u)]);
            }
            bool there = true;
            float v[kGatherLoads];
#pragma unroll
            for (int k = 0; k < kGatherLoads; ++k) {
                there = there && (uint32_t)(d[k] >> 32) == want;
                v[k] = mine + (uint32_t)(k * kGatherWaves * kWave) < a.per ? __builtin_bit_cast(float, (uint32_t)d[k]) : 0.0f;
            }
            // (in pairs: three roundings a round)
#pragma unroll
            for (int step = 1; step < kGatherLoads; step *= 2)
#pragma unroll
                for (int k = 0; k + step < kGatherLoads; k += 2 * step) v[k] += v[k + step];
            sum = v[0];
            if (__ballot(!there) == 0ull) break;
            if (++polls > a.patience) {
                // whole wavefront: every missing one of those it looks at (a lane's index beyond the end looks at the last)
#pragma unroll 1
                for (uint32_t k = 0; k < (uint32_t)kGatherLoads; ++k) {
                    const uint32_t at = mine + k * (uint32_t)(kGatherWaves * kWave);
                    const uint32_t i = first + (at < a.per ? at : a.per - 1u);
                    for (unsigned long long missing = __ballot((uint32_t)(load_descriptor(&ws.desc[i]) >> 32) != want); missing != 0ull;
                         missing &= missing - 1ull) {
                        const uint32_t which = (uint32_t)__builtin_amdgcn_readlane((int)i, __builtin_ctzll(missing));
                        const uint64_t begin = (uint64_t)which * a.span;
                        const float again = gather_span_sum<FORM, kGatherTiles, 2>(a.in, begin, span_end(begin), id);
                        if (id.lane == 0)
                            __hip_atomic_store(&ws.desc[which], pack_desc(ws.epoch, kStatusAggregate, again), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                polls = 0;                // (what this wavefront has stored itself it finds with its next look)
            } else {
                __builtin_amdgcn_s_sleep(1);
            }
        }
        acc += sum;
    }
    const float total = wave_sum(acc);
    if (id.lane == 0) s_total[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) a.out[seg] = pairwise_sum(s_total);
}

}  // namespace tcr
