// Sums (and sums of squares) of irregular segments in one launch, mostly for arrays of more than 2^23 elements.
//
// A workgroup of four wavefronts takes a range of consecutive tiles of 6144 elements.  It searches the offsets once, for the
// range's start, and from there on only reads entries: 512 at a time, each once, those of the next tile -- and its
// elements -- on their way while a tile is summed.  A tile's elements lie in LDS as they are, next to the sum of every
// group of 8 (two elements per v_dot2_f32_f16: exact products, added in binary32), and a segment's part of the tile is the
// groups that its two ends cut, masked, and the sums of the groups in between:
//   many short segments   one lane each (up to 8 groups in between; longer ones by eight lanes or the whole wavefront);
//   up to 64 in the tile  eight lanes each;
//   a handful             a wavefront each.
// Nothing is marked and nothing scanned: irregular_reduce_kernel, which forms running sums of every element that restart at
// segment starts and then picks the results from them, issues 119 vector instructions per 512 elements for sums of
// segments of 16 elements and 178 for both moments, this kernel 69 and 89 (2^26 elements).
//
// What reaches a tile from in front inside the range is one number (`carry`).  The part of the range's first result that
// lies in front of the range is added at the end: up to a tile of it from the elements, asked for at the start, more from
// the sums that the workgroups publish.  A sum that is not there after `patience` looks is added up again from the elements in
// the publishing workgroup's own order, so no wait depends on which workgroups run and no bit of a result on how they run.
//
// Bound: memory, and in front of it a range's start (two rounds of requests for the search, one for the entries): with one
// tile per workgroup those are half of a workgroup's time (64M elements, segments of 16: 51 us).  Against a look-up
// kernel, irregular_reduce_kernel and a finishing kernel, or up to 2^24 elements irregular_reduce_kernel with four
// searches per tile, us, n = 2^20 * 9 / 16 / 32 / 64 / 128: segments of 16 11.1 / 14.8 / 28.3 / 43.5 / 72.3 -> 8.9 / 12.0 / 21.2 / 36.6 /
// 66.2, both moments 13.0 / 21.3 / 36.9 / 57.5 / 99.0 -> 9.8 / 14.0 / 24.3 / 40.3 / 73.1.
// Registers: held to what seven workgroups per compute unit leave (both moments: six): 71 (77), with 48 (37) scalar ones spilled to
// lanes and nothing (20 bytes per lane) in scratch.
#pragma once
#include "tcr_irregular.hpp"

namespace tcr {

struct SegmentsReduce {
    const _Float16* in;           // `shift` elements in front of the caller's array, 16-byte aligned
    const uint64_t* offsets;      // nseg + 1 entries
    float* out;
    float* out2;                  // sums of squares (kBoth)
    uint64_t n;                   // elements counted from `in`
    uint64_t nseg;
    uint32_t shift;
    double per_elem;              // (nseg + 1) / n
    uint32_t grid_log2;           // distance of the first probes among the offsets
    uint32_t tiles;               // per workgroup
    uint32_t patience;
};

// Tiles of 6144 elements: 18.9 KiB of LDS (23.1 for both moments) leave room for the 7 (6) workgroups per compute unit that the
// registers do.  8192 elements, 24.6 KiB: 5 workgroups, 64M elements in segments of 16 42 us against 38; 4096: 45.
constexpr int kSegmentsU = 3, kSegmentsBatch = 2;        // 512-element sub-tiles per wavefront; entries per thread and batch
constexpr uint64_t kSegmentsTile = (uint64_t)kTile * kSegmentsU * 4;
// How a tile's segments are shared out, by their number m.  Segments of 512 / 128 / 64 elements (12 / 48 / 96 in a tile) at 64M
// elements, us: eight lanes each 34.3 / 36.4 / 42.5, one lane each (with eight for the long ones) 36.8 / 36.9 / 37.0.
constexpr uint32_t kFewEntries = 8, kSomeEntries = 64;
constexpr int kOneLaneMax = 8, kEightLanesMax = 64;      // groups of 8 elements between the two that the ends cut

typedef _Float16 half2d __attribute__((ext_vector_type(2)));

// acc + the sum (C = 0) or the sum of squares (C = 1) of eight elements.
template <int C>
__device__ __forceinline__ float dot8(half8 x, float acc) {
    const half2d one = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const half2d v = {x[2 * k], x[2 * k + 1]};
        acc = __builtin_amdgcn_fdot2(v, C == 0 ? one : v, acc, false);
    }
    return acc;
}

// What workgroup number `g` publishes, from its elements (whole wavefront; s0 is the workgroup's last segment start or lies
// in front of it), added in the order in which the workgroup itself adds.
template <int KIND, int C, int U, int WAVES>
__device__ __forceinline__ float segments_group_sum(const SegmentsReduce& a, uint64_t g, uint64_t s0, int lane) {
    constexpr uint64_t kChunk = (uint64_t)kTile * U;
    float run = 0.0f, total = 0.0f, v = 0.0f;
#pragma unroll 1
    for (uint32_t k = 0; k < a.tiles * (uint32_t)(U * WAVES); ++k) {
        const uint64_t at = g * a.tiles * (kChunk * WAVES) + (uint64_t)k * (uint64_t)kTile + 8 * (uint64_t)lane;
        const half8 x = load8_guarded<true>(a.in, at, a.n);
        v += dot8<C>(drop_leading(x, s0 > at ? (int)(s0 - at < 8 ? s0 - at : 8) : 0), 0.0f);
        if (k % U == U - 1) {
            total += wave_sum(v);
            v = 0.0f;
        }
        if (k % (U * WAVES) == U * WAVES - 1) {
            run += total;
            total = 0.0f;
        }
    }
    return run;
}

// This wavefront's share of the sum from position s0 to the start of workgroup `group` out of the published sums: the
// workgroup's wavefronts take turns at 64 * PER of them, all asked for before the first is looked at.
template <int KIND, int C, int U, int WAVES>
__device__ __forceinline__ float segments_linked_sum(const SegmentsReduce& a, const unsigned long long* desc, uint32_t epoch, uint32_t group,
                                                     uint64_t s0, int wave, int lane) {
    constexpr int PER = 4;
    constexpr uint32_t kSpan = PER * kWave;
    const uint64_t range = (uint64_t)(kTile * U * WAVES) * a.tiles;
    const uint32_t sums = group - (uint32_t)(s0 / range), want = epoch * 4u + kStatusAggregate;
    float acc = 0.0f;
    for (uint32_t at = (uint32_t)wave * kSpan; at < sums; at += WAVES * kSpan) {       // counted back from `group`
        const uint32_t span = sums - at < kSpan ? sums - at : kSpan, hi = group - at;
        float v[PER];
        for (uint32_t polls = 0;; ++polls) {
            unsigned long long d[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const uint32_t i = (uint32_t)(k * kWave + lane);
                d[k] = load_descriptor(&desc[hi - 1u - (i < span ? i : 0u)]);
            }
            uint32_t missing = 0u;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const bool counts = (uint32_t)(k * kWave + lane) < span;
                if (counts && (uint32_t)(d[k] >> 32) != want) missing |= 1u << k;
                v[k] = counts ? __builtin_bit_cast(float, (uint32_t)d[k]) : 0.0f;
            }
            if (__ballot(missing != 0u) == 0ull) break;
            if (polls >= a.patience) {
                for (unsigned long long lanes; (lanes = __ballot(missing != 0u)) != 0ull;) {
                    const int slot = __builtin_ctzll(lanes);
                    const int which = __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)missing, slot));
                    const float sum = segments_group_sum<KIND, C, U, WAVES>(a, hi - 1u - (uint32_t)(which * kWave + slot), s0, lane);
                    if (lane == slot) {
                        missing &= missing - 1u;
#pragma unroll
                        for (int k = 0; k < PER; ++k) v[k] = k == which ? sum : v[k];
                    }
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < PER; ++k) sum += v[k];
        acc += wave_sum(sum);
    }
    return acc;
}

// ws.desc: one sum per channel and workgroup, channel after channel.
template <int KIND>
__global__ __launch_bounds__(4 * kWave) __attribute__((amdgpu_waves_per_eu(KIND == kBoth ? 6 : 7))) void segments_reduce_kernel(SegmentsReduce a, ScanWorkspace ws_arg) {
    constexpr int WAVES = 4, U = kSegmentsU, K = kSegmentsBatch, CH = channels<KIND>();
    constexpr uint32_t kThreads = WAVES * kWave, kBatch = kThreads * K;      // entries read at once
    constexpr uint32_t kChunk = (uint32_t)kTile * U, kTileElems = kChunk * WAVES;
    constexpr uint32_t kPad = 16;                             // (groups behind the last one may be read, and count for nothing)
    static_assert(kTileElems <= 8192u, "");
    __shared__ __attribute__((aligned(16))) half8 s_data[kTileElems / 8 + kPad];
    // the bits of elements [lo, hi) of a group of 8, by 9 lo + hi
    __shared__ __attribute__((aligned(16))) uint4v s_mask[72];
    __shared__ uint16_t s_end[kBatch + 1];                    // where entry i of the batch lies: s_end[i + 1]
    __shared__ __attribute__((aligned(16))) uint32_t s_count[WAVES];
    __shared__ uint32_t s_list[CH][WAVES][kWave];             // segments for eight lanes each, then their sums
    __shared__ float s_total[CH][kTileElems / 8 + kPad];      // the sum of every group
    __shared__ float s_tail[CH][WAVES], s_ahead[CH][WAVES], s_kept[CH];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t range = (uint64_t)kTileElems * a.tiles;
    const uint64_t rb = (uint64_t)blockIdx.x * range;
    const uint64_t left = a.n - rb;                           // (a workgroup has at least one element)
    const uint32_t count = left < range ? (uint32_t)left : (uint32_t)range, whole_groups = count & ~7u;
    const uint32_t tiles = (count + kTileElems - 1) / kTileElems;
    if (threadIdx.x < 72) {
        const uint32_t lo = threadIdx.x / 9u, hi = threadIdx.x % 9u;
        const uint32_t bits = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
        uint4v m;
#pragma unroll
        for (int k = 0; k < 4; ++k) m[k] = ((bits >> (2 * k)) & 1u ? 0x0000ffffu : 0u) | ((bits >> (2 * k + 1)) & 1u ? 0xffff0000u : 0u);
        s_mask[threadIdx.x] = m;
    }

    // whole groups of 8 through the range check; the group that the array's end cuts is read again by element
    const __amdgpu_buffer_rsrc_t src = make_rsrc(a.in + rb, whole_groups * 2u);
    half8 x[U];
    const auto load_tile = [&](uint32_t at) {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = buffer_load8<true>(src, (at + (uint32_t)wave * kChunk + (uint32_t)(kTile * u + 8 * lane)) * 2u);
    };
    uint64_t entry[K];
    const auto load_entries = [&](uint64_t at) {
        const uint64_t rest = at <= a.nseg ? a.nseg + 1 - at : 0;
        const __amdgpu_buffer_rsrc_t from = make_rsrc(a.offsets + at, (uint32_t)(rest < (uint64_t)kBatch ? rest : (uint64_t)kBatch) * 8u);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t i = (uint32_t)k * kThreads + threadIdx.x;
            entry[k] = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(from, (int)(i * 8u), 0, 0));
        }
    };
    // at_entry: how many entries lie on rb or in front of it; s0: where the last of them, the start of the segment open at
    // rb, lies.  (Every wavefront looks for itself: one that looks for all four takes as long.  The range's first elements are
    // asked for behind the last round: what is asked for first arrives first.)
    const EntryFound found = find_entry(a.offsets, a.nseg + 1, rb + 1 > a.shift ? rb + 1 - a.shift : 0,
                                        (uint64_t)((double)rb * a.per_elem), a.grid_log2, lane, [&] { load_tile(0); }, [](uint64_t) { return false; });
    uint64_t at_entry = found.below;
    const uint64_t s0 = at_entry ? found.last + a.shift : rb;
    load_entries(at_entry);
    const bool open = at_entry >= 1 && at_entry <= a.nseg && s0 < rb;
    const bool far = open && rb - s0 > (uint64_t)kTileElems;
    if (rb == 0)                                              // entries on position 0 close empty segments in front of everything
        for (uint64_t s = 1 + (uint64_t)threadIdx.x; s < at_entry; s += kThreads) {
            a.out[s - 1] = 0.0f;
            if constexpr (CH == 2) a.out2[s - 1] = 0.0f;
        }
    if (open && !far) {
        float ahead[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) ahead[c] = 0.0f;
        const uint64_t at = rb - kTileElems + (uint64_t)wave * kChunk;
        if (at + kChunk > s0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint64_t mine = at + (uint64_t)(kTile * u + 8 * lane);
                const half8 y = drop_leading(load8<true>(a.in, mine), s0 > mine ? (int)(s0 - mine < 8 ? s0 - mine : 8) : 0);
                ahead[0] += dot8<0>(y, 0.0f);
                if constexpr (CH == 2) ahead[CH - 1] += dot8<1>(y, 0.0f);
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) ahead[c] = wave_sum(ahead[c]);
        }
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < CH; ++c) s_ahead[c][wave] = ahead[c];
    }

    float carry[CH];                                          // of the open segment: its elements in front of the tile
#pragma unroll
    for (int c = 0; c < CH; ++c) carry[c] = 0.0f;
    bool closed = false;                                      // a segment has ended
    const uint64_t first_segment = at_entry - 1;
    bool fresh = true;
    uint32_t from = 0;                                        // where the last segment in the tile has ended so far
    for (uint32_t t = 0; t < tiles;) {
        const uint64_t tb = rb + (uint64_t)t * kTileElems;
        if (fresh) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int g = wave * (int)(kChunk / 8) + u * kWave + lane;
                s_data[g] = x[u];
                s_total[0][g] = dot8<0>(x[u], 0.0f);
                if constexpr (CH == 2) s_total[CH - 1][g] = dot8<1>(x[u], 0.0f);
            }
            const uint32_t cut = (whole_groups - t * kTileElems) >> 3;        // (its own lane writes that group again)
            if (count != whole_groups && t + 1 == tiles && (cut & 63u) == (uint32_t)lane && cut / (kChunk / 8) == (uint32_t)wave) {
                const half8 y = load8_guarded(a.in, rb + whole_groups, a.n);
                s_data[cut] = y;
                s_total[0][cut] = dot8<0>(y, 0.0f);
                if constexpr (CH == 2) s_total[CH - 1][cut] = dot8<1>(y, 0.0f);
            }
        }
        if (threadIdx.x == 0) s_end[0] = (uint16_t)from;
        const uint64_t rest = at_entry <= a.nseg ? a.nseg + 1 - at_entry : 0;
        const uint32_t there = rest < (uint64_t)kBatch ? (uint32_t)rest : kBatch;
        const uint64_t base = tb - a.shift;                   // (modulo 2^64)
        uint32_t c_in = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t i = (uint32_t)k * kThreads + threadIdx.x;
            const int64_t p = (int64_t)(entry[k] - base);
            const bool in = i < there && p <= (int64_t)kTileElems;
            s_end[i + 1] = (uint16_t)(p > 0 ? (uint32_t)p : 0u);
            c_in += (uint32_t)__builtin_popcountll(__ballot(in));
        }
        if (lane == 0) s_count[wave] = c_in;
        lds_barrier();
        const uint4v counts = *reinterpret_cast<const uint4v*>(s_count);
        const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)(counts[0] + counts[1] + counts[2] + counts[3]));
        const bool more = m == kBatch;                        // (the next batch may lie in this tile as well)
        float* const out_at = a.out + at_entry;               // entry i of the batch closes segment at_entry + i - 1
        float* const out2_at = CH == 2 ? a.out2 + at_entry : nullptr;
        const uint32_t skip = at_entry == 0 ? 1u : 0u;        // (offsets[0] closes nothing)
        at_entry += m;
        if (fresh) load_tile((t + 1) * kTileElems);           // (behind the range: nothing)
        load_entries(at_entry);

        // where segment at_entry + i - 1 lies in the tile (i == m: nowhere).  Positions out of order are the caller's error; no
        // access leaves the tile for them.
        const auto place = [&](uint32_t i, uint32_t& begin, uint32_t& end) {
            begin = s_end[i < m ? i : 0u];
            end = s_end[i < m ? i + 1u : 0u];
            end = end < kTileElems ? end : kTileElems;
            begin = begin < end ? begin : end;
        };
        // the sum over a segment, the whole wavefront at once (the same arguments in every lane)
        const auto whole_wave = [&](uint32_t begin, uint32_t end, float (&value)[CH]) {
            const uint32_t g0 = begin >> 3, g1 = end >> 3;
            const bool same = g0 == g1;
#pragma unroll
            for (int c = 0; c < CH; ++c) value[c] = 0.0f;
            for (uint32_t g = g0 + 1u; g < g1; g += 4 * kWave) {
                float w[CH][4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t at = g + (uint32_t)(r * kWave + lane);
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const float v = s_total[c][at < g1 ? at : 0u];
                        w[c][r] = at < g1 ? v : 0.0f;
                    }
                }
#pragma unroll
                for (int c = 0; c < CH; ++c) value[c] += (w[c][0] + w[c][1]) + (w[c][2] + w[c][3]);
            }
            // (the cut groups to the first two lanes; in the others the masks leave nothing)
            const uint32_t lo = lane == 0 ? begin & 7u : 0u, hi = lane == 0 ? (same ? end & 7u : 8u) : (lane == 1 && !same ? end & 7u : 0u);
            const half8 cut = __builtin_bit_cast(half8, __builtin_bit_cast(uint4v, s_data[lane == 0 ? g0 : g1]) & s_mask[9u * lo + hi]);
            value[0] = wave_sum(value[0] + dot8<0>(cut, 0.0f));
            if constexpr (CH == 2) value[CH - 1] = wave_sum(value[CH - 1] + dot8<1>(cut, 0.0f));
        };
        // entry i's result, in the lane that `holds` it
        const auto finish = [&](bool holds, uint32_t i, float (&value)[CH]) {
            bool store = holds && i >= skip;
            if (i == 0u) {
#pragma unroll
                for (int c = 0; c < CH; ++c) value[c] += carry[c];
                if (!closed && open) {                        // its part in front of the range is added below
                    if (holds)
#pragma unroll
                        for (int c = 0; c < CH; ++c) s_kept[c] = value[c];
                    store = false;
                }
            }
            if (store) {
                out_at[(int)i - 1] = value[0];
                if constexpr (CH == 2) out2_at[(int)i - 1] = value[CH - 1];
            }
        };
        // entry i's segment, one lane each
        const auto take = [&](uint32_t i) {
            const bool active = i < m;
            uint32_t begin, end;
            place(active ? i : m, begin, end);
            const uint32_t g0 = begin >> 3, g1 = end >> 3;
            const bool same = g0 == g1;
            // (all reads before the first sum: one wait)
            uint4v head = __builtin_bit_cast(uint4v, s_data[g0]), foot = __builtin_bit_cast(uint4v, s_data[g1]);
            const uint4v head_mask = s_mask[9u * (begin & 7u) + (same ? end & 7u : 8u)], foot_mask = s_mask[same ? 0u : end & 7u];
            float near[CH][4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < CH; ++c) near[c][r] = s_total[c][g0 + 1u + (uint32_t)r];
            __builtin_amdgcn_sched_barrier(0);
            head &= head_mask;
            foot &= foot_mask;
            float value[CH];
            value[0] = dot8<0>(__builtin_bit_cast(half8, head), 0.0f) + dot8<0>(__builtin_bit_cast(half8, foot), 0.0f);
            if constexpr (CH == 2) value[CH - 1] = dot8<1>(__builtin_bit_cast(half8, head), 0.0f) + dot8<1>(__builtin_bit_cast(half8, foot), 0.0f);
            const int between = (int)g1 - (int)g0 - 1;
            const int mine = between <= kOneLaneMax ? between : 0;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < CH; ++c) value[c] += r < mine ? near[c][r] : 0.0f;
            if (__ballot(mine > 4) != 0ull) {
#pragma unroll
                for (int r = 4; r < kOneLaneMax; ++r)
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const float v = s_total[c][g0 + 1u + (uint32_t)r];
                        value[c] += r < mine ? v : 0.0f;
                    }
            }
            if (__ballot(between > kOneLaneMax) != 0ull) {
                // (a segment's groups in between by eight lanes, eight segments at once)
                const unsigned long long eight = __ballot(between > kOneLaneMax && between <= kEightLanesMax);
                const bool listed = (eight >> lane) & 1ull;
                const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(eight >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)eight, 0u));
                if (listed) s_list[0][wave][rank] = g0 | ((uint32_t)between << 16);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const uint32_t items = (uint32_t)__builtin_popcountll(eight);
                for (uint32_t p = 0; p < items; p += 8u) {
                    const uint32_t which = p + ((uint32_t)lane >> 3);
                    const uint32_t item = which < items ? s_list[0][wave][which] : 0u;
                    const uint32_t from_group = (item & 0xffffu) + 1u;
                    const int groups = (int)(item >> 16);
                    float part[CH];
#pragma unroll
                    for (int c = 0; c < CH; ++c) part[c] = 0.0f;
                    for (int g = lane & 7; __ballot(g < groups) != 0ull; g += 8)
#pragma unroll
                        for (int c = 0; c < CH; ++c) {
                            const float v = s_total[c][g < groups ? from_group + (uint32_t)g : 0u];
                            part[c] += g < groups ? v : 0.0f;
                        }
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const float sum = row_sum_to_last<8>(part[c]);
                        if ((lane & 7) == 7 && which < items) s_list[c][wave][which] = __builtin_bit_cast(uint32_t, sum);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if (listed) value[c] += __builtin_bit_cast(float, s_list[c][wave][rank]);
                for (unsigned long long all = __ballot(between > kEightLanesMax); all != 0ull; all &= all - 1ull) {
                    const int slot = __builtin_ctzll(all);
                    float sum[CH];
                    whole_wave((uint32_t)__builtin_amdgcn_readlane((int)begin, slot), (uint32_t)__builtin_amdgcn_readlane((int)end, slot), sum);
#pragma unroll
                    for (int c = 0; c < CH; ++c) value[c] = lane == slot ? sum[c] : value[c];
                }
            }
            finish(active, i, value);
        };
        if (m <= kFewEntries) {                               // a segment at a time to a whole wavefront
            for (uint32_t i = (uint32_t)wave; i < m; i += WAVES) {
                uint32_t begin, end;
                place(i, begin, end);
                float value[CH];
                whole_wave((uint32_t)__builtin_amdgcn_readfirstlane((int)begin), (uint32_t)__builtin_amdgcn_readfirstlane((int)end), value);
                finish(lane == 0, i, value);
            }
        } else if (m <= kSomeEntries) {                       // eight lanes per segment, one of over a thousand elements by all of them
            const uint32_t sub = (uint32_t)lane & 7u;
            for (uint32_t i = (uint32_t)wave + WAVES * ((uint32_t)lane >> 3); i - WAVES * ((uint32_t)lane >> 3) < m; i += 8 * WAVES) {
                const bool active = i < m;
                uint32_t begin, end;
                place(active ? i : m, begin, end);
                const uint32_t g0 = begin >> 3, g1 = end >> 3;
                const bool same = g0 == g1, far_apart = g1 - g0 > 2u * (uint32_t)kEightLanesMax;
                const uint32_t lo = sub == 0u ? begin & 7u : 0u, hi = sub == 0u ? (same ? end & 7u : 8u) : (sub == 1u && !same ? end & 7u : 0u);
                const half8 cut = __builtin_bit_cast(half8, __builtin_bit_cast(uint4v, s_data[sub == 0u ? g0 : g1]) & s_mask[9u * lo + hi]);
                float value[CH];
                value[0] = dot8<0>(cut, 0.0f);
                if constexpr (CH == 2) value[CH - 1] = dot8<1>(cut, 0.0f);
                const uint32_t stop = far_apart ? 0u : g1;
                for (uint32_t g = g0 + 1u + sub; __ballot(g < stop) != 0ull; g += 32u)
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        float w[4];
#pragma unroll
                        for (uint32_t r = 0; r < 4; ++r) {
                            const float v = s_total[c][g + 8u * r < stop ? g + 8u * r : 0u];
                            w[r] = g + 8u * r < stop ? v : 0.0f;
                        }
                        value[c] += (w[0] + w[1]) + (w[2] + w[3]);
                    }
#pragma unroll
                for (int c = 0; c < CH; ++c) value[c] = row_sum_to_last<8>(value[c]);
                for (unsigned long long rest = __ballot(active && far_apart && sub == 7u); rest != 0ull; rest &= rest - 1ull) {
                    const int slot = __builtin_ctzll(rest);
                    float sum[CH];
                    whole_wave((uint32_t)__builtin_amdgcn_readlane((int)begin, slot), (uint32_t)__builtin_amdgcn_readlane((int)end, slot), sum);
#pragma unroll
                    for (int c = 0; c < CH; ++c) value[c] = lane == slot ? sum[c] : value[c];
                }
                finish(active && sub == 7u, i, value);
            }
        } else if (m <= kThreads) {                           // a lane each, spread over the wavefronts
            if ((uint32_t)wave < m) take(WAVES * (uint32_t)lane + (uint32_t)wave);
        } else {                                              // a lane each, in 64s
            for (uint32_t first = (uint32_t)wave * kWave; first < m; first += kThreads)
                take(first + (uint32_t)lane);
        }
        if (m != 0u) {
            closed = true;
            from = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_end[m]);
            from = from < kTileElems ? from : kTileElems;
#pragma unroll
            for (int c = 0; c < CH; ++c) carry[c] = 0.0f;
        }
        if (!more) {                                          // what lies behind the last segment end, a quarter to each wavefront
            float sum[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) sum[c] = 0.0f;
            if (from < ((uint32_t)wave + 1u) * kChunk) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t g = (uint32_t)wave * (kChunk / 8) + (uint32_t)(u * kWave + lane);
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const float whole = s_total[c][g];
                        float v = 8u * g >= from ? whole : 0.0f;
                        if (g == from >> 3 && (from & 7u) != 0u) {
                            const half8 cut = __builtin_bit_cast(half8, __builtin_bit_cast(uint4v, s_data[g]) & s_mask[9u * (from & 7u) + 8u]);
                            v = c == 0 ? dot8<0>(cut, 0.0f) : dot8<1>(cut, 0.0f);
                        }
                        sum[c] += v;
                    }
                }
#pragma unroll
                for (int c = 0; c < CH; ++c) sum[c] = wave_sum(sum[c]);
            }
            if (lane == 0)
#pragma unroll
                for (int c = 0; c < CH; ++c) s_tail[c][wave] = sum[c];
        }
        lds_barrier();
        if (!more) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                float tail = 0.0f;
#pragma unroll
                for (int v = 0; v < WAVES; ++v) tail += s_tail[c][v];
                carry[c] += tail;
            }
            from = 0;
            ++t;
        }
        fresh = !more;
    }
    const ScanWorkspace ws = resolve_workspace(ws_arg);
    if (threadIdx.x == 0) {
        if (blockIdx.x == 0 && ws.state != nullptr && !ws.device_managed) ws.state[0] = ws.epoch;
#pragma unroll
        for (int c = 0; c < CH; ++c)
            __hip_atomic_store(&ws.desc[(uint64_t)c * gridDim.x + blockIdx.x], pack_desc(ws.epoch, kStatusAggregate, carry[c]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!open || !closed) return;                             // (the same in every wavefront)
    if (far) {
        const float sum = segments_linked_sum<KIND, 0, U, WAVES>(a, ws.desc, ws.epoch, blockIdx.x, s0, wave, lane);
        if (lane == 0) s_ahead[0][wave] = sum;
        if constexpr (CH == 2) {
            const float sum2 = segments_linked_sum<KIND, 1, U, WAVES>(a, ws.desc + gridDim.x, ws.epoch, blockIdx.x, s0, wave, lane);
            if (lane == 0) s_ahead[CH - 1][wave] = sum2;
        }
        lds_barrier();
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            float total = 0.0f;
#pragma unroll
            for (int v = 0; v < WAVES; ++v) total += s_ahead[c][v];
            (c == 0 ? a.out : a.out2)[first_segment] = s_kept[c] + total;
        }
    }
}

}  // namespace tcr
