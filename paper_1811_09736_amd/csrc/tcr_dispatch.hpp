// Host side of the library, part 2 of 3 (included by tcr_api.hip only): the dispatch from segment length
// to kernel and launch shape -- the role the paper gives its auto-tuner (Section 6) -- with the tuning
// table that tcr_autotune fills.
#pragma once
#include "tcr_workspace.hpp"

namespace tcr {
namespace host {

// ---------------------------------------------------------------------------- helpers
__global__ void fill_zero_kernel(float* out, uint64_t count) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = 0.0f;
}

inline bool is_pow2(uint64_t v) { return v != 0 && (v & (v - 1)) == 0; }
inline int log2u(uint64_t v) {
    int l = 0;
    while ((1ull << l) < v) ++l;
    return l;
}
inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

inline tcr_status check_launch(const char* what) {
    if (hip_failed(hipGetLastError(), what)) return TCR_ERR_HIP;
    return TCR_OK;
}


// ---------------------------------------------------------------------------- tuning table
// The paper selects algorithm, wavefronts per workgroup and coarsening per segment size with an
// auto-tuner (Section 6).  Here the defaults are frozen from sweeps on MI355X; tcr_autotune can
// re-time the candidates on the machine at hand and override the default for one class of
// segment lengths (index log2(seg_len), or kWholeClass for the one-segment operations).
constexpr int kWholeClass = 41;
// One table per kind of choice; an entry is -1 (the frozen default) or  id + 32 * formulation:
//   kTuneScan, kTuneReduce      powers of two from 16 and the one-segment operations, class = log2(seg_len) or
//                               kWholeClass.  id: a launch shape (small segments: kSmallScanShapes /
//                               kSmallReduceShapes; longer: kScanShapes incl. the two multi-kernel carry
//                               strategies / reduce_candidates); formulation 1 forces the cross-lane (DPP)
//                               arithmetic for the class (0: whatever tcr_set_variant says, matrix cores by default).
//   kTuneScanAny, kTuneReduceAny  every other seg_len, class = floor(log2(seg_len)).  id: which kernel takes the
//                               length (see scan_any_candidates / reduce_any_candidates).
//   kTuneIrregular              class 0: tile shape of tcr_irregular_reduce / _moments, class 1: of tcr_irregular_scan.
enum TuneTable { kTuneScan = 0, kTuneReduce = 1, kTuneScanAny = 2, kTuneReduceAny = 3, kTuneIrregular = 4, kTuneTables = 5 };
constexpr const char* kTuneTableNames[kTuneTables] = {"scan", "reduce", "scan_any", "reduce_any", "irregular"};
constexpr int kTuneFormBit = 32;
inline signed char g_tuned[kTuneTables][kWholeClass + 1];
inline bool g_tuning_initialised = false;
inline void init_tuning() {
    if (g_tuning_initialised) return;
    std::memset(g_tuned, -1, sizeof(g_tuned));
    g_tuning_initialised = true;
}
inline int tuning_class(uint64_t seg_len, bool whole) { return whole ? kWholeClass : log2u(seg_len); }
inline int floor_log2(uint64_t v) {
    int l = 0;
    while ((v >> (l + 1)) != 0) ++l;
    return l;
}
// The shape id chosen for a class (-1: none) and the formulation its kernels run.
inline int tuned_id(int table, int cls) {
    init_tuning();
    const int v = g_tuned[table][cls];
    return v < 0 ? -1 : (v & (kTuneFormBit - 1));
}
inline int tuned_formulation(int table, int cls) {
    init_tuning();
    const int v = g_tuned[table][cls];
    return (v >= 0 && (v & kTuneFormBit)) ? kDpp : g_variant.formulation;
}


// ---------------------------------------------------------------------------- reduce dispatch
// Launch shapes of the small-segment kernels (U tiles per wavefront, W wavefronts per workgroup); id 0 is the
// frozen default of each.
struct SmallShape { int u, w; };
constexpr SmallShape kSmallReduceShapes[] = {{kSmallReduceU, kSmallReduceW}, {1, 4}, {1, 8}, {4, 4}};
constexpr SmallShape kSmallScanShapes[] = {{1, kSmallScanW}, {1, 4}, {2, 2}, {2, 4}};
constexpr int kSmallShapeCount = 4;
// reduce_small keeps one result per lane: U * 512 / seg_len <= 64
inline bool small_reduce_shape_valid(int id, int log2l) {
    return id >= 0 && id < kSmallShapeCount && ((kTile >> log2l) * kSmallReduceShapes[id].u <= kWave);
}

template <int FORM, int U, int W>
inline void launch_reduce_small_shape(const _Float16* in, float* out, uint64_t n, int log2l, hipStream_t s) {
    const uint64_t blocks = ceil_div(n, (uint64_t)kTile * U * W);
    const dim3 grid((unsigned)blocks), block(W * kWave);
    switch (log2l) {
        case 4: if constexpr (U <= 2) reduce_small_kernel<FORM, 4, U, W><<<grid, block, 0, s>>>(in, out, n); break;
        case 5: reduce_small_kernel<FORM, 5, U, W><<<grid, block, 0, s>>>(in, out, n); break;
        case 6: reduce_small_kernel<FORM, 6, U, W><<<grid, block, 0, s>>>(in, out, n); break;
        case 7: reduce_small_kernel<FORM, 7, U, W><<<grid, block, 0, s>>>(in, out, n); break;
        case 8: reduce_small_kernel<FORM, 8, U, W><<<grid, block, 0, s>>>(in, out, n); break;
        default: reduce_small_kernel<FORM, 9, U, W><<<grid, block, 0, s>>>(in, out, n); break;
    }
}

template <int FORM>
inline tcr_status launch_reduce_small(const _Float16* in, float* out, uint64_t n, int log2l, hipStream_t s) {
    if (log2l < 4 || log2l > 9) return TCR_ERR_UNSUPPORTED;
    int shape = tuned_id(kTuneReduce, log2l);
    if (!small_reduce_shape_valid(shape, log2l)) shape = 0;
    if (FORM == kMfma && shape == 0 && g_variant.tile_load != kLoadDirect) {
        // the measured alternatives to loading operands directly (default shape only)
        constexpr int U = kSmallReduceU, W = kSmallReduceW;
        const dim3 grid((unsigned)ceil_div(n, (uint64_t)kTile * U * W)), block(W * kWave);
        const bool dma = g_variant.tile_load == kLoadLdsDma;
        switch (log2l) {
#define TCR_CASE(L) case L: if (dma) reduce_small_kernel<kMfma, L, U, W, kLoadLdsDma><<<grid, block, 0, s>>>(in, out, n); \
                            else reduce_small_kernel<kMfma, L, U, W, kLoadStaged><<<grid, block, 0, s>>>(in, out, n); break;
            TCR_CASE(4) TCR_CASE(5) TCR_CASE(6) TCR_CASE(7) TCR_CASE(8) TCR_CASE(9)
#undef TCR_CASE
        }
        return check_launch("reduce_small_kernel");
    }
    switch (shape) {
        case 1: launch_reduce_small_shape<FORM, 1, 4>(in, out, n, log2l, s); break;
        case 2: launch_reduce_small_shape<FORM, 1, 8>(in, out, n, log2l, s); break;
        case 3: launch_reduce_small_shape<FORM, 4, 4>(in, out, n, log2l, s); break;
        default: launch_reduce_small_shape<FORM, kSmallReduceU, kSmallReduceW>(in, out, n, log2l, s); break;
    }
    return check_launch("reduce_small_kernel");
}

template <int FORM>
inline tcr_status launch_reduce_span(const _Float16* in, float* dst, uint64_t n, uint64_t span, uint64_t nspans,
                              int combine_waves, hipStream_t s, const ReduceFinish* finish = nullptr) {
    const ReduceFinish none = {};
    if (finish != nullptr) {          // one partial per workgroup; the last workgroup adds them up
        if (combine_waves == 16) {
            const dim3 grid((unsigned)ceil_div(nspans, 16)), block(16 * kWave);
            if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 16, true, true><<<grid, block, 0, s>>>(in, dst, n, span, nspans, *finish);
            else if (span >= 4 * kTile) reduce_span_kernel<FORM, 4, 16, true, true><<<grid, block, 0, s>>>(in, dst, n, span, nspans, *finish);
            else reduce_span_kernel<FORM, 2, 16, true, true><<<grid, block, 0, s>>>(in, dst, n, span, nspans, *finish);
        } else if (combine_waves == 4) {
            reduce_span_kernel<FORM, 8, 4, true, true><<<dim3((unsigned)ceil_div(nspans, 4)), dim3(4 * kWave), 0, s>>>(
                in, dst, n, span, nspans, *finish);
        } else if (combine_waves == 2) {
            reduce_span_kernel<FORM, 8, 2, true, true><<<dim3((unsigned)ceil_div(nspans, 2)), dim3(2 * kWave), 0, s>>>(
                in, dst, n, span, nspans, *finish);
        } else {
            reduce_span_kernel<FORM, 8, 1, false, true><<<dim3((unsigned)nspans), dim3(kWave), 0, s>>>(in, dst, n, span, nspans,
                                                                                                       *finish);
        }
        return check_launch("reduce_span_kernel");
    }
    if (combine_waves == 16) {
        if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 16, true><<<dim3((unsigned)ceil_div(nspans, 16)), dim3(16 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
        else reduce_span_kernel<FORM, 4, 16, true><<<dim3((unsigned)ceil_div(nspans, 16)), dim3(16 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
    } else if (combine_waves == 8) {
        if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 8, true><<<dim3((unsigned)ceil_div(nspans, 8)), dim3(8 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
        else reduce_span_kernel<FORM, 4, 8, true><<<dim3((unsigned)ceil_div(nspans, 8)), dim3(8 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
    } else if (combine_waves == 4) {
        if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 4, true><<<dim3((unsigned)ceil_div(nspans, 4)), dim3(4 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
        else reduce_span_kernel<FORM, 4, 4, true><<<dim3((unsigned)ceil_div(nspans, 4)), dim3(4 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
    } else if (combine_waves == 2) {
        if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 2, true><<<dim3((unsigned)ceil_div(nspans, 2)), dim3(2 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
        else reduce_span_kernel<FORM, 4, 2, true><<<dim3((unsigned)ceil_div(nspans, 2)), dim3(2 * kWave), 0, s>>>(in, dst, n, span, nspans, none);
    } else {
        const dim3 grid((unsigned)nspans), block(kWave);
        if (span >= 8 * kTile) reduce_span_kernel<FORM, 8, 1, false><<<grid, block, 0, s>>>(in, dst, n, span, nspans, none);
        else if (span >= 4 * kTile) reduce_span_kernel<FORM, 4, 1, false><<<grid, block, 0, s>>>(in, dst, n, span, nspans, none);
        else reduce_span_kernel<FORM, 2, 1, false><<<grid, block, 0, s>>>(in, dst, n, span, nspans, none);
    }
    return check_launch("reduce_span_kernel");
}

struct ReducePlan {
    uint64_t span;      // elements per wavefront
    int combine;        // wavefronts per workgroup whose sums are added through LDS (1: none)
    uint64_t per;       // partials per segment left for reduce_final_kernel (1: results go straight to out)
    uint64_t nspans;    // wavefronts in total
    bool finish;        // the partials are added up by the workgroup that finishes last
};

// Arrays whose partials the last workgroup adds up: at most 128 of them, of a workgroup's share each, and one more per
// segment where segments end inside a share (one count on one address takes 12 ns).  Full reduction of 2^18 / 2^20 / 2^22 / 2^23 elements, us back to back: two kernels 6.8 / 6.9 /
// 6.7 / 6.7, one launch 4.5 / 4.5 / 5.9 / 7.0 -- and 3.3 us less for the host at every size, which is the longer of the two
// up to there.  (One workgroup and no partials at all up to 2^17: 3.7 at 2^16, 4.9 at 2^17.)
constexpr uint64_t kFinishElemsMax = 1ull << 23;
constexpr uint64_t kFinishSums = 32;                     // results that the last workgroup adds up
constexpr uint64_t kFinishShares = 128;
static_assert(kFinishShares + kFinishSums <= kFinishCount, "a launch counts each of its workgroups");
inline uint64_t finish_share(uint64_t n) {
    uint64_t share = 16384;
    while (ceil_div(n, share) > kFinishShares) share <<= 1;
    return share;
}

// How many wavefronts an array is shared among, if its size allows: a wavefront keeps 8 KiB of loads in flight, and 16
// wavefronts per compute unit is where more of them no longer help.
constexpr uint64_t kWavesWanted = 4096;
constexpr uint64_t kSpanMin = 2048;                      // no share below four tiles ...
constexpr uint64_t kOneGroupSegment = 1ull << 17;        // longest segment that one workgroup of 16 wavefronts takes
// Share of a wavefront when the array may be cut anywhere.
inline uint64_t free_span(uint64_t n) {
    uint64_t span = 4096;
    while (span < kWaveSpanMax && n / span > kWavesWanted) span <<= 1;
    return span;
}

// Reduce candidates for seg_len >= 1024 (power of two) or one segment: (span, combine) pairs.
struct ReduceShape { uint64_t span; int combine; };
inline int reduce_candidates(uint64_t n, uint64_t seg_len, bool whole, ReduceShape* c) {
    int k = 0;
    if (!whole && seg_len <= kWaveSpanMax) {
        c[k++] = {seg_len, 1};                                   // one wavefront per segment
        if (seg_len >= 8192) c[k++] = {seg_len / 2, 2};
        if (seg_len >= 16384) c[k++] = {seg_len / 4, 4};
        return k;
    }
    if (whole) {
        const uint64_t span = free_span(n);
        if (ceil_div(n, span) == 1) {
            c[k++] = {ceil_div(n, kTile) * kTile, 1};
            return k;
        }
        c[k++] = {span, kReduceBlockW};                          // default
        c[k++] = {span, 1};
        if (span > 16384) c[k++] = {span / 4, kReduceBlockW};
        if (span > 32768) c[k++] = {span / 2, kReduceBlockW};
        return k;
    }
    c[k++] = {kWaveSpanMax, (seg_len / kWaveSpanMax >= (uint64_t)kReduceBlockW) ? kReduceBlockW : 2};   // default
    c[k++] = {kWaveSpanMax, 1};
    c[k++] = {16384, 4};
    c[k++] = {32768, 4};
    return k;
}

// seg_len >= 1024 (a power of two), or one segment of any length (whole).
// coarse: no more partials than one per 65536 elements of a segment, or per 4096 of the array if it is one segment (a
// workspace that cannot be grown).  two_kernels: the partials, if any, are left to reduce_final_kernel.
inline ReducePlan plan_reduce(uint64_t n, uint64_t seg_len, bool whole, bool coarse = false, bool two_kernels = false) {
    ReduceShape cand[4];
    const int count = reduce_candidates(n, seg_len, whole, cand);
    bool finish = false;
    int pick = tuned_id(kTuneReduce, tuning_class(seg_len, whole));
    const bool untuned = pick < 0 || pick >= count;
    if (untuned) {
        // frozen defaults for an array that fills the chip whatever the split: segments of 8192 .. 32768 elements over
        // 2 or 4 wavefronts; from 2^18 elements on (and for one segment) every wavefront leaves a partial of its own
        // for the second kernel -- combining the wavefronts of a workgroup first holds each back to the slowest
        // (n = 2^28: 81.5-81.9 us against 83.9-86.1 us with 4 combined; 8 or 16 combined, which make a segment of 2^19
        // or 2^20 elements one workgroup's and the second kernel unnecessary, 84.1 and 90.8 us)
        if (whole || seg_len >= (1ull << 18)) pick = count > 1 ? 1 : 0;
        else pick = (seg_len < 8192 || seg_len > 32768) ? 0 : (seg_len == 8192 ? 1 : 2);
    }
    // (the tuner's first candidate, too, is run in one launch where that is possible: it has to find what untuned calls run)
    if (untuned || pick == 0) {
        const bool long_one = whole ? count > 1 : seg_len > kOneGroupSegment;
        if (whole && long_one && n <= kOneGroupSegment) {
            cand[pick = 0] = {ceil_div(ceil_div(n, 16), kTile) * kTile, 16};       // one workgroup, no partials
        } else if (long_one && n <= kFinishElemsMax && (whole || n / seg_len <= kFinishSums) && !coarse && !two_kernels && !g_variant.reduce_fused) {
            cand[pick = 0] = {finish_share(n) / 16, 16};
            finish = true;
        } else if (untuned && !whole) {
            ReduceShape c = cand[pick];
            if (seg_len <= kOneGroupSegment) {
                // too few wavefronts to fill the chip: halve their shares, up to one workgroup of 16 per segment
                const uint64_t w0 = seg_len / c.span;
                uint64_t w = w0;
                while (w < 16 && (n / seg_len) * w < kWavesWanted / 2 && seg_len / w > kSpanMin) w <<= 1;
                if (w != w0) c = {seg_len / w, (int)w};
            } else if (!coarse) {
                c.span = free_span(n);                           // (a divisor of seg_len: both are powers of two)
            }
            cand[pick = 0] = c;
        }
    }
    ReducePlan p;
    p.span = cand[pick].span;
    p.combine = cand[pick].combine;
    const uint64_t len = whole ? n : seg_len;
    p.per = ceil_div(len, p.span * (uint64_t)p.combine);
    p.nspans = whole ? ceil_div(n, p.span) : n / p.span;
    p.finish = finish && p.per > 1;
    return p;
}

// The second kernel of the device-level reduction: one workgroup per segment over its `per` partials.
// out2: a second set of nseg * per partials behind the first goes there (the sums of squares), in the same launch.
inline void launch_reduce_final(const float* partials, float* out, float* out2, uint64_t nseg, uint64_t per, hipStream_t s) {
    const dim3 grid((unsigned)nseg, out2 != nullptr ? 2u : 1u);
    if (per > kFinalThreads) reduce_final_kernel<kFinalThreadsMax><<<grid, dim3(kFinalThreadsMax), 0, s>>>(partials, out, out2, per, nseg * per);
    else reduce_final_kernel<kFinalThreads><<<grid, dim3(kFinalThreads), 0, s>>>(partials, out, out2, per, nseg * per);
}

// Partials of one wavefront each that the last workgroup of a segment collects (tcr_gather.hpp) instead of a second kernel.
// Several segments: whole workgroups each.  Not on a workspace whose launches a graph has recorded: there the descriptors cost a
// launch in front of this one, and it would again be two.
// Up to 2^24 elements, where two launches keep the host longer than one the device (8.0 to 9.4 us at any size up to 2^24; one launch 5.4
// to 6.1, 8.1 in some runs at 2^24).  Beyond, the two overlap and the collecting workgroup does not: two against one, n = 2^20 * 24 / 32 / 64 / 128 / 256 11.1 / 13.5 /
// 23.6 / 44.0 / 81.4 us against 11.2 / 14.5 / 23.9 / 46.0 / 83.6.
constexpr uint64_t kGatherElemsMax = 1ull << 24;
inline bool gather_better(const ReducePlan& p, uint64_t n, uint64_t nseg) {
    return n <= kGatherElemsMax && p.per > 1 && p.combine == 1 && !p.finish && p.span >= (uint64_t)(kGatherTiles * kTile) &&
           (nseg == 1 || p.per % kGatherWaves == 0);
}
template <int FORM>
inline tcr_status launch_reduce_gather(const _Float16* in, float* out, uint64_t n, const ReducePlan& p, Workspace* ws, hipStream_t s) {
    ScanWorkspace dev = {};
    tcr_status st = begin_lookback(ws, s, p.nspans, &dev, false);
    if (st != TCR_OK) return st;
    const ReduceGather a = {in, out, n, p.span, (uint32_t)p.per, (uint32_t)p.nspans, g_variant.scan_wait ? kOncePatience : 0u};
    const dim3 grid((unsigned)ceil_div(p.nspans, (uint64_t)kGatherWaves)), block(kGatherWaves * kWave);
    reduce_gather_kernel<FORM><<<grid, block, 0, s>>>(a, dev);
    st = check_launch("reduce_gather_kernel");
    if (st != TCR_OK) ws->dirty = true;
    return st;
}

inline tcr_status reduce_long(const _Float16* in, float* out, uint64_t n, uint64_t seg_len, bool whole, hipStream_t s) {
    ReducePlan p = plan_reduce(n, seg_len, whole);
    const int form = tuned_formulation(kTuneReduce, tuning_class(seg_len, whole));
    const uint64_t nseg = whole ? 1 : n / seg_len;
    float* dst = out;
    Workspace* ws = nullptr;
    bool capturing = false;
    if (p.per > 1) {
        tcr_status st = get_workspace(s, &ws, &capturing);
        if (st != TCR_OK) return st;
        uint32_t* counter = p.finish ? finish_counter(ws, capturing) : nullptr;
        if (p.finish && counter == nullptr) p = plan_reduce(n, seg_len, whole, false, true);
        if (nseg * p.per > partials_limit(ws, capturing)) p = plan_reduce(n, seg_len, whole, true);
        st = ensure_partials(ws, s, nseg * p.per, capturing);
        if (st != TCR_OK) return st;
        dst = ws->partials;
        if (p.finish) {
            const ReduceFinish fin = {out, nullptr, counter, 0u, (uint32_t)nseg, (uint32_t)p.per, 1u};
            return form == kMfma ? launch_reduce_span<kMfma>(in, dst, n, p.span, p.nspans, p.combine, s, &fin)
                                 : launch_reduce_span<kDpp>(in, dst, n, p.span, p.nspans, p.combine, s, &fin);
        }
    }
    if (gather_better(p, n, nseg) && !g_variant.reduce_fused && !capturing && !ws->device_managed && table_has_room(ws, p.nspans, capturing))
        return form == kMfma ? launch_reduce_gather<kMfma>(in, out, n, p, ws, s) : launch_reduce_gather<kDpp>(in, out, n, p, ws, s);
    if (p.per > 1 && g_variant.reduce_fused && nseg * p.per <= kFusedPartialsMax) {
        // one kernel: the workgroup that finishes last adds up the partials
        if (capturing || ws->device_managed) return TCR_ERR_UNSUPPORTED;     // its count base is a kernel argument
        ScanWorkspace dev = {};
        tcr_status st = begin_lookback(ws, s, 0, &dev, false);   // the running counter that also hands out scan tiles
        if (st != TCR_OK) return st;
        const ReduceFinish fin = {out, nullptr, dev.ticket, dev.ticket_base, (uint32_t)nseg, (uint32_t)p.per, 0u};
        st = form == kMfma ? launch_reduce_span<kMfma>(in, dst, n, p.span, p.nspans, p.combine, s, &fin)
                                            : launch_reduce_span<kDpp>(in, dst, n, p.span, p.nspans, p.combine, s, &fin);
        if (st != TCR_OK) {
            ws->dirty = true;
            return st;
        }
        ws->tickets_issued += (uint32_t)(nseg * p.per);   // one count per workgroup
        return TCR_OK;
    }
    tcr_status st = form == kMfma ? launch_reduce_span<kMfma>(in, dst, n, p.span, p.nspans, p.combine, s)
                                                   : launch_reduce_span<kDpp>(in, dst, n, p.span, p.nspans, p.combine, s);
    if (st != TCR_OK) return st;
    if (p.per > 1) {
        launch_reduce_final(dst, out, nullptr, nseg, p.per, s);
        st = check_launch("reduce_final_kernel");
    }
    return st;
}


// ---------------------------------------------------------------------------- scan dispatch
// MODE bit 0: exclusive, bit 1: binary16 output (TCR_SCAN_EXCLUSIVE, TCR_OUT_F16).
template <int FORM, int MODE, int U, int W>
inline void launch_scan_small_shape(const _Float16* in, void* out, uint64_t n, int log2l, hipStream_t s) {
    const uint64_t blocks = ceil_div(n, (uint64_t)kTile * U * W);
    const dim3 grid((unsigned)blocks), block(W * kWave);
    switch (log2l) {
        case 4: scan_small_kernel<FORM, 4, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
        case 5: scan_small_kernel<FORM, 5, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
        case 6: scan_small_kernel<FORM, 6, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
        case 7: scan_small_kernel<FORM, 7, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
        case 8: scan_small_kernel<FORM, 8, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
        default: scan_small_kernel<FORM, 9, U, W, MODE><<<grid, block, 0, s>>>(in, out, n); break;
    }
}

template <int FORM, int MODE>
inline tcr_status launch_scan_small(const _Float16* in, void* out, uint64_t n, int log2l, hipStream_t s) {
    if (log2l < 4 || log2l > 9) return TCR_ERR_UNSUPPORTED;
    int shape = tuned_id(kTuneScan, log2l);
    if (shape < 0 || shape >= kSmallShapeCount) shape = 0;
    if constexpr (FORM == kMfma && MODE == 0) {
        if (shape == 0 && g_variant.tile_load != kLoadDirect) {
            // the measured alternatives to loading operands directly (default shape, plain mode only)
            constexpr int W = kSmallScanW;
            const dim3 grid((unsigned)ceil_div(n, (uint64_t)kTile * W)), block(W * kWave);
            const bool dma = g_variant.tile_load == kLoadLdsDma;
            switch (log2l) {
#define TCR_CASE(L) case L: if (dma) scan_small_kernel<kMfma, L, 1, W, 0, kLoadLdsDma><<<grid, block, 0, s>>>(in, out, n); \
                            else scan_small_kernel<kMfma, L, 1, W, 0, kLoadStaged><<<grid, block, 0, s>>>(in, out, n); break;
                TCR_CASE(4) TCR_CASE(5) TCR_CASE(6) TCR_CASE(7) TCR_CASE(8) TCR_CASE(9)
#undef TCR_CASE
            }
            return check_launch("scan_small_kernel");
        }
    }
    switch (shape) {
        case 1: launch_scan_small_shape<FORM, MODE, 1, 4>(in, out, n, log2l, s); break;
        case 2: launch_scan_small_shape<FORM, MODE, 2, 2>(in, out, n, log2l, s); break;
        case 3: launch_scan_small_shape<FORM, MODE, 2, 4>(in, out, n, log2l, s); break;
        default: launch_scan_small_shape<FORM, MODE, 1, kSmallScanW>(in, out, n, log2l, s); break;
    }
    return check_launch("scan_small_kernel");
}

template <int FORM, int U, int W, int CARRY, int MODE>
inline void launch_scan_block(const _Float16* in, void* out, uint64_t n, uint64_t seg_mask, uint64_t seg_len,
                       const ScanWorkspace& dev, const float* prefix, hipStream_t s) {
    const unsigned blocks = (unsigned)ceil_div(n, (uint64_t)kTile * U * W);
    scan_block_kernel<FORM, U, W, CARRY, MODE><<<dim3(blocks), dim3(W * kWave), 0, s>>>(
        in, out, n, seg_mask, seg_len, dev, prefix);
}

// Launch shapes of scan_block_kernel.  Ids 0..6 take tiles in blockIdx order and need a whole
// segment inside one workgroup share; ids 7..9 hand tiles out by ticket (tiles are then processed
// in the order workgroups actually start, which keeps the tiles in flight contiguous in memory and
// measured 5-9 % faster for 1024-thread workgroups even without a carry) and chain workgroups
// through the look-back when a segment is longer than the share.  One ticket costs about 12 ns of
// a chip-wide serial resource, so ticketed shares start at 16384 elements.
// Ids 10 and 11 are scan_chain_kernel: persistent workgroups (one per compute unit) that take
// 32768-element tiles by ticket in a loop and keep three in flight (loading, aggregate published,
// carry looked up and stored); for segments of at least one tile and the one-segment scan,
// n a multiple of 8.  Id 10 runs most arrays as one tile per workgroup: those that the chip holds all at once (once_share) and, with
// carries from the relay, larger ones (chain_relayed).
struct ScanShape { int u, w; bool ticket; int persistent; };      // persistent: workgroups per compute unit (0: one per tile)
constexpr ScanShape kScanShapes[] = {{1, 2, false, 0}, {1, 4, false, 0}, {1, 8, false, 0}, {1, 16, false, 0},
                                     {2, 16, false, 0}, {4, 16, false, 0}, {8, 16, false, 0}, {2, 16, true, 0},
                                     {4, 16, true, 0}, {8, 16, true, 0}, {4, 16, true, 1}, {8, 8, true, 1}};
constexpr int kScanShapeCount = 12;
// Two more ids choose a multi-kernel carry strategy instead of a single-pass shape (segments longer than one
// 65536-element share only): the paper's three-kernel scan-then-propagate (Section 5) and reduce-then-scan.
// (14: one segment whose n is no multiple of 8 -- the chain over the whole groups of 8, then scan_tail_kernel)
constexpr int kScanIdReduceThenScan = 12, kScanIdScanThenPropagate = 13, kScanIdChainTail = 14, kScanIdCount = 15;
inline uint64_t scan_shape_tile(int id) { return (uint64_t)kTile * kScanShapes[id].u * kScanShapes[id].w; }

inline bool scan_shape_valid(int id, uint64_t len, bool whole) {      // len: seg_len, or n for the one-segment scan
    if (id == kScanIdReduceThenScan || id == kScanIdScanThenPropagate) return len > kCarryTile;
    if (id == kScanIdChainTail) return whole && len % 8 != 0 && len >= 2 * scan_shape_tile(10) && g_variant.scan_carry == kStrategyLookback;
    if (id < 0 || id >= kScanShapeCount) return false;
    if (kScanShapes[id].persistent)                             // (whole: len == n, which must be a multiple of 8)
        return whole ? len % 8 == 0 : len >= scan_shape_tile(id);
    return kScanShapes[id].ticket || scan_shape_tile(id) >= len;
}

// Compute units of the current device (cached per device id).
inline int compute_units() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int cu = 0;
        if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0) cu = 256;
        cached[dev] = cu;
    }
    return cached[dev];
}

// n: elements of the whole call (the defaults for segments of 8192 and 16384 depend on it).
inline int default_scan_shape(uint64_t n, uint64_t len, bool whole, int form) {
    if (len <= 1024) return 0;
    if (len <= 2048) return 1;
    if (len <= 4096) return 2;
    if (len < 8192 || (whole && len == 8192)) return 3;
    // one workgroup per segment, in blockIdx order while the array is not much larger than the memory-side cache (8192
    // elements: n = 2^20 / 2^24 / 2^26 / 2^27 3.8 / 20.8 / 70.5 / 136 us against 5.3 / 28.6 / 79.8 / 147 by ticket; 16384:
    // 4.4 / 23.3 / 76.6 / 151 against 5.3 / 28.9 / 77.5 / 141), by ticket in arrays that stream from memory
    if (!whole && len == 8192 && n < (1ull << 28)) return 3;
    if (!whole && len == 16384 && n < (1ull << 27)) return 4;
    if (!whole && len <= 16384) return 7;          // one ticketed share per segment (two segments of 8192)
    // the pipelined chain: segments of 32768 and more, one segment with n % 8 == 0.  (16 wavefronts of 4 tiles
    // for the matrix cores; the DPP arithmetic needs more registers and takes 8 wavefronts of 8 tiles.)
    if (scan_shape_valid(10, len, whole)) return form == kMfma ? 10 : 11;
    // n not a multiple of 8: one tile per workgroup where id 10 has that, else the chain over the whole groups of 8 and a second, tiny kernel for the rest (measured
    // at n = 2^28 - 3: 297 us against 307-323 us for scan_block_kernel with decoupled look-back, which short arrays keep)
    if (scan_shape_valid(kScanIdChainTail, len, whole)) return kScanIdChainTail;
    if (whole && len < (1u << 16)) return 7;       // a few shares (n = 2^15: 5.2 us against 7.4 with one large share)
    return (whole || len >= (1u << 20)) ? 9 : 8;
}

inline int pick_scan_shape(uint64_t n, uint64_t len, bool whole) {
    const int cls = tuning_class(len, whole);
    const int tuned = tuned_id(kTuneScan, cls);
    return scan_shape_valid(tuned, len, whole) ? tuned : default_scan_shape(n, len, whole, tuned_formulation(kTuneScan, cls));
}

template <int FORM, int CARRY, int MODE>
inline void launch_scan_shape(int id, const _Float16* in, void* out, uint64_t n, uint64_t seg_mask, uint64_t seg_len,
                       const ScanWorkspace& dev, const float* prefix, hipStream_t s) {
    // CARRY is kNoCarry for ids 0..6 and kLookback for ids 7..9
    if constexpr (CARRY == kNoCarry) {
        switch (id) {
            case 0: launch_scan_block<FORM, 1, 2, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 1: launch_scan_block<FORM, 1, 4, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 2: launch_scan_block<FORM, 1, 8, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 3: launch_scan_block<FORM, 1, 16, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 4: launch_scan_block<FORM, 2, 16, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 5: launch_scan_block<FORM, 4, 16, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            default: launch_scan_block<FORM, 8, 16, kNoCarry, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
        }
    } else {
        switch (id) {
            case 7: launch_scan_block<FORM, 2, 16, kLookback, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            case 8: launch_scan_block<FORM, 4, 16, kLookback, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
            default: launch_scan_block<FORM, 8, 16, kLookback, MODE>(in, out, n, seg_mask, seg_len, dev, prefix, s); break;
        }
    }
}

// Smallest blockIdx-ordered shape that holds `fit` elements (used by the multi-kernel strategies).
inline int nocarry_shape_for(uint64_t fit) {
    for (int id = 0; id < 7; ++id)
        if (scan_shape_tile(id) >= fit) return id;
    return 6;
}

// The chain as one tile per workgroup: tiles of 16 wavefronts with the result's number of 512-element tiles each -- the
// smallest of which there are no more than compute units and no more than `limit` (descriptors of a workspace that
// cannot be grown).  Segments that overhang their last tile may need more tiles than that; they take 32768-element
// tiles, up to the same size of array.  0: the array is too large for the chip to hold at once (2^24 elements: 22.5 us
// against 28.5 with the pipeline; 2^24 + 32768: 30.8 against 28.7).
inline uint64_t once_tiles(uint64_t n, uint64_t seg_len, int u) { return (n / seg_len) * ceil_div(seg_len, (uint64_t)(kTile * 16 * u)); }
inline int once_share(uint64_t n, uint64_t seg_len, uint64_t limit) {
    const uint64_t units = (uint64_t)compute_units();
    if (n > units * (uint64_t)(kTile * 16 * 8)) return 0;
    for (int u = 1; u <= 8; u *= 2) {
        if (u > 1 && (uint64_t)(kTile * 16 * u) > seg_len) break;
        const uint64_t tiles = once_tiles(n, seg_len, u);
        if (tiles <= units && tiles <= limit) return u;
    }
    return 4;
}
template <int MODE>
tcr_status launch_chain_once(const _Float16* in, void* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    ScanWorkspace dev = {};
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    const int u = once_share(n, seg_len, table_limit(ws, capturing));
    const uint64_t tiles = once_tiles(n, seg_len, u);
    st = begin_lookback(ws, s, tiles, &dev, capturing);
    if (st != TCR_OK) return st;
    const ChainGrid grid = {seg_len, (uint32_t)(tiles / (n / seg_len)), (uint32_t)tiles, g_variant.scan_wait ? kOncePatience : 0u};
    const dim3 blocks((unsigned)tiles), block(16 * kWave);
    if (u == 1) scan_chain_kernel<kMfma, 1, 16, MODE, false, kChainOnce><<<blocks, block, 0, s>>>(in, out, grid, dev, nullptr);
    else if (u == 2) scan_chain_kernel<kMfma, 2, 16, MODE, false, kChainOnce><<<blocks, block, 0, s>>>(in, out, grid, dev, nullptr);
    else if (u == 4) scan_chain_kernel<kMfma, 4, 16, MODE, false, kChainOnce><<<blocks, block, 0, s>>>(in, out, grid, dev, nullptr);
    else scan_chain_kernel<kMfma, 8, 16, MODE, false, kChainOnce><<<blocks, block, 0, s>>>(in, out, grid, dev, nullptr);
    st = check_launch("scan_chain_kernel");
    if (st != TCR_OK) ws->dirty = true;
    return st;
}

// The chain with carries from the relay (tcr_relay.hpp), in tiles of 8192 elements, for arrays larger than the chip holds at once: two
// words of the table per tile.  us, the persistent chain against this, n in 2^20, full scan:
//   binary32   n = 16.001  26.8/21.0   20  30.5/25.1   24  39.5/33.2   32  46.0/42.5   64  81.2/74.8   128  148/140   256  281/270   512  546/531
//   binary16       16.001  21.0/17.2   20  22.9/18.7   24  24.4/20.7   32  30.9/26.8   64  53.2/50.0   128  96.6/96.5   160  117/118   256  181/183
// (segments of 65536: 20 30.0/25.3, 256 276/271; of 65544: 24 44.2/36.4, 64 89.1/78.6, 128 160/148.)  And where one tile per compute unit would
// have to be one of 65536 elements (kChainOnce) and segments are long, full scan of 8.001 / 9 / 10 / 11 / 12 15.5/13.4, 15.7/14.3, 16.0/14.8, 16.3/15.8,
// 16.6/16.5; segments of 262144 9 / 11 15.1/14.3, 15.7/15.8; of 65536 9 14.2/14.3; binary16 10 9.8/12.5.
constexpr uint64_t kRelayTile = (uint64_t)(kTile * 4 * kRelayWaves);
inline uint64_t relay_tiles(uint64_t n, uint64_t seg_len) { return (n / seg_len) * ceil_div(seg_len, kRelayTile); }
inline bool chain_relayed(uint64_t n, uint64_t seg_len, bool f16) {
    const int once = once_share(n, seg_len, ~0ull);
    if (once != 0) return once == 8 && !f16 && seg_len >= (1ull << 18) && n <= (21ull << 19);
    return !f16 || n <= (3ull << 25);
}
// On a caller's buffer, which is ordinary memory, the relay costs more (2^20 * 80 / 96 elements, binary16: 7 and 8 % more than the persistent chain; none more up to 64
// and with binary32 results).
inline bool chain_relay_room(const Workspace* ws, bool capturing, uint64_t n, uint64_t seg_len, bool f16) {
    return !(ws->caller_owned && f16 && n > (1ull << 26)) && 2 * relay_tiles(n, seg_len) <= table_limit(ws, capturing);
}
template <int MODE>
tcr_status launch_chain_relay(Workspace* ws, bool capturing, const _Float16* in, void* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    const uint64_t tiles = relay_tiles(n, seg_len);
    ScanWorkspace dev = {};
    tcr_status st = begin_lookback(ws, s, 2 * tiles, &dev, capturing);
    if (st != TCR_OK) return st;
    const ChainGrid grid = {seg_len, (uint32_t)(tiles / (n / seg_len)), (uint32_t)tiles, g_variant.scan_wait ? kOncePatience : 0u};
    scan_chain_kernel<kMfma, 4, kRelayWaves, MODE, false, kChainRelay><<<dim3((unsigned)tiles + 1), dim3(kRelayWaves * kWave), 0, s>>>(in, out, grid, dev, nullptr);
    st = check_launch("scan_chain_kernel");
    if (st != TCR_OK) ws->dirty = true;
    return st;
}

// The persistent chain (shape 10 or 11) over segments of `seg_len` elements: any multiple of 8 that is at
// least one tile, or one segment of n elements (n a multiple of 8).  With `used` the caller reads the totals of the
// chain's own tiles out of the table afterwards, so the array is not run as one tile per workgroup, whatever its size.
template <int FORM, int MODE>
tcr_status launch_chain(int shape, const _Float16* in, void* out, uint64_t n, uint64_t seg_len, hipStream_t s,
                        ScanWorkspace* used = nullptr, uint32_t* used_tiles = nullptr) {
    const bool held = shape == 10 && used == nullptr && once_share(n, seg_len, ~0ull) != 0;
    const bool alone = shape == 10 && used == nullptr && chain_relayed(n, seg_len, (MODE & 2) != 0);
    if constexpr (FORM == kMfma) {
        if (held && !alone) return launch_chain_once<MODE>(in, out, n, seg_len, s);
    }
    const uint64_t tile = scan_shape_tile(shape);
    const uint64_t per_segment = ceil_div(seg_len, tile);
    const uint64_t tiles = (n / seg_len) * per_segment;
    ScanWorkspace dev = {};
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    if constexpr (FORM == kMfma) {
        if (alone && chain_relay_room(ws, capturing, n, seg_len, (MODE & 2) != 0)) return launch_chain_relay<MODE>(ws, capturing, in, out, n, seg_len, s);
        if (alone && held) return launch_chain_once<MODE>(in, out, n, seg_len, s);
    }
    st = begin_lookback(ws, s, tiles, &dev, capturing);
    if (st != TCR_OK) return st;
    const uint64_t resident = (uint64_t)compute_units() * (uint64_t)kScanShapes[shape].persistent;
    const uint64_t groups = tiles < resident ? tiles : resident;
    const ChainGrid grid = {seg_len, (uint32_t)per_segment, (uint32_t)tiles, 0};
    if (shape == 10) scan_chain_kernel<FORM, 4, 16, MODE><<<dim3((unsigned)groups), dim3(16 * kWave), 0, s>>>(in, out, grid, dev, nullptr);
    else scan_chain_kernel<FORM, 8, 8, MODE><<<dim3((unsigned)groups), dim3(8 * kWave), 0, s>>>(in, out, grid, dev, nullptr);
    st = check_launch("scan_chain_kernel");
    if (st != TCR_OK) {
        ws->dirty = true;
        return st;
    }
    ws->tickets_issued += (uint32_t)(tiles + 3 * groups);   // three drawn at the start of every workgroup, one per tile
    if (used != nullptr) *used = dev;
    if (used_tiles != nullptr) *used_tiles = (uint32_t)tiles;
    return TCR_OK;
}

// One segment of n elements, n no multiple of 8: the chain over the first n - n % 8, then the rest.
template <int FORM, int MODE>
tcr_status launch_chain_tail(const _Float16* in, void* out, uint64_t n, hipStream_t s) {
    if constexpr (FORM == kMfma) {
        // (these cut the last group themselves)
        const bool held = once_share(n, n, ~0ull) != 0;
        if (chain_relayed(n, n, (MODE & 2) != 0)) {
            Workspace* ws = nullptr;
            bool capturing = false;
            const tcr_status st = get_workspace(s, &ws, &capturing);
            if (st != TCR_OK) return st;
            if (chain_relay_room(ws, capturing, n, n, (MODE & 2) != 0)) return launch_chain_relay<MODE>(ws, capturing, in, out, n, n, s);
        }
        if (held) return launch_chain_once<MODE>(in, out, n, n, s);
    }
    const uint64_t n8 = n & ~7ull;
    ScanWorkspace dev = {};
    uint32_t tiles = 0;
    tcr_status st = launch_chain<FORM, MODE>(FORM == kMfma ? 10 : 11, in, out, n8, n8, s, &dev, &tiles);
    if (st != TCR_OK) return st;
    scan_tail_kernel<MODE><<<dim3(1), dim3(kTailThreads), 0, s>>>(in, out, n8, n, dev, tiles);
    return check_launch("scan_tail_kernel");
}

// seg_len >= 1024 (power of two), or the full scan (seg_len == n, any n).
template <int FORM, int MODE>
inline tcr_status scan_long(const _Float16* in, void* out, uint64_t n, uint64_t seg_len, bool whole, hipStream_t s) {
    const uint64_t seg_mask = whole ? ~0ull : seg_len - 1;
    const uint64_t host_seg_len = seg_len;            // decides the launch; the kernels see a saturated
    if (whole) seg_len = ~0ull;                       // length for the one-segment case (n need not be a power of two)
    // the carry strategy: forced by tcr_set_variant, else the class's tuned choice, else the single pass
    int strategy = g_variant.scan_carry;
    int shape = strategy == kStrategyLookback ? pick_scan_shape(n, host_seg_len, whole) : -1;
    if (shape == kScanIdReduceThenScan) strategy = kStrategyReduceThenScan;
    if (shape == kScanIdScanThenPropagate) strategy = MODE == 0 ? kStrategyScanThenPropagate : kStrategyLookback;
    if (shape == kScanIdChainTail) return launch_chain_tail<FORM, MODE>(in, out, n, s);
    if (shape >= kScanShapeCount) shape = default_scan_shape(n, host_seg_len, whole, FORM);    // (the strategies have fixed shapes)
    if (shape == kScanIdChainTail) shape = 9;             // (a forced multi-kernel strategy: its no-carry shares do not use it)
    const bool table = strategy != kStrategyLookback;     // the two multi-kernel strategies
    if (table && host_seg_len <= kCarryTile) {
        const ScanWorkspace none = {};
        launch_scan_shape<FORM, kNoCarry, MODE>(nocarry_shape_for(host_seg_len), in, out, n, seg_mask, seg_len, none, nullptr, s);
        return check_launch("scan_block_kernel");
    }
    if (!table) {
        if (!kScanShapes[shape].ticket) {
            const ScanWorkspace none = {};
            launch_scan_shape<FORM, kNoCarry, MODE>(shape, in, out, n, seg_mask, seg_len, none, nullptr, s);
            return check_launch("scan_block_kernel");
        }
        if (kScanShapes[shape].persistent) return launch_chain<FORM, MODE>(shape, in, out, n, host_seg_len, s);
        const uint64_t tiles = ceil_div(n, scan_shape_tile(shape));
        ScanWorkspace dev = {};
        Workspace* ws = nullptr;
        bool capturing = false;
        tcr_status st = get_workspace(s, &ws, &capturing);
        if (st != TCR_OK) return st;
        st = begin_lookback(ws, s, tiles, &dev, capturing);
        if (st != TCR_OK) return st;
        launch_scan_shape<FORM, kLookback, MODE>(shape, in, out, n, seg_mask, seg_len, dev, nullptr, s);
        st = check_launch("scan_block_kernel");
        if (st != TCR_OK) {
            ws->dirty = true;
            return st;
        }
        ws->tickets_issued += (uint32_t)tiles;      // one per workgroup; wraps modulo 2^32 like the device counter
        return TCR_OK;
    }
    if (strategy == kStrategyScanThenPropagate) {
        // the paper's three kernels; totals are read back from the binary32 inclusive output
        if (MODE != 0) return TCR_ERR_UNSUPPORTED;
        const uint64_t shares = ceil_div(n, kCarryTile);
        Workspace* w = nullptr;
        bool capturing = false;
        tcr_status st = get_workspace(s, &w, &capturing);
        if (st != TCR_OK) return st;
        st = ensure_partials(w, s, shares, capturing);
        if (st != TCR_OK) return st;
        const ScanWorkspace none = {};
        float* o = static_cast<float*>(out);
        launch_scan_block<FORM, kCarryU, kCarryW, kNoCarry, 0>(in, out, n, kCarryTile - 1, kCarryTile, none, nullptr, s);
        st = check_launch("scan_block_kernel");
        if (st != TCR_OK) return st;
        gather_totals_kernel<<<dim3((unsigned)ceil_div(shares, 256)), dim3(256), 0, s>>>(o, w->partials, kCarryTile, shares, n);
        st = check_launch("gather_totals_kernel");
        if (st != TCR_OK) return st;
        const uint64_t per = whole ? shares : host_seg_len / kCarryTile;
        scan_partials_kernel<<<dim3((unsigned)(whole ? 1 : n / host_seg_len)), dim3(kPartialsThreads), 0, s>>>(w->partials, per);
        st = check_launch("scan_partials_kernel");
        if (st != TCR_OK) return st;
        uniform_add_kernel<<<dim3((unsigned)ceil_div(n, 4096)), dim3(256), 0, s>>>(o, w->partials, kCarryTile, n);
        return check_launch("uniform_add_kernel");
    }
    const uint64_t tiles = ceil_div(n, kCarryTile);
    ScanWorkspace dev = {};
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    // reduce-then-scan: workgroup totals, their exclusive scan per segment, then the scan proper
    st = ensure_partials(ws, s, tiles, capturing);
    if (st != TCR_OK) return st;
    // one wavefront span per workgroup tile; spans are uniform because seg_len is a multiple of the tile (or one segment)
    st = launch_reduce_span<FORM>(in, ws->partials, n, kCarryTile, tiles, 1, s);
    if (st != TCR_OK) return st;
    const uint64_t per = whole ? tiles : host_seg_len / kCarryTile;
    const uint64_t groups = whole ? 1 : n / host_seg_len;
    scan_partials_kernel<<<dim3((unsigned)groups), dim3(kPartialsThreads), 0, s>>>(ws->partials, per);
    st = check_launch("scan_partials_kernel");
    if (st != TCR_OK) return st;
    launch_scan_block<FORM, kCarryU, kCarryW, kTable, MODE>(in, out, n, seg_mask, seg_len, dev, ws->partials, s);
    return check_launch("scan_block_kernel");
}

// Irregular segments: fixed tiles of the flat array, whatever the segments.  Tile shapes (U sub-tiles of 512
// elements per wavefront, W wavefronts); id 0 is the frozen default: 32768-element tiles for the chained scan,
// 8192-element tiles of four wavefronts for the reduction, whose tiles are independent (measured at n = 2^28:
// 90 us against 92 us with eight wavefronts of four sub-tiles on log-normal lengths, 143 against 153 us on
// segments of 16 elements on average: a tile's work is a chain of dependent steps -- its range of offsets
// entries, the entries, the marks, the sums -- and small workgroups keep more tiles in flight per compute unit).
constexpr SmallShape kIrregularScanShapes[] = {{4, 16}, {2, 16}};
constexpr SmallShape kIrregularReduceShapes[] = {{4, 4}, {4, 8}, {2, 8}};
constexpr int kIrregularScanShapeCount = 2, kIrregularReduceShapeCount = 3;
inline int irregular_shape(bool scan) {
    const int id = tuned_id(kTuneIrregular, scan ? 1 : 0);
    return (id >= 0 && id < (scan ? kIrregularScanShapeCount : kIrregularReduceShapeCount)) ? id : 0;
}
inline uint64_t irregular_tile_elems(bool scan, int shape) {
    const SmallShape t = scan ? kIrregularScanShapes[shape] : kIrregularReduceShapes[shape];
    return (uint64_t)kTile * t.u * t.w;
}
inline uint64_t irregular_tiles(bool scan, uint64_t n, int shape) { return ceil_div(n, irregular_tile_elems(scan, shape)); }
// 8-byte words of the partials area: the look-up table(s) of the tile boundaries, and for the reduction one
// carried-segment index and one pair per tile and channel.
inline uint64_t irregular_words(bool scan, uint64_t n, int shape, uint64_t ch = 1) {
    const uint64_t tiles = irregular_tiles(scan, n, shape);
    // (scan: the look-up table and one TileLink per tile)
    return scan ? 2 * tiles + 1 : 2 * (tiles + 1) + (1 + ch) * tiles;
}
// Reductions over segments of thousands of tiles also combine the pairs of every 64 tiles.  Segments of 1024 tiles on
// average, in arrays that do not run as one launch, us, without / with the combined pairs: one segment of 2^20 * 48 / 64 /
// 128 / 256 / 511 elements 22.8 / 27.8 / 50.0 / 95.8 / 186.9 against 22.0 / 26.6 / 46.5 / 87.8 / 170.3, two segments 21.8 / 26.3 /
// 47.1 / 89.5 / 176.4 against 22.0 / 26.4 / 45.7 / 85.7 / 167.7, seven 21.8 / 27.5 / 49.1 / 90.9 / 178.1 against 22.1 / 26.7 / 47.0 /
// 87.0 / 169.0, forty (818 tiles each at 2^28) 21.7 / 26.8 / 46.1 / 86.4 against 22.4 / 27.4 / 46.8 / 85.8; lognormal lengths
// 23.7 / 28.3 / 47.5 / 87.3 / 170.1 against 25.6 / 30.1 / 49.3 / 89.0 / 172.8.
inline uint64_t irregular_groups(uint64_t tiles) { return ceil_div(tiles, kWave); }
inline bool irregular_far(uint64_t tiles, uint64_t nseg) { return tiles > 4096 && tiles / 1024 >= nseg; }
// The largest of these over the tile shapes (the smallest tiles): what tcr_workspace_bytes reports.
inline uint64_t irregular_tiles_max(bool scan, uint64_t n) {
    uint64_t m = 0;
    for (int id = 0; id < (scan ? kIrregularScanShapeCount : kIrregularReduceShapeCount); ++id)
        if (irregular_tiles(scan, n, id) > m) m = irregular_tiles(scan, n, id);
    return m;
}
inline uint64_t irregular_words_max(bool scan, uint64_t n) {
    uint64_t m = 0;
    for (int id = 0; id < (scan ? kIrregularScanShapeCount : kIrregularReduceShapeCount); ++id)
        if (irregular_words(scan, n, id) > m) m = irregular_words(scan, n, id);
    return m;
}

// The tiles start at the 16-byte boundary at or below `in`: `shift` elements in front of it (0 for aligned arrays).
inline uint32_t alignment_shift(const _Float16* in) { return (uint32_t)((reinterpret_cast<uintptr_t>(in) & 15u) / 2u); }

// offsets == nullptr: regular segments of seg_len elements (no look-up table; MODE as for the other scans).
// in: 2-byte aligned; out: aligned to its element size.  shape: an id of kIrregularScanShapes.
template <int MODE, int U, int W>
inline void launch_irregular_scan_shape(bool regular, const _Float16* in, const uint64_t* offsets, void* out, uint64_t n, uint64_t nseg,
                                        const uint64_t* starts, uint64_t seg_len, uint32_t shift, uint32_t vector_stores,
                                        const ScanWorkspace& dev, uint64_t tiles, hipStream_t s) {
    const dim3 grid((unsigned)tiles), block(W * kWave);
    if (regular) irregular_scan_kernel<U, W, true, MODE><<<grid, block, 0, s>>>(in, nullptr, out, n, nseg, nullptr, seg_len, shift, vector_stores, dev);
    else irregular_scan_kernel<U, W, false, MODE><<<grid, block, 0, s>>>(in, offsets, out, n, nseg, starts, 0, shift, vector_stores, dev);
}

// Zeros to the positions of [shift, n) that no segment covers.
template <int F16>
inline tcr_status launch_fill_outside(const uint64_t* offsets, uint64_t nseg, void* out, uint64_t n, uint32_t shift, hipStream_t s) {
    fill_outside_kernel<F16><<<dim3((unsigned)compute_units()), dim3(256), 0, s>>>(offsets, nseg, out, n, shift);
    return check_launch("fill_outside_kernel");
}

// Distance of the 64 probes with which a workgroup's search among the offsets starts, as a power of two: they reach four standard deviations of
// where n / nseg uniform lengths put an entry to either side.
inline uint32_t search_grid_log2(uint64_t nseg) {
    uint32_t log2 = 6;
    while (log2 < 40 && (64ull << (2 * log2)) < nseg) ++log2;
    return log2;
}

// One tile per workgroup (tcr_once.hpp).  in, out, n: already counted from the 16-byte boundary below the caller's array.
template <int U, int W, int MODE, bool LOCAL, int SUMS = kSumsWide>
inline void launch_tile_scan(const TileScan& a, const ScanWorkspace& dev, hipStream_t s) {
    const dim3 grid((unsigned)ceil_div(a.n, (uint64_t)(kTile * U * W)) + (SUMS == kSumsRelayed ? 1u : 0u)), block(W * kWave);
    if (LOCAL || a.offsets == nullptr) tile_scan_kernel<U, W, true, MODE, LOCAL, SUMS><<<grid, block, 0, s>>>(a, dev);
    else if constexpr (!LOCAL) tile_scan_kernel<U, W, false, MODE, false, SUMS><<<grid, block, 0, s>>>(a, dev);
}
// Up to here the compute units hold all workgroups at once (256 units: 2^24 elements).
inline uint64_t scan_held_max() { return (uint64_t)compute_units() * (uint64_t)(kTile * 16 * 8); }
constexpr uint64_t kNearSevenMax = 39ull << 19;       // (irregular_sums)
template <int MODE>
inline tcr_status launch_scan_once(const _Float16* in, const uint64_t* offsets, void* out, uint64_t n, uint64_t nseg, uint64_t seg_len,
                                   uint32_t shift, bool fill, TileSums sums, hipStream_t s) {
    TileScan a = {};
    a.in = in;
    a.offsets = offsets;
    a.out = out;
    a.n = n;
    a.nseg = nseg;
    a.seg_len = seg_len;
    a.shift = shift;
    a.vector_stores = aligned(out, 16) ? 1u : 0u;
    a.fill = fill ? 1u : 0u;
    a.patience = g_variant.scan_wait ? kOncePatience : 0u;
    const bool local = offsets == nullptr && seg_len <= kLocalMax;
    if (offsets == nullptr) {
        a.per_elem = 1.0 / (double)seg_len;
        for (uint32_t i = 0; i < 8; ++i)
            if (i % seg_len == 0) a.pattern |= 1u << i;
    } else {
        a.per_elem = (double)(nseg + 1) / (double)n;
        a.grid_log2 = search_grid_log2(nseg);
    }
    ScanWorkspace dev = {};
    if (local && sums == kSumsWide) {
        a.magic = (uint32_t)(((1ull << 32) + seg_len - 1) / seg_len);
        // 8 wavefronts, so that the open part is a small share of what a workgroup reads -- unless segments are short and
        // the array streams from memory (seg_len 33 at n = 2^24 / 2^26 / 2^28: 23.2 / 74.8 / 285 us with 8, 23.6 / 73.3 /
        // 276 with 16; 2001: 22.7 / 74.4 / 277 and 24.0 / 77.8 / 290; binary16 results, 33 at 2^26 / 2^27 / 2^28: 42.2 / 91.9 /
        // 179 with 8, 43.8 / 100.8 / 196 with 16), or longer than 8 wavefronts can add up at once
        // Long open parts are added in binary64 beyond what the chip holds at once where the relay would take them (tiles_relayed) if it were as fast: 8191 elements in
        // 2^20 * 22 / off a boundary in 2^20 * 64 32.9 / 181.6 -> 32.7 / 179.5 us.  On a boundary 4097 to 6144 elements would lose 1 to 3 %.
        if (MODE < 2 && n > scan_held_max() && seg_len > (a.vector_stores != 0u ? 6144u : 4096u))
            tile_scan_kernel<1, 16, true, MODE, true, kSumsWide, 8, MODE < 2 ? kCarryExact : kCarryEarly><<<dim3((unsigned)ceil_div(n, (uint64_t)(kTile * 16))), dim3(16 * kWave), 0, s>>>(a, dev);
        else if (seg_len > 4096 || (!(MODE & 2) && seg_len <= 1024 && n > (1ull << 24))) launch_tile_scan<1, 16, MODE, true>(a, dev, s);
        else launch_tile_scan<1, 8, MODE, true>(a, dev, s);
        return check_launch("tile_scan_kernel");
    }
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    const uint64_t limit = table_limit(ws, capturing);
    if (sums != kSumsWide) {
        const uint64_t tiles = ceil_div(n, kRelayTile);
        // (looked-up sums need one; asked for where it can be had, so that the same call can be recorded with other offsets)
        st = begin_lookback(ws, s, sums == kSumsLookedUp && 2 * tiles > limit ? tiles : 2 * tiles, &dev, capturing);
        if (st != TCR_OK) return st;
        // (7 wavefronts per SIMD: up to 72 registers where the relay alone, with binary32 results, takes 49; none to 24 bytes of scratch
        // per lane, with binary16 results up to 76 with 64 registers)
        if (sums == kSumsLookedUp) tile_scan_kernel<4, kRelayWaves, false, MODE, false, kSumsLookedUp, 7><<<dim3((unsigned)tiles), dim3(kRelayWaves * kWave), 0, s>>>(a, dev);
        else if (sums == kSumsNear) {
            constexpr int MOST = MODE < 2 ? 8 : 7;
            if (n > kNearSevenMax) tile_scan_kernel<4, kRelayWaves, false, MODE, false, kSumsNear, MOST><<<dim3((unsigned)tiles + 1), dim3(kRelayWaves * kWave), 0, s>>>(a, dev);
            else tile_scan_kernel<4, kRelayWaves, false, MODE, false, kSumsNear, 7><<<dim3((unsigned)tiles + 1), dim3(kRelayWaves * kWave), 0, s>>>(a, dev);
        }
        else launch_tile_scan<4, kRelayWaves, MODE, false, kSumsRelayed>(a, dev, s);
        st = check_launch("tile_scan_kernel");
        if (st != TCR_OK) ws->dirty = true;
        return st;
    }
    // Workgroups of 8 wavefronts, small enough that the compute units get about equally many: with 4096, 8192 and 16384
    // elements a tile n = 2.2e6 7.6 / 7.2 / 8.4 us, 5.2e6 15.1 / 11.7 / 12.3, 8e6 20.5 / 16.5 / 14.7 (seven segments; lognormal
    // lengths and regular segments of 10802 and 198163 elements alike), 2^24 - / 31.7 / 27.4.  16 wavefronts, 16384 and
    // 32768 elements: 2.2e6 7.9 / 11.1, 5.2e6 15.0 / 13.1, 8e6 17.2 / 15.8, 2^24 33.6 / 27.2 -- better where every unit just
    // gets one (4.1e6: 9.5 us against 10.1), and 32768 where the table has no room for more tiles.
    const uint64_t units = (uint64_t)compute_units();
    const auto tiles_of = [n](int u, int w) { return ceil_div(n, (uint64_t)(kTile * u * w)); };
    int u = 4, w = 8;
    if (tiles_of(1, 8) <= 2 * units) u = 1;
    else if (tiles_of(2, 16) <= units && 4 * tiles_of(2, 16) > 3 * units) u = 2, w = 16;
    else if (tiles_of(2, 8) <= 3 * units) u = 2;
    if (tiles_of(u, w) > limit) u = 4, w = tiles_of(4, 8) > limit ? 16 : 8;
    st = begin_lookback(ws, s, tiles_of(u, w), &dev, capturing);
    if (st != TCR_OK) return st;
    // (regular segments where workgroups follow each other: six wavefronts per SIMD in place of eight.  9001 / 30003 elements, n = 2^26 76.3 / 77.9 against
    // 79.0 / 78.4 us, 2^28 275 / 278 against 287 / 279)
    if (u == 1) launch_tile_scan<1, 8, MODE, false>(a, dev, s);
    else if (u == 2 && w == 8) launch_tile_scan<2, 8, MODE, false>(a, dev, s);
    else if (u == 2) launch_tile_scan<2, 16, MODE, false>(a, dev, s);
    else if (w == 8 && offsets == nullptr && n > scan_held_max()) {
        // (in binary64 where results are stored by element, which hides it: 9001 / 30003 / 100003 elements off a boundary in 2^20 * 64 184.7 / 188.0 / 191.0 -> 184.8 / 187.3 / 190.1;
        // on one in 2^20 * 22 33.9 / 34.3 / - -> 34.5 / 34.7 / -)
        const dim3 grid((unsigned)tiles_of(4, 8)), block(8 * kWave);
        if (a.vector_stores == 0u) tile_scan_kernel<4, 8, true, MODE, false, kSumsWide, 6, MODE < 2 ? kCarryExact : kCarryLate><<<grid, block, 0, s>>>(a, dev);
        else tile_scan_kernel<4, 8, true, MODE, false, kSumsWide, 6><<<grid, block, 0, s>>>(a, dev);
    }
    else if (w == 8) launch_tile_scan<4, 8, MODE, false>(a, dev, s);
    else launch_tile_scan<4, 16, MODE, false>(a, dev, s);
    st = check_launch("tile_scan_kernel");
    if (st != TCR_OK) ws->dirty = true;
    return st;
}

// Scans in fixed tiles whose carries come from the relay: us, the other forms (the wavefronts add the open part up themselves or
// look up what tiles in front have published, or chained tiles) against this, n in 2^20.
// Irregular segments: beyond what the chip holds at once, up to 9 * 2^24 elements (below: irregular_sums).  What the others cost there goes by the longest
// segment, which the host does not know; the relay's does not.
//   binary32        n = 32          64          128         256
//     2              94.8/87.2   164.6/150.9
//     16             63.0/54.1   103.1/95.0  178.5/168.4 328/322
//     lognormal      55.1/48.0   90.3/83.6   158.9/155.3 294/299
//     seven          55.2/46.4   91.0/81.8   159.1/151.6 292/293
//     one, 1023 empty   -        98.8/84.9        -      293/302
//   binary16, exclusive
//     16             44.9/37.0   73.3/64.0   124.8/113.7 228/214
//     lognormal         -        61.1/56.6   107.2/106.1 197/202
//     seven             -        62.3/55.3   107.0/104.5 191/199
// Regular segments and seven irregular ones, of more than 2^20 elements on average: binary32 from 12 * 2^20 elements on (3000003 at 14.3: 21.7/19.4, 22.9: 32.6/30.8, 62.9:
// 91.3/76.7, 126: 167.9/143.8; seven at 12 / 14 / 16 18.6/18.4, 21.6/19.9, 22.8/21.5).
// Other regular ones, beyond 2^24, by length, type and alignment (chained tiles, which took some lengths of 4097 to 8191 elements: 64 85, 128 152, 256 287;
// binary16 64 50, 128 102, 256 190):
//   binary32   5001: 32 43.0/44.4, 48 61.0/61.8, 56 70.2/69.4, 128 151/146, 256 296/281; 8191: 18 28.4/28.9, 24 35.1/37.0 (from the memory-side cache 17
//              20.6/22.1), 28 equal, 64 81.8/78.2, 128 159/146, 256 313/281; 9001 (looked up): 24 33.0/33.7, 64 76.3/78.0, 256 275/281; 30003: 20 26.3/26.3,
//              64 77.9/77.7, 256 278/281; 50003: 17 22.9/22.3, 64 78.8/78.0; 100003: 17 23.1/22.3, 64 80.0/78.0, 128 148.2/145.2
//   binary16   2001: 64 49.8/50.3, 256 187/181; 3001: 48 39.8/41.9, 64 51.2/50.1, 128 97.9/94.5, 256 191/181; 5001: 17 17.0/18.1, 24 21.7/21.7, 28 26.9/25.1,
//              64 60.3/50.6; 8001: 17 18.2/18.1, 20 20.5/19.4, 64 62.4/50.4; 9001: 48 34.2/36.9, 128 92.5/97.1, 256 179/184; 40000: 128 95.1/97.6, 256 184/187;
//              100003: 48 3 % less, 128 97.7/98.5, 256 187/186; 500003: 17 17.9/18.9, 28 24.9/25.9, 32 29.2/27.5, 48 44.3/42.6; 3000003: 17 18.8/18.9,
//              23 22.5/21.6, 26 25.0/23.7
// Where input or results lie off a 16-byte boundary, results are stored by element, twice the time, and tiles that store in the order of the array are in each other's
// way:  binary32  5001: 64 6 % less, 256 701/735; 8191: 18 57.2/60.5, 24 73.4/78.8, 128 356/374, 256 702/734; 40000: 18 63.5/60.0, 24 78.3/78.4, 48 5 % less, 128
//                 363/374; 100003: 18 64.7/60.7, 128 366/374; 500003: 64 5 % more, 256 7 % more
//       binary16  3001: 128 194/211, 256 385/412; 5001: 28 51.7/54.2, 36 65.5/66.7, 48 85.4/85.3, 64 112/108, (chained tiles) 96 159/160, 128 205/210,
//                 256 393/411; 9001: 48 8 % less, 256 379/408; 262168: 48 4 % less, 256 8 % less; 1000003: equal
inline bool tiles_relayed(uint64_t n, uint64_t nseg, uint64_t seg_len, bool regular, bool f16, bool vector_stores) {
    const bool far = nseg << 20 < n;                     // more than 2^20 elements a segment
    if (n <= scan_held_max()) return far && !f16 && n > (3ull << 22);
    if (!regular) return n <= (9ull << 24);
    if (far) return true;
    if (!vector_stores && f16) return seg_len > 4096 && seg_len <= kLocalMax && n > (5ull << 23) && n <= (3ull << 25);
    if (!vector_stores) return seg_len > (1ull << 18) || (seg_len > 32768 && n <= (5ull << 23));
    if (f16 && seg_len > kLocalMax) return seg_len > (1ull << 18) && n > (5ull << 23);
    if (f16) return seg_len > 2048 && n > (seg_len > 4096 ? 3ull << 23 : 15ull << 22);
    return seg_len > 32768 || (seg_len > 4096 && seg_len <= kLocalMax && n > (seg_len > 6144 ? 13ull << 21 : 13ull << 22));
}
// And the only regular ones that are chained: binary16 results by element, where the open part costs more cache bandwidth to add up again than a look-back costs
// (above: 205 us, 216 where each tile adds it up).
inline bool tiles_chained(uint64_t n, uint64_t seg_len, bool f16, bool vector_stores) {
    return f16 && !vector_stores && seg_len > 4096 && seg_len <= kLocalMax && n > (3ull << 25);
}

// Where the irregular tiles that tiles_relayed names get the sum in front of them (TileSums).  Up to 7 * 2^22 elements the order in which the relay hands carries out
// costs more than it gives unless most elements lie in a few segments: a tile that takes long -- thousands of short segments, a million empty ones -- holds up all
// behind it.  So where most tiles hold many starts the four wavefronts look sums up, and where there is one for every few tiles at most those of the tiles near by;
// only for fewer segments, which are long whatever the offsets, all goes through the relay.  us, looked up / near by / relay, n = 2^20 * 17, 20, 28:
//   binary32   16             27.9/28.4/28.3   32.8/33.0/31.7   43.1/43.6/43.9      lognormal  29.2/29.1/29.7   33.0/32.8/32.7   43.1/43.5/41.7
//              3000           28.7/28.7/30.9   33.2/33.2/33.7   41.3/41.7/43.2      20000      29.2/29.0/31.7   32.8/32.4/33.2   43.0/43.5/41.6
//              half ones, half one segment  55.0/55.6/56.9   64.8/63.0/60.5   89.0/80.1/77.6     a hundredth of 16, one  37.6/33.6/32.9   41.8/36.0/34.8   56.0/44.7/43.7
//              100000         29.3/29.4/29.9   32.5/32.7/31.8   44.2/44.3/41.3      seven      34.3/35.0/29.3   38.1/37.7/31.3   53.1/48.5/40.5
//   binary16,  16             22.0/22.5/22.7   24.8/25.2/24.8   31.5/32.0/32.6      lognormal  22.3/22.3/22.9   24.1/24.2/25.3   30.1/30.0/31.3
//   exclusive  3000           21.2/21.3/22.7   23.0/23.2/25.0   28.8/29.1/31.1      20000      22.2/22.2/23.1   24.2/24.1/25.7   30.2/30.3/32.2
//              half ones, half one segment  46.6/52.5/54.0   54.0/55.4/56.0   72.8/71.3/71.3     a hundredth of 16, one  28.0/26.0/24.9   31.1/28.8/27.7   40.3/35.5/34.8
//              100000         22.2/22.0/21.8   24.0/23.9/24.4   30.8/31.0/32.0      seven      24.7/24.8/21.9   27.0/27.3/24.3   36.0/35.0/31.4
//              1000, and 2^20 * 0.17 empty ones in a row  24.8/28.0/28.8   26.0/30.2/29.9   32.9/38.3/37.0
// (results stored by element, 18 and 24: lognormal 59.7/60.2/63.5 and 77.4/77.2/79.3, binary16 38.0/38.0/40.6 and 47.7/48.2/48.5; 100000 38.9/38.7/41.6 and
// 48.5/48.5/51.4.)
// Binary32 results beyond 2^20 * 19.5: the relay for segments of up to 32 elements and long ones, those near by in between, where the relay lost; without scratch, so that
// 8 wavefronts per SIMD run (below 2^20 * 19.5 7 are faster: lognormal of mean 756 32.5/31.6).  us, before the relay / relay / near by, lognormal of mean 35, 147, 756, 1000
// (narrow), 3000 elements each, a tenth in 64s and one segment:
//   20   33.0/34.2/32.5   33.5/34.5/33.3   33.0/32.8/32.9   33.4/34.0/32.8   33.7/33.7/33.0   44.5/33.9/33.3
//   22   36.5/37.8/36.8   36.1/37.4/36.2   35.5/36.1/34.5   35.6/37.2/35.5   35.7/36.9/35.3   48.6/37.0/38.2
//   24   40.7/41.5/39.8   39.1/40.0/39.7   39.3/39.6/39.5   38.7/39.9/38.9   39.1/39.7/38.9   54.4/40.2/41.7
//   28   44.8/45.3/44.6   42.5/43.7/42.8   43.4/42.6/43.5   41.9/43.4/42.5   42.2/43.7/-      61.2/42.0/43.5
// (means of 4096 and more: the relay up to 6 % faster at 28; of 2048 to 4096 beyond 24 both ways: lognormal 43.5/42.2/44.1.)
constexpr uint64_t kIrregularLookedUpMax = 7ull << 22;
inline TileSums irregular_sums(uint64_t n, uint64_t nseg, bool f16, bool vector_stores) {
    if (n > (!vector_stores ? 27ull << 20 : kIrregularLookedUpMax)) return kSumsRelayed;
    if (vector_stores && !f16 && n > kNearSevenMax) return nseg < n >> 5 && nseg >= n >> (n > (3ull << 23) ? 11 : 12) ? kSumsNear : kSumsRelayed;
    if (nseg >= n >> 9) return kSumsLookedUp;
    return nseg >= n >> (!vector_stores ? 20 : f16 ? 18 : 16) ? kSumsNear : kSumsRelayed;
}

// The same on a caller's buffer, which is ordinary memory where the library's own tables are uncached: everybody's looks at the relay's carries cost
// more there.  us, n = 2^20 * 48, 64, 112, the relay against adding up or looking up: binary32, 5001 elements 61/61, 82/86, 131/136; 40000 60/65, 80/86, 132/141;
// 200003 equal up to 64, 112 4 % more; 300003 and more no more; binary16, 2501 (80) 60/66; 300003 (80, 96) 8 and 6 % more.
inline bool tiles_relayed_callers(uint64_t n, uint64_t seg_len, bool f16) {
    if (f16) return seg_len > 4096 && (seg_len <= kLocalMax || seg_len > (1ull << 20) || n <= (1ull << 26));
    return seg_len > (1ull << 18) || (seg_len > kLocalMax && n <= (5ull << 23));
}
// Beyond 2^27 elements, for which such a buffer has no room for the relay's words: chained tiles for lengths whose open part is much to add up or to look up
// (2^20 * 136 / 256 elements, that / chained, binary16: 5001 elements 11 / 16 % less, 8191 16 / 21; binary32: 8191 even / 4, 2000003 2 / 6, one segment off a
// boundary 28 / 66, with binary16 results 41 / 90; 100003 and less are looked up).
inline bool tiles_chained_callers(uint64_t n, uint64_t seg_len) {
    return n > (1ull << 27) && ((seg_len > 4096 && seg_len <= kLocalMax) || seg_len > (1ull << 18));
}

template <int MODE>
inline tcr_status launch_irregular_scan(const _Float16* in, const uint64_t* offsets, void* out, uint64_t n, uint64_t nseg,
                                        uint64_t seg_len, hipStream_t s, int shape = -1, bool fill = false) {
    if (shape < 0) shape = irregular_shape(true);
    const uint64_t elems = irregular_tile_elems(true, shape);
    const uint32_t shift = alignment_shift(in);
    in -= shift;
    out = static_cast<char*>(out) - (size_t)shift * ((MODE & 2) ? 2 : 4);
    n += shift;
    const uint32_t vector_stores = aligned(out, 16) ? 1u : 0u;
    const uint64_t tiles = irregular_tiles(true, n, shape);
    const bool regular = offsets == nullptr;
    // One tile per workgroup: with carries from the relay (tiles_relayed; irregular_sums says which irregular tiles look sums up instead), else regular
    // segments of nearly any length (tiles_chained) and, up to what the chip holds at once, irregular ones.  n = 2^20 / 2^24 / 2^26, us, by ticket and look-back against this: seg_len 1001 8.2 / 27 / 85 against
    // 4.1 / 22.8 / 74; 100003 8.7 / 28 / 89 against 5.1 / 20.4 / 78; irregular, lognormal lengths 10.9 / 31.8 against 5.5 / 21.0.
    const bool alone = shape == 0 && g_variant.formulation == kMfma && (regular ? seg_len >= 2 : g_variant.irregular_scan == 0);
    bool relay = alone && tiles_relayed(n, nseg, seg_len, regular, (MODE & 2) != 0, vector_stores != 0);
    bool chained = alone && !relay && regular && tiles_chained(n, seg_len, (MODE & 2) != 0, vector_stores != 0);
    if (alone && !relay && !chained && (regular || n <= scan_held_max())) return launch_scan_once<MODE>(in, offsets, out, n, nseg, seg_len, shift, fill, kSumsWide, s);
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    // Long segments -- fewer segments than a quarter of the tiles, so most tiles hold no segment start: the
    // pipelined chain scans the tiles without a start, a second kernel the others.  (Default tile shape, 16-byte
    // aligned arrays.)
    const bool two_kernels = !regular && shape == 0 && shift == 0 && vector_stores != 0 && g_variant.formulation == kMfma &&
                             g_variant.irregular_scan != 1 && (g_variant.irregular_scan == 2 || nseg <= tiles / 4);
    if (relay) {
        // without room for the relay's two words per tile: regular segments look up or add up what is in front of a tile; others look it up where that is as fast, in
        // one word, or are chained
        const uint64_t limit = table_limit(ws, capturing), words = ceil_div(n, kRelayTile);
        TileSums sums = regular || n <= scan_held_max() ? kSumsRelayed : irregular_sums(n, nseg, (MODE & 2) != 0, vector_stores != 0);
        if (!regular && n <= kIrregularLookedUpMax && n > scan_held_max() && 2 * words > limit) sums = kSumsLookedUp;
        const bool slower = regular && n > scan_held_max() && ws->caller_owned && !tiles_relayed_callers(n, seg_len, (MODE & 2) != 0);
        const bool room = !slower && (sums == kSumsLookedUp ? words : 2 * words) <= limit;
        chained = regular && !room && tiles_chained_callers(n, seg_len);
        const bool room_once = regular && !chained && (seg_len <= kLocalMax || ceil_div(n, (uint64_t)(kTile * 4 * 8)) <= limit);
        const bool room_chained = (two_kernels ? 2 * tiles : tiles) <= limit && (regular || 2 * irregular_words(true, n, shape) <= partials_limit(ws, capturing));
        if (room || room_once || !room_chained || n <= scan_held_max())
            return launch_scan_once<MODE>(in, offsets, out, n, nseg, seg_len, shift, fill, room ? sums : kSumsWide, s);
    }
    if (chained && !table_has_room(ws, tiles, capturing)) return launch_scan_once<MODE>(in, offsets, out, n, nseg, seg_len, shift, fill, kSumsWide, s);
    if (!regular) {
        st = ensure_partials(ws, s, 2 * irregular_words(true, n, shape), capturing);
        if (st != TCR_OK) return st;
    }
    ScanWorkspace dev = {};
    // (two kernels: a second table behind the first; asked for also where one kernel does, so that the same call can be recorded
    // with other offsets)
    const bool second_table = two_kernels || (!regular && !ws->caller_owned && !capturing);
    st = begin_lookback(ws, s, second_table ? 2 * tiles : tiles, &dev, capturing);
    if (st != TCR_OK) return st;
    uint64_t* starts = reinterpret_cast<uint64_t*>(ws->partials);
    TileLink* links = reinterpret_cast<TileLink*>(starts + (tiles + 1));
    if (!regular) {
        // (with `fill` it also clears what lies outside the segments: a launch of its own for that took 3 us of every call)
        const uint64_t searching = ceil_div(tiles + 1, kBoundsWaves * kBoundsPerWave), units = (uint64_t)compute_units();
        const FillOutside outside = {fill ? out : nullptr, n, (MODE >> 1) ? 2u : 4u, (uint32_t)searching};
        irregular_bounds_kernel<<<dim3((unsigned)(searching + (fill ? units : 0))), dim3(kBoundsWaves * kWave), 0, s>>>(
            offsets, nseg + 1, elems, tiles + 1, shift, starts, nullptr, two_kernels ? links : nullptr, outside);
        st = check_launch("irregular_bounds_kernel");
        if (st != TCR_OK) return st;
    }
    if (two_kernels) {
        const uint64_t resident = (uint64_t)compute_units();
        const uint64_t groups = tiles < resident ? tiles : resident;
        scan_chain_kernel<kMfma, 4, 16, MODE, true><<<dim3((unsigned)groups), dim3(16 * kWave), 0, s>>>(
            in, out, ChainGrid{n, (uint32_t)tiles, (uint32_t)tiles, 0}, dev, links);
        st = check_launch("scan_chain_kernel");
        if (st != TCR_OK) {
            ws->dirty = true;
            return st;
        }
        ws->tickets_issued += (uint32_t)(tiles + 3 * groups);
        // (every workgroup of the second kernel looks at up to 64 tiles)
        const uint64_t second = ceil_div(tiles, kWave) > resident ? ceil_div(tiles, kWave) : (tiles < resident ? tiles : resident);
        irregular_scan_kernel<4, 16, false, MODE, true><<<dim3((unsigned)second), dim3(16 * kWave), 0, s>>>(
            in, offsets, out, n, nseg, starts, 0, shift, vector_stores, dev, links);
        return check_launch("irregular_scan_kernel");
    }
    if (shape == 1) launch_irregular_scan_shape<MODE, 2, 16>(regular, in, offsets, out, n, nseg, starts, seg_len, shift, vector_stores, dev, tiles, s);
    else launch_irregular_scan_shape<MODE, 4, 16>(regular, in, offsets, out, n, nseg, starts, seg_len, shift, vector_stores, dev, tiles, s);
    st = check_launch("irregular_scan_kernel");
    if (st != TCR_OK) {
        ws->dirty = true;
        return st;
    }
    ws->tickets_issued += (uint32_t)tiles;
    return TCR_OK;
}

struct IrregularReduce {
    const _Float16* in;
    const uint64_t* offsets;      // nullptr: regular segments of seg_len elements (no look-up tables)
    float* out;
    float* out2;
    uint64_t n;
    const uint64_t* starts;
    const uint64_t* ends;
    uint64_t seg_len, nseg;
    uint32_t shift;
    TilePair* pairs;
    uint64_t* carried;
    uint64_t tiles;
    int kind;                     // kSum, kSquares (regular segments only), or kBoth with the sums of squares in out2
};
template <int U, int W, bool LINKED, bool REGULAR, int KIND>
inline void launch_irregular_reduce_kernel(const IrregularReduce& a, const ReduceLink& link, hipStream_t s) {
    irregular_reduce_kernel<U, W, REGULAR, KIND, LINKED><<<dim3((unsigned)a.tiles), dim3(W * kWave), 0, s>>>(
        a.in, a.offsets, a.out, a.out2, a.n, a.starts, a.ends, a.seg_len, a.nseg, a.shift, a.pairs, a.carried, link);
}
template <int U, int W, bool LINKED>
inline tcr_status launch_irregular_reduce_shape(const IrregularReduce& a, const ReduceLink& link, hipStream_t s) {
    if (a.offsets == nullptr) {
        if (a.kind == kBoth) launch_irregular_reduce_kernel<U, W, LINKED, true, kBoth>(a, link, s);
        else if (a.kind == kSquares) launch_irregular_reduce_kernel<U, W, LINKED, true, kSquares>(a, link, s);
        else launch_irregular_reduce_kernel<U, W, LINKED, true, kSum>(a, link, s);
    } else {
        if (a.kind == kBoth) launch_irregular_reduce_kernel<U, W, LINKED, false, kBoth>(a, link, s);
        else launch_irregular_reduce_kernel<U, W, LINKED, false, kSum>(a, link, s);
    }
    return check_launch("irregular_reduce_kernel");
}

// Irregular reductions by workgroups that walk ranges of tiles (tcr_segments.hpp).
// Tiles per workgroup: one while that makes no more than five workgroups per compute unit, two up to ten tiles per unit, then what makes
// four workgroups per unit, up to 11 tiles; four in larger arrays, and no more than 2^15 workgroups.  us, segments of 16 on average, one / two
// tiles: 2^20 * 7 / 8 / 9 / 12 elements 8.1 / 8.8, 9.1 / 8.8, 9.3 / 8.9, 12.4 / 9.8; two / three, 14 10.9 / 11.7, 16 12.3 / 12.0; 48 by 7 / 8 29.3 /
// 28.0; 64 by 4 / 6 / 8 / 9 / 11 / 14 37.3 / 40.5 / 37.9 / 36.5 / 36.4 / 40.6; 128 by 4 / 6 / 8 / 11 66.4 / 67.0 / 67.0 / 72.6.
// Segments of fewer than 8 elements keep their tile busy for so long that workgroups without any wait for the others: one tile up to
// seven workgroups per unit, sums no more than four.  Half the array in segments of one element and half in one segment, 2^20 * 8 / 32 / 64
// elements, by one / two / four / eleven tiles 27.1 / 39.1, - / 65.1 / 82.5, - / 115 / 126 / 194.
inline uint64_t segments_tiles(uint64_t n, uint64_t mean, int kind) {
    const uint64_t tiles = ceil_div(n, kSegmentsTile), units = (uint64_t)compute_units();
    if (tiles <= (mean < 8 ? 7 : 5) * units) return 1;
    const uint64_t most = ceil_div(tiles, 1ull << 15), even = tiles <= 10 * units ? 2 : ceil_div(tiles, 4 * units);
    return even <= (mean < 8 && kind == kSum ? 4 : 11) ? even : (most > 4 ? most : 4);
}
// Where that is the faster form, by the mean length of a segment: us, tiles of their own (one launch up to 2^24 or 2^25 elements, on
// workgroups of eight wavefronts up to 2^23; three beyond) against ranges:
//   sums      n = 2^20 *  5          8          9          12         16         24         32         64         96         128
//     2                 19.6/18.3  25.3/23.3  33.0/23.1  38.3/30.0  46.3/40.8  67.9/52.3  81.5/64.8  164/124    233/178    302/235
//     4                 11.5/12.8  15.0/16.5  20.1/17.1  23.9/20.7  29.8/26.6  43.9/33.6  52.6/41.6  85.3/69.1  128/106    174/143
//     8                 8.9/8.7    10.7/11.7  13.2/12.4  15.7/14.1  19.8/18.0  29.2/22.6  36.0/29.4  53.9/48.1  72.6/66.3  89.4/84.2
//     12                8.0/8.7    -          11.3/11.6  -          15.8/17.0  (faster from 2^24 on)
//     16                7.8/7.3    9.5/8.8    11.1/8.9   12.4/9.8   14.8/12.0  22.7/16.3  28.3/21.2  43.5/36.6  57.9/51.5  72.3/66.2
//     32                7.4/7.1    8.7/8.6    10.4/8.6   11.5/9.3   13.8/11.3  19.7/13.9  25.2/18.9  39.3/34.6  53.0/49.9  66.3/64.3
//     64                7.1/7.6    8.5/9.6    9.7/9.7    10.9/10.4  12.8/12.9  18.8/15.6  23.6/20.7  37.0/36.0  49.5/51.0  62.1/65.3
//     256               7.0/7.2    8.1/8.8    9.4/8.8    10.7/9.4   12.5/11.6  17.6/14.0  22.0/18.4  33.6/30.1  45.5/44.8  57.9/58.1
//     1024              6.8/7.4    7.6/9.2    8.5/9.2    9.7/9.9    11.2/12.4  16.4/15.0  20.1/19.5  30.1/31.7  40.3/42.7  50.8/54.4
//     16384             6.8/7.5    7.3/8.3    7.4/8.4    8.4/9.3    9.6/10.9   13.8/12.8  16.8/16.2  27.1/25.9  37.4/38.3  46.4/48.9
//     262144            6.7/6.5    6.8/7.4    6.8/7.2    8.2/7.8    8.8/9.1    11.9/11.0  14.8/14.0  26.4/24.1  36.0/33.8  45.8/43.4
//     lognormal (1892)  6.8/7.3    7.8/9.5    8.3/9.5    9.3/10.2   10.8/12.6  15.9/15.7  18.8/19.6  28.3/31.6  37.9/41.9  47.3/53.1
//   both moments
//     2                 22.6/21.1  28.0/26.4  35.8/26.2  51.2/34.1  60.9/47.0  84.3/60.5  107/86.6   231/160    340/224    450/291
//     4                 14.0/15.0  18.2/19.1  23.8/19.5  32.8/23.6  39.3/30.8  54.4/38.7  66.2/53.6  115/90.9   196/130    257/174
//     8                 10.4/9.8   12.9/13.3  16.3/14.1  22.5/16.1  27.1/21.1  37.9/26.0  44.3/34.3  70.5/56.0  97.2/77.3  125/99.8
//     16                9.0/7.9    10.9/9.6   13.0/9.8   17.9/11.0  21.3/14.0  30.7/18.2  36.9/24.3  57.5/40.3  78.6/56.6  99.0/73.1
//     64                8.1/8.3    9.9/10.7   11.5/10.8  14.7/11.8  18.3/15.1  25.5/18.6  30.3/24.9  51.0/42.0  70.5/58.4  89.0/74.7
//     256               8.2/7.9    9.5/9.3    11.2/9.3   14.2/10.2  17.7/12.7  24.9/15.4  29.3/20.3  47.5/33.7  66.2/49.9  85.6/64.2
//     1024              8.3/7.9    9.0/9.6    9.9/9.7    13.2/10.7  15.7/13.2  22.1/16.4  25.7/21.4  40.8/35.0  55.9/47.9  71.3/61.3
//     16384             8.2/8.2    8.8/9.2    9.1/9.4    11.0/10.3  13.4/12.3  18.1/14.3  20.8/18.5  31.5/27.9  42.8/42.7  54.1/54.3
//     262144            7.9/7.8    8.2/8.2    8.2/8.1    9.4/8.8    11.6/10.5  16.0/12.3  18.4/16.0  27.7/25.6  39.0/37.1  46.9/46.3
//     lognormal (1892)  8.1/8.4    9.4/10.1   10.1/10.4  12.6/11.3  15.1/13.8  20.1/16.6  23.2/21.6  35.7/34.1  48.4/46.0  61.0/58.4
// With segments of a thousand elements a tile has a handful of ends, and each is a chain of its own; below 14 (512 entries a tile) it
// takes more than one batch of entries.  2^20 segments of 16 at the end of an array that one segment fills (a mean of 32 up to 2^23
// elements): sums at 2^20 * 5 / 8 elements 6.9 / 8.0 against 7.9 / 9.3, both moments at 7 9.0 against 9.6.
inline bool segments_better(uint64_t n, uint64_t nseg, int kind) {
    const uint64_t mean = n / nseg;
    const auto from = [mean](uint64_t lo, uint64_t hi) { return mean >= lo && mean < hi; };
    if (n <= (1ull << 22)) return false;
    if (n <= (1ull << 23)) {
        if (from(14, 28)) return true;
        if (segments_tiles(n, mean, kind) != 1) return false;
        return from(8, 10) || (kind == kBoth && (from(0, 3) || from(96, 1500) || mean >= (1ull << 17)));
    }
    if (kind == kBoth) return n > (21ull << 19) || mean < 512 || mean >= (1ull << 17);
    if (mean >= (1ull << 15)) return n > (mean >= (1ull << 17) ? 1ull << 24 : 5ull << 22);
    if (mean >= 384) return n > (5ull << 22) && n <= (3ull << 23);
    if (mean >= 192) return n <= (3ull << 25);
    if (mean >= 64) return n > (21ull << 19) && n <= (5ull << 24);
    return n > (from(10, 14) ? 1ull << 24 : 1ull << 23) && n <= (1ull << 27);
}
inline tcr_status launch_irregular_reduce(const _Float16* in, const uint64_t* offsets, float* out, uint64_t n, uint64_t nseg,
                                          uint64_t seg_len, hipStream_t s, int kind = kSum, float* out2 = nullptr, int shape = -1) {
    const bool untuned = shape < 0 && tuned_id(kTuneIrregular, 0) < 0;
    if (shape < 0) shape = irregular_shape(false);
    const uint64_t elems = irregular_tile_elems(false, shape);
    const uint32_t shift = alignment_shift(in);
    in -= shift;
    n += shift;
    const uint64_t tiles = irregular_tiles(false, n, shape);
    const unsigned ch = kind == kBoth ? 2u : 1u;
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    // (also where the call does without them: the same call can then be recorded into a graph)
    const uint64_t words = irregular_words(false, n, shape, ch), groups = irregular_groups(tiles);
    const bool far = irregular_far(tiles, nseg) && 2 * (words + ch * groups) <= partials_limit(ws, capturing);
    st = ensure_partials(ws, s, 2 * (words + (far ? ch * groups : 0)), capturing);
    if (st != TCR_OK) return st;
    if (offsets != nullptr && shape == 0 && segments_better(n, nseg, kind)) {
        const uint64_t group_tiles = segments_tiles(n, n / nseg, kind), wgs = ceil_div(n, group_tiles * kSegmentsTile);
        if (table_has_room(ws, ch * wgs, capturing)) {
            ScanWorkspace dev = {};
            st = begin_lookback(ws, s, ch * wgs, &dev, capturing);
            if (st != TCR_OK) return st;
            const SegmentsReduce a = {in, offsets, out, out2, n, nseg, shift, (double)(nseg + 1) / (double)n, search_grid_log2(nseg),
                                      (uint32_t)group_tiles, g_variant.scan_wait ? kOncePatience : 0u};
            const dim3 grid((unsigned)wgs), block(4 * kWave);
            if (kind == kBoth) segments_reduce_kernel<kBoth><<<grid, block, 0, s>>>(a, dev);
            else segments_reduce_kernel<kSum><<<grid, block, 0, s>>>(a, dev);
            st = check_launch("segments_reduce_kernel");
            if (st != TCR_OK) ws->dirty = true;
            return st;
        }
    }
    // One launch, whose tiles search the offsets and add what reaches them from in front themselves, out of one descriptor
    // per tile and channel; against a look-up kernel in front and a finishing kernel behind, us, segments of 16 elements /
    // lognormal lengths / seven segments: n = 2^20 8.0 / 6.2 / 5.5 -> 5.6 / 5.3 / 5.3, 2^22 10.6 / 9.0 / 8.6 -> 7.4 / 6.2 / 6.2, 2^24
    // 19.0 / 13.1 / 12.9 -> 17.3 / 11.8 / 10.4, 2^25 29.8 / 20.1 / 19.0 -> 29.3 / 19.6 / 16.1, both moments at 2^24 25.5 / 17.5 / 14.0
    // -> 22.9 / 16.0 / 12.3.  Beyond, the searches are what the tiles wait for (2^26 43.6 / 29.8 / 28.2 -> 52.0 / 34.2 / 25.4) and
    // for both moments and regular segments the sums of thousands of tiles behind one result (one segment of 2^26 elements:
    // 25.9 -> 31.0).  Not where the descriptors cannot be had.
    const bool linked = table_has_room(ws, ch * tiles, capturing) && shape != 1 && tiles <= (offsets != nullptr && kind == kSum ? 4096u : 2048u);
    // (up to four tiles per compute unit twice the wavefronts per tile: segments of 16 elements, n = 2^20 / 2^22 / 2^23 / 2^24
    // 7.1 / 8.6 / 12.0 / 17.3 us with 4 wavefronts, 5.6 / 7.4 / 11.2 / 19.3 with 8)
    if (linked && untuned && tiles <= 4 * (uint64_t)compute_units()) shape = 2;
    ReduceLink link = {};
    if (linked) {
        st = begin_lookback(ws, s, ch * tiles, &link.ws, capturing);
        if (st != TCR_OK) return st;
        link.patience = g_variant.scan_wait ? kOncePatience : 0u;
        const IrregularReduce a = {in, offsets, out, out2, n, nullptr, nullptr, seg_len, nseg, shift, nullptr, nullptr, tiles, kind};
        st = shape == 2 ? launch_irregular_reduce_shape<2, 8, true>(a, link, s) : launch_irregular_reduce_shape<4, 4, true>(a, link, s);
        if (st != TCR_OK) ws->dirty = true;
        return st;
    }
    uint64_t* starts = reinterpret_cast<uint64_t*>(ws->partials);
    uint64_t* ends = starts + (tiles + 1);
    uint64_t* carried = ends + (tiles + 1);
    TilePair* pairs = reinterpret_cast<TilePair*>(carried + tiles);              // ch * tiles
    const IrregularReduce a = {in, offsets, out, out2, n, starts, ends, seg_len, nseg, shift, pairs, carried, tiles, kind};
    if (offsets != nullptr) {
        irregular_bounds_kernel<<<dim3((unsigned)ceil_div(tiles + 1, kBoundsWaves * kBoundsPerWave)), dim3(kBoundsWaves * kWave), 0, s>>>(
            offsets, nseg + 1, elems, tiles + 1, shift, starts, ends);
        st = check_launch("irregular_bounds_kernel");
        if (st != TCR_OK) return st;
    }
    st = shape == 1 ? launch_irregular_reduce_shape<4, 8, false>(a, link, s)
                    : (shape == 2 ? launch_irregular_reduce_shape<2, 8, false>(a, link, s) : launch_irregular_reduce_shape<4, 4, false>(a, link, s));
    if (st != TCR_OK || tiles == 1) return st;          // a single tile has nothing in front of it
    if (far) {
        TilePair* group_pairs = pairs + ch * tiles;
        const dim3 grid((unsigned)ceil_div(groups, kCarryWaves), ch);
        irregular_groups_kernel<<<grid, dim3(kCarryWaves * kWave), 0, s>>>(pairs, tiles, group_pairs);
        st = check_launch("irregular_groups_kernel");
        if (st != TCR_OK) return st;
        irregular_carry_kernel<<<grid, dim3(kCarryWaves * kWave), 0, s>>>(pairs, group_pairs, carried, tiles, out, out2);
        return check_launch("irregular_carry_kernel");
    }
    irregular_finish_kernel<kFinishThreads, kFinishFar><<<dim3((unsigned)ceil_div(tiles, kFinishThreads), ch), dim3(kFinishThreads), 0, s>>>(
        pairs, carried, tiles, out, out2);
    return check_launch("irregular_finish_kernel");
}

// Regular segments from 17 elements on, no power of two: whole segments per workgroup, masked row products
// (tcr_rows.hpp).  `in` needs only 2-byte alignment.  kind: kSum, or kBoth with the sums of squares in out2.
// Measured at n = 2^28 against the kernels that took these lengths before: sums 77-98 us from 33 to 8000
// elements (fixed tiles with marked starts: 114-157 us below 1000; one wavefront per segment over masked tiles:
// 114 us at 1000, 89 at 2000, 80 from 3000 on); both moments 88-108 us (fixed tiles 184-249 us; masked tiles 119 us
// at 1000, 93 at 2000, 82 from 3000 on, where they stay).  From 17 to 31 elements (two boundaries per row): sums
// 102-110 us (fixed tiles 117-150 us), both moments 140-170 us (177-217 us).
// (Below 17 -- two or three whole segments per row -- it only equals the fixed tiles at 11-15 elements, 123-130 us
// either way, and loses to them at 9 and 10, 170 against 144-168 us.)
constexpr uint64_t kRowsReduceMin = 17, kRowsMomentsMin = 17, kRowsReduceMax = kRowsMaxSegLen, kRowsMomentsMax = 2999;
inline bool rows_reduce_takes(uint64_t seg_len, int kind = kSum) {
    return g_variant.rows_reduce && seg_len >= (kind == kBoth ? kRowsMomentsMin : kRowsReduceMin) &&
           seg_len <= (kind == kBoth ? kRowsMomentsMax : kRowsReduceMax);
}
// A workgroup's share: 16320 elements by eight wavefronts, or, in arrays that do not give every compute unit several such workgroups, 8128 by
// eight (1) or 4032 by four (2); in all of them whole segments.  us, the first against these, n in 2^20:
//   both moments, 8128   25: 4 6.3/5.0, 16 12.7/11.8, 64 37.3/36.6, 128 68.9/68.8, 256 131.7/133.9; 33: 4 5.1/4.3, 16 9.6/9.1, 24 12.6/12.4, 32 15.9/16.1;
//                        100: 1 3.9/3.5, 6 5.4/5.0, 20 10.7/10.4, 24 12.0/11.9, 32 14.8/15.0; 784: 2 3.9/3.6, 4 5.1/4.2, 6 5.4/4.9, 8 6.5/5.8,
//                        20 10.3/10.1, 32 14.2/14.5; 1999: 8 6.3/5.9, 20 10.0/10.0; 2500: 8 6.4/5.9, 16 8.8/8.6, 20 10.0/10.1;
//                        2999 (two segments): 8 6.4/6.4, 12 7.5/8.4
//   sums, 4032           17: 1 3.7/3.6, 4 4.9/4.0, 8 6.5/5.7, 12 7.9/7.3, 14 8.3/8.2; 100: 2 3.6/3.8, 4 4.1/3.9, 8 5.2/5.0, 10 5.6/5.6, 12 6.4/6.2,
//                        14 6.9/6.6; 784: 4 4.1/3.9, 12 6.5/6.1, 14 6.6/6.9; 2000: 4 4.0/3.9, 8 5.2/4.7, 12 6.3/6.0; 2500 (one): 6 4.3/5.0
// (inputs read from memory; from the memory-side cache the gains up to 2^20 * 6 are hidden behind the call.)  How many segments a smaller share holds matters: 1355
// elements fill 83 % of 8128 and all of 16320, 2035 75 %.  moments  1200 (89 %): 8 6 % less, 14 3 % more, 18 4 to 8 % more; 1355: 8 6 % less, 11 3 to 7 % more;
// 1640 (81 %): 8 8 % less, 10 3 % more, 13 6 to 8 % more; 2035: 5 9 % less, 6 4 % more, 11 14 to 18 % more; 1500, 2500 (92 %): 12 7 % less, 14 3 to 6 % more; 1999
// (98 %): 16 4 % less, 18 1 to 6 % more.  sums  784: 8 5 to 8 % less, 10 and 11 5 % more, 12 4 % less; 1355 (67 %): 8 even, 12 6 to 9 % more; 1700 (84 %): 12 6 % less.
inline int rows_shape(uint64_t n, uint64_t seg_len, int kind) {
    if (kind == kBoth) {
        if (seg_len > 2709) return 0;
        const uint64_t filled = 8128 / seg_len * seg_len;
        if (seg_len < 32) return n <= (1ull << 26) ? 1 : 0;
        if (filled > 7720) return n <= (seg_len <= 1625 ? 5ull << 22 : 1ull << 24) ? 1 : 0;
        return n <= (filled > 7315 ? 13ull << 20 : filled > 6340 ? 1ull << 23 : 5ull << 20) ? 1 : 0;
    }
    if (seg_len > 2016) return 0;
    if (seg_len < 32) return n <= (7ull << 21) ? 2 : 0;
    return n > (3ull << 20) && (n <= (9ull << 20) || (n > (23ull << 19) && n <= (13ull << 20) && 4032 / seg_len * seg_len > 3350)) ? 2 : 0;
}
template <int U, int W>
inline void launch_rows_shape(const _Float16* in, float* out, float* out2, RowsGrid grid, int kind, hipStream_t s) {
    grid.per_group = (uint32_t)((U * W * kTile - 64) / grid.seg_len);
    const dim3 blocks((unsigned)ceil_div(grid.nseg, grid.per_group)), block(W * kWave);
    if (grid.seg_len < 32) {             // 17 .. 31: two boundaries per row and a whole segment between them
        if (kind == kBoth) rows_reduce_kernel<kBoth, U, W, 1><<<blocks, block, 0, s>>>(in, out, out2, grid);
        else rows_reduce_kernel<kSum, U, W, 1><<<blocks, block, 0, s>>>(in, out, nullptr, grid);
    } else {
        if (kind == kBoth) rows_reduce_kernel<kBoth, U, W><<<blocks, block, 0, s>>>(in, out, out2, grid);
        else rows_reduce_kernel<kSum, U, W><<<blocks, block, 0, s>>>(in, out, nullptr, grid);
    }
}
inline tcr_status launch_rows_reduce(const _Float16* in, float* out, float* out2, uint64_t n, uint64_t seg_len, int kind,
                                     hipStream_t s) {
    const uint32_t shift = alignment_shift(in);
    RowsGrid grid;
    grid.seg_len = seg_len;
    grid.nseg = n / seg_len;
    grid.n = n + shift;
    grid.shift = shift;
    grid.magic = (uint32_t)(((1ull << 32) + seg_len - 1) / seg_len);
    switch (rows_shape(n, seg_len, kind)) {
        case 1: launch_rows_shape<2, 8>(in - shift, out, out2, grid, kind, s); break;
        case 2: launch_rows_shape<2, 4>(in - shift, out, out2, grid, kind, s); break;
        default: launch_rows_shape<4, 8>(in - shift, out, out2, grid, kind, s); break;
    }
    return check_launch("rows_reduce_kernel");
}

// Regular segments of 3 to 30 elements that pack into rows of an even number of at most 32 elements (every even
// length that is no power of two, odd lengths up to 15): one product per 16 rows with a masked constant matrix
// (tcr_packed.hpp).  `in` 4-byte aligned.  kind: kSum, or kBoth with the sums of squares in out2.
// Measured at n = 2^28 against the kernels that took these lengths before -- sums: 3 elements 162 us (one thread per
// segment: 274), 5 to 7 107-116 (fixed tiles with marked starts 162-183), 9 to 15 98-104 (125-148), even lengths
// from 18 to 30 91-99 (masked rows of the array 102-106); both moments: 3 elements 310 (one thread per segment
// 320-345), 5 to 7 153-190 (213-250), 9 to 15 110-134 (180-216), 18 to 30 100-110 (140-170).
// Two launch shapes: eight tiles per wavefront where a row's width is no multiple of 8 (rows of 18 elements: 99
// against 113 us; 22: 97 against 105; 26 to 30: 94-96 against 97-99), four where it is (24: 90 against 96 us); twelve
// or sixteen tiles, or two or eight wavefronts, change nothing.  (U, W) = (8, 4) and (4, 4).
// (4 and 8 elements as well: sums 117 and 102 us against 125 and 110 for the kernel with whole segments inside a
// lane's eight elements, both moments 208 and 128 against 272 and 219 with one thread per segment; 2 elements: 178
// against 167 us, and 16 rows of P for the squares -- left where they are)
inline bool packed_reduce_takes(uint64_t seg_len) {
    return g_variant.rows_reduce && packed_per_row(seg_len) != 0 && (!is_pow2(seg_len) || seg_len == 4 || seg_len == 8);
}
template <int KIND, int U, int W>
inline void launch_packed_shape(const _Float16* in, float* out, float* out2, const PackedGrid& grid, hipStream_t s) {
    const uint64_t rows = ceil_div(grid.nseg, (uint64_t)grid.per_row);
    const size_t staging = (size_t)W * channels<KIND>() * 16 * U * grid.per_row * sizeof(float);      // at most 40 KiB
    packed_rows_reduce_kernel<KIND, U, W><<<dim3((unsigned)ceil_div(rows, (uint64_t)(16 * U * W))), dim3(W * kWave), staging, s>>>(in, out, out2, grid);
}
// Fewer tiles per wavefront in smaller arrays, where rows of no multiple of 8 elements take eight: a wavefront's tiles follow each other, and for the
// squares each is a product per segment of the row.  us, eight against fewer, n in 2^20:
//   both moments   one    3: 1/16 11.5/4.2, 1 12.0/5.7; 7: 1/16 6.6/3.5, 1 6.7/3.7, 2 7.0/5.0 (two 4.9)
//                  two    3: 3 12.7/8.8; 7: 2 7.0/4.9, 4 8.6/6.2; 15: 4 6.4/4.9; 22: 4 5.4/4.6
//                  four   3: 5 15.6/11.9, 12 21.8/20.0, 64 82.1/72.0, 128 145/133; 5: 8 14.3/12.4, 24 25.2/23.4, 32 30.4/29.6, 64 48.2/49.1; 7: 8 10.8/9.6,
//                         12 14.2/12.9, 24 19.8/20.5; 9: 8 9.0/8.6, 12 12.0/12.1, 16 14.3/14.6; 15: 12 10.0/9.3; 22: 12 9.1/8.6, 16 9.8/10.8
//   sums           two    3: 3 4.4/3.8; 7: 1 3.8/3.4, 4 4.7/3.7; 15: 4 4.6/3.7; 22: 3 4.3/3.8
//                  four   3: 6 6.2/5.5, 12 9.8/9.1, 16 11.4/12.2; 7: 8 6.0/5.3, 12 7.6/7.0; 15: 10 6.0/5.7; 22: 8 5.3/5.0, 12 6.8/7.2
// Narrow rows fill less of a tile: rows of 18 (9 elements): moments 10 and 11 2 to 7 % more, sums 4 % more; of 20: moments 11 to 13 2 to 9 % more, sums 11 7 % more;
// of 22: moments 12 2 %; 30: none up to 12.
inline int packed_tiles(uint64_t n, uint32_t width, uint32_t per_row, int kind) {
    if (kind == kBoth && n <= (5ull << 18)) return 1;
    if (n <= (9ull << 19)) return 2;
    const uint64_t few = (uint64_t)width << 19;
    if (kind == kBoth) return (n <= few && n <= (3ull << 22)) || per_row >= 10 || (per_row >= 6 && n <= (1ull << 25)) ? 4 : 8;
    return n <= few && n <= (11ull << 20) ? 4 : 8;
}
// Both moments of 4 and 8 elements: whole segments inside a lane's eight.  us, packed rows against this, n in 2^20: 4 elements 1/16 5.8/3.7, 4 8.0/3.8,
// 8 12.5/7.3, 16 18.0/13.2, 64 51.1/42.9, 256 192/167 (two groups of eight per lane: 64 40.7 against 41.7 with one, 256 185 against 171); 8 elements 1
// 4.4/3.9, 8 8.0/5.1, 16 12.8/10.4, 64 36/34.6, 256 138/131 (one group: 8 5.1 against 4.7, 256 132 against 130).
inline tcr_status launch_tiny_moments(const _Float16* in, float* sum, float* sumsq, uint64_t n, uint64_t seg_len, hipStream_t s) {
    if (seg_len == 4) tiny_moments_kernel<2, 1><<<dim3((unsigned)ceil_div(n, 8 * kGenericThreads)), dim3(kGenericThreads), 0, s>>>(in, sum, sumsq, n);
    else tiny_moments_kernel<3, 2><<<dim3((unsigned)ceil_div(n, 16 * kGenericThreads)), dim3(kGenericThreads), 0, s>>>(in, sum, sumsq, n);
    return check_launch("tiny_moments_kernel");
}
// Tiles per wavefront.  alt (a choice of the tuning table, whose meaning does not go by n): eight for rows of a multiple of 8 elements, which take four, four for
// others.
inline int packed_shape(uint64_t n, uint64_t seg_len, int kind, bool alt) {
    const uint32_t per_row = packed_per_row(seg_len), width = (uint32_t)seg_len * per_row;
    if ((width % 8u == 0) != alt) return 4;
    return alt ? 8 : packed_tiles(n, width, per_row, kind);
}
inline tcr_status launch_packed_reduce(const _Float16* in, float* out, float* out2, uint64_t n, uint64_t seg_len, int kind,
                                       hipStream_t s, bool alt = false) {
    const PackedGrid grid = {n, n / seg_len, (uint32_t)seg_len, packed_per_row(seg_len)};
    const int tiles = packed_shape(n, seg_len, kind, alt);
    if (kind == kBoth) {
        if (tiles == 1) launch_packed_shape<kBoth, 1, 4>(in, out, out2, grid, s);
        else if (tiles == 2) launch_packed_shape<kBoth, 2, 4>(in, out, out2, grid, s);
        else if (tiles == 4) launch_packed_shape<kBoth, 4, 4>(in, out, out2, grid, s);
        else launch_packed_shape<kBoth, 8, 4>(in, out, out2, grid, s);
    } else {
        if (tiles == 2) launch_packed_shape<kSum, 2, 4>(in, out, nullptr, grid, s);
        else if (tiles == 4) launch_packed_shape<kSum, 4, 4>(in, out, nullptr, grid, s);
        else launch_packed_shape<kSum, 8, 4>(in, out, nullptr, grid, s);
    }
    return check_launch("packed_rows_reduce_kernel");
}

// Any other seg_len >= 1 (no power of two, or below 16): no kernel is tuned for it.
// Scans from 2 elements on and reductions of 8 to 999 elements run on the fixed tiles of the irregular
// kernels with the multiples of seg_len as segment starts.  Measured at n = 2^28: scans 300-325 us
// whatever the length (one thread or one wavefront per segment took 440-5600 us below 256 elements,
// 350-400 us above, and 13 ms for 15 segments of 2^24 + 1 elements); reductions 146-231 us (against
// 230-1060 us).  Longer reductions keep one wavefront per segment over zero-masked tiles (116 us at
// 1000 elements, 85 us at 3001), the shortest segments one thread each.
constexpr uint64_t kTiledScanMin = 2;
// (sums from 5 elements on: 161-183 us at 5..7 against 193-210 us with one thread per segment, 274 either way at 3;
// both moments from 8 on: below, one thread per segment is faster, 213-232 against 231-259 us)
constexpr uint64_t kTiledReduceMin = 5, kTiledMomentsMin = 8, kTiledReduceMax = 1000;

// Which kernel takes a reduction whose seg_len is no power of two (or below 16); class = floor(log2(seg_len)).
// The default is the first valid one of: rows, tiles, the rest (one wavefront per segment over masked tiles from
// 1000 elements, one thread per segment below 5).
enum ReduceAny { kReduceAnyRows = 0, kReduceAnyTiles = 1, kReduceAnyTilesAlt = 2, kReduceAnyMasked = 3, kReduceAnyPacked = 4, kReduceAnyPackedAlt = 5, kReduceAnyCount = 6 };
constexpr uint64_t kMaskedReduceMin = 256;              // (valid for any length; pointless for short segments)
inline bool reduce_any_valid(int id, uint64_t seg_len) {
    switch (id) {
        case kReduceAnyRows: return rows_reduce_takes(seg_len);
        case kReduceAnyTiles:
        case kReduceAnyTilesAlt: return seg_len >= kTiledReduceMin && seg_len < kTiledReduceMax;
        case kReduceAnyMasked: return seg_len >= kMaskedReduceMin;
        case kReduceAnyPacked:
        case kReduceAnyPackedAlt: return packed_reduce_takes(seg_len);
        default: return false;
    }
}
// packed_ok: the array is 4-byte aligned (the packed rows need that; kernel names are given for aligned arrays)
inline int pick_reduce_any(uint64_t seg_len, bool packed_ok = true) {
    const int tuned = tuned_id(kTuneReduceAny, floor_log2(seg_len));
    if (reduce_any_valid(tuned, seg_len) && ((tuned != kReduceAnyPacked && tuned != kReduceAnyPackedAlt) || packed_ok)) return tuned;
    if (packed_ok && reduce_any_valid(kReduceAnyPacked, seg_len)) return kReduceAnyPacked;
    if (reduce_any_valid(kReduceAnyRows, seg_len)) return kReduceAnyRows;
    if (reduce_any_valid(kReduceAnyTiles, seg_len)) return kReduceAnyTiles;
    return kReduceAnyMasked;                            // (or one thread per segment, below 8 elements)
}

// Sums (kSum) or both moments (kBoth, the second in out2) over masked tiles of the array.
// Wavefronts per segment: one where that fills the chip or the segment is one step of a wavefront, else 4 or 16 (W
// wavefronts of a workgroup take 4096 elements each per step).  Longer segments than one workgroup should walk are cut
// into pieces of four wavefronts' free shares -- of one wavefront's where the array fills the chip anyway: the
// wavefronts of a workgroup then need not wait for each other.  At n = 2^24 one wavefront per segment or per
// 65536-element piece took 22.6 us at 50001 elements, 41.5 at 100001 and 30 at 300001 and 1000001.
template <int KIND, int W>
inline void launch_masked_pieces(const _Float16* in, float* dst, float* dst2, uint64_t nseg, uint64_t seg_len, uint64_t span,
                                 uint64_t per, hipStream_t s, const ReduceFinish& fin = {}) {
    const dim3 grid((unsigned)ceil_div(nseg * per, W == 1 ? kMaskedWaves : 1)), block(masked_group_waves<W>() * kWave);
    const bool four = W == 1 && seg_len > 4096;          // a wavefront that takes several steps: shorter ones (8192 elements: 21.7 against 22.8 us)
    if constexpr (KIND == kBoth) {
        if (per > 1) masked_moments_kernel<8, W, true><<<grid, block, 0, s>>>(in, dst, dst2, nseg, seg_len, span, per, fin);
        else if (four) masked_moments_kernel<4, W, false><<<grid, block, 0, s>>>(in, dst, dst2, nseg, seg_len, span, per, fin);
        else masked_moments_kernel<8, W, false><<<grid, block, 0, s>>>(in, dst, dst2, nseg, seg_len, span, per, fin);
    } else {
        if (per > 1) masked_span_reduce_kernel<W><<<grid, block, 0, s>>>(in, dst, nseg, seg_len, span, per, fin);
        else if (four) masked_wave_reduce_kernel<4, W><<<grid, block, 0, s>>>(in, dst, nseg, seg_len);
        else masked_wave_reduce_kernel<8, W><<<grid, block, 0, s>>>(in, dst, nseg, seg_len);
    }
}
inline bool masked_finishes(uint64_t n, uint64_t seg_len, uint64_t ch) {
    return seg_len > 2 * kWaveSpanMax && n <= kFinishElemsMax && ch * (n / seg_len) <= kFinishSums;
}
template <int KIND>
inline tcr_status launch_masked(const _Float16* in, float* out, float* out2, uint64_t n, uint64_t seg_len, hipStream_t s) {
    const uint64_t nseg = n / seg_len;
    if (seg_len <= 2 * kWaveSpanMax) {
        if (seg_len <= 4096 || nseg >= (seg_len <= 8192 ? kWavesWanted / 2 : kWavesWanted)) launch_masked_pieces<KIND, 1>(in, out, out2, nseg, seg_len, seg_len, 1, s);
        else if (seg_len <= 16384 || 4 * nseg >= kWavesWanted / 2) launch_masked_pieces<KIND, 4>(in, out, out2, nseg, seg_len, seg_len, 1, s);
        else launch_masked_pieces<KIND, 16>(in, out, out2, nseg, seg_len, seg_len, 1, s);
        return check_launch("masked_wave_reduce_kernel");
    }
    // pieces, then the paper's second kernel over the pieces (for each moment)
    constexpr uint64_t ch = KIND == kBoth ? 2 : 1;
    Workspace* ws = nullptr;
    bool capturing = false;
    tcr_status st = get_workspace(s, &ws, &capturing);
    if (st != TCR_OK) return st;
    uint32_t* counter = masked_finishes(n, seg_len, ch) ? finish_counter(ws, capturing) : nullptr;
    uint64_t span = counter != nullptr ? finish_share(n) : free_span(n);
    const bool grouped = span < kWaveSpanMax;
    if (grouped && counter == nullptr) span *= 4;
    // (a workspace that cannot be grown and is too small for that: pieces of 65536 elements, as few as there need be)
    if (span < kWaveSpanMax && ch * nseg * ceil_div(seg_len, span) > partials_limit(ws, capturing)) span = kWaveSpanMax;
    uint64_t per = ceil_div(seg_len, span);
    if (span < seg_len) span = ceil_div(ceil_div(seg_len, per), 8 * (uint64_t)kTile) * (8 * (uint64_t)kTile);   // pieces of one size, in whole steps
    per = ceil_div(seg_len, span);
    const uint64_t pieces = nseg * per;
    st = ensure_partials(ws, s, ch * pieces, capturing);
    if (st != TCR_OK) return st;
    if (counter != nullptr) {
        const ReduceFinish fin = {out, KIND == kBoth ? out2 : nullptr, counter, 0u, (uint32_t)nseg, (uint32_t)per, 1u};
        if (span <= 32768) launch_masked_pieces<KIND, 4>(in, ws->partials, ws->partials + pieces, nseg, seg_len, span, per, s, fin);
        else launch_masked_pieces<KIND, 16>(in, ws->partials, ws->partials + pieces, nseg, seg_len, span, per, s, fin);
        return check_launch("masked_span_reduce_kernel");
    }
    if (grouped) launch_masked_pieces<KIND, 4>(in, ws->partials, ws->partials + pieces, nseg, seg_len, span, per, s);
    else launch_masked_pieces<KIND, 1>(in, ws->partials, ws->partials + pieces, nseg, seg_len, span, per, s);
    st = check_launch("masked_span_reduce_kernel");
    if (st != TCR_OK) return st;
    launch_reduce_final(ws->partials, out, out2, nseg, per, s);
    return check_launch("reduce_final_kernel");
}

template <bool SCAN>
inline tcr_status launch_generic(const _Float16* in, void* out, uint64_t n, uint64_t seg_len, uint32_t flags, hipStream_t s,
                                 int tiles_shape = 0) {
    const uint64_t nseg = n / seg_len;
    const bool excl = (flags & TCR_SCAN_EXCLUSIVE) != 0, f16 = (flags & TCR_OUT_F16) != 0;
    // 1, 2, 4 or 8 elements (scans: the plain binary32 inclusive one): whole segments inside a lane's 8 elements.
    // `out` is 16-byte aligned for scans; reductions need it for their 128-bit stores.
    // 4 and 8 elements: reductions on rows of whole segments unless the tuning table or the variant says otherwise
    const bool packed_first = !SCAN && (seg_len == 4 || seg_len == 8) && packed_reduce_takes(seg_len) && aligned(in, 4) &&
                              (pick_reduce_any(seg_len) == kReduceAnyPacked || pick_reduce_any(seg_len) == kReduceAnyPackedAlt);
    if (is_pow2(seg_len) && seg_len <= 8 && !packed_first && (SCAN ? flags == 0 : aligned(out, 16))) {
        const dim3 grid((unsigned)ceil_div(n, (uint64_t)kGenericThreads * 8)), block(kGenericThreads);
        float* o = static_cast<float*>(out);
        if constexpr (SCAN) {
            switch (seg_len) {
                case 1: tiny_scan_kernel<0><<<grid, block, 0, s>>>(in, o, n); break;
                case 2: tiny_scan_kernel<1><<<grid, block, 0, s>>>(in, o, n); break;
                case 4: tiny_scan_kernel<2><<<grid, block, 0, s>>>(in, o, n); break;
                default: tiny_scan_kernel<3><<<grid, block, 0, s>>>(in, o, n); break;
            }
            return check_launch("tiny_scan_kernel");
        }
        switch (seg_len) {
            case 1: tiny_reduce_kernel<0><<<grid, block, 0, s>>>(in, o, n); break;
            case 2: tiny_reduce_kernel<1><<<grid, block, 0, s>>>(in, o, n); break;
            case 4: tiny_reduce_kernel<2><<<grid, block, 0, s>>>(in, o, n); break;
            default: tiny_reduce_kernel<3><<<grid, block, 0, s>>>(in, o, n); break;
        }
        return check_launch("tiny_reduce_kernel");
    }
    if constexpr (SCAN) {
        if (seg_len >= kTiledScanMin) {
            switch (flags & 3u) {
                case 0: return launch_irregular_scan<0>(in, nullptr, out, n, nseg, seg_len, s, tiles_shape);
                case 1: return launch_irregular_scan<1>(in, nullptr, out, n, nseg, seg_len, s, tiles_shape);
                case 2: return launch_irregular_scan<2>(in, nullptr, out, n, nseg, seg_len, s, tiles_shape);
                default: return launch_irregular_scan<3>(in, nullptr, out, n, nseg, seg_len, s, tiles_shape);
            }
        }
    } else {
        const int pick = pick_reduce_any(seg_len, aligned(in, 4));
        if (pick == kReduceAnyPacked || pick == kReduceAnyPackedAlt)
            return launch_packed_reduce(in, static_cast<float*>(out), nullptr, n, seg_len, kSum, s, pick == kReduceAnyPackedAlt);
        if (pick == kReduceAnyRows) return launch_rows_reduce(in, static_cast<float*>(out), nullptr, n, seg_len, kSum, s);
        if (pick == kReduceAnyTiles || pick == kReduceAnyTilesAlt)
            return launch_irregular_reduce(in, nullptr, static_cast<float*>(out), n, nseg, seg_len, s, kSum, nullptr,
                                           pick == kReduceAnyTilesAlt ? 1 : 0);
    }
    if (SCAN || seg_len < kTiledReduceMin) {         // (also reductions of 3 elements from an array that is not 4-byte aligned)
        generic_thread_kernel<SCAN><<<dim3((unsigned)ceil_div(nseg, kGenericThreads)), dim3(kGenericThreads), 0, s>>>(
            in, out, nseg, seg_len, excl, f16);
        return check_launch("generic_thread_kernel");
    }
    // reductions from 1000 elements on: masked 512-element tiles of the array
    return launch_masked<kSum>(in, static_cast<float*>(out), nullptr, n, seg_len, s);
}

// The tuned scan paths for one (formulation, mode) pair.
template <int FORM, int MODE>
inline tcr_status scan_tuned(const _Float16* x, void* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    if (seg_len == n) return scan_long<FORM, MODE>(x, out, n, n, true, s);
    if (seg_len <= kTile) return launch_scan_small<FORM, MODE>(x, out, n, log2u(seg_len), s);
    return scan_long<FORM, MODE>(x, out, n, seg_len, false, s);
}

// First two moments of every segment, any seg_len >= 1 that divides n.
template <int LOG2L>
inline void launch_moments_small(const _Float16* in, float* sum, float* sumsq, uint64_t n, hipStream_t s) {
    const uint64_t per_group = (uint64_t)kTile * kSmallReduceU * kSmallReduceW;
    moments_small_kernel<LOG2L, kSmallReduceU, kSmallReduceW><<<dim3((unsigned)ceil_div(n, per_group)), dim3(kSmallReduceW * kWave), 0, s>>>(
        in, sum, sumsq, n);
}

inline tcr_status launch_moments(const _Float16* in, float* sum, float* sumsq, uint64_t n, uint64_t seg_len, hipStream_t s) {
    const uint64_t nseg = n / seg_len;
    if (is_pow2(seg_len) && seg_len >= 16 && seg_len <= kTile) {
        switch (log2u(seg_len)) {
            case 4: launch_moments_small<4>(in, sum, sumsq, n, s); break;
            case 5: launch_moments_small<5>(in, sum, sumsq, n, s); break;
            case 6: launch_moments_small<6>(in, sum, sumsq, n, s); break;
            case 7: launch_moments_small<7>(in, sum, sumsq, n, s); break;
            case 8: launch_moments_small<8>(in, sum, sumsq, n, s); break;
            default: launch_moments_small<9>(in, sum, sumsq, n, s); break;
        }
        return check_launch("moments_small_kernel");
    }
    if ((seg_len == 4 || seg_len == 8) && aligned(in, 16)) return launch_tiny_moments(in, sum, sumsq, n, seg_len, s);
    if (packed_reduce_takes(seg_len) && aligned(in, 4)) return launch_packed_reduce(in, sum, sumsq, n, seg_len, kBoth, s);
    if (rows_reduce_takes(seg_len, kBoth)) return launch_rows_reduce(in, sum, sumsq, n, seg_len, kBoth, s);
    if (seg_len >= kTiledMomentsMin && seg_len < kTiledReduceMax) {
        // fixed tiles with the segment starts marked, both moments as two channels of one pass
        return launch_irregular_reduce(in, nullptr, sum, n, nseg, seg_len, s, kBoth, sumsq);
    }
    if (seg_len < kTiledMomentsMin) {        // under 8 elements: one thread per segment
        generic_moments_kernel<<<dim3((unsigned)ceil_div(nseg, kGenericThreads)), dim3(kGenericThreads), 0, s>>>(
            in, sum, sumsq, nseg, seg_len);
        return check_launch("generic_moments_kernel");
    }
    return launch_masked<kBoth>(in, sum, sumsq, n, seg_len, s);
}

// Segment lengths that are no power of two, a multiple of 8, and fit one workgroup: scan_segment_kernel with the
// smallest share that holds a segment.
inline bool segment_kernel_takes(uint64_t seg_len) {
    return g_variant.formulation == kMfma && seg_len % 8 == 0 && seg_len > kTile && seg_len < 2 * scan_shape_tile(10);
}

template <int U, int W, int MODE>
void launch_scan_segment_shape(const _Float16* in, void* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    scan_segment_kernel<U, W, MODE><<<dim3((unsigned)(n / seg_len)), dim3(W * kWave), 0, s>>>(in, out, seg_len);
}

// Shares in steps of at most a third, so that few wavefronts of a workgroup lie beyond the segment's end.
template <int MODE>
tcr_status launch_scan_segment(const _Float16* in, void* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    const uint64_t t = ceil_div(seg_len, kTile);           // tiles per segment
    if (t <= 2) launch_scan_segment_shape<1, 2, MODE>(in, out, n, seg_len, s);
    else if (t <= 3) launch_scan_segment_shape<1, 3, MODE>(in, out, n, seg_len, s);
    else if (t <= 4) launch_scan_segment_shape<1, 4, MODE>(in, out, n, seg_len, s);
    else if (t <= 6) launch_scan_segment_shape<1, 6, MODE>(in, out, n, seg_len, s);
    else if (t <= 8) launch_scan_segment_shape<1, 8, MODE>(in, out, n, seg_len, s);
    else if (t <= 12) launch_scan_segment_shape<1, 12, MODE>(in, out, n, seg_len, s);
    else if (t <= 16) launch_scan_segment_shape<1, 16, MODE>(in, out, n, seg_len, s);
    else if (t <= 24) launch_scan_segment_shape<2, 12, MODE>(in, out, n, seg_len, s);
    else if (t <= 32) launch_scan_segment_shape<2, 16, MODE>(in, out, n, seg_len, s);
    else if (t <= 48) launch_scan_segment_shape<4, 12, MODE>(in, out, n, seg_len, s);
    else if (t <= 64) launch_scan_segment_shape<4, 16, MODE>(in, out, n, seg_len, s);
    else if (t <= 96) launch_scan_segment_shape<8, 12, MODE>(in, out, n, seg_len, s);
    else launch_scan_segment_shape<8, 16, MODE>(in, out, n, seg_len, s);
    return check_launch("scan_segment_kernel");
}

// Segment lengths that are no power of two but long enough for the persistent chain (its ragged last tile per
// segment is cut off by the buffer range check, which works on whole 8-element groups).
inline bool chain_takes_any_length(uint64_t seg_len) {
    return g_variant.formulation == kMfma && g_variant.scan_carry == kStrategyLookback && seg_len % 8 == 0 &&
           seg_len >= 2 * scan_shape_tile(10);
}

// Which kernel takes a scan whose seg_len is no power of two (or below 16); class = floor(log2(seg_len)).  The
// default: the chain where it is valid, one workgroup per segment where that is known to win, else the tiles.
enum ScanAny { kScanAnyTiles = 0, kScanAnyTilesAlt = 1, kScanAnySegment = 2, kScanAnyChain = 3, kScanAnyCount = 4 };
inline bool scan_any_valid(int id, uint64_t seg_len) {
    switch (id) {
        case kScanAnyTiles:
        case kScanAnyTilesAlt: return seg_len >= kTiledScanMin;
        case kScanAnySegment: return segment_kernel_takes(seg_len);
        case kScanAnyChain: return chain_takes_any_length(seg_len);
        default: return false;
    }
}
// One workgroup per segment beats the fixed tiles (284-291 us at n = 2^28 whatever the length) where the segments
// start on 128-byte boundaries and fill at least four fifths of the workgroup's share of one tile per wavefront:
// 270-282 us at 1280, 1536, 2560, 3584, 7168 and 8000 elements; 293-372 us at 520, 1000, 2056, 3000, 4088, 4104
// (short of the share, or rows of the tiles that straddle cache lines), 300-315 us from 12000 elements on (two
// tiles per wavefront).
inline bool segment_kernel_preferred(uint64_t seg_len) {
    if (!segment_kernel_takes(seg_len) || seg_len % 64 != 0 || seg_len > 16 * (uint64_t)kTile) return false;
    const uint64_t t = ceil_div(seg_len, kTile);
    const uint64_t share = t <= 4 ? t : (t <= 6 ? 6 : (t <= 8 ? 8 : (t <= 12 ? 12 : 16)));     // as launch_scan_segment picks it
    return 5 * seg_len >= 4 * share * kTile;
}
inline int pick_scan_any(uint64_t seg_len) {
    const int tuned = tuned_id(kTuneScanAny, floor_log2(seg_len));
    if (scan_any_valid(tuned, seg_len)) return tuned;
    if (scan_any_valid(kScanAnyChain, seg_len)) return kScanAnyChain;
    if (segment_kernel_preferred(seg_len)) return kScanAnySegment;
    return kScanAnyTiles;
}

inline tcr_status scan_any(const void* in, void* out, uint64_t n, uint64_t seg_len, uint32_t flags, hipStream_t s) {
    const _Float16* x = static_cast<const _Float16*>(in);
    const int mode = (int)(flags & 3u);
    if (seg_len != n && (!is_pow2(seg_len) || seg_len < 16)) {
        const int pick = pick_scan_any(seg_len);
        if (pick == kScanAnyChain) {
            // long segments of any length that keeps 8-element groups whole: the chain on a per-segment tile grid
            switch (mode) {
                case 0: return launch_chain<kMfma, 0>(10, x, out, n, seg_len, s);
                case 1: return launch_chain<kMfma, 1>(10, x, out, n, seg_len, s);
                case 2: return launch_chain<kMfma, 2>(10, x, out, n, seg_len, s);
                default: return launch_chain<kMfma, 3>(10, x, out, n, seg_len, s);
            }
        }
        if (pick == kScanAnySegment) {
            switch (mode) {
                case 0: return launch_scan_segment<0>(x, out, n, seg_len, s);
                case 1: return launch_scan_segment<1>(x, out, n, seg_len, s);
                case 2: return launch_scan_segment<2>(x, out, n, seg_len, s);
                default: return launch_scan_segment<3>(x, out, n, seg_len, s);
            }
        }
        return launch_generic<true>(x, out, n, seg_len, flags, s, pick == kScanAnyTilesAlt ? 1 : 0);
    }
    // the cross-lane alternative is kept for the default mode only
    const int form = tuned_formulation(kTuneScan, tuning_class(seg_len, seg_len == n));
    if (form == kDpp && mode == 0) return scan_tuned<kDpp, 0>(x, out, n, seg_len, s);
    if (g_variant.formulation == kDpp) return TCR_ERR_UNSUPPORTED;        // forced for every class: the other modes have no kernels
    switch (mode) {
        case 0: return scan_tuned<kMfma, 0>(x, out, n, seg_len, s);
        case 1: return scan_tuned<kMfma, 1>(x, out, n, seg_len, s);
        case 2: return scan_tuned<kMfma, 2>(x, out, n, seg_len, s);
        default: return scan_tuned<kMfma, 3>(x, out, n, seg_len, s);
    }
}

// The scan with a binary16 accumulator (TCR_ACC_F16): powers of two and the one-segment scan, 16-byte aligned arrays.
template <int U, int W, int CARRY, int EXCL>
inline void launch_scan_half_shape(const _Float16* in, _Float16* out, uint64_t n, uint64_t seg_mask, uint64_t seg_len,
                                   const ScanWorkspace& dev, hipStream_t s) {
    const unsigned blocks = (unsigned)ceil_div(n, (uint64_t)kTile * U * W);
    scan_half_kernel<U, W, CARRY, EXCL><<<dim3(blocks), dim3(W * kWave), 0, s>>>(in, out, n, seg_mask, seg_len, dev);
}

template <int EXCL>
inline tcr_status scan_half(const _Float16* in, _Float16* out, uint64_t n, uint64_t seg_len, hipStream_t s) {
    const bool whole = seg_len == n;
    if (!whole && !is_pow2(seg_len)) return TCR_ERR_UNSUPPORTED;
    if (!aligned(in, 16) || !aligned(out, 16)) return TCR_ERR_UNSUPPORTED;
    const uint64_t len = seg_len;                                  // decides the launch shape
    const uint64_t seg_mask = (whole && !is_pow2(n)) ? ~0ull : seg_len - 1;
    if (whole && !is_pow2(n)) seg_len = ~0ull;                     // one segment of any length: never restarts
    const ScanWorkspace none = {};
    if (len <= 1024) launch_scan_half_shape<1, 2, kNoCarry, EXCL>(in, out, n, seg_mask, seg_len, none, s);
    else if (len <= 4096) launch_scan_half_shape<1, 8, kNoCarry, EXCL>(in, out, n, seg_mask, seg_len, none, s);
    else if (len <= 16384) launch_scan_half_shape<2, 16, kNoCarry, EXCL>(in, out, n, seg_mask, seg_len, none, s);
    else if (len <= 65536) launch_scan_half_shape<8, 16, kNoCarry, EXCL>(in, out, n, seg_mask, seg_len, none, s);
    else {
        const uint64_t tiles = ceil_div(n, (uint64_t)kTile * 8 * 16);
        ScanWorkspace dev = {};
        Workspace* ws = nullptr;
        bool capturing = false;
        tcr_status st = get_workspace(s, &ws, &capturing);
        if (st != TCR_OK) return st;
        st = begin_lookback(ws, s, tiles, &dev, capturing);
        if (st != TCR_OK) return st;
        launch_scan_half_shape<8, 16, kLookback, EXCL>(in, out, n, seg_mask, seg_len, dev, s);
        st = check_launch("scan_half_kernel");
        if (st != TCR_OK) {
            ws->dirty = true;
            return st;
        }
        ws->tickets_issued += (uint32_t)tiles;
        return TCR_OK;
    }
    return check_launch("scan_half_kernel");
}

// out_align: the natural alignment of the output's elements.
inline tcr_status validate(const void* in, const void* out, uint64_t n, uint64_t seg_len, uintptr_t out_align) {
    if (seg_len == 0) return TCR_ERR_INVALID_ARG;
    if (n % seg_len != 0) return TCR_ERR_INVALID_ARG;
    if (n == 0) return TCR_OK;
    if (in == nullptr || out == nullptr) return TCR_ERR_INVALID_ARG;
    if (!aligned(in, 2) || !aligned(out, out_align)) return TCR_ERR_INVALID_ARG;
    if (n > kMaxElements) return TCR_ERR_UNSUPPORTED;
    return TCR_OK;
}


}  // namespace host
}  // namespace tcr
