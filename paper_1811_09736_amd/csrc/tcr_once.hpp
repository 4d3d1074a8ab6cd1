// Scans of segments that start anywhere -- regular ones of a length no tuned kernel takes, and irregular ones -- with one
// tile of the array per workgroup and nothing drawn or chained between workgroups.
//
// A tile needs one number from in front of it: the sum of its open segment, from that segment's start s0 to the tile's
// own start.  s0 is known without asking another workgroup -- by a division for regular segments, from the offsets
// entry in front of the tile for irregular ones -- and so is the way the sum is found:
//   * s0 at most a tile or so in front: the workgroup adds those elements up itself, 512 to a wavefront, while its own
//     data is on its way (they are a neighbour's data, mostly found in a cache);
//   * further away: the published sums of the tiles from the one that holds s0 on, read in one round trip, or, in most larger
//     arrays, the carry that the relay makes of them (tcr_relay.hpp).  As in the chained scan of arrays that the chip holds at
//     once, what is not there after `patience` looks is added up from the elements, so no wait depends on which workgroups run.
// Bound: memory for large arrays, the chain of dependent steps for the smaller ones.  The ticket, the look-back and, for
// regular segments, the bitmap of the starts and its two barriers are what this form does without.
// (The tile arithmetic is that of irregular_scan_kernel, the chained form: running sums that restart at heads inside a
// lane's eight elements, pairs of (head, sum) across lanes and wavefronts.)
#pragma once
#include "tcr_irregular.hpp"

namespace tcr {

struct TileScan {
    const _Float16* in;           // `shift` elements in front of the caller's array, 16-byte aligned
    const uint64_t* offsets;      // irregular: nseg + 1 entries
    void* out;                    // `shift` elements in front of the caller's array
    uint64_t n;                   // elements counted from `in`
    uint64_t nseg;
    uint64_t seg_len;             // regular
    double per_elem;              // regular: 1 / seg_len; irregular: (nseg + 1) / n
    uint32_t grid_log2;           // irregular: distance of a search's first probes among the offsets
    uint32_t magic;               // regular, seg_len <= kLocalMax: ceil(2^32 / seg_len)
    uint32_t pattern;             // regular: bit i set iff i is a multiple of seg_len, i < 8
    uint32_t shift;
    uint32_t vector_stores;       // `out` is 16-byte aligned
    uint32_t fill;                // irregular: positions outside the segments are set to 0
    uint32_t patience;
};
constexpr uint64_t kLocalMax = 8192;          // longest regular segment whose open part the workgroup adds up itself

// 512 elements from position `at` (a multiple of 512 inside the array) of which those in front of `from` do not count:
// their sum, by one wavefront.
__device__ __forceinline__ float masked_tile_sum(half8 x, uint64_t at, uint64_t from, int lane) {
    const uint64_t mine = at + 8 * (uint64_t)lane;
    const half8 kept = drop_leading(x, from > mine ? (int)(from - mine < 8 ? from - mine : 8) : 0);
    return read_lane(row_sum_to_last<16>(mfma(const_ones(), kept, splat(0.0f))[0]), 15);
}

// The elements of tile t from position s0 on: their sum, by one wavefront.
__device__ __forceinline__ float open_tile_sum(const TileScan& a, uint32_t t, uint64_t s0, int tile_log2, int lane) {
    const uint64_t begin = (uint64_t)t << tile_log2;
    float sum = 0.0f;
    for (uint64_t at = begin; at < begin + (1ull << tile_log2); at += (uint64_t)kTile)
        if (at + (uint64_t)kTile > s0) sum += masked_tile_sum(load8(a.in, at + 8 * (uint64_t)lane), at, s0, lane);
    return sum;
}

// One wavefront: the sum from position s0 to the start of `tile` out of what the tiles in between have published, 64 at a time, the
// nearest first; number `looker` of LOOKERS that take turns.  TAILS: tiles publish either status (with a relay).  What is not there after
// `patience` looks is added up from the elements, or (GIVE_UP) the result is false.
// T: what the sums are added in.
template <bool GIVE_UP, int LOOKERS = 1, bool TAILS = false, typename T>
__device__ __forceinline__ bool lookup_open_sum(const TileScan& a, const ScanWorkspace& ws, uint32_t tile, uint64_t s0, int tile_log2, int lane,
                                                T& sum, int looker = 0) {
    const uint32_t first = (uint32_t)(s0 >> tile_log2);
    const uint32_t want = ws.epoch * 4u + kStatusAggregate;
    T acc = 0;
    const uint32_t skipped = 64u * (uint32_t)looker;
    for (uint32_t hi = tile - first > skipped ? tile - skipped : first; hi > first;) {
        const uint32_t span = hi - first > 64u ? 64u : hi - first;
        bool need = (uint32_t)lane < span;
        float v = 0.0f;
        uint32_t polls = 0;
        while (true) {
            if (need) {
                const unsigned long long d = load_descriptor(&ws.desc[hi - 1u - (uint32_t)lane]);
                if (TAILS ? (uint32_t)(d >> 34) == ws.epoch : (uint32_t)(d >> 32) == want) {
                    v = __builtin_bit_cast(float, (uint32_t)d);
                    need = false;
                }
            }
            unsigned long long missing = __ballot(need);
            if (missing == 0ull) break;
            if (++polls > a.patience) {
                if constexpr (GIVE_UP) return false;
                for (; missing != 0ull; missing &= missing - 1ull) {
                    const int slot = __builtin_ctzll(missing);
                    const float elements = open_tile_sum(a, hi - 1u - (uint32_t)slot, s0, tile_log2, lane);
                    if (lane == slot) v = elements;
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        acc += (T)v;
        if constexpr (LOOKERS == 1) hi -= span;
        else hi = hi - first > 64u * LOOKERS ? hi - 64u * LOOKERS : first;
    }
    sum = wave_sum(acc);                                 // (added per lane first: one chain of roundings of the whole sum's size, not one per look)
    return true;
}

// Where the sum in front of a tile comes from if it is more than the tile's wavefronts add up themselves.  kSumsWide: arrays whose workgroups run all
// at once, and regular segments; one wavefront looks it up.  The others are for arrays whose workgroups follow each other, in workgroups of four
// wavefronts: they take turns at looking it up (kSumsLookedUp), the relay hands it out (kSumsRelayed, tcr_relay.hpp), or they look up the sums of up to
// kNearTiles tiles, one look each, and wait for the relay only further away from the segment's start (kSumsNear).
enum TileSums { kSumsWide = 0, kSumsLookedUp = 1, kSumsNear = 2, kSumsRelayed = 3 };
constexpr uint32_t kNearTiles = 64 * kRelayWaves;

// How the sum in front reaches a lane's elements.  It may be millions of times one of them, so kCarryLate adds it once, behind the lane's eight additions, not in front of
// them.  Where workgroups follow each other (tiles of four wavefronts, and regular ones beyond what the chip holds at once) the two more operations per element are
// free; where all run at once they cost 5 to 10 % (seven segments in 2^24 elements: 23.5 us, 25.3 with them).  kCarryExact: and what goes into that sum --
// the wavefronts' values, what is looked up, the parts of the open sum -- is added up in binary64, the wavefronts' by one scan over the lanes in place
// of a loop over up to sixteen of them.  Error against 64 bits (2-norms, uniform values; early / late / exact): 8191 elements, added up by each tile, 6.0e-8 / 5.2e-8 / 3.4e-8;
// 100003, looked up, - / 5.4e-8 / 4.4e-8 (the relay's tiles 4.4e-8 and 4.5e-8).  Binary16 results don't show it.
enum CarryKind { kCarryEarly = 0, kCarryLate = 1, kCarryExact = 2 };

// LOCAL (regular segments of 2 to WAVES * 512 elements): no sum is ever looked up, no workspace.
// Relayed regular tiles all wait for the relay, in the order of the array; irregular ones only where it is more than the four
// wavefronts add up themselves (segments of 16 in 2^27 elements 165 us, 174 where all wait; seven segments 151 and 149).  The
// entries of tiles of four wavefronts are found with one search of two rounds around where they are likely to be (GUIDED), not two of four over the whole array.
// Registers: at most 64, so that 8 wavefronts per SIMD run.  A wavefront that has waited in vain loads its elements again behind the
// additions, so that they need not be held across them: 43 to 55 registers where four sub-tiles took 64 and 44 bytes of scratch
// (lognormal lengths / segments of 16 / seven segments in 2^24 elements 21.7 / 23.9 / 23.6 -> 21.0 / 23.5 / 22.7 us).  Not with fewer
// sub-tiles, which lose 2 to 5 %, nor with binary16 results (15.7 -> 16.0): 64 registers, 28 to 76 bytes.
// MOST: wavefronts per SIMD at most.
template <int U, int WAVES, bool REGULAR, int MODE, bool LOCAL, int SUMS = kSumsWide, int MOST = 8,
          int CARRY = SUMS != kSumsWide || (!LOCAL && MOST < 8) ? kCarryLate : kCarryEarly>
__global__ __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(U < 4 ? 4 : MOST, MOST))) void tile_scan_kernel(TileScan a, ScanWorkspace ws_arg) {
    static_assert(!LOCAL || REGULAR, "");
    static_assert(SUMS == kSumsWide || (WAVES == kRelayWaves && !LOCAL), "");
    constexpr bool RELAY = SUMS == kSumsNear || SUMS == kSumsRelayed;
    constexpr bool GUIDED = !REGULAR && SUMS != kSumsWide;    // (how a tile's entries are found)
    constexpr int LOOKERS = SUMS == kSumsLookedUp || SUMS == kSumsNear ? WAVES : 1;
    constexpr int EXCL = MODE & 1, F16 = MODE >> 1;
    constexpr uint32_t kChunk = (uint32_t)kTile * U;          // one wavefront's share
    constexpr uint32_t kBlockTile = kChunk * WAVES;           // one workgroup's share
    constexpr uint64_t kBackMax = (uint64_t)kTile * WAVES;    // the open part that the wavefronts add up themselves
    constexpr int kTileLog2 = __builtin_ctz(kBlockTile);
    __shared__ uint32_t s_heads[REGULAR ? 1 : kBlockTile / 32];
    __shared__ uint64_t s_bound[4];
    __shared__ float s_wave_value[WAVES], s_back[WAVES];      // (s_back: parts of the open sum, added up or looked up)
    // Sums looked up by all, added as the relay adds, in binary64 (lognormal lengths in 2^20 * 17 / 24 elements 5.1e-8 / 6.5e-8 off 64 bits in binary32,
    // 4.5e-8 / 4.6e-8 so, in the same time; with binary16 results, which don't show it, 1 % more).
    using Far = std::conditional_t<F16 != 0, float, double>;
    __shared__ Far s_far[LOOKERS > 1 ? WAVES : 1];
    __shared__ uint32_t s_wave_flag[WAVES];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (RELAY) {
        __shared__ RelayShared relay;
        if (blockIdx.x == 0u) {
            relay_carries(resolve_workspace(ws_arg), gridDim.x - 1u, relay, wave, lane);
            return;
        }
    }
    const uint32_t tile = blockIdx.x - (RELAY ? 1u : 0u);
    const uint64_t tb = (uint64_t)tile * kBlockTile;
    const uint64_t base = tb + (uint64_t)wave * kChunk;
    // the wavefront's share: whole groups of 8 through the range check, the group that the array's end cuts by element
    const uint64_t left = base < a.n ? a.n - base : 0;
    const uint32_t count = left < kChunk ? (uint32_t)left : kChunk, whole = count & ~7u;
    const __amdgpu_buffer_rsrc_t src = make_rsrc(a.in + (count ? base : 0), whole * 2u);
    half8 x[U];
    const auto load_share = [&] {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = buffer_load8(src, (uint32_t)(kTile * u + 8 * lane) * 2u);
    };
    const auto load_cut_group = [&] {
        if (count != whole) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((uint32_t)(kTile * u + 8 * lane) == whole) x[u] = load8_guarded(a.in, base + whole, a.n);
        }
    };
    if constexpr (REGULAR) load_share();
    // Irregular tiles that search for themselves, all at the same time: what every wavefront asked for in front of the search each of its rounds
    // would wait behind (lognormal lengths in 2^24 elements 24.4 us), and behind it memory idles during the search.  So in every other
    // workgroup of an XCD (they follow each other in eights) the wavefronts that do not search ask for their elements first: lognormal lengths / segments of 16 / of 200
    // / one segment, 2^24 elements, 21.2 / 23.6 / 21.5 / 25.0 -> 20.4 / 23.1 / 20.5 / 24.3; in every workgroup 21.5, in three of four 21.0,
    // in every other one all wavefronts 20.8.
    constexpr bool STAGGERED = !REGULAR && !GUIDED && U == 4 && WAVES == 8;
    const bool early = STAGGERED && wave >= 2 && (blockIdx.x & 8u) != 0u;
    if (early) load_share();

    // where the open segment starts (tb: nothing reaches into the tile), and which part of the array lies in a segment
    uint64_t s0 = tb, first = a.shift, last = a.n;
    uint32_t head = 0;                        // regular: position of the tile's first head
    bool has_heads = true;
    if constexpr (REGULAR) {
        if (tb < a.shift) {
            head = a.shift;                   // (the first tile of an array that is not 16-byte aligned)
        } else {
            const uint64_t p = tb - a.shift;
            uint64_t q = (uint64_t)((double)p * a.per_elem);                  // p / seg_len, one off at most
            if (q * a.seg_len > p) --q;
            if ((q + 1) * a.seg_len <= p) ++q;
            const uint64_t back = p - q * a.seg_len;
            s0 = tb - back;
            const uint64_t h = back ? a.seg_len - back : 0;
            head = h < kBlockTile ? (uint32_t)h : kBlockTile;
        }
    } else {
        for (uint32_t i = threadIdx.x; i < kBlockTile / 32; i += WAVES * kWave) s_heads[i] = 0u;
        // entry s lies on position offsets[s] + shift
        const auto mark = [&](uint64_t entry) {
            const uint64_t pos = entry + a.shift - tb;
            const bool in = pos < (uint64_t)kBlockTile;
            if (in) atomicOr(&s_heads[pos >> 5], 1u << (pos & 31u));
            return in;
        };
        if constexpr (!GUIDED) {
            if (wave < 2) {
                const uint64_t edge = tb + (wave ? (uint64_t)kBlockTile : 0);
                const uint64_t below = wave_lower_bound(a.offsets, a.nseg + 1, edge > a.shift ? edge - a.shift : 0, lane);
                if (lane == 0) s_bound[wave] = below;
            }
            first = a.offsets[0] + a.shift;
            last = a.offsets[a.nseg] + a.shift;
            if (last > a.n) last = a.n;
            lds_barrier();
            if (!early) load_share();
            const uint64_t lo = s_bound[0], hi = s_bound[1];
            has_heads = lo < hi;
            for (uint64_t s = lo + threadIdx.x; s < hi; s += (uint64_t)(WAVES * kWave)) mark(a.offsets[s]);
            // (nothing is open in front of the first entry and behind the last; an entry on tb itself restarts there)
            if (lo > 0 && lo <= a.nseg) {
                const uint64_t at = a.offsets[lo - 1] + a.shift;
                if (at < tb) s0 = at;
            }
        } else {
            // One wavefront finds the entries in front of the tile, the last of them (the start of the segment open there) and, among
            // those that the search's last round has read, the tile's first ones -- mostly all of them where segments are not
            // short.  Nothing else is asked for meanwhile: in an array that the chip holds at once all workgroups search at the same
            // time, and behind everybody's elements every round would wait for them (2^24 elements, seven segments: 24.4 us with
            // the other wavefronts' elements asked for in front of the search).
            lds_barrier();                        // (the bits are cleared)
            if (wave == 0) {
                const EntryFound found = find_entry(a.offsets, a.nseg + 1, tb > a.shift ? tb - a.shift : 0, (uint64_t)((double)tb * a.per_elem),
                                                    a.grid_log2, lane, [] {}, mark);
                if (lane == 0) {
                    s_bound[0] = found.below;
                    s_bound[1] = found.last;
                    s_bound[2] = found.below + found.wanted == found.seen ? found.seen : ~0ull;       // where more may follow
                    s_bound[3] = found.wanted;
                }
            }
            first = a.offsets[0] + a.shift;
            last = a.offsets[a.nseg] + a.shift;
            if (last > a.n) last = a.n;
            lds_barrier();
            load_share();
            const uint64_t lo = s_bound[0], next = s_bound[2];
            has_heads = s_bound[3] != 0u;
            // (nothing is open in front of the first entry and behind the last; an entry on tb itself restarts there)
            if (lo > 0 && lo <= a.nseg && s_bound[1] + a.shift < tb) s0 = s_bound[1] + a.shift;
            if (next <= a.nseg) {                 // (the same in every wavefront)
                // 64 entries per wavefront and half of a turn; a wavefront that has found one behind the tile is done
                constexpr uint64_t kTurn = 2 * WAVES * kWave;
                for (uint64_t at = next;;) {
                    const uint64_t rest = at <= a.nseg ? a.nseg + 1 - at : 0;
                    const uint32_t there = rest < kTurn ? (uint32_t)rest : (uint32_t)kTurn;
                    const __amdgpu_buffer_rsrc_t entries = make_rsrc(a.offsets + (rest ? at : 0), there * 8u);
                    // (read with the entries of the turn, for below)
                    const bool ahead = at != next && at + 64 * kTurn <= a.nseg;
                    const uint64_t here = a.offsets[ahead ? at : 0], further = a.offsets[ahead ? at + kTurn : 0];
                    uint64_t entry[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        entry[k] = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(entries, (int)((threadIdx.x + (uint32_t)(k * WAVES * kWave)) * 8u), 0, 0));
                    bool filled = true;
#pragma unroll
                    for (int k = 0; k < 2; ++k) filled = __ballot(threadIdx.x + (uint32_t)(k * WAVES * kWave) < there && mark(entry[k])) == ~0ull;
                    if (!filled) break;
                    // Empty segments.  Where a run of them goes on for long this turn has
                    // marked their position; on with the turn in which they end, the same one for every wavefront (a million of them between
                    // segments of 16 in 2^26 elements: 1975 us -> 99; looked for from the second turn on and not only behind as many entries
                    // as the tile has elements, since all tiles behind this one wait: segments of 1000 and 2^20 * 0.24 empty ones in a row in 2^20 * 24 elements
                    // 44.1 -> 38.7.  Tiles of kSumsWide take every entry: 2^20 * 3 empty ones in 2^20 * 12 elements 2630).
                    uint64_t turns = 1;
                    if (ahead && here == further && here == a.offsets[at + 64 * kTurn]) {
                        const uint64_t behind = wave_lower_bound(a.offsets, a.nseg + 1, here + 1, lane);
                        if (behind >= at + 2 * kTurn) turns = (behind - at) / kTurn;
                    }
                    at += turns * kTurn;
                }
                has_heads = true;
                lds_barrier();                    // the heads are marked
            }
        }
    }
    const uint64_t back = tb - s0;
    const bool far = RELAY && REGULAR ? true : !LOCAL && back > kBackMax;
    const bool looks = LOOKERS > 1 && far && (!RELAY || tile - (uint32_t)(s0 >> kTileLog2) <= kNearTiles);     // (all four wavefronts do)
    // the wavefront's 512 elements of the open part, counted back from the tile's start
    const uint64_t behind = (uint64_t)kTile * (uint64_t)wave;
    const bool mine = !far && behind < back;
    const uint64_t back_at = mine ? tb - behind - (uint64_t)kTile : 0;
    half8 back_x = {};
    if constexpr (!(RELAY && REGULAR)) {
        const __amdgpu_buffer_rsrc_t back_src = make_rsrc(a.in + back_at, mine ? (uint32_t)kTile * 2u : 0u);
        back_x = buffer_load8(back_src, 16u * (uint32_t)lane);
    }
    if constexpr (!REGULAR && !GUIDED) __syncthreads();   // the heads are marked

    load_cut_group();
    uint32_t heads[(U + 3) / 4] = {};             // the lane's heads: a byte per sub-tile
    uint64_t flag_before[U];                      // bit l: a head in a lane in front of lane l inside the sub-tile
    uint32_t seen_before[U];                      // a head in a sub-tile in front
    float lane_value[U], before[U], run = 0.0f;
    uint32_t chunk_flag = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint32_t bits;
        if constexpr (REGULAR) {
            // the lane's first head, counted from its first element (the heads are head, head + seg_len, ...)
            const uint32_t at = (uint32_t)wave * kChunk + (uint32_t)(kTile * u + 8 * lane);
            uint32_t c;
            if constexpr (LOCAL) {
                const uint32_t t = at - head;
                c = at <= head ? head - at : __umulhi(t + (uint32_t)a.seg_len - 1u, a.magic) * (uint32_t)a.seg_len - t;
            } else {
                // (longer than kLocalMax: the next heads by repeated addition, a few at most per tile)
                uint64_t h = head;
                while (h < at) h += a.seg_len;
                c = h - at < 8u ? (uint32_t)(h - at) : 8u;
            }
            bits = c < 8u ? (a.pattern << c) & 0xffu : 0u;
        } else {
            bits = has_heads ? (uint32_t)reinterpret_cast<const uint8_t*>(s_heads)[wave * (kChunk / 8) + (kTile / 8) * u + lane] : 0u;
        }
        heads[u / 4] |= bits << (8 * (u % 4));
        uint64_t flags = __ballot(bits != 0u);
        float v[1] = {0.0f};
#pragma unroll
        for (int e = 0; e < 8; ++e) v[0] = ((bits >> e) & 1u ? 0.0f : v[0]) + (float)x[u][e];
        flags = wave_seg_scan_inclusive_bits<1>(flags, v);
        flag_before[u] = flags << 1;
        const uint32_t sub_flag = (uint32_t)(flags >> 63);
        seen_before[u] = chunk_flag;
        lane_value[u] = wave_shr1(v[0]);
        const float sub_value = read_lane(v[0], 63);
        before[u] = run;
        run = sub_flag ? sub_value : run + sub_value;
        chunk_flag |= sub_flag;
    }
    const float back_sum = mine ? masked_tile_sum(back_x, back_at, s0, lane) : 0.0f;
    if (lane == 0) {
        s_wave_value[wave] = run;
        s_wave_flag[wave] = chunk_flag;
        s_back[wave] = back_sum;
    }
    __syncthreads();
    constexpr bool LATE = CARRY != kCarryEarly, EXACT = CARRY == kCarryExact;
    static_assert(!EXACT || (SUMS == kSumsWide && REGULAR), "");
    // the wavefronts' values and, in the row of lanes behind them (LOCAL), the parts of the open sum
    double waves[1] = {};
    uint64_t waves_flags = 0;
    if constexpr (EXACT) {
        static_assert(WAVES <= 16, "");
        waves[0] = lane < WAVES ? s_wave_value[lane] : LOCAL && lane >= 16 && lane < 16 + WAVES ? s_back[lane - 16] : 0.0f;
        waves_flags = wave_seg_scan_inclusive_bits<1>(__ballot(lane < WAVES && s_wave_flag[lane] != 0u) | 1ull << 16, waves);
    }
    if constexpr (!LOCAL) {
        const ScanWorkspace ws = resolve_workspace(ws_arg);
        if (wave == 0) {
            // what later tiles may need of this one: the sum behind its last head
            float total = 0.0f;
            bool tail = false;
            if constexpr (EXACT) {
                total = (float)read_lane(waves[0], WAVES - 1);
            } else {
                for (int v = WAVES - 1; v >= 0; --v) {
                    total += s_wave_value[v];
                    if (s_wave_flag[v]) {
                        tail = true;
                        break;
                    }
                }
            }
            if (lane == 0) {
                if (!RELAY && tile == 0 && ws.state != nullptr && !ws.device_managed) ws.state[0] = ws.epoch;
                __hip_atomic_store(&ws.desc[tile], pack_desc(ws.epoch, RELAY && tail ? kStatusTail : kStatusAggregate, total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            if ((RELAY || LOOKERS == 1) && far && !looks) {
                float pre = 0.0f;
                constexpr bool AGAIN = RELAY || (U == 4 && !F16);      // (elements asked for again by a wavefront that has waited in vain)
                bool got;
                if constexpr (RELAY) got = relay_wait(ws, gridDim.x - 1u, tile, a.patience, pre);
                else {
                    std::conditional_t<EXACT, double, float> looked_up = 0;
                    got = lookup_open_sum<AGAIN>(a, ws, tile, s0, kTileLog2, lane, looked_up);
                    pre = (float)looked_up;
                }
                if constexpr (AGAIN) {
                    if (__builtin_expect(!got, 0)) {
                        pre = add_up_in_front<RELAY>(ws, gridDim.x - 1u, (uint32_t)(s0 >> kTileLog2), tile,
                                                     [&](uint32_t t) { return open_tile_sum(a, t, s0, kTileLog2, lane); });
                        if constexpr (U >= 4 && !F16) {
                            load_share();
                            load_cut_group();
                        }
                    }
                }
                if (lane == 0) s_back[0] = pre;
            }
        }
        if constexpr (LOOKERS > 1) {
            if (looks) {
                Far pre = 0;
                lookup_open_sum<false, LOOKERS, RELAY>(a, ws, tile, s0, kTileLog2, lane, pre, wave);
                if (lane == 0) s_far[wave] = pre;
            }
        }
        if (far) __syncthreads();
    }
    // carry from the wavefronts in front, back to the nearest one that holds a head, else from in front of the tile
    float ext = 0.0f;
    if constexpr (EXACT) {
        double carried = wave != 0 ? read_lane(waves[0], wave - 1) : 0.0;
        if ((wave == 0 || ((waves_flags >> (wave - 1)) & 1ull) == 0ull) && back != 0) {
            if constexpr (LOCAL) {
                carried += read_lane(waves[0], 31);
            } else {
#pragma unroll
                for (int v = 0; v < WAVES; ++v) carried += (double)s_back[v];
            }
        }
        ext = (float)carried;
    } else {
        bool open = true;
        for (int v = wave - 1; v >= 0; --v) {
            ext += s_wave_value[v];
            if (s_wave_flag[v]) {
                open = false;
                break;
            }
        }
        if (open && back != 0) {
            float sum = 0.0f;
            if constexpr (LOOKERS > 1) {
                sum = looks ? (float)((s_far[0] + s_far[1]) + (s_far[2] + s_far[3])) : pairwise_sum(s_back);
            } else {
#pragma unroll
                for (int v = 0; v < WAVES; ++v) sum += s_back[v];
            }
            ext += sum;
        }
    }
    const uint32_t valid_lo = first > base ? (uint32_t)(first - base < kChunk ? first - base : kChunk) : 0u;
    const uint32_t valid_hi = last > base ? (uint32_t)(last - base < kChunk ? last - base : kChunk) : 0u;
    const bool inside = valid_lo == 0u && valid_hi == kChunk && a.vector_stores != 0u;
    void* const dst = F16 ? static_cast<void*>(static_cast<_Float16*>(a.out) + base) : static_cast<void*>(static_cast<float*>(a.out) + base);
    // A whole share that lies in no segment (the middle third of 2^20 * 24 / 64 / 128 elements in segments of 37, the rest in none: 66 / 150 / 293 us ->
    // 38 / 83 / 157).  Not with kSumsNear and binary16 results, whose other shares lose 2 %, nor with kSumsWide (lognormal lengths in 2^24 elements 20.4 -> 20.5).
    if constexpr (!REGULAR && SUMS != kSumsWide && !(F16 && SUMS == kSumsNear)) {
        if (a.fill != 0u && a.vector_stores != 0u && count == kChunk && base >= a.shift && (valid_lo == kChunk || valid_hi == 0u)) {
#pragma unroll
            for (int u = 0; u < U; ++u) store8_t<F16>(dst, (uint32_t)(kTile * u + 8 * lane), splat(0.0f), splat(0.0f));
            return;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float carry = !LATE || seen_before[u] ? 0.0f : ext;
        const float into_sub = LATE || seen_before[u] ? before[u] : before[u] + ext;
        const bool after_head = __builtin_amdgcn_inverse_ballot_w64(flag_before[u]);
        float q = after_head ? lane_value[u] : lane_value[u] + into_sub;
        if constexpr (LATE) carry = after_head ? 0.0f : carry;
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool head = (heads[u / 4] >> (8 * (u % 4) + e)) & 1u;
            const float kept = head ? 0.0f : q;
            q = kept + (float)x[u][e];
            p[e] = EXCL ? kept : q;
            if constexpr (LATE) {
                carry = head ? 0.0f : carry;
                p[e] += carry;
            }
        }
        const uint32_t k = (uint32_t)(kTile * u + 8 * lane);
        if (inside) {
            store8_t<F16>(dst, k, (float4v){p[0], p[1], p[2], p[3]}, (float4v){p[4], p[5], p[6], p[7]});
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in_segment = k + e >= valid_lo && k + e < valid_hi;
                const bool cleared = !REGULAR && a.fill && !in_segment && k + e < count && base + k + e >= a.shift;
                if (in_segment || cleared) {
                    const float r = in_segment ? p[e] : 0.0f;
                    if constexpr (F16) static_cast<_Float16*>(dst)[k + e] = (_Float16)r;
                    else static_cast<float*>(dst)[k + e] = r;
                }
            }
        }
    }
}

}  // namespace tcr
