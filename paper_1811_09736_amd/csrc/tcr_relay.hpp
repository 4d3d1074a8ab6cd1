// Carries between workgroups: the descriptors in which tiles publish their sums, and the relay, in which one workgroup turns them
// into carries for all the others.
//
// The relay: every workgroup but the first takes one tile, publishes its sum and waits for its carry; the first one reads the
// sums, 64 tiles to a wavefront, adds them up in order -- from wavefront to wavefront through LDS -- and writes each tile's carry
// into a second table (into the word that held its sum: everybody polls the lines that everybody writes, 267 -> 283 us at 2^28).  A carry is two trips through memory behind the slowest sum in front, whatever the distance to
// the segment's start, a tile reads one word instead of a table, and no ticket is drawn.  Bound: memory.  What the form does for a
// large array beside that: tiles get their carries, and so write their results, in the order of the array, also those that need
// none (n = 2^28 in segments of 32768: 269 us, 285 where a segment's first tile does not wait).
// Tiles of 8192 elements by four wavefronts: eight of them per compute unit hide the two trips.  Full scan of 2^20 * 24 / 64 / 128 /
// 256 elements, us: the persistent chain 39.8 / 81.2 / 148.6 / 280.6, this 34.7 / 73.7 / 138.2 / 267.0, segments of 4096, which
// need no carry, 29.5 / 70.0 / 134.0 / 264.1; tiles half as large 39.4 / 92.0 / 178.7 / -, twice as large 31.4 / 81.6 / 150.0 /
// 288.0.  128 tiles at a time per wavefront: 35.0 / 77.6 / 145.8 / 282.6; carries handed out before all 64 sums are there: no gain.
// Progress: nothing guarantees that the first workgroup or those of lower tiles run, so a tile that has not got its carry after
// `patience` looks adds it up itself, from the published sums and, where there are none, from the elements; every workgroup ends,
// so every sum is published in the end and the first workgroup ends too.
#pragma once
#include "tcr_device.hpp"

namespace tcr {

// ------------------------------------------------------------------------------ look-back state
// One 64-bit word per workgroup tile: high half = tag, low half = binary32 value.
// tag = epoch * 4 + status; a word whose epoch differs from the launch's is "not yet written",
// so the table never needs clearing between launches.
constexpr uint32_t kStatusAggregate = 1;   // value = total of this tile only
constexpr uint32_t kStatusPrefix = 2;      // value = total of this tile and all earlier tiles of its segment
constexpr uint32_t kStatusTail = 2;      // (relay) value = sum behind this tile's last segment start
constexpr uint32_t kStatusCarry = 3;     // (relay, second table) value = sum that reaches this tile
constexpr int kSpinLimit = 1 << 20;        // polls of one look-back window before giving up

struct ScanWorkspace {
    unsigned long long* desc;   // [tiles]; the relay's carries and other second tables lie behind
    uint32_t* ticket;           // running count of tiles handed out since the workspace was created
    uint32_t* gave_up;          // set to 1 if a bounded wait expired
    uint32_t ticket_base;       // value of *ticket when this launch starts
    uint32_t epoch;
    // state[0]: epoch of the latest launch, state[1]: *ticket at its start.  Host-managed workspaces
    // (device_managed == 0) pass epoch and ticket_base above and the launch only records its epoch in
    // state[0]; device-managed ones (launches recorded into HIP graphs, whose arguments are frozen)
    // take both from state[], which chain_begin_kernel advances in front of every launch.
    uint32_t* state;
    uint32_t device_managed;
};

__device__ __forceinline__ ScanWorkspace resolve_workspace(ScanWorkspace w) {
    if (w.state != nullptr && w.device_managed) {
        w.epoch = w.state[0];
        w.ticket_base = w.state[1];
    }
    return w;
}

__device__ __forceinline__ unsigned long long pack_desc(uint32_t epoch, uint32_t status, float v) {
    return ((unsigned long long)(epoch * 4u + status) << 32) | (unsigned long long)__builtin_bit_cast(uint32_t, v);
}

// Descriptor words live in uncached device memory and are read with agent scope: the tiles of
// one chain run on different XCDs, whose L2 caches are not coherent with each other.  (A read
// that only bypasses the first-level cache was tried and does see stale words.)
__device__ __forceinline__ unsigned long long load_descriptor(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------------------ the relay
constexpr int kRelayWaves = 4;
constexpr uint32_t kRelaySlots = 2 * kRelayWaves;
struct RelayShared {
    double carry[kRelaySlots];
    uint32_t round[kRelaySlots];          // carry[i] is what reaches group round[i] of 64 tiles
};

// Workgroup 0, all of its kRelayWaves wavefronts: turns the published sums of `tiles` tiles into carries, adding them up
// in binary64: thousands follow each other.  Ends also if a sum never comes; its tiles help themselves.
__device__ __forceinline__ void relay_carries(const ScanWorkspace& ws, uint32_t tiles, RelayShared& sh, int wave, int lane) {
    if (threadIdx.x < kRelaySlots) sh.round[threadIdx.x] = 0u;
    __syncthreads();
    if (threadIdx.x == 0 && ws.state != nullptr && !ws.device_managed) ws.state[0] = ws.epoch;
    __builtin_amdgcn_s_setprio(3);                   // (the other workgroups of this compute unit wait for it too)
    for (uint32_t group = (uint32_t)wave; group <= (tiles - 1u) >> 6; group += (uint32_t)kRelayWaves) {
        const uint32_t tile = group * 64u + (uint32_t)lane;
        bool need = tile < tiles, tail = false;
        double v[1] = {0.0};
        for (int polls = 0;; ++polls) {
            const unsigned long long d = load_descriptor(&ws.desc[tile < tiles ? tile : tiles - 1u]);
            const uint32_t tag = (uint32_t)(d >> 32);
            if (need && (tag >> 2) == ws.epoch) {
                need = false;
                v[0] = (double)__builtin_bit_cast(float, (uint32_t)d);
                tail = (tag & 3u) == kStatusTail;
            }
            if (__ballot(need) == 0ull) break;
            if (polls > kSpinLimit) return;
        }
        const uint64_t flags = wave_seg_scan_inclusive_bits<1>(__ballot(tail), v);
        const double in_front = dpp_move<0x138, 0xf, true>(v[0]), all = read_lane(v[0], 63);       // (the lane in front; 0 for the first)
        double carry = 0.0;
        if (group != 0u) {
            const uint32_t slot = group % kRelaySlots;
            for (int looks = 0; __hip_atomic_load(&sh.round[slot], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != group; ++looks)
                if (looks > 4 * kSpinLimit) return;
            carry = sh.carry[slot];
        }
        if (lane == 0) {
            const uint32_t slot = (group + 1u) % kRelaySlots;
            sh.carry[slot] = (flags >> 63) ? all : carry + all;
            __hip_atomic_store(&sh.round[slot], group + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        const bool restarted = __builtin_amdgcn_inverse_ballot_w64(flags << 1);
        const float mine = (float)(restarted ? in_front : carry + in_front);
        if (tile < tiles) __hip_atomic_store(&ws.desc[tiles + tile], pack_desc(ws.epoch, kStatusCarry, mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One whole wavefront, behind the publication of its tile's sum: whether the carry of `tile` has come within `patience` looks.
__device__ __forceinline__ bool relay_wait(const ScanWorkspace& ws, uint32_t tiles, uint32_t tile, uint32_t patience, float& carry) {
    for (uint32_t polls = 0; polls < patience; ++polls) {
        const unsigned long long d = load_descriptor(&ws.desc[tiles + tile]);
        if ((uint32_t)(d >> 32) == ws.epoch * 4u + kStatusCarry) {
            carry = __builtin_bit_cast(float, (uint32_t)d);
            return true;
        }
        __builtin_amdgcn_s_sleep(8);
    }
    return false;
}
// Where it has not, one whole wavefront: the carry, from what is published of tiles first .. tile - 1 (also without a relay), and elements where
// nothing is; `first` is the tile in which the segment starts.  64 tiles at a time, the nearest first, as far as the nearest one whose carry is
// there; added in binary64, as the relay does: thousands may follow each other, and which way a tile takes is a matter of time (one segment
// of 2^20 * 7 / 11 elements, no tile waiting: 7.1e-8 / 7.8e-8 off 64 bits, 3.0e-7 / 2.0e-7 with the sums added one after the other in binary32,
// 7.5e-8 / 8.1e-8 where tiles wait).  What a tile finds out this way it keeps to itself: carries made of each other's would be rounded once per
// tile.
// total_of(t): what tile t contributes, from its elements.  (Called where the tile's own elements are no longer held; they are loaded
// again: held across this, they would cost the other form registers or scratch.)
template <bool RELAY, typename TOTAL>
__device__ __forceinline__ float add_up_in_front(const ScanWorkspace& ws, uint32_t tiles, uint32_t first, uint32_t tile, TOTAL total_of) {
    const uint32_t lane = threadIdx.x & (uint32_t)(kWave - 1);
    double sum = 0.0;
    for (uint32_t hi = tile; hi > first;) {
        const uint32_t span = hi - first > (uint32_t)kWave ? (uint32_t)kWave : hi - first;
        const uint32_t t = hi - 1u - (lane < span ? lane : 0u);
        const unsigned long long c = RELAY ? load_descriptor(&ws.desc[tiles + t]) : 0ull, d = load_descriptor(&ws.desc[t]);
        const bool carried = RELAY && t != first && (uint32_t)(c >> 32) == ws.epoch * 4u + kStatusCarry;
        const uint64_t carries = __ballot(lane < span && carried);
        const uint32_t last = carries != 0ull ? (uint32_t)__builtin_ctzll(carries) : span - 1u;      // lanes 0 .. last count
        const bool there = (uint32_t)(d >> 34) == ws.epoch;
        float v = there ? __builtin_bit_cast(float, (uint32_t)d) : 0.0f;
        for (uint64_t missing = __ballot(lane <= last && !there); missing != 0ull; missing &= missing - 1ull) {
            const uint32_t slot = (uint32_t)__builtin_ctzll(missing);
            const float elements = total_of(hi - 1u - slot);
            if (lane == slot) v = elements;
        }
        if (lane <= last) sum += (double)v;
        if (carries != 0ull) {
            if (lane == last) sum += (double)__builtin_bit_cast(float, (uint32_t)c);
            break;
        }
        hi -= span;
    }
    return (float)wave_sum(sum);
}

}  // namespace tcr
