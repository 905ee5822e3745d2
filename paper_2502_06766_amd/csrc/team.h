// The threads that work on one head together, and their prefix sums and ranges.
#pragma once
#include "device_utils.h"

namespace tka {

// A whole workgroup, or one wave of it.
template <int NT_>
struct WorkgroupTeam {
    static constexpr int NT = NT_, NW = NT_ / kWave;
    static __device__ __forceinline__ int rank() { return (int)threadIdx.x; }
    static __device__ __forceinline__ void sync() { __syncthreads(); }
};
struct WaveTeam {
    static constexpr int NT = kWave, NW = 1;
    static __device__ __forceinline__ int rank() { return lane_id(); }
    static __device__ __forceinline__ void sync() { wave_sync(); }
};

// Exclusive prefix sum of n over the team; `total` for all.  One barrier; `slot` alternates between two places so that
// the next call need not wait for the readers of this one.
template <class Team, class SM>
__device__ __forceinline__ uint32_t team_prefix(uint32_t n, uint32_t& total, SM& sm, int slot) {
    const int lane = lane_id();
    const uint32_t inc = wave_scan_add(n);
    if (Team::NW == 1) {
        total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        return inc - n;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (lane == kWave - 1) sm.tot[slot][wave] = inc;
    Team::sync();
    const uint32_t t = row_scan_add((lane & 15) < Team::NW ? sm.tot[slot][lane & 15] : 0u);
    total = (uint32_t)__builtin_amdgcn_readlane((int)t, Team::NW - 1);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)t, wave - 1) : 0u;
    return before + inc - n;
}

// Smallest and largest of every thread's (lo, hi) over the team, one barrier.
template <class Team, class SM>
__device__ __forceinline__ void team_range(float& lo, float& hi, SM& sm, int slot) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    lo = wave_min(lo); hi = wave_max(hi);
    if (Team::NW == 1) { Team::sync(); return; }
    if (lane == 0) { sm.red[slot][0][wave] = lo; sm.red[slot][1][wave] = hi; }
    Team::sync();
    const int w = lane < Team::NW ? lane : 0;
    lo = wave_min(sm.red[slot][0][w]); hi = wave_max(sm.red[slot][1][w]);
}

}  // namespace tka
