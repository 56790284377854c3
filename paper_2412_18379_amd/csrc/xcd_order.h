// The order in which a walk's blocks take the points.
//
// Workgroups go to the 8 XCDs round-robin by id, each with an L2 of its own; consecutive blocks of points, whose paths
// share elements, would so meet in no cache.  Here each XCD takes chunks of consecutive blocks instead, chunk by chunk
// in turn: chunks as long as `longest` allows, all of nearly the same length (one chunk per XCD would leave an XCD
// with the longest walks of the point order to run alone at the end).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cnnsns {

struct XcdOrder {
    unsigned blocks, chunk;  // chunk 0: in order of id
    // In order: walks of a few blocks an XCD, and those whose grid, up to 8 `longest` larger, could reach the 2^32
    // threads (2^24 blocks of 256) that a launch may not have.
    __host__ __device__ XcdOrder(unsigned n, unsigned longest) : blocks(n), chunk(0)
    {
        if (n <= 64 || n > (1u << 24) - 8 * longest) return;
        const unsigned per = n / 8 + (n % 8 != 0);  // blocks of an XCD
        const unsigned chunks = per / longest + (per % longest != 0);
        chunk = per / chunks + (per % chunks != 0);
    }
    // workgroups to launch: whole rounds of a chunk on every XCD
    __host__ __device__ unsigned grid() const { return chunk ? (blocks + 8 * chunk - 1) / (8 * chunk) * (8 * chunk) : blocks; }
    // the block of points of workgroup `id` (chunk > 0); those past the last one have none
    __host__ __device__ unsigned block(unsigned id) const
    {
        const unsigned r = id / 8;
        return (r / chunk * 7 + id % 8) * chunk + r;
    }
    __device__ __forceinline__ unsigned block() const { return block(blockIdx.x); }
};

// x of the lane before in a row of 16 (0 for the first)
__device__ __forceinline__ double lane_before(double x)
{
    const uint64_t b = __double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)b, 0x111, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), 0x111, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Whether this lane's point lies within sqrt(near2) of the lane before's, in a row of 16 lanes.
template <class... X>
__device__ __forceinline__ bool near_lane_before(double near2, X... x)
{
    return (((x - lane_before(x)) * (x - lane_before(x))) + ...) <= near2;
}

}  // namespace cnnsns
