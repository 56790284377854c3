// The order in which a walk's blocks take the points.
//
// Workgroups go to the 8 XCDs round-robin by id, each with an L2 of its own; consecutive blocks of points, whose paths
// share elements, would so meet in no cache.  Here each XCD takes chunks of consecutive blocks instead, chunk by chunk
// in turn: chunks as long as `longest` allows, all of nearly the same length (one chunk per XCD would leave an XCD
// with the longest walks of the point order to run alone at the end).
#pragma once

#include <hip/hip_runtime.h>

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

}  // namespace cnnsns
