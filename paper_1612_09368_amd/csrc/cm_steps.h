// Rotating counters of the step machines, and how far one workgroup may run
// ahead of the others' reads of them.  Host code too: tests/host/chain_check.cpp
// plays the steps through.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cm {

// A queue's tail exists three times: step r reads one, pushes to the next and
// clears the third, which step r + 1 pushes to.
__host__ __device__ constexpr int slot_read(int32_t r) { return r % 3; }
__host__ __device__ constexpr int slot_push(int32_t r) { return (r + 1) % 3; }
__host__ __device__ constexpr int slot_clear(int32_t r) { return (r + 2) % 3; }

// After a grid barrier every workgroup looks at the counters (slot_read of the
// next step) by itself, in its own time, and workgroup 0 may already run that
// step.  One step leaves what the others still read alone; the step after it
// clears it (slot_clear(r + 1) == slot_read(r)), and a workgroup that looks only
// then would take another way than the rest.  So workgroup 0 runs this many
// steps of a chain at once, and goes on when every other workgroup has arrived
// at the barrier that ends the chain, thus has looked (chain_alone).
constexpr int CHAIN_FREE = 1;

// A chain of local steps looks at its time slice when (steps & mask) == 0: every
// 16 steps (the look takes two workgroup barriers, and 16 steps of the default
// bounds take well under a millisecond), but after each one where the bounds let
// a single step take milliseconds, so that 16 of them could outlast a barrier wait.
__host__ __device__ constexpr int slice_mask(int32_t local_edges, int32_t local_items, int32_t local_work) {
    return local_edges > (1 << 16) || local_items > (1 << 14) || local_work > (1 << 20) ? 0 : 15;
}

}  // namespace cm
