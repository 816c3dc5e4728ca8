// launch.h -- host-side launchers of the gfx950 kernels (internal to the
// library; the public surface is include/omprt.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "sched.h"

namespace omprt {

// Bytes of one cross-team partial slot: 4 tagged 64-bit words (payloads up to
// 16 bytes, 32 bits per word).
constexpr int kSlotBytes = 32;

// Header in front of the slots: 256 bytes with the election counter, the epoch
// and the status word, then the counters of the election's groups.
constexpr int kHeaderBytes = 256 + kElectGroups * kElectGroupBytes;

// Device words a launch of the plain kernels uses for the cross-team step.
struct CrossTeamArgs {
    void* slots;          // teams * kSlotBytes, zero-filled at allocation
    uint32_t* counter;    // election counter, 0 between launches
    uint32_t* epoch;      // launch epoch
    uint32_t* status;     // poll-timeout flag
    int32_t groups = 0;   // election in kElectGroups groups (elect_groups)
};

// Whether a launch's election goes in groups.  One counter serves T teams 13 ns
// apart, which is what a short launch's teams wait for as they all end at once
// (us, one counter -> groups: fp32 max 2^22 in 256 teams 7.6 -> 5.7, 2^18 in
// 2048 29.0 -> 8.2; 64 teams 5.6 -> 5.9); a long one's end spread out, and there
// a second increment is a round trip more (2^28 in 256 teams 149.0 -> 149.4),
// short of a thousand teams (2048: 169.9 -> 162.2).
inline int32_t elect_groups(int teams, int64_t bytes) {
    return teams >= 1024 || (teams >= 128 && bytes <= ((int64_t)128 << 20));
}

// True if (dtype, op, vec_bytes, unroll) has a compiled reduce kernel.
bool reduce_variant_exists(int dtype, int op, int vec_bytes, int unroll);

// Plain reduction (team-block streaming + wave/LDS tree + last-team combine).
hipError_t launch_reduce(int dtype, int op, int vec_bytes, int unroll, const void* in,
                         int64_t n, void* x, int teams, int threads, const CrossTeamArgs& ct,
                         hipStream_t stream);

// Iteration map of a static schedule (threads = logical P, 1..1024).
hipError_t launch_static_map(int64_t n, int teams, int threads, int64_t dist_chunk,
                             int64_t chunk, int32_t* owner, uint32_t* count,
                             hipStream_t stream);

// The plain reduction (sum, max, min) with every thread reducing exactly its
// schedule(static) run of the team's block (exact.hip).
hipError_t launch_reduce_exact(int dtype, int op, const void* in, int64_t n, void* x, int teams,
                               int threads, const CrossTeamArgs& ct, hipStream_t stream);

// y <- fmaf(a, x, y) with the exact static mapping, fused compensated sum.
hipError_t launch_axpy_sum(float a, const float* x, float* y, float* sum, int64_t n,
                           int teams, int threads, int64_t dist_chunk, int64_t chunk,
                           const CrossTeamArgs& ct, hipStream_t stream);

// Empty target region over n iterations with reduction(+: iters) of one
// count per iteration (iters may be NULL); inconsistencies set status bit 16.
hipError_t launch_empty_region(int64_t n, int teams, int threads, int64_t dist_chunk,
                               int64_t chunk, int64_t* iters, const CrossTeamArgs& ct,
                               hipStream_t stream);

}  // namespace omprt
