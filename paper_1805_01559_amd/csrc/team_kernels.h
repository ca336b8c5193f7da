// The instances of a batch as teams: the cooperative phase of a single solve
// (persist_kernels.h), run for many instances by one launch that fills the
// GPU with one workgroup per CU. Each instance belongs to a team of as many
// workgroups as its stabilised kernel needs LDS for, which solves it to the
// end (iterations, exact check) or to the launch's cap of iterations before its
// members go on to their next one.
// The host assigns teams (longest first, each to the workgroups with the
// least work so far) and gives every workgroup its list of (instance, rank).
// The lists follow one order of all instances, so the first unfinished
// instance always has every member free of earlier ones, and no set of teams
// can wait in a circle. An instance's team size and row split follow from its
// own I and J, and no sum depends on which workgroup has which rank: results
// are bitwise independent of the rest of the batch.
//
// Why: a batch's sweeps read every cost once per iteration and recompute its
// exponentials (0.73 GB and 265 us per iteration for 256 uneven instances,
// about 100 iterations until the slowest ends); a team reads its cost three
// times in all: 16.8 -> 13.7 ms with their plans, 6.8 ms of them this kernel. What
// bounds it: the exchange and the rows, 3 and 2 to 3 of 5.5 - 7 us per iteration,
// while a CU's LDS is taken.
#pragma once

#include "persist_kernels.h"

namespace otk {

// Lanes per row and cells per lane by class: up to 64, 128, 256 and 512 columns.
// One more (13 cells for up to 416 columns) saved less in the row sums, a quarter
// of an iteration, than it cost in registers.
__host__ __device__ constexpr int team_class(int J) { return J <= 64 ? 0 : J <= 128 ? 1 : J <= 256 ? 2 : 3; }
__host__ __device__ constexpr int team_lpr(int cls) { return cls == 0 ? 16 : 32; }
__host__ __device__ constexpr int team_cpl(int cls) { return cls <= 1 ? 4 : cls == 2 ? 8 : 16; }
__host__ __device__ constexpr int team_rows(int cls) { return 8 * kWave / team_lpr(cls); }  // of a workgroup's step

struct TeamJob {
    PersistArgs A;
    DenseSrc<float> src;
    int nb;
    int cls;
};

// Zeroes the exchange blocks of a launch (a zero slot carries the tag of no
// first iteration: every launch starts an instance at a multiple of 4).
static __global__ __launch_bounds__(256) void k_team_clear(const TeamJob* jobs) {
    const TeamJob& J = jobs[blockIdx.y];
    const size_t n = persist_exchange_doubles(J.nb, J.A.J);
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x)
        J.A.xch[q] = 0.0;
}

// items[start[b]] .. items[start[b + 1] - 1]: workgroup b's instances and its rank in their teams.
static __global__ __launch_bounds__(512) void k_team(const TeamJob* __restrict__ jobs, const int2* __restrict__ items,
                                                     const int* __restrict__ start) {
    __shared__ PersistShared ps;
    const int q1 = __builtin_amdgcn_readfirstlane(start[blockIdx.x + 1]);
    for (int q = __builtin_amdgcn_readfirstlane(start[blockIdx.x]); q < q1; ++q) {
        const int2 it{__builtin_amdgcn_readfirstlane(items[q].x), __builtin_amdgcn_readfirstlane(items[q].y)};
        // (word by word through the first lane: the same for all lanes, so it
        // belongs in scalar registers)
        TeamJob J;
        static_assert(sizeof(TeamJob) % 4 == 0, "copied word by word");
        const int* from = reinterpret_cast<const int*>(jobs + it.x);
#pragma unroll
        for (int u = 0; u < (int)(sizeof(TeamJob) / 4); ++u) {
            int v = __builtin_amdgcn_readfirstlane(from[u]);
            asm volatile("" : "+s"(v));  // (now, not at each use)
            reinterpret_cast<int*>(&J)[u] = v;
        }
        using S = DenseSrc<float>;
        switch (J.cls) {
            case 0: persist_run<S, team_cpl(0), team_lpr(0), 8, false, true>(J.A, J.src, J.nb, it.y, ps); break;
            case 1: persist_run<S, team_cpl(1), team_lpr(1), 8, false, true>(J.A, J.src, J.nb, it.y, ps); break;
            case 2: persist_run<S, team_cpl(2), team_lpr(2), 8, false, true>(J.A, J.src, J.nb, it.y, ps); break;
            default: persist_run<S, team_cpl(3), team_lpr(3), 8, false, true>(J.A, J.src, J.nb, it.y, ps); break;
        }
        __syncthreads();  // LDS is the next instance's
    }
}

}  // namespace otk
