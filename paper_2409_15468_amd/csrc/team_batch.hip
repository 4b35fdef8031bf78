// Many small systems per launch, a team of workgroups each (team_solve.hpp):
// the batched solver's main path.
//
// A system is G units, one per workgroup of its team, consecutive in the list of
// units; a workgroup takes the next unit from an atomic ticket when it has
// finished one.  Units are taken in order, so at most the last system begun has
// an incomplete team, and the workgroups of all others, which finish, complete
// it.  (Launches of as many whole teams as fit, one after the other, each waited
// for its slowest system: 2560 systems of 400 rows of which every 256th runs 2000
// steps took 267 ms, now 40; one workgroup per system 98.)
//
// One workgroup per system (batch.hip) left most of the GPU idle behind the
// largest one: 48 systems of 1024 to 16384 rows took 190 ms, as long as the
// largest alone; by teams 29 ms.  A team takes 1024 rows a workgroup (cs = 4): at n = 16384
// a step is 26 us with 16 workgroups, 19 us with 32 (cs = 8), 43 us with 8 (cs =
// 2), so cs = 4 serves 1.5 times as many rows per second and CU as cs = 8 and
// keeps the largest system's time near its best.  The shape depends on the
// system's rows only, so its result does not depend on the rest of the batch.
#include "cb_internal.hpp"
#include "team.hpp"
#include "team_solve.hpp"

namespace cb {

using namespace dev;

// The solve as a function of its own: inlined for six formats into one kernel it
// spills 130 registers.  (The shared memory has a fixed address.)
static __shared__ TeamShared S;
template <int FMT>
static __device__ __attribute__((noinline)) void solve_one(int rank) {
    team_solve<FMT, kSlotsOf<FMT>>(rank, S);
}

// Unit i is workgroup units[i] >> 32 of the team that solves system
// (uint32_t)units[i].  *next reads 0 at launch.
__global__ __launch_bounds__(kTeamThreads, 2) void k_team_many(const TeamArgs* __restrict__ args,
                                                               const uint64_t* __restrict__ units, unsigned count,
                                                               unsigned* next) {
    __shared__ unsigned at;
    for (;;) {
        if (threadIdx.x == 0) at = atomicAdd(next, 1u);
        __syncthreads();
        const unsigned i = uniform(at);
        if (i >= count) return;
        const uint64_t who = uniform(ld_ctl(units + i));
        static_assert(sizeof(TeamArgs) % 8 == 0 && sizeof(TeamArgs) / 8 <= 64, "copied by one wave");
        if (threadIdx.x < sizeof(TeamArgs) / 8)
            reinterpret_cast<uint64_t*>(&S.args)[threadIdx.x] =
                ld_ctl(reinterpret_cast<const uint64_t*>(args + (uint32_t)who) + threadIdx.x);
        __syncthreads();
        const int rank = (int)(who >> 32);
        switch (uniform(S.args.format)) {
        case CB_F64: solve_one<CB_F64>(rank); break;
        case CB_F32: solve_one<CB_F32>(rank); break;
        case CB_F16: solve_one<CB_F16>(rank); break;
        case CB_FRSZ2_16: solve_one<CB_FRSZ2_16>(rank); break;
        case CB_FRSZ2_21: solve_one<CB_FRSZ2_21>(rank); break;
        default: solve_one<CB_FRSZ2_32>(rank); break;
        }
        __syncthreads();  // S is free for the next unit
    }
}

TeamShape team_batch_shape(int32_t n) {
    const int tiles = (int)((padded_rows(n) + kTile - 1) / kTile);
    const int cs = tiles > 1 ? 4 : 8;
    return {(tiles + 8 / cs - 1) / (8 / cs), cs};
}

void launch_team_many(const TeamArgs* args, const uint64_t* units, unsigned count, unsigned* next, int groups,
                      hipStream_t s) {
    k_team_many<<<groups, kTeamThreads, 0, s>>>(args, units, count, next);
}

}  // namespace cb
