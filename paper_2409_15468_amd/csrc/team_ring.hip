// The serving ring: a persistent launch that takes small solves from a ring of
// descriptors the host publishes while it runs (continuous batching), each
// solved by a team of workgroups (team_solve.hpp) of the shape the batched
// solver gives it, so that a request's result is the batched solver's, bit for
// bit; if other programs' work keeps a team from forming, the host solves the
// system like the batch does then.  (With one workgroup a request, a system of 16384 rows took 190 ms;
// with a team of 16, 16 ms.)
//
// A published system is G units, one per workgroup of its team, consecutive in
// the ring of units.  A workgroup claims the next published unit with a
// compare-and-swap on a device counter (so nothing is claimed before it is
// published), copies its rows' inputs from host memory into the system's device
// buffers, solves with the others, writes its rows of x back, and the team's
// last workgroup raises the slot's done word (system-scope release).  Units are
// claimed in order, so the earliest system whose team is not complete gets the
// next workgroups that come free, and workgroups ahead of it always come free:
// their teams are complete.
//
// The launch ends as one: a workgroup that sees the host's `stop`, that found
// nothing to claim for `idle_polls` polls, or that finds the launch older than
// `slice` ticks of the 100 MHz real-time counter (so that streams sharing its
// hardware queue are not held up for long) closes the counter, which is
// possible only where no system is partly claimed; then nothing is claimed any
// more and every workgroup leaves after the system it works on.  (Workgroups
// leaving one by one could leave a team that never completes.)  The host
// starts the next launch while work is pending.
//
// The descriptors, the inputs they point to (CSR, b, x0), the output x, the
// results and the control words live in host memory that is pinned, mapped and
// coherent.  Loads and stores of it are system-scope atomics, so they bypass
// the GPU caches: a staging area that held an earlier system's inputs is never
// read from a stale cache line.  Polls are relaxed (an acquire at system scope
// would invalidate the caches on every poll); the descriptor loads that follow
// a successful claim are issued only after the claim's result has been seen.
//
// Each slot has exchange words of its own, cleared once; a system's tags start
// above the last the slot's earlier systems used (which the result reports),
// so no word left there can be taken for one of this system.
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "cb_internal.hpp"
#include "ring_claim.hpp"
#include "team.hpp"
#include "team_solve.hpp"

namespace cb {

using namespace dev;

namespace {

constexpr int kRingUnits = 1 << 16;  // units published and unclaimed at most (a power of two)

struct RingDesc {
    TeamArgs a;
    const int32_t* h_row_ptr;
    const int32_t* h_col;
    const double* h_val;
    const double* h_b;
    const double* h_x0;
    double* h_x;
    uint64_t seq;
};

// The ring's control words: tail (units published) and stop in cache lines of
// their own, then per slot the done word (sequence number + 1 once the slot's
// result is final) and the launch that served it, and the units (slot | rank << 16).
struct RingCtl {
    unsigned tail;
    unsigned pad0[31];
    unsigned stop;
    unsigned pad1[31];
    unsigned done[kRingSlots];
    unsigned served_by[kRingSlots];
    unsigned units[kRingUnits];
};

template <class T>
__device__ __forceinline__ T ld_sys(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// host memory -> device memory
template <class T>
__device__ __forceinline__ void copy_in(const T* __restrict__ src, T* __restrict__ dst, int64_t i0, int64_t i1) {
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kTeamThreads) dst[i] = ld_sys(src + i);
}

struct ClaimMemory {
    const RingCtl* ctl;
    uint64_t* h;
    __device__ __forceinline__ uint64_t head() const {
        const uint64_t v = ld_ctl(h);
        __builtin_amdgcn_s_waitcnt(0);  // the tail's load goes out after this one's value is here
        return v;
    }
    __device__ __forceinline__ uint32_t tail() const { return ld_sys(&ctl->tail); }
    __device__ __forceinline__ uint32_t unit(uint32_t i) const { return ld_sys(&ctl->units[i & (kRingUnits - 1)]); }
    __device__ __forceinline__ bool stop() const { return ld_sys(&ctl->stop) != 0; }
    __device__ __forceinline__ bool cas(uint64_t from, uint64_t to) const {
        return atomicCAS(reinterpret_cast<unsigned long long*>(h), from, to) == from;
    }
};

// The next unit (slot | rank << 16), or -1 once the launch is closed.
__device__ int claim(const RingCtl* ctl, uint64_t* head, int idle_polls, uint64_t t_start, uint64_t slice) {
    ClaimMemory m{ctl, head};
    for (int idle = 0;;) {
        const bool late = __builtin_amdgcn_s_memrealtime() - t_start >= slice;
        const int r = claim_step(m, late, idle >= idle_polls);
        if (r >= 0 || r == kClaimClosed) return r;
        if (r == kClaimAgain) continue;  // look again at once
        __builtin_amdgcn_s_sleep(127);  // ~8k cycles between polls of the bus
        ++idle;
    }
}

// The solve as a function of its own: inlined six times into the claim loop, it
// spills 800 registers; called, none.  (The shared memory has a fixed address.)
__shared__ TeamShared S;
template <int FMT>
__device__ __attribute__((noinline)) void ring_solve(int rank) {
    team_solve<FMT, kSlotsOf<FMT>>(rank, S);
}

__global__ void k_ring_open(uint64_t* head) { *head = ld_ctl(head) & ~kRingClosed; }

__global__ __launch_bounds__(kTeamThreads, 2) void k_team_ring(const RingDesc* __restrict__ descs, RingCtl* ctl,
                                                               uint64_t* head, unsigned* arrived, int idle_polls,
                                                               uint64_t slice, uint32_t launch_id) {
    __shared__ int unit;
    __shared__ RingDesc D;
    const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
    for (;;) {
        if (threadIdx.x == 0) unit = claim(ctl, head, idle_polls, t_start, slice);
        __syncthreads();
        const int u = uniform(unit);
        if (u < 0) return;
        const int slot = u & 0xFFFF, rank = u >> 16;
        // this CU's first-level cache may still hold lines of an earlier system
        // that used the same device memory: drop them
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        static_assert(sizeof(RingDesc) % 8 == 0, "descriptor size");
        if (threadIdx.x < sizeof(RingDesc) / 8)
            reinterpret_cast<uint64_t*>(&D)[threadIdx.x] =
                ld_sys(reinterpret_cast<const uint64_t*>(descs + slot) + threadIdx.x);
        __syncthreads();
        if (threadIdx.x == 0) S.args = D.a;
        // the inputs of this workgroup's rows into the device buffers (x0 into x)
        const int64_t rows = (int64_t)(kTW / D.a.cs) * kTile;
        const int64_t r0 = min((int64_t)rank * rows, (int64_t)D.a.n), r1 = min(r0 + rows, (int64_t)D.a.n);
        copy_in(D.h_row_ptr, const_cast<int32_t*>(D.a.rp), r0, r1 + 1);
        const int64_t k0 = ld_sys(D.h_row_ptr + r0), k1 = ld_sys(D.h_row_ptr + r1);
        copy_in(D.h_col, const_cast<int32_t*>(D.a.ci), k0, k1);
        copy_in(D.h_val, const_cast<double*>(D.a.val), k0, k1);
        copy_in(D.h_b, const_cast<double*>(D.a.b), r0, r1);
        for (int64_t i = r0 + threadIdx.x; i < r1; i += kTeamThreads)
            __hip_atomic_store(D.a.x + i, ld_sys(D.h_x0 + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        switch (uniform(S.args.format)) {
        case CB_F64: ring_solve<CB_F64>(rank); break;
        case CB_F32: ring_solve<CB_F32>(rank); break;
        case CB_F16: ring_solve<CB_F16>(rank); break;
        case CB_FRSZ2_16: ring_solve<CB_FRSZ2_16>(rank); break;
        case CB_FRSZ2_21: ring_solve<CB_FRSZ2_21>(rank); break;
        default: ring_solve<CB_FRSZ2_32>(rank); break;
        }
        __builtin_amdgcn_s_waitcnt(0);  // this wave's rows of x are in place
        __syncthreads();
        for (int64_t i = r0 + threadIdx.x; i < r1; i += kTeamThreads)
            __hip_atomic_store(D.h_x + i, ld_ctl(D.a.x + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");  // this thread's writes, system scope
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned n = __hip_atomic_fetch_add(&arrived[slot], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (n == (unsigned)D.a.G - 1u) {
                __hip_atomic_store(&arrived[slot], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(D.a.join, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&ctl->served_by[slot], launch_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(&ctl->done[slot], (unsigned)D.seq + 1u, __ATOMIC_RELEASE,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        __syncthreads();  // D and S are free for the next unit
    }
}

}  // namespace

struct BatchRing {
    unsigned char* host = nullptr;  // pinned, mapped, coherent: RingCtl, descriptors, results
    RingCtl* ctl = nullptr;
    RingDesc* descs = nullptr;
    State* results = nullptr;
    RingCtl* ctl_dev = nullptr;
    RingDesc* descs_dev = nullptr;
    State* results_dev = nullptr;
    unsigned char* mem = nullptr;   // device: claim counter, whole teams, arrivals per slot, exchange words per slot
    uint64_t* head = nullptr;
    unsigned* busy = nullptr;
    unsigned* arrived = nullptr;
    uint64_t* ll = nullptr;
    int64_t ll_words = 0;           // per slot
    hipEvent_t ended = nullptr;     // recorded after each launch
    bool launched = false;
    uint32_t published = 0;         // units
    uint32_t next_seq = 0;
    uint32_t launches = 0;
    std::vector<int> free_slots;
    std::vector<uint32_t> epoch;    // last tag used per slot
    std::vector<uint32_t> seq_of;   // per slot
    std::unique_ptr<TeamSeats> seats;
    int grid = 0, cap = 0, idle_polls = 4096;
    uint64_t slice = 0;             // real-time counter ticks (100 MHz)
};

BatchRing* ring_create(int grid, int idle_polls, double slice_s) {
    std::unique_ptr<BatchRing> r(new BatchRing());
    r->cap = team_device_groups();
    r->grid = grid < r->cap ? grid : r->cap;
    const TeamShape largest = team_batch_shape(kRingMaxN);
    if (r->grid < largest.G) {
        set_error("a device of %d CUs does not hold a team of %d workgroups", r->cap, largest.G);
        return nullptr;
    }
    r->idle_polls = idle_polls;
    r->slice = (uint64_t)(slice_s * 1e8);
    for (int i = kRingSlots; i-- > 0;) r->free_slots.push_back(i);
    r->epoch.assign(kRingSlots, 0);
    r->seq_of.assign(kRingSlots, 0);
    const size_t o_desc = (sizeof(RingCtl) + 255) & ~size_t(255);
    const size_t o_res = o_desc + ((kRingSlots * sizeof(RingDesc) + 255) & ~size_t(255));
    const size_t total = o_res + kRingSlots * sizeof(State);
    r->ll_words = team_ll_words(largest.G, kBatchMaxRestart);
    const int64_t words = 32 + kRingSlots / 2 + kRingSlots * r->ll_words;
    void* h = nullptr;
    void* dptr = nullptr;
    if (hipHostMalloc(&h, total, hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess) return nullptr;
    std::memset(h, 0, total);
    r->host = static_cast<unsigned char*>(h);
    if (hipHostGetDevicePointer(&dptr, h, 0) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&r->mem), (size_t)words * 8) != hipSuccess ||
        hipMemset(r->mem, 0, (size_t)words * 8) != hipSuccess ||
        hipEventCreateWithFlags(&r->ended, hipEventDisableTiming) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {
        ring_destroy(r.release());
        return nullptr;
    }
    r->head = reinterpret_cast<uint64_t*>(r->mem);
    r->busy = reinterpret_cast<unsigned*>(r->mem + 128);
    r->arrived = reinterpret_cast<unsigned*>(r->mem + 256);
    r->ll = reinterpret_cast<uint64_t*>(r->mem) + 32 + kRingSlots / 2;
    unsigned char* d = static_cast<unsigned char*>(dptr);
    r->ctl = reinterpret_cast<RingCtl*>(r->host);
    r->descs = reinterpret_cast<RingDesc*>(r->host + o_desc);
    r->results = reinterpret_cast<State*>(r->host + o_res);
    r->ctl_dev = reinterpret_cast<RingCtl*>(d);
    r->descs_dev = reinterpret_cast<RingDesc*>(d + o_desc);
    r->results_dev = reinterpret_cast<State*>(d + o_res);
    return r.release();
}

int ring_publish(BatchRing* r, const cb_batch_item& q, const int32_t* h_row_ptr, const int32_t* h_col,
                 const double* h_val, const double* h_b, const double* h_x0, double* h_x, uint32_t* seq) {
    if (q.A.n < 1 || q.A.n > kRingMaxN || q.A.nnz < 0 || q.m < 1 || q.m > kBatchMaxRestart ||
        !(q.tol > 0.0) || !batch_format(q.format) || !q.b || !q.x || !q.workspace || !q.A.row_ptr ||
        (q.A.nnz > 0 && (!q.A.col || !q.A.val)) || !h_row_ptr || !h_b || !h_x0 || !h_x ||
        (q.A.nnz > 0 && (!h_col || !h_val)) || !aligned(q.x, 16) || !aligned(q.b, 16) ||
        !aligned(q.workspace, 256) || (int64_t)q.workspace_bytes < batch_workspace_bytes(q.A.n, q.m, q.format))
        return fail(CB_ERR_INVALID_ARG, "ring: bad system");
    if (r->free_slots.empty()) return fail(CB_ERR_WORKSPACE, "ring: all %d slots busy", kRingSlots);
    const int slot = r->free_slots.back();
    uint64_t* ll = r->ll + slot * r->ll_words;
    if (r->epoch[slot] > UINT32_MAX / 2) {  // the tags would run out: clear the slot's words
        if (hipMemset(ll, 0, (size_t)r->ll_words * 8) != hipSuccess || hipDeviceSynchronize() != hipSuccess)
            return fail(CB_ERR_HIP, "ring: clearing a slot failed");
        r->epoch[slot] = 0;
    }
    RingDesc d{};
    d.a = team_batch_args(q);
    d.a.eta = kDefaultEta;
    d.a.max_iters = kDefaultMaxIters;
    team_exchange(d.a, ll);
    d.a.st = r->results_dev + slot;
    d.a.wait_us = team_wait_us();
    d.a.poll_ticks = team_poll_ticks();
    d.a.busy = r->busy;
    d.a.epoch0 = r->epoch[slot];
    d.h_row_ptr = h_row_ptr;
    d.h_col = h_col;
    d.h_val = h_val;
    d.h_b = h_b;
    d.h_x0 = h_x0;
    d.h_x = h_x;
    const uint32_t s = r->next_seq++;
    d.seq = s;
    r->free_slots.pop_back();
    r->seq_of[slot] = s;
    r->descs[slot] = d;
    std::memset(&r->results[slot], 0, sizeof(State));
    __atomic_store_n(&r->ctl->done[slot], 0u, __ATOMIC_RELAXED);
    for (int g = 0; g < d.a.G; ++g)
        r->ctl->units[(r->published + (uint32_t)g) & (kRingUnits - 1)] = (unsigned)slot | (unsigned)g << 16;
    r->published += (uint32_t)d.a.G;
    __atomic_store_n(&r->ctl->tail, r->published, __ATOMIC_RELEASE);  // the descriptor and units before the count
    *seq = (uint32_t)slot;
    return CB_OK;
}

bool ring_poll(BatchRing* r, uint32_t seq, cb_result* res, uint32_t* launch, bool* solved) {
    const int slot = (int)seq;
    if (__atomic_load_n(&r->ctl->done[slot], __ATOMIC_ACQUIRE) != r->seq_of[slot] + 1u) return false;
    const State& st = r->results[slot];
    team_waited(st.status != kTeamAbandoned);
    *solved = st.status != kTeamAbandoned && st.status != kTeamLost;
    if (res) fill_result(res, st, 0.0);
    // (a lost team may have used tags past those its first workgroup reports, one
    // that never formed has used none)
    if (st.status == kTeamLost) r->epoch[slot] = UINT32_MAX;
    else if (st.status != kTeamAbandoned) r->epoch[slot] = (uint32_t)st.pad0;
    if (launch) *launch = r->ctl->served_by[slot];
    r->free_slots.push_back(slot);
    return true;
}

bool ring_running(BatchRing* r) {
    if (r->launched && hipEventQuery(r->ended) == hipErrorNotReady) return true;
    if (r->launched) r->seats.reset();  // the launch has ended: its CUs are free
    r->launched = false;
    return false;
}

void ring_idle(BatchRing* r) {
    if (ring_running(r) && r->seats && r->seats->wanted()) __atomic_store_n(&r->ctl->stop, 1u, __ATOMIC_RELEASE);
}

uint32_t ring_kick(BatchRing* r, hipStream_t s, int* status) {
    *status = CB_OK;
    if (ring_running(r)) return 0;
    if (!r->seats) r->seats.reset(new TeamSeats(r->grid, r->cap));
    if (!r->seats->ready()) return 0;  // not its turn yet
    const uint32_t id = ++r->launches;
    __atomic_store_n(&r->ctl->stop, 0u, __ATOMIC_RELEASE);
    k_ring_open<<<1, 1, 0, s>>>(r->head);
    k_team_ring<<<r->grid, kTeamThreads, 0, s>>>(r->descs_dev, r->ctl_dev, r->head, r->arrived, r->idle_polls,
                                                  r->slice, id);
    if (hipGetLastError() != hipSuccess || hipEventRecord(r->ended, s) != hipSuccess) {
        (void)hipStreamSynchronize(s);  // whatever did start has ended
        r->seats.reset();
        *status = fail(CB_ERR_HIP, "ring launch failed");
        return 0;
    }
    r->launched = true;
    return id;
}

void ring_stop(BatchRing* r) {
    __atomic_store_n(&r->ctl->stop, 1u, __ATOMIC_RELEASE);
    if (r->launched) (void)hipEventSynchronize(r->ended);
    r->launched = false;
    r->seats.reset();
    __atomic_store_n(&r->ctl->stop, 0u, __ATOMIC_RELEASE);
}

void ring_destroy(BatchRing* r) {
    if (!r) return;
    if (r->ctl) ring_stop(r);
    if (r->ended) (void)hipEventDestroy(r->ended);
    if (r->mem) (void)hipFree(r->mem);
    if (r->host) (void)hipHostFree(r->host);
    delete r;
}

}  // namespace cb
