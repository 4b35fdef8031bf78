// Launches of team solves (team_solve.hpp): one system per launch, and the
// ledger that keeps the teams in flight within the GPU's CUs.
#include <condition_variable>
#include <mutex>

#include "cb_internal.hpp"
#include "team.hpp"
#include "team_solve.hpp"

namespace cb {

using namespace dev;

namespace {

template <int FMT, int N>
__global__ __launch_bounds__(kTeamThreads, 2) void k_team(TeamArgs a) {
    __shared__ TeamShared S;
    if (threadIdx.x == 0) S.args = a;
    __syncthreads();
    team_solve<FMT, N>(blockIdx.x, S);
}

__global__ void k_team_clear(uint64_t* __restrict__ ll, int64_t words) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) ll[i] = 0;
}

// The CUs that team workgroups of this process occupy, per device, in arrival
// order: a solve waits until its whole team fits, so two teams never hold parts of
// the GPU that the other needs to become whole (seats_of).
constexpr int kLedgerDevices = 16;
struct Ledger {
    std::mutex mu;
    std::condition_variable cv;
    uint64_t next = 0, serving = 0;
    int used = 0;
};
Ledger g_ledger[kLedgerDevices];

}  // namespace

int team_device_groups() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kLedgerDevices ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return cus < kTeamMaxGroups ? cus : kTeamMaxGroups;
}

int team_stream_groups(hipStream_t s) {
    const int cap = team_device_groups();
    int dev = 0, cus = 0;
    uint32_t mask[32] = {};
    if (!s || s == hipStreamLegacy || s == hipStreamPerThread || cap == 0 || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return cap;
    if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return cap;
    }
    int enabled = 0;
    for (uint32_t w : mask) enabled += __builtin_popcount(w);
    return enabled < cus ? 0 : cap;
}

// Workgroup w of a launch runs on XCD w % kXcds whatever else runs there, so a
// team of 9 takes two CUs of the first: seats are counted in rows of one per XCD.
static int seats_of(int groups, int capacity) {
    const int rows = (groups + kXcds - 1) / kXcds;
    return rows * kXcds < capacity ? rows * kXcds : capacity;
}

TeamSeats::TeamSeats(int groups, int capacity) : groups_(seats_of(groups, capacity)), capacity_(capacity) {
    if (hipGetDevice(&dev_) != hipSuccess || dev_ < 0 || dev_ >= kLedgerDevices) dev_ = 0;
    std::lock_guard<std::mutex> lk(g_ledger[dev_].mu);
    ticket_ = g_ledger[dev_].next++;
}
bool TeamSeats::ready() {
    Ledger& L = g_ledger[dev_];
    std::lock_guard<std::mutex> lk(L.mu);
    if (!seated_ && L.serving == ticket_ && L.used + groups_ <= capacity_) {
        seated_ = true;
        L.serving += 1;
        L.used += groups_;
        L.cv.notify_all();
    }
    return seated_;
}
void TeamSeats::wait() {
    Ledger& L = g_ledger[dev_];
    {
        std::unique_lock<std::mutex> lk(L.mu);
        L.cv.wait(lk, [&] { return L.serving == ticket_ && L.used + groups_ <= capacity_; });
    }
    ready();
}
bool TeamSeats::wanted() const {
    Ledger& L = g_ledger[dev_];
    std::lock_guard<std::mutex> lk(L.mu);
    return seated_ && L.serving != L.next;
}
TeamSeats::~TeamSeats() {
    if (!seated_) wait();  // a ticket is used up in its turn
    Ledger& L = g_ledger[dev_];
    {
        std::lock_guard<std::mutex> lk(L.mu);
        L.used -= groups_;
    }
    L.cv.notify_all();
}

bool team_shape(int32_t n, int32_t m, int capacity, TeamShape* s) {
    if (m > kTeamMaxRestart || capacity < 1) return false;
    const int64_t tiles = (padded_rows(n) + kTile - 1) / kTile;
    // At least two waves to a tile (half a million rows on 256 CUs).  With one, a
    // wave walks all columns of its tile as the launch-per-kernel path's do: at n =
    // 10^6 a solve alone took 68.9 -> 65.9 ms (frsz2_32), 48.9 -> 44.9 (frsz2_16)
    // and 105 -> 95 (float64), but it holds every CU for that long, and what a team
    // gains alone it loses beside others (four host threads' solves of 493,000
    // rows, frsz2_32: 13.0 ms each by teams, 9.0 by launches).
    for (int cs = 8; cs >= 2; cs /= 2) {
        const int64_t G = (tiles + 8 / cs - 1) / (8 / cs);
        if (G <= capacity) {
            s->cs = cs;
            s->G = (int)G;
            return true;
        }
    }
    return false;
}

int64_t team_ll_words(int G, int m) {
    return kJoinWords + (G <= kDirect ? (int64_t)4 * G * (m + 2) : (int64_t)2 * (G + 1) * (m + 2));
}

static thread_local int32_t g_wait_us = -1, g_wait_skip = 0, g_missed = 0, g_poll_us = -1;
int32_t team_poll_us() { return g_poll_us < 0 ? kTeamPollUs : g_poll_us; }
int32_t team_wait_setting() { return g_wait_us; }
int32_t team_wait_us() {
    if (g_wait_us >= 0 && g_wait_skip-- <= 0) return g_wait_us;
    const int32_t us = kTeamWaitUs >> 2 * g_missed;
    return us > kTeamWaitLeastUs ? us : kTeamWaitLeastUs;
}
void team_waited(bool formed) { g_missed = formed ? 0 : g_missed < 8 ? g_missed + 1 : 8; }

void launch_team_clear(uint64_t* ll, int64_t words, hipStream_t s) {
    k_team_clear<<<(unsigned)((words + 255) / 256), 256, 0, s>>>(ll, words);
}

void launch_team(int fmt, const TeamArgs& a, hipStream_t s) {
    launch_team_clear(reinterpret_cast<uint64_t*>(a.join), team_ll_words(a.G, a.m), s);
#define CB_TEAM_CASE(F)                                                                    \
    case F:                                                                                \
        if (a.cs >= 4) k_team<F, kSlotsOf<F>><<<a.G, kTeamThreads, 0, s>>>(a);              \
        else k_team<F, 0><<<a.G, kTeamThreads, 0, s>>>(a);                                 \
        break;
    switch (kernel_format(fmt)) {
        CB_TEAM_CASE(CB_F64)
        CB_TEAM_CASE(CB_F32)
        CB_TEAM_CASE(CB_F16)
        CB_TEAM_CASE(CB_FRSZ2_16)
        CB_TEAM_CASE(CB_FRSZ2_21)
        CB_TEAM_CASE(CB_FRSZ2_GEN)
        CB_TEAM_CASE(CB_FRSZ2_16_B64)
        CB_TEAM_CASE(CB_FRSZ2_32_B64)
        default:
        CB_TEAM_CASE(CB_FRSZ2_32)
    }
#undef CB_TEAM_CASE
}

}  // namespace cb

// (for tests) The wait after a team that formed or did not.
extern "C" int32_t cb_internal_team_waited(int32_t formed) {
    cb::team_waited(formed != 0);
    return cb::team_wait_us();
}
extern "C" int32_t cb_internal_team_seats(int32_t groups, int32_t capacity) { return cb::seats_of(groups, capacity); }

// How long the teams of this host thread's solves wait for their workgroups, in
// microseconds (negative: the default), from the launch after the next
// `launches` on.  With 0 no team forms, and the tests reach the paths that solve
// such systems.
extern "C" void cb_internal_team_wait(int32_t us, int32_t launches) {
    cb::g_wait_us = us;
    cb::g_wait_skip = launches;
}

// The limit of an exchange in the launches of this host thread, in microseconds
// (negative: the default).  With 0 a team whose workgroups wait for one that is
// slower by some hundred polls is lost, and the tests reach what follows.
extern "C" void cb_internal_team_poll(int32_t us) { cb::g_poll_us = us; }
