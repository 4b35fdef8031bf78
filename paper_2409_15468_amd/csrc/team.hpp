// Whole solves by a team of resident workgroups (team.hip).
#pragma once

#include "cb_internal.hpp"

namespace cb {

constexpr int kTeamThreads = 512;
constexpr int kTeamMaxRestart = 104;  // R, the rotations and the sums of a step sit in LDS
constexpr int kTeamMaxGroups = 256;   // one workgroup per CU
// State::status of a solve whose workgroups did not come together: nothing but
// this word has been written
constexpr int kTeamAbandoned = -1;
// ... and of one in which a workgroup that had come was not heard of for kTeamPollUs
// (its queue was taken off the GPU): x holds each row before or after the last
// cycle's update, the counters are those of the cycles before
constexpr int kTeamLost = -2;
// How long a team may take to come together before its solve goes the other way.
// Kernels of the process's other streams end (the longest of this library take
// milliseconds), and waiting for them keeps a result independent of them; what
// never ends, a resident kernel of another program, should not cost every
// solve that time.  So each team in a row that does not form cuts the next
// one's wait to a quarter, down to kTeamWaitLeastUs, for the host thread whose
// solves they are, and one that forms restores it.
constexpr int32_t kTeamWaitUs = 500000;
constexpr int32_t kTeamWaitLeastUs = 2000;
constexpr int32_t kTeamPollUs = 20000000;
constexpr int kJoinWords = 16;  // ahead of the exchange slots, in a line of its own

struct State;

struct TeamArgs {
    const int32_t* rp;
    const int32_t* ci;
    const double* val;   // A
    const double* aval;  // the operator of the Arnoldi steps: A, or A M^-1
    const double* b;
    double* x;
    const double* dinv;  // Jacobi preconditioner, or NULL
    BasisView V;
    double* w;           // n doubles: the vector the next SpMV reads
    uint64_t* ll;        // exchange slots
    unsigned* join;      // workgroups that have come; top bit: the team does not form
    unsigned* busy;      // NULL, or the teams of this launch that are whole: while there are any, others
                         // wait for their workgroups
    double* x0;          // NULL, or n doubles that get x as it was on entry
    State* st;
    double* hist;        // NULL, or |g_{j+1}| per step of this launch
    double tol, eta;
    int64_t col_total;   // bytes of a column with its exponents
    uint64_t poll_ticks; // a whole team's exchange takes this long at most (100 MHz)
    int32_t n, m, G, cs;
    int32_t max_iters, max_cycles, literal;
    int32_t hist_cap;    // entries of hist; the launch ends when a cycle may not fit
    int32_t resume;      // the counters continue from *st
    int32_t batch;       // one of many systems: what the batch does and counts where it differs
    int32_t format;      // basis format (launches of many systems)
    int32_t wait_us;     // the team's workgroups come within this time or not at all (0: not at all)
    uint32_t epoch0;     // tags of this solve are above it; the slots hold none that are
};

struct TeamShape {
    int G, cs;  // workgroups, waves per 512-row tile
};

// Workgroups a team may have on the current device (0: no teams).
int team_device_groups();
// ... for work on stream s: 0 if it may not use all CUs (a CU mask), since a team
// needs the CUs it counts on.
int team_stream_groups(hipStream_t s);
// The team for n rows and restart length m; false if it does not fit.
bool team_shape(int32_t n, int32_t m, int capacity, TeamShape* s);
int64_t team_ll_words(int G, int m);
// a.join and a.ll in team_ll_words words at p.
inline void team_exchange(TeamArgs& a, uint64_t* p) {
    a.join = reinterpret_cast<unsigned*>(p);
    a.ll = p + kJoinWords;
}
// The wait of this host thread's next launch: by kTeamWaitUs, or what
// cb_internal_team_wait has set; and what came of one.
int32_t team_wait_us();
void team_waited(bool formed);
int32_t team_wait_setting();
// kTeamPollUs, or what cb_internal_team_poll has set for this host thread.
int32_t team_poll_us();
inline uint64_t team_poll_ticks() { return (uint64_t)team_poll_us() * 100u; }
// Clear the words at a.join and start the team on stream s.
void launch_team(int fmt, const TeamArgs& a, hipStream_t s);
// The team for one of many systems; depends on its rows only.
TeamShape team_batch_shape(int32_t n);
// Its arguments but for ll, st, eta, max_iters and literal.
TeamArgs team_batch_args(const cb_batch_item& q);
void launch_team_clear(uint64_t* ll, int64_t words, hipStream_t s);
// One launch of `groups` workgroups, at least the largest team, that take the
// `count` units in order (args and units on the device; *next, the busy word and
// the exchange words clear).
void launch_team_many(const TeamArgs* args, const uint64_t* units, unsigned count, unsigned* next, int groups,
                      hipStream_t s);

// The statistics of a solve as the caller gets them.
void fill_result(cb_result* res, const State& hs, double seconds);

// CUs reserved for a team's workgroups while it runs, in arrival order.
class TeamSeats {
public:
    TeamSeats(int groups, int capacity);  // joins the queue
    ~TeamSeats();                         // leaves it, or gives the CUs back
    bool ready();                         // true once the CUs are reserved
    void wait();
    bool wanted() const;                  // others queue behind these seats
    TeamSeats(const TeamSeats&) = delete;
    TeamSeats& operator=(const TeamSeats&) = delete;

private:
    int dev_ = 0, groups_, capacity_;
    uint64_t ticket_ = 0;
    bool seated_ = false;
};

}  // namespace cb

extern "C" void cb_internal_team_wait(int32_t us, int32_t launches);
extern "C" void cb_internal_team_poll(int32_t us);
