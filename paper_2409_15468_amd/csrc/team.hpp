// Whole solves by a team of resident workgroups (team.hip).
#pragma once

#include "cb_internal.hpp"

namespace cb {

constexpr int kTeamThreads = 512;
constexpr int kTeamMaxRestart = 104;  // R, the rotations and the sums of a step sit in LDS
constexpr int kTeamMaxGroups = 256;   // one workgroup per CU
// State::status of a solve whose workgroups did not find each other in time
constexpr int kTeamAbandoned = -1;

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
    uint64_t* ll;        // exchange slots, team_ll_words of them
    State* st;
    double* hist;        // NULL, or |g_{j+1}| per step of this launch
    double tol, eta;
    int64_t col_total;   // bytes of a column with its exponents
    int32_t n, m, G, cs;
    int32_t max_iters, max_cycles, literal;
    int32_t hist_cap;    // entries of hist; the launch ends when a cycle may not fit
    int32_t resume;      // the counters continue from *st
    int32_t format;      // basis format (launches of many systems)
    int32_t patience;    // 2 s units a poll waits before the solve is abandoned (0: one)
    uint32_t epoch0;     // tags of this solve are above it; the slots hold none that are
};

struct TeamShape {
    int G, cs;  // workgroups, waves per 512-row tile
};

// Workgroups a team may have on the current device (0: no teams).
int team_device_groups();
// The team for n rows and restart length m; false if it does not fit.
bool team_shape(int32_t n, int32_t m, int capacity, TeamShape* s);
int64_t team_ll_words(int G, int m);
// Clear the slots and start the team on stream s.
void launch_team(int fmt, const TeamArgs& a, hipStream_t s);
// The team for one of many systems; depends on its rows only.
TeamShape team_batch_shape(int32_t n);
// Its arguments but for ll, st, eta, max_iters and literal.
TeamArgs team_batch_args(const cb_batch_item& q);
void launch_team_clear(uint64_t* ll, int64_t words, hipStream_t s);
// One launch of `groups` workgroups: workgroup w is workgroup map[w] >> 32 of
// the team of system (uint32_t)map[w] (args and map on the device, slots clear).
void launch_team_many(const TeamArgs* args, const uint64_t* map, int groups, hipStream_t s);

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
