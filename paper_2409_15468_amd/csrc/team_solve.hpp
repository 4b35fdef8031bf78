// Whole solves by a team of workgroups that stay on the GPU from the first
// residual to the last update (Fig. 1 with restarts), for short-row systems of
// up to a few hundred thousand rows.
//
// At these sizes a step of the launch-per-kernel solver is not bound by bytes:
// its four launches take 43 us at n = 4096 and 72 us at n = 227,000 (float64
// basis) where their data take 0.2 and 28 us at the HBM rate; what they pay is
// launch gaps, the two-level ticket reductions and one wave walking all
// columns of its tile.  Here one launch runs many cycles.  A step is three
// exchanges between the workgroups instead of four launches:
//
//   encode v_j, w = A v_j, h = V^T w          -> exchange h, ||w||^2
//   w -= V h, u = V^T w, ||w||^2              -> exchange u, ||w||^2
//   h += u, w -= V u, publish w, ||w||^2      -> exchange ||w||^2
//
// Rows are cut into 512-row tiles.  A workgroup has 8 waves and owns 8 / cs
// consecutive tiles; the cs waves of a tile (cs = 8, 4 or 2, the largest
// for which the team fits the GPU at one workgroup per CU) hold its rows of w
// in registers and split the columns: wave p of a tile projects the columns p,
// p + cs, ... and forms its part of V h, and the parts are added in the order
// p = 0, 1, ... through LDS.  Every workgroup computes the scalars (Givens
// rotations, tests, R, g) from the same sums, so nothing else is exchanged;
// all branches are uniform over the team.
//
// Exchange.  A partial sum travels as two 8-byte words that carry half of the
// double and a 32-bit tag each (the exchange's number in this launch); the
// reader polls the data itself until both tags match, so a sum costs one store
// and one load latency, without a separate flag, counter or wait for the
// store's completion.  Up to kDirect workgroups, every workgroup reads every
// partial; above, workgroup c sums column c and publishes the sum.  Sums are
// formed in a fixed order that depends on the number of rows and the GPU's CU
// count only.  A slot is written again only after every reader of its last
// content has gone on (a workgroup takes part in an exchange only after it has
// read the one before; the direct form alternates between two sets of slots).
//
// A workgroup first waits until the whole team is on the GPU (gather).  The host
// keeps the teams in flight within the GPU's CUs (one workgroup fills a CU's
// registers), so only other programs' work can keep a team from forming; after
// wait_us it then leaves as one, before it has written anything, and the host
// solves the system by a path that needs no team.  Behind the gather every
// workgroup runs, and a poll waits for the others' work only.  Its limit of 20 s
// ends the launch where the GPU takes the team off its CUs for that long: a
// workgroup whose poll expires tags what it still sends with 0, for which nobody
// waits, so no sum that lacks a part is ever used.
#pragma once

#include "cb_internal.hpp"
#include "codec.hpp"
#include "epilogue.hpp"
#include "reduce.hpp"
#include "team.hpp"
#include "tiles.hpp"

namespace cb {

namespace dev {

constexpr int kTW = kTeamThreads / 64;  // waves per workgroup
constexpr int kTM = kTeamMaxRestart;
constexpr int kTC = kTM + 2;            // columns of one exchange at most
constexpr int kDirect = 32;             // workgroups up to which everyone reads all partials
constexpr int kStage = 512;             // nonzeros of a 64-row block staged in LDS
constexpr int64_t kStreamBytes = (int64_t)192 << 20;  // columns that the Infinity Cache does not keep
constexpr unsigned kNoTeam = 1u << 31;      // in the join word

struct TeamShared {
    TeamArgs args;
    double red[kTW][kTC];   // per tile of the workgroup: column sums
    double part[kTW][kTC];
    double tot[kTC];        // the exchanged sums
    double h[kTC], u[kTC];
    double cs[kTM], sn[kTM], g[kTM + 1], y[kTM];
    double R[kTM * (kTM + 1) / 2];  // packed by columns: column i at i(i+1)/2
    union {  // an exchange lies between the SpMV and the updates
        double xch[kTW][8][64];  // the waves' parts of V h
        double prod[kTW][kStage];
    };
    double w[kTW * kPadTile];  // the workgroup's rows of w (padded())
    State st;      // what the solve reports, kept by thread 0
    double carry;  // column j's entry after the old rotations
    int bad, dead;
    int reorths0;  // S.st.reorths at the start of the cycle
};
static_assert(sizeof(TeamShared) <= 148 * 1024, "team LDS (and 10.5 KB of frsz2_21 tiles)");

// (pointers come back from LDS as pointers to global memory)
template <class T>
__device__ __forceinline__ T* global(T* p) { return global_ptr(p); }
__device__ __forceinline__ BasisView global(BasisView V) {
    V.values = global(V.values);
    V.exps = global(V.exps);
    return V;
}
template <class T>
__device__ __forceinline__ T global(T v) { return v; }

struct Ctx {
    TeamShared& S;
    int n, m, rank, G, cs, lcs, R;  // rows, restart, workgroup, team size, waves per tile (and log2), tiles per workgroup
    int wave, lane, t, p;      // tile of the wave in the workgroup, its column phase
    int tile0;                 // first row of the wave's tile
    bool full;                 // the tile lies inside the padded column
    uint32_t epoch;

    // An argument, read from LDS into scalar registers where it is used: held
    // for the whole kernel they do not fit, and spill.
    template <class T>
    __device__ __forceinline__ T arg(T TeamArgs::*f) const { return global(uniform(S.args.*f)); }
};

__device__ __forceinline__ void ll_store(uint64_t* s, double v, uint32_t tag) {
    const uint64_t t = (uint64_t)tag << 32;
    __hip_atomic_store(s, t | lo32(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(s + 1, t | hi32(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits for K slots at once (those with live[k]); after poll_ticks the team is lost,
// and S.dead says so.
template <int K>
__device__ __forceinline__ bool ll_load(const Ctx& x, const uint64_t* const* s, const bool* live, uint32_t tag, double* v) {
    uint64_t t_end = 0;
    for (unsigned it = 0;; ++it) {
        uint64_t a[K], b[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            a[k] = live[k] ? ld_ctl(s[k]) : (uint64_t)tag << 32;
            b[k] = live[k] ? ld_ctl(s[k] + 1) : (uint64_t)tag << 32;
        }
        bool ok = true;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ok = ok && (uint32_t)(a[k] >> 32) == tag && (uint32_t)(b[k] >> 32) == tag;
            v[k] = make_double((uint32_t)b[k], (uint32_t)a[k]);
        }
        if (ok) return true;
        if ((it & 255u) == 255u) {
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (t_end == 0) t_end = now + x.S.args.poll_ticks;
            else if (now > t_end) {
                x.S.dead = 1;
                return false;
            }
        }
    }
}

// True once all G workgroups of the team are on the GPU; false, in every one of
// them, if they are not within wait_us (all threads).  Where a launch's
// workgroups go on to other systems, the time counts while none of its teams is
// whole: then every workgroup of it that the GPU has is in this one.  The count
// and the decision against the team share a word: a workgroup gives up by setting
// the top bit of a count that is not full, and a count with that bit is never full.
__device__ __forceinline__ bool gather(Ctx& x) {
    if (threadIdx.x == 0) {
        unsigned* join = x.arg(&TeamArgs::join);
        const int us = x.arg(&TeamArgs::wait_us);
        if (us <= 0) __hip_atomic_fetch_or(join, kNoTeam, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned v = __hip_atomic_fetch_add(join, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
        unsigned* busy = x.arg(&TeamArgs::busy);
        uint64_t t0 = __builtin_amdgcn_s_memrealtime();
        while (v != (unsigned)x.G && !(v & kNoTeam)) {
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (busy && ld_ctl(busy) != 0u) {
                t0 = now;
            } else if (now - t0 > (uint64_t)us * 100u) {
                if (__hip_atomic_compare_exchange_strong(join, &v, v | kNoTeam, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT))
                    v |= kNoTeam;
                continue;  // (else v is the word as it now is)
            }
            __builtin_amdgcn_s_sleep(1);
            v = ld_ctl(join);
        }
        x.S.dead = v & kNoTeam ? 1 : 0;
        if (busy && x.rank == 0 && !(v & kNoTeam))
            __hip_atomic_fetch_add(busy, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return uniform(x.S.dead) == 0;
}

// tot[c] = sum over the team of red[.][c], c < nc: post sends the workgroup's
// sums, collect waits for the team's (all threads; synchronised on return;
// false: the team is lost, and nothing the workgroup sends from then on counts).  Rows published before post are visible to
// every workgroup after collect.
__device__ __forceinline__ uint64_t* slots(const Ctx& x) {
    const bool two_sets = x.G <= kDirect;
    return x.arg(&TeamArgs::ll) + (two_sets ? (int64_t)(x.epoch & 1u) * 2 * x.G * (x.m + 2) : 0);
}
// (of a workgroup that has lost the team, one that nobody waits for)
__device__ __forceinline__ uint32_t tag_of(const Ctx& x) { return x.S.dead ? 0u : x.epoch; }
__device__ __forceinline__ void post(Ctx& x, int nc, bool may_be_lost) {
    TeamShared& S = x.S;
    const int tid = threadIdx.x, G = x.G, ncs = x.m + 2;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's published rows have arrived
    __syncthreads();
    ++x.epoch;
    uint64_t* ll = slots(x);
    if (tid < nc) {
        const uint32_t tag = may_be_lost ? tag_of(x) : x.epoch;
        double s = S.red[0][tid];
        for (int k = 1; k < x.R; ++k) s += S.red[k][tid];
        if (G == 1) S.tot[tid] = s;
        else if (G <= kDirect) ll_store(ll + 2 * ((int64_t)x.rank * ncs + tid), s, tag);
        else ll_store(ll + 2 * ((int64_t)tid * G + x.rank), s, tag);
    }
}
__device__ __forceinline__ bool collect(Ctx& x, int nc) {
    TeamShared& S = x.S;
    const int tid = threadIdx.x, G = x.G, ncs = x.m + 2;
    uint64_t* ll = slots(x);
    if (G > 1 && G <= kDirect) {
        // wave q adds the partials of workgroups q, q + 8, ... in order, then
        // the waves' sums are added in order
        constexpr int K = kDirect / kTW;
        if (x.wave < G) {
            for (int c = x.lane; c < nc; c += 64) {
                const uint64_t* s[K];
                bool live[K];
                double v[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int g = x.wave + kTW * k;
                    live[k] = g < G;
                    s[k] = ll + 2 * ((int64_t)g * ncs + c);
                }
                ll_load<K>(x, s, live, x.epoch, v);
                double sum = 0.0;
#pragma unroll
                for (int k = 0; k < K; ++k) sum += live[k] ? v[k] : 0.0;
                S.part[x.wave][c] = sum;
            }
        }
        __syncthreads();
        if (tid < nc) {
            double s = S.part[0][tid];
            for (int k = 1; k < min(kTW, G); ++k) s += S.part[k][tid];
            S.tot[tid] = s;
        }
    } else if (G > 1) {
        uint64_t* out = ll + 2 * (int64_t)ncs * G;
        for (int c = x.rank; c < nc; c += G) {
            const uint64_t* s[1] = {ll + 2 * ((int64_t)c * G + tid)};
            const bool live[1] = {tid < G};
            double v[1];
            ll_load<1>(x, s, live, x.epoch, v);
            const double q = wave_sum(live[0] ? v[0] : 0.0);
            if (x.lane == 0) S.part[x.wave][0] = q;
            __syncthreads();
            if (tid == 0) {
                const uint32_t tag = tag_of(x);
                double t = S.part[0][0];
                for (int k = 1; k < kTW; ++k) t += S.part[k][0];
                ll_store(out + 2 * c, t, tag);
            }
            __syncthreads();
        }
        if (tid < nc) {
            const uint64_t* s[1] = {out + 2 * tid};
            const bool live[1] = {true};
            double v[1];
            ll_load<1>(x, s, live, x.epoch, v);
            S.tot[tid] = v[0];
        }
    }
    __syncthreads();
    return uniform(S.dead) == 0;
}

// The entries of a 64-row block, loaded ahead of the operand.
struct Entries {
    int c0, c1, k0, k1;  // the lane's row, the block's run
    int cc[kStage / 64];
    double vv[kStage / 64];
};
__device__ __forceinline__ void load_entries(const Ctx& x, const double* val, int blk, Entries& e) {
    const int32_t* rp = x.arg(&TeamArgs::rp);
    const int32_t* ci = x.arg(&TeamArgs::ci);
    const int r = x.rank * x.R * kTile + blk * 64 + x.lane;
    e.c0 = rp[min(r, x.n)];
    e.c1 = rp[min(r + 1, x.n)];
    e.k0 = __builtin_amdgcn_readfirstlane(e.c0);
    e.k1 = __builtin_amdgcn_readlane(e.c1, 63);
    if (e.k1 > e.k0 && e.k1 - e.k0 <= kStage) {
#pragma unroll
        for (int c = 0; c < kStage / 64; ++c) {
            const int k = min(e.k0 + c * 64 + x.lane, e.k1 - 1);
            e.cc[c] = ci[k];
            e.vv[c] = val[k];
        }
    }
}
// The rows of a block of which one has most of the entries, more than fit the
// staging buffer: the wave takes the run in pieces, values and operands staged
// side by side, and each lane adds what a piece holds of its row, in CSR order.
// That is one entry at a time of the block, from LDS, against one at a time of
// each row, from memory, which takes four times as long: n = 500,000 with one row
// of 300,000 entries 8182 -> 1983 ms (7499 by one launch per operation).  So it
// pays where a row has a quarter of the block's entries; rows of 200 entries
// each, 4096 of them, take 8.0 ms a lane per row and 14.5 so.
__device__ __forceinline__ void long_rows(const Ctx& x, const double* val, const double* xs, double d, int c0, int c1,
                                          int k0, int k1, double* stage, double& s) {
    constexpr int H = kStage / 2, C = H / 64;
    const int32_t* ci = x.arg(&TeamArgs::ci);
    for (int q = k0; q < k1; q += H) {
        double vv[C], xv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int k = min(q + c * 64 + x.lane, k1 - 1);
            vv[c] = val[k];
            xv[c] = ld_ctl(xs + ci[k]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            stage[c * 64 + x.lane] = vv[c];
            stage[H + c * 64 + x.lane] = xv[c] / d;
        }
        __builtin_amdgcn_wave_barrier();
        const int end = min(c1, q + H);
        for (int k = max(c0, q); k < end; ++k) s = fma(stage[k - q], stage[H + k - q], s);
        __builtin_amdgcn_wave_barrier();
    }
}
// S.w = A (xs / d), or b - A (xs / d), over the workgroup's rows: as
// spmv_rows_staged (64 rows a wave, products staged in LDS, each row summed in
// CSR order), the operand read with device-scope loads since other workgroups
// write it.  e holds the entries of the wave's first block, loaded while the
// team's sums travelled.
__device__ __forceinline__ void team_spmv(Ctx& x, Entries& e, const double* val, const double* xs, double d,
                                          const double* b) {
    const int nblk = x.R * (kTile / 64);
    const int row0 = x.rank * x.R * kTile;
    double* prod = x.S.prod[x.wave];
    constexpr int C = kStage / 64;
    for (int blk = x.wave; blk < nblk; blk += kTW) {
        const int r = row0 + blk * 64 + x.lane;
        const int c0 = e.c0, c1 = e.c1, k0 = uniform(e.k0), k1 = uniform(e.k1);
        const double bv = b && r < x.n ? b[r] : 0.0;
        double s = 0.0;
        if (k1 - k0 <= kStage) {
            if (k1 > k0) {
                double xv[C];
#pragma unroll
                for (int c = 0; c < C; ++c) xv[c] = ld_ctl(xs + e.cc[c]);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const bool live = k0 + c * 64 + x.lane < k1;
                    prod[c * 64 + x.lane] = live ? e.vv[c] * (xv[c] / d) : 0.0;
                }
            }
            if (blk + kTW < nblk) load_entries(x, val, blk + kTW, e);
            __builtin_amdgcn_wave_barrier();
            for (int k = c0; k < c1; ++k) s += prod[k - k0];
            __builtin_amdgcn_wave_barrier();
        } else {
            if (__any(c1 - c0 >= (k1 - k0) / 4)) {
                long_rows(x, val, xs, d, c0, c1, k0, k1, prod, s);
            } else {
                const int32_t* ci = x.arg(&TeamArgs::ci);
                for (int k = c0; k < c1; ++k) s = fma(val[k], ld_ctl(xs + ci[k]) / d, s);
            }
            if (blk + kTW < nblk) load_entries(x, val, blk + kTW, e);
        }
        x.S.w[padded(blk * 64 + x.lane)] = b ? bv - s : s;  // rows past n: 0
    }
    __syncthreads();
}

// the wave's rows of its tile from S.w
template <int FMT>
__device__ __forceinline__ void read_rows(const Ctx& x, double* wv) {
    const double* w = x.S.w + x.t * kPadTile;
#pragma unroll
    for (int q = 0; q < 8; ++q) wv[q] = w[padded(Map<FMT>::row(x.lane, q))];
}

// The wave's first kSlots columns (p, p + cs, ...) of its tile stay in registers
// for the whole cycle, in their stored form; later columns are read from
// memory in each pass.  As many as fit beside the passes' own registers at two
// waves per SIMD (64 registers of tiles; more spill).
template <int FMT>
constexpr int kSlotsOf = FMT == CB_F64 ? 2 : FMT == CB_FRSZ2_32 || FMT == CB_FRSZ2_32_B64 || FMT == CB_FRSZ2_21 ? 6
                     : is_generic<FMT> ? 3 : 8;
// the wave's columns among the first jc
__device__ __forceinline__ int columns_of(const Ctx& x, int jc) { return (jc - x.p + x.cs - 1) >> x.lcs; }
// S.red[t][c] = <D(v_c), w> over the tile for the wave's columns c < jc; the
// columns in memory from the last to the first, the next 8 in flight while the
// wave reduces the current ones, then the resident ones
template <int FMT, int N, int LM>
__device__ __forceinline__ void project_cols(const Ctx& x, const BasisView& V, int K, const double* wv) {
    // columns loaded at once: 4 where 8 tiles do not fit beside the rest
    constexpr int U = N > 0 || FMT == CB_F64 || FMT == CB_FRSZ2_21 || is_generic<FMT> ? 4 : 8;
    const int ks = x.lane >> 3;
    Tile<FMT> tl[U];
    auto load = [&](int k) {
        int cols[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cols[u] = x.p + x.cs * min(k + u, K - 1);
        load_tiles<FMT, U, LM>(tl, V, cols, x.tile0, x.lane);
    };
    const int last = N + (K - 1 - N) / 8 * 8;
    load(last);
    for (int k0 = last; k0 >= N; k0 -= 8) {
        double s[8];
#pragma unroll
        for (int part = 0; part < 8 / U; ++part) {
#pragma unroll
            for (int u = 0; u < U; ++u) s[part * U + u] = tl[u].dot(wv);
            if (part + 1 < 8 / U) load(k0 + (part + 1) * U);
        }
        if (U == 8 && k0 > N) load(k0 - 8);
        const double sum = wave_sum8(s);
        if (U < 8 && k0 > N) load(k0 - 8);
        if ((x.lane & 7) == 0 && k0 + ks < K) x.S.red[x.t][x.p + x.cs * (k0 + ks)] = sum;
    }
}
template <int FMT, int N>
__device__ __forceinline__ void team_project(const Ctx& x, Tile<FMT>* rs, int jc, const double* wv, bool stream) {
    const int K = columns_of(x, jc);
    if (K > N) {
        const BasisView V = x.arg(&TeamArgs::V);
        if (!x.full) project_cols<FMT, N, 0>(x, V, K, wv);
        else if (N == 0 && stream) project_cols<FMT, N, kFull | kStream>(x, V, K, wv);
        else project_cols<FMT, N, kFull>(x, V, K, wv);
    }
    if (N == 0 || K <= 0) return;
    double s[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        s[u] = 0.0;
        if (u < N) {
            opaque<FMT>(rs[u]);
            if (u < K) s[u] = rs[u].dot(wv);
        }
    }
    const double sum = wave_sum8(s);
    const int ks = x.lane >> 3;
    if ((x.lane & 7) == 0 && ks < min(K, N)) x.S.red[x.t][x.p + x.cs * ks] = sum;
}

// acc += sum over the wave's columns k0 <= k < K of coef[c] D(v_c); the next 4
// columns in flight behind the current ones where the registers allow
template <int FMT, int N, int LM>
__device__ __forceinline__ void combine_cols(const Ctx& x, const BasisView& V, int k0, int K, const double* coef,
                                             double* acc) {
    constexpr int U = 4;
    auto load = [&](Tile<FMT>* tl, int k) {
        int cols[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cols[u] = x.p + x.cs * min(k + u, K - 1);
        load_tiles<FMT, U, LM>(tl, V, cols, x.tile0, x.lane);
    };
    auto apply = [&](const Tile<FMT>* tl, int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) tl[u].axpy(k + u < K ? coef[x.p + x.cs * min(k + u, K - 1)] : 0.0, acc);
    };
    if (k0 >= K) return;
    Tile<FMT> tl[U];
    if constexpr (N > 0 || FMT == CB_F64 || is_generic<FMT>) {
        for (; k0 < K; k0 += U) {
            load(tl, k0);
            apply(tl, k0);
        }
    } else {
        Tile<FMT> nx[U];
        load(tl, k0);
        for (; k0 < K; k0 += U) {
            const bool more = k0 + U < K;
            if (more) load(nx, k0 + U);
            apply(tl, k0);
            if (more) {
#pragma unroll
                for (int u = 0; u < U; ++u) tl[u] = nx[u];
            }
        }
    }
}
// The values q of a tile's lanes with q % cs == p are wave p's share: it adds
// the waves' parts of them in wave order and hands f(row in the workgroup, sum).
template <int FMT, class F>
__device__ __forceinline__ void add_parts(const Ctx& x, const double* acc, F&& f) {
    TeamShared& S = x.S;
#pragma unroll
    for (int q = 0; q < 8; ++q) S.xch[x.wave][q][x.lane] = acc[q];
    __syncthreads();
    const int w0 = x.t * x.cs;
    for (int q = x.p; q < 8; q += x.cs) {
        double s = S.xch[w0][q][x.lane];
        for (int k = 1; k < x.cs; ++k) s += S.xch[w0 + k][q][x.lane];
        f(x.t * kTile + Map<FMT>::row(x.lane, q), s);
    }
}
// out[row] = S.w for the wave's share of its tile, visible to the team after
// the next exchange
template <int FMT>
__device__ __forceinline__ void publish(const Ctx& x, double* out) {
    const int row0 = x.rank * x.R * kTile;
    for (int q = x.p; q < 8; q += x.cs) {
        const int r = x.t * kTile + Map<FMT>::row(x.lane, q);
        if (row0 + r < x.n)
            __hip_atomic_store(out + row0 + r, x.S.w[padded(r)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// the tile's sum of squares into S.red[t][c]
__device__ __forceinline__ void put_sumsq(const Ctx& x, const double* wv, int c) {
    if (x.p != 0) return;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s = fma(wv[q], wv[q], s);
    s = wave_sum(s);
    if (x.lane == 0) x.S.red[x.t][c] = s;
}

// S.args holds the arguments (all threads synchronised).
template <int FMT, int N>
__device__ __forceinline__ void team_solve(int rank, TeamShared& S) {
    using M = Map<FMT>;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // nothing here is moved out of a caller's loop
    // (the wave's index in a scalar register: what depends on it is uniform)
    Ctx x{S, 0, 0, rank, 0, 0, 0, 0, wave_index(), tid & 63, 0, 0, 0, false, uniform(S.args.epoch0)};
    x.n = x.arg(&TeamArgs::n);
    x.m = x.arg(&TeamArgs::m);
    x.G = x.arg(&TeamArgs::G);
    x.cs = x.arg(&TeamArgs::cs);
    x.lcs = x.cs == 8 ? 3 : x.cs == 4 ? 2 : 1;
    x.R = kTW >> x.lcs;
    x.t = x.wave >> x.lcs;
    x.p = x.wave & (x.cs - 1);
    x.tile0 = (rank * x.R + x.t) * kTile;
    x.full = x.tile0 + kTile <= x.arg(&TeamArgs::V).np;
    if (tid == 0) S.bad = 0;
    if (!gather(x)) {
        if (rank == 0 && tid == 0) x.arg(&TeamArgs::st)->status = kTeamAbandoned;
        return;
    }
    if (double* x0 = x.arg(&TeamArgs::x0)) {
        const double* xv = x.arg(&TeamArgs::x);
        for (int i = tid; i < x.R * kTile; i += kTeamThreads) {
            const int r = rank * x.R * kTile + i;
            if (r < x.n) x0[r] = ld_ctl(xv + r);
        }
    }
    int iters = 0, cycles = 0, status = CB_OK, stop = 0, recorded = 0;
    double nb = 0.0;
    if (x.arg(&TeamArgs::resume)) {
        const State* st = x.arg(&TeamArgs::st);
        iters = uniform(ld_ctl(&st->iters));
        cycles = uniform(ld_ctl(&st->cycles));
        if (tid == 0) {
            S.st = State{};
            S.st.iters = iters;
            S.st.cycles = cycles;
            S.st.reorths = ld_ctl(&st->reorths);
            S.st.breakdowns = ld_ctl(&st->breakdowns);
            S.st.basis_bytes = ld_ctl(&st->basis_bytes);
            S.st.gabs = ld_ctl(&st->gabs);
            S.st.counted_fused = ld_ctl(&st->counted_fused);
        }
    } else if (tid == 0) {
        S.st = State{};
        S.st.gabs = -1.0;
        S.st.counted_fused = FMT != CB_F64 && !x.arg(&TeamArgs::batch);
    }
    if (tid == 0) {
        S.st.rel = -1.0;
        S.reorths0 = S.st.reorths;
    }
    // One loop, so that each piece of code exists once: the phase of an
    // iteration is ||b||, the residual of a restart, an Arnoldi step (j) or the
    // update of x; each ends in an exchange of a squared norm.
    enum : int { kNormB, kResidual, kStep, kUpdate };
    int phase = kNormB;
    double d = 1.0;
    int j = 0, steps = 0;
    bool nonfinite = false;
    double wv[8];
    Tile<FMT> rs[N > 0 ? N : 1];
    Entries ent;
    load_entries(x, x.arg(&TeamArgs::val), x.wave, ent);
    __syncthreads();
    for (;;) {
        // keeps the address arithmetic of every piece below from being hoisted
        // out of the loop, where it would hold a hundred registers
        asm volatile("" : "+v"(x.lane));
        // the same in every lane, which the compiler does not see through the
        // loop: in scalar registers, or every branch below would be a divergent one
        phase = uniform(phase);
        j = uniform(j);
        steps = uniform(steps);
        d = uniform(d);
        x.epoch = uniform(x.epoch);
        iters = uniform(iters);
        recorded = uniform(recorded);
        const int jc = j + 1;
        double omega = 0.0, hn = 0.0;
        bool again = false;
        if (phase == kNormB) {
            const double* b = x.arg(&TeamArgs::b);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int r = x.tile0 + M::row(x.lane, q);
                wv[q] = r < x.n ? b[r] : 0.0;
            }
        } else if (phase == kUpdate) {
            // step 17: R y = g by columns (wave 0; rows lane and lane + 64), x += V y
            if (x.wave == 0) {
                double r0 = x.lane < steps ? S.g[x.lane] : 0.0;
                double r1 = x.lane + 64 < steps ? S.g[x.lane + 64] : 0.0;
                for (int i = steps - 1; i >= 0; --i) {
                    const double* Rc = S.R + i * (i + 1) / 2;
                    const double gi = i < 64 ? readlane_f64(r0, i) : readlane_f64(r1, i - 64);
                    const double yi = gi / Rc[i];
                    if (x.lane == 0) S.y[i] = yi;
                    if (x.lane < i) r0 -= Rc[x.lane] * yi;
                    if (x.lane + 64 < i) r1 -= Rc[x.lane + 64] * yi;
                }
            }
            __syncthreads();
            double acc[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = 0.0;
            const BasisView V = x.arg(&TeamArgs::V);
            combine_cols<FMT, 1, 0>(x, V, 0, columns_of(x, steps), S.y, acc);
            double* xv = x.arg(&TeamArgs::x);
            const double* dinv = x.arg(&TeamArgs::dinv);
            const int row0 = rank * x.R * kTile;
            add_parts<FMT>(x, acc, [&](int r, double s) {
                r += row0;
                if (r >= x.n) return;
                const double xo = ld_ctl(xv + r);
                const double xn = dinv ? __dadd_rn(xo, __dmul_rn(dinv[r], s)) : xo + s;
                __hip_atomic_store(xv + r, xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
        } else {
            if (phase == kStep && x.p == (j & (x.cs - 1))) {
                // v_j = w / d, V_j = Q(v_j), by one wave of each tile
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = wv[q] / d;
                const BasisView V = x.arg(&TeamArgs::V);
                const bool nf = encode_tile<FMT>(
                    const_cast<unsigned char*>(V.values) + (int64_t)j * V.col_bytes,
                    const_cast<uint32_t*>(V.exps) + (int64_t)j * V.exp_stride, V.np, x.tile0, x.lane, v, V.bits,
                    V.bs_log);
                if (__any(nf) && x.lane == 0) S.bad = 1;
            }
            // the residual reads x, a step w (an operand divided by 1 is itself)
            if (phase == kStep) team_spmv(x, ent, x.arg(&TeamArgs::aval), x.arg(&TeamArgs::w), d, nullptr);
            else team_spmv(x, ent, x.arg(&TeamArgs::val), x.arg(&TeamArgs::x), 1.0, x.arg(&TeamArgs::b));
            read_rows<FMT>(x, wv);
        }
        if (phase == kStep) {
            // the new column joins the resident ones of the wave that wrote it
            if (N > 0 && x.p == (j & (x.cs - 1))) {
                Tile<FMT> nt;
                nt.template load<0>(x.arg(&TeamArgs::V), j, x.tile0, x.lane);
                const int k = j >> x.lcs;
#pragma unroll
                for (int u = 0; u < N; ++u)
                    if (k == u) rs[u] = nt;
            }
            // Gram-Schmidt: the first pass, then the second projection with the
            // first update's norm (formed whether or not step 7 asks for it)
            const bool stream = N == 0 && (int64_t)jc * x.arg(&TeamArgs::col_total) > kStreamBytes;
            for (int pass = 0; pass < 2; ++pass) {
                asm volatile("" : "+v"(x.lane));
                put_sumsq(x, wv, jc);
                team_project<FMT, N>(x, rs, jc, wv, stream);
                post(x, jc + 1, false);
                // (lost: the exchange below fails in its turn; a way out of both loops
                // from here costs them 40 registers)
                if (!collect(x, jc + 1)) break;
                const double t = sqrt(uniform(S.tot[jc]));
                if (tid < jc) {
                    S.u[tid] = S.tot[tid];
                    if (pass == 0) S.h[tid] = S.tot[tid];
                }
                if (pass == 0) {
                    omega = t;
                } else {
                    hn = t;
                    again = hn < x.arg(&TeamArgs::eta) * omega;
                    if (!again) break;
                    if (tid < jc) S.h[tid] += S.tot[tid];
                }
                __syncthreads();
                double acc[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[q] = 0.0;
                const int K = columns_of(x, jc);
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    opaque<FMT>(rs[u]);
                    if (u < K) rs[u].axpy(S.u[x.p + x.cs * u], acc);
                }
                if (K > N) {
                    const BasisView V = x.arg(&TeamArgs::V);
                    // (the first update's columns are read again right away)
                    if (!x.full) combine_cols<FMT, N, 0>(x, V, N, K, S.u, acc);
                    else if (N == 0 && stream && pass > 0) combine_cols<FMT, N, kFull | kStream>(x, V, N, K, S.u, acc);
                    else combine_cols<FMT, N, kFull>(x, V, N, K, S.u, acc);
                }
                add_parts<FMT>(x, acc, [&](int r, double s) { S.w[padded(r)] -= s; });
                __syncthreads();
                read_rows<FMT>(x, wv);
            }
        }
        if (phase == kStep || phase == kResidual) publish<FMT>(x, x.arg(&TeamArgs::w));
        put_sumsq(x, wv, 0);
        if (x.p == 0 && x.lane == 0) S.red[x.t][1] = x.t == 0 && S.bad ? 1.0 : 0.0;
        post(x, 2, true);
        // while the sums travel: the entries of the next SpMV, and by one
        // thread the old rotations on column j (steps 15-16)
        load_entries(x, x.arg(phase == kStep || phase == kResidual ? &TeamArgs::aval : &TeamArgs::val), x.wave, ent);
        if (phase == kStep && tid == kTeamThreads - 64) {
            double* Rc = S.R + j * (j + 1) / 2;
            double carry = S.h[0];
            for (int i0 = 0; i0 < j; i0 += 8) {
                double b1[8], c[8], s[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int i = min(i0 + k, j - 1);
                    b1[k] = S.h[i + 1];
                    c[k] = S.cs[i];
                    s[k] = S.sn[i];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (i0 + k < j) {
                        Rc[i0 + k] = c[k] * carry + s[k] * b1[k];
                        carry = -s[k] * carry + c[k] * b1[k];
                    }
                }
            }
            S.carry = carry;
        }
        if (!collect(x, 2)) {
            status = kTeamLost;
            break;
        }
        const double norm = sqrt(uniform(S.tot[0]));
        if (phase == kNormB) {
            nb = norm;
            if (nb == 0.0) {
                double* xv = x.arg(&TeamArgs::x);
                for (int i = tid; i < x.R * kTile; i += kTeamThreads) {
                    const int r = rank * x.R * kTile + i;
                    if (r < x.n) xv[r] = 0.0;
                }
                if (tid == 0) {
                    S.st.converged = 1;
                    S.st.rel = S.st.gabs = 0.0;
                }
                stop = 1;
                break;
            }
            if (!isfinite(nb)) {
                stop = 1;
                status = CB_ERR_NONFINITE;
                break;
            }
            phase = kResidual;
        } else if (phase == kResidual) {
            // steps 1 and 18: beta and the stop test of Eq. 4
            if (tid == 0) S.st.rel = norm / nb;
            if (!isfinite(norm) || uniform(S.tot[1]) != 0.0) {
                stop = 1;
                status = CB_ERR_NONFINITE;
            } else if (norm <= x.arg(&TeamArgs::tol) * nb) {
                stop = 1;
                if (tid == 0) S.st.converged = 1;
            } else if (nonfinite) {
                stop = 1;
            } else if (iters >= x.arg(&TeamArgs::max_iters)) {
                stop = 1;
                status = CB_ERR_NOT_CONVERGED;
            }
            // (or no room for a cycle's history: the next launch goes on)
            if (stop || recorded + x.m > x.arg(&TeamArgs::hist_cap)) break;
            if (tid == 0) {
                S.st.iters = iters;
                S.st.cycles = cycles;
            }
            cycles += 1;
            for (int i = tid; i <= x.m; i += kTeamThreads) S.g[i] = i == 0 ? norm : 0.0;
            d = norm;
            steps = 0;
            j = 0;
            phase = kStep;
            __syncthreads();
        } else if (phase == kStep) {
            int bd = 0;
            if (again) {
                const double omega_pre = hn;
                hn = norm;
                const double eta = x.arg(&TeamArgs::eta);
                bd = x.arg(&TeamArgs::literal) ? (hn < eta * omega) : (hn < eta * omega_pre);
            }
            bool over;
            double gabs = 0.0;
            if (!isfinite(hn)) {
                nonfinite = over = true;
                status = CB_ERR_NONFINITE;
                bd = 0;
                if (x.arg(&TeamArgs::batch)) {  // (the batch leaves x as the cycle found it)
                    stop = 1;
                    break;
                }
            } else {
                // the new rotation and g, by every thread from the same values
                if (hn == 0.0) bd = 1;
                const double carry = uniform(S.carry), gj = uniform(S.g[j]);
                const double rho = sqrt(carry * carry + hn * hn);
                const double c = carry / rho, s = hn / rho;
                const double g1 = -s * gj;
                gabs = fabs(g1);
                __syncthreads();  // every thread has read g_j
                if (tid == 0) {
                    S.cs[j] = c;
                    S.sn[j] = s;
                    S.R[j * (j + 1) / 2 + j] = rho;
                    S.g[j + 1] = g1;
                    S.g[j] = c * gj;
                    S.st.gabs = gabs;
                    double* hist = x.arg(&TeamArgs::hist);
                    if (rank == 0 && hist) hist[recorded + j] = gabs;
                }
                iters += 1;
                steps = jc;
                d = hn;
                over = gabs <= x.arg(&TeamArgs::tol) * nb || bd || iters >= x.arg(&TeamArgs::max_iters) || jc == x.m;
            }
            if (tid == 0) {
                // the passes over the columns as the other paths make them: fused
                // updates form u whether or not it is asked for, separate ones
                // (a float64 basis, the batch, cycles that follow one with few
                // second passes) only if it is
                const int passes = S.st.counted_fused ? 3 + again : 2 + 2 * again;
                S.st.basis_bytes += (double)passes * jc * (double)x.arg(&TeamArgs::V).col_bytes;
                S.st.reorths += again;
                if (over) {
                    S.st.breakdowns += bd;
                    if (FMT != CB_F64 && !x.arg(&TeamArgs::batch))
                        S.st.counted_fused = steps > 0 && 2 * (S.st.reorths - S.reorths0) >= steps;
                    S.reorths0 = S.st.reorths;
                }
            }
            if (over) {
                recorded += steps;
                phase = kUpdate;
                __syncthreads();
            } else {
                j += 1;
            }
        } else {
            if (tid == 0) S.st.basis_bytes += (double)steps * (double)x.arg(&TeamArgs::V).col_bytes;
            const int max_cycles = x.arg(&TeamArgs::max_cycles);
            if (max_cycles > 0 && cycles >= max_cycles) {
                stop = 1;
                if (status == CB_OK) {
                    status = CB_ERR_NOT_CONVERGED;
                    if (tid == 0) S.st.rel = -1.0;
                }
                break;
            }
            phase = kResidual;
        }
    }
    if (rank != 0) return;
    if (tid == 0) {
        if (unsigned* busy = x.arg(&TeamArgs::busy))
            __hip_atomic_fetch_sub(busy, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        S.st.nb = nb;
        if (status != kTeamLost) {
            S.st.iters = iters;
            S.st.cycles = cycles;
        }
        S.st.stop = stop;
        S.st.status = status;
        S.st.steps = recorded;
        S.st.pad0 = (int)x.epoch;  // the last tag used
    }
    __syncthreads();
    static_assert(sizeof(State) % 8 == 0, "copied by words");
    if (tid < (int)(sizeof(State) / 8))
        reinterpret_cast<uint64_t*>(x.arg(&TeamArgs::st))[tid] = reinterpret_cast<const uint64_t*>(&S.st)[tid];
}

}  // namespace dev
}  // namespace cb
