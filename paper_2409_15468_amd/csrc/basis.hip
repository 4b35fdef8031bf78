// Basis kernels: normalise+encode (store), decode (load), the fused
// decode + classical Gram-Schmidt projection and update, the fused decode +
// solution update, and the fixed-order second reduction stage.
//
// Row partition: workgroup g of the row kernels owns rows
// [2048 g, 2048 (g+1)) -- 64 FRSZ2 blocks -- and thread t of it the 8 rows
// from 2048 g + 8 t.  The partition depends on n only (and, for the fused
// update + projection, on the device's resident capacity), so every reduction
// (per-thread chain, then a fixed shuffle tree, then the 4 waves in order,
// then the workgroups in order) is the same on every run and for every caller.
#include <atomic>

#include "cb_internal.hpp"
#include "codec.hpp"
#include "epilogue.hpp"
#include "reduce.hpp"
#include "tiles.hpp"

namespace cb {

using namespace dev;

// ----------------------------------------------------------------- store (encode)
// Workgroup g, wave w encodes the 512-row tile starting at 2048 g + 512 w.
// The codes go out with non-temporal stores: over launches that encode
// different columns they sustain 2-3% more.  (Of the solver's columns only
// each cycle's first is stored here; the steps' columns are encoded by the
// store + SpMV kernel with ordinary stores, as the next kernel reads them.)
template <int FMT>
__global__ __launch_bounds__(kThreads) void k_store(unsigned char* __restrict__ values,
                                                    uint32_t* __restrict__ exps, int n, int np,
                                                    const double* w, const double* __restrict__ divisor,
                                                    double* v_out, int32_t* __restrict__ flag,
                                                    const int* __restrict__ guard, int bits, int bs_log) {
    if (guard && ld_ctl(guard) == 0) return;
    const int lane = threadIdx.x & 63;
    const int tile0 = blockIdx.x * kRowsPerWG + wave_index() * kTile;
    double v[8];
    load_rows<FMT>(w, tile0, lane, n, v);
    if (divisor) {
        const double d = ld_ctl(divisor);
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = v[q] / d;  // IEEE division per entry
    }
    __shared__ double stage[kThreads / 64][kTile];
    if (v_out) store_rows_lds<FMT>(v_out, tile0, lane, n, v, stage[threadIdx.x >> 6]);
    const bool bad = encode_tile<FMT, true>(values, exps, np, tile0, lane, v, bits, bs_log);
    if (flag && bad) atomicOr(flag, 1);
}

// ----------------------------------------------------------------- load (decode)
// Workgroup g, wave w decodes the 512-row tile starting at 2048 g + 512 w:
// one tile per wave and many waves (a loop over several tiles per wave with
// the next tile's loads in flight measured 6% slower: the wave then waits for
// its own stores, where fresh waves do not).  The output goes out with
// non-temporal stores: ordinary stores leave it in the Infinity Cache as dirty
// lines that later launches (or the next kernel's traffic) must write back,
// and measured over launches that decode different columns into different
// vectors they sustain 6% less.
template <int FMT>
__global__ __launch_bounds__(kThreads) void k_load(BasisView V, int col, double* __restrict__ x) {
    const int lane = threadIdx.x & 63, wave = wave_index();
    const int tile0 = blockIdx.x * kRowsPerWG + wave * kTile;
    Tile<FMT> t[1];
    const int cols[1] = {col};
    if (tile0 + kTile <= V.np) load_tiles<FMT, 1, kFull | kStream>(t, V, cols, tile0, lane);
    else load_tiles<FMT, 1, kStream>(t, V, cols, tile0, lane);
    double out[8];
    t[0].decode(out);
    __shared__ double stage[kThreads / 64][kTile];
    store_rows_lds<FMT, true>(x, tile0, lane, V.n, out, stage[wave]);
}

// ----------------------------------------------------------------- CGS projection
// Workgroup (g, y) takes the row groups g, g + G, g + 2G, ... (2048 rows each;
// G <= kProjectGroups keeps the partials few) and the columns
// [y cw, (y+1) cw), and writes partials[c * G + g], its sum of D(v_c) * w:
// per column the waves accumulate over their row groups in order and the waves
// are then added in order.  The last workgroup forms the sums over g
// (epilogue.hpp).  Small n gets several column chunks so that the launch still
// has enough waves to keep HBM busy.
template <int FMT>
__global__ __launch_bounds__(kThreads) void k_project(BasisView V, int j,
                                                      const double* __restrict__ w,
                                                      double* __restrict__ partials, int G, int cw,
                                                      int stream, const int* __restrict__ guard, Epi e) {
    if (guard && ld_ctl(guard) == 0) return;
    __shared__ double red[kThreads / 64][kMaxRestart + 1];
    __shared__ double elds[kEpiLds];
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int g = blockIdx.x;
    const int ngroups = row_groups_dev(V.np);
    const int c0 = blockIdx.y * cw;  // this workgroup's columns [c0, c1)
    const int c1 = min(j, c0 + cw);
    for (int i = lane; i < c1 - c0; i += 64) red[wave][i] = 0.0;
    for (int rg = g; rg < ngroups; rg += G) {
        const int tile0 = rg * kRowsPerWG + wave * kTile;
        double wv[8];
        load_rows<FMT>(w, tile0, lane, V.n, wv);
        const bool full = tile0 + kTile <= V.np;
        if (stream) {
            if (full) project_tile<FMT, kFull | kStream>(V, c0, c1, tile0, lane, wv, red[wave]);
            else project_tile<FMT, kStream>(V, c0, c1, tile0, lane, wv, red[wave]);
        } else {
            if (full) project_tile<FMT, kFull>(V, c0, c1, tile0, lane, wv, red[wave]);
            else project_tile<FMT, 0>(V, c0, c1, tile0, lane, wv, red[wave]);
        }
    }
    __syncthreads();
    for (int i = tid; i < c1 - c0; i += kThreads) {
        double s = red[0][i];
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) s += red[k][i];
        store_partial(partials + (int64_t)(c0 + i) * G + g, s);
    }
    if (e.mode != EPI_PARTIALS) epilogue(e, partials, elds);
}

// The projection of a short vector in one launch: workgroup c forms
// h[c] = <D(v_c), w> over all rows, wave p of it over the tiles p, p + 8, ....
// Nothing is left to sum, so it spares the caller the second launch, which at
// these sizes costs more than the work.
template <int FMT>
__global__ __launch_bounds__(512) void k_project_column(BasisView V, const double* __restrict__ w,
                                                        double* __restrict__ h) {
    __shared__ double part[8];
    const int lane = threadIdx.x & 63, wave = wave_index(), ntiles = (V.np + kTile - 1) / kTile;
    double s = 0.0;
    for (int t = wave; t < ntiles; t += 16) {
        // two tiles in flight (of one past the last nothing is read)
        Tile<FMT> a, b;
        double wa[8], wb[8];
        const int ta = t * kTile, tb = min(t + 8, ntiles) * kTile;
        a.template load<kBound>(V, blockIdx.x, ta, lane);
        b.template load<kBound>(V, blockIdx.x, tb, lane);
        load_rows<FMT>(w, ta, lane, V.n, wa);
        load_rows<FMT>(w, tb, lane, V.n, wb);
        s += a.dot(wa);
        s += b.dot(wb);
    }
    s = wave_sum(s);
    if (lane == 0) part[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = part[0];
        for (int k = 1; k < 8; ++k) sum += part[k];
        h[blockIdx.x] = sum;
    }
}

// ----------------------------------------------------------------- CGS update / x update
// Start of the update kernels: the guard, the device-side count jdev (if any;
// the host's j then bounds it) and the coefficients h[0 .. j) are loaded
// together -- one memory round trip, not three -- and the coefficients go to
// hc in LDS (the caller synchronises before reading them).  Returns 0 if the
// guard says the launch has nothing to do; j becomes the count to use.
__device__ __forceinline__ int load_coefficients(const int* __restrict__ guard, const int* __restrict__ jdev,
                                                 const double* __restrict__ h, int& j, double* hc) {
    constexpr int HR = (kMaxRestart + 1 + kThreads - 1) / kThreads;
    const int go = guard ? ld_ctl(guard) : 1;
    const int jd = jdev ? ld_ctl(jdev) : j;
    double hv[HR];
#pragma unroll
    for (int k = 0; k < HR; ++k) hv[k] = j > 0 ? ld_ctl(&h[min((int)threadIdx.x + kThreads * k, j - 1)]) : 0.0;
    if (go == 0) return 0;
    j = jd;
#pragma unroll
    for (int k = 0; k < HR; ++k) {
        const int i = (int)threadIdx.x + kThreads * k;
        if (i < j) hc[i] = hv[k];
    }
    return 1;
}

// w[k] += sign * sum_{c<j} h[c] * D(v_c)[k] over the row groups g, g + G, ...
// of workgroup g; partials[g] = sum of w[k]^2 over those rows after the update
// (row groups in order, then the waves in order), if partials != NULL, and
// then the epilogue.
// frsz2_21 leaves the lanes' addresses to the compiler: with scalar bases its
// loop took 51.6 us instead of 48.6 at 10^6 x 90 and 33.8 instead of 32.2 at
// 1000003 x 60 (909 and 912 at 2^24 x 101), and a solve at 10^6 x 100 58.4 ms
// instead of 57.8; its projection takes the same time either way.
template <int FMT, int U>
__global__ __launch_bounds__(kThreads) void k_subtract(BasisView V, int j, const int* __restrict__ jdev,
                                                       const double* __restrict__ h,
                                                       double* __restrict__ w,
                                                       double* __restrict__ partials, int sign, int stream,
                                                       const int* __restrict__ guard, Epi e) {
    constexpr int A = FMT == CB_FRSZ2_21 ? kLane : 0;
    __shared__ double elds[kEpiLds];
    // the coefficients (written by an earlier kernel), read once into LDS
    __shared__ double hc[kMaxRestart + 1];
    __shared__ double stage[kThreads / 64][kTile];
    const int go = load_coefficients(guard, jdev, h, j, hc);
    if (!go) return;
    __syncthreads();
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int ngroups = row_groups_dev(V.np);
    double nrm = 0.0;
    for (int rg = blockIdx.x; rg < ngroups; rg += gridDim.x) {
        const int tile0 = rg * kRowsPerWG + wave * kTile;
        double acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0;
        const bool full = tile0 + kTile <= V.np;
        if (stream) {
            if (full) subtract_tile<FMT, U, kFull | kStream | A>(V, j, hc, tile0, lane, acc);
            else subtract_tile<FMT, U, kStream | A>(V, j, hc, tile0, lane, acc);
        } else {
            if (full) subtract_tile<FMT, U, kFull | A>(V, j, hc, tile0, lane, acc);
            else subtract_tile<FMT, U, A>(V, j, hc, tile0, lane, acc);
        }
        double wv[8];
        load_rows<FMT>(w, tile0, lane, V.n, wv);
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            wv[q] = sign > 0 ? wv[q] + acc[q] : wv[q] - acc[q];
            t = fma(wv[q], wv[q], t);  // rows >= n hold 0
        }
        nrm += t;
        store_rows_lds<FMT>(w, tile0, lane, V.n, wv, stage[wave]);
    }
    if (partials) {
        const double t = block_sum<kThreads>(nrm);
        if (tid == 0) store_partial(partials + blockIdx.x, t);
        if (e.mode != EPI_PARTIALS) epilogue(e, partials, elds);
    }
}

// Columns a wave of k_subtract_project keeps at most, by the registers a tile
// takes (16 of float64, 4 or 5 of the 16-bit formats): more spill.
template <int FMT>
constexpr int kResidentColumns = FMT == CB_F64 ? 8 : FMT == CB_F32 ? 16
                               : FMT == CB_F16 || FMT == CB_FRSZ2_16 || FMT == CB_FRSZ2_16_B64 ? 16 : 13;
constexpr int sub_proj_threads(int W) { return W == 8 ? 512 : 256; }

// The first Gram-Schmidt update fused with the second projection (Fig. 1 steps
// 5b-6 and 8): w -= sum_{c<j} h[c] D(v_c), then u_c = <D(v_c), w> for c < j on
// the updated rows.  partials[c * G + g] holds the workgroup's u_c for c < j
// and its ||w||^2 at c = j; the epilogue (FUSED_CHECK) keeps u only if step 7
// asks for the second pass.
//
// Bound by the reads of the basis, so each column is read once: W waves share
// a 512-row tile, wave p of them takes the columns p, p + W, ..., and keeps
// the first N in registers, in their stored form, from the update to the
// projection (later ones are read again).  The waves' parts of V h are added
// in wave order through LDS.  The loads of the next tile go out as the
// projection releases the registers, so they are in flight behind it and the
// reductions.  W = 1 has nothing to exchange; with more, each tile costs two
// barriers' waits.
//
// One wave per tile that read every column twice took, at 10^6 x 100, 136 us
// with frsz2_32 and 255 with float64; this 92 and 156 (at 2^21 x 12 43 and 65,
// now 34 and 42).  The formats whose decoding bounds them gain less, since each
// column is still decoded twice (frsz2_21 at 10^6 x 100 103 -> 93).
template <int FMT, int W, int N>
__global__ __launch_bounds__(sub_proj_threads(W), 2) void k_subtract_project(BasisView V, int j,
                                                                          const double* __restrict__ h,
                                                                          double* __restrict__ w,
                                                                          double* __restrict__ partials,
                                                                          const int* __restrict__ guard, Epi e) {
    constexpr int NW = sub_proj_threads(W) / 64, T = NW / W;  // waves, tiles at a time
    constexpr int S = 8 / W;                                  // values of a lane's 8 that are a wave's share
    constexpr int B = W == 1 ? 1 : 2;
    __shared__ double hc[kMaxRestart + 1];
    __shared__ double red[T][kMaxRestart + 2];
    __shared__ double part[NW];
    __shared__ double rows[B][T][kPadTile];
    __shared__ union {
        double xch[W == 1 ? 1 : NW][8][64];
        double epi[kEpiLds];
    } lds;
    const int go = load_coefficients(guard, nullptr, h, j, hc);
    if (!go) return;
    const int wave = wave_index(), ti = wave / W;
    int p = wave % W;
    const int slot = (int)threadIdx.x - ti * W * 64;  // the thread among those of its tile
    int lane = threadIdx.x & 63;
    const int G = gridDim.x, ntiles = (V.np + kTile - 1) / kTile, ngroups = (ntiles + T - 1) / T;
    int K = (j - p + W - 1) / W;  // the wave's columns
    auto col = [&](int k) { return min(p + W * max(min(k, K - 1), 0), j - 1); };
    auto barrier = [] {
        if (W > 1) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
    };
    Tile<FMT> rs[N];
    double wn[S];
    // a thread moves pairs of rows (single rows where it has one)
    constexpr int P = S > 1 ? 2 : 1;
    auto row = [&](int i) { return P * slot + i * W * 64; };  // (i a multiple of P)
    auto load_w = [&](int t) {
#pragma unroll
        for (int i = 0; i < S; i += P) {
            const int r = t * kTile + row(i);
            if (P == 2 && r + 1 < V.n) {
                const double2 x = *reinterpret_cast<const double2*>(w + r);
                wn[i] = x.x;
                wn[i + P - 1] = x.y;
            } else {
                wn[i] = r < V.n ? w[r] : 0.0;
                if (P == 2) wn[i + P - 1] = 0.0;
            }
        }
    };
    // (of a tile past the last nothing is read)
    auto load = [&](int u, int t) {
        if (u < K) rs[u].template load<kBound>(V, p + W * u, t * kTile, lane);
    };
    int tg = blockIdx.x;
    {
        const int t = min(tg * T + ti, ntiles);
        load_w(t);
#pragma unroll
        for (int u = 0; u < N; ++u) load(u, t);
    }
    for (int i = slot; i <= j; i += W * 64) red[ti][i] = 0.0;
    __syncthreads();
    double nrm = 0.0;
    for (int buf = 0; tg < ngroups; tg += G, buf ^= B - 1) {
        // keeps the columns' addresses from being held over the loop (they spill)
        asm volatile("" : "+v"(lane));
        asm volatile("" : "+s"(p), "+s"(K));
        const int t = min(tg * T + ti, ntiles);
        double* sw = rows[buf][ti];
#pragma unroll
        for (int i = 0; i < S; ++i) sw[padded(row(i & -P)) + i % P] = wn[i];
        double acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0;
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (u < K) rs[u].axpy(hc[p + W * u], acc);
        for (int k = N; k < K; k += 4) {
            Tile<FMT> tl[4];
            const int cols[4] = {col(k), col(k + 1), col(k + 2), col(k + 3)};
            load_tiles<FMT, 4, kBound>(tl, V, cols, t * kTile, lane);
#pragma unroll
            for (int u = 0; u < 4; ++u) tl[u].axpy(k + u < K ? hc[col(k + u)] : 0.0, acc);
        }
        double wv[8];
        if constexpr (W > 1) {
#pragma unroll
            for (int q = 0; q < 8; ++q) lds.xch[wave][q][lane] = acc[q];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const int q = p + i * W;
                double s = lds.xch[ti * W][q][lane];
#pragma unroll
                for (int k = 1; k < W; ++k) s += lds.xch[ti * W + k][q][lane];
                sw[padded(Map<FMT>::row(lane, q))] -= s;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 8; ++q) wv[q] = sw[padded(Map<FMT>::row(lane, q))];
        } else {
            barrier();
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                double& x = sw[padded(Map<FMT>::row(lane, q))];
                wv[q] = x - acc[q];
                x = wv[q];
            }
            barrier();
        }
#pragma unroll
        for (int i = 0; i < S; i += P) {
            const int r = t * kTile + row(i);
            double2 x;
            x.x = sw[padded(row(i))];
            x.y = P == 2 ? sw[padded(row(i)) + 1] : 0.0;
            nrm = fma(x.y, x.y, fma(x.x, x.x, nrm));  // rows >= n hold 0
            if (P == 2 && r + 1 < V.n) *reinterpret_cast<double2*>(w + r) = x;
            else if (r < V.n) w[r] = x.x;
        }
        for (int k = N; k < K; k += 4) {
            Tile<FMT> tl[4];
            const int cols[4] = {col(k), col(k + 1), col(k + 2), col(k + 3)};
            load_tiles<FMT, 4, kBound>(tl, V, cols, t * kTile, lane);
            double d[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) d[u] = u < 4 ? tl[u & 3].dot(wv) : 0.0;
            const double sum = wave_sum8(d);
            const int kk = k + (lane >> 3);
            if ((lane & 7) == 0 && lane < 32 && kk < K) red[ti][p + W * kk] += sum;
        }
        const int next = min((tg + G) * T + ti, ntiles);
        if (W == 1) barrier();  // the rows have been read
        load_w(next);
#pragma unroll
        for (int k = 0; k < N; k += 8) {
            double d[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                d[u] = 0.0;
                if (k + u < N) {
                    opaque<FMT>(rs[k + u]);
                    if (k + u < K) d[u] = rs[k + u].dot(wv);
                    load(k + u, next);
                }
            }
            const double sum = wave_sum8(d);
            const int kk = k + (lane >> 3);
            if ((lane & 7) == 0 && kk < min(K, N)) red[ti][p + W * kk] += sum;
        }
    }
    nrm = wave_sum(nrm);
    if (lane == 0) part[wave] = nrm;
    __syncthreads();
    // the epilogue is 256 threads' work
    if (wave >= kThreads / 64) return;
    for (int i = threadIdx.x; i <= j; i += kThreads) {
        double s;
        if (i == j) {
            s = part[0];
            for (int k = 1; k < NW; ++k) s += part[k];
        } else {
            s = red[0][i];
#pragma unroll
            for (int k = 1; k < T; ++k) s += red[k][i];
        }
        store_partial(partials + (int64_t)i * G + blockIdx.x, s);
    }
    if (e.mode != EPI_PARTIALS) epilogue(e, partials, lds.epi);
}

// The same for the few columns of a solver step's start, each read twice, the
// second time from the cache: one wave per tile and no registers held.  In a
// solve the data come from HBM behind the SpMV, and what counts is how soon
// the loads go out (launch_subtract_project says when).
// At most 256 registers (two waves per SIMD): with one, a launch of more
// workgroups than CUs runs in two rounds and pays its start-up twice.
template <int FMT, int U>
__global__ __launch_bounds__(kThreads, 2) void k_subtract_project_few(BasisView V, int j,
                                                               const double* __restrict__ h,
                                                               double* __restrict__ w,
                                                               double* __restrict__ partials,
                                                               const int* __restrict__ guard, Epi e) {
    __shared__ double elds[kEpiLds];
    __shared__ double hc[kMaxRestart + 1];
    __shared__ double red[kThreads / 64][kMaxRestart + 2];
    __shared__ double stage[kThreads / 64][kTile];
    const int go = load_coefficients(guard, nullptr, h, j, hc);
    if (!go) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int G = gridDim.x;
    const int ngroups = row_groups_dev(V.np);
    for (int i = lane; i < j; i += 64) red[wave][i] = 0.0;
    __syncthreads();
    double nrm = 0.0;
    for (int rg = blockIdx.x; rg < ngroups; rg += G) {
        const int tile0 = rg * kRowsPerWG + wave * kTile;
        double acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0;
        const bool full = tile0 + kTile <= V.np;
        if (full) subtract_tile<FMT, U, kFull>(V, j, hc, tile0, lane, acc);
        else subtract_tile<FMT, U, 0>(V, j, hc, tile0, lane, acc);
        double wv[8];
        load_rows<FMT>(w, tile0, lane, V.n, wv);
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            wv[q] = wv[q] - acc[q];
            t = fma(wv[q], wv[q], t);  // rows >= n hold 0
        }
        nrm += t;
        store_rows_lds<FMT>(w, tile0, lane, V.n, wv, stage[wave]);
        if (full) project_tile_narrow<FMT, kFull>(V, 0, j, tile0, lane, wv, red[wave]);
        else project_tile_narrow<FMT, 0>(V, 0, j, tile0, lane, wv, red[wave]);
    }
    const double wn = wave_sum(nrm);
    if (lane == 0) red[wave][j] = wn;
    __syncthreads();
    for (int i = tid; i <= j; i += kThreads) {
        double s = red[0][i];
#pragma unroll
        for (int k = 1; k < kThreads / 64; ++k) s += red[k][i];
        store_partial(partials + (int64_t)i * G + blockIdx.x, s);
    }
    epilogue(e, partials, elds);
}

// ----------------------------------------------------------------- stage 2
__global__ __launch_bounds__(256) void k_reduce(const double* __restrict__ partials, int G,
                                                double* __restrict__ out, int op,
                                                const int* __restrict__ guard) {
    if (guard && ld_ctl(guard) == 0) return;
    const int c = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < G; i += 256) s += partials[(int64_t)c * G + i];
    s = block_sum<256>(s);
    if (threadIdx.x == 0) out[c] = op ? ld_ctl(&out[c]) + s : s;
}

__global__ void k_fill(double* __restrict__ x, double v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// ----------------------------------------------------------------- launchers
#define CB_DISPATCH(fmt, KERNEL_CALL)                      \
    switch (kernel_format(fmt)) {                          \
    case CB_F64: { constexpr int F = CB_F64; KERNEL_CALL; break; }           \
    case CB_F32: { constexpr int F = CB_F32; KERNEL_CALL; break; }           \
    case CB_F16: { constexpr int F = CB_F16; KERNEL_CALL; break; }           \
    case CB_FRSZ2_16: { constexpr int F = CB_FRSZ2_16; KERNEL_CALL; break; } \
    case CB_FRSZ2_21: { constexpr int F = CB_FRSZ2_21; KERNEL_CALL; break; } \
    case CB_FRSZ2_GEN: { constexpr int F = CB_FRSZ2_GEN; KERNEL_CALL; break; } \
    case CB_FRSZ2_16_B64: { constexpr int F = CB_FRSZ2_16_B64; KERNEL_CALL; break; } \
    case CB_FRSZ2_32_B64: { constexpr int F = CB_FRSZ2_32_B64; KERNEL_CALL; break; } \
    default: { constexpr int F = CB_FRSZ2_32; KERNEL_CALL; break; }          \
    }

// Non-temporal basis loads pay off once the columns one pass reads no longer
// fit in the 256 MB Infinity Cache next to the rest of the working set; below
// that, the solver's four passes per step over the same columns hit in it.
constexpr int kResidentWaves = 2048;

// Rows up to which the projection runs a column per workgroup: a call takes 8.5
// us against 11.5 of the two launches from 1000 to 32768 rows, 11 against 12 at
// 65536, 20 against 12 at 131072 (17 and 100 columns alike).
constexpr int kColumnRows = 1 << 15;

static int streams_basis(const BasisView& b, int j) {
    constexpr int64_t kCacheResident = (int64_t)192 << 20;
    return (int64_t)j * (b.col_bytes + 4 * b.exp_stride) > kCacheResident;
}

void launch_store(int fmt, const cb_basis& V, int col, const double* w, const double* divisor,
                  double* v_out, int32_t* flag, const int* guard, hipStream_t s) {
    BasisView b = view_of(V);
    unsigned char* vals = static_cast<unsigned char*>(V.values) + (int64_t)col * b.col_bytes;
    uint32_t* ex = V.exps ? V.exps + (int64_t)col * b.exp_stride : nullptr;
    dim3 grid((unsigned)row_groups(V.n));
    CB_DISPATCH(fmt, (k_store<F><<<grid, kThreads, 0, s>>>(vals, ex, b.n, b.np, w, divisor, v_out,
                                                           flag, guard, b.bits, b.bs_log)));
}

void launch_load(int fmt, const cb_basis& V, int col, double* x, hipStream_t s) {
    BasisView b = view_of(V);
    dim3 grid((unsigned)row_groups(V.n));
    CB_DISPATCH(fmt, (k_load<F><<<grid, kThreads, 0, s>>>(b, col, x)));
}

int launch_project(int fmt, const cb_basis& V, int j, const double* w, double* partials,
                    const int* guard, const Epi& e, hipStream_t s) {
    BasisView b = view_of(V);
    const int G = dot_groups(V.n);
    // Column chunks (multiples of 8 columns) only while the launch has fewer
    // waves than the GPU keeps resident (~2048 at this kernel's register
    // use): every workgroup pays a fixed tail (its partial stores and ticket),
    // so workgroups are made as long as the resident waves allow.
    int chunks = kResidentWaves / (4 * G);
    chunks = chunks < 1 ? 1 : chunks;
    int max_chunks = (j + 15) / 16;
    const int ngroups = (G + kTicketGroup - 1) / kTicketGroup;  // ticket groups per chunk
    if (max_chunks > kMaxTicketGroups / ngroups) max_chunks = kMaxTicketGroups / ngroups;
    chunks = chunks > max_chunks ? max_chunks : chunks;
    chunks = chunks < 1 ? 1 : chunks;
    int cw = (j + chunks - 1) / chunks;
    cw = (cw + 7) / 8 * 8;
    chunks = (j + cw - 1) / cw;
    dim3 grid((unsigned)G, (unsigned)chunks);
    Epi ee = e;
    ee.G = G;
    ee.ncols = j;
    ee.cw = cw;
    const int stream = streams_basis(b, j);
    CB_DISPATCH(fmt, (k_project<F><<<grid, kThreads, 0, s>>>(b, j, w, partials, G, cw, stream, guard, ee)));
    return G;
}

bool launch_project_column(int fmt, const cb_basis& V, int j, const double* w, double* h, hipStream_t s) {
    if (V.n > kColumnRows) return false;
    BasisView b = view_of(V);
    CB_DISPATCH(fmt, (k_project_column<F><<<j, 512, 0, s>>>(b, w, h)));
    return true;
}

constexpr int kFewCus = 32;  // CUs of the smallest partition of the GPU: so many workgroups are one round
static int current_device() {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess ? dev : -1;
}
// Workgroups of `kernel` the current device holds at once (its occupancy per
// CU times the CU count), cached per device and kernel; 0 if the runtime
// cannot say.
static int resident_groups(const void* kernel, int id, int threads, int dev) {
    constexpr int kDevs = 16, kIds = 112;
    static std::atomic<int> cache[kDevs][kIds];
    if (dev < 0 || dev >= kDevs || id < 0 || id >= kIds) return 0;
    int r = cache[dev][id].load(std::memory_order_relaxed);
    if (r > 0) return r;
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess)
        return 0;
    r = cus * per_cu;
    if (r > 0) cache[dev][id].store(r, std::memory_order_relaxed);
    return r;
}

int launch_subtract(int fmt, const cb_basis& V, int j, const int* jdev, const double* h,
                     double* w, double* partials, const int* guard, int sign, const Epi& e,
                     hipStream_t s) {
    BasisView b = view_of(V);
    int G = project_groups(V.n);
    // Whole rounds of resident workgroups: three frsz2_21 ones fit a CU, and 1024
    // ran as 768 and then 256, one to a CU, 982 us at 2^24 x 101 where 768 that loop
    // over the row groups take 907 (frsz2_12 734 and 633; two or four to a CU: as before).
    int R = 0;
    if (G > kFewCus)
        CB_DISPATCH(fmt, (R = resident_groups(reinterpret_cast<const void*>(&k_subtract<F, 4>), 96 + F, kThreads,
                                              current_device())));
    if (R > 0 && G > R) G = G / R * R;
    dim3 grid((unsigned)G);
    Epi ee = e;
    ee.G = G;
    ee.ncols = 1;
    ee.cw = 1;
    // with the count on the device, size the policy for the largest count j
    const int stream = streams_basis(b, j);
    CB_DISPATCH(fmt, (k_subtract<F, 4><<<grid, kThreads, 0, s>>>(b, j, jdev, h, w, partials, sign, stream,
                                                                guard, ee)));
    return G;
}

// The solver's launches read few columns twice: up to 12 that together take up to
// 56 MB, but of float64.  From traces of solves with n = 2^15 to 2^22, banded and
// stencil, six formats, each step by both kernels: over the first 12 steps of a
// cycle this choice is 1.9% above the faster kernel at each step, one read always
// 6.9%, 12 columns of any size 6.7% (us a step, one read / two: n = 2^19 x 8
// frsz2_16 15.8 / 13.5, frsz2_32 16.8 / 14.1; 2^21 x 11 frsz2_16 32.0 / 28.7, 2^21 x 8
// float32 27.9 / 34.4, float64 36.1 / 52.2; 2^15 x 16 frsz2_32 13.1 / 14.7).  Over 100
// steps either choice is within 1.3%.  (The primitive's launches, hot in the
// cache, are faster read once at any count.)
constexpr int kFewColumns = 12;
constexpr int64_t kFewBytes = 56000000;

// What the exchange between a tile's waves costs a round of the one-read kernel,
// in columns.  Over 91 random sizes timed with each W (eight formats, 6*10^4 to
// 2*10^6 rows, 3 to 52 columns) the choice with one is 1.3% above the fastest, with
// four 2.2%: that stays with few waves too long (frsz2b64_32 at 597306 x 22 24.8 us
// with W = 2, 22.1 with 8; float32 at 1230550 x 16 26.1 with 1, 21.1 with 4).
constexpr int kExchangeColumns = 1;

// Workgroups of that kernel with W waves a tile: what the GPU holds, cut to the
// partial sums there is room for (capacity doubles) and to the fewest that take
// the same number of rounds over the tiles.
struct SubProjGrid {
    int G;
    int64_t rounds;
};
template <int FMT, int W, int N>
static SubProjGrid sub_proj_grid(const BasisView& b, int j, int64_t capacity, int dev) {
    constexpr int threads = sub_proj_threads(W), T = threads / 64 / W;
    const int ngroups = ((b.np + kTile - 1) / kTile + T - 1) / T;
    const int R = resident_groups(reinterpret_cast<const void*>(&k_subtract_project<FMT, W, N>),
                                  FMT * 5 + (W > 1) + (W > 2) + (W > 4) + (N < kResidentColumns<FMT> ? 4 : 0), threads,
                                  dev);
    int64_t G = R > 0 ? R : 256;
    if (G > capacity / (j + 1)) G = capacity / (j + 1);
    if (G > kTicketGroup * kMaxTicketGroups) G = kTicketGroup * kMaxTicketGroups;
    const int64_t rounds = (ngroups + G - 1) / G;
    G = (ngroups + rounds - 1) / rounds;
    return {(int)G, rounds};
}
template <int FMT, int W, int N>
static int run_subtract_project(const BasisView& b, int j, const double* h, double* w, double* partials,
                                int64_t capacity, int dev, const int* guard, Epi e, hipStream_t s) {
    const int G = sub_proj_grid<FMT, W, N>(b, j, capacity, dev).G;
    e.G = G;
    e.ncols = j + 1;  // u_0 .. u_{j-1} and the norm
    e.cw = j + 1;
    k_subtract_project<FMT, W, N><<<(unsigned)G, sub_proj_threads(W), 0, s>>>(b, j, h, w, partials, guard, e);
    return G;
}

int launch_subtract_project(int fmt, const cb_basis& V, int j, const double* h, double* w, double* partials,
                            int64_t capacity, const int* guard, const Epi& e, hipStream_t s) {
    BasisView b = view_of(V);
    const int dev = current_device();
    int G = 0;
    if (e.mode != EPI_PARTIALS && j <= kFewColumns && j * (b.col_bytes + 4 * b.exp_stride) <= kFewBytes &&
        fmt != CB_F64) {
        G = project_groups(V.n);
        CB_DISPATCH(fmt, ({
            if constexpr (F != CB_F64) {
                // whole waves of resident workgroups
                const int R = resident_groups(reinterpret_cast<const void*>(&k_subtract_project_few<F, 4>), 80 + F,
                                              kThreads, dev);
                if (R > 0 && G > R) G = G / R * R;
                Epi ee = e;
                ee.G = G;
                ee.ncols = j + 1;
                ee.cw = j + 1;
                k_subtract_project_few<F, 4><<<G, kThreads, 0, s>>>(b, j, h, w, partials, guard, ee);
            }
        }));
        return G;
    }
    CB_DISPATCH(fmt, ({
        constexpr int N = kResidentColumns<F>;
        // among the W whose waves hold the columns (8 if none does) the one with
        // the fewest rounds over the tiles, each as long as a wave has columns and,
        // with more than one wave, an exchange; the smallest such W.  The rounds are
        // those of the grids that will run, whose partial sums have to fit
        // (reckoned with 2048 resident waves and no exchange, frsz2_16 at 200003 x 40
        // took 24.4 us, now 20.0; two reads of the columns 21.3)
        int W = 0;
        int64_t best = INT64_MAX;
        auto weigh = [&](int v, int64_t rounds) {
            const int64_t cost = rounds * ((j + v - 1) / v + (v > 1 ? kExchangeColumns : 0));
            if (cost < best) {
                best = cost;
                W = v;
            }
        };
        if (N >= j) weigh(1, sub_proj_grid<F, 1, N>(b, j, capacity, dev).rounds);
        if (2 * N >= j) weigh(2, sub_proj_grid<F, 2, N>(b, j, capacity, dev).rounds);
        if (4 * N >= j) weigh(4, sub_proj_grid<F, 4, N>(b, j, capacity, dev).rounds);
        weigh(8, sub_proj_grid<F, 8, N>(b, j, capacity, dev).rounds);
        // few columns in fewer registers, where a third workgroup then fits a CU
        // (2^21 x 8: float32 22.4 -> 21.8 us, frsz2_16 21.8 -> 21.4)
        constexpr int Few = N > 13 ? 8 : N;
        if (W == 1 && j <= Few) G = run_subtract_project<F, 1, Few>(b, j, h, w, partials, capacity, dev, guard, e, s);
        else if (W == 1) G = run_subtract_project<F, 1, N>(b, j, h, w, partials, capacity, dev, guard, e, s);
        else if (W == 2) G = run_subtract_project<F, 2, N>(b, j, h, w, partials, capacity, dev, guard, e, s);
        else if (W == 4) G = run_subtract_project<F, 4, N>(b, j, h, w, partials, capacity, dev, guard, e, s);
        else G = run_subtract_project<F, 8, N>(b, j, h, w, partials, capacity, dev, guard, e, s);
    }));
    return G;
}

void launch_reduce(const double* partials, int G, int ncols, double* out, int op, const int* guard,
                   hipStream_t s) {
    if (ncols <= 0) return;
    k_reduce<<<ncols, 256, 0, s>>>(partials, G, out, op, guard);
}

void launch_fill(double* x, double v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    k_fill<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, v, n);
}

}  // namespace cb
