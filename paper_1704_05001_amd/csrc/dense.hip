// Direct solves on the coarsest level of each system: the dense operator of a
// system's block rows, its inverse by Gauss-Jordan elimination with partial
// pivoting (blocked, the updates on the FP64 matrix cores: in one workgroup's
// LDS up to 128 unknowns, over the whole chip panel by panel up to 4096), and
// the inverse's transpose for the transposed cycle.  A batched hierarchy holds many such systems
// ("segments": a contiguous range of block rows each) on one level.
#include <algorithm>
#include <vector>

#include "common.h"
#include "mfma_tile.h"

namespace nair {
namespace {

constexpr int kGJThreads = 1024;

template <int V>
struct Ctrl {
    static constexpr int v = V;
};
// v of lane l (the same l in every lane)
__device__ inline double lane_value(double v, int l) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(u), l);
    const int hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), l);
    return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// Segment k = blockIdx.y: block row blk0[k] + blockIdx.x into the dense n x n
// matrix at M + off[k] (n = nbk[k] * bs, columns relative to blk0[k]).
__global__ __launch_bounds__(256) void k_bsr_to_dense(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                     const double *__restrict__ vals, int bs,
                                                     const int *__restrict__ blk0, const int *__restrict__ nbk,
                                                     const int64_t *__restrict__ off, double *__restrict__ M) {
    const int k = blockIdx.y;
    const int i = blockIdx.x;
    if (i >= nbk[k]) return;
    const int b0 = blk0[k];
    const int I = b0 + i;
    const int n = nbk[k] * bs;
    const int bb = bs * bs;
    double *Mk = M + off[k];
    for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
        const int J = colidx[t] - b0;
        for (int e = threadIdx.x; e < bb; e += blockDim.x) {
            const int a = e / bs, b = e - a * bs;
            Mk[static_cast<int64_t>(i * bs + a) * n + J * bs + b] = vals[static_cast<int64_t>(t) * bb + e];
        }
    }
}

// Orders past 4096 (a level cut off by max_levels; a stalled splitting of that
// size is refused): the elimination a column at a time in one workgroup, from
// global memory.
__global__ __launch_bounds__(kGJThreads) void k_gauss_jordan(double *__restrict__ M, double *__restrict__ Inv, int n,
                                                            double *__restrict__ colk, int *__restrict__ singular) {
    __shared__ double rv[kGJThreads];
    __shared__ int ri[kGJThreads];
    const int tid = threadIdx.x;
    const int64_t nn = static_cast<int64_t>(n) * n;
    for (int64_t e = tid; e < nn; e += kGJThreads) Inv[e] = (e / n == e % n) ? 1.0 : 0.0;
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        double v = -1.0;
        int idx = n;
        for (int i = k + tid; i < n; i += kGJThreads) {
            const double av = fabs(M[static_cast<int64_t>(i) * n + k]);
            if (av > v || (av == v && i < idx)) {
                v = av;
                idx = i;
            }
        }
        rv[tid] = v;
        ri[tid] = idx;
        __syncthreads();
        for (int s = kGJThreads / 2; s > 0; s >>= 1) {
            if (tid < s) {
                const double ov = rv[tid + s];
                const int oi = ri[tid + s];
                if (ov > rv[tid] || (ov == rv[tid] && oi < ri[tid])) {
                    rv[tid] = ov;
                    ri[tid] = oi;
                }
            }
            __syncthreads();
        }
        const double best = rv[0];
        const int p = ri[0];
        __syncthreads();
        if (!(best > 0.0)) {
            if (tid == 0) *singular = 1;
            return;
        }
        if (p != k) {
            for (int j = tid; j < n; j += kGJThreads) {
                double t = M[static_cast<int64_t>(k) * n + j];
                M[static_cast<int64_t>(k) * n + j] = M[static_cast<int64_t>(p) * n + j];
                M[static_cast<int64_t>(p) * n + j] = t;
                t = Inv[static_cast<int64_t>(k) * n + j];
                Inv[static_cast<int64_t>(k) * n + j] = Inv[static_cast<int64_t>(p) * n + j];
                Inv[static_cast<int64_t>(p) * n + j] = t;
            }
        }
        __syncthreads();
        const double piv = M[static_cast<int64_t>(k) * n + k];
        __syncthreads();
        for (int j = tid; j < n; j += kGJThreads) {
            M[static_cast<int64_t>(k) * n + j] /= piv;
            Inv[static_cast<int64_t>(k) * n + j] /= piv;
        }
        __syncthreads();
        for (int i = tid; i < n; i += kGJThreads) colk[i] = M[static_cast<int64_t>(i) * n + k];
        __syncthreads();
        for (int64_t e = tid; e < nn; e += kGJThreads) {
            const int i = static_cast<int>(e / n);
            if (i == k) continue;
            const int j = static_cast<int>(e - static_cast<int64_t>(i) * n);
            const double f = colk[i];
            if (f == 0.0) continue;
            if (j > k) M[e] -= f * M[static_cast<int64_t>(k) * n + j];
            Inv[e] -= f * Inv[static_cast<int64_t>(k) * n + j];
        }
        __syncthreads();
    }
}

// Blocked in-place Gauss-Jordan inversion with partial pivoting.  A panel of
// PW columns is eliminated in registers, a row per lane: for each column the
// largest entry of a row not yet a pivot row is the pivot, the pivot row is
// scaled (a_pk replaced by 1) and every other row eliminates (a_ik replaced by
// 0).  Rows are never exchanged: prow[k] is column k's pivot row, upos its
// inverse.  What is left in the panel, G, turns the other columns' entries into
// a_i <- (a_i, or 0 on the panel's pivot rows) + sum_k G_ik a_prow(k): a rank-PW
// update that runs on the FP64 matrix cores.  After the last panel
// inv[k][prow[j]] = a[prow[k]][j].

// Largest v of the wave (the same value in every lane).
__device__ inline double wave_max(double v) {
    auto mv = [](double x, auto ctrl) {
        const long long u = __double_as_longlong(x);
        const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), decltype(ctrl)::v, 0xF, 0xF, false);
        const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), decltype(ctrl)::v, 0xF, 0xF, false);
        return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
    };
    v = fmax(v, mv(v, Ctrl<0xB1>{}));    // quad_perm 1,0,3,2
    v = fmax(v, mv(v, Ctrl<0x4E>{}));    // quad_perm 2,3,0,1
    v = fmax(v, mv(v, Ctrl<0x141>{}));   // row_half_mirror
    v = fmax(v, mv(v, Ctrl<0x140>{}));   // row_mirror
    return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}

// One column's elimination in this lane's R rows: `row` is the unscaled pivot
// row (its entry c the pivot), mine[r] the lane's r-th row, is_piv its flag.
template <int R, int PW>
__device__ inline void eliminate(double (&mine)[R][PW], const bool (&is_piv)[R], const double (&row)[PW], int c) {
    const double inv = 1.0 / row[c];
    double f[R];
#pragma unroll
    for (int r = 0; r < R; ++r) f[r] = mine[r][c];
#pragma unroll
    for (int j = 0; j < PW; ++j) {
        const double s = j == c ? inv : row[j] * inv;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double old = j == c ? 0.0 : mine[r][j];
            mine[r][j] = is_piv[r] ? s : __builtin_fma(-f[r], s, old);
        }
    }
}

constexpr int kInvThreads = 512;
constexpr int kLdsOrder = 128;   // largest order inverted in one workgroup's LDS
constexpr int kPanel = 16;

// One workgroup per listed segment k = sel[blockIdx.x]: the n x n matrix at
// Mall + off[k] (n = nbk[k] * bs <= 128) inverted into invall + off[k] in one
// launch, the matrix in LDS, padded to whole 16 x 16 tiles by an identity.  The
// first wave eliminates a panel (two rows per lane, the pivot row broadcast by
// readlane: no barrier inside a panel), then every wave updates whole 16-column
// strips, so a strip's pivot rows are read before the wave overwrites them.
// Bound by the panels' serial chain (below 1 us per column): 112 us at n = 108
// (140 with the pivot's selects on both rows of a lane), where a column at a time
// over the whole workgroup, with six barriers per column, took 420 us at n = 126.
__global__ __launch_bounds__(kInvThreads) void k_invert_lds(const double *__restrict__ Mall,
                                                           double *__restrict__ invall,
                                                           const int *__restrict__ sel, const int *__restrict__ nbk,
                                                           int bs, const int64_t *__restrict__ off,
                                                           int *__restrict__ singular_all) {
    extern __shared__ double a[];
    __shared__ int prow[kLdsOrder], upos[kLdsOrder];
    __shared__ int bad;
    const int seg = sel[blockIdx.x];
    const int n = nbk[seg] * bs;
    const int np = (n + kPanel - 1) / kPanel * kPanel;
    const int ld = np + 1;   // (rows on different banks)
    const double *Min = Mall + off[seg];
    double *inv = invall + off[seg];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row16 = lane & 15, kk = lane >> 4;
    for (int e = tid; e < np * np; e += kInvThreads) {
        const int i = e / np, j = e - i * np;
        a[i * ld + j] = (i < n && j < n) ? Min[static_cast<int64_t>(i) * n + j] : (i == j ? 1.0 : 0.0);
    }
    if (tid < kLdsOrder) upos[tid] = -1;
    if (tid == 0) bad = 0;
    __syncthreads();
    bool used[2] = {lane >= np, lane + 64 >= np};   // (first wave) rows that are pivot rows already, or do not exist
    for (int k0 = 0; k0 < np; k0 += kPanel) {
        if (wave == 0) {
            double p[2][kPanel];
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < kPanel; ++j) p[r][j] = lane + 64 * r < np ? a[(lane + 64 * r) * ld + k0 + j] : 0.0;
            bool ok = true;
#pragma unroll
            for (int c = 0; c < kPanel; ++c) {   // (no exit from the loop: unrolled, p stays in registers)
                const double v0 = used[0] ? -1.0 : fabs(p[0][c]), v1 = used[1] ? -1.0 : fabs(p[1][c]);
                const double best = wave_max(fmax(v0, v1));
                ok = ok && best > 0.0;
                const unsigned long long b0 = __ballot(v0 == best), b1 = __ballot(v1 == best);
                const int l = __builtin_ctzll(b0 ? b0 : (b1 ? b1 : 1ull));
                // (the pivot row's half is the same in every lane: only its rows need the pivot's select)
                const bool is_piv[2] = {b0 != 0ull && lane == l, b0 == 0ull && lane == l};
                double row[kPanel];
                if (b0) {
#pragma unroll
                    for (int j = 0; j < kPanel; ++j) row[j] = lane_value(p[0][j], l);
                    const bool piv[2] = {lane == l, false};
                    eliminate<2, kPanel>(p, piv, row, c);
                } else {
#pragma unroll
                    for (int j = 0; j < kPanel; ++j) row[j] = lane_value(p[1][j], l);
                    const bool piv[2] = {false, lane == l};
                    eliminate<2, kPanel>(p, piv, row, c);
                }
                used[0] = used[0] || is_piv[0];
                used[1] = used[1] || is_piv[1];
                if (lane == 0 && ok) {
                    const int pr = l + (b0 ? 0 : 64);
                    prow[k0 + c] = pr;
                    upos[pr] = k0 + c;
                }
            }
            if (!ok) {
                if (lane == 0) bad = 1;
            } else {
#pragma unroll
                for (int r = 0; r < 2; ++r)
                    if (lane + 64 * r < np)
#pragma unroll
                        for (int j = 0; j < kPanel; ++j) a[(lane + 64 * r) * ld + k0 + j] = p[r][j];
            }
        }
        __syncthreads();
        if (bad) {
            if (tid == 0) singular_all[seg] = 1;
            return;
        }
        for (int st = wave; st * kPanel < np; st += kInvThreads / 64) {
            const int j0 = st * kPanel;
            if (j0 == k0) continue;
            double b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) b[q] = a[prow[k0 + 4 * q + kk] * ld + j0 + row16];
            for (int i0 = 0; i0 < np; i0 += kPanel) {
                double4_t acc;
                double g[4], old[4];
                int u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {   // (every read first)
                    const int i = i0 + kk + 4 * q;
                    g[q] = a[(i0 + row16) * ld + k0 + 4 * q + kk];
                    u[q] = upos[i];
                    old[q] = a[i * ld + j0 + row16];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = (u[q] >= k0 && u[q] < k0 + kPanel) ? 0.0 : old[q];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(g[q], b[q], acc, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) a[(i0 + kk + 4 * q) * ld + j0 + row16] = acc[q];
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < n * n; e += kInvThreads) {
        const int k = e / n, m = e - k * n;
        inv[e] = a[prow[k] * ld + upos[m]];
    }
}

// The same inversion for larger orders, one launch per panel and one workgroup
// per 16-column strip of each listed segment (blockIdx.y): step t applies panel
// t - 1 to the strips, and workgroup 0 takes strip t / the next panel's columns
// first and then eliminates that panel, while the others still update theirs.
// A panel's G stays in its columns, prow / upos (at off of their own) in global
// memory.  R rows per thread hold a panel of PW columns in registers, so n <=
// 512 R.  Each column is one barrier: every wave offers its best row whole, the
// workgroup takes the best of the eight.  Bound by that chain (28, 53 and 95 us
// per panel at one, two and four rows per thread).  Setup of a directly solved
// system of 250 / 825 / 2000 unknowns: 0.68 / 3.1 / 12.6 ms, against 11.3 / 514
// / 7219 ms with one workgroup taking a column at a time from global memory
// (k_gauss_jordan, which is left the orders past 4096).
template <int R, int PW>
__global__ __launch_bounds__(kInvThreads) void k_invert_step(double *__restrict__ Mall, const int *__restrict__ sel,
                                                            const int *__restrict__ nbk, int bs,
                                                            const int64_t *__restrict__ off,
                                                            const int *__restrict__ poff, int t,
                                                            int *__restrict__ prow_all, int *__restrict__ upos_all,
                                                            int *__restrict__ singular_all) {
    constexpr int kWaves = kInvThreads / 64;
    constexpr int KQ = PW / 4;
    __shared__ double cand[2][kWaves][PW];
    __shared__ double candv[2][kWaves];
    __shared__ int candr[2][kWaves];
    const int seg = sel[blockIdx.y];
    const int n = nbk[seg] * bs;
    // (launch t marks a singular segment with t + 1: a mark of this very launch is not acted on,
    // so all threads of a workgroup decide alike)
    const int mark = singular_all[seg];
    if (mark != 0 && mark <= t) return;
    const int nst = (n + PW - 1) / PW;   // panels, and update strips per segment
    if (t > nst) return;
    double *M = Mall + off[seg];
    int *prow = prow_all + poff[blockIdx.y], *upos = upos_all + poff[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row16 = lane & 15, kk = lane >> 4;
    // strips of 16 columns: workgroup 0 takes the one that holds panel t's columns (PW = 16: strip t)
    const int ncol16 = (n + 15) / 16;
    const int mine = t < nst ? (t * PW) / 16 : -1;
    int st = static_cast<int>(blockIdx.x);
    if (mine >= 0) st = st == 0 ? mine : (st <= mine ? st - 1 : st);
    if (t > 0 && st < ncol16) {
        const int k0 = (t - 1) * PW;
        const int w = min(PW, n - k0);   // columns of the panel
        const int j = st * 16 + row16;
        const bool in = j < n && !(j >= k0 && j < k0 + w);   // the panel's own columns hold G
        double b[KQ];
#pragma unroll
        for (int q = 0; q < KQ; ++q)
            b[q] = (4 * q + kk < w && in) ? M[static_cast<int64_t>(prow[k0 + 4 * q + kk]) * n + j] : 0.0;
        __syncthreads();   // every wave holds the pivot rows of its strip before one overwrites them
        const int jc = min(j, n - 1);
        for (int i0 = wave * 16; i0 < n; i0 += kWaves * 16) {
            // every load first, at indices clamped into the matrix, then the selections
            double4_t acc;
            double g[KQ], old[4];
            int u[4];
            const int ig = i0 + row16;
#pragma unroll
            for (int q = 0; q < KQ; ++q)
                g[q] = M[static_cast<int64_t>(min(ig, n - 1)) * n + k0 + min(4 * q + kk, w - 1)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = min(i0 + kk + 4 * r, n - 1);
                u[r] = upos[i];
                old[r] = M[static_cast<int64_t>(i) * n + jc];
            }
#pragma unroll
            for (int q = 0; q < KQ; ++q)
                if (ig >= n || 4 * q + kk >= w) g[q] = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = (u[r] >= k0 && u[r] < k0 + w) ? 0.0 : old[r];
#pragma unroll
            for (int q = 0; q < KQ; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(g[q], b[q], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + kk + 4 * r;
                if (i < n && in) M[static_cast<int64_t>(i) * n + j] = acc[r];
            }
        }
    }
    if (blockIdx.x != 0 || t >= nst) return;
    __syncthreads();   // the panel's columns are up to date
    const int k0 = t * PW, w = min(PW, n - k0);
    double p[R][PW];
    bool used[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = tid + kInvThreads * r;
        used[r] = i >= n || upos[i] >= 0;
#pragma unroll
        for (int j = 0; j < PW; ++j) p[r][j] = (i < n && j < w) ? M[static_cast<int64_t>(i) * n + k0 + j] : 0.0;
    }
    bool ok = true;   // (the same in every thread; the unrolled loop has no exit, so p stays in registers)
#pragma unroll
    for (int c = 0; c < PW; ++c) {
        if (!ok || c >= w) continue;
        double v = -1.0;
        int vr = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double av = used[r] ? -1.0 : fabs(p[r][c]);
            if (av > v) {
                v = av;
                vr = r;
            }
        }
        const double wb = wave_max(v);
        const int sl = c & 1;   // (two slots: the next column's offers do not overwrite rows still being read)
        const unsigned long long bal = __ballot(v == wb);
        if (lane == __builtin_ctzll(bal ? bal : 1ull)) {
            candv[sl][wave] = wb;
            candr[sl][wave] = tid + kInvThreads * vr;
#pragma unroll
            for (int j = 0; j < PW; ++j) {
                double x = p[0][j];
#pragma unroll
                for (int r = 1; r < R; ++r) x = r == vr ? p[r][j] : x;
                cand[sl][wave][j] = x;
            }
        }
        __syncthreads();
        double best = candv[sl][0];
        int bw = 0;
#pragma unroll
        for (int k = 1; k < kWaves; ++k) {
            const double ov = candv[sl][k];
            if (ov > best) {
                best = ov;
                bw = k;
            }
        }
        ok = best > 0.0;
        const int pr = candr[sl][bw];
        double row[PW];
#pragma unroll
        for (int j = 0; j < PW; ++j) row[j] = cand[sl][bw][j];
        bool is_piv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            is_piv[r] = tid + kInvThreads * r == pr;
            used[r] = used[r] || is_piv[r];
        }
        eliminate<R, PW>(p, is_piv, row, c);
        if (tid == 0 && ok) {
            prow[k0 + c] = pr;
            upos[pr] = k0 + c;
        }
    }
    if (!ok) {
        if (tid == 0) singular_all[seg] = t + 1;
        return;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = tid + kInvThreads * r;
        if (i < n)
#pragma unroll
            for (int j = 0; j < PW; ++j)
                if (j < w) M[static_cast<int64_t>(i) * n + k0 + j] = p[r][j];
    }
}

// inv[k][prow[j]] = a[prow[k]][j] of the listed segments, read and written along rows of inv
__global__ __launch_bounds__(256) void k_invert_unpermute(const double *__restrict__ Mall, const int *__restrict__ sel,
                                                         const int *__restrict__ nbk, int bs,
                                                         const int64_t *__restrict__ off, const int *__restrict__ poff,
                                                         const int *__restrict__ prow_all,
                                                         const int *__restrict__ upos_all,
                                                         const int *__restrict__ singular_all,
                                                         double *__restrict__ invall) {
    const int seg = sel[blockIdx.y];
    if (singular_all[seg]) return;
    const int n = nbk[seg] * bs;
    const int *prow = prow_all + poff[blockIdx.y], *upos = upos_all + poff[blockIdx.y];
    const double *M = Mall + off[seg];
    double *inv = invall + off[seg];
    for (int k = blockIdx.x; k < n; k += gridDim.x) {
        const double *src = M + static_cast<int64_t>(prow[k]) * n;
        for (int m = threadIdx.x; m < n; m += blockDim.x) inv[static_cast<int64_t>(k) * n + m] = src[upos[m]];
    }
}

__global__ __launch_bounds__(256) void k_transpose_dense(const double *__restrict__ M, double *__restrict__ MT,
                                                        const int *__restrict__ nbk, int bs,
                                                        const int64_t *__restrict__ off) {
    const int k = blockIdx.y;
    const int n = nbk[k] * bs;
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= static_cast<int64_t>(n) * n) return;
    const int i = static_cast<int>(e / n), j = static_cast<int>(e - static_cast<int64_t>(i) * n);
    MT[off[k] + static_cast<int64_t>(j) * n + i] = M[off[k] + e];
}

}  // namespace

int dense_inverse_segments(const DevBSR &A, int nseg, const int *blk0_h, const int *nbk_h, const int64_t *off_h,
                           double *inv, double *invT, hipStream_t s) {
    if (nseg <= 0) return -1;
    const int bs = A.bs;
    int max_nb = 0;
    for (int k = 0; k < nseg; ++k) max_nb = std::max(max_nb, nbk_h[k]);
    const int64_t last_n = static_cast<int64_t>(nbk_h[nseg - 1]) * bs;
    const int64_t total = off_h[nseg - 1] + last_n * last_n;
    const int64_t max_n = static_cast<int64_t>(max_nb) * bs;
    // without the dynamic LDS every segment takes the panel launches
    auto lds_bytes = [](int n) {
        const size_t np = static_cast<size_t>((n + kPanel - 1) / kPanel) * kPanel;
        return sizeof(double) * np * (np + 1);
    };
    const bool lds_ok = allow_lds(reinterpret_cast<const void *>(k_invert_lds), lds_bytes(kLdsOrder));
    std::vector<int> sel_lds, sel_big;
    for (int k = 0; k < nseg; ++k)
        (lds_ok && static_cast<int64_t>(nbk_h[k]) * bs <= kLdsOrder ? sel_lds : sel_big).push_back(k);
    DBuf<double> M(static_cast<size_t>(total));
    DBuf<int> blk0(nseg), nbk(nseg), sing(nseg), sel(sel_lds.empty() ? 1 : sel_lds.size());
    DBuf<int64_t> off(nseg);
    NAIR_HIP(hipMemsetAsync(M.get(), 0, sizeof(double) * static_cast<size_t>(total), s));
    const std::vector<int> none(static_cast<size_t>(nseg), 0);
    const size_t ib = sizeof(int) * static_cast<size_t>(nseg);
    PutJobs J;
    if (J.add(sing.get(), none.data(), ib) && J.add(blk0.get(), blk0_h, ib) && J.add(nbk.get(), nbk_h, ib) &&
        J.add(off.get(), off_h, 2 * ib) && J.add(sel.get(), sel_lds.data(), sizeof(int) * sel_lds.size())) {
        launch_put_words(J, s);
    } else {
        NAIR_HIP(hipMemsetAsync(sing.get(), 0, ib, s));
        NAIR_HIP(hipMemcpyAsync(blk0.get(), blk0_h, ib, hipMemcpyHostToDevice, s));
        NAIR_HIP(hipMemcpyAsync(nbk.get(), nbk_h, ib, hipMemcpyHostToDevice, s));
        NAIR_HIP(hipMemcpyAsync(off.get(), off_h, 2 * ib, hipMemcpyHostToDevice, s));
        if (!sel_lds.empty())
            NAIR_HIP(hipMemcpyAsync(sel.get(), sel_lds.data(), sizeof(int) * sel_lds.size(), hipMemcpyHostToDevice, s));
    }
    k_bsr_to_dense<<<dim3(static_cast<unsigned>(max_nb), static_cast<unsigned>(nseg)), 256, 0, s>>>(
        A.rowptr.get(), A.colidx.get(), A.vals.get(), bs, blk0.get(), nbk.get(), off.get(), M.get());
    NAIR_HIP(hipGetLastError());
    if (!sel_lds.empty()) {
        int lds_n = 0;
        for (int k : sel_lds) lds_n = std::max(lds_n, nbk_h[k] * bs);
        k_invert_lds<<<static_cast<unsigned>(sel_lds.size()), kInvThreads, lds_bytes(lds_n), s>>>(
            M.get(), inv, sel.get(), nbk.get(), bs, off.get(), sing.get());
        NAIR_HIP(hipGetLastError());
    }
    // segments of similar order share their panel launches: up to 512 R unknowns with R rows per thread
    struct Group {
        int max_n;
        std::vector<int> seg;
    } groups[] = {{512, {}}, {1024, {}}, {2048, {}}, {4096, {}}};
    DBuf<double> colk;
    for (int k : sel_big) {
        const int n = nbk_h[k] * bs;
        Group *g = groups;
        while (g != groups + 4 && n > g->max_n) ++g;
        if (g != groups + 4) {
            g->seg.push_back(k);
            continue;
        }
        if (!colk.get()) colk.alloc(static_cast<size_t>(max_n));
        k_gauss_jordan<<<1, kGJThreads, 0, s>>>(M.get() + off_h[k], inv + off_h[k], n, colk.get(), sing.get() + k);
        NAIR_HIP(hipGetLastError());
    }
    std::vector<std::vector<int>> tables;   // (host memory the copies below read until the stream is waited for)
    std::vector<DBuf<int>> keep;
    for (const Group &g : groups) {
        const int m = static_cast<int>(g.seg.size());
        if (m == 0) continue;
        int np = 0, gn = 0;
        std::vector<int> table(g.seg);   // the segments, then where each one's pivot tables start
        for (int k : g.seg) {
            table.push_back(np);
            np += nbk_h[k] * bs;
            gn = std::max(gn, nbk_h[k] * bs);
        }
        tables.push_back(std::move(table));
        keep.emplace_back(static_cast<size_t>(2 * m));
        const int *seld = keep.back().get(), *poff = seld + m;
        NAIR_HIP(hipMemcpyAsync(keep.back().get(), tables.back().data(), sizeof(int) * 2 * m, hipMemcpyHostToDevice, s));
        keep.emplace_back(static_cast<size_t>(2 * np));
        int *prow = keep.back().get(), *upos = prow + np;
        launch_fill_ints({{prow, 2 * static_cast<int64_t>(np), -1}}, s);
        const int pw = gn > 2048 ? kPanel / 2 : kPanel;
        const dim3 grid(static_cast<unsigned>((gn + 15) / 16), static_cast<unsigned>(m));
        for (int t = 0; t <= (gn + pw - 1) / pw; ++t) {
#define NAIR_STEP(R, PW) \
    k_invert_step<R, PW><<<grid, kInvThreads, 0, s>>>(M.get(), seld, nbk.get(), bs, off.get(), poff, t, prow, upos, sing.get())
            if (gn > 2048) NAIR_STEP(8, kPanel / 2);
            else if (gn > 1024) NAIR_STEP(4, kPanel);
            else if (gn > 512) NAIR_STEP(2, kPanel);
            else NAIR_STEP(1, kPanel);
#undef NAIR_STEP
            NAIR_HIP(hipGetLastError());
        }
        k_invert_unpermute<<<dim3(static_cast<unsigned>(std::min(gn, 1024)), static_cast<unsigned>(m)), 256, 0, s>>>(
            M.get(), seld, nbk.get(), bs, off.get(), poff, prow, upos, sing.get(), inv);
        NAIR_HIP(hipGetLastError());
    }
    // (the flags come back with the transposes done: the host arrays and temporaries end here)
    k_transpose_dense<<<dim3(grid_for(max_n * max_n, 256), static_cast<unsigned>(nseg)), 256, 0, s>>>(
        inv, invT, nbk.get(), bs, off.get());
    NAIR_HIP(hipGetLastError());
    std::vector<int> hs(nseg);
    read_ints(sing.get(), hs.data(), nseg, s);
    for (int k = 0; k < nseg; ++k)
        if (hs[k] != 0) return k;
    return -1;
}

}  // namespace nair
