// Row-wise block SpGEMM (Gustavson order): the symbolic phase sorts a row's
// products by (output column, number) within a group of lanes, which gives the
// pattern and per-output-block
// pair lists in the fixed accumulation order; and numeric kernels that walk
// them (FP64 matrix cores for 9x9 and 16x16 blocks, one thread per block row
// otherwise); union-add of two block matrices; and the Galerkin product
// K = R A P with the one-point P and the drop filter.
//
// Determinism: every output entry is one fma chain over the inner block
// index K ascending (the order of X's sorted row, with X's implicit identity
// block merged in at its column), c ascending within a block product,
// starting from +0.  Rows are independent, and each output block's pairs are
// applied in list order by the one wave or thread that owns the block.
#include <algorithm>

#include <climits>

#include "common.h"
#include "mfma_tile.h"

#pragma clang fp contract(off)

namespace nair {
namespace {

constexpr int kWave = 64;

// Inclusive prefix sum of x over the wave's 64 lanes by DPP moves (no LDS
// round trips): shifts by 1, 2, 4, 8 within each row of 16 lanes, then each
// row's last lane added into the rows after it.  A lane whose source lies
// outside its row (or a row the step leaves out) receives 0.
template <int CTRL, int ROWS = 0xF>
__device__ inline int dpp_add(int x) {
    return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, false);
}
__device__ inline int wave_incl_scan(int x) {
    x = dpp_add<0x111>(x);          // row_shr:1
    x = dpp_add<0x112>(x);          // row_shr:2
    x = dpp_add<0x114>(x);          // row_shr:4
    x = dpp_add<0x118>(x);          // row_shr:8
    x = dpp_add<0x142, 0xA>(x);     // row_bcast:15 into rows 1 and 3
    x = dpp_add<0x143, 0xC>(x);     // row_bcast:31 into rows 2 and 3
    return x;
}

// ------------------------------------------------------------- key sorts

// The value of lane (lane ^ D): within rows of 16 lanes by DPP moves.
template <int D>
__device__ inline uint32_t lane_xor32(uint32_t x) {
    const int v = static_cast<int>(x);
    if constexpr (D == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);   // quad_perm 1 0 3 2
    if constexpr (D == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm 2 3 0 1
    if constexpr (D == 4)   // half rows mirrored (xor 7), then quads mirrored (xor 3)
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true), 0x1B, 0xF,
                                           0xF, true);
    if constexpr (D == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);   // row_ror:8
    return static_cast<uint32_t>(__shfl_xor(v, D, kWave));
}
template <int D>
__device__ inline uint32_t lane_xor(uint32_t x) { return lane_xor32<D>(x); }
template <int D>
__device__ inline uint64_t lane_xor(uint64_t x) {
    return static_cast<uint64_t>(lane_xor32<D>(static_cast<uint32_t>(x))) |
           static_cast<uint64_t>(lane_xor32<D>(static_cast<uint32_t>(x >> 32))) << 32;
}

// Bitonic network over the W E keys of each group of W lanes, ascending; key
// number s = lane * E + e.
template <int E, int KK, int J, typename KEY>
__device__ inline void sort_step(KEY (&key)[E], int gl) {
    if constexpr (J >= E) {
        const bool lower = (gl & (J / E)) == 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const KEY o = lane_xor<J / E>(key[e]);
            const bool asc = ((gl * E + e) & KK) == 0;
            key[e] = (lower == asc) == (o < key[e]) ? o : key[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (e & J) continue;
            const KEY a = key[e], b = key[e | J];
            const bool asc = ((gl * E + e) & KK) == 0;
            key[e] = asc == (b < a) ? b : a;
            key[e | J] = asc == (b < a) ? a : b;
        }
    }
    if constexpr (J > 1) sort_step<E, KK, J / 2>(key, gl);
}
template <int W, int E, int KK = 2, typename KEY>
__device__ inline void group_sort(KEY (&key)[E], int gl) {
    sort_step<E, KK, KK / 2>(key, gl);
    if constexpr (KK < W * E) group_sort<W, E, KK * 2>(key, gl);
}

// A sorted group's keys are (column << B | place); a head is the first key of a
// column.  heads(): how many the group has, and per key how many lie at or before it.
template <int W, int E, int B, typename KEY>
__device__ inline int heads(const KEY (&key)[E], int gl, int lane, bool (&head)[E], int (&upto)[E]) {
    const KEY none = ~static_cast<KEY>(0);
    const KEY before = __shfl_up(key[E - 1], 1, W);
    const uint64_t group = W == 64 ? ~0ull : (((1ull << (W & 63)) - 1) << (lane & ~(W - 1)));
    int n = 0, mine = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const KEY prev = e > 0 ? key[e > 0 ? e - 1 : 0] : before;
        head[e] = key[e] != none && ((gl == 0 && e == 0) || (key[e] >> B) != (prev >> B));
        const uint64_t bits = __ballot(head[e]) & group;
        n += __popcll(bits);
        mine += __popcll(bits & ((1ull << lane) - 1));   // lanes before this one
    }
#pragma unroll
    for (int e = 0; e < E; ++e) upto[e] = mine += head[e] ? 1 : 0;
    return n;
}

// ------------------------------------------------------------ upper bounds

// Rows that one wave takes: at most 64 inner slots and 256 products.
constexpr int kWaveProducts = 256;
__device__ inline bool wave_row(int products, int slots) { return products <= kWaveProducts && slots <= kWave; }

// ub[i] = sum of the lengths of Y's rows touched by X's row i (plus the identity's row).
__global__ __launch_bounds__(256) void k_row_upper_bound(const int *__restrict__ xrowptr, const int *__restrict__ xcol,
                                                        const int *__restrict__ xdiag, const int *__restrict__ yrowptr,
                                                        int m, int *__restrict__ ub, int *__restrict__ big_list,
                                                        int *__restrict__ big_count,
                                                        int large_cap, int *__restrict__ too_dense) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int64_t s = 0;
    for (int q = xrowptr[i]; q < xrowptr[i + 1]; ++q) s += yrowptr[xcol[q] + 1] - yrowptr[xcol[q]];
    if (xdiag) s += yrowptr[xdiag[i] + 1] - yrowptr[xdiag[i]];
    const int v = s > 0x3fffffff ? 0x3fffffff : static_cast<int>(s);
    ub[i] = v;
    if (!wave_row(v, xrowptr[i + 1] - xrowptr[i] + (xdiag ? 1 : 0))) {
        if (v > large_cap) atomicMax(too_dense, v);
        big_list[atomicAdd(big_count, 1)] = i;
    }
}

// ------------------------------------------------------------- union add

__global__ __launch_bounds__(256) void k_add_count(const int *__restrict__ srp, const int *__restrict__ sc,
                                                  const int *__restrict__ wrp, const int *__restrict__ wc, int m,
                                                  int *__restrict__ cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int p = srp[i], q = wrp[i];
    const int pe = srp[i + 1], qe = wrp[i + 1];
    int n = 0;
    while (p < pe || q < qe) {
        if (q >= qe || (p < pe && sc[p] < wc[q])) ++p;
        else if (p >= pe || wc[q] < sc[p]) ++q;
        else {
            ++p;
            ++q;
        }
        ++n;
    }
    cnt[i] = n;
}

__global__ __launch_bounds__(256) void k_add_fill(const int *__restrict__ srp, const int *__restrict__ sc,
                                                 const int *__restrict__ wrp, const int *__restrict__ wc, int m,
                                                 const int *__restrict__ orp, int *__restrict__ oc,
                                                 int *__restrict__ srcS, int *__restrict__ srcW) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int p = srp[i], q = wrp[i];
    const int pe = srp[i + 1], qe = wrp[i + 1];
    int o = orp[i];
    while (p < pe || q < qe) {
        if (q >= qe || (p < pe && sc[p] < wc[q])) {
            oc[o] = sc[p];
            srcS[o] = p++;
            srcW[o] = -1;
        } else if (p >= pe || wc[q] < sc[p]) {
            oc[o] = wc[q];
            srcS[o] = -1;
            srcW[o] = q++;
        } else {
            oc[o] = sc[p];
            srcS[o] = p++;
            srcW[o] = q++;
        }
        ++o;
    }
}

// blocks t < *count of O (count on the device)
__global__ __launch_bounds__(256) void k_add_values(const int *__restrict__ count, int bb, const double *__restrict__ S,
                                                   const int *__restrict__ srcS, const double *__restrict__ W,
                                                   const int *__restrict__ srcW, double *__restrict__ O) {
    const int64_t total = static_cast<int64_t>(*count) * bb;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t t = g / bb;
        const int e = static_cast<int>(g - t * bb);
        const int a = srcS[t], b = srcW[t];
        double v;
        if (a >= 0 && b >= 0) v = S[static_cast<int64_t>(a) * bb + e] + W[static_cast<int64_t>(b) * bb + e];
        else if (a >= 0) v = S[static_cast<int64_t>(a) * bb + e];
        else v = W[static_cast<int64_t>(b) * bb + e];
        O[g] = v;
    }
}

// The same with one wave per block (blocks of 64 entries or more).
__global__ __launch_bounds__(256) void k_add_values_wave(const int *__restrict__ count, int bb,
                                                        const double *__restrict__ S, const int *__restrict__ srcS,
                                                        const double *__restrict__ W, const int *__restrict__ srcW,
                                                        double *__restrict__ O) {
    const int lane = threadIdx.x & 63;
    const int64_t nblk = *count;
    const int64_t stride = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    for (int64_t t = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6; t < nblk; t += stride) {
        const int a = srcS[t], b = srcW[t];
        const double *sp = S + static_cast<int64_t>(a < 0 ? 0 : a) * bb;
        const double *wp = W + static_cast<int64_t>(b < 0 ? 0 : b) * bb;
        double *o = O + t * bb;
        for (int e = lane; e < bb; e += 64) {
            double v;
            if (a >= 0 && b >= 0) v = sp[e] + wp[e];
            else if (a >= 0) v = sp[e];
            else v = wp[e];
            o[e] = v;
        }
    }
}

// ------------------------------------------------- one-point Galerkin merge

constexpr int kRowBlocks = 1024;   // longest operator row that the merge takes

// A P's pattern: row i's blocks A_it with pmap[t] >= 0, merged by column pmap[t].
// mode 0: cnt[i] columns and ccnt[i] contributing blocks; mode 1: the sorted
// columns at kcol + krp[i], each one's blocks (ascending) from kptr in klist
// (row i's from crow[i]).  One sort of (column, place in the row) by a group of
// lanes gives all of it.
struct MergeArgs {
    const int *rarp, *racol, *pmap;
    int m;
    int *cnt, *ccnt;
    const int *krp;
    int *kcol;
    const int *crow;
    int *kptr, *klist;
};

constexpr int kMergeBits = 10;

template <int W, int E, int MODE, typename KEY>
__device__ inline void merge_row(const MergeArgs &M, int i, int lane) {
    const int gl = lane & (W - 1);
    const bool active = i < M.m;
    const int r0 = active ? M.rarp[i] : 0, n = active ? M.rarp[i + 1] - r0 : 0;
    int col[E];
#pragma unroll
    for (int e = 0; e < E; ++e) col[e] = gl * E + e < n ? M.racol[r0 + gl * E + e] : -1;
    KEY key[E];
    int c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = col[e] >= 0 ? M.pmap[col[e]] : -1;
        key[e] = t >= 0 ? static_cast<KEY>(t) << kMergeBits | static_cast<KEY>(gl * E + e) : ~static_cast<KEY>(0);
        c += t >= 0 ? 1 : 0;
    }
    group_sort<W, E>(key, gl);
    bool head[E];
    int upto[E];
    const int nk = heads<W, E, kMergeBits>(key, gl, lane, head, upto);
    if (MODE == 0) {
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
        if (active && gl == 0) {
            M.cnt[i] = nk;
            M.ccnt[i] = c;
        }
        return;
    }
    const int k0 = active ? M.krp[i] : 0, R0 = active ? M.crow[i] : 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (key[e] == ~static_cast<KEY>(0)) continue;
        const int at = R0 + gl * E + e;
        M.klist[at] = r0 + static_cast<int>(key[e] & ((1 << kMergeBits) - 1));
        if (head[e]) {
            M.kcol[k0 + upto[e] - 1] = static_cast<int>(key[e] >> kMergeBits);
            M.kptr[k0 + upto[e] - 1] = at;
        }
    }
}

// A wave takes four consecutive rows at a time, all four, two or one at once as
// the longest allows.  (rows past 1,024 blocks are reported and left out)
template <int MODE, typename KEY>
__global__ __launch_bounds__(256) void k_merge_rows(MergeArgs M, int *__restrict__ too_dense) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (MODE == 1 && blockIdx.x == 0 && threadIdx.x == 0) M.kptr[M.krp[M.m]] = M.crow[M.m];   // end of the last list
    for (int i0 = (blockIdx.x * 4 + w) * 4; i0 < M.m; i0 += gridDim.x * 16) {
        const int i = i0 + (lane >> 4);
        const int n = i < M.m ? M.rarp[i + 1] - M.rarp[i] : 0;
        int len[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) len[k] = __builtin_amdgcn_readlane(n, 16 * k);
        if (max(max(len[0], len[1]), max(len[2], len[3])) <= 16) {
            merge_row<16, 1, MODE, KEY>(M, i, lane);
            continue;
        }
#pragma unroll 1
        for (int h = 0; h < 4; h += 2) {
            const int a = h ? len[2] : len[0], b = h ? len[3] : len[1];
            if (max(a, b) <= 32) {
                merge_row<32, 1, MODE, KEY>(M, i0 + h + (lane >> 5), lane);
                continue;
            }
#pragma unroll 1
            for (int k = 0; k < 2; ++k) {
                const int l = k ? b : a, row = i0 + h + k;
                if (l <= 64) merge_row<64, 1, MODE, KEY>(M, row, lane);
                else if (l <= 256) merge_row<64, 4, MODE, KEY>(M, row, lane);
                else if (l <= kRowBlocks) merge_row<64, 16, MODE, KEY>(M, row, lane);
                else if (MODE == 0 && lane == 0) atomicMax(too_dense, l);
            }
        }
    }
}

// The kept blocks' columns, places, sizes and (rmask) row masks.
__global__ __launch_bounds__(256) void k_compact_fill(const int *__restrict__ krp, const int *__restrict__ kcol,
                                                     const uint8_t *__restrict__ keep,
                                                     const double *__restrict__ knorm,
                                                     const uint32_t *__restrict__ kbits, int m,
                                                     const int *__restrict__ orp, int *__restrict__ ocol,
                                                     int *__restrict__ osrc, double *__restrict__ onorm,
                                                     uint32_t *__restrict__ obits) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int o = orp[i];
    for (int t = krp[i]; t < krp[i + 1]; ++t)
        if (keep[t]) {
            ocol[o] = kcol[t];
            osrc[o] = t;
            onorm[o] = knorm[t];
            if (obits) obits[o] = kbits[t];
            ++o;
        }
}

unsigned cap_grid(int64_t g) { return static_cast<unsigned>(g > 65536 * 16 ? 65536 * 16 : (g < 1 ? 1 : g)); }

}  // namespace

namespace {

// Symbolic product C = X Y (X with an implicit identity block at column xdiag[i]
// merged into its row i).  A row's products are numbered flat, ascending inner
// index first; sorting (output column, number) gives the row's columns in order and
// each output block's pair list in ascending inner index (a Y row feeds a block at
// most once).  mode 0: cnt[i] columns; mode 1: columns at ccol + crowptr[i], pairs at
// prow[i] ..., block t's from pairptr[t].
struct SymArgs {
    const int *xrowptr, *xcol, *xdiag, *yrowptr, *ycol;
    int m;
    const int *ub;
    int *cnt;
    const int *crowptr;
    int *ccol;
    const int *prow;
    int *pairptr;
    int2 *pairs;
};

constexpr int kPairBits = 10;   // (up to 1,024 products a wave)

// One row per group of W lanes, E products per lane: one inner slot per lane, then
// product p's slot by binary search over the lanes' offsets.
template <int W, int E, int MODE, typename KEY>
__device__ inline void product_row(const SymArgs &S, int i, int lane) {
    const int gl = lane & (W - 1);
    const bool active = i < S.m;
    int q0 = 0, nx = 0, dcol = 0;
    if (active) {
        q0 = S.xrowptr[i];
        nx = S.xrowptr[i + 1] - q0;
        if (S.xdiag) dcol = S.xdiag[i];
    }
    int K = gl < nx ? S.xcol[q0 + gl] : INT_MAX, q = q0 + gl;
    bool slot = gl < nx;
    if (S.xdiag) {   // the identity takes its place, the slots from there on move up by one
        const uint64_t group = W == 64 ? ~0ull : (((1ull << (W & 63)) - 1) << (lane & ~(W - 1)));
        const int dslot = __popcll(__ballot(slot && K < dcol) & group);
        const int Kp = __shfl_up(K, 1, W);
        if (gl > dslot) {
            K = Kp;
            --q;
        } else if (gl == dslot) {
            K = dcol;
            q = -1;
        }
        slot = active && gl <= nx;
    }
    int ybeg = 0, len = 0;
    if (slot) {
        ybeg = S.yrowptr[K];
        len = S.yrowptr[K + 1] - ybeg;
    }
    int excl = len;
#pragma unroll
    for (int d = 1; d < W; d <<= 1) {
        const int y = __shfl_up(excl, d, W);
        excl += gl >= d ? y : 0;
    }
    const int total = __shfl(excl, W - 1, W);
    excl -= len;
    auto slot_of = [&](int p) {   // the last slot that starts at or before p (empty slots lie before their successor)
        int j = 0;
#pragma unroll
        for (int step = W / 2; step > 0; step >>= 1) j += __shfl(excl, j + step, W) <= p ? step : 0;
        return j;
    };
    KEY key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = gl * E + e, j = slot_of(p);
        const int u = __shfl(ybeg, j, W) + p - __shfl(excl, j, W);
        key[e] = p < total ? static_cast<KEY>(S.ycol[u]) << kPairBits | static_cast<KEY>(p) : ~static_cast<KEY>(0);
    }
    group_sort<W, E>(key, gl);
    bool head[E];
    int upto[E];
    const int n = heads<W, E, kPairBits>(key, gl, lane, head, upto);
    if (MODE == 0) {
        if (active && gl == 0) S.cnt[i] = n;
        return;
    }
    const int c0 = active ? S.crowptr[i] : 0, P0 = active ? S.prow[i] : 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = static_cast<int>(key[e] & ((1 << kPairBits) - 1)), j = slot_of(p);
        const int fq = __shfl(q, j, W), fu = __shfl(ybeg, j, W) + p - __shfl(excl, j, W);
        if (key[e] == ~static_cast<KEY>(0)) continue;
        const int at = P0 + gl * E + e;
        S.pairs[at] = make_int2(fq, fu);
        if (head[e]) {
            S.ccol[c0 + upto[e] - 1] = static_cast<int>(key[e] >> kPairBits);
            S.pairptr[c0 + upto[e] - 1] = at;
        }
    }
}

// A wave takes four consecutive rows at a time: all four at once in 16 lanes each,
// two in 32, or one after the other, as the longest needs (products and inner
// slots); rows of more than kWaveProducts products or kWave slots are left to
// k_product_large.  Bound by the row's chain of loads (row range, inner columns,
// their rows, their columns) and the sort's about 60 to 500 lane moves.  One row per
// wave with LDS hash tables, per-block counts and 64-step ranks took 40 ms of the
// setup of 64 Q2 transport operators (2.0 M rows; products, merges and their lists
// together), this takes 8.
template <int MODE, typename KEY>
__global__ __launch_bounds__(256) void k_product_rows(SymArgs S) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (MODE == 1 && blockIdx.x == 0 && threadIdx.x == 0) S.pairptr[S.crowptr[S.m]] = S.prow[S.m];   // last list's end
    for (int i0 = (blockIdx.x * 4 + w) * 4; i0 < S.m; i0 += gridDim.x * 16) {
        const int i = i0 + (lane >> 4);
        int n = 0;
        if (i < S.m) {
            const int slots = S.xrowptr[i + 1] - S.xrowptr[i] + (S.xdiag ? 1 : 0), products = S.ub[i];
            n = wave_row(products, slots) ? max(products, slots) : INT_MAX;
        }
        int len[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) len[k] = __builtin_amdgcn_readlane(n, 16 * k);
        if (max(max(len[0], len[1]), max(len[2], len[3])) <= 16) {
            product_row<16, 1, MODE, KEY>(S, i, lane);
            continue;
        }
#pragma unroll 1
        for (int h = 0; h < 4; h += 2) {
            const int a = h ? len[2] : len[0], b = h ? len[3] : len[1];
            if (max(a, b) <= 32) {
                product_row<32, 1, MODE, KEY>(S, i0 + h + (lane >> 5), lane);
                continue;
            }
#pragma unroll 1
            for (int k = 0; k < 2; ++k) {
                const int l = k ? b : a, row = i0 + h + k;
                if (l <= 64) product_row<64, 1, MODE, KEY>(S, row, lane);
                else if (l <= 128) product_row<64, 2, MODE, KEY>(S, row, lane);
                else if (l <= kWaveProducts) product_row<64, 4, MODE, KEY>(S, row, lane);
            }
        }
    }
}

// The rows in big_list: up to 1,024 products and 64 slots a wave each, up to
// kLargeProducts products the workgroup together, keys and pairs in LDS (rows past
// the limit are reported on the host).
constexpr int kLargeProducts = 4096;
constexpr int kLargeBits = 12;
constexpr int kLargeGrid = 512;

template <int MODE, typename KEY>
__global__ __launch_bounds__(256) void k_product_large(SymArgs S, const int *__restrict__ big_list,
                                                      const int *__restrict__ big_count) {
    extern __shared__ uint64_t lkey[];                             // [kLargeProducts]
    int2 *pay = reinterpret_cast<int2 *>(lkey + kLargeProducts);   // [kLargeProducts], mode 1
    __shared__ int sq[256], sy[256], se[256], wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto block_excl = [&](int v, int &total) {   // exclusive scan over the workgroup
        const int x = wave_incl_scan(v);
        __syncthreads();
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        int before = 0;
        for (int k = 0; k < w; ++k) before += wsum[k];
        total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        return before + x - v;
    };
    const int nbig = *big_count;
    auto kind = [&](int b) {   // of list entry b: 0 a wave's 512 products, 1 its 1,024, 2 the workgroup's, 3 none
        if (b >= nbig) return 3;
        const int i = big_list[b], products = S.ub[i];
        const int slots = S.xrowptr[i + 1] - S.xrowptr[i] + (S.xdiag ? 1 : 0);
        return products > kLargeProducts ? 3 : (products > 1024 || slots > kWave ? 2 : (products > 512 ? 1 : 0));
    };
    for (int b0 = blockIdx.x * 4; b0 < nbig; b0 += gridDim.x * 4) {
        const int mine = __builtin_amdgcn_readfirstlane(kind(b0 + w));
        if (mine == 0) product_row<64, 8, MODE, KEY>(S, big_list[b0 + w], lane);
        else if (mine == 1) product_row<64, 16, MODE, KEY>(S, big_list[b0 + w], lane);
        for (int b = b0; b < b0 + 4; ++b) {
            if (kind(b) != 2) continue;   // (the same in every thread)
            const int i = big_list[b];
            const int q0 = S.xrowptr[i], nx = S.xrowptr[i + 1] - q0;
            int dslot = INT_MAX, dcol = 0;
            if (S.xdiag) {
                dcol = S.xdiag[i];
                int lo = 0, hi = nx;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (S.xcol[q0 + mid] < dcol) lo = mid + 1;
                    else hi = mid;
                }
                dslot = lo;
            }
            const int nk = nx + (S.xdiag ? 1 : 0);
            int flat = 0;   // products of the slots before this chunk
            for (int base = 0; base < nk; base += 256) {
                const int qq = base + tid;
                int q = -1, ybeg = 0, len = 0;
                if (qq < nk) {
                    if (qq != dslot) q = q0 + qq - (qq > dslot ? 1 : 0);
                    const int K = q < 0 ? dcol : S.xcol[q];
                    ybeg = S.yrowptr[K];
                    len = S.yrowptr[K + 1] - ybeg;
                }
                int total;
                const int excl = block_excl(len, total);
                sq[tid] = q;
                sy[tid] = ybeg;
                se[tid] = excl;
                __syncthreads();
                for (int p = tid; p < total; p += 256) {
                    int j = 0;
    #pragma unroll
                    for (int step = 128; step > 0; step >>= 1) j += se[j + step] <= p ? step : 0;
                    const int u = sy[j] + p - se[j];
                    lkey[flat + p] = static_cast<uint64_t>(S.ycol[u]) << kLargeBits | static_cast<uint64_t>(flat + p);
                    if (MODE == 1) pay[flat + p] = make_int2(sq[j], u);
                }
                flat += total;
                __syncthreads();
            }
            int N = 256;
            while (N < flat) N <<= 1;
            for (int t = flat + tid; t < N; t += 256) lkey[t] = ~0ull;
            __syncthreads();
            for (int k = 2; k <= N; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int t = tid; t < N / 2; t += 256) {
                        const int x = 2 * t - (t & (j - 1)), y = x + j;
                        const uint64_t a = lkey[x], c = lkey[y];
                        if (((x & k) == 0) == (c < a)) {
                            lkey[x] = c;
                            lkey[y] = a;
                        }
                    }
                    __syncthreads();
                }
            const int per = N / 256, t0 = tid * per;
            int n = 0;
            for (int t = t0; t < t0 + per && t < flat; ++t)
                n += (t == 0 || (lkey[t] >> kLargeBits) != (lkey[t - 1] >> kLargeBits)) ? 1 : 0;
            int total;
            int at = block_excl(n, total);
            if (MODE == 0) {
                if (tid == 0) S.cnt[i] = total;
            } else {
                const int c0 = S.crowptr[i], P0 = S.prow[i];
                for (int t = t0; t < t0 + per && t < flat; ++t)
                    if (t == 0 || (lkey[t] >> kLargeBits) != (lkey[t - 1] >> kLargeBits)) {
                        S.ccol[c0 + at] = static_cast<int>(lkey[t] >> kLargeBits);
                        S.pairptr[c0 + at] = P0 + t;
                        ++at;
                    }
                for (int t = tid; t < flat; t += 256) S.pairs[P0 + t] = pay[lkey[t] & (kLargeProducts - 1)];
            }
            __syncthreads();
        }
    }
}

// C[t] entry (a,b) = fma chain over the pairs of block t (ascending inner index)
// and c ascending, from +0; identity pairs add Y's entry plainly.  One thread
// per (output block, block row a) keeps the row's bs accumulators in registers
// and reads contiguous rows of X and Y.
template <int BS>
__global__ __launch_bounds__(256) void k_spgemm_pairs(int64_t nnz, int bs_rt, const int *__restrict__ pairptr,
                                                     const int2 *__restrict__ pairs, const double *__restrict__ X,
                                                     const double *__restrict__ Y, double *__restrict__ C) {
    constexpr int NB = BS > 0 ? BS : kMaxBs;
    const int bs = BS > 0 ? BS : bs_rt;
    const int bb = bs * bs;
    const int64_t total = nnz * bs;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t t = g / bs;
        const int a = static_cast<int>(g - t * bs);
        double acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = 0.0;
        for (int k = pairptr[t]; k < pairptr[t + 1]; ++k) {
            const int2 pr = pairs[k];
            const double *y = Y + static_cast<int64_t>(pr.y) * bb;
            if (pr.x < 0) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (BS > 0 || b < bs) acc[b] = acc[b] + y[a * bs + b];
            } else {
                const double *x = X + static_cast<int64_t>(pr.x) * bb + a * bs;
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    if (BS == 0 && c >= bs) break;
                    const double xc = x[c];
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (BS > 0 || b < bs) acc[b] = __builtin_fma(xc, y[c * bs + b], acc[b]);
                }
            }
        }
        double *out = C + t * bb + a * bs;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (BS > 0 || b < bs) out[b] = acc[b];
    }
}

// The same sums on the matrix cores (bs 9, 16, 25; mfma_tile.h).  One wave
// holds one output block in 16x16 FP64 accumulator tiles; each pair adds
// ceil(bs/4) 16x16x4 steps per tile over c = 4q .. 4q+3, zero beyond bs.  A
// 16x16x4 FP64 step updates each entry as the fma chain over its four c in
// ascending order, so the sums are the per-thread chains above (padding adds
// exact zeros); identity pairs add Y's entries plainly, in their place in the
// pair order.  The block is written as 0 + the accumulator.
//
// A pair's two blocks are read with consecutive lanes on consecutive words
// (ceil(bs^2/64) loads per lane and block), written to the wave's LDS slot,
// and the fragments taken from there.  The sums are short (a few pairs per
// block), so a wave that started each block from its index would wait on
// three dependent loads per block (the pair range, the pair, the blocks):
// instead each workgroup owns a contiguous range of output blocks, its four
// waves take every fourth block of it, and each wave keeps ahead of itself --
// the pair range two blocks on, the pair indices of the next block, and the
// next pair's blocks (of this block or the next) in registers while the
// current pair's steps run.  Also writes each block's max-abs size and the bit
// mask of its nonzero rows (knorm == nullptr: neither).
// lane src's pair (src the same in every lane: a read of one lane's registers)
__device__ inline int2 shfl_pair(int2 v, int src) {
    return int2{__builtin_amdgcn_readlane(v.x, src), __builtin_amdgcn_readlane(v.y, src)};
}

template <int BS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_pair_sums(
    int64_t nnz, int64_t per_wg, const int *__restrict__ pairptr, const int2 *__restrict__ pairs,
    const double *__restrict__ X, const double *__restrict__ Y, const double *__restrict__ Y2,
    double *__restrict__ K, double *__restrict__ knorm, uint32_t *__restrict__ kmask) {
    constexpr int BB = BS * BS;
    constexpr int NL = (BB + 63) / 64;   // loads per lane and block
    constexpr int NT = MfmaShape<BS>::NT, KQ = MfmaShape<BS>::KQ;
    __shared__ double slot[4][2 * BB];
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kk = lane >> 4;
    const int64_t lo = static_cast<int64_t>(blockIdx.x) * per_wg;
    const int64_t hi = lo + per_wg < nnz ? lo + per_wg : nnz;
    int64_t t = lo + w;
    if (t >= hi) return;   // whole waves; no workgroup barrier below
    double *xs = slot[w], *ys = slot[w] + BB;
    double xv[NL], yv[NL];
    auto load = [&](const int2 q) {
        // (a pair's y < 0 names block -y-1 of the second store)
        const double *y = q.y >= 0 ? Y + static_cast<int64_t>(q.y) * BB : Y2 + static_cast<int64_t>(-q.y - 1) * BB;
        // (an identity pair's x is never read: it loads its y block again, so that every
        // load is unconditional -- as are the words past the block, read from its last)
        const double *x = q.x >= 0 ? X + static_cast<int64_t>(q.x) * BB : y;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int e = lane + 64 * i < BB ? lane + 64 * i : BB - 1;
            yv[i] = y[e];
            xv[i] = x[e];
        }
    };
    auto chunk = [&](int from, int end) { return from + lane < end ? pairs[from + lane] : int2{0, 0}; };
    // this block: pair range and the first 64 pair indices
    int pb = pairptr[t], pe = pairptr[t + 1];
    int2 cp = chunk(pb, pe);
    // the next block: range and pair indices; the one after: range
    int64_t tn = t + 4;
    int npb = 0, npe = 0;
    if (tn < hi) {
        npb = pairptr[tn];
        npe = pairptr[tn + 1];
    }
    int2 ncp = tn < hi ? chunk(npb, npe) : int2{0, 0};
    int64_t tnn = tn + 4;
    int nnpb = 0, nnpe = 0;
    if (tnn < hi) {
        nnpb = pairptr[tnn];
        nnpe = pairptr[tnn + 1];
    }
    bool pend = false;   // xv / yv hold (or are loading) the next pair to run
    for (;;) {
        const int cnt = pe - pb;
        MfmaAcc<BS> acc;
        acc.zero();
        for (int j = 0; j < cnt; ++j) {
            if (j > 0 && (j & 63) == 0) cp = chunk(pb + j, pe);   // (more than 64 pairs: the next 64)
            const int2 pr = shfl_pair(cp, j & 63);
            if (!pend) load(pr);
            // this pair's blocks to LDS (the previous pair's fragment reads were issued before)
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int e = lane + 64 * i;
                if (e < BB) {
                    xs[e] = xv[i];
                    ys[e] = yv[i];
                }
            }
            pend = false;
            // the following pair's blocks load while this pair's steps run
            if (j + 1 < cnt) {
                if (((j + 1) & 63) != 0) {
                    load(shfl_pair(cp, (j + 1) & 63));
                    pend = true;
                }
            } else if (tn < hi && npe > npb) {
                load(shfl_pair(ncp, 0));
                pend = true;
            }
            if (pr.x < 0) {   // identity pair: Y's entries added plainly
#pragma unroll
                for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                    for (int tj = 0; tj < NT; ++tj)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * ti + kk + 4 * r, jj = 16 * tj + row;
                            if (i < BS && jj < BS) acc.t[ti][tj][r] = acc.t[ti][tj][r] + ys[i * BS + jj];
                        }
            } else {
#pragma unroll
                for (int q = 0; q < KQ; ++q) {
                    const int c = 4 * q + kk;
                    double a[NT], b[NT];
#pragma unroll
                    for (int u = 0; u < NT; ++u) {
                        const int i = 16 * u + row;
                        a[u] = (i < BS && c < BS) ? xs[i * BS + c] : 0.0;
                        b[u] = (i < BS && c < BS) ? ys[c * BS + i] : 0.0;
                    }
#pragma unroll
                    for (int ti = 0; ti < NT; ++ti)
#pragma unroll
                        for (int tj = 0; tj < NT; ++tj)
                            acc.t[ti][tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ti], b[tj], acc.t[ti][tj], 0, 0, 0);
                    // (one step's fragments at a time: the LDS reads are not hoisted past its MFMAs)
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        double *out = K + t * BB;
        double m = 0.0;
        uint32_t bits = 0u;
        mfma_for_entries<BS>(acc, row, kk, [&](int i, int jj, double v) {
            const double o = 0.0 + v;
            out[i * BS + jj] = o;
            m = fmax(m, fabs(o));
            if (o != 0.0) bits |= 1u << i;
        });
        if (knorm) {   // (a plain sparse product takes no sizes)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                m = fmax(m, __shfl_xor(m, o, 64));
                bits |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(bits), o, 64));
            }
            if (lane == 0) {
                knorm[t] = m;
                kmask[t] = bits;
            }
        }
        // on to the next block
        t = tn;
        if (t >= hi) break;
        pb = npb;
        pe = npe;
        cp = ncp;
        tn = tnn;
        npb = nnpb;
        npe = nnpe;
        ncp = tn < hi ? chunk(npb, npe) : int2{0, 0};
        tnn = tn + 4;
        if (tnn < hi) {
            nnpb = pairptr[tnn];
            nnpe = pairptr[tnn + 1];
        }
    }
}

// Sums of pair lists for nnz output blocks on the matrix cores (bs 9, 16, 25).
void launch_pair_sums(int bs, int64_t nnz, const int *pairptr, const int2 *pairs, const double *X, const double *Y,
                      const double *Y2, double *K, double *knorm, uint32_t *kmask, hipStream_t s) {
    if (nnz <= 0) return;
    // up to 24,576 workgroups of contiguous ranges: each wave still runs through several
    // blocks with the next ones in flight, and the chains are short enough that the tail
    // balances (at 25 x 25 blocks 12k-36k workgroups all did best, 3,072 1.4% worse)
    const int64_t nwg = std::min<int64_t>((nnz + 3) / 4, 24576);
    const int64_t per_wg = (nnz + nwg - 1) / nwg;
    const int64_t grid = (nnz + per_wg - 1) / per_wg;
    if (bs == 9)
        k_pair_sums<9><<<static_cast<unsigned>(grid), 256, 0, s>>>(nnz, per_wg, pairptr, pairs, X, Y, Y2, K, knorm,
                                                                   kmask);
    else if (bs == 16)
        k_pair_sums<16><<<static_cast<unsigned>(grid), 256, 0, s>>>(nnz, per_wg, pairptr, pairs, X, Y, Y2, K, knorm,
                                                                    kmask);
    else if (bs == 25)
        k_pair_sums<25><<<static_cast<unsigned>(grid), 256, 0, s>>>(nnz, per_wg, pairptr, pairs, X, Y, Y2, K, knorm,
                                                                    kmask);
    else
        fail(NAIR_EDEVICE, "launch_pair_sums: matrix-core block sizes only");
    NAIR_HIP(hipGetLastError());
}

// --------------------------------------------------- Galerkin merged values

__global__ __launch_bounds__(256) void k_rap_values(int64_t nnz, int bb, const int *__restrict__ kptr,
                                                   const int *__restrict__ klist, const double *__restrict__ RA,
                                                   double *__restrict__ K) {
    const int64_t total = nnz * bb;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t t = g / bb;
        const int e = static_cast<int>(g - t * bb);
        double s = 0.0;
        for (int k = kptr[t]; k < kptr[t + 1]; ++k) s = s + RA[static_cast<int64_t>(klist[k]) * bb + e];
        K[g] = s;
    }
}

// The same with one wave per block (blocks of 64 entries or more).
__global__ __launch_bounds__(256) void k_rap_values_wave(int64_t nnz, int bb, const int *__restrict__ kptr,
                                                        const int *__restrict__ klist, const double *__restrict__ RA,
                                                        double *__restrict__ K) {
    const int lane = threadIdx.x & 63;
    const int64_t stride = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    for (int64_t t = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6; t < nnz; t += stride) {
        const int k0 = kptr[t], k1 = kptr[t + 1];
        for (int e = lane; e < bb; e += 64) {
            double v = 0.0;
            for (int k = k0; k < k1; ++k) v = v + RA[static_cast<int64_t>(klist[k]) * bb + e];
            K[t * bb + e] = v;
        }
    }
}

// A P blocks with one contributor are that A block itself; the others (flag 1)
// are summed into a second store.  ymap[t]: the A block, or -(merged index)-1.
__global__ __launch_bounds__(256) void k_ap_flags(int64_t nnz, const int *__restrict__ kptr, int *__restrict__ flag) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t < nnz) flag[t] = (kptr[t + 1] - kptr[t] > 1) ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_ap_map(int64_t nnz, const int *__restrict__ kptr,
                                               const int *__restrict__ klist, const int *__restrict__ midx,
                                               int *__restrict__ ymap, int *__restrict__ mblk) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= nnz) return;
    if (kptr[t + 1] - kptr[t] > 1) {
        ymap[t] = -midx[t] - 1;
        mblk[midx[t]] = static_cast<int>(t);
    } else {
        ymap[t] = klist[kptr[t]];
    }
}

// merged block q = sum of A P block mblk[q]'s contributors, one wave per block
// (NCH: 64-word chunks that cover a block, at most 16 for bs <= 32)
template <int NCH>
__global__ __launch_bounds__(256) void k_ap_merged(int nm, int bb, const int *__restrict__ mblk,
                                                  const int *__restrict__ kptr, const int *__restrict__ klist,
                                                  const double *__restrict__ A, double *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t stride = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    for (int64_t q = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6; q < nm; q += stride) {
        const int t = mblk[q];
        const int k0 = kptr[t], k1 = kptr[t + 1];
        // contributors outermost, two at a time: their entries load together (one wait
        // per two contributors, not per entry); every entry still sums its contributors
        // in order.  (Words past a block repeat its last, unused.)
        constexpr int kChunks = NCH;
        double v[kChunks];
#pragma unroll
        for (int i = 0; i < kChunks; ++i) v[i] = 0.0;
        int k = k0;
        for (; k + 1 < k1; k += 2) {
            const double *a0 = A + static_cast<int64_t>(klist[k]) * bb;
            const double *a1 = A + static_cast<int64_t>(klist[k + 1]) * bb;
            double u0[kChunks], u1[kChunks];
#pragma unroll
            for (int i = 0; i < kChunks; ++i) {
                const int e = lane + 64 * i < bb ? lane + 64 * i : bb - 1;
                u0[i] = a0[e];
                u1[i] = a1[e];
            }
#pragma unroll
            for (int i = 0; i < kChunks; ++i) v[i] = (v[i] + u0[i]) + u1[i];
        }
        if (k < k1) {
            const double *a = A + static_cast<int64_t>(klist[k]) * bb;
#pragma unroll
            for (int i = 0; i < kChunks; ++i) {
                const int e = lane + 64 * i;
                if (e < bb) v[i] = v[i] + a[e];
            }
        }
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const int e = lane + 64 * i;
            if (e < bb) out[q * bb + e] = v[i];
        }
    }
}

// pairs[k].x = xmap[pairs[k].x] where x >= 0 (identity pairs keep x < 0)
__global__ __launch_bounds__(256) void k_remap_x(int64_t n, const int *__restrict__ xmap, int2 *__restrict__ pairs) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int x = pairs[k].x;
    if (x >= 0) pairs[k].x = xmap[x];
}

__global__ __launch_bounds__(256) void k_remap_y(int64_t n, const int *__restrict__ ymap, int2 *__restrict__ pairs) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p < n) pairs[p].y = ymap[pairs[p].y];
}

// Drop filter: keep the diagonal and blocks with size > drop * size(diagonal).
// One wave per row, its lanes over the row's blocks.
__global__ __launch_bounds__(256) void k_drop_mark(const int *__restrict__ krp, const int *__restrict__ kcol,
                                                  const double *__restrict__ knorm, int m, double drop,
                                                  uint8_t *__restrict__ keep, int *__restrict__ kept,
                                                  int *__restrict__ margin) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    if (i >= m) return;   // whole waves
    const int lo = krp[i], hi = krp[i + 1];
    double dn = 0.0;   // the diagonal block's size (0 if the row has none)
    for (int base = lo; base < hi; base += 64) {
        const int t = base + lane;
        const bool isd = t < hi && kcol[t] == i;
        const double v = isd ? knorm[t] : 0.0;
        const unsigned long long b = __ballot(isd);
        if (b != 0ull) {
            dn = __shfl(v, static_cast<int>(__builtin_ctzll(b)), 64);
            break;
        }
    }
    const double thr = drop * dn;
    int c = 0, nties = 0;
    for (int t = lo + lane; t < hi; t += 64) {
        const bool diag = kcol[t] == i;
        const double kn = knorm[t];
        const bool k = diag || (kn > thr);
        keep[t] = k ? 1 : 0;
        c += k ? 1 : 0;
        // audit: the two sides of the drop test within 1e-12 relative
        if (!diag && fabs(kn - thr) <= 1e-12 * fmax(fabs(kn), fabs(thr))) ++nties;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o, 64);
        nties += __shfl_xor(nties, o, 64);
    }
    if (lane == 0) {
        kept[i] = c;
        if (nties) atomicAdd(margin + 3, nties);
    }
}


}  // namespace

#define NAIR_BS_DISPATCH(bs, KERNEL, ...)            \
    switch (bs) {                                    \
        case 2: KERNEL<2> __VA_ARGS__; break;        \
        case 3: KERNEL<3> __VA_ARGS__; break;        \
        case 4: KERNEL<4> __VA_ARGS__; break;        \
        case 6: KERNEL<6> __VA_ARGS__; break;        \
        case 9: KERNEL<9> __VA_ARGS__; break;        \
        case 10: KERNEL<10> __VA_ARGS__; break;      \
        case 16: KERNEL<16> __VA_ARGS__; break;      \
        case 25: KERNEL<25> __VA_ARGS__; break;      \
        default: KERNEL<0> __VA_ARGS__; break;       \
    }

namespace {

// The pair lists of a product's blocks (pairs[pairptr[t]] ... for block t).
struct Pairs {
    DBuf<int> pairptr;
    DBuf<int2> pairs;
    int64_t n = 0;   // pairs
};

// C's pattern (rowptr, colidx, nnzb) and the pair lists of its blocks; C.vals
// is left unallocated.
void spgemm_structure(const DevBSR &X, const int *xdiag, const DevBSR &Y, DevBSR &C, Pairs &P, int *flags,
                      hipStream_t s) {
    const int m = X.nb;
    const int bs = X.bs;
    C.nb = m;
    C.ncols = Y.ncols;
    C.bs = bs;
    C.rowptr.alloc(static_cast<size_t>(m) + 1);
    if (m == 0) {
        NAIR_HIP(hipMemsetAsync(C.rowptr.get(), 0, sizeof(int), s));
        C.nnzb = 0;
        C.colidx.alloc(0);
        return;
    }
    // flags: big-row count, too-dense row, then the scans' totals (nnz, pairs), read in one copy
    DBuf<int> ub(m), cnt(m), big_list(m), prow(static_cast<size_t>(m) + 1);
    int *big_count = flags;
    k_row_upper_bound<<<grid_for(m, 256), 256, 0, s>>>(X.rowptr.get(), X.colidx.get(), xdiag, Y.rowptr.get(), m,
                                                      ub.get(), big_list.get(), big_count, kLargeProducts,
                                                      flags + 1);
    SymArgs S{X.rowptr.get(), X.colidx.get(), xdiag, Y.rowptr.get(), Y.colidx.get(), m, ub.get(), cnt.get()};
    const unsigned gs = cap_grid((m + 15) / 16);
    const bool narrow = Y.ncols < (1 << (32 - kPairBits));   // (column, product) fit 32 bits, no key all ones
    if (narrow) k_product_rows<0, uint32_t><<<gs, 256, 0, s>>>(S);
    else k_product_rows<0, uint64_t><<<gs, 256, 0, s>>>(S);
    {
        TimerScope ts(TK_SPGEMM_SYM, g_timer_level, s);
        constexpr size_t lds = sizeof(uint64_t) * kLargeProducts;
        if (narrow) k_product_large<0, uint32_t><<<kLargeGrid, 256, lds, s>>>(S, big_list.get(), big_count);
        else k_product_large<0, uint64_t><<<kLargeGrid, 256, lds, s>>>(S, big_list.get(), big_count);
    }
    NAIR_HIP(hipGetLastError());
    scan_exclusive2(cnt.get(), C.rowptr.get(), m, flags + 2, ub.get(), prow.get(), m, flags + 3, s);
    int hflags[4] = {0, 0, 0, 0};
    read_ints(flags, hflags, 4, s);
    const int nnz = hflags[2], npairs = hflags[3];
    if (hflags[1] > 0)
        fail(NAIR_ENOMEM, "sparse product row has " + std::to_string(hflags[1]) + " candidate blocks (limit " +
                              std::to_string(kLargeProducts) + ")");
    C.nnzb = nnz;
    C.colidx.alloc(nnz);
    if (nnz == 0) return;
    P.pairptr.alloc(static_cast<size_t>(nnz) + 1);
    P.pairs.alloc(npairs);
    P.n = npairs;
    S.crowptr = C.rowptr.get();
    S.ccol = C.colidx.get();
    S.prow = prow.get();
    S.pairptr = P.pairptr.get();
    S.pairs = P.pairs.get();
    if (narrow) k_product_rows<1, uint32_t><<<gs, 256, 0, s>>>(S);
    else k_product_rows<1, uint64_t><<<gs, 256, 0, s>>>(S);
    if (hflags[0] > 0) {
        constexpr size_t lds = (sizeof(uint64_t) + sizeof(int2)) * kLargeProducts;
        auto kern = narrow ? k_product_large<1, uint32_t> : k_product_large<1, uint64_t>;
        if (!allow_lds(reinterpret_cast<const void *>(kern), lds))
            fail(NAIR_EDEVICE, "the device refuses the sparse product's " + std::to_string(lds) + " bytes of LDS");
        kern<<<kLargeGrid, 256, lds, s>>>(S, big_list.get(), big_count);
    }
    NAIR_HIP(hipGetLastError());
}

// C's values from its pair lists (C.vals allocated by the caller).
void spgemm_values(const double *xvals, const DevBSR &Y, const Pairs &P, DevBSR &C, hipStream_t s) {
    const int64_t nnz = C.nnzb;
    const int bs = C.bs;
    if (nnz == 0) return;
    const int64_t total = nnz * bs;
    const unsigned grid = cap_grid((total + 255) / 256);
    TimerScope ts(TK_SPGEMM_NUM, g_timer_level, s);
    if (use_matrix_cores(bs)) {
        launch_pair_sums(bs, nnz, P.pairptr.get(), P.pairs.get(), xvals, Y.vals.get(), nullptr, C.vals.get(), nullptr,
                         nullptr, s);
    } else {
        NAIR_BS_DISPATCH(bs, k_spgemm_pairs, <<<grid, 256, 0, s>>>(nnz, bs, P.pairptr.get(), P.pairs.get(), xvals,
                                                                   Y.vals.get(), C.vals.get()));
    }
    NAIR_HIP(hipGetLastError());
}

}  // namespace

void spgemm(const DevBSR &X, const int *xdiag, const DevBSR &Y, DevBSR &C, int *zeros, hipStream_t s,
            const double *xvals, const int *xmap) {
    Pairs P;
    spgemm_structure(X, xdiag, Y, C, P, zeros, s);
    if (xmap && P.n > 0) {   // X's block x is block xmap[x] of xvals
        k_remap_x<<<grid_for(P.n, 256), 256, 0, s>>>(P.n, xmap, P.pairs.get());
        NAIR_HIP(hipGetLastError());
    }
    C.vals.alloc(static_cast<size_t>(C.nnzb) * C.bs * C.bs);
    spgemm_values(xmap ? xvals : X.vals.get(), Y, P, C, s);
}

void bsr_add(const DevBSR &S, const DevBSR &W, DevBSR &O, hipStream_t s, DBuf<int> *srcS_out, DBuf<int> *srcW_out) {
    const int m = S.nb;
    const int bs = S.bs;
    O.nb = m;
    O.ncols = S.ncols;
    O.bs = bs;
    O.rowptr.alloc(static_cast<size_t>(m) + 1);
    DBuf<int> cnt(m);
    if (m > 0)
        k_add_count<<<grid_for(m, 256), 256, 0, s>>>(S.rowptr.get(), S.colidx.get(), W.rowptr.get(), W.colidx.get(),
                                                     m, cnt.get());
    scan_exclusive(cnt.get(), O.rowptr.get(), m, s);
    // the union has at most the two counts together; the exact count stays on the device
    const int64_t cap = S.bound() + W.bound();
    O.nnzb = -1;
    O.cap = cap;
    O.colidx.alloc(static_cast<size_t>(cap));
    const bool pattern_only = srcS_out && srcW_out;
    if (!pattern_only) O.vals.alloc(static_cast<size_t>(cap) * bs * bs);
    if (cap == 0 || m == 0) return;
    DBuf<int> srcS(static_cast<size_t>(cap)), srcW(static_cast<size_t>(cap));
    k_add_fill<<<grid_for(m, 256), 256, 0, s>>>(S.rowptr.get(), S.colidx.get(), W.rowptr.get(), W.colidx.get(), m,
                                                O.rowptr.get(), O.colidx.get(), srcS.get(), srcW.get());
    if (pattern_only) {
        NAIR_HIP(hipGetLastError());
        *srcS_out = std::move(srcS);
        *srcW_out = std::move(srcW);
        return;
    }
    const int64_t total = cap * bs * bs;
    if (bs * bs >= 64)
        k_add_values_wave<<<cap_grid((cap + 3) / 4), 256, 0, s>>>(O.rowptr.get() + m, bs * bs, S.vals.get(),
                                                                   srcS.get(), W.vals.get(), srcW.get(), O.vals.get());
    else
        k_add_values<<<cap_grid((total + 255) / 256), 256, 0, s>>>(O.rowptr.get() + m, bs * bs, S.vals.get(),
                                                                  srcS.get(), W.vals.get(), srcW.get(), O.vals.get());
    NAIR_HIP(hipGetLastError());
}

namespace {

// AP = A P for one-point P: A's columns merged through pmap, each AP block the
// sum of its A blocks in ascending column (from +0).  Z's block count comes
// back with the same read when it is still on the device.  With `ymap`, only
// the blocks with several contributors are summed (into `merged`); ymap[t]
// names block t's values: A's block, or -(merged index)-1 (a lone block is
// its A block, up to the sign of a zero entry).
void merge_columns(const DevBSR &A, const int *pmap, int nc, DevBSR &Z, DevBSR &AP, int *flags, hipStream_t s,
                   DBuf<int> *ymap = nullptr, DBuf<double> *merged = nullptr) {
    const int m = A.nb, bs = A.bs, bb = bs * bs;
    AP.nb = m;
    AP.ncols = nc;
    AP.bs = bs;
    DBuf<int> cnt(m), ccnt(m), crow(static_cast<size_t>(m) + 1);
    AP.rowptr.alloc(static_cast<size_t>(m) + 1);
    const unsigned gs = cap_grid((m + 15) / 16);
    MergeArgs M{A.rowptr.get(), A.colidx.get(), pmap, m, cnt.get(), ccnt.get()};
    const bool narrow = nc < (1 << (32 - kMergeBits));   // (column, place) fit 32 bits, no key all ones
    if (narrow) k_merge_rows<0, uint32_t><<<gs, 256, 0, s>>>(M, flags);
    else k_merge_rows<0, uint64_t><<<gs, 256, 0, s>>>(M, flags);
    NAIR_HIP(hipGetLastError());
    scan_exclusive2(cnt.get(), AP.rowptr.get(), m, flags + 1, ccnt.get(), crow.get(), m, flags + 2, s);
    int hflags[3] = {0, 0, 0};
    int zcount = 0;
    const bool zdev = Z.nnzb < 0;
    read_device({{flags, hflags, sizeof(int) * 3},
                 {zdev ? Z.rowptr.get() + Z.nb : nullptr, &zcount, zdev ? sizeof(int) : 0}},
                s);
    if (zdev) Z.nnzb = zcount;
    if (hflags[0] > 0)
        fail(NAIR_ENOMEM, "operator row has " + std::to_string(hflags[0]) + " blocks (limit " +
                              std::to_string(kRowBlocks) + ")");
    const int nnz = hflags[1], ncontrib = hflags[2];
    AP.nnzb = nnz;
    AP.colidx.alloc(static_cast<size_t>(nnz));
    if (!ymap) AP.vals.alloc(static_cast<size_t>(nnz) * bb);
    if (nnz == 0) return;
    DBuf<int> kptr(static_cast<size_t>(nnz) + 1), klist(static_cast<size_t>(ncontrib));
    M.krp = AP.rowptr.get();
    M.kcol = AP.colidx.get();
    M.crow = crow.get();
    M.kptr = kptr.get();
    M.klist = klist.get();
    if (narrow) k_merge_rows<1, uint32_t><<<gs, 256, 0, s>>>(M, flags);
    else k_merge_rows<1, uint64_t><<<gs, 256, 0, s>>>(M, flags);
    if (ymap) {
        DBuf<int> flag(static_cast<size_t>(nnz)), midx(static_cast<size_t>(nnz) + 1);
        k_ap_flags<<<grid_for(nnz, 256), 256, 0, s>>>(nnz, kptr.get(), flag.get());
        scan_exclusive(flag.get(), midx.get(), nnz, s);
        const int nm = read_int(midx.get() + nnz, s);
        ymap->alloc(static_cast<size_t>(nnz));
        merged->alloc(static_cast<size_t>(std::max(nm, 1)) * bb);
        DBuf<int> mblk(static_cast<size_t>(std::max(nm, 1)));
        k_ap_map<<<grid_for(nnz, 256), 256, 0, s>>>(nnz, kptr.get(), klist.get(), midx.get(), ymap->get(), mblk.get());
        if (nm > 0) {
            // the instance for blocks of at most 64, 128, 256 or 640 entries, else 16 chunks
            void (*kern)(int, int, const int *, const int *, const int *, const double *, double *) = k_ap_merged<16>;
            switch ((bb + 63) / 64) {
                case 1: kern = k_ap_merged<1>; break;
                case 2: kern = k_ap_merged<2>; break;
                case 4: kern = k_ap_merged<4>; break;
                case 10: kern = k_ap_merged<10>; break;
                default: break;
            }
            kern<<<cap_grid((static_cast<int64_t>(nm) + 3) / 4), 256, 0, s>>>(nm, bb, mblk.get(), kptr.get(),
                                                                             klist.get(), A.vals.get(), merged->get());
        }
        NAIR_HIP(hipGetLastError());
        return;
    }
    if (bb >= 64)
        k_rap_values_wave<<<cap_grid((static_cast<int64_t>(nnz) + 3) / 4), 256, 0, s>>>(nnz, bb, kptr.get(),
                                                                                      klist.get(), A.vals.get(),
                                                                                      AP.vals.get());
    else
        k_rap_values<<<cap_grid((static_cast<int64_t>(nnz) * bb + 255) / 256), 256, 0, s>>>(
            nnz, bb, kptr.get(), klist.get(), A.vals.get(), AP.vals.get());
    NAIR_HIP(hipGetLastError());
}

}  // namespace

void galerkin(DevBSR &Z, const int *cpts, const DevBSR &A, const int *pmap, int nc, double drop, DevBSR &K,
              int *margin, DBuf<double> &knext, DBuf<uint32_t> &kmask, int *zeros, hipStream_t s) {
    // A P first (P is one unit block per row: a merge of A's columns), then
    // K = R (A P) with R = [Z I]: its pattern and pair lists, and each block's
    // sum on the matrix cores (with its size and row mask) or by pairs
    const int bs = A.bs;
    const int bb = bs * bs;
    const bool fused = use_matrix_cores(bs);
    DevBSR AP;
    DBuf<int> ymap;
    DBuf<double> merged;
    merge_columns(A, pmap, nc, Z, AP, zeros, s, fused ? &ymap : nullptr, fused ? &merged : nullptr);
    DevBSR RK;
    Pairs P;
    spgemm_structure(Z, cpts, AP, RK, P, zeros + kSpgemmZeros, s);
    if (fused && P.n > 0) {   // the pairs name A's block or a merged block
        k_remap_y<<<grid_for(P.n, 256), 256, 0, s>>>(P.n, ymap.get(), P.pairs.get());
        NAIR_HIP(hipGetLastError());
    }
    const int m = nc;
    const int nnz = static_cast<int>(RK.nnzb);
    DBuf<double> kval, knorm(static_cast<size_t>(nnz));
    DBuf<uint32_t> kbits(fused ? nnz : 0);
    DBuf<uint8_t> keep(static_cast<size_t>(nnz));
    DBuf<int> kept(static_cast<size_t>(m));
    if (fused) {
        kval.alloc(static_cast<size_t>(nnz) * bb);
        if (nnz > 0) {
            TimerScope ts(TK_RAP, g_timer_level, s);
            launch_pair_sums(bs, nnz, P.pairptr.get(), P.pairs.get(), Z.vals.get(), A.vals.get(), merged.get(),
                             kval.get(), knorm.get(), kbits.get(), s);
        }
    } else {
        RK.vals.alloc(static_cast<size_t>(nnz) * bb);
        {
            TimerScope ts(TK_RAP, g_timer_level, s);
            spgemm_values(Z.vals.get(), AP, P, RK, s);
        }
        kval = std::move(RK.vals);
        launch_block_maxabs(kval.get(), nnz, bs, knorm.get(), s);
    }
    const int *krp = RK.rowptr.get();
    const int *kcol = RK.colidx.get();
    k_drop_mark<<<static_cast<unsigned>(std::max((m + 3) / 4, 1)), 256, 0, s>>>(krp, kcol, knorm.get(), m, drop,
                                                                               keep.get(), kept.get(), margin);
    NAIR_HIP(hipGetLastError());
    K.nb = nc;
    K.ncols = nc;
    K.bs = bs;
    K.rowptr.alloc(static_cast<size_t>(nc) + 1);
    scan_exclusive(kept.get(), K.rowptr.get(), m, s);
    // the kept count stays on the device (the next level reads it back with its first read)
    K.nnzb = -1;
    K.cap = nnz;
    K.colidx.alloc(static_cast<size_t>(nnz));
    K.vals.alloc(static_cast<size_t>(nnz) * bb);
    knext.alloc(static_cast<size_t>(nnz));
    const int *nk = K.rowptr.get() + m;
    DBuf<int> src(static_cast<size_t>(nnz));
    if (fused && nnz > 0) kmask.alloc(static_cast<size_t>(nnz));
    // (a block's size is its max-abs entry)
    k_compact_fill<<<grid_for(m, 256), 256, 0, s>>>(krp, kcol, keep.get(), knorm.get(), kbits.get(), m,
                                                    K.rowptr.get(), K.colidx.get(), src.get(), knext.get(),
                                                    kmask.get());
    NAIR_HIP(hipGetLastError());
    launch_block_gather(nnz, bs, kval.get(), src.get(), K.vals.get(), s, nk);
}

}  // namespace nair
