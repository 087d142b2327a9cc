// Collapsed coarse cycle: on a small level (kCollapse) the cycle below it is a
// linear operator of that order, kept as one dense matrix.
//
// A cycle's small levels are a chain of launches of 3 to 6 us each (restriction,
// interpolation, sweeps, per level) that move next to no data: latency bounds
// them, not bytes.  One dense product takes 3 us at order 540, 5.7 us at 1440.  The
// matrix is formed at setup by running the cycle on all unit vectors at once:
// every vector of the levels concerned becomes an array [unknowns of the level]
// [order] with the columns across the lanes of a wave, so that an operator entry
// is one scalar for 64 columns and each step is one launch (0.15 ms in all at
// order 1440).  Everything is FP64, also under an FP32-stored hierarchy.
// One Q1 61 x 61 cycle 123 -> 96 us, FC solves at Q2 64 x 64 2.8 -> 1.9 ms,
// F-cycle solves at Q2 160 x 160 28.1 -> 22.5 ms.
#include <vector>

#include "hier.h"

namespace nair {
namespace {

constexpr int kCols = 64;    // columns per workgroup: one per lane
constexpr int kWaves = 4;    // a row's blocks are dealt to the waves (a single wave's chain of loads sets the time)

// Block sizes with an instance of their own; the others run the 32-wide one.
template <int BS>
struct Dim {
    static constexpr int kN = BS > 0 ? BS : kMaxBs;
};

// y[a] (LDS, stride kCols, this lane's column) += row a of the bs x bs block (the same for all lanes) times x,
// for a = first, first + step, ...
template <int BS>
__device__ inline void add_block(const double *__restrict__ blk, const double (&x)[Dim<BS>::kN], double *y, int bs,
                                 int first = 0, int step = 1) {
    for (int a = first; a < bs; a += step) {
        double s = y[a * kCols];
#pragma unroll
        for (int c = 0; c < Dim<BS>::kN; ++c)
            if (BS > 0 || c < bs) s = __builtin_fma(blk[a * bs + c], x[c], s);
        y[a * kCols] = s;
    }
}

// This lane's column of block J of v ([rows][ld]); zero past the columns.
template <int BS>
__device__ inline void load_block(const double *__restrict__ v, int64_t J, int64_t ld, int col, bool in, int bs,
                                  double (&x)[Dim<BS>::kN]) {
#pragma unroll
    for (int c = 0; c < Dim<BS>::kN; ++c) x[c] = (in && (BS > 0 || c < bs)) ? v[(J * bs + c) * ld + col] : 0.0;
}

// The workgroup's lanes: column, wave (a scalar), and this lane's column of the wave's LDS part [bs][kCols].
struct ColLane {
    int col, wave;
    bool in;
    double *y;
    __device__ ColLane(double *lds, int bs, int64_t ld) {
        wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kCols);
        col = blockIdx.y * kCols + static_cast<int>(threadIdx.x) % kCols;
        in = col < ld;
        y = lds + wave * bs * kCols + static_cast<int>(threadIdx.x) % kCols;
    }
};

// Sum over the row's blocks in columns J >= 0 (cmap nullable: J = cmap[column]) other than `skip`, into
// each wave's y; then, behind a barrier, the waves' sums of entry c.
template <int BS>
__device__ inline void row_blocks(const ColLane &L, const int *__restrict__ colidx, const int *__restrict__ cmap,
                                  const double *__restrict__ vals, int lo, int hi, int skip, int bs, int64_t ld,
                                  const double *__restrict__ v) {
    for (int a = 0; a < bs; ++a) L.y[a * kCols] = 0.0;
    double x[Dim<BS>::kN];
    for (int t = lo + L.wave; t < hi; t += kWaves) {
        const int J = colidx[t];
        const int p = J == skip ? -1 : (cmap ? cmap[J] : J);
        if (p < 0) continue;
        load_block<BS>(v, p, ld, L.col, L.in, bs, x);
        add_block<BS>(vals + static_cast<int64_t>(t) * bs * bs, x, L.y, bs);
    }
    __syncthreads();
}
__device__ inline double row_sum(const ColLane &L, int c, int bs) {
    const double *y = L.y - L.wave * bs * kCols + c * kCols;
    double s = y[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s += y[w * bs * kCols];
    return s;
}

// rc_i = r_{cpts[i]} + sum_t Z_it r_{col t}: workgroup (i, 64 columns)
template <int BS>
__global__ __launch_bounds__(kCols *kWaves) void k_cols_restrict(const int *__restrict__ zrp,
                                                                const int *__restrict__ zcol,
                                                                const double *__restrict__ zval, int bs_rt,
                                                                int64_t ld, const double *__restrict__ r,
                                                                const int *__restrict__ cpts,
                                                                double *__restrict__ rc) {
    extern __shared__ double lds[];
    const int bs = BS > 0 ? BS : bs_rt;
    const int i = blockIdx.x;
    const ColLane L(lds, bs, ld);
    row_blocks<BS>(L, zcol, nullptr, zval, zrp[i], zrp[i + 1], -1, bs, ld, r);
    if (L.in)
        for (int a = L.wave; a < bs; a += kWaves)
            rc[(static_cast<int64_t>(i) * bs + a) * ld + L.col] =
                r[(static_cast<int64_t>(cpts[i]) * bs + a) * ld + L.col] + row_sum(L, a, bs);
}

// One Jacobi sweep over the rows with cf == which: out_I = D_I^{-1}(r_I - sum_{J != I} A_IJ in_J).
// FIRST: `in` is e_c on the coarse level, read through pmap (zero where it is negative), and
// the other rows take P e_c in both out and out2; else, with copy, the other rows of out copy in.
template <int BS, bool FIRST>
__global__ __launch_bounds__(kCols *kWaves) void k_cols_sweep(const int *__restrict__ rowptr,
                                                             const int *__restrict__ colidx,
                                                             const double *__restrict__ vals,
                                                             const double *__restrict__ dinv, int bs_rt, int64_t ld,
                                                             const int8_t *__restrict__ cf, int which, bool copy,
                                                             const int *__restrict__ pmap,
                                                             const double *__restrict__ r,
                                                             const double *__restrict__ in_v,
                                                             double *__restrict__ out, double *__restrict__ out2) {
    extern __shared__ double lds[];
    const int bs = BS > 0 ? BS : bs_rt;
    const int I = blockIdx.x;
    const ColLane L(lds, bs, ld);
    if (cf[I] != which) {   // (the whole workgroup)
        if (!FIRST && !copy) return;
        const int p = FIRST ? pmap[I] : I;
        if (L.in)
            for (int a = L.wave; a < bs; a += kWaves) {
                const int64_t o = (static_cast<int64_t>(I) * bs + a) * ld + L.col;
                const double v = p >= 0 ? in_v[(static_cast<int64_t>(p) * bs + a) * ld + L.col] : 0.0;
                out[o] = v;
                if (FIRST) out2[o] = v;
            }
        return;
    }
    row_blocks<BS>(L, colidx, FIRST ? pmap : nullptr, vals, rowptr[I], rowptr[I + 1], I, bs, ld, in_v);
    double x[Dim<BS>::kN];
    load_block<BS>(r, I, ld, L.col, L.in, bs, x);
#pragma unroll
    for (int c = 0; c < Dim<BS>::kN; ++c)
        if (BS > 0 || c < bs) x[c] -= row_sum(L, c, bs);
    __syncthreads();   // (the sums are read: the waves' parts take D^{-1}'s product)
    for (int a = L.wave; a < bs; a += kWaves) L.y[a * kCols] = 0.0;
    add_block<BS>(dinv + static_cast<int64_t>(I) * bs * bs, x, L.y, bs, L.wave, kWaves);
    if (L.in)
        for (int a = L.wave; a < bs; a += kWaves) out[(static_cast<int64_t>(I) * bs + a) * ld + L.col] = L.y[a * kCols];
}

// out_I = r_I - (A x)_I on every row
template <int BS>
__global__ __launch_bounds__(kCols *kWaves) void k_cols_residual(const int *__restrict__ rowptr,
                                                                const int *__restrict__ colidx,
                                                                const double *__restrict__ vals, int bs_rt,
                                                                int64_t ld, const double *__restrict__ r,
                                                                const double *__restrict__ xv,
                                                                double *__restrict__ out) {
    extern __shared__ double lds[];
    const int bs = BS > 0 ? BS : bs_rt;
    const int I = blockIdx.x;
    const ColLane L(lds, bs, ld);
    row_blocks<BS>(L, colidx, nullptr, vals, rowptr[I], rowptr[I + 1], -1, bs, ld, xv);
    if (L.in)
        for (int a = L.wave; a < bs; a += kWaves) {
            const int64_t o = (static_cast<int64_t>(I) * bs + a) * ld + L.col;
            out[o] = r[o] - row_sum(L, a, bs);
        }
}

// out = M x for the dense n x n M: workgroup (row, 64 columns), every fourth term to a wave
__global__ __launch_bounds__(kCols *kWaves) void k_cols_dense(const double *__restrict__ M, int n, int64_t ld,
                                                             const double *__restrict__ x,
                                                             double *__restrict__ out) {
    extern __shared__ double lds[];
    const int i = blockIdx.x;
    const ColLane L(lds, 1, ld);
    const double *m = M + static_cast<int64_t>(i) * n;
    double s = 0.0;
    if (L.in) {
#pragma unroll 8
        for (int k = L.wave; k < n; k += kWaves) s = __builtin_fma(m[k], x[k * ld + L.col], s);
    }
    L.y[0] = s;
    __syncthreads();
    if (L.in && L.wave == 0) out[i * ld + L.col] = row_sum(L, 0, 1);
}

__global__ __launch_bounds__(256) void k_cols_identity(double *__restrict__ x, int n) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (g < static_cast<int64_t>(n) * n) x[g] = g / n == g % n ? 1.0 : 0.0;
}

// dst = src (add: dst += src)
__global__ __launch_bounds__(256) void k_cols_copy(double *__restrict__ dst, const double *__restrict__ src, int64_t n,
                                                  bool add) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (g < n) dst[g] = add ? dst[g] + src[g] : src[g];
}

__global__ __launch_bounds__(256) void k_square_transpose(const double *__restrict__ M, double *__restrict__ MT, int n) {
    __shared__ double tile[16][17];
    const int i0 = blockIdx.y * 16, j0 = blockIdx.x * 16, x = threadIdx.x & 15, y = threadIdx.x >> 4;
    if (i0 + y < n && j0 + x < n) tile[y][x] = M[static_cast<int64_t>(i0 + y) * n + j0 + x];
    __syncthreads();
    if (j0 + y < n && i0 + x < n) MT[static_cast<int64_t>(j0 + y) * n + i0 + x] = tile[x][y];
}

// y = M x: one wave per row of the n x n M
template <typename VT>
__global__ __launch_bounds__(256) void k_collapsed_mv(const double *__restrict__ M, int n, const VT *__restrict__ x,
                                                     VT *__restrict__ y) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    if (row >= n) return;
    const double *m = M + static_cast<int64_t>(row) * n;
    double s = 0.0;
    // every load first (at most kCollapse / 64 words of each per lane)
    constexpr int kW = kCollapse / 64;
    double mv[kW], xv[kW];
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        const int j = lane + 64 * i;
        mv[i] = j < n ? m[j] : 0.0;
        xv[i] = j < n ? static_cast<double>(x[j]) : 0.0;
    }
#pragma unroll
    for (int i = 0; i < kW; ++i) s += mv[i] * xv[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) y[row] = static_cast<VT>(s);
}

// The cycle of solve.cpp on all columns at once, from level m down.
struct ColsCycle {
    Hier &h;
    int m;
    int64_t ld;
    hipStream_t s;
    std::vector<DBuf<double>> r, e0, e1, fsave;   // by level - m

    ColsCycle(Hier &hh, int mm, hipStream_t st)
        : h(hh), m(mm), ld(static_cast<int64_t>(hh.lv[mm]->A.nb) * hh.bs), s(st) {
        const size_t k = h.lv.size() - m;
        r.resize(k);
        e0.resize(k);
        e1.resize(k);
        fsave.resize(k);
        for (size_t i = 0; i < k; ++i) {
            const size_t n = static_cast<size_t>(h.lv[m + i]->A.nb) * h.bs * ld;
            r[i].alloc(n);
            e0[i].alloc(n);
            e1[i].alloc(n);
            if (h.prm.cycle == 1) fsave[i].alloc(n);
        }
    }
    dim3 grid(int rows) const { return dim3(static_cast<unsigned>(rows), static_cast<unsigned>((ld + kCols - 1) / kCols)); }
    size_t lds() const { return sizeof(double) * kCols * kWaves * h.bs; }

    const double *cycle(int l, bool fcyc) {
        Level &L = *h.lv[l];
        const int bs = h.bs, i = l - m, nb = L.A.nb;
        if (L.coarsest) {
            k_cols_dense<<<grid(nb * bs), kCols * kWaves, sizeof(double) * kCols * kWaves, s>>>(L.dense_inv.get(), nb * bs, ld, r[i].get(), e0[i].get());
            NAIR_HIP(hipGetLastError());
            return e0[i].get();
        }
#define NAIR_COLS(KERNEL, ROWS, ...)                                                       \
    switch (bs) {                                                                          \
        case 1: KERNEL(1)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;            \
        case 4: KERNEL(4)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;            \
        case 9: KERNEL(9)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;            \
        case 16: KERNEL(16)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;          \
        case 25: KERNEL(25)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;          \
        default: KERNEL(0)<<<grid(ROWS), kCols * kWaves, lds(), s>>>(__VA_ARGS__); break;           \
    }                                                                                      \
    NAIR_HIP(hipGetLastError())
#define RESTRICT_K(BS) k_cols_restrict<BS>
#define FIRST_K(BS) k_cols_sweep<BS, true>
#define SWEEP_K(BS) k_cols_sweep<BS, false>
#define RESIDUAL_K(BS) k_cols_residual<BS>
        NAIR_COLS(RESTRICT_K, L.nc, L.Z.rowptr.get(), L.Z.colidx.get(), L.Z.vals.get(), bs, ld, r[i].get(),
                  L.cpts.get(), r[i + 1].get());
        const double *ec = coarse(l + 1, fcyc);
        double *cur = e0[i].get(), *oth = e1[i].get();
        NAIR_COLS(FIRST_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld, L.cf.get(), 0,
                  false, L.pmap.get(), r[i].get(), ec, cur, oth);
        for (int k = 1; k <= h.prm.degree; ++k) {
            NAIR_COLS(SWEEP_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld,
                      L.cf.get(), 0, false, L.pmap.get(), r[i].get(), cur, oth, nullptr);
            std::swap(cur, oth);
        }
        if (h.prm.relax == 1) {
            NAIR_COLS(SWEEP_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld,
                      L.cf.get(), 1, true, L.pmap.get(), r[i].get(), cur, oth, nullptr);
            std::swap(cur, oth);
        }
        return cur;
    }
    const double *coarse(int l, bool fcyc) {
        if (!fcyc) return cycle(l, false);
        Level &L = *h.lv[l];
        const int bs = h.bs, i = l - m;
        const int64_t n = static_cast<int64_t>(L.A.nb) * bs * ld;
        copy(fsave[i].get(), cycle(l, true), n, false);
        // (e0 is free: the V-cycle below writes it anew)
        NAIR_COLS(RESIDUAL_K, L.A.nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), bs, ld, r[i].get(),
                  fsave[i].get(), e0[i].get());
        copy(r[i].get(), e0[i].get(), n, false);
        copy(fsave[i].get(), cycle(l, false), n, true);
        return fsave[i].get();
    }
#undef NAIR_COLS
    void copy(double *dst, const double *src, int64_t n, bool add) {
        k_cols_copy<<<grid_for(n, 256), 256, 0, s>>>(dst, src, n, add);
        NAIR_HIP(hipGetLastError());
    }
    void identity() {
        k_cols_identity<<<grid_for(ld * ld, 256), 256, 0, s>>>(r[0].get(), static_cast<int>(ld));
        NAIR_HIP(hipGetLastError());
    }
};

}  // namespace

void build_collapse(Hier &h, hipStream_t s) {
    h.collapse = 0;
    if (h.nsys != 1) return;
    for (size_t l = 1; l + 1 < h.lv.size(); ++l) {
        const int64_t n = static_cast<int64_t>(h.lv[l]->A.nb) * h.bs;
        if (n > kCollapse || h.lv[l]->A.nb > kCollapseRows) continue;
        ColsCycle C(h, static_cast<int>(l), s);
        // (an F-cycle's coarse solves are F-cycles on its way down and V-cycles after)
        for (int f = 0; f <= (h.prm.cycle == 1 ? 1 : 0); ++f) {
            if (h.prm.cycle == 1 && f == 0 && l == 1) continue;   // the finest level's cycle is the F-cycle
            C.identity();
            h.coarse_op[f].alloc(static_cast<size_t>(n * n));
            C.copy(h.coarse_op[f].get(), C.coarse(static_cast<int>(l), f == 1), n * n, false);
        }
        h.collapse = static_cast<int>(l);
        return;
    }
}

void collapse_transpose(Hier &h, hipStream_t s) {
    if (h.collapse == 0) return;
    const int n = h.lv[h.collapse]->A.nb * h.bs;
    for (int f = 0; f < 2; ++f) {
        if (!h.coarse_op[f].get() || h.coarse_opT[f].get()) continue;
        h.coarse_opT[f].alloc(static_cast<size_t>(n) * n);
        const unsigned g = static_cast<unsigned>((n + 15) / 16);
        k_square_transpose<<<dim3(g, g), 256, 0, s>>>(h.coarse_op[f].get(), h.coarse_opT[f].get(), n);
        NAIR_HIP(hipGetLastError());
    }
}

template <typename VT>
void launch_collapsed(const Hier &h, bool fcyc, bool trans, const VT *r, VT *e, hipStream_t s) {
    const int n = h.lv[h.collapse]->A.nb * h.bs;
    const double *M = (trans ? h.coarse_opT : h.coarse_op)[fcyc ? 1 : 0].get();
    if (n > kCollapse || !M) fail(NAIR_EDEVICE, "launch_collapsed: no collapsed coarse cycle");
    TimerScope ts(TK_DENSE, h.collapse, s);
    k_collapsed_mv<VT><<<grid_for(n, 4), 256, 0, s>>>(M, n, r, e);
    NAIR_HIP(hipGetLastError());
}
template void launch_collapsed<double>(const Hier &, bool, bool, const double *, double *, hipStream_t);
template void launch_collapsed<float>(const Hier &, bool, bool, const float *, float *, hipStream_t);

}  // namespace nair
