// Collapsed coarse cycle: on a small level (kCollapse) the cycle below it is a
// linear operator of that order, kept as one dense matrix.
//
// A cycle's small levels are a chain of launches of 3 to 6 us each (restriction,
// interpolation, sweeps, per level) that move next to no data: latency bounds
// them, not bytes.  One dense product takes 3 us at order 540, 5.7 us at 1440.
// The matrix is formed at setup from the coarsest level's inverse upwards: a
// level's matrix is its cycle run on all its unit vectors at once, with the
// matrix of the level below as the coarse solve.  Every vector becomes an array
// [unknowns of the level] [order] with the columns across the lanes of a wave, so
// that an operator entry is one scalar for 64 columns and each step is one launch.
// At order 1512 (Q2 97 x 97) that is 0.19 ms of kernels in 15 launches.  Beside the
// matrix it needs 1.7 times its bytes while it runs (19 MiB at order 1192; an F-cycle's
// 3.8 times, 44 MiB): running the whole cycle from the level down on one set of columns
// took 0.17 ms and 5.6 times (60 MiB; F-cycle 81), and an F-cycle's launches grew with
// the square of the levels (setup of Q3 40 x 40 2.87 ms, 2.77 this way).
// Everything is FP64, also under an FP32-stored hierarchy.  The matrix is a copy of
// what the levels hold: where the device or the caller's allocator has no room
// for it, the cycle visits the levels instead.
// One Q1 61 x 61 cycle 123 -> 96 us, FC solves at Q2 64 x 64 2.8 -> 1.9 ms,
// F-cycle solves at Q2 160 x 160 28.1 -> 22.5 ms.
#include <algorithm>
#include <vector>

#include "hier.h"
#include "mfma_tile.h"

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

// This lane's column of block J of v ([rows][ld]; null: the unit vectors); zero past the columns.
template <int BS>
__device__ inline void load_block(const double *__restrict__ v, int64_t J, int64_t ld, int col, bool in, int bs,
                                  double (&x)[Dim<BS>::kN]) {
    if (!v) {
#pragma unroll
        for (int c = 0; c < Dim<BS>::kN; ++c) x[c] = (in && (BS > 0 || c < bs) && J * bs + c == col) ? 1.0 : 0.0;
        return;
    }
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

// Entry i of column `col` of v (null: the unit vectors)
__device__ inline double col_entry(const double *__restrict__ v, int64_t i, int64_t ld, int col) {
    return v ? v[i * ld + col] : (i == col ? 1.0 : 0.0);
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
                col_entry(r, static_cast<int64_t>(cpts[i]) * bs + a, ld, L.col) + row_sum(L, a, bs);
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
            const int64_t i = static_cast<int64_t>(I) * bs + a;
            out[i * ld + L.col] = col_entry(r, i, ld, L.col) - row_sum(L, a, bs);
        }
}

// out = M x for the dense n x n M on the matrix cores: workgroup (16 rows, 64
// columns), a quarter of the terms to a wave, four 16 x 16 tiles a wave.  Each step
// loads 16 terms before it multiplies them.  Order 675, 1512 columns: 49 us, against
// 83 us for eight rows of a lane on the vector units.
constexpr int kDenseRows = 16;
__global__ __launch_bounds__(kCols *kWaves) void k_cols_dense(const double *__restrict__ M, int n, int64_t ld,
                                                             const double *__restrict__ x,
                                                             double *__restrict__ out) {
    constexpr int T = kCols / 16, U = 4;
    __shared__ double lds[kWaves * kDenseRows * kCols];
    const int i0 = blockIdx.x * kDenseRows, j0 = blockIdx.y * kCols;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row16 = lane & 15, kk = lane >> 4;
    const int part = ((n + kWaves - 1) / kWaves + 3) / 4 * 4, k0 = wave * part, k1 = min(n, k0 + part);
    const double *m = M + static_cast<int64_t>(min(i0 + row16, n - 1)) * n;
    int64_t col[T];   // (rows, columns and terms past the last repeat it, terms with a zero of M)
#pragma unroll
    for (int t = 0; t < T; ++t) col[t] = min(static_cast<int64_t>(j0 + 16 * t + row16), ld - 1);
    double4_t acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = double4_t{0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < k1; k += 4 * U) {
        double a[U], b[U][T];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = k + 4 * u + kk, qc = min(q, k1 - 1);
            const double v = m[qc];
            a[u] = q < k1 ? v : 0.0;
#pragma unroll
            for (int t = 0; t < T; ++t) b[u][t] = x[qc * ld + col[t]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u][t], acc[t], 0, 0, 0);
    }
    double *y = lds + wave * kDenseRows * kCols;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[(kk + 4 * r) * kCols + 16 * t + row16] = acc[t][r];
    __syncthreads();
    for (int e = threadIdx.x; e < kDenseRows * kCols; e += kCols * kWaves) {
        const int i = i0 + e / kCols;
        const int64_t c = j0 + e % kCols;
        if (i < n && c < ld) {
            double v = lds[e];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) v += lds[w * kDenseRows * kCols + e];
            out[i * ld + c] = v;
        }
    }
}

// dst = a + b (dst may be a)
__global__ __launch_bounds__(256) void k_cols_sum(double *dst, const double *a, const double *__restrict__ b,
                                                 int64_t n) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (g < n) dst[g] = a[g] + b[g];
}

__global__ __launch_bounds__(256) void k_square_transpose(const double *__restrict__ M, double *__restrict__ MT, int n) {
    __shared__ double tile[16][17];
    const int i0 = blockIdx.y * 16, j0 = blockIdx.x * 16, x = threadIdx.x & 15, y = threadIdx.x >> 4;
    if (i0 + y < n && j0 + x < n) tile[y][x] = M[static_cast<int64_t>(i0 + y) * n + j0 + x];
    __syncthreads();
    if (j0 + y < n && i0 + x < n) MT[static_cast<int64_t>(j0 + y) * n + i0 + x] = tile[x][y];
}

// y = M x (TRANS: M^T x, the same sums read down M's columns): one wave per entry of y
template <typename VT, bool TRANS>
__global__ __launch_bounds__(256) void k_collapsed_mv(const double *__restrict__ M, int n, const VT *__restrict__ x,
                                                     VT *__restrict__ y) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    if (row >= n) return;
    const double *m = M + (TRANS ? row : static_cast<int64_t>(row) * n);
    double s = 0.0;
    // every load first (at most kCollapse / 64 words of each per lane)
    constexpr int kW = kCollapse / 64;
    double mv[kW], xv[kW];
#pragma unroll
    for (int i = 0; i < kW; ++i) {
        const int j = lane + 64 * i;
        mv[i] = j < n ? m[TRANS ? static_cast<int64_t>(j) * n : j] : 0.0;
        xv[i] = j < n ? static_cast<double>(x[j]) : 0.0;
    }
    // (a zero of M is no dependence: a NaN or infinity of x stays out of the rows that do not depend on it)
#pragma unroll
    for (int i = 0; i < kW; ++i) s += mv[i] != 0.0 ? mv[i] * xv[i] : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) y[row] = static_cast<VT>(s);
}

// The cycle of solve.cpp on all columns at once, level by level.
struct ColsCycle {
    Hier &h;
    hipStream_t s;
    int64_t ld = 0;   // columns: the unknowns of the level whose matrix is being formed

    dim3 grid(int rows) const { return dim3(static_cast<unsigned>(rows), static_cast<unsigned>((ld + kCols - 1) / kCols)); }
    size_t lds() const { return sizeof(double) * kCols * kWaves * h.bs; }
    int order(int l) const { return h.lv[l]->A.nb * h.bs; }

    void dense(const double *M, int n, const double *x, double *out) {
        k_cols_dense<<<grid((n + kDenseRows - 1) / kDenseRows), kCols * kWaves, 0, s>>>(M, n, ld, x, out);
        NAIR_HIP(hipGetLastError());
    }
    void sum(double *dst, const double *a, const double *b, int64_t n) {
        k_cols_sum<<<grid_for(n, 256), 256, 0, s>>>(dst, a, b, n);
        NAIR_HIP(hipGetLastError());
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

    // out = level l's cycle of the columns r (null: the unit vectors), Mc the coarse solve on level l + 1;
    // tmp as large as out, ec of level l + 1's unknowns
    void cycle(int l, const double *r, const double *Mc, double *out, double *tmp, double *ec) {
        const Level &L = *h.lv[l];
        const int bs = h.bs, nb = L.A.nb;
        double *rc = tmp;   // (read before the first sweep)
        NAIR_COLS(RESTRICT_K, L.nc, L.Z.rowptr.get(), L.Z.colidx.get(), L.Z.vals.get(), bs, ld, r, L.cpts.get(), rc);
        dense(Mc, order(l + 1), rc, ec);
        const int sweeps = h.prm.degree + 1 + (h.prm.relax == 1 ? 1 : 0);
        double *cur = sweeps % 2 == 0 ? out : tmp, *oth = sweeps % 2 == 0 ? tmp : out;   // the last sweep writes out
        NAIR_COLS(FIRST_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld, L.cf.get(), 0,
                  false, L.pmap.get(), r, ec, oth, cur);
        std::swap(cur, oth);
        for (int k = 1; k <= h.prm.degree; ++k) {
            NAIR_COLS(SWEEP_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld,
                      L.cf.get(), 0, false, L.pmap.get(), r, cur, oth, nullptr);
            std::swap(cur, oth);
        }
        if (h.prm.relax == 1)
            NAIR_COLS(SWEEP_K, nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), L.dinv.get(), bs, ld,
                      L.cf.get(), 1, true, L.pmap.get(), r, cur, oth, nullptr);
    }
    // out = I - A x on level l
    void residual(int l, const double *x, double *out) {
        const Level &L = *h.lv[l];
        const int bs = h.bs;
        NAIR_COLS(RESIDUAL_K, L.A.nb, L.A.rowptr.get(), L.A.colidx.get(), L.A.vals.get(), bs, ld, nullptr, x, out);
    }
#undef NAIR_COLS

    // V = the V-cycle on level l, F (nullable) = its coarse solve in an F-cycle, F r + V (r - A F r), from those of
    // the level below
    void matrices(int l, const double *Vc, const double *Fc, double *V, double *F) {
        const int n = order(l);
        ld = n;
        const int64_t nn = static_cast<int64_t>(n) * n;
        if (h.lv[l]->coarsest) {   // (V: the dense inverse itself)
            const double *D = h.lv[l]->dense_inv.get();
            if (F) {
                DBuf<double> res(nn);
                residual(l, D, res.get());
                dense(D, n, res.get(), F);
                sum(F, F, D, nn);
            }
            return;
        }
        DBuf<double> tmp(nn), ec(static_cast<size_t>(order(l + 1)) * n);
        if (V) cycle(l, nullptr, Vc, V, tmp.get(), ec.get());
        if (F) {
            DBuf<double> res(nn), out(nn);
            cycle(l, nullptr, Fc, F, tmp.get(), ec.get());
            residual(l, F, res.get());
            cycle(l, res.get(), Vc, out.get(), tmp.get(), ec.get());
            sum(F, F, out.get(), nn);
        }
    }
};

}  // namespace

void build_collapse(Hier &h, hipStream_t s) {
    h.collapse = 0;
    if (h.nsys != 1) return;
    for (size_t l = 1; l + 1 < h.lv.size(); ++l) {
        const int64_t n = static_cast<int64_t>(h.lv[l]->A.nb) * h.bs;
        if (n > kCollapse || h.lv[l]->A.nb > kCollapseRows) continue;
        try {
            ColsCycle C{h, s};
            // (the finest level's own cycle is the F-cycle: its coarse solve never is a V-cycle)
            const bool fc = h.prm.cycle == 1, want[2] = {!fc || l > 1, fc};
            DBuf<double> below[2];
            for (size_t k = h.lv.size() - 1; k >= l; --k) {
                const size_t nn = static_cast<size_t>(C.order(static_cast<int>(k))) * C.order(static_cast<int>(k));
                DBuf<double> M[2];
                const bool last = h.lv[k]->coarsest;
                if (!last && (k > l || want[0])) M[0].alloc(nn);
                if (fc) M[1].alloc(nn);
                const double *Vc = !last && h.lv[k + 1]->coarsest ? h.lv[k + 1]->dense_inv.get() : below[0].get();
                C.matrices(static_cast<int>(k), Vc, below[1].get(), M[0].get(), M[1].get());
                for (int f = 0; f < 2; ++f) below[f] = std::move(M[f]);
            }
            for (int f = 0; f < 2; ++f) h.coarse_op[f] = std::move(below[f]);
            h.collapse = static_cast<int>(l);
        } catch (const Error &e) {
            if (e.code != NAIR_ENOMEM) throw;   // (no room: the cycle visits the levels)
        }
        return;
    }
}

void collapse_transpose(Hier &h, hipStream_t s) {
    if (h.collapse == 0) return;
    const int n = h.lv[h.collapse]->A.nb * h.bs;
    for (int f = 0; f < 2; ++f) {
        if (!h.coarse_op[f].get() || h.coarse_opT[f].get()) continue;
        try {
            h.coarse_opT[f].alloc(static_cast<size_t>(n) * n);
        } catch (const Error &e) {
            if (e.code != NAIR_ENOMEM) throw;
            continue;   // (no room: the transposed products read down M's columns)
        }
        const unsigned g = static_cast<unsigned>((n + 15) / 16);
        k_square_transpose<<<dim3(g, g), 256, 0, s>>>(h.coarse_op[f].get(), h.coarse_opT[f].get(), n);
        NAIR_HIP(hipGetLastError());
    }
}

template <typename VT>
void launch_collapsed(const Hier &h, bool fcyc, bool trans, const VT *r, VT *e, hipStream_t s) {
    const int n = h.lv[h.collapse]->A.nb * h.bs;
    const double *M = h.coarse_op[fcyc ? 1 : 0].get(), *MT = h.coarse_opT[fcyc ? 1 : 0].get();
    if (n > kCollapse || !M) fail(NAIR_EDEVICE, "launch_collapsed: no collapsed coarse cycle");
    TimerScope ts(TK_DENSE, h.collapse, s);
    const unsigned g = grid_for(n, 4);
    if (trans && !MT) k_collapsed_mv<VT, true><<<g, 256, 0, s>>>(M, n, r, e);
    else k_collapsed_mv<VT, false><<<g, 256, 0, s>>>(trans ? MT : M, n, r, e);
    NAIR_HIP(hipGetLastError());
}
template void launch_collapsed<double>(const Hier &, bool, bool, const double *, double *, hipStream_t);
template void launch_collapsed<float>(const Hier &, bool, bool, const float *, float *, hipStream_t);

}  // namespace nair
