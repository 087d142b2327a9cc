// The sweeps' own copies of F rows.  Split copies (SplitCopy: the forward sweeps
// of the large levels), short rows (ShortRows: the small levels) and sweep copies:
// the F rows of a level operator (or its transpose) in F-list
// order, each without its diagonal block, with D_F^{-1} in the same order
// (SweepCopy).  A Jacobi F sweep then streams its matrix entries, column
// indices and inverse blocks contiguously instead of picking F rows out from
// between the C rows.  Built once per level and direction: an exact count of
// every row's off-diagonal blocks, a scan, and one wave per row copying its
// column indices, blocks (or face masks and rectangles) and D^{-1} block with
// consecutive lanes on consecutive words.  Nothing is read back to the host.
#include <algorithm>
#include <climits>

#include "common.h"

namespace nair {
namespace {

__global__ __launch_bounds__(256) void k_sweep_count(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                    const int *__restrict__ flist, int nF, int *__restrict__ cnt) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nF) return;
    const int I = flist[f];
    int c = 0;
    for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) c += colidx[t] != I ? 1 : 0;
    cnt[f] = c;
}

// One wave per F row f (I = flist[f]): blocks of A's row I other than the
// diagonal go to positions orp[f] ... in order: their column indices, and
// with FACE the face copy's masks and rc-word rectangles, else the source
// block index (osrc) for the row-compressed copy made next; D_I^{-1} goes to
// position f with the coefficient of input c for output a at c * bb/bs + a
// (dtrans: D_I^{-1} transposed; else as it is, for the sweeps that apply
// D^{-T}).  Nothing is written at or past cap.
template <bool FACE>
__global__ __launch_bounds__(256) void k_sweep_fill(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                   const double *__restrict__ src, const uint64_t *__restrict__ fmeta,
                                                   const double *__restrict__ dinv, const int *__restrict__ flist,
                                                   int nF, int w, int bs, bool dtrans, int64_t cap,
                                                   const int *__restrict__ orp,
                                                   int *__restrict__ ocol, uint64_t *__restrict__ ometa,
                                                   double *__restrict__ ovals, int *__restrict__ osrc,
                                                   double *__restrict__ odinv) {
    const int lane = threadIdx.x & 63;
    const int f = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    if (f >= nF) return;   // whole waves
    const int bb = bs * bs;
    const int I = flist[f];
    const int lo = rowptr[I], hi = rowptr[I + 1];
    const int o = orp[f];
    // the diagonal block's position (hi if the row has none)
    int dp = hi;
    for (int base = lo; base < hi; base += 64) {
        const int t = base + lane;
        const unsigned long long b = __ballot(t < hi && colidx[t] == I);
        if (b != 0ull) {
            dp = base + __builtin_ctzll(b);
            break;
        }
    }
    const int n = hi - lo;
    for (int k = lane; k < n; k += 64) {
        const int t = lo + k;
        const int64_t d = static_cast<int64_t>(o) + k - (t > dp ? 1 : 0);
        if (t == dp || d >= cap) continue;
        ocol[d] = colidx[t];
        if constexpr (FACE) ometa[d] = fmeta[t];
        else osrc[d] = t;
    }
    if constexpr (FACE) {
        const int64_t total = static_cast<int64_t>(n) * w;
        for (int64_t e = lane; e < total; e += 64) {
            const int k = static_cast<int>(e / w);
            const int64_t q = e - static_cast<int64_t>(k) * w;
            const int t = lo + k;
            const int64_t d = static_cast<int64_t>(o) + k - (t > dp ? 1 : 0);
            if (t == dp || d >= cap) continue;
            ovals[d * w + q] = src[static_cast<int64_t>(t) * w + q];
        }
    }
    const double *Di = dinv + static_cast<int64_t>(I) * bb;
    double *Do = odinv + static_cast<int64_t>(f) * bb;
    // every load of the inverse first (bs <= 32: at most 16 words per lane; words past
    // the block repeat its last, unused), then the stores
    constexpr int kChunks = 16;
    double v[kChunks];
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int e = lane + 64 * i < bb ? lane + 64 * i : bb - 1;
        const int c = e / bs, a = e - c * bs;   // output position: input c, output a
        v[i] = Di[dtrans ? a * bs + c : e];
    }
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int e = lane + 64 * i;
        if (e < bb) Do[e] = v[i];
    }
}

// mask[t] = masks[src[t]] (src null: masks[t]) and size[t] for t < count (past it empty).
__global__ __launch_bounds__(256) void k_rb_take(const uint32_t *__restrict__ masks, int64_t n, int bs,
                                                const int *__restrict__ src, const int *__restrict__ count,
                                                uint32_t *__restrict__ mask, int *__restrict__ size) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const uint32_t m = t < (count ? *count : n) ? masks[src ? src[t] : t] : 0u;
    mask[t] = m;
    size[t] = __popc(m) * bs;
}

// Block t's nonzero rows, in order, to out[off[t] ...]: one wave per block
// (four per workgroup), lane q of the stored entries taking entry c of the
// block's (q / bs)-th nonzero row, so consecutive lanes read consecutive
// words of a row and write consecutive words of the copy.
__global__ __launch_bounds__(256) void k_rb_fill(const double *__restrict__ vals, int64_t n, int bs,
                                                const int *__restrict__ src, const int *__restrict__ count,
                                                const uint32_t *__restrict__ mask, const int *__restrict__ off,
                                                double *__restrict__ out) {
    const int64_t bb = static_cast<int64_t>(bs) * bs;
    const int lane = threadIdx.x & 63;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (t >= (count ? *count : n)) return;
    const uint32_t m = mask[t];
    const int stored = __popc(m) * bs;
    const double *blk = vals + (src ? src[t] : t) * bb;
    double *o = out + off[t];
    // every load first, then the stores (at most bs * bs <= 1024 entries: 16 per lane)
    constexpr int kChunks = 16;
    double v[kChunks];
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int q = lane + 64 * i;
        v[i] = 0.0;
        if (q < stored) {
            const int k = q / bs, c = q - k * bs;
            uint32_t mm = m;
            for (int j = 0; j < k; ++j) mm &= mm - 1u;   // drop the k lower nonzero rows
            const int a = __ffs(static_cast<int>(mm)) - 1;
            v[i] = blk[a * bs + c];
        }
    }
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int q = lane + 64 * i;
        if (q < stored) o[q] = v[i];
    }
}

// Depth class of F row f (I = flist[f]) as a flag in one of three lists one
// after another (class 2, 1, 0): whether row I has an F-F block, and whether one
// of those F neighbours has one itself.  Index work only: the pattern rows of I
// and of its F neighbours.
__global__ __launch_bounds__(256) void k_depth_class(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                    const int8_t *__restrict__ cf, const int *__restrict__ flist,
                                                    int nF, int *__restrict__ flag) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nF) return;
    const int I = flist[f];
    int d = 0;
    for (int t = rowptr[I]; t < rowptr[I + 1] && d < 2; ++t) {
        const int J = colidx[t];
        if (J == I || cf[J] != 0) continue;
        d = 1;
        for (int q = rowptr[J]; q < rowptr[J + 1] && d < 2; ++q) {
            const int K = colidx[q];
            if (K != J && cf[K] == 0) d = 2;
        }
    }
    for (int c = 0; c < 3; ++c) flag[static_cast<int64_t>(c) * nF + f] = d == 2 - c ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_depth_place(const int *__restrict__ flist, const int *__restrict__ flag,
                                                    const int *__restrict__ pos, int nF, int *__restrict__ out,
                                                    int *__restrict__ counts) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f < 2) counts[f] = pos[(f + 1) * static_cast<int64_t>(nF)];
    if (f >= nF) return;
    for (int c = 0; c < 3; ++c) {
        const int64_t k = static_cast<int64_t>(c) * nF + f;
        if (flag[k]) out[pos[k]] = flist[f];
    }
}

// Blocks of F row f in columns outside F -> cnt[f], in F columns other than its own -> cnt[nF + f].
__global__ __launch_bounds__(256) void k_split_count(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                    const int8_t *__restrict__ cf, const int *__restrict__ flist,
                                                    int nF, int *__restrict__ cnt) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nF) return;
    const int I = flist[f];
    int c = 0, e = 0;
    for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
        const int J = colidx[t];
        if (J == I) continue;
        if (cf[J] == 0) ++e;
        else ++c;
    }
    cnt[f] = c;
    cnt[nF + f] = e;
}

// One wave per F row: its blocks' columns, coarse columns and source block
// indices (with FACE also the face masks) to their places, both parts in order.
template <bool FACE>
__global__ __launch_bounds__(256) void k_split_fill(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                   const int8_t *__restrict__ cf, const int *__restrict__ pmap,
                                                   const uint64_t *__restrict__ fmeta,
                                                   const int *__restrict__ flist, int nF, int64_t cap,
                                                   const int *__restrict__ orp, int *__restrict__ ocol,
                                                   int *__restrict__ occol, uint64_t *__restrict__ ometa,
                                                   int *__restrict__ osrc) {
    const int lane = threadIdx.x & 63;
    const int f = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    if (f >= nF) return;   // whole waves
    const int I = flist[f];
    const int lo = rowptr[I], hi = rowptr[I + 1];
    const unsigned long long below = (1ull << lane) - 1ull;
    int64_t oc = orp[f], of = orp[nF + f];
    for (int base = lo; base < hi; base += 64) {
        const int t = base + lane;
        const int J = t < hi ? colidx[t] : I;
        const bool keep = J != I;
        const bool inF = keep && cf[J] == 0;
        const unsigned long long bf = __ballot(inF), bc = __ballot(keep && !inF);
        const int64_t d = inF ? of + __popcll(bf & below) : oc + __popcll(bc & below);
        if (keep && d < cap) {
            ocol[d] = J;
            occol[d] = pmap[J];
            osrc[d] = t;
            if constexpr (FACE) ometa[d] = fmeta[t];
        }
        of += __popcll(bf);
        oc += __popcll(bc);
    }
}

// out's w-word rectangle d = vals' rectangle src[d], d < *count: one thread per word
__global__ __launch_bounds__(256) void k_take_rects(const double *__restrict__ vals, const int *__restrict__ src,
                                                   const int *__restrict__ count, int64_t cap, int w,
                                                   double *__restrict__ out) {
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t d = g / w;
    if (d >= cap || d >= *count) return;
    out[g] = vals[static_cast<int64_t>(src[d]) * w + (g - d * w)];
}

// One wave per F row: U_I, the union of its F-F blocks' nonzero rows (low words
// of the face masks, or row masks), and D_I^{-1} column by column, the columns
// outside U_I first (coefficient of the k-th such column for output a at k bs + a).
__global__ __launch_bounds__(256) void k_split_dinv(const double *__restrict__ dinv, const int *__restrict__ flist,
                                                   int nF, int bs, const int *__restrict__ orp,
                                                   const uint64_t *__restrict__ meta,
                                                   const uint32_t *__restrict__ rmask, uint32_t *__restrict__ umask,
                                                   double *__restrict__ odinv) {
    __shared__ int cols[4][32];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int f = blockIdx.x * 4 + wv;
    if (f >= nF) return;   // whole waves
    uint32_t u = 0;
    for (int t = orp[nF + f]; t < orp[nF + f + 1]; ++t) u |= meta ? static_cast<uint32_t>(meta[t]) : rmask[t];
    if (lane == 0) umask[f] = u;
    const int nN = bs - __popc(u);
    if (lane < bs) {
        const uint32_t below = (1u << lane) - 1u;
        const int pos = (u >> lane) & 1u ? nN + __popc(u & below) : __popc(~u & below);
        cols[wv][pos] = lane;
    }
    __builtin_amdgcn_wave_barrier();   // (each wave its own LDS row)
    const int bb = bs * bs;
    const double *Di = dinv + static_cast<int64_t>(flist[f]) * bb;
    double *Do = odinv + static_cast<int64_t>(f) * bb;
    // every load first (bs <= 32: at most 16 words per lane; words past the block repeat its last), then the stores
    constexpr int kChunks = 16;
    double v[kChunks];
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int e = lane + 64 * i < bb ? lane + 64 * i : bb - 1;
        const int k = e / bs, a = e - k * bs;
        v[i] = Di[a * bs + cols[wv][k]];
    }
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
        const int e = lane + 64 * i;
        if (e < bb) Do[e] = v[i];
    }
}

// Headers and columns of F rows f < nF and of Z's rows i < nc (ShortRows): one thread per row.
__global__ __launch_bounds__(256) void k_short_rows(const int *__restrict__ rowptr, const int *__restrict__ colidx,
                                                   const int *__restrict__ flist, int nF,
                                                   const int *__restrict__ pmap, const int *__restrict__ zrp,
                                                   const int *__restrict__ zcol, const int *__restrict__ cpts, int nc,
                                                   int4 *__restrict__ hdr, int2 *__restrict__ ent,
                                                   int4 *__restrict__ zhdr, int *__restrict__ zent) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < nF) {
        const int I = flist[g], lo = rowptr[I], hi = rowptr[I + 1];
        int n = 0, before = 0;
        for (int t = lo; t < hi; ++t) {
            const int J = colidx[t];
            if (J == I) continue;
            if (J < I) ++before;
            if (n < kShort) ent[static_cast<int64_t>(g) * kShort + n] = int2{J, pmap[J]};
            ++n;
        }
        for (int k = n; k < kShort; ++k) ent[static_cast<int64_t>(g) * kShort + k] = int2{0, -1};
        hdr[g] = int4{I, n, lo, before};
    } else if (g - nF < nc) {
        const int i = g - nF, lo = zrp[i], n = zrp[i + 1] - lo;
        for (int k = 0; k < kShort; ++k) zent[static_cast<int64_t>(i) * kShort + k] = k < n ? zcol[lo + k] : 0;
        zhdr[i] = int4{cpts[i], n, lo, 0};
    }
}

}  // namespace

void build_short_rows(const DevBSR &A, const DevBSR &Z, const int *flist, int nF, const int *cpts, int nc,
                      const int *pmap, ShortRows &S, hipStream_t s) {
    S = ShortRows();
    if (nF <= 0 || nc <= 0 || A.bs > 32) return;
    S.hdr.alloc(static_cast<size_t>(nF));
    S.ent.alloc(static_cast<size_t>(nF) * kShort);
    S.zhdr.alloc(static_cast<size_t>(nc));
    S.zent.alloc(static_cast<size_t>(nc) * kShort);
    k_short_rows<<<grid_for(static_cast<int64_t>(nF) + nc, 256), 256, 0, s>>>(
        A.rowptr.get(), A.colidx.get(), flist, nF, pmap, Z.rowptr.get(), Z.colidx.get(), cpts, nc, S.hdr.get(),
        S.ent.get(), S.zhdr.get(), S.zent.get());
    NAIR_HIP(hipGetLastError());
    S.on = true;
}

DBuf<int> order_by_depth(const DevBSR &A, const int8_t *cf, const int *flist, int nF, int *counts, hipStream_t s) {
    DBuf<int> flag(static_cast<size_t>(nF) * 3), pos(static_cast<size_t>(nF) * 3 + 1), out(static_cast<size_t>(nF));
    const unsigned grid = grid_for(nF, 256);
    k_depth_class<<<grid, 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), cf, flist, nF, flag.get());
    NAIR_HIP(hipGetLastError());
    scan_exclusive(flag.get(), pos.get(), 3 * nF, s);
    k_depth_place<<<grid, 256, 0, s>>>(flist, flag.get(), pos.get(), nF, out.get(), counts);
    NAIR_HIP(hipGetLastError());
    return out;
}

bool split_fits(const DevBSR &A, const FaceCopy &F, int nF) {
    const int64_t bb = static_cast<int64_t>(A.bs) * A.bs;
    return nF > 0 && nF <= INT_MAX / 3 && A.bs <= 32 &&
           (F.on || std::max<int64_t>(A.nnzb - nF, 1) * bb <= INT_MAX);
}

void build_split(const DevBSR &A, const FaceCopy &F, const double *dinv, const int8_t *cf, const int *pmap,
                 DBuf<int> &&list, int nF, int n1, int n2, SplitCopy &S, hipStream_t s, const uint32_t *amask) {
    S = SplitCopy();
    const int bs = A.bs;
    if (!split_fits(A, F, nF)) return;
    const bool face = F.on;
    S.flist = std::move(list);
    const int *flist = S.flist.get();
    S.nF = nF;
    S.n1 = n1;
    S.n2 = n2;
    S.rc = face ? F.rc : 0;
    S.cmax = face ? F.cmax : 0;
    S.cap = std::max<int64_t>(A.nnzb - nF, 1);   // (every row holds its diagonal block)
    S.rowptr.alloc(2 * static_cast<size_t>(nF) + 1);
    S.colidx.alloc(static_cast<size_t>(S.cap));
    S.ccol.alloc(static_cast<size_t>(S.cap));
    S.umask.alloc(static_cast<size_t>(nF));
    S.dinv.alloc(static_cast<size_t>(nF) * bs * bs);
    S.s.alloc(static_cast<size_t>(n1) * bs);
    S.w.alloc(static_cast<size_t>(n1) * bs);
    DBuf<int> cnt(2 * static_cast<size_t>(nF)), src(static_cast<size_t>(S.cap));
    k_split_count<<<grid_for(nF, 256), 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), cf, flist, nF, cnt.get());
    NAIR_HIP(hipGetLastError());
    scan_exclusive(cnt.get(), S.rowptr.get(), 2 * nF, s);
    const int *total = S.rowptr.get() + 2 * static_cast<int64_t>(nF);
    const unsigned grid = static_cast<unsigned>((nF + 3) / 4);
    if (face) {
        S.meta.alloc(static_cast<size_t>(S.cap));
        S.vals.alloc(static_cast<size_t>(S.cap) * F.rc);
        k_split_fill<true><<<grid, 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), cf, pmap, F.meta.get(), flist, nF,
                                                S.cap, S.rowptr.get(), S.colidx.get(), S.ccol.get(), S.meta.get(),
                                                src.get());
        NAIR_HIP(hipGetLastError());
        k_take_rects<<<grid_for(S.cap * F.rc, 256), 256, 0, s>>>(F.vals.get(), src.get(), total, S.cap, F.rc,
                                                                S.vals.get());
        NAIR_HIP(hipGetLastError());
    } else {
        k_split_fill<false><<<grid, 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), cf, pmap, nullptr, flist, nF, S.cap,
                                                 S.rowptr.get(), S.colidx.get(), S.ccol.get(), nullptr, src.get());
        NAIR_HIP(hipGetLastError());
        if (!build_row_blocks(A.vals.get(), S.cap, bs, S.rows, s, src.get(), total, amask))
            fail(NAIR_EDEVICE, "build_split: the level's rows exceed int32 offsets");
    }
    k_split_dinv<<<grid, 256, 0, s>>>(dinv, flist, nF, bs, S.rowptr.get(), face ? S.meta.get() : nullptr,
                                      S.rows.mask.get(), S.umask.get(), S.dinv.get());
    NAIR_HIP(hipGetLastError());
    S.on = true;
}

void split_to_float(SplitCopy &S, int bs, hipStream_t s) {
    if (!S.on) return;
    if (S.rc > 0) {
        if (S.vals32.get()) return;
        const int64_t nv = S.cap * S.rc;
        S.vals32.alloc(static_cast<size_t>(nv));
        launch_to_float(S.vals.get(), S.vals32.get(), nv, s);
    } else {
        row_blocks_to_float(S.rows, S.cap, bs, s);
    }
}

bool build_row_blocks(const double *vals, int64_t n, int bs, RowBlocks &R, hipStream_t s, const int *src,
                      const int *count, const uint32_t *masks) {
    R = RowBlocks();
    const int64_t bb = static_cast<int64_t>(bs) * bs;
    if (n <= 0 || bs < 1 || bs > 32 || n * bb > INT_MAX) return false;
    R.mask.alloc(static_cast<size_t>(n));
    R.off.alloc(static_cast<size_t>(n) + 1);
    R.vals.alloc(static_cast<size_t>(n * bb));   // (the rows kept take less; the total is not read back)
    DBuf<int> size(static_cast<size_t>(n));
    if (masks) {   // the blocks' row masks are known: no pass over their entries
        k_rb_take<<<grid_for(n, 256), 256, 0, s>>>(masks, n, bs, src, count, R.mask.get(), size.get());
        NAIR_HIP(hipGetLastError());
    } else {   // mask[t] and size[t] = nonzero rows * bs of block src[t] (t < count; past it empty)
        launch_block_scan(vals, n, bs, src, count, nullptr, nullptr, R.mask.get(), size.get(), s);
    }
    scan_exclusive(size.get(), R.off.get(), static_cast<int>(n), s);
    k_rb_fill<<<grid_for(n, 4), 256, 0, s>>>(vals, n, bs, src, count, R.mask.get(), R.off.get(), R.vals.get());
    NAIR_HIP(hipGetLastError());
    R.on = true;
    return true;
}

void row_blocks_to_float(RowBlocks &R, int64_t n, int bs, hipStream_t s) {
    if (!R.on || R.vals32.get()) return;
    const int64_t nv = n * bs * bs;
    R.vals32.alloc(static_cast<size_t>(nv));
    launch_to_float(R.vals.get(), R.vals32.get(), nv, s, R.off.get() + n);   // the rows kept: off[n] entries
}

void build_sweep(const DevBSR &A, const FaceCopy &F, const double *dinv, const int *flist, int nF, SweepCopy &S,
                 hipStream_t s, bool trans, const uint32_t *amask) {
    S = SweepCopy();
    if (nF <= 0 || A.nb == 0 || !dinv || !flist) return;
    const int bs = A.bs;
    const int bb = bs * bs;
    const bool face = F.on;
    const int w = face ? F.rc : bb;
    S.nF = nF;
    S.rc = face ? F.rc : 0;
    S.cmax = face ? F.cmax : 0;
    // every row of a level operator holds its diagonal block, so the F rows
    // hold at most nnzb - nF others
    S.cap = std::max<int64_t>(A.nnzb - nF, 1);
    S.rowptr.alloc(static_cast<size_t>(nF) + 1);
    S.colidx.alloc(static_cast<size_t>(S.cap));
    if (face) {
        S.vals.alloc(static_cast<size_t>(S.cap) * w);
        S.meta.alloc(static_cast<size_t>(S.cap));
    }
    S.dinv.alloc(static_cast<size_t>(nF) * bb);
    DBuf<int> cnt(static_cast<size_t>(nF));
    k_sweep_count<<<grid_for(nF, 256), 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), flist, nF, cnt.get());
    NAIR_HIP(hipGetLastError());
    scan_exclusive(cnt.get(), S.rowptr.get(), nF, s);
    const unsigned grid = static_cast<unsigned>((nF + 3) / 4);
    if (face) {
        k_sweep_fill<true><<<grid, 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), F.vals.get(), F.meta.get(), dinv,
                                                flist, nF, w, bs, !trans, S.cap, S.rowptr.get(), S.colidx.get(),
                                                S.meta.get(), S.vals.get(), nullptr, S.dinv.get());
        NAIR_HIP(hipGetLastError());
    } else {
        DBuf<int> src(static_cast<size_t>(S.cap));
        k_sweep_fill<false><<<grid, 256, 0, s>>>(A.rowptr.get(), A.colidx.get(), nullptr, nullptr, dinv, flist, nF,
                                                 w, bs, !trans, S.cap, S.rowptr.get(), S.colidx.get(), nullptr,
                                                 nullptr, src.get(), S.dinv.get());
        NAIR_HIP(hipGetLastError());
        if (!build_row_blocks(A.vals.get(), S.cap, bs, S.rows, s, src.get(), S.rowptr.get() + nF, amask)) return;
    }
    S.on = true;
}

void sweep_to_float(SweepCopy &S, int bs, hipStream_t s) {
    if (!S.on) return;
    if (S.rc > 0) {
        if (S.vals32.get()) return;
        const int64_t nv = S.cap * S.rc;
        S.vals32.alloc(static_cast<size_t>(nv));
        launch_to_float(S.vals.get(), S.vals32.get(), nv, s);
    } else {
        row_blocks_to_float(S.rows, S.cap, bs, s);
    }
}

}  // namespace nair
