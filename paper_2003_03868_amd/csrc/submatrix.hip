// Submatrix method (section "Submatrix Method"): the density matrix from
// one small dense problem per block column instead of sparse products over
// the whole matrix.
//
// For block column j let N_j be the block rows with a stored block in
// column j (ascending; j itself included).  T_j = H[N_j, N_j] is the dense
// principal submatrix over those block rows, P_j = (I - sign(T_j - mu I))/2
// its density matrix, and block column j of P is P_j's block column of j,
// on H's pattern; P is filtered with the block-norm rule at the end.
//
// Each sign(T_j - mu I) is taken by the dense Newton-Schulz iteration
//   X_0 = (T_j - mu I) / ||T_j - mu I||_inf
//   k = 0, 1, ...:  Y = X_k X_k;  r_k = ||Y - I||_F / n_j;  stop if r_k < tol
//                   X_{k+1} = 1.5 X_k - 0.5 X_k Y
// with every submatrix of a batch advanced together and each stopped on its
// own residual.  Submatrices live densely in HBM, padded to multiples of 32
// (the padding stays zero through both products); the products run on the
// FP64 matrix cores in one launch over the 64 x 64 tiles of all active
// submatrices, the last tile row and column 32 wide where the edge ends there.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "bsm_internal.h"
#include "lds_dma.h"

namespace bsm {

namespace {

constexpr int kTile = 64;      // output tile edge of the dense product
constexpr int kPad = 32;       // submatrix edges are padded to a multiple of this
constexpr int kTk = 16;        // k depth staged per LDS stage

typedef double d4 __attribute__((ext_vector_type(4)));

struct SubGemm {
    const int4 *tiles;         // (submatrix, tile row, tile column, buffer of X)
    int32_t ntiles;
    const int64_t *base;       // per submatrix: offset (doubles) in every buffer
    const int32_t *npad;       // per submatrix: padded edge (multiple of 32)
    const int32_t *ndim;       // per submatrix: true edge n_j
    double *buf0, *buf1, *ybuf;
    int32_t mode;              // 0: Y = X X (+ residual partials); 1: X' = 1.5 X - 0.5 X Y
    double *partial;           // mode 0: per tile, sum over its entries of (Y - I)^2
};

typedef __attribute__((address_space(3))) double lds_double;

// One 64 x 64 tile of D = A B (mode 0: A = B = X, D = Y; mode 1: A = X,
// B = Y, D = 1.5 X - 0.5 A B into the other X buffer).  Four waves, each a
// 32 x 32 quarter as 2 x 2 tiles of V_MFMA_F64_16X16X4_F64: lane l feeds
// A(i = l % 16, k = l / 16) and B(k = l / 16, j = l % 16) and receives
// D(i = 4 r + l / 16, j = l % 16) in register r.  Sums ascend in k.
//
// Operands go from memory to LDS past the registers, 16 k at a time and
// double-buffered: step i + 1 is on its way while step i is multiplied, with
// one barrier a step.  B's stage holds 16 rows of 64 columns; a step reads
// four rows at a time, so their 16-column groups are stored turned by the row
// (group g of row k at g ^ k % 4) and the 64 lanes spread over all banks.
//
// SYM (H is its own transpose, so X and Y are too): the launch lists the
// tiles on and above the diagonal, a quarter below it is skipped, and every
// element is stored with its mirror image; A(i, k) = X(k, i) is staged from
// X's rows like B.  Both images hold the same bits: one computed for itself
// would differ by rounding, a difference that the iteration doubles.
// Without SYM, A's stage holds 64 rows of 16 k, the 16-byte chunk c of row i
// at c ^ i / 2 % 8, for the same reason.
//
// A tile that reaches past the padded edge is 32 rows or columns wide: the
// waves of its missing half skip their products and stores, and the staging
// loads of that half are folded into the square (data that only those idle
// waves would read).
template <bool SYM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_sub_gemm(SubGemm g) {
    // consecutive tiles (one submatrix) on one XCD: workgroups b, b+8, ...
    // share an XCD's L2
    const int per = (g.ntiles + kXcds - 1) / kXcds;
    const int tix = static_cast<int>(blockIdx.x % kXcds) * per + static_cast<int>(blockIdx.x / kXcds);
    if (tix >= g.ntiles) return;
    const int4 td = g.tiles[tix];
    const int sub = td.x;
    const int ld = g.npad[sub], n = g.ndim[sub];
    const int64_t base = g.base[sub];
    const double *X = (td.w ? g.buf1 : g.buf0) + base;
    const double *Bm = g.mode == 0 ? X : g.ybuf + base;
    double *D = g.mode == 0 ? g.ybuf + base : (td.w ? g.buf0 : g.buf1) + base;
    const int r0 = td.y * kTile, c0 = td.z * kTile;
    const int vr = min(kTile, ld - r0), vc = min(kTile, ld - c0);   // 32 or 64

    __shared__ __attribute__((aligned(16))) double stage[2][2][kTk * kTile];   // [buffer][A, B]
    __shared__ double red[4];

    const int t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l16 = lane & 15, l4 = lane >> 4;
    const int wr = (w >> 1) * 32, wc = (w & 1) * 32;
    const bool busy = wr < vr && wc < vc && !(SYM && r0 + wr > c0 + wc);   // wave-uniform

    // A wave copies two kilobytes of either stage; byte offsets of the lane's
    // 16 from (row k or k 0 of the step, first row or column of the tile).
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (lds_double *)&stage[0][0][0]));
    uint32_t va[2], vb[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int k = (2 * w + q) * 2 + (lane >> 5), c = lane & 31;
        const int grp = (c >> 3) ^ (k & 3);
        vb[q] = (static_cast<uint32_t>(k) * ld + (grp & (vc / 16 - 1)) * 16 + (c & 7) * 2) * 8;
        if (SYM) {
            va[q] = (static_cast<uint32_t>(k) * ld + (grp & (vr / 16 - 1)) * 16 + (c & 7) * 2) * 8;
        } else {
            const int i = (2 * w + q) * 8 + (lane >> 3);
            va[q] = (static_cast<uint32_t>(i & (vr - 1)) * ld + ((lane & 7) ^ ((i >> 1) & 7)) * 2) * 8;
        }
    }
    const double *pa = SYM ? X + r0 : X + static_cast<int64_t>(r0) * ld;
    const double *pb = Bm + c0;
    const int64_t stepb = static_cast<int64_t>(kTk) * ld, stepa = SYM ? stepb : kTk;
    auto copy = [&](int buf) {
        const uint32_t slot = lds0 + buf * (2 * kTk * kTile * 8) + w * 2048;
        dma16(slot, va[0], pa);
        dma16(slot + 1024, va[1], pa);
        dma16(slot + kTk * kTile * 8, vb[0], pb);
        dma16(slot + kTk * kTile * 8 + 1024, vb[1], pb);
        pa += stepa;
        pb += stepb;
    };

    d4 acc[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[s][u] = d4{0.0, 0.0, 0.0, 0.0};
    // the lane's operands in a stage (doubles): columns of the quarter's two
    // 16-wide halves, row l4 of four
    int oa[2], ob[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        oa[s] = l4 * kTile + ((wr / 16 + s) ^ l4) * 16 + l16;
        ob[s] = l4 * kTile + ((wc / 16 + s) ^ l4) * 16 + l16;
    }
    auto compute = [&](int buf) {
        const double *A = stage[buf][0], *B = stage[buf][1];
#pragma unroll
        for (int kk = 0; kk < kTk / 4; ++kk) {
            double a[2], b[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                b[s] = B[kk * 4 * kTile + ob[s]];
                if (SYM) a[s] = A[kk * 4 * kTile + oa[s]];
                else a[s] = A[(wr + 16 * s + l16) * kTk + ((2 * kk + (l4 >> 1)) ^ (l16 >> 1)) * 2 + (l4 & 1)];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[s][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[u], acc[s][u], 0, 0, 0);
        }
    };

    // k steps up to the edge rounded to kTk (the padding beyond it is zero,
    // so the remaining steps would add nothing): nk >= 1
    const int nk = (n + kTk - 1) / kTk;
    copy(0);
    for (int i = 0; i < nk; ++i) {
        wait_dma();                       // the wave's part of step i has arrived;
        group_barrier();                   // all parts have, and step i - 1 is read
        if (i + 1 < nk) copy((i + 1) & 1);
        if (busy) compute(i & 1);
    }

    double res = 0.0;
    if (busy) {
        const bool diag = SYM && r0 + wr == c0 + wc;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = r0 + wr + 16 * s + 4 * e + l4, c = c0 + wc + 16 * u + l16;
                    if (diag && r > c) continue;
                    const int64_t o = static_cast<int64_t>(r) * ld + c;
                    double v = acc[s][u][e];
                    if (g.mode == 0) {
                        const double d = v - ((r == c && r < n) ? 1.0 : 0.0);
                        res += (SYM && r != c) ? 2.0 * (d * d) : d * d;
                    } else {
                        v = 1.5 * X[o] - 0.5 * v;
                    }
                    D[o] = v;
                    if (SYM && r != c) D[static_cast<int64_t>(c) * ld + r] = v;
                }
    }
    if (g.mode == 0) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) res += __shfl_xor(res, off);
        if (lane == 0) red[w] = res;
        __syncthreads();
        if (t == 0) g.partial[tix] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// Workgroups of the kernels over block rows, which take rows in turn.
constexpr int kRowGroups = 4096;

// Adds to *mirrored (zero beforehand) the number of stored blocks (i, j) with a
// stored (j, i) of the mirrored values: H is its own transpose where that is
// all of them.  One workgroup per block row at a time, a wave per block; NaN
// is unequal to itself.
__global__ __launch_bounds__(256) void k_sub_symmetric(const int64_t *row_ptr, const int32_t *col_idx,
                                                       const int64_t *blk_off, const double *vals,
                                                       const int32_t *rbs, int32_t nb,
                                                       unsigned long long *mirrored) {
    __shared__ unsigned long long cnt[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long n = 0;
    for (int i = blockIdx.x; i < nb; i += gridDim.x) {
        const int bi = rbs[i];
        for (int64_t t = row_ptr[i] + w; t < row_ptr[i + 1]; t += 4) {
            const int j = col_idx[t];
            int64_t lo = row_ptr[j], hi = row_ptr[j + 1];
            const int64_t end = hi;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (col_idx[mid] < i) lo = mid + 1; else hi = mid;
            }
            bool same = lo < end && col_idx[lo] == i;
            if (same) {
                const int bj = rbs[j];
                const double *a = vals + blk_off[t], *b = vals + blk_off[lo];
                for (int u = lane; u < bi * bj; u += 64) same = same && a[u] == b[u % bj * bi + u / bj];
            }
            if (__all(same)) ++n;
        }
    }
    if (lane == 0) cnt[w] = n;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(mirrored, cnt[0] + cnt[1] + cnt[2] + cnt[3]);
}

// r = ||Y - I||_F / n per active submatrix from its tiles' partial sums
// (tiles of one submatrix are consecutive; summed in tile order).
__global__ void k_sub_resid(const double *partial, const int32_t *act_sub, const int32_t *tile_lo,
                            const int32_t *tile_hi, const int32_t *ndim, double *r, int32_t nact) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= nact) return;
    double s = 0.0;
    for (int u = tile_lo[a]; u < tile_hi[a]; ++u) s += partial[u];
    r[a] = sqrt(s) / static_cast<double>(ndim[act_sub[a]]);
}

// Row sums of |H - mu I| of every stored block, one per row: those of block t
// at sums[t max_b].  One workgroup per block row at a time, a thread per row of
// a block.
__global__ __launch_bounds__(256) void k_sub_block_sums(const int64_t *row_ptr, const int32_t *col_idx,
                                                        const int64_t *blk_off, const double *vals,
                                                        const int32_t *rbs, int32_t nb, double mu,
                                                        int max_b, double *sums) {
    for (int i = blockIdx.x; i < nb; i += gridDim.x) {
        const int bi = rbs[i];
        const int64_t t0 = row_ptr[i], n = (row_ptr[i + 1] - t0) * bi;
        for (int64_t q = threadIdx.x; q < n; q += blockDim.x) {
            const int64_t t = t0 + q / bi;
            const int u = static_cast<int>(q % bi), j = col_idx[t], bj = rbs[j];
            const double *h = vals + blk_off[t] + static_cast<int64_t>(u) * bj;
            double s = 0.0;
            for (int v = 0; v < bj; ++v) s += fabs(h[v] - ((j == i && u == v) ? mu : 0.0));
            sums[t * max_b + u] = s;
        }
    }
}

// Stored block (i, k) among the columns of block row i, or p1.
__device__ inline int64_t sub_find(const int32_t *col_idx, int64_t p0, int64_t p1, int32_t k) {
    int64_t lo = p0, hi = p1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col_idx[mid] < k) lo = mid + 1; else hi = mid;
    }
    return lo < p1 && col_idx[lo] == k ? lo : p1;
}

// ||T_j - mu I||_inf per submatrix from the blocks' row sums, into the bits of
// scale[sub] (zero beforehand): one 64-lane group per (submatrix, block row
// a), lane f looking up block column f of the submatrix, lane u keeping row u.
// Reading the assembled T_j instead took 0.51 ms for 1.9 GB, and scaling it
// afterwards 0.81 ms; this way the gather writes scaled values (MI355X, 6192
// submatrices of mean edge 189).
__global__ void k_sub_norm(const int64_t *row_ptr, const int32_t *col_idx, int max_b,
                           const double *sums, const int32_t *rbs, const int32_t *ent_row,
                           const int32_t *ent_sub, const int64_t *sub_ent0, double *scale,
                           int64_t nent) {
    const int64_t e = blockIdx.x;
    if (e >= nent) return;
    const int sub = ent_sub[e], i = ent_row[e], bi = rbs[i];
    const int lane = threadIdx.x;
    const int64_t p0 = row_ptr[i], p1 = row_ptr[i + 1], f1 = sub_ent0[sub + 1];
    double row = 0.0;
    for (int64_t f0 = sub_ent0[sub]; f0 < f1; f0 += 64) {
        const int64_t t = f0 + lane < f1 ? sub_find(col_idx, p0, p1, ent_row[f0 + lane]) : p1;
        const double *b = t < p1 ? sums + t * max_b : nullptr;
        for (int u = 0; u < bi; ++u) {
            double s = b ? b[u] : 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
            if (lane == u) row += s;
        }
    }
    double mx = row > 0.0 ? row : 0.0;      // a NaN sum is left to the residual
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    // sums are not negative: their bits are ordered like the values
    if (lane == 0)
        atomicMax(reinterpret_cast<unsigned long long *>(scale) + sub,
                  static_cast<unsigned long long>(__double_as_longlong(mx)));
}

// X_0 = (T_j - mu I) / scale from the stored blocks: one 64-lane group per
// (submatrix, block row a); lane f looks block column f of the submatrix up in
// H's row N_j[a] and copies it when stored.  The buffer is zero beforehand.
__global__ void k_sub_gather(const int64_t *row_ptr, const int32_t *col_idx, const int64_t *blk_off,
                             const double *vals, const int32_t *rbs, const int32_t *ent_row,
                             const int32_t *ent_soff, const int32_t *ent_sub,
                             const int64_t *sub_ent0, const int64_t *base, const int32_t *npad,
                             const double *scale, double mu, double *X, int64_t nent) {
    const int64_t e = blockIdx.x;
    if (e >= nent) return;
    const int sub = ent_sub[e];
    const int i = ent_row[e];
    const int ra = ent_soff[e];
    const int bi = rbs[i];
    const int ld = npad[sub];
    const double scl = 1.0 / scale[sub];
    double *T = X + base[sub];
    const int64_t p0 = row_ptr[i], p1 = row_ptr[i + 1];
    for (int64_t f = sub_ent0[sub] + threadIdx.x; f < sub_ent0[sub + 1]; f += blockDim.x) {
        const int k = ent_row[f];
        const int64_t t = sub_find(col_idx, p0, p1, k);
        if (t >= p1) continue;
        const int bk = rbs[k];
        const int cb = ent_soff[f];
        const double *src = vals + blk_off[t];
        for (int u = 0; u < bi; ++u)
            for (int v = 0; v < bk; ++v)
                T[static_cast<int64_t>(ra + u) * ld + cb + v] =
                    (src[u * bk + v] - ((k == i && u == v) ? mu : 0.0)) * scl;
    }
}

// Block (N_j[a], j) of P = (delta - X_j[a-th rows, j's columns]) / 2 into P's
// values (H's pattern); one 64-lane group per (submatrix, block row a).
__global__ void k_sub_extract(const int64_t *row_ptr, const int32_t *col_idx, const int64_t *blk_off,
                              const int32_t *rbs, const int32_t *ent_row, const int32_t *ent_soff,
                              const int32_t *ent_sub, const int32_t *sub_col,
                              const int32_t *sub_csoff, const int64_t *base, const int32_t *npad,
                              const int32_t *parity, const double *buf0, const double *buf1,
                              double *pvals, int64_t nent) {
    const int64_t e = blockIdx.x;
    if (e >= nent) return;
    const int sub = ent_sub[e];
    const int i = ent_row[e], j = sub_col[sub];
    const int ra = ent_soff[e], cj = sub_csoff[sub];
    const int bi = rbs[i], bj = rbs[j];
    const int ld = npad[sub];
    const double *Xs = (parity[sub] ? buf1 : buf0) + base[sub];
    int64_t lo = row_ptr[i], hi = row_ptr[i + 1];
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col_idx[mid] < j) lo = mid + 1; else hi = mid;
    }
    if (lo >= row_ptr[i + 1] || col_idx[lo] != j) return;   // cannot happen: i is in N_j
    double *dst = pvals + blk_off[lo];
    for (int u = threadIdx.x; u < bi * bj; u += blockDim.x) {
        const int p = u / bj, q = u % bj;
        const double xv = Xs[static_cast<int64_t>(ra + p) * ld + cj + q];
        dst[u] = 0.5 * (((i == j && p == q) ? 1.0 : 0.0) - xv);
    }
}

template <class T>
int upload(T **d, const std::vector<T> &h, hipStream_t s) {
    BSM_TRY(dalloc(d, std::max<size_t>(h.size(), 1), s));
    if (!h.empty())
        BSM_HIP(hipMemcpyAsync(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, s));
    return BSM_OK;
}

size_t batch_bytes_cap() {
    const char *e = std::getenv("BSM_SUB_BATCH_BYTES");
    if (e) {
        const long long v = std::atoll(e);
        if (v > 0) return static_cast<size_t>(v);
    }
    return size_t(48) << 30;
}

}  // namespace

int submatrix_density(Mat &H, double mu, const bsm_sign_opts &o, Mat **p_out, bsm_sub_stats *st,
                      hipStream_t s) {
    *p_out = nullptr;
    if (H.nbrows != H.nbcols || H.h_rbs != H.h_cbs) {
        set_error("submatrix: H must be square with square diagonal blocks");
        return BSM_EINVAL;
    }
    if (!std::isfinite(mu) || !(o.eps_filter >= 0.0) || !std::isfinite(o.eps_filter) ||
        !(o.tol > 0.0) || o.max_iter < 0 || o.max_iter > 120 ||
        (o.norm != BSM_NORM_FROB && o.norm != BSM_NORM_MAXABS)) {
        set_error("submatrix: need a finite mu, eps_filter >= 0, tol > 0, 0 <= max_iter <= 120, "
                  "a known norm");
        return BSM_EINVAL;
    }
    // pattern on the host: the column sets N_j (rows ascending)
    const int nb = H.nbrows;
    std::vector<int64_t> rp(nb + 1);
    std::vector<int32_t> ci(H.nnzb);
    BSM_HIP(hipMemcpyAsync(rp.data(), H.row_ptr, sizeof(int64_t) * (nb + 1), hipMemcpyDeviceToHost, s));
    if (H.nnzb)
        BSM_HIP(hipMemcpyAsync(ci.data(), H.col_idx, sizeof(int32_t) * H.nnzb, hipMemcpyDeviceToHost, s));
    BSM_HIP(hipStreamSynchronize(s));
    std::vector<int64_t> cp(nb + 1, 0);
    for (int64_t t = 0; t < H.nnzb; ++t) cp[ci[t] + 1]++;
    for (int j = 0; j < nb; ++j) cp[j + 1] += cp[j];
    std::vector<int32_t> crow(H.nnzb);
    {
        std::vector<int64_t> fill(cp.begin(), cp.end() - 1);
        for (int i = 0; i < nb; ++i)
            for (int64_t t = rp[i]; t < rp[i + 1]; ++t) crow[fill[ci[t]]++] = i;
    }
    std::vector<int32_t> dim(nb), pad(nb), csoff(nb);
    for (int j = 0; j < nb; ++j) {
        int64_t n = 0;
        int pos = -1;
        for (int64_t u = cp[j]; u < cp[j + 1]; ++u) {
            if (crow[u] == j) { pos = static_cast<int>(u - cp[j]); csoff[j] = static_cast<int32_t>(n); }
            n += H.h_rbs[crow[u]];
        }
        if (pos < 0) {
            set_error("submatrix: block column %d has no stored diagonal block", j);
            return BSM_EINVAL;
        }
        if (n > (1 << 15)) {
            set_error("submatrix: block column %d spans %lld rows (at most 32768)", j,
                      static_cast<long long>(n));
            return BSM_EINVAL;
        }
        dim[j] = static_cast<int32_t>(n);
        pad[j] = static_cast<int32_t>((n + kPad - 1) / kPad * kPad);
    }

    hipEvent_t t0, t1;
    BSM_HIP(hipEventCreate(&t0));
    BSM_HIP(hipEventCreate(&t1));
    BSM_HIP(hipEventRecord(t0, s));
    Mat *P = nullptr;
    int rc = copy_mat(H, &P, s);

    st->n_sub = nb;
    double sum_dim = 0.0;
    for (int j = 0; j < nb; ++j) {
        st->max_dim = std::max(st->max_dim, dim[j]);
        sum_dim += dim[j];
    }
    st->mean_dim = nb ? sum_dim / nb : 0.0;

    // whether H is its own transpose, read back with the first batch's norms:
    // half of every product is then the mirror image of the other
    bool symmetric = false;
    auto gemm = k_sub_gemm<false>;
    const size_t cap = batch_bytes_cap();
    std::vector<std::pair<hipEvent_t, hipEvent_t>> gev;
    double *d_sums = nullptr;        // row sums of |H - mu I| per block
    if (rc == BSM_OK) rc = dalloc(&d_sums, std::max<int64_t>(H.nnzb * H.max_rbs, 1), s);
    if (rc == BSM_OK && nb > 0) {
        hipLaunchKernelGGL(k_sub_block_sums, dim3(std::min(nb, kRowGroups)), dim3(256), 0, s, H.row_ptr,
                           H.col_idx, H.blk_off, H.values, H.rbs, nb, mu, H.max_rbs, d_sums);
        if (hipGetLastError() != hipSuccess) { set_error("submatrix: row sums failed"); rc = BSM_EDEVICE; }
    }
    int64_t n_noconv = 0;            // submatrices left above tol (every batch still runs)
    int j0 = 0;
    while (rc == BSM_OK && j0 < nb) {
        // the batch: consecutive block columns while three padded squares fit
        size_t bytes = 0;
        int j1 = j0;
        while (j1 < nb) {
            const size_t b = size_t(3) * sizeof(double) * size_t(pad[j1]) * size_t(pad[j1]);
            if (j1 > j0 && bytes + b > cap) break;
            bytes += b;
            ++j1;
        }
        const int ns = j1 - j0;
        st->n_batches++;
        std::vector<int64_t> base(ns), ent0(ns + 1, 0);
        std::vector<int32_t> npad(ns), ndim(ns), scol(ns), scs(ns), ent_row, ent_soff, ent_sub;
        int64_t tot = 0;
        for (int q = 0; q < ns; ++q) {
            const int j = j0 + q;
            base[q] = tot;
            tot += int64_t(pad[j]) * pad[j];
            npad[q] = pad[j];
            ndim[q] = dim[j];
            scol[q] = j;
            scs[q] = csoff[j];
            int32_t off = 0;
            for (int64_t u = cp[j]; u < cp[j + 1]; ++u) {
                ent_row.push_back(crow[u]);
                ent_soff.push_back(off);
                ent_sub.push_back(q);
                off += H.h_rbs[crow[u]];
            }
            ent0[q + 1] = static_cast<int64_t>(ent_row.size());
        }
        const int64_t nent = static_cast<int64_t>(ent_row.size());
        int64_t *d_base = nullptr, *d_ent0 = nullptr;
        int32_t *d_npad = nullptr, *d_ndim = nullptr, *d_scol = nullptr, *d_scs = nullptr,
                *d_erow = nullptr, *d_esoff = nullptr, *d_esub = nullptr, *d_par = nullptr;
        double *buf0 = nullptr, *buf1 = nullptr, *ybuf = nullptr, *d_scale = nullptr,
               *d_r = nullptr, *d_part = nullptr;
        int4 *d_tiles = nullptr;
        int32_t *d_act = nullptr, *d_tlo = nullptr, *d_thi = nullptr;
        auto release = [&]() {
            dfree(d_base, s); dfree(d_ent0, s); dfree(d_npad, s); dfree(d_ndim, s);
            dfree(d_scol, s); dfree(d_scs, s); dfree(d_erow, s); dfree(d_esoff, s);
            dfree(d_esub, s); dfree(d_par, s); dfree(buf0, s); dfree(buf1, s); dfree(ybuf, s);
            dfree(d_scale, s); dfree(d_r, s); dfree(d_part, s); dfree(d_tiles, s);
            dfree(d_act, s); dfree(d_tlo, s); dfree(d_thi, s);
        };
        rc = upload(&d_base, base, s);
        if (rc == BSM_OK) rc = upload(&d_ent0, ent0, s);
        if (rc == BSM_OK) rc = upload(&d_npad, npad, s);
        if (rc == BSM_OK) rc = upload(&d_ndim, ndim, s);
        if (rc == BSM_OK) rc = upload(&d_scol, scol, s);
        if (rc == BSM_OK) rc = upload(&d_scs, scs, s);
        if (rc == BSM_OK) rc = upload(&d_erow, ent_row, s);
        if (rc == BSM_OK) rc = upload(&d_esoff, ent_soff, s);
        if (rc == BSM_OK) rc = upload(&d_esub, ent_sub, s);
        if (rc == BSM_OK) rc = dalloc(&buf0, static_cast<size_t>(tot), s);
        if (rc == BSM_OK) rc = dalloc(&buf1, static_cast<size_t>(tot), s);
        if (rc == BSM_OK) rc = dalloc(&ybuf, static_cast<size_t>(tot), s);
        if (rc == BSM_OK) rc = dalloc(&d_scale, static_cast<size_t>(ns) + 1, s);
        if (rc == BSM_OK) rc = dalloc(&d_r, static_cast<size_t>(ns), s);
        if (rc != BSM_OK) { release(); break; }

        // X_0 = (T - mu I) / ||T - mu I||_inf, zero padding
        // (the products write the whole padded squares of the other buffers)
        if (hipMemsetAsync(buf0, 0, sizeof(double) * tot, s) != hipSuccess ||
            hipMemsetAsync(d_scale, 0, sizeof(double) * (ns + 1), s) != hipSuccess) {
            set_error("submatrix: memset failed");
            rc = BSM_EDEVICE;
            release();
            break;
        }
        if (nent > 0)
            hipLaunchKernelGGL(k_sub_norm, dim3(static_cast<unsigned>(nent)), dim3(64), 0, s,
                               H.row_ptr, H.col_idx, H.max_rbs, d_sums, H.rbs, d_erow, d_esub,
                               d_ent0, d_scale, nent);
        if (j0 == 0)                 // into the word behind the norms
            hipLaunchKernelGGL(k_sub_symmetric, dim3(std::min(nb, kRowGroups)), dim3(256), 0, s, H.row_ptr,
                               H.col_idx, H.blk_off, H.values, H.rbs, nb,
                               reinterpret_cast<unsigned long long *>(d_scale + ns));
        std::vector<double> scale(ns + 1);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess)
            e = hipMemcpyAsync(scale.data(), d_scale, sizeof(double) * (ns + 1), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            set_error("submatrix: %s", hipGetErrorString(e));
            rc = BSM_EDEVICE;
            release();
            break;
        }
        if (j0 == 0) {
            unsigned long long mirrored;
            std::memcpy(&mirrored, &scale[ns], sizeof mirrored);
            symmetric = mirrored == static_cast<unsigned long long>(H.nnzb);
            if (symmetric) gemm = k_sub_gemm<true>;
        }
        for (int q = 0; q < ns && rc == BSM_OK; ++q) {
            if (!std::isfinite(scale[q])) {
                set_error("submatrix: H holds NaN or Inf (block column %d)", j0 + q);
                rc = BSM_ENONFINITE;
            } else if (scale[q] == 0.0) {
                set_error("submatrix: T - mu I is zero for block column %d", j0 + q);
                rc = BSM_EINVAL;
            }
        }
        if (rc != BSM_OK) { release(); break; }
        if (nent > 0)
            hipLaunchKernelGGL(k_sub_gather, dim3(static_cast<unsigned>(nent)), dim3(64), 0, s,
                               H.row_ptr, H.col_idx, H.blk_off, H.values, H.rbs, d_erow, d_esoff,
                               d_esub, d_ent0, d_base, d_npad, d_scale, mu, buf0, nent);

        // Newton-Schulz on every submatrix of the batch
        std::vector<int32_t> parity(ns, 0), active;
        for (int q = 0; q < ns; ++q) active.push_back(q);
        std::vector<int> iters(ns, 0);
        std::vector<double> rfin(ns, 0.0);
        size_t tiles_cap = 0;
        for (int32_t k = 0; rc == BSM_OK && !active.empty(); ++k) {
            std::vector<int4> tiles;
            std::vector<int32_t> tlo, thi;
            for (int q : active) {
                const int nt = (npad[q] + kTile - 1) / kTile;
                tlo.push_back(static_cast<int32_t>(tiles.size()));
                for (int a = 0; a < nt; ++a)
                    for (int b = symmetric ? a : 0; b < nt; ++b) tiles.push_back(make_int4(q, a, b, parity[q]));
                thi.push_back(static_cast<int32_t>(tiles.size()));
            }
            if (tiles.size() > static_cast<size_t>(INT32_MAX / 2)) {
                set_error("submatrix: too many tiles in one batch");
                rc = BSM_EINVAL;
                break;
            }
            if (tiles.size() > tiles_cap) {
                dfree(d_tiles, s); dfree(d_part, s);
                d_tiles = nullptr; d_part = nullptr;
                tiles_cap = tiles.size();
                rc = dalloc(&d_tiles, tiles_cap, s);
                if (rc == BSM_OK) rc = dalloc(&d_part, tiles_cap, s);
                if (rc != BSM_OK) break;
            }
            dfree(d_act, s); dfree(d_tlo, s); dfree(d_thi, s);
            d_act = d_tlo = d_thi = nullptr;
            rc = upload(&d_act, active, s);
            if (rc == BSM_OK) rc = upload(&d_tlo, tlo, s);
            if (rc == BSM_OK) rc = upload(&d_thi, thi, s);
            if (rc != BSM_OK) break;
            if (hipMemcpyAsync(d_tiles, tiles.data(), sizeof(int4) * tiles.size(),
                               hipMemcpyHostToDevice, s) != hipSuccess) {
                set_error("submatrix: tile upload failed");
                rc = BSM_EDEVICE;
                break;
            }
            SubGemm g{d_tiles, static_cast<int32_t>(tiles.size()), d_base, d_npad, d_ndim,
                      buf0, buf1, ybuf, 0, d_part};
            const unsigned grid = static_cast<unsigned>((tiles.size() + kXcds - 1) / kXcds * kXcds);
            hipEvent_t e0, e1;
            (void)hipEventCreate(&e0);
            (void)hipEventCreate(&e1);
            (void)hipEventRecord(e0, s);
            hipLaunchKernelGGL(gemm, dim3(grid), dim3(256), 0, s, g);       // Y = X X
            (void)hipEventRecord(e1, s);
            gev.emplace_back(e0, e1);
            for (int q : active) st->flops += 2.0 * double(ndim[q]) * ndim[q] * ndim[q];
            const int nact = static_cast<int>(active.size());
            hipLaunchKernelGGL(k_sub_resid, dim3(grid_for(nact, 128)), dim3(128), 0, s, d_part,
                               d_act, d_tlo, d_thi, d_ndim, d_r, nact);
            std::vector<double> r(nact);
            if (hipMemcpyAsync(r.data(), d_r, sizeof(double) * nact, hipMemcpyDeviceToHost, s) !=
                    hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                set_error("submatrix: %s", hipGetErrorString(hipGetLastError()));
                rc = BSM_EDEVICE;
                break;
            }
            std::vector<int32_t> next;
            for (int a = 0; a < nact; ++a) {
                const int q = active[a];
                rfin[q] = r[a];
                iters[q] = k;
                if (!std::isfinite(r[a])) {
                    set_error("submatrix: residual not finite (block column %d)", j0 + q);
                    rc = BSM_ENONFINITE;
                } else if (!(r[a] < o.tol)) {
                    next.push_back(q);
                }
            }
            if (rc != BSM_OK) break;
            if (next.empty()) { active.clear(); break; }
            if (k >= o.max_iter) {
                n_noconv += static_cast<int64_t>(next.size());   // keep their last iterates
                break;
            }
            // X' = 1.5 X - 0.5 X Y for those not yet converged (their tiles
            // only; the list is rebuilt in the order of `next`)
            if (next.size() != active.size()) {
                tiles.clear();
                for (int q : next) {
                    const int nt = (npad[q] + kTile - 1) / kTile;
                    for (int a = 0; a < nt; ++a)
                        for (int b = symmetric ? a : 0; b < nt; ++b) tiles.push_back(make_int4(q, a, b, parity[q]));
                }
                if (hipMemcpyAsync(d_tiles, tiles.data(), sizeof(int4) * tiles.size(),
                                   hipMemcpyHostToDevice, s) != hipSuccess) {
                    set_error("submatrix: tile upload failed");
                    rc = BSM_EDEVICE;
                    break;
                }
            }
            g.ntiles = static_cast<int32_t>(tiles.size());
            g.mode = 1;
            const unsigned grid2 = static_cast<unsigned>((tiles.size() + kXcds - 1) / kXcds * kXcds);
            hipEvent_t f0, f1;
            (void)hipEventCreate(&f0);
            (void)hipEventCreate(&f1);
            (void)hipEventRecord(f0, s);
            hipLaunchKernelGGL(gemm, dim3(grid2), dim3(256), 0, s, g);
            (void)hipEventRecord(f1, s);
            gev.emplace_back(f0, f1);
            for (int q : next) {
                st->flops += 2.0 * double(ndim[q]) * ndim[q] * ndim[q];
                parity[q] ^= 1;
            }
            active.swap(next);
        }
        if (rc == BSM_OK) {
            for (int q = 0; q < ns; ++q) {
                st->max_iterations = std::max(st->max_iterations, iters[q]);
                st->r_max = std::max(st->r_max, rfin[q]);
            }
            int r2 = upload(&d_par, parity, s);
            if (r2 == BSM_OK && nent > 0)
                hipLaunchKernelGGL(k_sub_extract, dim3(static_cast<unsigned>(nent)), dim3(64), 0, s,
                                   P->row_ptr, P->col_idx, P->blk_off, P->rbs, d_erow, d_esoff,
                                   d_esub, d_scol, d_scs, d_base, d_npad, d_par, buf0, buf1,
                                   P->values, nent);
            if (r2 != BSM_OK) rc = r2;
        }
        release();
        if (rc != BSM_OK) break;
        j0 = j1;
    }
    dfree(d_sums, s);
    if (rc == BSM_OK) {
        const int r2 = filter_inplace(*P, o.eps_filter, o.norm, s);
        if (r2 != BSM_OK) rc = r2;
    }
    if (rc == BSM_OK && n_noconv > 0) {
        set_error("submatrix: %lld submatrices above tol after max_iter",
                  static_cast<long long>(n_noconv));
        rc = BSM_ENOCONV;
    }
    (void)hipEventRecord(t1, s);
    (void)hipEventSynchronize(t1);
    float ms = 0.f;
    for (auto &p : gev) {
        if (hipEventElapsedTime(&ms, p.first, p.second) == hipSuccess) st->gemm_ms += ms;
        (void)hipEventDestroy(p.first);
        (void)hipEventDestroy(p.second);
    }
    if (hipEventElapsedTime(&ms, t0, t1) == hipSuccess) st->device_ms = ms;
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    if (rc == BSM_OK || rc == BSM_ENOCONV) {
        st->nnzb = P->nnzb;
        *p_out = P;
    } else {
        free_mat(P, s);
    }
    return rc;
}

}  // namespace bsm
