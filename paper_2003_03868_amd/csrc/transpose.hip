// Block-sparse transpose B = A^T (section "DBCSR library": transpose is one
// of the operations the library provides besides multiply, sum and trace).
// Block (i, j) of A, an m x n row-major block, becomes block (j, i) of B,
// its n x m transpose; B's block rows have A's column sizes and vice versa.
//
// Pattern: blocks are counted per column of A, the counts scanned into B's
// row pointers, and every block placed into its row of B through an atomic
// cursor; each row of B is then put into the order of its columns (A's rows)
// by counting, which makes the result independent of the order the atomics
// ran in.  Values: one wave per block of B turns the block through LDS.
#include <algorithm>

#include "bsm_internal.h"

namespace bsm {

namespace {

__global__ void k_t_count(const int64_t *row_ptr, const int32_t *col_idx, int32_t nbrows,
                          unsigned long long *cnt, int32_t *rows) {
    const int32_t i = blockIdx.x;
    if (i >= nbrows) return;
    for (int64_t t = row_ptr[i] + threadIdx.x; t < row_ptr[i + 1]; t += blockDim.x) {
        rows[t] = i;
        atomicAdd(&cnt[col_idx[t]], 1ull);
    }
}

__global__ void k_t_place(const int32_t *col_idx, const int32_t *rows, int64_t nnzb,
                          const int64_t *rp_out, unsigned long long *cursor, int32_t *key,
                          int64_t *src) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (t >= nnzb) return;
    const int32_t j = col_idx[t];
    const int64_t p = rp_out[j] + static_cast<int64_t>(atomicAdd(&cursor[j], 1ull));
    key[p] = rows[t];
    src[p] = t;
}

// Each row of B in the order of its columns (A's rows, unique within the
// row): a block's place is the number of smaller keys in its row.  One thread
// per block, whatever the rows' lengths are; neighbours read the same keys.
// Bound by the reads, n per block of a row of n blocks.  Whole transposes with
// an insertion sort by one thread per row, with a workgroup per row and with
// this kernel, the next one as it is now (ms): a million rows of 5 blocks of
// 6 x 6 3.4, 5.4, 3.3; 4096 rows of 92 mixed blocks 1.81, 0.61, 0.51, of 1024
// blocks of 6 x 6 23 (with one thread) and 2.3; one row of 100,000 blocks 1650
// (with one workgroup) and 5.5.
constexpr int kSortThreads = 256;
__global__ void __launch_bounds__(kSortThreads)
k_t_sort(const int64_t *rp_out, const int32_t *a_col_idx, const int32_t *key, const int64_t *src,
         int64_t nnzb, int32_t *key_out, int64_t *src_out) {
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kSortThreads + threadIdx.x;
    if (p >= nnzb) return;
    const int64_t t = src[p];
    const int32_t j = a_col_idx[t], k = key[p];
    const int64_t b = rp_out[j], e = rp_out[j + 1];
    int64_t place = b;
#pragma unroll 8
    for (int64_t u = b; u < e; ++u) place += key[u] < k ? 1 : 0;
    key_out[place] = k;
    src_out[place] = t;
}

// One wave per block of B, four per workgroup: the block is read in order into
// LDS and written in the order of its transpose, so that both sides move
// whole lines; stored as it was read, lanes wrote 8 bytes every block row.
// Bound by memory (0.84 GB read and written for 375,000 mixed blocks): 657 us
// with strided writes, 458 us this way.  Rows of n doubles lie n + 1 apart
// for even n, which keeps a column's elements on different banks.  The LDS of
// a launch is what its largest block needs: with room for 32 x 32 always,
// small blocks had half the waves (a million rows of 5 blocks of 6 x 6, whole
// transpose 4.5 ms and 3.2 then, 2.9 with blocks of up to 64 elements stored
// as they were read).
constexpr int kTWaves = 4;
__global__ void __launch_bounds__(64 * kTWaves)
k_t_values(const int64_t *src, const int32_t *key, const int32_t *a_col_idx,
           const int64_t *a_blk_off, const double *a_vals, const int32_t *a_rbs,
           const int32_t *a_cbs, const int64_t *b_blk_off, double *b_vals, int64_t nnzb, int per_wave) {
    extern __shared__ double lds[];                    // per_wave: doubles of the largest block
    const int wv = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int64_t p = static_cast<int64_t>(blockIdx.x) * kTWaves + wv;
    if (p >= nnzb) return;
    double *sm = lds + wv * per_wave;
    const int64_t t = src[p];
    const int m = a_rbs[key[p]], n = a_cbs[a_col_idx[t]];
    const double *in = a_vals + a_blk_off[t];
    double *out = b_vals + b_blk_off[p];
    const int pitch = n | 1;
    // u / d for u < 1024, d <= 32: u (65536 / d rounded up) / 65536 is exact
    const unsigned by_n = (65536u + n - 1) / n, by_m = (65536u + m - 1) / m;
    const int len = m * n;
    if (len <= kWave) {                                // one store of a few lines: no turn needed
        const int r = (lane * by_n) >> 16;
        if (lane < len) out[(lane - r * n) * m + r] = in[lane];
        return;
    }
    for (int u0 = lane; u0 < len; u0 += 8 * kWave) {     // eight loads in flight
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (u0 + q * kWave < len) v[q] = in[u0 + q * kWave];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int u = u0 + q * kWave, r = (u * by_n) >> 16;
            if (u < len) sm[r * pitch + (u - r * n)] = v[q];   // in[r][c]
        }
    }
    __builtin_amdgcn_wave_barrier();                   // one wave: LDS operations are in order
    for (int u = lane; u < len; u += kWave) {
        const int c = (u * by_m) >> 16;
        out[u] = sm[(u - c * m) * pitch + c];          // out[c][r]
    }
}

}  // namespace

int transpose_mat(const Mat &a, Mat **out, hipStream_t s) {
    *out = nullptr;
    if (a.nnzb > INT32_MAX) { set_error("transpose: more than 2^31 blocks"); return BSM_EINVAL; }
    Mat *m = nullptr;
    BSM_TRY(new_mat_sizes(a, true, a, true, &m, s));
    unsigned long long *cnt = nullptr, *cursor = nullptr;
    int32_t *rows = nullptr;
    int st = dalloc(&m->row_ptr, static_cast<size_t>(m->nbrows) + 1, s);
    if (st == BSM_OK) st = dalloc(&m->col_idx, std::max<int64_t>(a.nnzb, 1), s);
    if (st == BSM_OK) st = dalloc(&cnt, static_cast<size_t>(m->nbrows) + 1, s);
    if (st == BSM_OK) st = dalloc(&cursor, static_cast<size_t>(m->nbrows) + 1, s);
    if (st == BSM_OK) st = dalloc(&rows, std::max<int64_t>(a.nnzb, 1), s);
    int64_t *src = nullptr, *placed = nullptr;
    int32_t *key = nullptr;
    if (st == BSM_OK) st = dalloc(&src, std::max<int64_t>(a.nnzb, 1), s);
    if (st == BSM_OK) st = dalloc(&placed, std::max<int64_t>(a.nnzb, 1), s);
    if (st == BSM_OK) st = dalloc(&key, std::max<int64_t>(a.nnzb, 1), s);
    if (st == BSM_OK) {
        hipError_t e = hipMemsetAsync(cnt, 0, sizeof(unsigned long long) * (m->nbrows + 1), s);
        if (e == hipSuccess)
            e = hipMemsetAsync(cursor, 0, sizeof(unsigned long long) * (m->nbrows + 1), s);
        if (e != hipSuccess) { set_error("transpose: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    if (st == BSM_OK && a.nbrows > 0 && a.nnzb > 0)
        k_t_count<<<a.nbrows, 64, 0, s>>>(a.row_ptr, a.col_idx, a.nbrows, cnt, rows);
    // counts are non-negative int64 values: scan them as such
    if (st == BSM_OK) st = scan_i64(reinterpret_cast<const int64_t *>(cnt), m->row_ptr, m->nbrows, s);
    if (st == BSM_OK && a.nnzb > 0) {
        k_t_place<<<grid_for(a.nnzb, 256), 256, 0, s>>>(a.col_idx, rows, a.nnzb, m->row_ptr, cursor,
                                                        key, placed);
        k_t_sort<<<grid_for(a.nnzb, kSortThreads), kSortThreads, 0, s>>>(m->row_ptr, a.col_idx, key, placed,
                                                                        a.nnzb, m->col_idx, src);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) { set_error("transpose: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    if (st == BSM_OK) {
        m->nnzb = a.nnzb;
        st = compute_blk_off(*m, s);
    }
    if (st == BSM_OK) {
        m->nvalues = a.nvalues;
        st = dalloc(&m->values, std::max<int64_t>(a.nvalues, 1), s);
    }
    if (st == BSM_OK && a.nnzb > 0) {
        const int per_wave = a.max_rbs * (a.max_cbs | 1);
        k_t_values<<<grid_for(a.nnzb, kTWaves), 64 * kTWaves, sizeof(double) * kTWaves * per_wave, s>>>(
            src, m->col_idx, a.col_idx, a.blk_off, a.values, a.rbs, a.cbs, m->blk_off, m->values, a.nnzb,
            per_wave);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) { set_error("transpose: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    dfree(cnt, s);
    dfree(cursor, s);
    dfree(rows, s);
    dfree(src, s);
    dfree(placed, s);
    dfree(key, s);
    if (st != BSM_OK) { free_mat(m, s); return st; }
    *out = m;
    return BSM_OK;
}

}  // namespace bsm
