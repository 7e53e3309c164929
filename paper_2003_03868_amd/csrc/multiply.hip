// C = alpha*A*B + beta*C with the norm filter: the device pipeline.
//
//   1. count     per C block row: C blocks, C scalars, products, flops
//   2. scans     row pointers of C and of the product list (device), then one
//                wait to learn the sizes
//   3. pattern   C col_idx / owning row / matching C_in block
//   4. offsets   C block value offsets (device scan)
//   5. per chunk of block rows (bounded product count, like the paper's
//                bounded batches): product stacks (for the quad kernel merged
//                per 2 x 2 group of C blocks, quad.hip), then the block products
//   6. filter    drop blocks failing the norm test and compact (device)
//
// C's old arrays stay alive until everything that reads them is queued, so C
// may be the same handle as A or B.
//
// With a plan requested, the symbolic results (stacks per chunk, sorted work
// lists, the launches, the filter's keep-set and compaction maps) are kept in
// plan-owned memory for numeric-only repetitions (plan.hip).
#include <algorithm>
#include <climits>
#include <cstring>
#include <vector>

#include "plan.h"
#include "symbolic.h"

namespace bsm {

// Products per chunk: bounds the stack memory (8 bytes per product; about
// 6 for the quads' entry lists), 4 GiB at the default 2^29, which keeps the
// launches few and large (on the sign workload 2^29 ran 4% faster per step
// than 2^27; 2^30 no faster).  BSM_CHUNK_PRODUCTS overrides it (tests use a
// small value to force chunks).
static int64_t chunk_products() {
    const char *e = getenv("BSM_CHUNK_PRODUCTS");
    const long long x = e ? atoll(e) : 0;
    return x > 0 ? static_cast<int64_t>(x) : (int64_t{1} << 29);
}

// Block-product kernel variant; BSM_SMM_VARIANT overrides the default
// (tests and the tuner compare variants).
int smm_variant() {
    const char *e = getenv("BSM_SMM_VARIANT");
    return e ? atoi(e) : kSmmF64Quad;
}

// Work order of the quads: bands of QR row pairs by QC column pairs
// (BSM_QUAD_TILE_ROWS / BSM_QUAD_TILE_COLS; rows 0 keeps row-pair order).
static int quad_tile(const char *name, int dflt) {
    const char *e = getenv(name);
    return e ? atoi(e) : dflt;
}

// Fewest products per C block for the FP64 group kernels where nothing else
// is known of the size (BSM_QUAD_MIN_REUSE overrides it).
static double quad_min_reuse() {
    const char *e = getenv("BSM_QUAD_MIN_REUSE");
    return e ? atof(e) : 8.0;
}

// The same for a size m with a one-block kernel of its own (below).
static double fp64_least_reuse(int m) { return m == 23 ? 12.5 : (m == 13 || m == 32) ? 20.0 : 64.0; }

// FP64 groups for a size m with a one-block kernel of its own, `reuse`
// products per C block, unless BSM_SMM_VARIANT names a kernel or screening
// needs the groups.  Their lists cost a symbolic pass and two host waits
// (0.1 ms, more with many block rows), and what a group saves is operand
// traffic, which small blocks and few products have little of.  Whole
// multiplies, groups and one block per wave, ms, at reuse: size 5 (6 alike)
// 18 4.3 and 3.7, 47 5.6 and 5.3, 92 9.6 and 10.0; 13 15 6.2 and 6.0, 19 4.9 and
// 4.6, 25 6.3 and 6.9, 92 22 and 30; 23 9 3.3 and 2.8, 11 9.0 and 8.6, 15 14.9
// and 15.4, 18 21.7 and 24.0; 26 18 43.5 and 39.4, 47 66.4 and 65.0, 92 126 and
// 133; 32 18 74.0 and 73.4, 25 56.4 and 56.8, 92 242 and 250.  Few products
// (7e5, reuse 18): 13 0.59 and 0.43, 23 0.96 and 0.74.  A sign iteration with
// device-sized graphs (`iter`) has its multiplies from the graphs where they run
// in groups, and keeps to them.
// All of those are neighbour lists along a Morton curve, about 5 products per 4 x 4
// entry and more (`share`).  Where neighbouring rows and columns have little in
// common, a group stages an operand for one or two products; one block and
// groups then, ms: 23 share 1.1 69 and 113, 1.4 100 and 125, 1.9 48 and 48, 2.2
// 613 and 500; 13 1.4 32 and 52, 2.0 15.7 and 19.3, 2.2 207 and 202; 5 2.2 56 and
// 106, 4.6 25.6 and 27.8, 7.7 55 and 48; 26 2.2 854 and 1259, 4.6 386 and 395, 7.7
// 790 and 685; 32 1.9 120 and 129, 4.6 658 and 668, 7.7 1402 and 1339.
static bool fp64_groups(int m, double reuse, double share, int64_t nprod, bool iter) {
    if (iter || getenv("BSM_QUAD_MIN_REUSE")) return reuse >= quad_min_reuse();
    return reuse >= fp64_least_reuse(m) && nprod >= 1000000 && share >= (m == 23 || m == 13 ? 2.1 : 5.0);
}

// Mixed sizes: 4 x 4 groups of consecutive block rows and columns.  Whole
// multiplies with the one-block kernels and with groups, ms:
//   any sizes ({4, 9, 13, 18, 22, 31}; the persistent kernel): 5e2 products
//     0.23 and 0.28, 2e3 0.30 and 0.31, 2e4 0.55 and 0.46, 1.7e5 1.32 and
//     0.67; 14.7 products per C block 18.5 and 7.9, 126 250 and 69.  The persistent
//     kernel takes 12 ns per C block (its counter) or 1.9 per product, whichever
//     is more, groups 16 ns each and 1.45 per entry ({1, 2, 3, 4}: 1.1 per product
//     and 0.4 per entry).  With few products per entry, groups are many: a
//     million C blocks of one product each, all in groups of their own, 13.2 and
//     17.8; 1.3e6 products, 1.05 C blocks per group, 4.2 and 7.7; 4.2e6 products,
//     3.6 C blocks per group, 45 and 24;
//   {5, 13, 23, 26} (a launch per (m, n) class): 8.6e6 products, 15 per C block 5.9
//     and 7.2; 4.8e7, 47 28.1 and 27.9; 2.7e8, 257 162 and 129, with 4.6 products
//     per entry instead of 8.7 165 and 156, of 6.8e7 with 1.1 44 and 112.  Below
//     50000 products per class the launches count, 0.4 ms against 0.25 for four
//     sizes: 6e4 products 0.51 and 0.37, 2.3e5 0.67 and 0.54; with as many groups
//     as C blocks, 6.5e4 0.50 and 0.93, 1.5e5 0.76 and 1.08; only 5 and 13 6e4 0.27
//     and 0.32.
// groups: at most so many; v: mean m n k of a product; classes: pairs of sizes.
static bool mixed_groups(bool basis, double reuse, double share, double nprod, double n_c, double groups,
                         double v, int classes) {
    const double entries = nprod / share;
    if (basis)
        return (reuse >= 64.0 && share >= 4.5) ||
               (nprod <= 50000.0 * classes && 16.0 * groups + (0.35 + v / 4500.0) * entries <
                                                  12000.0 * (classes - 4) + (0.1 + v / 5000.0) * nprod);
    return nprod >= 4000.0 && 16.0 * groups + (0.4 + v / 4000.0) * entries <
                                  std::max(12.0 * n_c, (1.1 + v / 5000.0) * nprod);
}

// Groups of C blocks for reduced-precision products (uniform block size m,
// `reuse` products per C block): BSM_LOWP_QUAD = 1 always, 0 never; by
// default where they measured faster than one C block per wave.  Building the
// groups costs a small multiply 0.1 ms, and FP32 products are so short of
// other work that they gain only where operands are shared by many products.
// Whole multiplies, one-block kernel and groups, ms:
//   three parts  172e3 products (100 block rows) size 5 0.37 and 0.41, 13 0.38
//     and 0.42, 23 0.49 and 0.48, 32 0.65 and 0.50; 743e3 (256) 5 0.65 and 0.58,
//     23 1.13 and 0.83; 2048 block rows, reuse 9.4, 23 7.1 and 5.1; 18 30 and 20;
//   two parts    172e3 5 0.35 and 0.41, 23 0.40 and 0.44, 32 0.47 and 0.42; 743e3
//     5 0.51 and 0.51, 23 0.75 and 0.72; reuse 9.4, 5 2.2 and 2.0, 23 4.2 and 4.1;
//   FP32         743e3 5 0.43 and 0.52, 23 0.87 and 1.03, 32 1.29 and 1.20; reuse
//     9.4, 5 1.45 and 1.81, 13 1.88 and 2.03; 18, 5 5.7 and 4.4, 13 7.6 and 6.1,
//     23 21.3 and 23.3, 26 25.0 and 26.6; 47, 23 31.1 and 29.8, 26 36.3 and 33.6.
// With few products per entry (`share`; FP64 above), groups / one block:
//   three parts  1.1 1.6 .. 2.3, 1.3 0.99 .. 1.28, 1.4 0.96 .. 1.09, 1.9 0.77 .. 0.95
//     (32 the last of each), 4.6 0.47 .. 0.68;
//   two parts    1.1 1.4 .. 2.4, 1.4 1.0 .. 1.6, 1.9 0.68 (32), 0.97 .. 1.19, 2.6 0.76
//     (32), 1.06 (26), 4.6 0.42 .. 0.68;
//   FP32         1.1 1.7 .. 2.5, 1.9 1.11 (32), 1.2 .. 1.6, 2.6 1.02 (32), 3.4 0.90
//     (32), 1.23 (26), 4.6 0.71 (32, 13), 1.0 .. 1.06 (26, 23), 6.4 0.67 .. 0.97.
// Small blocks with few products per C block gain from the groups' shorter
// stacks all the same where the groups are full (`full`; 2.3 products per C
// block, share 1.1: three parts 5 0.54, 13 0.73, two parts 0.82, 0.98).
static double fp32_least_reuse(int m) { return m == 32 ? 0.0 : m <= 13 ? 14.0 : 32.0; }
static bool lowp_groups(int prec, int m, double reuse, double share, bool full, int64_t nprod) {
    const char *e = getenv("BSM_LOWP_QUAD");
    if (e) return atoi(e) != 0;
    const bool many = nprod >= 400000;
    if (prec == BSM_FP32)
        return many && reuse >= fp32_least_reuse(m) &&
               share >= (m == 32 ? 2.6 : m <= 13 ? 4.0 : 6.0);
    if (!many && static_cast<double>(nprod) * m < 4e6) return false;
    if (m <= 13 && reuse < 4.0 && full) return true;
    return share >= (prec == BSM_SPLIT_BF16X3 ? (m == 32 ? 1.7 : 1.4) : (m == 32 ? 1.8 : 2.6));
}

// k segments of the group lists' symbolic walk (one workgroup per row group
// and segment; the walk over the merged A rows is serial, so it is nseg times
// shorter).  One per 4 block columns of A, at most 16, above 1024 block
// columns at most 8.  Whole multiplies of size 23, 1 / 4 / 8 / 16 / 32
// segments: 64 block rows 0.55 / 0.45 / 0.43 / 0.41 / 0.41 ms; 300: 2.71 /
// 2.23 / 2.12 / 2.06 / 2.14; 800 (11% filled): 6.35 / 6.03 / 5.91 / 5.98 /
// 6.06; 2048 (4.5%): 15.16 / 15.18 / 14.98 / 15.09 / 15.51 (every segment
// marks the row group's columns again).  BSM_QUAD_KSEG overrides it.
int32_t quad_ksegments(int32_t nbk) {
    const char *e = getenv("BSM_QUAD_KSEG");
    int32_t v = e ? atoi(e) : std::min(nbk / 4, nbk > 1024 ? 8 : 16);
    if (v > 64) v = 64;
    return v < 1 ? 1 : v;
}

// Kernel family for a chunk with mixed block sizes (uniform sizes keep the
// requested variant).  Default: one launch per (m, n) class when every size
// is in {5, 13, 23, 26} (measured fastest on the 4096-site mixed workload:
// 7.1 s per sign step, against 8.8 s for the paired-group kernel of
// kSmmF64MQuad, whose one persistent launch per multiply shares operands but
// waits at a barrier per entry for products that are small on average),
// else the run-time-shape persistent kernel.
static int mixed_variant(const SmmArgs &a, int requested) {
    const bool uniform = a.uni_m && a.uni_n && a.uni_k;
    if (uniform) return requested;
    if ((requested == kSmmF64Class || requested == kSmmF64MQuad) && !a.fused_ok) return kSmmF64Fused;
    if (requested == kSmmF64Fixed || requested == kSmmF64Quad)
        return a.fused_ok ? kSmmF64Class : kSmmF64Fused;
    return requested;
}

namespace {
struct Events {
    bool on = false;
    hipEvent_t t0{}, t1{};
    std::vector<std::pair<hipEvent_t, hipEvent_t>> smm;
    std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> cls;   // per-class launches
    ~Events() {
        if (!on) return;
        (void)hipEventDestroy(t0);
        (void)hipEventDestroy(t1);
        for (auto &p : smm) { (void)hipEventDestroy(p.first); (void)hipEventDestroy(p.second); }
        for (auto &p : cls) { (void)hipEventDestroy(p.second.first); (void)hipEventDestroy(p.second.second); }
    }
};
struct Scratch {
    hipStream_t s;
    std::vector<void *> ptrs;
    explicit Scratch(hipStream_t st) : s(st) {}
    template <class T>
    int get(T **p, size_t n) {
        int st = dalloc(p, n, s);
        if (st == BSM_OK) ptrs.push_back(*p);
        return st;
    }
    ~Scratch() { for (void *p : ptrs) dfree(p, s); }
};
}  // namespace

static int check_shapes(const Mat &A, const Mat &B, const Mat &C) {
    if (A.nbcols != B.nbrows || C.nbrows != A.nbrows || C.nbcols != B.nbcols) {
        set_error("block grids do not match: A %dx%d, B %dx%d, C %dx%d", A.nbrows, A.nbcols,
                  B.nbrows, B.nbcols, C.nbrows, C.nbcols);
        return BSM_EINVAL;
    }
    if (A.h_cbs != B.h_rbs) { set_error("A column block sizes differ from B row block sizes"); return BSM_EINVAL; }
    if (C.h_rbs != A.h_rbs || C.h_cbs != B.h_cbs) {
        set_error("C block sizes must be A's row sizes by B's column sizes");
        return BSM_EINVAL;
    }
    if (B.nbcols > kMaxBlockCols) {
        set_error("at most %d block columns are supported (got %d)", kMaxBlockCols, B.nbcols);
        return BSM_EINVAL;
    }
    if (A.nnzb >= (int64_t{1} << 31) || B.nnzb >= (int64_t{1} << 31)) {
        set_error("operands with 2^31 or more stored blocks are not supported");
        return BSM_EINVAL;
    }
    return BSM_OK;
}

// Most bytes that one list of the group kernels or one operand's image may
// take (BSM_GROUP_BYTES; no bound by default).
static size_t group_bytes_cap() {
    const char *e = getenv("BSM_GROUP_BYTES");
    return e ? static_cast<size_t>(strtoull(e, nullptr, 10)) : SIZE_MAX;
}

// `groups`: in, whether a rule may choose groups of C blocks; out, whether one did.
static int multiply_once(double alpha, Mat &A, Mat &B, double beta, Mat &C, double eps, int norm, int prec,
                         bsm_mult_stats *stats, hipStream_t s, MulPlan **plan, double tau, MulSizes *sizes,
                         bool *groups_io) {
    BSM_TRY(check_shapes(A, B, C));
    if (!(tau >= 0.0) || !std::isfinite(tau)) { set_error("eps_screen must be finite and >= 0"); return BSM_EINVAL; }
    if (tau > 0.0 && (prec != BSM_FP64 || plan)) {
        set_error("product screening needs FP64 products and no retained plan");
        return BSM_EINVAL;
    }
    if (!(eps >= 0.0) || !std::isfinite(eps)) { set_error("eps_filter must be finite and >= 0"); return BSM_EINVAL; }
    if (norm != BSM_NORM_FROB && norm != BSM_NORM_MAXABS) { set_error("unknown norm %d", norm); return BSM_EINVAL; }
    if (prec != BSM_FP64 && prec != BSM_FP32 && prec != BSM_SPLIT_BF16 && prec != BSM_SPLIT_BF16X3) {
        set_error("unknown precision %d", prec);
        return BSM_EINVAL;
    }
    if (!std::isfinite(alpha) || !std::isfinite(beta)) { set_error("alpha and beta must be finite"); return BSM_EINVAL; }

    const int32_t nbr = A.nbrows;
    const bool use_c = (beta != 0.0) && C.nnzb > 0;
    const int64_t cin_nnzb = C.nnzb;
    Events ev;
    if (stats) {
        ev.on = true;
        BSM_HIP(hipEventCreate(&ev.t0));
        BSM_HIP(hipEventCreate(&ev.t1));
        BSM_HIP(hipEventRecord(ev.t0, s));
    }
    Scratch tmp(s);
    MulPlan *pl = plan ? new MulPlan : nullptr;
    if (pl) pl->s = s;
    // buffers the plan keeps (plan mode) or that die with this call
    auto keep_buf = [&](auto **ptr, size_t n) -> int {
        if (!pl) return tmp.get(ptr, n);
        const int r = dalloc(ptr, n, s);
        if (r == BSM_OK) pl->owned.push_back(*ptr);
        return r;
    };
    struct PlanGuard {
        MulPlan *&p;
        ~PlanGuard() { free_plan(p); }
    } plan_guard{pl};

    SymArgs sa{};
    sa.nbrows = nbr; sa.nbcols = B.nbcols;
    sa.a_row_ptr = A.row_ptr; sa.a_col_idx = A.col_idx;
    sa.b_row_ptr = B.row_ptr; sa.b_col_idx = B.col_idx;
    sa.k_size = A.cbs; sa.c_rbs = A.rbs; sa.c_cbs = B.cbs;
    sa.use_c = use_c ? 1 : 0;
    sa.c_in_row_ptr = use_c ? C.row_ptr : nullptr;
    sa.c_in_col_idx = use_c ? C.col_idx : nullptr;

    // 1-2. counts and scans
    // The sums that the host reads sit in one buffer: a copy to pageable
    // memory waits for the stream each time (four copies took 30 us of the
    // 240 us of an 832 x 832 multiply, two 15).
    int64_t *c_row_ptr = nullptr, *sums = nullptr;
    BSM_TRY(dalloc(&c_row_ptr, nbr + 1, s));      // becomes the new C's row_ptr
    const int64_t ns = nbr + 1;
    const int parts = count_entries_parts(A);
    int st = tmp.get(&sums, 3 * ns + parts);
    int64_t *c_nval = sums, *p_row_ptr = sums + ns, *d_entries = sums + 3 * ns;
    double *flops_row = reinterpret_cast<double *>(sums + 2 * ns);
    if (st == BSM_OK) st = sym_count(sa, c_row_ptr, c_nval, p_row_ptr, flops_row, s);
    if (st == BSM_OK) st = scan_i64(c_row_ptr, c_row_ptr, nbr, s);
    if (st == BSM_OK) st = scan_i64(c_nval, c_nval, nbr, s);
    if (st == BSM_OK) st = scan_i64(p_row_ptr, p_row_ptr, nbr, s);
    // the entries that 4 x 4 groups would have, where a rule below looks at them:
    // counted along with the rest (8 us, 30 on a whole multiply) where as many
    // products are to be expected; by themselves for sizes that seldom have
    // enough of them per C block, and for mixed sizes that need them to decide
    const int variant = smm_variant();
    const bool mixed_sizes = !(A.uni_r && A.uni_c && B.uni_c);
    const bool square = A.uni_r && A.uni_r == A.uni_c && A.uni_r == B.uni_c;
    const bool may_group = variant == kSmmF64Quad && tau == 0.0 && square && !getenv("BSM_SMM_VARIANT") &&
                           !getenv("BSM_QUAD_MIN_REUSE") &&
                           (prec == BSM_FP64 ? smm_tile_available(A.uni_r)
                                             : smm_lowp_available(A.uni_r, A.uni_r, A.uni_r));
    const bool own = prec == BSM_FP64 && square && smm_quad_available(A.uni_r, A.uni_r, A.uni_r);
    const double least_reuse = own ? fp64_least_reuse(A.uni_r) : prec == BSM_FP32 ? fp32_least_reuse(A.uni_r) : 0.0;
    const double least_products =                               // below, no rule looks at them
        own ? 1e6 : prec == BSM_FP32 ? 4e5 : std::min(4e5, 4e6 / std::max(1, A.uni_r));
    int32_t *b_groups = nullptr;
    auto count = [&]() -> int {
        BSM_TRY(tmp.get(&b_groups, std::max(1, B.nbrows)));
        return count_entries(A, B, b_groups, d_entries, s);
    };
    if (st == BSM_OK && may_group &&
        (sizes || (least_reuse <= 20.0 &&
                   static_cast<double>(A.nnzb) * static_cast<double>(B.nnzb) >= 0.5 * least_products * A.nbcols)))
        st = count();
    std::vector<int64_t> h_crp(ns), h_sums(3 * ns + parts);
    if (st == BSM_OK) {
        hipError_t e = hipMemcpyAsync(h_crp.data(), c_row_ptr, sizeof(int64_t) * ns, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(h_sums.data(), sums, sizeof(int64_t) * (3 * ns + (b_groups ? parts : 0)), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { set_error("multiply: reading sizes failed: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    auto sum_entries_of = [&]() {
        int64_t n = 0;
        for (int p = 0; b_groups && p < parts; ++p) n += h_sums[3 * ns + p];
        return n;
    };
    auto count_now = [&]() -> int {
        BSM_TRY(count());
        BSM_HIP(hipMemcpyAsync(&h_sums[3 * ns], d_entries, sizeof(int64_t) * parts, hipMemcpyDeviceToHost, s));
        BSM_HIP(hipStreamSynchronize(s));
        return BSM_OK;
    };
    if (st == BSM_OK && may_group && !b_groups && static_cast<double>(h_sums[2 * ns - 1]) >= least_products &&
        static_cast<double>(h_sums[2 * ns - 1]) >= least_reuse * static_cast<double>(h_crp[nbr]))
        st = count_now();
    if (st != BSM_OK) { dfree(c_row_ptr, s); return st; }
    const int64_t nnzb_c = h_crp[nbr];
    const int64_t *h_prp = h_sums.data() + ns;
    const int64_t nprod = h_prp[nbr], nval_c = h_sums[nbr];
    double flops = 0.0;
    for (int32_t i = 0; i < nbr; ++i) {
        double f;
        std::memcpy(&f, &h_sums[2 * ns + i], sizeof f);
        flops += f;
    }

    // 3-4. pattern and value offsets of the new C
    Mat nc;
    nc.nbrows = nbr; nc.nbcols = B.nbcols; nc.rbs = A.rbs; nc.cbs = B.cbs;
    nc.row_ptr = c_row_ptr;
    nc.nnzb = nnzb_c;
    nc.nvalues = nval_c;
    int32_t *c_row = nullptr;
    int64_t *cin_map = nullptr;
    double *sq = nullptr, *mx = nullptr;
    int *flags = nullptr;
    st = dalloc(&nc.col_idx, nnzb_c, s);
    if (st == BSM_OK) st = dalloc(&nc.values, nval_c, s);
    if (st == BSM_OK) st = keep_buf(&c_row, nnzb_c);
    if (st == BSM_OK && use_c) st = keep_buf(&cin_map, nnzb_c);
    if (st == BSM_OK) st = keep_buf(&sq, nnzb_c);
    if (st == BSM_OK) st = keep_buf(&mx, nnzb_c);
    if (st == BSM_OK) st = tmp.get(&flags, 1);
    if (st == BSM_OK) {
        hipError_t e = hipMemsetAsync(flags, 0, sizeof(int), s);
        if (e != hipSuccess) { set_error("memset: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    if (st == BSM_OK) st = sym_pattern(sa, c_row_ptr, nc.col_idx, c_row, cin_map, s);
    if (st == BSM_OK) st = compute_blk_off(nc, s);

    // 5. tiled work order, then chunks of whole row bands with a bounded
    //    number of products
    const int rb = tile_rows();
    int64_t *worklist = nullptr, *worklist2 = nullptr;
    if (st == BSM_OK) st = keep_buf(&worklist, nnzb_c);
    if (st == BSM_OK) st = keep_buf(&worklist2, nnzb_c);  // target of the work-list sorts
    if (st == BSM_OK) st = tile_order(c_row_ptr, nc.col_idx, nbr, B.nbcols, rb, worklist, s);
    // mixed sizes in {5, 13, 23, 26}: groups over paired rows and columns
    // (FP64, no screening), unless another kernel variant is asked for
    bool mixed_ok = true;
    for (const auto *v : {&A.h_rbs, &A.h_cbs, &B.h_cbs})
        for (int32_t b : *v)
            if (b != 5 && b != 13 && b != 23 && b != 26) mixed_ok = false;
    const bool use_mquad = prec == BSM_FP64 && tau == 0.0 && mixed_sizes && mixed_ok &&
                           variant == kSmmF64MQuad;
    std::vector<int32_t> cuts{0};
    {
        // whole row bands; a step that is a multiple of 4 keeps the row
        // groups of the group kernel (2 or 4 rows) in one chunk, one of
        // kPairBand the paired rows of the mixed-size groups
        const int64_t lim = chunk_products();
        const int step = use_mquad ? (rb + kPairBand - 1) / kPairBand * kPairBand : (rb + 3) / 4 * 4;
        int32_t r0 = 0;
        while (r0 < nbr) {
            int32_t r1 = std::min(nbr, r0 + step);
            while (r1 < nbr && h_prp[std::min(nbr, r1 + step)] - h_prp[r0] <= lim)
                r1 = std::min(nbr, r1 + step);
            cuts.push_back(r1);
            r0 = r1;
        }
    }
    int64_t max_p = 0, max_c = 0;
    for (size_t q = 0; q + 1 < cuts.size(); ++q) {
        max_p = std::max(max_p, h_prp[cuts[q + 1]] - h_prp[cuts[q]]);
        max_c = std::max(max_c, h_crp[cuts[q + 1]] - h_crp[cuts[q]]);
    }
    // the quad kernel serves uniform sizes with a compile-time shape unless
    // the tuning table picks another kernel family for them
    const double reuse = nnzb_c ? static_cast<double>(nprod) / static_cast<double>(nnzb_c) : 0.0;
    // products per entry of 4 x 4 groups (unknown: large), and a bound of the groups
    const int64_t entries = sum_entries_of();
    const double share = entries > 0 ? static_cast<double>(nprod) / static_cast<double>(entries) : 1e300;
    auto most_groups = [&]() {
        const int64_t ncg = (B.nbcols + 3) / 4;
        int64_t n = 0;
        for (int32_t i = 0; i < nbr; i += 4) n += std::min(ncg, h_crp[std::min(nbr, i + 4)] - h_crp[i]);
        return n;
    };
    bool use_quad = false;
    if (prec == BSM_FP64 && variant == kSmmF64Quad && A.uni_r && A.uni_c && B.uni_c &&
        smm_quad_available(A.uni_r, B.uni_c, A.uni_c)) {
        SmmParams tp;
        use_quad = !(table_lookup(A.uni_r, B.uni_c, A.uni_c, &tp) && tp.family != 3);
        if (use_quad && tau == 0.0 && !getenv("BSM_SMM_VARIANT"))
            use_quad = fp64_groups(A.uni_r, reuse, share, nprod, sizes != nullptr);
    }
    // the other uniform sizes: 4 x 4 groups instead of the run-time-shape
    // kernel where the table has no choice for the size, C blocks and entries
    // (`share`) have enough products, and the time saved exceeds the 0.1 ms that
    // building the groups adds to a small multiply.  Products per C block, products, whole multiply
    // with the run-time-shape kernel and with groups: size 9 11.6, 1.9e5, 0.30
    // and 0.34 ms; 14.7, 2.1e6, 9.5 and 5.7; 172, 1.8e8, 90 and 29; size 17
    // 11.6, 1.9e5, 0.43 and 0.40; 172, 1.8e8, 196 and 83; size 31 11.6, 1.9e5,
    // 0.93 and 0.75; 172, 1.8e8, 617 and 251; size 4 11.6, 1.9e5, 0.25 and 0.30;
    // 172, 1.8e8, 40 and 13.  At share 1.1 the run-time-shape kernel and groups
    // take 15.8 and 29.6 ms (size 4), 35 and 44 (9), 73 and 90 (17), 86 and 113 (22),
    // 234 and 362 (31); 1.3 2.3 and 3.5 (4), 4.8 and 4.6 (9), 10.1 and 9.4 (17), 11.4
    // and 12.7 (22); 1.55 5.4 and 6.3 (4), 27.5 and 25.2 (22), 74 and 76 (31); 1.9 11.1
    // and 10.7 (4), 60 and 48 (22), 166 and 142 (31).
    if (prec == BSM_FP64 && variant == kSmmF64Quad && tau == 0.0 && A.uni_r && A.uni_r == A.uni_c &&
        A.uni_r == B.uni_c && !smm_quad_available(A.uni_r, A.uni_r, A.uni_r) && smm_tile_available(A.uni_r)) {
        SmmParams tp;
        use_quad = !table_lookup(A.uni_r, A.uni_r, A.uni_r, &tp) && reuse >= quad_min_reuse() &&
                   static_cast<double>(nprod) * A.uni_r >= 5e5 * quad_min_reuse() &&
                   share >= (A.uni_r < 9 ? 2.0 : A.uni_r <= 20 ? 1.25 : A.uni_r <= 24 ? 1.4 : 1.65);
    }
    // mixed sizes: classes that the table has a kernel for keep their launches
    bool use_mtile = false;
    if (prec == BSM_FP64 && tau == 0.0 && variant == kSmmF64Quad && mixed_sizes && nprod > 0) {
        auto distinct = [](const std::vector<int32_t> &v) {
            uint32_t m = 0;
            for (int32_t b : v) m |= 1u << b;
            return __builtin_popcount(m);
        };
        // as if entries and groups were as few as they can be, as many, as they are
        const double n_c = static_cast<double>(nnzb_c), p = static_cast<double>(nprod);
        auto pays = [&](double sh, double groups) {
            return mixed_groups(mixed_ok, reuse, sh, p, n_c, groups, 0.5 * flops / p,
                                mixed_ok ? distinct(A.h_rbs) * distinct(B.h_cbs) : 0);
        };
        const int64_t most = most_groups();
        use_mtile = pays(16.0, n_c / 16.0);
        if (use_mtile && !pays(1.0, static_cast<double>(most)) && st == BSM_OK) {
            st = count_now();
            const int64_t e = sum_entries_of();
            if (e > 0) use_mtile = pays(p / static_cast<double>(e), static_cast<double>(use_c ? most : std::min(most, e)));
        }
        if (const char *e = getenv("BSM_MIXED_TILE")) use_mtile = atoi(e) != 0;
        for (int b = 0; mixed_ok && b < 16; ++b) {
            static const int sz[4] = {5, 13, 23, 26};
            SmmParams tp;
            if (table_lookup(sz[b / 4], sz[b % 4], 0, &tp) && tp.family != 2) use_mtile = false;
        }
        use_quad = use_mtile;
    }
    // reduced precision: 4 x 4 groups where they pay, unless another kernel
    // variant is asked for
    bool lowp_tile = false;
    if (prec != BSM_FP64 && variant == kSmmF64Quad && A.uni_r && A.uni_c && B.uni_c &&
        smm_lowp_available(A.uni_r, B.uni_c, A.uni_c))
        use_quad = lowp_tile = lowp_groups(prec, A.uni_r, reuse, share,
                                           nnzb_c >= 8 * std::min(most_groups(), use_c || !entries ? INT64_MAX : entries),
                                           nprod);
    if (!*groups_io) use_quad = use_mtile = lowp_tile = false;
    *groups_io = use_quad;
    // group shape: quads, or other shapes on request (FP64 only); screening
    // runs through the quads' product masks
    int GR = 2, GC = 2;
    if (use_mtile || lowp_tile) GR = GC = 4;
    else if (use_quad && prec == BSM_FP64 && tau == 0.0) quad_shape(A.uni_r, reuse, share, &GR, &GC);
    if (st == BSM_OK && tau > 0.0 && !use_quad) {
        set_error("product screening needs uniform block sizes 5, 6, 13, 23, 26 or 32 and the "
                  "default kernel variant");
        st = BSM_EINVAL;
    }
    // squared block norms of the operands, and the count of kept products
    double *a_sq = nullptr, *b_sq = nullptr;
    unsigned long long *kept = nullptr;
    if (st == BSM_OK && tau > 0.0) {
        st = tmp.get(&a_sq, A.nnzb);
        if (st == BSM_OK) st = block_sqnorms(A, a_sq, s);
        if (st == BSM_OK && &A != &B) st = tmp.get(&b_sq, B.nnzb);
        if (st == BSM_OK && &A != &B) st = block_sqnorms(B, b_sq, s);
        if (&A == &B) b_sq = a_sq;
        if (st == BSM_OK) st = tmp.get(&kept, 1);
        if (st == BSM_OK) {
            hipError_t e = hipMemsetAsync(kept, 0, sizeof(unsigned long long), s);
            if (e != hipSuccess) { set_error("memset: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
        }
    }
    const int NE = (GR + GC + 3) / 4;                        // int4 per group entry

    // pair maps of the mixed-size groups (host-built, copied to the device)
    MixedPairs mp;
    int32_t *d_rg = nullptr, *d_cgrp = nullptr, *d_cslot = nullptr, *d_cmap = nullptr;
    unsigned long long *mq_counter = nullptr;
    if (st == BSM_OK && use_mquad) {
        mixed_pairs(A.h_rbs, B.h_cbs, &mp);
        st = keep_buf(&d_rg, mp.rg.size());
        if (st == BSM_OK) st = keep_buf(&d_cgrp, mp.cgrp.size());
        if (st == BSM_OK) st = keep_buf(&d_cslot, mp.cslot.size());
        if (st == BSM_OK) st = keep_buf(&d_cmap, mp.cmap.size());
        if (st == BSM_OK) st = keep_buf(&mq_counter, 1);
        hipError_t e = hipSuccess;
        auto up = [&](int32_t *d, const std::vector<int32_t> &h) {
            if (e == hipSuccess && !h.empty())
                e = hipMemcpyAsync(d, h.data(), sizeof(int32_t) * h.size(), hipMemcpyHostToDevice, s);
        };
        if (st == BSM_OK) { up(d_rg, mp.rg); up(d_cgrp, mp.cgrp); up(d_cslot, mp.cslot); up(d_cmap, mp.cmap); }
        if (e != hipSuccess) { set_error("pair maps: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }

    // one set of stack buffers reused by every chunk; a plan keeps one per
    // chunk; the group kernels build their own lists
    int64_t *seg = nullptr;
    int32_t *stk_a = nullptr, *stk_b = nullptr;
    const bool groups = use_quad || use_mquad;
    if (st == BSM_OK && !pl && !groups) st = tmp.get(&seg, max_c + 1);
    if (st == BSM_OK && !pl && !groups) st = tmp.get(&stk_a, max_p);
    if (st == BSM_OK && !pl && !groups) st = tmp.get(&stk_b, max_p);

    SmmArgs ma{};
    ma.c_row = c_row; ma.c_col = nc.col_idx; ma.c_blk_off = nc.blk_off; ma.c_vals = nc.values;
    ma.c_rbs = A.rbs; ma.c_cbs = B.cbs;
    ma.a_col_idx = A.col_idx; ma.a_blk_off = A.blk_off; ma.a_vals = A.values; ma.k_size = A.cbs;
    ma.b_blk_off = B.blk_off; ma.b_vals = B.values;
    ma.cin_map = cin_map;
    ma.cin_blk_off = use_c ? C.blk_off : nullptr;
    ma.cin_vals = use_c ? C.values : nullptr;
    ma.alpha = alpha; ma.beta = beta;
    ma.sq_out = sq; ma.mx_out = mx; ma.flags = flags;
    ma.max_m = A.max_rbs; ma.max_n = B.max_cbs; ma.max_k = A.max_cbs;
    ma.nbr = nbr; ma.nbc = B.nbcols;
    ma.uni_m = A.uni_r; ma.uni_n = B.uni_c; ma.uni_k = A.uni_c;
    {
        auto in_set = [](const std::vector<int32_t> &v) {
            for (int32_t b : v)
                if (b != 5 && b != 13 && b != 23 && b != 26) return false;
            return true;
        };
        ma.fused_ok = (in_set(A.h_rbs) && in_set(A.h_cbs) && in_set(B.h_cbs)) ? 1 : 0;
    }
    ma.prec = prec;
    ma.seg = seg; ma.stk_a = stk_a; ma.stk_b = stk_b;
    ma.worklist = worklist;
    if (st == BSM_OK) st = keep_buf(&ma.counter, 1);         // persistent kernels' counter

    if (st == BSM_OK && prec != BSM_FP64) {
        if (!(A.uni_r && A.uni_c && B.uni_c && smm_lowp_available(A.uni_r, B.uni_c, A.uni_c))) {
            set_error("reduced-precision products need uniform block sizes 5, 13, 23, 26 or 32");
            st = BSM_EINVAL;
        }
        uint32_t *apk = nullptr, *bpk = nullptr;
        const int size = lowp_tile ? A.uni_r : 0;
        auto words = [&](const Mat &m) {
            return size ? lowp_image_words(m.nnzb, size, prec) : lowp_words(m.nvalues, prec);
        };
        if (size && sizeof(uint32_t) * std::max(words(A), words(B)) > group_bytes_cap()) {
            set_error("operand images above BSM_GROUP_BYTES");
            st = BSM_ENOMEM;
        }
        if (st == BSM_OK) st = keep_buf(&apk, words(A));
        if (st == BSM_OK) st = pack_operand(A, size, prec, false, apk, s);
        if (&A != &B || size) {
            if (st == BSM_OK) st = keep_buf(&bpk, words(B));
            if (st == BSM_OK) st = pack_operand(B, size, prec, true, bpk, s);
        } else {
            bpk = apk;
        }
        ma.a_pk = apk;
        ma.b_pk = bpk;
        ma.a_pk_n = A.nvalues;
        ma.b_pk_n = B.nvalues;
        if (pl) { pl->apk = apk; pl->bpk = bpk; pl->image_size = size; }
    }

    int32_t n_launch = 0;
    int64_t sum_groups = 0, sum_entries = 0;
    auto launch = [&](const MulOp &op) -> int {
        ++n_launch;
        const int r = run_op(op, s);
        if (r == BSM_OK && pl) pl->ops.push_back(op);
        return r;
    };

    for (size_t q = 0; st == BSM_OK && q + 1 < cuts.size(); ++q) {
        const int32_t r0 = cuts[q], r1 = cuts[q + 1];
        ma.c0 = h_crp[r0];
        ma.nC = h_crp[r1] - h_crp[r0];
        if (ma.nC == 0) continue;
        if (groups) {
            // groups of this chunk's C blocks and their merged entry lists;
            // without a plan the buffers live for this chunk only
            Scratch ctmp(s);
            auto qbuf = [&](auto **ptr, size_t n) -> int {
                if (n * sizeof(**ptr) > group_bytes_cap()) { set_error("group lists above BSM_GROUP_BYTES"); return BSM_ENOMEM; }
                return pl ? keep_buf(ptr, n) : ctmp.get(ptr, n);
            };
            int32_t g0 = 0;
            int64_t npairs = (static_cast<int64_t>(r1 - r0) + GR - 1) / GR;
            if (use_mquad) {
                g0 = mp.band_g0[r0 / kPairBand];
                npairs = mp.band_g0[(r1 + kPairBand - 1) / kPairBand] - g0;
            }
            int64_t *q_off = nullptr, *q_cblk = nullptr, *e_off = nullptr, *q_order = nullptr,
                    *e_seg = nullptr;
            int32_t *pm = nullptr;
            int32_t *q_col = nullptr;
            int4 *ent = nullptr;
            int64_t nq = 0, ne = 0;
            auto read_total = [&](const int64_t *d, int64_t *h) -> int {
                hipError_t e = hipMemcpyAsync(h, d, sizeof(int64_t), hipMemcpyDeviceToHost, s);
                if (e == hipSuccess) e = hipStreamSynchronize(s);
                if (e != hipSuccess) { set_error("quads: %s", hipGetErrorString(e)); return BSM_EDEVICE; }
                return BSM_OK;
            };
            QuadSymArgs qa{};
            qa.r0 = r0; qa.r1 = r1; qa.nbcols = B.nbcols; qa.gr = GR; qa.gc = GC;
            // one workgroup per row group and segment, fewer than 2^32 threads
            qa.nseg = static_cast<int32_t>(std::min<int64_t>(
                quad_ksegments(A.nbcols), std::max<int64_t>(1, kQuadListGroups / std::max<int64_t>(1, npairs))));
            qa.kseg = (A.nbcols + qa.nseg - 1) / qa.nseg;
            if (qa.kseg < 1) qa.kseg = 1;
            qa.a_row_ptr = A.row_ptr; qa.a_col_idx = A.col_idx;
            qa.b_row_ptr = B.row_ptr; qa.b_col_idx = B.col_idx;
            qa.c_row_ptr = c_row_ptr; qa.c_col_idx = nc.col_idx;
            qa.a_sq = a_sq; qa.b_sq = b_sq; qa.tau2 = tau * tau; qa.kept = kept;
            if (use_mquad) {
                qa.map = 1;
                qa.g0 = g0;
                qa.ngroups = npairs;
                qa.ncg = static_cast<int32_t>(mp.cmap.size() / 2);
                qa.rg = d_rg; qa.cgrp = d_cgrp; qa.cslot = d_cslot; qa.cmap = d_cmap;
            }
            st = qbuf(&q_off, npairs + 1);
            if (st == BSM_OK) st = quad_pairs(qa, q_off, s);
            if (st == BSM_OK) st = scan_i64(q_off, q_off, npairs, s);
            if (st == BSM_OK) st = read_total(q_off + npairs, &nq);
            if (st == BSM_OK) st = qbuf(&q_cblk, static_cast<size_t>(GR) * GC * nq);
            if (st == BSM_OK) st = qbuf(&e_off, nq + 1);
            if (st == BSM_OK && qa.nseg > 1) st = qbuf(&e_seg, static_cast<size_t>(nq) * qa.nseg + 1);
            if (qa.nseg == 1) e_seg = e_off;
            if (st == BSM_OK) st = qbuf(&q_col, nq);
            qa.q_off = q_off;
            qa.q_cblk = q_cblk;
            qa.q_col = q_col;
            qa.e_off = e_seg;
            if (st == BSM_OK) st = quad_stack(qa, false, s);
            const int qr = quad_tile("BSM_QUAD_TILE_ROWS", 0), qc = quad_tile("BSM_QUAD_TILE_COLS", 16);
            if (st == BSM_OK && qr > 0 && nq > 0 && !use_mquad) {
                st = qbuf(&q_order, nq);
                if (st == BSM_OK)
                    st = tile_order(q_off, q_col, static_cast<int32_t>(npairs), (B.nbcols + GC - 1) / GC,
                                    qr, q_order, s, qc);
            }
            const int64_t nsl = nq * qa.nseg;                       // (group, segment) counts
            if (st == BSM_OK) st = scan_i64(e_seg, e_seg, nsl, s);
            if (st == BSM_OK && qa.nseg > 1) st = quad_seg_starts(e_seg, qa.nseg, nq, e_off, s);
            if (st == BSM_OK) st = read_total(e_seg + nsl, &ne);
            if (st == BSM_OK && ne > INT32_MAX) {
                // the fill pass keeps entry offsets inside a row group as int32
                set_error("more than 2^31 group entries in one chunk; lower BSM_CHUNK_PRODUCTS");
                st = BSM_EINVAL;
            }
            sum_groups += nq;
            sum_entries += ne;
            if (st == BSM_OK) st = qbuf(&ent, static_cast<size_t>(ne) * NE);
            if (st == BSM_OK && tau > 0.0) st = qbuf(&pm, ne);
            qa.ent = ent;
            qa.pm = pm;
            if (st == BSM_OK) st = quad_stack(qa, true, s);
            if (st != BSM_OK) break;
            MulOp op;
            op.a = ma;
            op.kind = use_mquad ? kOpMQuad : kOpQuad;
            op.a.counter = use_mquad ? mq_counter : ma.counter;
            op.a.n_quads = nq;
            op.a.q_cblk = q_cblk;
            op.a.q_seg = e_off;
            op.a.q_ent = ent;
            if (st == BSM_OK && use_mquad && nq > 0) {
                int8_t *rank = nullptr;
                st = ctmp.get(&rank, nq);
                if (st == BSM_OK) st = qbuf(&q_order, nq);
                if (st == BSM_OK) st = mquad_order(op.a, rank, q_order, s);
                if (st != BSM_OK) break;
            }
            op.a.q_order = q_order;
            op.a.q_gr = GR;
            op.a.q_gc = GC;
            op.a.q_pm = pm;
            std::pair<hipEvent_t, hipEvent_t> pe{};
            if (ev.on) {
                BSM_HIP(hipEventCreate(&pe.first));
                BSM_HIP(hipEventCreate(&pe.second));
                BSM_HIP(hipEventRecord(pe.first, s));
            }
            st = launch(op);
            if (ev.on) {
                BSM_HIP(hipEventRecord(pe.second, s));
                ev.smm.push_back(pe);
            }
            continue;
        }
        if (pl) {
            const int64_t np = h_prp[r1] - h_prp[r0];
            st = keep_buf(&seg, ma.nC + 1);
            if (st == BSM_OK) st = keep_buf(&stk_a, np);
            if (st == BSM_OK) st = keep_buf(&stk_b, np);
            if (st != BSM_OK) break;
            ma.seg = seg; ma.stk_a = stk_a; ma.stk_b = stk_b;
        }
        st = sym_stack(sa, r0, r1, c_row_ptr, p_row_ptr, seg, stk_a, stk_b, s);
        if (st != BSM_OK) break;

        // mixed sizes: cost-sorted list for the fused persistent launch, or
        // class-sorted list for one launch per (m, n) class
        const int var = (prec == BSM_FP64) ? mixed_variant(ma, variant) : -1;
        int64_t hist[64] = {0};
        if (var == kSmmF64Fused || var == kSmmF64Class) {
            if (worklist2 == nullptr) { set_error("internal: no sort buffer"); st = BSM_EDEVICE; break; }
            st = sort_worklist(worklist, worklist2, ma.c0, ma.nC,
                               var == kSmmF64Fused ? kKeyCost : kKeyClass, c_row, nc.col_idx,
                               A.rbs, B.cbs, seg, var == kSmmF64Class ? hist : nullptr, s);
            if (st != BSM_OK) break;
            ma.worklist = worklist2;
        } else {
            ma.worklist = worklist;
        }
        std::pair<hipEvent_t, hipEvent_t> pe{};
        if (ev.on) {
            BSM_HIP(hipEventCreate(&pe.first));
            BSM_HIP(hipEventCreate(&pe.second));
            BSM_HIP(hipEventRecord(pe.first, s));
        }
        MulOp op;
        op.a = ma;
        if (prec != BSM_FP64) {
            op.kind = kOpLowp;
            st = launch(op);
        } else if (var == kSmmF64Class) {
            int64_t off = 0;
            for (int b = 0; b < 17 && st == BSM_OK; ++b) {
                if (hist[b] == 0) continue;
                op.a.worklist = worklist2 + off;
                op.a.nC = hist[b];
                // per class: the (m, n)-specialised kernel unless the tuning
                // table holds run-time-kernel parameters for (m, n, any k)
                static const int sz[4] = {5, 13, 23, 26};
                SmmParams prm;
                if (b < 16 && !(table_lookup(sz[b / 4], sz[b % 4], 0, &prm) && prm.family != 2)) {
                    op.kind = kOpClass;
                    op.id = b;
                } else if (b < 16) {
                    op.kind = kOpRt;
                    op.prm = prm;
                } else {
                    op.kind = kOpVariant;
                    op.id = kSmmF64Tuned;
                }
                std::pair<hipEvent_t, hipEvent_t> ce{};
                if (ev.on && b < 16) {
                    BSM_HIP(hipEventCreate(&ce.first));
                    BSM_HIP(hipEventCreate(&ce.second));
                    BSM_HIP(hipEventRecord(ce.first, s));
                }
                st = launch(op);
                if (ev.on && b < 16) {
                    BSM_HIP(hipEventRecord(ce.second, s));
                    ev.cls.push_back({b, ce});
                }
                off += hist[b];
            }
        } else {
            op.kind = kOpVariant;
            op.id = var;
            st = launch(op);
        }
        if (ev.on) {
            BSM_HIP(hipEventRecord(pe.second, s));
            ev.smm.push_back(pe);
        }
    }

    // 6. filter
    int64_t nnzb_after = nnzb_c;
    CompactKeep ck;
    if (st == BSM_OK && eps > 0.0)
        st = compact_by_norm(nc, sq, mx, eps, norm, s, &nnzb_after, pl ? &ck : nullptr);
    if (pl) {
        // the plan owns the keep maps and the unfiltered layout
        for (void *q : {static_cast<void *>(ck.kidx), static_cast<void *>(ck.koff),
                        static_cast<void *>(ck.row_ptr), static_cast<void *>(ck.col_idx),
                        static_cast<void *>(ck.blk_off), static_cast<void *>(ck.values)})
            if (q) pl->owned.push_back(q);
        if (st == BSM_OK) {
            pl->compacted = ck.compacted;
            if (ck.compacted) {
                pl->c_row_ptr_u = ck.row_ptr;
                pl->c_col_u = ck.col_idx;
                pl->c_blk_off_u = ck.blk_off;
                pl->c_vals_u = ck.values;
            } else {
                st = keep_buf(&pl->c_col_u, nnzb_c);
                if (st == BSM_OK) st = keep_buf(&pl->c_blk_off_u, nnzb_c + 1);
                if (st == BSM_OK) st = keep_buf(&pl->c_row_ptr_u, nbr + 1);
                hipError_t e = hipSuccess;
                if (st == BSM_OK)
                    e = hipMemcpyAsync(pl->c_row_ptr_u, nc.row_ptr, sizeof(int64_t) * (nbr + 1),
                                       hipMemcpyDeviceToDevice, s);
                if (st == BSM_OK && e == hipSuccess && nnzb_c)
                    e = hipMemcpyAsync(pl->c_col_u, nc.col_idx, sizeof(int32_t) * nnzb_c,
                                       hipMemcpyDeviceToDevice, s);
                if (st == BSM_OK && e == hipSuccess)
                    e = hipMemcpyAsync(pl->c_blk_off_u, nc.blk_off, sizeof(int64_t) * (nnzb_c + 1),
                                       hipMemcpyDeviceToDevice, s);
                if (e != hipSuccess) { set_error("plan copy: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
            }
            for (MulOp &o : pl->ops) { o.a.c_col = pl->c_col_u; o.a.c_blk_off = pl->c_blk_off_u; }
        }
    }
    int h_flags = 0;
    if (st == BSM_OK) {
        hipError_t e = hipMemcpyAsync(&h_flags, flags, sizeof(int), hipMemcpyDeviceToHost, s);
        if (ev.on && e == hipSuccess) e = hipEventRecord(ev.t1, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { set_error("multiply: %s", hipGetErrorString(e)); st = BSM_EDEVICE; }
    }
    if (st != BSM_OK) {
        dfree(nc.row_ptr, s); dfree(nc.col_idx, s); dfree(nc.blk_off, s); dfree(nc.values, s);
        return st;
    }

    // swap the new arrays into C (old ones are freed in stream order)
    free_mat_arrays(C, s);
    C.row_ptr = nc.row_ptr; C.col_idx = nc.col_idx; C.blk_off = nc.blk_off; C.values = nc.values;
    C.nnzb = nc.nnzb; C.nvalues = nc.nvalues;
    C.stream = s;

    if (sizes) {
        sizes->nnzb_u = nnzb_c;
        sizes->nnzb = nnzb_after;
        sizes->nval_u = nval_c;
        sizes->nval = nc.nvalues;
        sizes->n_products = nprod;
        sizes->share = share;
        sizes->n_groups = sum_groups;
        sizes->n_entries = sum_entries;
        sizes->gr = GR;
        sizes->groups = (use_quad && prec == BSM_FP64) || use_mquad;
    }
    if (stats) {
        stats->n_products = nprod;
        stats->flops = flops;
        stats->nnzb_unfiltered = nnzb_c;
        stats->nnzb = nnzb_after;
        stats->smm_launches = n_launch;
        if (tau > 0.0 && kept) {
            unsigned long long h_kept = 0;
            if (hipMemcpyAsync(&h_kept, kept, sizeof(h_kept), hipMemcpyDeviceToHost, s) == hipSuccess &&
                hipStreamSynchronize(s) == hipSuccess)
                stats->n_screened = nprod - static_cast<int64_t>(h_kept);
            // uniform blocks: every product costs the same, so the flops
            // actually done scale with the kept count
            if (nprod > 0) stats->flops = flops * static_cast<double>(h_kept) / static_cast<double>(nprod);
        }
        float ms = 0.f;
        double smm = 0.0;
        for (auto &p : ev.smm) {
            if (hipEventElapsedTime(&ms, p.first, p.second) == hipSuccess) smm += ms;
        }
        stats->smm_ms = smm;
        stats->total_ms = (hipEventElapsedTime(&ms, ev.t0, ev.t1) == hipSuccess) ? ms : 0.0;
        for (int b = 0; b < 16; ++b) stats->class_ms[b] = 0.0;
        for (auto &p : ev.cls)
            if (hipEventElapsedTime(&ms, p.second.first, p.second.second) == hipSuccess)
                stats->class_ms[p.first] += ms;
    }
    if (pl) {
        pl->alpha = alpha; pl->beta = beta; pl->eps = eps; pl->norm = norm; pl->prec = prec;
        pl->use_c = use_c;
        pl->same_ab = (&A == &B);
        pl->a_nnzb = A.nnzb; pl->b_nnzb = B.nnzb; pl->a_nval = A.nvalues; pl->b_nval = B.nvalues;
        pl->cin_nnzb = use_c ? cin_nnzb : 0;
        pl->nnzb_u = nnzb_c; pl->nval_u = nval_c;
        pl->nnzb = nc.nnzb; pl->nval = nc.nvalues;
        pl->flops = flops; pl->nprod = nprod;
        pl->sq = sq; pl->mx = mx;
        pl->kidx = ck.kidx; pl->koff = ck.koff;
    }
    if (h_flags & kFlagNonFinite) {
        set_error("a product block holds NaN or Inf");
        return BSM_ENONFINITE;
    }
    if (pl) { *plan = pl; pl = nullptr; }
    return BSM_OK;
}

// The lists of groups take up to four times the memory of the stacks (32 bytes
// an entry, 8 a product), and images of both operands more than one packed
// copy: where they do not fit, the multiply is done over again, one C block per
// wave (C is only replaced at its end).  Screening has its products in groups
// only.
int multiply(double alpha, Mat &A, Mat &B, double beta, Mat &C, double eps, int norm, int prec,
             bsm_mult_stats *stats, hipStream_t s, MulPlan **plan, double tau, MulSizes *sizes) {
    bool groups = true;
    int st = multiply_once(alpha, A, B, beta, C, eps, norm, prec, stats, s, plan, tau, sizes, &groups);
    if (st == BSM_ENOMEM && groups && tau == 0.0) {
        clear_error();
        groups = false;
        st = multiply_once(alpha, A, B, beta, C, eps, norm, prec, stats, s, plan, tau, sizes, &groups);
    }
    return st;
}

}  // namespace bsm
