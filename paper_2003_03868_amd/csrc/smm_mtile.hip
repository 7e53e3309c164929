// FP64 block products for mixed block sizes (any size up to 32), one
// workgroup of eight waves per 4 x 4 group of consecutive C block rows and
// columns, two C blocks per wave, with the group's merged product list (built
// in quad.hip as for uniform sizes).  Each C block's products are summed in
// ascending k with V_MFMA_F64_4X4X4_4B_F64, as in the one-block kernels (same
// bits).
//
// The one-block kernels read both operands of every product, 4.5 KB on
// average for sizes {5, 13, 23, 26}, at 4 to 5.4 TB/s; a group of consecutive
// rows and columns, whose neighbours overlap most, reads 1.7 to 2.0 KB per
// product whatever their sizes are.  Operands are copied from memory to LDS
// past the registers, packed one behind the other; a step holds as many
// entries as fit in half the LDS (three of them on average), and the next
// step's blocks land in the other half meanwhile, so that one barrier serves
// a step.  What an entry's operands need (source, size, place) is worked out
// once per chunk of 64 entries, one operand per thread, into a table in LDS.
// The four C blocks of a SIMD's two waves lie in different rows and columns.
// Measured (MI355X, whole multiplies): sizes {4, 9, 13, 18, 22, 31}, 1024
// block rows, 14.7 products per C block 18.5 (persistent one-block kernel)
// and 7.9 ms, 126 products 250 and 69 ms; sizes {5, 13, 23, 26}, 126 products
// 95.7 (one launch per class) and 73.1 ms.  It is bound by the wait for LDS in
// the step of a product (steps of 16 instructions at most between waits, four
// waves per SIMD: two groups share a CU's LDS) and, with few entries per group, by the chain of loads that
// starts a group.  Tried: sixteen waves of one C block, one group per CU and
// twice the stage: 11 .. 8% slower.
#include "lds_dma.h"
#include "smm_group.h"

namespace bsm {

namespace {

typedef __attribute__((address_space(3))) double lds_double;

__device__ inline int64_t lane64(int64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

// What a wave's products of one C block share.
struct RunArgs {
    uint32_t off;      // LDS address of the chunk's first byte in this stage
    uint32_t rb;       // lane's offset in a B block
    int row, x;        // lane's A row in eight, k in a step
    uint32_t bstep;    // bytes of four B rows
};

// The wave's products of a step (set bits of m) for a C block of HR x HC pairs
// of 4 x 4 tiles; ca: A's place in doubles with k in the top seven bits, cb: B's
// place.  A rows and B columns past the block read what follows in LDS, which
// reaches only accumulator elements that are never stored; k's past the block
// are zeroed on both sides.
template <int HR, int HC>
__device__ inline void run(uint64_t m, int ca, int cb, const RunArgs &g, double (&acc)[4][4]) {
    while (m) {
        const int t = __builtin_ctzll(m);
        m &= m - 1;
        const uint32_t wa = __builtin_amdgcn_readlane(ca, t);
        const int k = wa >> 25;
        uint32_t pa = g.off + (wa & 0x1ffffffu) * 8 + (g.row * k + g.x) * 8;
        uint32_t pb = g.off + __builtin_amdgcn_readlane(cb, t) * 8 + g.rb;
        const uint32_t ts = 64 * k;                      // bytes of eight A rows
        const int steps = (k + 3) >> 2;
        const bool ok = 4 * (steps - 1) + g.x < k;       // this lane's k of the last step exists
        double av[2][HR], bv[2][HC];
        auto load = [&](int h) {
#pragma unroll
            for (int q = 0; q < HR; ++q) av[h][q] = *reinterpret_cast<const lds_double *>(static_cast<uintptr_t>(pa + q * ts));
#pragma unroll
            for (int q = 0; q < HC; ++q) bv[h][q] = *reinterpret_cast<const lds_double *>(static_cast<uintptr_t>(pb + q * 32));
            pa += 32;
            pb += g.bstep;
        };
        auto mul = [&](int h) {
#pragma unroll
            for (int q = 0; q < HR; ++q)
#pragma unroll
                for (int u = 0; u < HC; ++u)
                    acc[q][u] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[h][q], bv[h][u], acc[q][u], 0, 0, 0);
        };
        // pairs of steps; an odd count starts with a zero step
        int s = steps & 1;
        if (s) {
#pragma unroll
            for (int q = 0; q < HR; ++q) av[0][q] = 0.0;
#pragma unroll
            for (int q = 0; q < HC; ++q) bv[0][q] = 0.0;
        } else {
            load(0);
        }
        load(1);
        for (s = 2 - s; s < steps; s += 2) {
            mul(0);
            mul(1);
            load(0);
            load(1);
        }
#pragma unroll
        for (int q = 0; q < HR; ++q) av[1][q] = ok ? av[1][q] : 0.0;
#pragma unroll
        for (int q = 0; q < HC; ++q) bv[1][q] = ok ? bv[1][q] : 0.0;
        mul(0);
        mul(1);
    }
}

// run() for an m x n C block.  One test after another, kept apart: merged
// into a switch, each case would copy the accumulators.
__device__ inline void run_any(int m, int n, uint64_t todo, int ca, int cb, const RunArgs &g, double (&acc)[4][4]) {
    int cls = 4 * ((m + 7) >> 3) + ((n + 7) >> 3);
#define BSM_RUN(HR, HC)                                      \
    if (cls == 4 * HR + HC) run<HR, HC>(todo, ca, cb, g, acc);   \
    asm volatile("" : "+s"(cls));
    if (cls < 12) {
        BSM_RUN(1, 1) BSM_RUN(1, 2) BSM_RUN(1, 3) BSM_RUN(1, 4)
        BSM_RUN(2, 1) BSM_RUN(2, 2) BSM_RUN(2, 3)
    }
    asm volatile("" : "+s"(cls));
    if (cls >= 12) {
        BSM_RUN(2, 4) BSM_RUN(3, 1) BSM_RUN(3, 2) BSM_RUN(3, 3) BSM_RUN(3, 4)
        BSM_RUN(4, 1) BSM_RUN(4, 2) BSM_RUN(4, 3) BSM_RUN(4, 4)
    }
#undef BSM_RUN
}

// alpha * sum + beta * C_in of C block c (m x n) and its filter norms.
__device__ inline void store(const SmmArgs &a, int64_t c, int m, int n, int lane, const double (&acc)[4][4]) {
    const int x = lane >> 4, blk = (lane >> 2) & 3, y = lane & 3;
    const int bh = blk >> 1, bw = blk & 1, hc = (n + 7) >> 3;
    if (c < 0) return;
    const int64_t co = a.c_blk_off[c];
    const double *cin = nullptr;
    if (a.cin_map) {
        const int64_t t = a.cin_map[c];
        if (t >= 0) cin = a.cin_vals + a.cin_blk_off[t];
    }
    double sq = 0.0, mx = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = 4 * (2 * t + bh) + x, col = 4 * (bw * hc + u) + y;
            if (u < hc && row < m && col < n) {
                double v = a.alpha * acc[t][u];
                if (cin) v += a.beta * cin[row * n + col];
                a.c_vals[co + row * n + col] = v;
                sq += v * v;
                mx = fmax(mx, fabs(v));
            }
        }
    sq = group_wave_sum(sq);
    mx = group_wave_max(mx);
    if (lane == 0) {
        a.sq_out[c] = sq;
        a.mx_out[c] = mx;
        if (!isfinite(sq)) atomicOr(a.flags, kFlagNonFinite);
    }
}

// CAP: bytes of one stage; an entry that is larger is multiplied alone, in both.
template <int CAP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_smm_f64_mtile(SmmArgs a) {
    constexpr int G = 4, NOP = 2 * G, NE = NOP / 4;
    constexpr int TAIL = 3072;                           // padded reads past the last block
    constexpr int CAP16 = CAP / 16;
    constexpr int kChunk = 64;
    static_assert(CAP % 16 == 0 && 2 * CAP >= NOP * 8208, "two stages hold any entry");
    __shared__ __align__(16) char lds[2 * CAP + TAIL];
    __shared__ int4 table[kChunk * NOP];                 // per operand: source, place, pieces
    __shared__ int tend[kChunk];                         // pieces up to and with the entry
    __shared__ int wsum[8];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) char *)lds));
    const int64_t it = group_item(a);
    if (it < 0) return;
    const int64_t item = a.q_order ? a.q_order[it] : it;
    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
    // the wave's two C blocks: the waves of a SIMD (equal wv % 4) own four of
    // different rows and columns
    const int R0 = wv / 4 * 2, R1 = R0 + 1, C0 = (wv - R0) & 3, C1 = (wv - R1) & 3;
    const int x = lane >> 4, blk = (lane >> 2) & 3, y = lane & 3;
    const int bh = blk >> 1, bw = blk & 1;

    // block sizes of the group's rows (lanes 0 .. 3) and columns (4 .. 7),
    // repeated every eight lanes
    const int64_t cl = lane < G * G ? a.q_cblk[G * G * item + lane] : -1;
    const int64_t cf = lane64(cl, __builtin_ctzll(__ballot(cl >= 0) | 1ull << 63));
    int szl = 0;
    if (cf >= 0) {
        const int z = lane % NOP;
        const int q = z < G ? (a.c_row[cf] & ~(G - 1)) + z : (a.c_col[cf] & ~(G - 1)) + z - G;
        if (z < G) { if (q < a.nbr) szl = a.c_rbs[q]; }
        else if (q < a.nbc) szl = a.c_cbs[q];
    }
    const int m0 = __builtin_amdgcn_readlane(szl, R0), n0 = __builtin_amdgcn_readlane(szl, G + C0);
    const int m1 = __builtin_amdgcn_readlane(szl, R1), n1 = __builtin_amdgcn_readlane(szl, G + C1);
    RunArgs g0, g1;
    g0.row = g1.row = 4 * bh + y;                        // A(4 (2 t + bh) + y, 4 s + x)
    g0.x = g1.x = x;
    g0.rb = (x * n0 + 4 * bw * ((n0 + 7) >> 3) + y) * 8; // B(4 s + x, 4 (bw hc + u) + y)
    g1.rb = (x * n1 + 4 * bw * ((n1 + 7) >> 3) + y) * 8;
    g0.bstep = 32 * n0;
    g1.bstep = 32 * n1;

    double acc0[4][4], acc1[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc0[t][u] = acc1[t][u] = 0.0;

    const int64_t e0 = a.q_seg[item];
    const int ne = __builtin_amdgcn_readfirstlane(static_cast<int>(a.q_seg[item + 1] - e0));
    const int *ent = reinterpret_cast<const int *>(a.q_ent + NE * e0);
    auto lanes_below = [](int l) { return l >= 64 ? ~0ull : (1ull << l) - 1ull; };
    for (int base = 0; base < ne; base += kChunk) {
        const int cn = ne - base < kChunk ? ne - base : kChunk;
        // the chunk's operands, one per thread: source, size, place
        int pos = 0, end = 0;
        int4 rec = make_int4(0, 0, 0, 0);
        const int e = threadIdx.x / NOP, z = threadIdx.x % NOP;
        const int id = e < cn ? ent[NOP * (base + e) + z] : -1;
        int k = id >= 0 && z < G ? a.k_size[a.a_col_idx[id]] : 0;
        const int64_t off = id >= 0 ? (z < G ? a.a_blk_off : a.b_blk_off)[id] : 0;
        for (int o = 1; o < NOP; o <<= 1) k = max(k, __shfl_xor(k, o, kWave));
        const int odd = static_cast<int>(off) & 1;
        const int elems = szl * k;
        const int cnt = id >= 0 ? (elems + 2) >> 1 : 0;
        end = cnt;
        for (int o = 1; o < kWave; o <<= 1) {
            const int v = __shfl_up(end, o, kWave);
            if (lane >= o) end += v;
        }
        pos = end - cnt;
        if (lane == kWave - 1) wsum[wv] = end;
        const uint64_t src = reinterpret_cast<uint64_t>(z < G ? a.a_vals : a.b_vals) +
                             static_cast<uint64_t>(off - odd) * 8;
        rec.x = static_cast<int>(src);
        rec.y = static_cast<int>(src >> 32);
        rec.w = id >= 0 ? ((odd + elems + 1) >> 1) | odd << 16 | k << 20 : 0;
        __syncthreads();
        for (int w = 0; w < 8; ++w) {
            const int v = wsum[w];
            if (w < wv) { pos += v; end += v; }
        }
        rec.z = pos;
        table[threadIdx.x] = rec;
        if (threadIdx.x % NOP == NOP - 1) tend[threadIdx.x / NOP] = end;
        __syncthreads();
        // entry base + lane: this wave's operands (place in doubles, k above),
        // the entries with a product of this wave, those with an operand it stages
        auto operands = [&](int r, int c, int &oa, int &ob) {
            const int2 ra = *reinterpret_cast<const int2 *>(&table[lane * NOP + r].z);
            const int2 rb = *reinterpret_cast<const int2 *>(&table[lane * NOP + G + c].z);
            oa = (2 * ra.x + ((ra.y >> 16) & 1)) | (ra.y >> 20) << 25;
            ob = 2 * rb.x + ((rb.y >> 16) & 1);
            return __ballot(ra.y != 0 && rb.y != 0);
        };
        int oa0, ob0, oa1, ob1;
        const uint64_t have0 = operands(R0, C0, oa0, ob0), have1 = operands(R1, C1, oa1, ob1);
        const uint64_t mine = __ballot(table[lane * NOP + wv].w != 0);
        const int cend = tend[lane];

        int s0 = 0, s1 = 0, sb = 0;                      // lanes [s0, s1) of a step, pieces before it
        bool big = false;                                // an entry that needs both stages
        auto next_step = [&]() {
            sb = s1 ? __builtin_amdgcn_readlane(cend, s1 - 1) : 0;
            s0 = s1;
            s1 = __popcll(__ballot(cend <= sb + CAP16));
            s1 = s1 < cn ? s1 : cn;
            big = s1 == s0;
            s1 = big ? s0 + 1 : s1;
        };
        auto stage = [&](uint32_t at) {
            uint64_t w = mine & lanes_below(s1) & ~lanes_below(s0);
            while (w) {
                const int t = __builtin_ctzll(w);
                w &= w - 1;
                const int4 r = table[t * NOP + wv];
                const uint64_t src =
                    static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(r.x)) |
                    static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(r.y))) << 32;
                stage_pieces(src, at + (__builtin_amdgcn_readfirstlane(r.z) - sb) * 16,
                             __builtin_amdgcn_readfirstlane(r.w) & 0xffff, lane * 16);
            }
        };
        next_step();
        uint32_t par = 0;
        stage(lds0);
        for (;;) {
            const uint64_t span = lanes_below(s1) & ~lanes_below(s0);
            g0.off = g1.off = lds0 + par - sb * 16;
            const bool more = s1 < cn, alone = big;
            if (more) next_step();
            wait_dma();
            group_barrier();
            const bool ahead = more && !alone && !big;
            if (ahead) {
                par = par ? 0 : CAP;
                stage(lds0 + par);
            }
            run_any(m0, n0, have0 & span, oa0, ob0, g0, acc0);
            run_any(m1, n1, have1 & span, oa1, ob1, g1, acc1);
            if (!more) break;
            if (!ahead) {
                group_barrier();
                par = 0;
                stage(lds0);
            }
        }
        group_barrier();                                 // table and stages are free
    }

    store(a, lane64(cl, G * R0 + C0), m0, n0, lane, acc0);
    store(a, lane64(cl, G * R1 + C1), m1, n1, lane, acc1);
}

}  // namespace

int launch_mtile(const SmmArgs &a, hipStream_t s) {
    return launch_groups(a, 512, [&](const SmmArgs &b, unsigned grid) {
        BSM_LAUNCH((k_smm_f64_mtile<34816>), grid, 512, 0, s)(b);
    });
}

}  // namespace bsm
