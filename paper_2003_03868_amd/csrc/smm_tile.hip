// FP64 block products for uniform block sizes 4 .. 32, one workgroup of
// sixteen waves per 4 x 4 group of C blocks, one C block per wave, with the
// group's merged product list (built in quad.hip).  Sums and instructions are those
// of the quad kernel (smm_quad.hip): ascending k, V_MFMA_F64_4X4X4_4B_F64,
// so the results are the same bits.
//
// What bounds it (size 23): the 2 x 2 quads moved 1.19 operand blocks per product
// through L2 (5.1 TB/s of misses on the sign workload's settled products),
// and the board's power limit held the clock to 2.0 GHz with the matrix
// cores 58% busy.  A 4 x 4 group moves 0.72 blocks per product.  Four things
// make that pay:
//   * operands go from memory to LDS without passing registers
//     (global_load_lds_dwordx4), double-buffered, one barrier per entry, so
//     two groups of sixteen waves share a CU with 59 registers a wave;
//   * the four waves of a SIMD own C blocks of different rows and columns of
//     the group, so that the products of an entry (half of the sixteen are
//     there) spread evenly: with a SIMD per column its load was 2.1 times
//     the mean, this way 1.1 times;
//   * entry indices are taken 64 at a time, one per lane, and turned into
//     bit masks and LDS offsets there: per entry a wave tests a bit and reads
//     a lane.  Worked out per entry by every wave, this integer work alone
//     took 69 ms where the products took 190;
//   * nothing is done for a C block without a product in the entry.
// Measured (MI355X, square of a settled iterate, 2048 block rows, 25%
// filled, 5.4e8 products): 395 ms with quads (33 TFLOP/s), 314 ms here
// (42 TFLOP/s); first square of the iteration (4.5% filled): 15.3 and 13.9
// ms.  Now the matrix cores are busy 71% of the time at 2.06 GHz.
// Tried and slower on the settled product: 4 x 4 groups of four waves with
// 2 x 2 C blocks each (409 ms), 8 x 8 groups of sixteen such waves (359 ms,
// 0.44 blocks per product, but one group per CU leaves nothing to run while
// it waits at its barrier), eight waves of 2 x 1 C blocks (322 -> 330 ms),
// groups ordered in square tiles (346 -> 354 .. 363 ms).
#include "lds_dma.h"
#include "smm_group.h"

namespace bsm {

namespace {

typedef __attribute__((address_space(3))) double lds_double;

template <int S>
struct TShape {
    static constexpr int B2 = S * S;
    static constexpr int KS = (S + 3) / 4, H = (KS + 1) / 2;
    static constexpr int KLAST = S - 4 * (KS - 1);                // valid x in the last k-step
    static constexpr int PIECES = (B2 * 8 + (B2 & 1) * 8) / 16;   // 16-byte pieces of a staged block
    static constexpr int SLOT = PIECES * 16;                      // LDS bytes of a staged block
    // padded reads past the last block: A rows up to 8 H, B rows up to 4 KS
    static constexpr int TAIL = (8 * H * S - B2 + 64) * 8;
};

// The wave's product of an entry: 4 x 4 x 4 steps in ascending k.  A rows and
// B columns past S read what follows in LDS, which reaches only accumulator
// elements that are never stored; the k's past S are zeroed on both sides.
template <int S>
__device__ inline void tile_product(const lds_double *ap, const lds_double *bp, bool klast_ok,
                                    double (&acc)[TShape<S>::H][TShape<S>::H]) {
    using T = TShape<S>;
    constexpr int H = T::H;
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks) {
        double av[H], bv[H];
#pragma unroll
        for (int t = 0; t < H; ++t) {
            const double v = ap[4 * t * S + 4 * ks];
            av[t] = (ks == T::KS - 1 && T::KLAST < 4 && !klast_ok) ? 0.0 : v;
        }
#pragma unroll
        for (int u = 0; u < H; ++u) {
            const double v = bp[4 * u + 4 * ks * S];
            bv[u] = (ks == T::KS - 1 && T::KLAST < 4 && !klast_ok) ? 0.0 : v;
        }
#pragma unroll
        for (int t = 0; t < H; ++t)
#pragma unroll
            for (int u = 0; u < H; ++u)
                acc[t][u] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[t], bv[u], acc[t][u], 0, 0, 0);
    }
}

// Wave wv owns C block (R, C) = (wv / 4, (wv - wv / 4) mod 4) of the group and
// stages operand wv mod 8 (A rows 0 .. 3, B columns 0 .. 3) of every entry
// (waves 0 .. 7; EPS > 1: waves 0 .. 7 of the even, 8 .. 15 of the odd ones).
// Two stages of EPS entries of eight blocks in LDS: the EPS entries of a step
// are multiplied from one while the next EPS land in the other.  The barrier
// of a step follows every wave's wait for its copies of the step and its last
// LDS reads of the step before, so after it the step is whole and the other
// stage is free.  WPE: waves per SIMD (two groups per CU up to size 24, whose
// stages share its LDS; one above).
template <int S, int EPS, int WPE>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
k_smm_f64_tile(SmmArgs a) {
    using T = TShape<S>;
    constexpr int H = T::H;
    constexpr int G = 4, NOP = 2 * G, NE = NOP / 4;
    constexpr int ENTRY = NOP * T::SLOT, STAGE = EPS * ENTRY;    // LDS bytes of an entry, of a stage
    __shared__ __align__(16) char lds[2 * STAGE + T::TAIL];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) char *)lds));
    const int64_t it = group_item(a);
    if (it < 0) return;
    const int64_t item = a.q_order ? a.q_order[it] : it;
    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
    const int R = wv / 4, C = (wv - wv / 4) & 3;
    const int x = lane >> 4, blk = (lane >> 2) & 3, y = lane & 3;
    const int bh = blk >> 1, bw = blk & 1;
    // LDS addresses of A(4 (bh H + t) + y, 4 ks + x) and B(4 ks + x, 4 (bw H + u) + y)
    const uint32_t ra0 = lds0 + ((4 * bh * H + y) * S + x) * 8 + R * T::SLOT;
    const uint32_t rb0 = lds0 + (x * S + 4 * bw * H + y) * 8 + (G + C) * T::SLOT;
    const bool klast_ok = x < T::KLAST;

    double acc[H][H];
#pragma unroll
    for (int t = 0; t < H; ++t)
#pragma unroll
        for (int u = 0; u < H; ++u) acc[t][u] = 0.0;

    const int64_t e0 = a.q_seg[item];
    const int ne = __builtin_amdgcn_readfirstlane(static_cast<int>(a.q_seg[item + 1] - e0));
    const int *ent = reinterpret_cast<const int *>(a.q_ent + NE * e0);
    // Entries base .. base + 63, one per lane: the wave's row's and column's
    // operand, and the operand it stages of the entry EPS further on (-1: none).
    const int Z = wv % NOP, first = wv / NOP;
    auto ids = [&](int base, int &ia, int &ib, int &io) {
        const int e = base + lane;
        ia = e < ne ? ent[NOP * e + R] : -1;
        ib = e < ne ? ent[NOP * e + G + C] : -1;
        io = e + EPS < ne ? ent[NOP * (e + EPS) + Z] : -1;
    };
    const double *vals = Z < G ? a.a_vals : a.b_vals;
    // Blocks of odd sizes start on 8 bytes: an odd block is copied from one
    // double before it (its even neighbour's last), an even one with one double
    // after it (its neighbour's first or, for the last block, the padding of the
    // allocation, whose size is a multiple of 256 bytes), and the reader adds
    // the block's parity to its offset.
    auto source = [&](int id) {                          // 16-byte aligned start of a block
        return (reinterpret_cast<uint64_t>(vals) +
                static_cast<uint64_t>(static_cast<uint32_t>(id)) * (T::B2 * 8)) & ~15ull;
    };
    const uint32_t slot = lds0 + Z * T::SLOT;
    const uint32_t voff = lane * 16;
    int ia, ib, io;
    ids(0, ia, ib, io);
#pragma unroll
    for (int i = 0; i < EPS; ++i) {
        const int id = i < ne && i % 2 == first ? __builtin_amdgcn_readfirstlane(ent[NOP * i + Z]) : -1;
        if (id >= 0) stage_pieces<T::PIECES>(source(id), slot + i * ENTRY, voff);
    }
    for (int base = 0; base < ne; base += kWave) {
        const uint64_t have = __ballot(ia >= 0 && ib >= 0);
        const uint64_t mine = __ballot(io >= 0) &
                              (EPS == 1 ? (first == 0 ? ~0ull : 0ull)
                                        : (first == 0 ? 0x5555555555555555ull : 0xaaaaaaaaaaaaaaaaull));
        const int in = ((lane / EPS) & 1) * STAGE + lane % EPS * ENTRY;
        const int oa = in + ((T::B2 & 1) ? (ia & 1) * 8 : 0);
        const int ob = in + ((T::B2 & 1) ? (ib & 1) * 8 : 0);
        const uint64_t sp = source(io);
        const int slo = static_cast<int>(sp), shi = static_cast<int>(sp >> 32);
        ids(base + kWave, ia, ib, io);
        const int n = ne - base < kWave ? ne - base : kWave;
        for (int t = 0; t < n; t += EPS) {
            wait_dma();
            group_barrier();
            const uint32_t to = (t & EPS) ? slot : slot + STAGE;
#pragma unroll
            for (int i = 0; i < EPS; ++i)
                if ((mine >> (t + i)) & 1) {
                    const uint64_t src =
                        static_cast<uint32_t>(__builtin_amdgcn_readlane(slo, t + i)) |
                        static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(shi, t + i))) << 32;
                    stage_pieces<T::PIECES>(src, to + i * ENTRY, voff);
                }
#pragma unroll
            for (int i = 0; i < EPS; ++i)
                if ((have >> (t + i)) & 1) {
                    const uint32_t pa = ra0 + __builtin_amdgcn_readlane(oa, t + i);
                    const uint32_t pb = rb0 + __builtin_amdgcn_readlane(ob, t + i);
                    tile_product<S>(reinterpret_cast<const lds_double *>(static_cast<uintptr_t>(pa)),
                                    reinterpret_cast<const lds_double *>(static_cast<uintptr_t>(pb)),
                                    klast_ok, acc);
                }
        }
    }

    // alpha * sum + beta * C_in and the block's filter norms
    const int64_t c = a.q_cblk[G * G * item + G * R + C];
    if (c < 0) return;
    const int64_t co = a.c_blk_off[c];
    const double *cin = nullptr;
    if (a.cin_map) {
        const int64_t t = a.cin_map[c];
        if (t >= 0) cin = a.cin_vals + a.cin_blk_off[t];
    }
    double sq = 0.0, mx = 0.0;
#pragma unroll
    for (int t = 0; t < H; ++t)
#pragma unroll
        for (int u = 0; u < H; ++u) {
            const int row = 4 * (bh * H + t) + x, col = 4 * (bw * H + u) + y;
            if (row < S && col < S) {
                double v = a.alpha * acc[t][u];
                if (cin) v += a.beta * cin[row * S + col];
                a.c_vals[co + row * S + col] = v;
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

}  // namespace

// Entries per stage: a barrier serves more of them where the products are
// short, as long as two groups share a CU's LDS.  Settled squares of 1024
// block rows (41% filled), 1 / 2 / 4 entries: size 5 18.7 / 14.1 / 12.5 ms, 9
// 30.7 / 27.5 / 26.1, 13 38.1 / 36.1, 17 80.9 / 79.6.
constexpr int tile_eps(int s) { return s <= 12 ? 4 : s <= 17 ? 2 : 1; }

template <int S>
static int launch_size(const SmmArgs &a, hipStream_t s) {
    constexpr int EPS = tile_eps(S), WPE = S <= 24 ? 8 : 4;
    note_kernelf("k_smm_f64_tile<%d, %d, %d>", S, EPS, WPE);
    return launch_groups(a, 1024, [&](const SmmArgs &b, unsigned grid) {
        k_smm_f64_tile<S, EPS, WPE><<<grid, 1024, 0, s>>>(b);
    });
}

bool smm_tile_available(int m) { return m >= 4 && m <= kMaxBlock; }

int launch_tile(const SmmArgs &a, hipStream_t s) {
    switch (a.uni_m) {
#define BSM_TILE(S) \
        case S: return launch_size<S>(a, s);
        BSM_TILE(4) BSM_TILE(5) BSM_TILE(6) BSM_TILE(7) BSM_TILE(8) BSM_TILE(9) BSM_TILE(10)
        BSM_TILE(11) BSM_TILE(12) BSM_TILE(13) BSM_TILE(14) BSM_TILE(15) BSM_TILE(16) BSM_TILE(17)
        BSM_TILE(18) BSM_TILE(19) BSM_TILE(20) BSM_TILE(21) BSM_TILE(22) BSM_TILE(23) BSM_TILE(24)
        BSM_TILE(25) BSM_TILE(26) BSM_TILE(27) BSM_TILE(28) BSM_TILE(29) BSM_TILE(30) BSM_TILE(31)
        BSM_TILE(32)
#undef BSM_TILE
        default: set_error("no 4 x 4 tile kernel for block size %d", a.uni_m); return BSM_EINVAL;
    }
}

}  // namespace bsm
