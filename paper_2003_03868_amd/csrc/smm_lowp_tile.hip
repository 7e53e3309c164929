// Reduced-precision block products (smm_lowp.hip) over 4 x 4 groups of C
// blocks (the groups of the FP64 tile kernel, smm_tile.hip): one workgroup of
// eight waves per group, two C blocks per wave.  The instructions of a product
// and their order, and the FP64 sums in ascending k, are those of the
// one-block kernels, so the results are the same bits.
//
// What bounds it (three parts, size 23): power.  The 2 x 2 quads used before
// unpacked every operand into LDS, three 2-byte stores per element, and read
// 1.19 operand blocks per product from L2.  Here the operands are packed once
// per multiply into images that the matrix instructions read as they are, 16
// bytes a lane, so that a block goes from memory to LDS without passing
// registers, and a 4 x 4 group reads 0.72 blocks per product.  What is left per
// product is 12 matrix instructions, 16 LDS reads and 24 FP64 additions and
// conversions; the matrix cores are busy 52% of the time at 1.54 GHz (2.4 GHz
// is the highest clock), with 4 TB/s of L2 misses.
// Measured (MI355X, block products of the square of a 1024-row iterate, 21%
// filled, 4.8e7 products of size 23): three parts 32.1 ms with quads, 20.5
// here; two parts 19.4 and 13.7; FP32 31.1 (one-block kernel 27.2) and 26.2.
// FP32 has 24 matrix instructions of 32 cycles per product, 70% busy.
// Tried: sixteen waves of one C block, two entries a stage 23.1 ms (three
// parts); 4 x 2 groups of eight waves, three per CU, 20.5 (two parts 14.1).
#include "bf16_split.h"
#include "lds_dma.h"
#include "smm_group.h"

namespace bsm {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) const us8 lds_us8;
typedef __attribute__((address_space(3))) const float lds_float;

// Image of a block, as the matrix instructions read it.  T = 2 or 3 parts of
// BF16: per part, per eight k's, 16 bytes for every row of A (column of B);
// the k's past S are zero.  T = 0, FP32: S values (rows of A, columns of B)
// for every k, k's up to the next multiple of 4 zero.
template <int S, int T>
struct LImage {
    static constexpr int KC = (S + 7) / 8;               // BF16: groups of eight k's
    static constexpr int KS = T ? (S + 15) / 16 : (S + 3) / 4;   // k steps of the instruction
    static constexpr int PART = KC * S * 16;             // bytes of a part
    static constexpr int PIECES = T ? T * KC * S : (4 * KS * S * 4 + 15) / 16;
    static constexpr int BYTES = PIECES * 16;
};

// The block's image from its FP64 values (one workgroup).
template <int S, int T, bool B>
__device__ inline void pack_image(const double *src, char *dst) {
    using I = LImage<S, T>;
    if constexpr (T == 0) {
        for (int u = threadIdx.x; u < I::BYTES / 4; u += 64) {
            const int k = u / S, i = u % S;
            const double x = k < S ? src[B ? k * S + i : i * S + k] : 0.0;
            reinterpret_cast<float *>(dst)[u] = __double2float_rn(x);
        }
    } else {
        for (int u = threadIdx.x; u < I::KC * S; u += 64) {
            const int c = u / S, i = u % S;
            us8 part[T];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 8 * c + e;
                const double x = k < S ? src[B ? k * S + i : i * S + k] : 0.0;
                uint32_t p[3];
                split_bf16(x, T, p);
#pragma unroll
                for (int q = 0; q < T; ++q) part[q][e] = static_cast<unsigned short>(p[q]);
            }
#pragma unroll
            for (int q = 0; q < T; ++q) *reinterpret_cast<us8 *>(dst + q * I::PART + u * 16) = part[q];
        }
    }
}

// One workgroup per block, or in turn where the blocks are more than a launch
// may have workgroups.
template <int S, int T, bool B>
__global__ __launch_bounds__(64) void k_pack_image(const double *v, int64_t n, uint32_t *out) {
    for (int64_t t = blockIdx.x; t < n; t += gridDim.x)
        pack_image<S, T, B>(v + t * (S * S), reinterpret_cast<char *>(out) + t * LImage<S, T>::BYTES);
}

// Wave w owns C blocks w and w + 8 of the group in the order of the FP64 tile
// kernel (a SIMD's blocks are of different rows and columns) and stages operand
// w (A rows 0 .. 3, B columns 0 .. 3) of every entry.  Two stages of EPS entries
// of eight images in LDS: EPS entries are multiplied from one while the next
// land in the other.  The barrier of a step follows every wave's wait for its
// copies of the step and its last LDS reads of the step before, so after it the
// step is whole and the other stage is free.  At most 128 registers a wave: two
// workgroups per CU for size 23.
template <int S, int T, int EPS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_lowp_tile(SmmArgs a) {
    using I = LImage<S, T>;
    constexpr int G = 4, NW = 8, NB = G * G / NW, NOP = 2 * G, NE = NOP / 4;
    static_assert(NOP == NW, "wave w stages operand w of an entry");
    constexpr int ENTRY = NOP * I::BYTES, STAGE = EPS * ENTRY;
    // BF16 with an odd number of k groups: the upper lanes of the last step
    // read zeros, for every part
    constexpr bool ODD = T > 0 && I::KC % 2 == 1;
    constexpr int ZERO = ODD ? (T - 1) * I::PART + 512 : 0;
    // past the last image: rows (columns) up to 32 of its last k's, which
    // reach only elements that are never stored
    constexpr int TAIL = 512;
    __shared__ __align__(16) char lds[2 * STAGE + TAIL + ZERO];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) char *)lds));
    constexpr uint32_t zero0 = 2 * STAGE + TAIL;
    const int64_t it = group_item(a);
    if (it < 0) return;
    const int64_t item = a.q_order ? a.q_order[it] : it;
    const int lane = threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
    // C block b of the wave
    int R[NB], C[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int id = wv + NW * b;
        R[b] = id / G;
        C[b] = (id - id / G) & (G - 1);
    }
    for (uint32_t z = threadIdx.x * 4; z < ZERO; z += NW * 256)
        *reinterpret_cast<uint32_t *>(lds + zero0 + z) = 0u;

    // LDS addresses of the lane's first operands; `last`: of the last k step,
    // whose stage offset is masked away where zeros are read
    const int r32 = lane & 31, h = lane >> 5, r16 = lane & 15, kq = lane >> 4;
    const uint32_t own = T ? (h * S + r32) * 16 : (kq * S + r16) * 4;
    const bool zl = ODD && h == 1;
    constexpr uint32_t LAST = T ? 2 * (I::KS - 1) * S * 16 : 0;
    const uint32_t zero = lds0 + zero0 + r32 * 16, keep = zl ? 0u : ~0u;

    // BF16: registers 4 g .. 4 g + 3 of the result hold rows 8 g .. 8 g + 7
    constexpr int NQ = T ? 4 * ((S + 7) / 8) : 16;
    double acc[NB][NQ];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[b][q] = 0.0;

    const int64_t e0 = a.q_seg[item];
    const int ne = __builtin_amdgcn_readfirstlane(static_cast<int>(a.q_seg[item + 1] - e0));
    const int *ent = reinterpret_cast<const int *>(a.q_ent + NE * e0);
    // ids: entries base .. base + 63, one per lane: the operands of the
    // wave's blocks, and the one it stages of the entry EPS further on (-1:
    // none)
    auto ids = [&](int base, int (&ia)[NB], int (&ib)[NB], int &io) {
        const int e = base + lane;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            ia[b] = e < ne ? ent[NOP * e + R[b]] : -1;
            ib[b] = e < ne ? ent[NOP * e + G + C[b]] : -1;
        }
        io = e + EPS < ne ? ent[NOP * (e + EPS) + wv] : -1;
    };
    const uint32_t *img = wv < G ? a.a_pk : a.b_pk;
    auto source = [&](int id) {
        return reinterpret_cast<uint64_t>(img) +
               static_cast<uint64_t>(static_cast<uint32_t>(id)) * I::BYTES;
    };
    const uint32_t slot = lds0 + wv * I::BYTES;
    const uint32_t voff = lane * 16;
    int ia[NB], ib[NB], io;
    ids(0, ia, ib, io);
#pragma unroll
    for (int i = 0; i < EPS; ++i) {
        const int id = i < ne ? __builtin_amdgcn_readfirstlane(ent[NOP * i + wv]) : -1;
        if (id >= 0) stage_pieces<I::PIECES>(source(id), slot + i * ENTRY, voff);
    }
    for (int base = 0; base < ne; base += kWave) {
        uint64_t have[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) have[b] = __ballot(ia[b] >= 0 && ib[b] >= 0);
        const uint64_t mine = __ballot(io >= 0);
        const uint64_t sp = source(io);
        const int slo = static_cast<int>(sp), shi = static_cast<int>(sp >> 32);
        ids(base + kWave, ia, ib, io);
        const int n = ne - base < kWave ? ne - base : kWave;
        for (int t = 0; t < n; t += EPS) {
            wait_dma();
            group_barrier();
            const uint32_t to = (t & EPS) ? slot : slot + STAGE;
            const uint32_t from = (t & EPS) ? STAGE : 0;
#pragma unroll
            for (int i = 0; i < EPS; ++i)
                if ((mine >> (t + i)) & 1) {
                    const uint64_t src =
                        static_cast<uint32_t>(__builtin_amdgcn_readlane(slo, t + i)) |
                        static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(shi, t + i))) << 32;
                    stage_pieces<I::PIECES>(src, to + i * ENTRY, voff);
                }
#pragma unroll
            for (int p = 0; p < EPS * NB; ++p) {
                const int i = p / NB, b = p % NB;
                if ((have[b] >> (t + i)) & 1) {
                    const uint32_t in = from + i * ENTRY;
                    const uint32_t ra = lds0 + R[b] * I::BYTES + own, rb = lds0 + (G + C[b]) * I::BYTES + own;
                    const uint32_t ra_last = zl ? zero : ra + LAST, rb_last = zl ? zero : rb + LAST;
                    if constexpr (T > 0) {
                        auto ld = [&](uint32_t base_, uint32_t last_, int ks, int q) {
                            const uint32_t p = ks == I::KS - 1 ? last_ + (in & keep)
                                                               : base_ + in + ks * 2 * S * 16;
                            return __builtin_bit_cast(bf8, *reinterpret_cast<lds_us8 *>(
                                static_cast<uintptr_t>(p + q * I::PART)));
                        };
                        f16v part = {};
#pragma unroll
                        for (int ks = 0; ks < I::KS; ++ks) {
                            const bf8 ah = ld(ra, ra_last, ks, 0), bh = ld(rb, rb_last, ks, 0);
                            if constexpr (T == 3) {
                                const bf8 am = ld(ra, ra_last, ks, 1), al = ld(ra, ra_last, ks, 2);
                                const bf8 bm = ld(rb, rb_last, ks, 1), bl = ld(rb, rb_last, ks, 2);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bm, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bm, part, 0, 0, 0);
                                asm volatile("" ::: "memory");
                            } else {
                                const bf8 al = ld(ra, ra_last, ks, 1), bl = ld(rb, rb_last, ks, 1);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, part, 0, 0, 0);
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, part, 0, 0, 0);
                            }
                        }
                        if constexpr (T == 3) {
                            // the leading parts again, read anew: held from
                            // above they cost sixteen registers
#pragma unroll
                            for (int ks = 0; ks < I::KS; ++ks)
                                part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    ld(ra, ra_last, ks, 0), ld(rb, rb_last, ks, 0), part, 0, 0, 0);
                        }
#pragma unroll
                        for (int q = 0; q < NQ; ++q) acc[b][q] += static_cast<double>(part[q]);
                    } else {
                        constexpr int MT = (S + 15) / 16;
                        f4 part[MT][MT] = {};
                        lds_float *pa = reinterpret_cast<lds_float *>(static_cast<uintptr_t>(ra + in));
                        lds_float *pb = reinterpret_cast<lds_float *>(static_cast<uintptr_t>(rb + in));
#pragma unroll
                        for (int ks = 0; ks < I::KS; ++ks) {
                            float av[MT], bv[MT];
#pragma unroll
                            for (int u = 0; u < MT; ++u) {
                                av[u] = pa[4 * ks * S + 16 * u];
                                bv[u] = pb[4 * ks * S + 16 * u];
                            }
#pragma unroll
                            for (int u = 0; u < MT; ++u)
#pragma unroll
                                for (int v = 0; v < MT; ++v)
                                    part[u][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[v],
                                                                                      part[u][v], 0, 0, 0);
                        }
#pragma unroll
                        for (int u = 0; u < MT; ++u)
#pragma unroll
                            for (int v = 0; v < MT; ++v)
#pragma unroll
                                for (int q = 0; q < 4; ++q)
                                    acc[b][(u * 2 + v) * 4 + q] += static_cast<double>(part[u][v][q]);
                    }
                }
                asm volatile("" ::: "memory");
            }
        }
    }

    // alpha * sum + beta * C_in and the block's filter norms
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t cb = a.q_cblk[G * G * item + G * R[b] + C[b]];
        if (cb < 0) continue;
        const int64_t co = a.c_blk_off[cb];
        const double *cin = nullptr;
        if (a.cin_map) {
            const int64_t tt = a.cin_map[cb];
            if (tt >= 0) cin = a.cin_vals + a.cin_blk_off[tt];
        }
        double sq = 0.0, mx = 0.0;
        constexpr int MT = (S + 15) / 16;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            int row, col;
            if (T > 0) {
                row = 8 * (q >> 2) + 4 * h + (q & 3);
                col = r32;
            } else {
                const int u = q >> 3, v = (q >> 2) & 1;
                row = 16 * u + 4 * kq + (q & 3);
                col = 16 * v + r16;
                if (u >= MT || v >= MT) row = 1 << 20;
            }
            if (row < S && col < S) {
                double v = a.alpha * acc[b][q];
                if (cin) v += a.beta * cin[row * S + col];
                a.c_vals[co + row * S + col] = v;
                sq += v * v;
                mx = fmax(mx, fabs(v));
            }
        }
        sq = group_wave_sum(sq);
        mx = group_wave_max(mx);
        if (lane == 0) {
            a.sq_out[cb] = sq;
            a.mx_out[cb] = mx;
            if (!isfinite(sq)) atomicOr(a.flags, kFlagNonFinite);
        }
    }
}

template <int S>
int64_t image_words(int prec) {
    return (prec == BSM_FP32 ? LImage<S, 0>::BYTES : prec == BSM_SPLIT_BF16 ? LImage<S, 2>::BYTES
                                                                            : LImage<S, 3>::BYTES) / 4;
}

template <int S, int T>
void pack_side(const double *v, int64_t n, bool b_side, uint32_t *out, hipStream_t s) {
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>(n, (int64_t{1} << 32) / 64 - 1));
    if (b_side) k_pack_image<S, T, true><<<grid, 64, 0, s>>>(v, n, out);
    else k_pack_image<S, T, false><<<grid, 64, 0, s>>>(v, n, out);
}

}  // namespace

// Entries per stage: a barrier serves more of them where the products are
// short.  Whole squares, reuse 18, of 2048 block rows with 1 / 2 / 4 entries:
// size 5 two parts 5.5 / 5.0 / 4.9 ms, FP32 5.0 / 4.5 / 4.4; 13 two parts 7.6 /
// 7.0 / 6.9, FP32 6.5 / 6.1 / 6.7.
constexpr int lowp_eps(int s) { return s <= 5 ? 4 : s <= 13 ? 2 : 1; }

template <int S, int T>
static int launch_size(const SmmArgs &a, hipStream_t s) {
    constexpr int EPS = lowp_eps(S);
    note_kernelf("k_lowp_tile<%d, %d, %d>", S, T, EPS);
    return launch_groups(a, 512, [&](const SmmArgs &b, unsigned grid) {
        k_lowp_tile<S, T, EPS><<<grid, 512, 0, s>>>(b);
    });
}

#define BSM_LT_SIZES(X) X(5) X(13) X(23) X(26) X(32)

int64_t lowp_image_words(int64_t nblocks, int size, int prec) {
    switch (size) {
#define BSM_LT(S) case S: return nblocks * image_words<S>(prec);
        BSM_LT_SIZES(BSM_LT)
#undef BSM_LT
        default: return 0;
    }
}

int pack_lowp_image(const double *v, int64_t nblocks, int size, int prec, bool b_side, uint32_t *out,
                    hipStream_t s) {
    if (nblocks == 0) return BSM_OK;
    switch (size) {
#define BSM_LT(S)                                                              \
        case S:                                                                \
            if (prec == BSM_FP32) pack_side<S, 0>(v, nblocks, b_side, out, s); \
            else if (prec == BSM_SPLIT_BF16) pack_side<S, 2>(v, nblocks, b_side, out, s); \
            else pack_side<S, 3>(v, nblocks, b_side, out, s);                  \
            break;
        BSM_LT_SIZES(BSM_LT)
#undef BSM_LT
        default: set_error("no reduced-precision image for block size %d", size); return BSM_EINVAL;
    }
    BSM_HIP(hipGetLastError());
    return BSM_OK;
}

int launch_lowp_tile(const SmmArgs &a, hipStream_t s) {
    switch (a.uni_m) {
#define BSM_LT(S)                                                                                      \
        case S:                                                                                        \
            return a.prec == BSM_FP32         ? launch_size<S, 0>(a, s)                                \
                   : a.prec == BSM_SPLIT_BF16 ? launch_size<S, 2>(a, s)                                \
                                              : launch_size<S, 3>(a, s);
        BSM_LT_SIZES(BSM_LT)
#undef BSM_LT
        default: set_error("no reduced-precision tile kernel for block size %d", a.uni_m); return BSM_EINVAL;
    }
}

}  // namespace bsm
