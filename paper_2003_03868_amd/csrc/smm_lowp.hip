// Reduced-precision block products (the approximate-computing direction of
// the paper: lower or mixed precision where FP64 accuracy is not needed,
// "Approximate Computing" section and the DBCSR "Outlook").
//
// Two forms, both accumulating each block product in FP32 on the matrix
// cores and adding it into an FP64 accumulator per C block (so the error of
// one product does not grow with the length of the product stack); the
// result, its norms and the filter stay FP64:
//
//  * FP32:       operands rounded to FP32; V_MFMA_F32_16X16X4_F32.
//  * split-BF16: x = hi + lo with hi = bf16(x), lo = bf16(x - hi) (both
//                round-to-nearest-even); A*B ~ lo*hi + hi*lo + hi*hi with
//                V_MFMA_F32_32X32X16_BF16 (the lo*lo term is dropped).
//                Each operand keeps about 17 significant bits.
//  * three-term split-BF16: x = hi + mid + lo, each part the RNE bf16 of
//                what the previous parts leave; with |mid| <= 2^-9 |x| and
//                |lo| <= 2^-18 |x| the products are kept down to size
//                2^-18 of hi*hi: mid*mid + hi*lo + lo*hi + mid*hi + hi*mid
//                + hi*hi (small terms first).  About 26 bits per operand,
//                so the FP32 accumulation sets the error, as in FP32 mode.
//
// Operands are packed once per multiply: one 32-bit word per element (the
// FP32 bits, or hi << 16 | lo), and for the three-term split hi << 16 | mid
// followed by an array of the lo parts (uint16).  The kernels here take one C
// block per wave, for uniform block sizes (compile-time shapes, up to 32);
// larger products run over groups of C blocks (smm_lowp_tile.hip).
#include "bf16_split.h"
#include "smm.h"

namespace bsm {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short us8 __attribute__((ext_vector_type(8)));

// --------------------------------------------------------------- packing

__global__ void k_pack_lowp(const double *v, int64_t n, uint32_t *out, int prec) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = v[i];
    if (prec == BSM_FP32) {
        out[i] = __float_as_uint(__double2float_rn(x));
    } else {
        uint32_t p[3];
        split_bf16(x, prec == BSM_SPLIT_BF16X3 ? 3 : 2, p);
        out[i] = (p[0] << 16) | p[1];
        if (prec == BSM_SPLIT_BF16X3)
            reinterpret_cast<unsigned short *>(out + n)[i] = static_cast<unsigned short>(p[2]);
    }
}

int pack_lowp(const double *v, int64_t n, uint32_t *out, int prec, hipStream_t s) {
    if (n == 0) return BSM_OK;
    k_pack_lowp<<<grid_for(n, 256), 256, 0, s>>>(v, n, out, prec);
    BSM_HIP(hipGetLastError());
    return BSM_OK;
}

__device__ inline int64_t lp_item(int64_t n_items) {
    const int64_t per = (n_items + kXcds - 1) / kXcds;
    return static_cast<int64_t>(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

__device__ inline double lp_wave_sum(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}
__device__ inline double lp_wave_max(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// Epilogue shared by both forms: out(row, col) for the lane's 16 slots.
template <int M, int N, class RowCol>
__device__ inline void lp_store(const SmmArgs &a, int64_t c, const double (&acc)[16],
                                RowCol rc) {
    const int64_t co = a.c_blk_off[c];
    const double *cin = nullptr;
    if (a.cin_map) {
        const int64_t t = a.cin_map[c];
        if (t >= 0) cin = a.cin_vals + a.cin_blk_off[t];
    }
    double sq = 0.0, mx = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        int row, col;
        rc(q, row, col);
        if (row < M && col < N) {
            double v = a.alpha * acc[q];
            if (cin) v += a.beta * cin[row * N + col];
            a.c_vals[co + row * N + col] = v;
            sq += v * v;
            mx = fmax(mx, fabs(v));
        }
    }
    sq = lp_wave_sum(sq);
    mx = lp_wave_max(mx);
    if (threadIdx.x == 0) {
        a.sq_out[c] = sq;
        a.mx_out[c] = mx;
        if (!isfinite(sq)) atomicOr(a.flags, kFlagNonFinite);
    }
}

// ------------------------------------------------------------ split-BF16
// One wavefront per C block, the block padded to one 32 x 32 tile.
// LDS: A_hi, A_lo as [32][LDK] and B_hi^T, B_lo^T as [32][LDK] (bf16), so
// each lane reads its 8 consecutive k values with one 16-byte load.
// Lane layout of V_MFMA_F32_32X32X16_BF16 (measured on gfx950):
// A(i,k): lane i + 32*(k/8), element k%8; B(k,j): lane j + 32*(k/8),
// element k%8; D(i,j): lane j + 32*((i/4)%2), register 4*(i/8) + i%4.
// One split block product over KS k steps of 16, added into the FP64
// accumulator.  T = 2: LDS planes hi, lo of A then of B, per k step
// lo*hi + hi*lo + hi*hi.  T = 3: planes hi, mid, lo; first every correction
// term (mid*mid, lo*hi, hi*lo, mid*hi, hi*mid) of all k steps, then hi*hi of
// all k steps, so that the small terms are summed while the FP32 sum is
// still small and are not rounded to the precision of hi*hi.
template <int T, int KS, int LDK, int PLANE>
__device__ inline void bf16_split_product(const unsigned short *as, const unsigned short *bs,
                                          int base, double (&acc)[16]) {
    auto ld = [&](const unsigned short *p, int q, int ks) {
        return __builtin_bit_cast(bf8, *reinterpret_cast<const us8 *>(p + q * PLANE + base + 16 * ks));
    };
    f16v part = {};
    if (T == 3) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf8 ah = ld(as, 0, ks), am = ld(as, 1, ks), al = ld(as, 2, ks);
            const bf8 bh = ld(bs, 0, ks), bm = ld(bs, 1, ks), bl = ld(bs, 2, ks);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bm, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bm, part, 0, 0, 0);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld(as, 0, ks), ld(bs, 0, ks), part, 0, 0, 0);
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf8 ah = ld(as, 0, ks), al = ld(as, 1, ks), bh = ld(bs, 0, ks), bl = ld(bs, 1, ks);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, part, 0, 0, 0);
            part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, part, 0, 0, 0);
        }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] += static_cast<double>(part[q]);
}

template <int M, int N, int K, int T>
__global__ void __launch_bounds__(64)
k_smm_bf16x3(SmmArgs a) {
    constexpr int LDK = 40;                         // 80-byte rows: conflict-free 16 B reads
    constexpr int PLANE = 32 * LDK;
    constexpr int KS = (K + 15) / 16;
    constexpr int NA = (M * K + kWave - 1) / kWave, NB = (K * N + kWave - 1) / kWave;
    __shared__ __attribute__((aligned(16))) unsigned short sm[2 * T * PLANE];
    unsigned short *as = sm, *bs = sm + T * PLANE;
    const int64_t item = lp_item(a.nC);
    if (item >= a.nC) return;
    const int lane = threadIdx.x;
    const int64_t c = a.worklist ? a.worklist[a.c0 + item] : a.c0 + item;
    for (int e = lane; e < 2 * T * PLANE; e += kWave) sm[e] = 0;
    const unsigned short *alo3 = reinterpret_cast<const unsigned short *>(a.a_pk + a.a_pk_n);
    const unsigned short *blo3 = reinterpret_cast<const unsigned short *>(a.b_pk + a.b_pk_n);

    int oa[NA], ob[NB];
#pragma unroll
    for (int q = 0; q < NA; ++q) {
        const int e = lane + q * kWave;
        oa[q] = (e < M * K) ? (e / K) * LDK + (e % K) : -1;
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int e = lane + q * kWave;
        ob[q] = (e < K * N) ? (e % N) * LDK + (e / N) : -1;
    }
    const int r32 = lane & 31, h = lane >> 5;

    double acc[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0;

    const int64_t p0 = a.seg[c - a.c0];
    const int np = __builtin_amdgcn_readfirstlane(static_cast<int>(a.seg[c - a.c0 + 1] - p0));
    StackLane stk(a, p0, np);
    uint32_t pa[NA], pb[NB];
    unsigned short la[T == 3 ? NA : 1], lb[T == 3 ? NB : 1];
    auto prefetch = [&](int p) {
        int ia, ib;
        stk.get(p, ia, ib);
        const int64_t oa0 = static_cast<int64_t>(ia) * (M * K), ob0 = static_cast<int64_t>(ib) * (K * N);
        const uint32_t *ga = a.a_pk + oa0;
        const uint32_t *gb = a.b_pk + ob0;
#pragma unroll
        for (int q = 0; q < NA; ++q) pa[q] = (oa[q] >= 0) ? ga[lane + q * kWave] : 0u;
#pragma unroll
        for (int q = 0; q < NB; ++q) pb[q] = (ob[q] >= 0) ? gb[lane + q * kWave] : 0u;
        if (T == 3) {
#pragma unroll
            for (int q = 0; q < NA; ++q) la[q] = (oa[q] >= 0) ? alo3[oa0 + lane + q * kWave] : 0;
#pragma unroll
            for (int q = 0; q < NB; ++q) lb[q] = (ob[q] >= 0) ? blo3[ob0 + lane + q * kWave] : 0;
        }
    };
    if (np > 0) prefetch(0);
    __syncthreads();
    for (int p = 0; p < np; ++p) {
#pragma unroll
        for (int q = 0; q < NA; ++q)
            if (oa[q] >= 0) {
                as[oa[q]] = static_cast<unsigned short>(pa[q] >> 16);
                as[PLANE + oa[q]] = static_cast<unsigned short>(pa[q] & 0xFFFFu);
                if (T == 3) as[2 * PLANE + oa[q]] = la[q];
            }
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (ob[q] >= 0) {
                bs[ob[q]] = static_cast<unsigned short>(pb[q] >> 16);
                bs[PLANE + ob[q]] = static_cast<unsigned short>(pb[q] & 0xFFFFu);
                if (T == 3) bs[2 * PLANE + ob[q]] = lb[q];
            }
        __syncthreads();
        if (p + 1 < np) prefetch(p + 1);
        bf16_split_product<T, KS, LDK, PLANE>(as, bs, r32 * LDK + 8 * h, acc);
        __syncthreads();
    }
    lp_store<M, N>(a, c, acc, [&](int q, int &row, int &col) {
        row = 8 * (q >> 2) + 4 * h + (q & 3);
        col = r32;
    });
}

// ------------------------------------------------------------------ FP32
// One wavefront per C block as a 2 x 2 grid of 16 x 16 tiles.
// Lane layout of V_MFMA_F32_16X16X4_F32 (measured on gfx950):
// A(i,k): lane i + 16k; B(k,j): lane j + 16k; D(i,j): lane j + 16*(i/4),
// register i%4.
template <int M, int N, int K>
__global__ void __launch_bounds__(64)
k_smm_f32(SmmArgs a) {
    constexpr int LDA = 33, LDB = 32;               // A rows in distinct banks
    constexpr int KP = 4 * ((K + 3) / 4);
    constexpr int MT = (M + 15) / 16, NT = (N + 15) / 16;
    constexpr int NA = (M * K + kWave - 1) / kWave, NB = (K * N + kWave - 1) / kWave;
    __shared__ float sA[32 * LDA];
    __shared__ float sB[KP * LDB];
    const int64_t item = lp_item(a.nC);
    if (item >= a.nC) return;
    const int lane = threadIdx.x;
    const int64_t c = a.worklist ? a.worklist[a.c0 + item] : a.c0 + item;
    for (int e = lane; e < 32 * LDA; e += kWave) sA[e] = 0.f;
    for (int e = lane; e < KP * LDB; e += kWave) sB[e] = 0.f;
    int oa[NA], ob[NB];
#pragma unroll
    for (int q = 0; q < NA; ++q) {
        const int e = lane + q * kWave;
        oa[q] = (e < M * K) ? (e / K) * LDA + (e % K) : -1;
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int e = lane + q * kWave;
        ob[q] = (e < K * N) ? (e / N) * LDB + (e % N) : -1;
    }
    const int r16 = lane & 15, kq = lane >> 4;
    double acc[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0;

    const int64_t p0 = a.seg[c - a.c0];
    const int np = __builtin_amdgcn_readfirstlane(static_cast<int>(a.seg[c - a.c0 + 1] - p0));
    StackLane stk(a, p0, np);
    uint32_t pa[NA], pb[NB];
    auto prefetch = [&](int p) {
        int ia, ib;
        stk.get(p, ia, ib);
        const uint32_t *ga = a.a_pk + static_cast<int64_t>(ia) * (M * K);
        const uint32_t *gb = a.b_pk + static_cast<int64_t>(ib) * (K * N);
#pragma unroll
        for (int q = 0; q < NA; ++q) pa[q] = (oa[q] >= 0) ? ga[lane + q * kWave] : 0u;
#pragma unroll
        for (int q = 0; q < NB; ++q) pb[q] = (ob[q] >= 0) ? gb[lane + q * kWave] : 0u;
    };
    if (np > 0) prefetch(0);
    __syncthreads();
    for (int p = 0; p < np; ++p) {
#pragma unroll
        for (int q = 0; q < NA; ++q)
            if (oa[q] >= 0) sA[oa[q]] = __uint_as_float(pa[q]);
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (ob[q] >= 0) sB[ob[q]] = __uint_as_float(pb[q]);
        __syncthreads();
        if (p + 1 < np) prefetch(p + 1);
        f4 part[2][2] = {};
#pragma unroll
        for (int ks = 0; ks < KP / 4; ++ks) {
            float av[2], bv[2];
#pragma unroll
            for (int t = 0; t < MT; ++t) av[t] = sA[(16 * t + r16) * LDA + 4 * ks + kq];
#pragma unroll
            for (int u = 0; u < NT; ++u) bv[u] = sB[(4 * ks + kq) * LDB + 16 * u + r16];
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u)
                    part[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t], bv[u], part[t][u],
                                                                      0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[(t * 2 + u) * 4 + r] += static_cast<double>(part[t][u][r]);
        __syncthreads();
    }
    lp_store<M, N>(a, c, acc, [&](int q, int &row, int &col) {
        const int tile = q >> 2, r = q & 3;
        const int t = tile >> 1, u = tile & 1;
        row = 16 * t + 4 * kq + r;
        col = 16 * u + r16;
        if (t >= MT || u >= NT) row = 1 << 20;   // tile not present
    });
}

bool smm_lowp_available(int m, int n, int k) {
    return (m == n && n == k) && (m == 5 || m == 13 || m == 23 || m == 26 || m == 32);
}

int smm_launch_lowp(const SmmArgs &a, hipStream_t s) {
    if (a.nC <= 0) return BSM_OK;
    const int64_t per = (a.nC + kXcds - 1) / kXcds;
    const unsigned grid = static_cast<unsigned>(per * kXcds);
    if (!(a.uni_m && smm_lowp_available(a.uni_m, a.uni_n, a.uni_k))) {
        set_error("reduced-precision products need uniform block sizes 5, 13, 23, 26 or 32");
        return BSM_EINVAL;
    }
#define BSM_LP(SZ)                                                                  \
    case SZ:                                                                        \
        if (a.prec == BSM_FP32) BSM_LAUNCH((k_smm_f32<SZ, SZ, SZ>), grid, 64, 0, s)(a);       \
        else if (a.prec == BSM_SPLIT_BF16X3) BSM_LAUNCH((k_smm_bf16x3<SZ, SZ, SZ, 3>), grid, 64, 0, s)(a); \
        else BSM_LAUNCH((k_smm_bf16x3<SZ, SZ, SZ, 2>), grid, 64, 0, s)(a);                    \
        break;
    switch (a.uni_m) {
        BSM_LP(5)
        BSM_LP(13)
        BSM_LP(23)
        BSM_LP(26)
        BSM_LP(32)
        default: break;
    }
#undef BSM_LP
    BSM_HIP(hipGetLastError());
    return BSM_OK;
}

}  // namespace bsm
