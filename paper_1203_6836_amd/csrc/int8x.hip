// Reduced-precision SP2 product on int8 MFMA with exact integer accumulation
// (an error-free split of FP64 operands into integer slices whose products
// are exact in integer arithmetic, the Ozaki scheme for matrix products).
//
// The FP64 master X_n is split row by row into fixed-point digit planes:
// with the row scale s_i = (1 + 2^-7) max_j |X_ij| (row_scale), y = X_ij / s_i
// lies in [-0.993, 0.993] and is written as y ~ sum_t d_t 2^-(e0 + W t), W
// bits per digit (digit_bits), e0 = W - 1:
//   W = 8: the integer m = rint(y 2^(8S - 1)) (|m| < 0.9961 2^(8S - 1), the
//     range of the excess code below) is written in base 256 with digits in
//     [-128, 127]: the bytes of m + 0x80..80 (S bytes), each read back as a
//     byte minus 128.  One rounding, error <= 2^-(8S) s_i; the top digit
//     uses its whole byte, since the row maximum sits just inside the range
//     (a power-of-two scale would leave it between 1/4 and 1/2 of it, one
//     to two bits less per operand);
//   W = 7: digits |d_t| <= 64 taken by successive round-to-nearest of the
//     remainder (each remainder exact in FP64) with weights 2^-(6 + 7 t), 7
//     bits a digit, for larger K.
// Because X is symmetric,
//     (X^2)_ij = sum_k X_ik X_jk ~ s_i s_j sum_{t,u} 2^-(2 e0 + W(t+u)) sum_k d_t[i,k] d_u[j,k],
// i.e. every digit product reads contiguous rows of the digit planes for both
// operands.  Products of planes t, u < S with level L = t + u < NL are kept,
// NL = S (the triangle) or S + 1 (the next level's products of the inner
// planes too: with 8-bit digits this is the accuracy of rounding each
// operand to 8S bits, for S - 1 more products).  Those of one level share an
// int32 accumulator, which is exact: a level has at most S products, and
// W = 8: |acc| <= S 2^14 K < 2^31 by the choice of W; W = 7: |d| <= 64,
// K <= 65536.  Levels are combined in FP64 in the epilogue, which then
// applies the SP2 update exactly like the FP64 product.  The plane count may
// change from product to product (the host picks each launch's), so the
// digit width is a function of (ld, S) that encode and product agree on.
//
// Work layout, storage and staging: see the comments at the kernels.
#include <atomic>
#include <algorithm>

#include "fold.h"
#include "split_internal.h"

namespace sp2 {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ double wred_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wred_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Digit planes are stored blocked: plane t, row i, column j lives in the
// 1 KiB block (i / 32, j / 32) (blocks row-major, ld / 32 per block row), at
// byte (i % 32) * 32 + 16 * (((j / 16) % 2) ^ swz(i % 32)) + j % 16.  One
// block is one MFMA operand fragment for 32 rows and 32 k: a wave stages it
// with one contiguous 16-byte-per-lane load, and the swizzle
// swz(r) = ((r >> 2) ^ (r >> 3)) & 1 makes the fragment reads (lane l: row
// l % 32, k-half l / 32) free of LDS bank conflicts.
__device__ __forceinline__ int dswz(int r) { return ((r >> 2) ^ (r >> 3)) & 1; }

// --------------------------------------------------------------- encoding
// Bits per digit of an S-plane split of operands with K = ld: 8 while every
// level accumulator provably fits int32 (at most S products of |d| <= 128
// per level), else 7.
__host__ __device__ __forceinline__ int digit_bits(int ld, int S) {
    return (long long)S * 16384LL * ld < 2147483648LL ? 8 : 7;
}
// Exponent of the top digit's weight, 2^-e0.
__host__ __device__ __forceinline__ int digit_e0(int W) { return W == 8 ? 7 : 6; }

// Row scale s = (1 + 2^-7) m of a row with maximum m (1 for a zero row) and
// its reciprocal, the factor that maps the row into [-0.993, 0.993] (one
// rounding each: |X_ij| inv <= (1 + 2^-51) / (1 + 2^-7)).  Every encoder
// takes both from here, so they agree bit for bit.
__device__ __forceinline__ double row_scale(double m, double* s_out) {
    const double s = m > 0.0 ? m * 1.0078125 : 1.0;
    if (s_out) *s_out = s;
    return 1.0 / s;
}

// W = 8: m + 0x80..80 (S bytes) for m = rint(y 2^(8S - 1)), |y| <= 0.993 (so
// -0x80..80 <= m < 0x7F..7F80, the range whose excess code has S bytes);
// byte S - 1 - t of it XOR 0x80 is digit t as an int8.
__device__ __forceinline__ unsigned long long excess_digits(double y, int S) {
    const long long m = (long long)rint(y * ldexp(1.0, 8 * S - 1));
    return (unsigned long long)m + (0x8080808080808080ull >> (8 * (8 - S)));
}
__device__ __forceinline__ unsigned excess_digit(unsigned long long u, int S, int t) {
    return (unsigned)((u >> (8 * (S - 1 - t))) & 0xFFull) ^ 0x80u;
}

// Digits of eight values y (|y| <= 0.993) into eight packed bytes per plane.
template <int S>
__device__ __forceinline__ void pack_digits8(double (&y)[8], int W, unsigned long long (&packed)[S]) {
    if (W == 8) {
        unsigned long long u[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) u[q] = excess_digits(y[q], S);
#pragma unroll
        for (int t = 0; t < S; ++t) {
            unsigned long long p = 0ull;
#pragma unroll
            for (int q = 0; q < 8; ++q) p |= (unsigned long long)excess_digit(u[q], S, t) << (8 * q);
            packed[t] = p;
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < S; ++t) {
        const double w = ldexp(1.0, 6 + 7 * t);      // digit weight 2^-(6+7t)
        const double iw = ldexp(1.0, -(6 + 7 * t));
        unsigned long long p = 0ull;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double d = rint(y[q] * w);        // |d| <= 64
            y[q] -= d * iw;                          // exact remainder
            p |= (unsigned long long)(uint8_t)(int8_t)d << (8 * q);
        }
        packed[t] = p;
    }
}

// One wave per padded row: row scale and `slices` digit planes of columns
// [c0, c1) (multiples of 32; the row is zero outside them).
template <int S>
__device__ __forceinline__ void encode_row(const double* __restrict__ X, int ld, int i, int lane, int8_t* __restrict__ digits,
                           double* __restrict__ scale, int c0, int c1) {
    const double* row = X + (size_t)i * ld;
    const int W = digit_bits(ld, S);
    double m = 0.0;
    for (int j = c0 + 8 * lane; j < c1; j += 512) {
        const double4 a = *reinterpret_cast<const double4*>(row + j);
        const double4 b = *reinterpret_cast<const double4*>(row + j + 4);
        m = fmax(m, fmax(fmax(fabs(a.x), fabs(a.y)), fmax(fabs(a.z), fabs(a.w))));
        m = fmax(m, fmax(fmax(fabs(b.x), fabs(b.y)), fmax(fabs(b.z), fabs(b.w))));
    }
    m = wred_max(m);
    double sc;
    const double inv = row_scale(m, &sc);
    if (lane == 0) scale[i] = sc;
    const size_t plane = (size_t)ld * ld;
    const size_t rowblk = (size_t)(i >> 5) * (ld >> 5);
    const int r32 = i & 31;
    for (int j = c0 + 8 * lane; j < c1; j += 512) {
        double y[8];
        const double4 a = *reinterpret_cast<const double4*>(row + j);
        const double4 b = *reinterpret_cast<const double4*>(row + j + 4);
        y[0] = a.x * inv; y[1] = a.y * inv; y[2] = a.z * inv; y[3] = a.w * inv;
        y[4] = b.x * inv; y[5] = b.y * inv; y[6] = b.z * inv; y[7] = b.w * inv;
        const size_t off = (rowblk + (j >> 5)) * 1024 + r32 * 32 + 16 * (((j >> 4) & 1) ^ dswz(r32)) + (j & 15);
        unsigned long long packed[S];
        pack_digits8<S>(y, W, packed);
#pragma unroll
        for (int t = 0; t < S; ++t) *reinterpret_cast<unsigned long long*>(digits + t * plane + off) = packed[t];
    }
}

// One wave per padded row: row scale and `slices` digit planes of X_n.
template <int S>
__global__ __launch_bounds__(256) void k_encode_int8(const double* __restrict__ buf0,
                                                     const double* __restrict__ buf1, int ld,
                                                     const State* __restrict__ st,
                                                     int8_t* __restrict__ digits,
                                                     double* __restrict__ scale) {
    if (st->done || st->phase != 1) return;
    encode_row<S>(st->cur ? buf1 : buf0, ld, blockIdx.x * 4 + (threadIdx.x >> 6), threadIdx.x & 63, digits, scale,
                  0, ld);
}

// One workgroup per padded row, the row held in registers between the max and
// the digit pass (one HBM read of X instead of two).  Thread t takes columns
// 8 t + 2048 c .. +8 for c < CH, so rows up to 2048 CH columns fit.  Blocks
// are mapped to rows XCD-contiguously (block b runs on XCD b % 8 and takes
// row (b % 8) ld / 8 + b / 8), so the four rows whose 32-byte pieces share a
// 128-byte line of a digit block are written through one L2 at nearly the
// same time.  Same digits as encode_row (the row maximum is order-free).
constexpr int ENC_CH = 8;

template <int S>
__global__ __launch_bounds__(256) void k_encode_int8_reg(const double* __restrict__ buf0,
                                                         const double* __restrict__ buf1, int ld,
                                                         const State* __restrict__ st,
                                                         int8_t* __restrict__ digits,
                                                         double* __restrict__ scale) {
    if (st->done || st->phase != 1) return;
    const double* __restrict__ X = st->cur ? buf1 : buf0;
    const int b = blockIdx.x;
    const int i = (b & 7) * (ld >> 3) + (b >> 3);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const double* row = X + (size_t)i * ld;
    double4 va[ENC_CH], vb[ENC_CH];
    double m = 0.0;
#pragma unroll
    for (int c = 0; c < ENC_CH; ++c) {
        const int j = 8 * tid + 2048 * c;
        if (j < ld) {
            va[c] = *reinterpret_cast<const double4*>(row + j);
            vb[c] = *reinterpret_cast<const double4*>(row + j + 4);
            m = fmax(m, fmax(fmax(fabs(va[c].x), fabs(va[c].y)), fmax(fabs(va[c].z), fabs(va[c].w))));
            m = fmax(m, fmax(fmax(fabs(vb[c].x), fabs(vb[c].y)), fmax(fabs(vb[c].z), fabs(vb[c].w))));
        }
    }
    m = wred_max(m);
    __shared__ double wm[4];
    if (lane == 0) wm[w] = m;
    __syncthreads();
    m = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
    double sc;
    const double inv = row_scale(m, &sc);
    if (tid == 0) scale[i] = sc;
    const size_t plane = (size_t)ld * ld;
    const size_t rowblk = (size_t)(i >> 5) * (ld >> 5);
    const int r32 = i & 31;
#pragma unroll
    for (int c = 0; c < ENC_CH; ++c) {
        const int j = 8 * tid + 2048 * c;
        if (j < ld) {
            double y[8] = {va[c].x * inv, va[c].y * inv, va[c].z * inv, va[c].w * inv,
                           vb[c].x * inv, vb[c].y * inv, vb[c].z * inv, vb[c].w * inv};
            const size_t off = (rowblk + (j >> 5)) * 1024 + r32 * 32 + 16 * (((j >> 4) & 1) ^ dswz(r32)) + (j & 15);
            unsigned long long packed[S];
            pack_digits8<S>(y, digit_bits(ld, S), packed);
#pragma unroll
            for (int t = 0; t < S; ++t) *reinterpret_cast<unsigned long long*>(digits + t * plane + off) = packed[t];
        }
    }
}

// Upper-triangle encode.  When the products write only their upper tiles
// (upper-only mode), X_n is valid on and above the diagonal and rmax[i]
// holds max_j |X_ij| as a bit pattern (accumulated by the product that wrote
// X_n).  One workgroup per 32 x 32 block (I, J), I <= J: the block is read
// once and written as digit block (I, J) with the scales of rows I and, read
// back transposed from LDS, as digit block (J, I) with the scales of rows J.
// Same digits as encode_row (same scale, same per-element arithmetic).  The
// diagonal blocks also write the row scales and clear rmax_next, which the
// next product fills.
__device__ __forceinline__ void pack_digits4(const double (&x)[4], double inv, int S, int W, int8_t* __restrict__ out,
                                             size_t plane) {
    double y[4] = {x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv};
    if (W == 8) {
        unsigned long long u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = excess_digits(y[q], S);
        for (int t = 0; t < S; ++t) {
            uint32_t packed = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) packed |= excess_digit(u[q], S, t) << (8 * q);
            *reinterpret_cast<uint32_t*>(out + t * plane) = packed;
        }
        return;
    }
    for (int t = 0; t < S; ++t) {
        const double wt = ldexp(1.0, 6 + 7 * t);
        const double iw = ldexp(1.0, -(6 + 7 * t));
        uint32_t packed = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double d = rint(y[q] * wt);
            y[q] -= d * iw;
            packed |= (uint32_t)(uint8_t)(int8_t)d << (8 * q);
        }
        *reinterpret_cast<uint32_t*>(out + t * plane) = packed;
    }
}

__device__ __forceinline__ double scale_inv(unsigned long long bits, double* s_out) {
    return row_scale(__longlong_as_double((long long)bits), s_out);
}

// Block (I, J), I <= J, at index t of the upper triangle of nb x nb blocks, row-major.
__device__ __forceinline__ void upper_block(int t, int nb, int& I, int& J) {
    I = (int)((2.0 * nb + 1.0 - sqrt((2.0 * nb + 1.0) * (2.0 * nb + 1.0) - 8.0 * (double)t)) / 2.0);
    I = max(0, min(I, nb - 1));
    while (I > 0 && I * nb - I * (I - 1) / 2 > t) --I;
    while (I + 1 < nb && (I + 1) * nb - (I + 1) * I / 2 <= t) ++I;
    J = I + (t - (I * nb - I * (I - 1) / 2));
}

template <int S, bool FOLD>
__global__ __launch_bounds__(256) void k_encode_int8_upper(const double* __restrict__ buf0,
                                                           const double* __restrict__ buf1, int ld,
                                                           const State* __restrict__ st,
                                                           int8_t* __restrict__ digits,
                                                           double* __restrict__ scale,
                                                           unsigned long long* __restrict__ rmax, FoldArgs f) {
    if (!FOLD && (st->done || st->phase != 1)) return;
    __shared__ FoldShared fsh;
    FoldPart fp;
    if (FOLD) fp.load(f);
    const int cur = FOLD ? f.g & 1 : st->cur;
    const double* __restrict__ X = cur ? buf1 : buf0;
    const unsigned long long* __restrict__ rm = rmax + (size_t)cur * ld;
    unsigned long long* __restrict__ rm_next = rmax + (size_t)(1 - cur) * ld;
    const int nb = ld >> 5;
    int I, J;
    upper_block(blockIdx.x, nb, I, J);
    const int tid = threadIdx.x;
    const int r = tid >> 3, c0 = (tid & 7) * 4;
    const size_t plane = (size_t)ld * ld;
    const double4 v = *reinterpret_cast<const double4*>(X + (size_t)(I * 32 + r) * ld + J * 32 + c0);
    const double x[4] = {v.x, v.y, v.z, v.w};
    const unsigned long long mi = rm[I * 32 + r], mj = rm[J * 32 + r];
    if (FOLD) {
        int done, br;
        fold_decide<false>(f, fp, fsh, &done, &br);
        if (done) return;
    }
    double sc;
    const double inv = scale_inv(mi, &sc);
    pack_digits4(x, inv, S, digit_bits(ld, S), digits + ((size_t)I * nb + J) * 1024 + r * 32 + 16 * ((c0 >> 4) ^ dswz(r)) + (c0 & 15),
                 plane);
    if (I == J) {
        if ((tid & 7) == 0) {
            scale[I * 32 + r] = sc;
            rm_next[I * 32 + r] = 0ull;
        }
        return;
    }
    __shared__ double T[32][33];
    T[r][c0] = x[0];
    T[r][c0 + 1] = x[1];
    T[r][c0 + 2] = x[2];
    T[r][c0 + 3] = x[3];
    __syncthreads();
    // row J*32 + r of X, columns I*32 + c0 .. + 3 = column r of the block, rows c0 ..
    const double xt[4] = {T[c0][r], T[c0 + 1][r], T[c0 + 2][r], T[c0 + 3][r]};
    const double invt = scale_inv(mj, nullptr);
    pack_digits4(xt, invt, S, digit_bits(ld, S), digits + ((size_t)J * nb + I) * 1024 + r * 32 + 16 * ((c0 >> 4) ^ dswz(r)) + (c0 & 15),
                 plane);
}

// Grouped: work item = one upper 32 x 32 block of one system, as
// k_encode_int8_upper; fixed grid, grid-stride loop.
template <int S>
__global__ __launch_bounds__(256) void k_encode_int8_grouped(const GroupDesc* __restrict__ g) {
    __shared__ double T[32][33];
    const int total = g->total_blks;
    const int tid = threadIdx.x, r = tid >> 3, c0 = (tid & 7) * 4;
    for (int item = blockIdx.x; item < total; item += gridDim.x) {
        const int s = group_find(g->blk_off, g->nsys, item);
        const SysView& v = g->sys[s];
        const State* st = v.st;
        if (st->done || st->phase != 1) continue;
        const int ld = v.ld, nb = ld >> 5, t = item - g->blk_off[s], cur = st->cur;
        int I, J;
        upper_block(t, nb, I, J);
        const double* __restrict__ X = cur ? v.buf1 : v.buf0;
        const unsigned long long* __restrict__ rm = v.rmax + (size_t)cur * ld;
        unsigned long long* __restrict__ rm_next = v.rmax + (size_t)(1 - cur) * ld;
        const size_t plane = (size_t)ld * ld;
        const double4 x4 = *reinterpret_cast<const double4*>(X + (size_t)(I * 32 + r) * ld + J * 32 + c0);
        const unsigned long long mi = rm[I * 32 + r], mj = rm[J * 32 + r];
        const double x[4] = {x4.x, x4.y, x4.z, x4.w};
        double sc;
        const double inv = scale_inv(mi, &sc);
        const int W = digit_bits(ld, S), off = r * 32 + 16 * ((c0 >> 4) ^ dswz(r)) + (c0 & 15);
        pack_digits4(x, inv, S, W, v.digits + ((size_t)I * nb + J) * 1024 + off, plane);
        if (I == J) {
            if ((tid & 7) == 0) {
                v.scale[I * 32 + r] = sc;
                rm_next[I * 32 + r] = 0ull;
            }
            continue;
        }
        __syncthreads();   // the item before has read T
        T[r][c0] = x[0];
        T[r][c0 + 1] = x[1];
        T[r][c0 + 2] = x[2];
        T[r][c0 + 3] = x[3];
        __syncthreads();
        const double xt[4] = {T[c0][r], T[c0 + 1][r], T[c0 + 2][r], T[c0 + 3][r]};
        pack_digits4(xt, scale_inv(mj, nullptr), S, W, v.digits + ((size_t)J * nb + I) * 1024 + off, plane);
    }
}

// ------------------------------------------------------------------ product
// One 512-thread workgroup per upper-triangular 128 x 128 tile; wave w
// covers rows 32 (w >> 1) .. +32 and columns 64 (w & 1) .. +64 as two 32 x 32
// blocks of v_mfma_i32_32x32x32_i8 per level (NL x 2 accumulators of 16
// int32).  Each K stage stages 2 operands x S planes x 4 row blocks x KS
// k blocks of 1 KiB through an LDS ring in the blocked layout, filled by
// global -> LDS loads one stage ahead of the products.
constexpr int QB = 128;          // tile
constexpr int QK = 32;           // k bytes per block

// K stage: KS blocks of 32 k-bytes; ring depth NST.  Configuration C = 0
// (the default): up to five planes fit a 64-byte stage twice in LDS
// (2 x 80 KiB at five), which halves the barriers per product against
// 32-byte stages; six planes keep 32-byte stages three deep (3 x 48 KiB).
// C = 1: 32-byte stages three deep; C = 2: 32-byte stages four deep (up to
// five planes).  The autotuner picks C per size for dense products.
template <int S, int C = 0> struct I8Stage {
    static constexpr int KS = (C == 0 && S <= 5) ? 2 : 1;
    static constexpr int NST = C == 0 ? (S <= 5 ? 2 : 3) : (C == 1 ? 3 : 4);
    static_assert(NST * 2 * S * 4 * KS <= 160, "stage ring exceeds the LDS");
};
// Configurations valid for S planes.
__host__ __device__ constexpr bool i8_cfg_ok(int S, int C) { return C == 0 || C == 1 || (C == 2 && S <= 5); }

// The staging ring; after the K loop the same LDS holds half of the finished
// tile, transposed, so the mirrored (lower-triangle) copy is written as
// whole rows instead of one 8-byte element per row.  Row stride 129 doubles
// spreads the column-wise LDS stores over the banks.
constexpr int TR_LD = 129;

template <int S, int C = 0>
struct I8Smem {
    union {
        int8_t buf[I8Stage<S, C>::NST][2 * S * 4 * I8Stage<S, C>::KS][1024];   // [stage][((op S + slice) 4 + row block) KS + k block][block]
        double tr[64][TR_LD];                  // [tile column (one half)][tile row]
        struct {
            double xs[128][128];                   // the X_n tile (upper-only mode), staged for the update
            unsigned long long rm[128], cm[128];   // tile row / column maxima (upper-only mode)
            double red[4][8];                      // per-wave partials, after the last use of tr / rm / cm
        } mx;
    };
};

// One 128 x 128 output tile (bi, bj) of one system; all 512 threads of the
// workgroup take part (the body contains barriers).  kmode 0: the whole
// tile; kmode 1: only K stages [kc0, kc1), whose int32 level accumulators are
// stored to chunk_acc (one chunk of a tile split along K); kmode 2: no K
// loop, the accumulators are the sum of the nchunks chunks at chunk_acc (the
// integer sums are exact, so a split tile equals an unsplit one), then the
// epilogue.  Chunk layout: int4 [NL][2][4][512 threads] (accumulator elements
// 4q .. 4q + 3 of level L, column block c), so that each wave moves 1 KiB
// per instruction.  UPPER: write the tile
// only (no mirrored copy below the diagonal) and fold its row and column
// maxima of |X_{n+1}| into rmax_next (bit patterns of non-negative doubles
// order like the values, so atomicMax on them is exact and order-free).
template <int S, int NL, bool THR, bool UPPER, int C = 0>
__device__ __forceinline__ void int8x_tile(double* __restrict__ buf0, double* __restrict__ buf1, int ld,
                           const State* __restrict__ st, const int8_t* __restrict__ digits,
                           const double* __restrict__ scale, double* __restrict__ part, int bi, int bj,
                           I8Smem<S, C>& sm, const int* __restrict__ env,
                           unsigned long long* __restrict__ rmax_next, int kmode = 0, int kc0 = 0,
                           int kc1 = -1, int* __restrict__ chunk_acc = nullptr, int nchunks = 0) {
    const int nt = ld / QB;
    const int t = tri_index(bi, bj, nt);
    const int i0 = bi * QB, j0 = bj * QB;
    const double* __restrict__ Xc = st->cur ? buf1 : buf0;
    double* __restrict__ Xn = st->cur ? buf0 : buf1;
    const size_t plane = (size_t)ld * ld;
    const int nb = ld >> 5;          // blocks per block row

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;

    constexpr int KS = I8Stage<S, C>::KS, NST = I8Stage<S, C>::NST;
    constexpr int NBLK = 2 * S * 4 * KS;        // 1 KiB blocks per stage
    constexpr int PER = NBLK * 64 / 512;        // 16-byte chunks per thread
    static_assert((NBLK * 64) % 512 == 0, "stage must split evenly over 512 threads");

    static_assert(NL == S || NL == S + 1, "levels: the triangle or one more");
    v16i acc[NL][2];
#pragma unroll
    for (int L = 0; L < NL; ++L)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[L][c][r] = 0;

    // fragment address inside a block: row lane % 32, k-half lane / 32
    const int fr = lane & 31;
    const int foff = fr * 32 + 16 * ((lane >> 5) ^ dswz(fr));
    // K stages: all of them (or chunk [kc0, kc1)), or for a thresholded X
    // those holding a 32-column block set in both panels' block masks (the
    // other stages multiply a zero block on one side)
    int ks = 0, nk = ld / (QK * KS);
    if (kc1 >= 0) {
        ks = kc0;
        nk = kc1;
    }
    const int nbk = ld / QK;
    bool holes = false;
    const unsigned long long* mk = THR ? env_mask(env, nt) : nullptr;
    const unsigned long long* mi = THR ? mk + (size_t)bi * mask_words(ld) : nullptr;
    const unsigned long long* mj = THR ? mk + (size_t)bj * mask_words(ld) : nullptr;
    if (THR) {
        // the stages between the first and the last common block; when some
        // stage in between has none (the blocks are scattered, not banded),
        // the loop below visits the working stages only
        const unsigned long long mword = common_mask_word(mi, mj, nbk);
        // per lane: stages of its word holding a common block (KS divides
        // 64, so no stage straddles two words) and its last common block;
        // then the wave's sum and maximum
        int stages = 0, b1 = -1;
        if (mword) {
            unsigned long long m = mword;
            if (KS == 2) m = (m | (m >> 1)) & 0x5555555555555555ull;
            stages = __popcll(m);
            b1 = (lane << 6) + 63 - __builtin_clzll(mword);
        }
        for (int o = 32; o > 0; o >>= 1) {
            stages += __shfl_xor(stages, o, 64);
            b1 = max(b1, __shfl_xor(b1, o, 64));
        }
        if (b1 < 0) {
            ks = nk = 0;
        } else {
            ks = next_block_in_wave(mword, 0, nbk) / KS;
            nk = b1 / KS + 1;
            holes = stages < nk - ks;
        }
    }

    // Fragment reads are written in order of first use (B plane 0, the A
    // planes, B planes 1 ..), the products in level order, and the scheduler
    // is held to a pattern of one read per two products that keeps every
    // read LA product pairs ahead of its first use, so a stage starts after
    // 3 + LA reads instead of the whole set.
    auto compute = [&](int stg) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            auto rdA = [&](int sl) {
                return *reinterpret_cast<const v4i*>(&sm.buf[stg][(sl * 4 + wr) * KS + kk][foff]);
            };
            auto rdB = [&](int uu, int c) {
                return *reinterpret_cast<const v4i*>(&sm.buf[stg][(S * 4 + uu * 4 + wc * 2 + c) * KS + kk][foff]);
            };
            v4i a[S], b[S][2];
            b[0][0] = rdB(0, 0);
            b[0][1] = rdB(0, 1);
#pragma unroll
            for (int tt = 0; tt < S; ++tt) a[tt] = rdA(tt);
#pragma unroll
            for (int uu = 1; uu < S; ++uu) {
                b[uu][0] = rdB(uu, 0);
                b[uu][1] = rdB(uu, 1);
            }
            // level tt + uu accumulates a[tt] b[uu]
#pragma unroll
            for (int uu = 0; uu < S; ++uu)
#pragma unroll
                for (int tt = 0; tt < S && tt < NL - uu; ++tt)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[tt + uu][c] =
                            __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tt], b[uu][c], acc[tt + uu][c], 0, 0, 0);
        }
        constexpr int LA = 2;                                  // lookahead in reads
        constexpr int R = 3 * S * KS, P = (S * (S + 1) / 2 + (NL - S) * (S - 1)) * KS;   // reads, product pairs
        constexpr int MID = R - 3 - LA;
        __builtin_amdgcn_sched_group_barrier(0x100, 3 + LA, 0);
#pragma unroll
        for (int q = 0; q < MID; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * (P - MID), 0);
    };
    // Global -> LDS loads without register staging: wave w moves blocks w,
    // w + 8, ... of a stage, one 1 KiB block per instruction (16 bytes per
    // lane).  Stage kt + NST - 1 is issued while stage kt is multiplied;
    // before reading stage kt a wave waits for its own loads of stage kt (at
    // most the PER loads of stage kt + 1 stay outstanding in a three-deep
    // ring), and a barrier then makes every wave's blocks visible.
    auto issue = [&](int kb, int stg) {
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const int blk = w + 8 * m;
            const int kk = blk % KS, ob = blk / KS;
            const int op = ob / (S * 4);
            const int rem = ob - op * (S * 4);
            const int sl = rem >> 2, rb = rem & 3;
            const int grb = ((op ? j0 : i0) >> 5) + rb;
            const int8_t* g = digits + sl * plane + ((size_t)grb * nb + kb * KS + kk) * 1024 + 16 * lane;
            __builtin_amdgcn_global_load_lds((const void*)g,
                                             (__attribute__((address_space(3))) void*)&sm.buf[stg][blk][0], 16, 0, 0);
        }
    };
    if (kmode == 2) nk = ks;          // accumulators come from the chunks
    if (!holes) {
        // every stage of [ks, nk) works: a plain loop
        for (int q = 0; q < NST - 1; ++q)
            if (ks + q < nk) issue(ks + q, q);
        for (int kt = ks; kt < nk; ++kt) {
            // this wave's blocks of stage kt have landed in LDS once only
            // stage kt + 1's loads (three-deep ring) or none (two-deep) are
            // outstanding; the bare barrier (no fence, which would wait for
            // every outstanding load) then covers the other waves' blocks, and
            // every wave has finished reading the buffer that stage
            // kt + NST - 1 overwrites
            if (NST == 4 && kt + 2 < nk) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * PER));   // vmcnt(2 PER)
            else if (NST >= 3 && kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0F70 | PER);   // vmcnt(PER)
            else __builtin_amdgcn_s_waitcnt(0x0F70);                                      // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            if (kt + NST - 1 < nk) issue(kt + NST - 1, (kt + NST - 1 - ks) % NST);
            compute((kt - ks) % NST);
        }
    }
    // with holes: the working stages in increasing order go round the ring:
    // ic is the next stage to issue, n_iss / n_done count stages issued /
    // multiplied (the common mask is reloaded here, so that it is not live
    // across the plain loop)
    const unsigned long long mword = (THR && holes) ? common_mask_word(mi, mj, nbk) : 0ull;
    auto next_stage = [&](int s) -> int {      // first working stage >= s, or nk
        const int b = next_block_in_wave(mword, s * KS, nbk);
        return b >= nbk ? nk : b / KS;
    };
    int ic = holes ? next_stage(ks) : nk, n_iss = 0, n_done = 0;
    while (n_iss < NST - 1 && ic < nk) {
        issue(ic, n_iss % NST);
        ++n_iss;
        ic = next_stage(ic + 1);
    }
    while (n_done < n_iss) {
        // this wave's blocks of the stage in ring slot n_done have landed in
        // LDS once only the next stage's loads (three-deep ring) or none
        // (two-deep) are outstanding; the bare barrier (no fence, which would
        // wait for every outstanding load) then covers the other waves'
        // blocks, and every wave has finished reading the slot that the next
        // issue overwrites
        if (NST == 4 && n_iss - n_done == 3) __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * PER));   // vmcnt(2 PER)
        else if (NST >= 3 && n_iss - n_done >= 2) __builtin_amdgcn_s_waitcnt(0x0F70 | PER);   // vmcnt(PER)
        else __builtin_amdgcn_s_waitcnt(0x0F70);                                              // vmcnt(0)
        __builtin_amdgcn_s_barrier();
        if (ic < nk) {
            issue(ic, n_iss % NST);
            ++n_iss;
            ic = next_stage(ic + 1);
        }
        compute(n_done % NST);
        ++n_done;
    }
    __syncthreads();
    constexpr int CH = NL * 2 * 16 * 512;   // int32 per chunk
    if (kmode == 1) {
        int4* out = reinterpret_cast<int4*>(chunk_acc);
#pragma unroll
        for (int L = 0; L < NL; ++L)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    out[((L * 2 + c) * 4 + q) * 512 + tid] =
                        make_int4(acc[L][c][4 * q], acc[L][c][4 * q + 1], acc[L][c][4 * q + 2], acc[L][c][4 * q + 3]);
        return;
    }
    if (kmode == 2) {
        for (int ch = 0; ch < nchunks; ++ch) {
            const int4* in = reinterpret_cast<const int4*>(chunk_acc + (size_t)ch * CH);
#pragma unroll
            for (int L = 0; L < NL; ++L)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int4 v = in[((L * 2 + c) * 4 + q) * 512 + tid];
                        acc[L][c][4 * q] += v.x;
                        acc[L][c][4 * q + 1] += v.y;
                        acc[L][c][4 * q + 2] += v.z;
                        acc[L][c][4 * q + 3] += v.w;
                    }
        }
    }

    if constexpr (UPPER) {
        // the X_n tile to LDS in one burst (16 rows of 1 KiB per wave, all in
        // flight at once) instead of dependent global loads inside the
        // update; the ring is free once every wave is past its last stage
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int row = w + 8 * m;
            __builtin_amdgcn_global_load_lds((const void*)(Xc + (size_t)(i0 + row) * ld + j0 + 2 * lane),
                                             (__attribute__((address_space(3))) void*)&sm.mx.xs[row][0], 16, 0, 0);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        __syncthreads();
    }
    // epilogue: combine levels in FP64, apply the SP2 update, partials.
    // Partial sums are kept per column block c in row order and added at the
    // end, the same order in both layouts (so both give identical partials).
    const int br = st->branch;
    const bool mirror = bi != bj;
    const int W = digit_bits(ld, S), E2 = 2 * digit_e0(W);
    double trc[2] = {0.0, 0.0}, froc[2] = {0.0, 0.0}, idmc[2] = {0.0, 0.0};
    auto element = [&](int c, int r, int gi, int gj, double sj) -> double {
        double v = 0.0;
#pragma unroll
        for (int L = NL - 1; L >= 0; --L) v += ldexp((double)acc[L][c][r], -(E2 + W * L));
        // s_i s_j first: the product is then the same for (i, j) and (j, i)
        // (the diagonal tiles form both), so X stays exactly symmetric
        double p = v * (scale[gi] * sj);
        // p rounded once for every use, as in the 64 x 64 tile
        if constexpr (!UPPER) asm("" : "+v"(p));
        const double x = UPPER ? sm.mx.xs[gi - i0][gj - j0] : Xc[(size_t)gi * ld + gj];
        const double xn = br ? 2.0 * x - p : p;
        Xn[(size_t)gi * ld + gj] = xn;
        if (gi == gj) trc[c] += xn;
        froc[c] += xn * xn;
        idmc[c] += (p - x) * (p - x);
        return xn;
    };
    // v_mfma_i32_32x32x32_i8 result: lane l, element r is row 8 (r/4) + 4 (l/32) + r%4, column l%32
    auto row_of = [&](int r) { return i0 + wr * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
    if (UPPER) {
        // tile row and column maxima are combined in LDS, then one global
        // atomic per row (and per column off the diagonal) of the tile
        if (tid < 128) sm.mx.rm[tid] = 0ull;
        else if (tid < 256) sm.mx.cm[tid - 128] = 0ull;
        __syncthreads();
        const int gj0 = j0 + wc * 64 + (lane & 31), gj1 = gj0 + 32;
        const double sj0 = scale[gj0], sj1 = scale[gj1];
        double cmx0 = 0.0, cmx1 = 0.0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int gi = row_of(r);
            const double a = fabs(element(0, r, gi, gj0, sj0));
            const double b = fabs(element(1, r, gi, gj1, sj1));
            cmx0 = fmax(cmx0, a);
            cmx1 = fmax(cmx1, b);
            // row maximum over the wave's 64 columns (32 lanes of this half)
            double m = fmax(a, b);
            for (int o = 16; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
            if ((lane & 31) == 0) atomicMax(&sm.mx.rm[gi - i0], (unsigned long long)__double_as_longlong(m));
        }
        if (mirror) {
            // column maxima over the wave's 32 rows: row maxima of rows gj over
            // these columns of their lower part (a diagonal tile is symmetric)
            cmx0 = fmax(cmx0, __shfl_xor(cmx0, 32, 64));
            cmx1 = fmax(cmx1, __shfl_xor(cmx1, 32, 64));
            if (lane < 32) {
                atomicMax(&sm.mx.cm[gj0 - j0], (unsigned long long)__double_as_longlong(cmx0));
                atomicMax(&sm.mx.cm[gj1 - j0], (unsigned long long)__double_as_longlong(cmx1));
            }
        }
        __syncthreads();
        if (tid < 128) atomicMax(rmax_next + i0 + tid, sm.mx.rm[tid]);
        else if (mirror && tid < 256) atomicMax(rmax_next + j0 + tid - 128, sm.mx.cm[tid - 128]);
    } else {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int gj = j0 + wc * 64 + c * 32 + (lane & 31);
            const double sj = scale[gj];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int gi = row_of(r);
                const double xn = element(c, r, gi, gj, sj);
                if (mirror) sm.tr[wc * 32 + (lane & 31)][gi - i0] = xn;
            }
            if (mirror) {
                // columns j0 + 64 wc' + 32 c + (0..31) of every wave: 64 rows of
                // the mirrored block, 128 doubles each, written one half row per
                // wave and instruction
                __syncthreads();
#pragma unroll 4
                for (int q = 0; q < 16; ++q) {
                    const int rh = w + 8 * q;
                    const int jj = rh >> 1, col = (rh & 1) * 64 + lane;
                    const int gr = j0 + (jj >> 5) * 64 + c * 32 + (jj & 31);
                    Xn[(size_t)gr * ld + i0 + col] = sm.tr[jj][col];
                }
                __syncthreads();
            }
        }
    }
    double tr = trc[0] + trc[1], fro = froc[0] + froc[1], idm = UPPER ? idmc[0] + idmc[1] : idmc[0];
    tr = wred_sum(tr);
    fro = wred_sum(fro);
    idm = wred_sum(idm);
    const double idm1 = UPPER ? 0.0 : wred_sum(idmc[1]);
    double (*red)[8] = sm.mx.red;
    if (lane == 0) {
        red[0][w] = tr;
        red[1][w] = fro;
        red[2][w] = idm;
        red[3][w] = idm1;
    }
    __syncthreads();
    if (tid == 0) {
        const double wgt = mirror ? 2.0 : 1.0;
        for (int q = 0; q < (UPPER ? 3 : 2); ++q)
            part[3 * t + q] = (q ? wgt : 1.0) * (((red[q][0] + red[q][1]) + (red[q][2] + red[q][3])) +
                                                 ((red[q][4] + red[q][5]) + (red[q][6] + red[q][7])));
        if (!UPPER) {
            // by 32 x 32 blocks within 64 x 64 quadrants, the order of the
            // work-list product on 64 x 64 tiles (the lower quadrant of a
            // diagonal tile counted as the upper one's mirror)
            auto quad = [&](int qr, int qc) {
                const int a = 4 * qr + qc, b = a + 2;
                return (red[2][a] + red[3][a]) + (red[2][b] + red[3][b]);
            };
            part[3 * t + 2] = mirror ? (2.0 * quad(0, 0) + 2.0 * quad(0, 1)) + (2.0 * quad(1, 0) + 2.0 * quad(1, 1))
                                     : (quad(0, 0) + 2.0 * quad(0, 1)) + (0.0 + quad(1, 1));
        }
    }
}

// Workgroups [0, t_full): whole tiles at visiting positions [0, t_full),
// dealt over the XCDs.  Workgroups from t_full on: the tiles at positions
// t_full, t_full + 1, ... (the last, partly filled wave of a launch), each
// split into nsplit chunks of the K loop whose accumulators go to chunk_acc;
// k_gemm_int8x_tail finishes them.
//
// THR: tiles are visited diagonal by diagonal (bj - bi = 0, 1, ..), so the
// tiles of a banded X, the only ones with a K range, are the first ones
// dispatched and spread over every CU (the XCD-dealt super-tile order would
// put most of them on the XCDs that take the short rows near the end of the
// triangle); tile_group does not apply.
// Tile at position pos of the diagonal-major order of the upper triangle of
// nt x nt tiles: diagonal d starts at d nt - d (d - 1) / 2.
__device__ __forceinline__ void diag_tile(int pos, int nt, int& bi, int& bj) {
    const double b = 2.0 * nt + 1.0;
    int d = (int)((b - sqrt(b * b - 8.0 * pos)) * 0.5);
    auto start = [nt](int e) { return e * nt - e * (e - 1) / 2; };
    while (d > 0 && start(d) > pos) --d;
    while (d + 1 < nt && start(d + 1) <= pos) ++d;
    bi = pos - start(d);
    bj = bi + d;
}

template <int S, int NL, bool THR, bool UPPER, int C = 0>
__global__ __launch_bounds__(512) void k_gemm_int8x(double* __restrict__ buf0, double* __restrict__ buf1,
                                                    int ld, const State* __restrict__ st,
                                                    const int8_t* __restrict__ digits,
                                                    const double* __restrict__ scale,
                                                    double* __restrict__ part, const int* __restrict__ env,
                                                    unsigned long long* __restrict__ rmax, int tile_group,
                                                    int t_full, int nsplit, int* __restrict__ chunk_acc,
                                                    int when_full) {
    if (st->done || st->phase != 1 || (when_full && !st->full_fill)) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem<S, C>& sm = *reinterpret_cast<I8Smem<S, C>*>(smem_raw);
    const int nt = ld / QB, w = blockIdx.x;
    int pos, kmode = 0, kc0 = 0, kc1 = -1;
    int* cacc = nullptr;
    if (THR) {
        pos = w;
    } else if (w < t_full) {
        pos = xcd_deal(w, t_full);
    } else {
        const int j = w - t_full, p = j / nsplit, ch = j - p * nsplit, nk = ld / (QK * I8Stage<S, C>::KS);
        pos = t_full + p;
        kmode = 1;
        kc0 = ch * nk / nsplit;
        kc1 = (ch + 1) * nk / nsplit;
        cacc = chunk_acc + (size_t)j * (NL * 2 * 16 * 512);
    }
    int bi, bj;
    if (THR) diag_tile(pos, nt, bi, bj);
    else order_tile(pos, nt, tile_group, bi, bj);
    int8x_tile<S, NL, THR, UPPER, C>(buf0, buf1, ld, st, digits, scale, part, bi, bj, sm, env,
                              UPPER ? rmax + (size_t)(1 - st->cur) * ld : nullptr, kmode, kc0, kc1, cacc, 0);
}

// ---- 64 x 64 output tiles (dense upper-only products of small and middle N)
//
// With 128 x 128 tiles a product of N = 720 has 21 workgroups for 256 CUs, and
// each walks its K loop and its epilogue alone.  Here one 256-thread workgroup
// covers an upper 64 x 64 tile; wave w its 32 x 32 block (w >> 1, w & 1) with
// NL accumulators of 16 int32, so two workgroups share a CU and one's epilogue
// runs beside the other's products.  The digit sums are exact and the
// epilogue's arithmetic per element is that of int8x_tile, so X_{n+1} and its
// row maxima are the same bit for bit.  4 planes, 5 levels, per product (encode
// included): N = 256 24 -> 11 us, 720 40 -> 17, 1024 48 -> 20, 1536 65 -> 37,
// 2048 81 -> 74, 3072 232 -> 174.  What bounds it at N = 2048: alone, the loads
// take 37 us (553 MB from L2 at 15 TB/s), the MFMAs 40 us (528 tiles on 256 CUs,
// three on some) and the LDS reads and writes about 30 us of the same LDS; a
// deeper ring or 32-k stages changed nothing.  Above N = 3400 the operand
// traffic, twice that of 128 x 128 tiles, costs more than the balance gives.
constexpr int QT = 64;
static_assert(kGroupTile == QT, "grouped products run this tile");

template <int S> struct I8Stage64 {
    static constexpr int KS = S <= 5 ? 2 : 1;    // 32-k blocks per stage
    static constexpr int NST = S <= 5 ? 2 : 3;   // ring depth
    static constexpr int NBLK = 2 * S * 2 * KS;    // 1 KiB blocks per stage
    static constexpr int PER = NBLK / 4;           // blocks per wave
};

template <int S>
struct I8Smem64 {
    union {
        int8_t buf[I8Stage64<S>::NST][I8Stage64<S>::NBLK][1024];   // [stage][((op S + plane) 2 + row block) KS + k block]
        struct {
            double ax[QT][QT + 1];                 // |X_{n+1}| of the tile, for its row and column maxima
            double red[3][4];
        } e;
    };
};

//
// THR: quadrant th.q of a 128 x 128 tile of a thresholded X: K stages with a
// 32-column block set in both masks (of the tile's two row panels) only; the
// threshold is applied here, by the wave to its block, with the sums in the
// order of threshold_tile; the mirrored copy is written too, rmax_next is not
// used, and of the partials only the idempotency one is written, to
// part[slot], beside what k_tile_finish needs of each block.
struct Thr64 {
    const unsigned long long* mi;
    const unsigned long long* mj;
    double tau;
    int elem;
    double* blk;    // of the 128 x 128 tile: ||block||_F^2 of its 16 blocks, -1 where dropped
    double* tr;     // of a diagonal tile: traces of its 4 diagonal blocks
    int q;
    bool diag;      // the 128 x 128 tile is a diagonal one
    bool x_zero;    // X_n is zero here whatever its memory holds
};

template <int S, int NL, bool THR = false>
__device__ __forceinline__ void int8x_tile64(double* __restrict__ buf0, double* __restrict__ buf1, int ld,
                                             const State* __restrict__ st, const int8_t* __restrict__ digits,
                                             const double* __restrict__ scale, double* __restrict__ part, int bi,
                                             int bj, I8Smem64<S>& sm, unsigned long long* __restrict__ rmax_next,
                                             int slot, const Thr64& th = {}) {
    using G = I8Stage64<S>;
    constexpr int KS = G::KS, NST = G::NST, PER = G::PER;
    static_assert(NL == S || NL == S + 1, "levels: the triangle or one more");
    static_assert(G::NBLK % 4 == 0, "stage must split evenly over 4 waves");
    const int i0 = bi * QT, j0 = bj * QT;
    const double* __restrict__ Xc = st->cur ? buf1 : buf0;
    double* __restrict__ Xn = st->cur ? buf0 : buf1;
    const size_t plane = (size_t)ld * ld;
    const int nb = ld >> 5;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;

    v16i acc[NL];
#pragma unroll
    for (int L = 0; L < NL; ++L)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[L][r] = 0;
    const int fr = lane & 31;
    const int foff = fr * 32 + 16 * ((lane >> 5) ^ dswz(fr));

    auto compute = [&](int stg) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            v4i a[S], b[S];
            b[0] = *reinterpret_cast<const v4i*>(&sm.buf[stg][(S * 2 + wc) * KS + kk][foff]);
#pragma unroll
            for (int tt = 0; tt < S; ++tt)
                a[tt] = *reinterpret_cast<const v4i*>(&sm.buf[stg][(tt * 2 + wr) * KS + kk][foff]);
#pragma unroll
            for (int uu = 1; uu < S; ++uu)
                b[uu] = *reinterpret_cast<const v4i*>(&sm.buf[stg][(S * 2 + uu * 2 + wc) * KS + kk][foff]);
#pragma unroll
            for (int uu = 0; uu < S; ++uu)
#pragma unroll
                for (int tt = 0; tt < S && tt < NL - uu; ++tt)
                    acc[tt + uu] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[tt], b[uu], acc[tt + uu], 0, 0, 0);
        }
        constexpr int LA = 2;                                  // lookahead in reads
        constexpr int R = 2 * S * KS, P = (S * (S + 1) / 2 + (NL - S) * (S - 1)) * KS;
        constexpr int MID = R - 2 - LA < P ? R - 2 - LA : P;
        __builtin_amdgcn_sched_group_barrier(0x100, 2 + LA, 0);
#pragma unroll
        for (int q = 0; q < MID; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, P - MID, 0);
    };
    auto issue = [&](int kb, int stg) {
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const int blk = w + 4 * m;
            const int kk = blk % KS, ob = blk / KS;
            const int op = ob / (S * 2);
            const int rem = ob - op * (S * 2);
            const int sl = rem >> 1, rb = rem & 1;
            const int grb = ((op ? j0 : i0) >> 5) + rb;
            const int8_t* g = digits + sl * plane + ((size_t)grb * nb + kb * KS + kk) * 1024 + 16 * lane;
            __builtin_amdgcn_global_load_lds((const void*)g,
                                             (__attribute__((address_space(3))) void*)&sm.buf[stg][blk][0], 16, 0, 0);
        }
    };
    const int nk = ld / (QK * KS);
    if constexpr (THR) {
        const unsigned long long mword = common_mask_word(th.mi, th.mj, nb);
        auto next_stage = [&](int s) -> int {      // first working stage >= s, or nk
            const int b = next_block_in_wave(mword, s * KS, nb);
            return b >= nb ? nk : b / KS;
        };
        int ic = next_stage(0), n_iss = 0, n_done = 0;
        while (n_iss < NST - 1 && ic < nk) {
            issue(ic, n_iss % NST);
            ++n_iss;
            ic = next_stage(ic + 1);
        }
        while (n_done < n_iss) {
            if (NST >= 3 && n_iss - n_done >= 2) __builtin_amdgcn_s_waitcnt(0x0F70 | PER);   // vmcnt(PER)
            else __builtin_amdgcn_s_waitcnt(0x0F70);                                         // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            if (ic < nk) {
                issue(ic, n_iss % NST);
                ++n_iss;
                ic = next_stage(ic + 1);
            }
            compute(n_done % NST);
            ++n_done;
        }
    } else {
        for (int q = 0; q < NST - 1; ++q)
            if (q < nk) issue(q, q);
        for (int kt = 0; kt < nk; ++kt) {
            // as in int8x_tile: this wave's blocks of stage kt have landed, the
            // barrier covers the other waves'
            if (NST >= 3 && kt + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0F70 | PER);   // vmcnt(PER)
            else __builtin_amdgcn_s_waitcnt(0x0F70);                                 // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            if (kt + NST - 1 < nk) issue(kt + NST - 1, (kt + NST - 1) % NST);
            compute(kt % NST);
        }
    }

    const int br = st->branch;
    const bool mirror = bi != bj;
    const int W = digit_bits(ld, S), E2 = 2 * digit_e0(W);
    const int gj = j0 + wc * 32 + (lane & 31);
    auto row_of = [&](int r) { return wr * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };
    // X_n of the wave's block and the row scales in one burst
    double x[16], si[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        x[r] = THR && th.x_zero ? 0.0 : Xc[(size_t)(i0 + row_of(r)) * ld + gj];
        si[r] = scale[i0 + row_of(r)];
    }
    const double sj = scale[gj];
    double tr = 0.0, fro = 0.0, idm = 0.0;
    __syncthreads();   // every wave is past the ring, which ax overlays
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int gi = i0 + row_of(r);
        double v = 0.0;
#pragma unroll
        for (int L = NL - 1; L >= 0; --L) v += ldexp((double)acc[L][r], -(E2 + W * L));
        double p = v * (si[r] * sj);
        if constexpr (THR) asm("" : "+v"(p));
        const double xn = br ? 2.0 * x[r] - p : p;
        if constexpr (!THR) {
            Xn[(size_t)gi * ld + gj] = xn;
            if (gi == gj) tr += xn;
            fro += xn * xn;
        }
        idm += (p - x[r]) * (p - x[r]);
        sm.e.ax[row_of(r)][wc * 32 + (lane & 31)] = THR ? xn : fabs(xn);
    }
    if constexpr (!THR) {
        tr = wred_sum(tr);
        fro = wred_sum(fro);
    }
    idm = wred_sum(idm);
    if (lane == 0) {
        if constexpr (!THR) {
            sm.e.red[0][w] = tr;
            sm.e.red[1][w] = fro;
        }
        sm.e.red[2][w] = idm;
    }
    __syncthreads();
    if constexpr (THR) {
        // the wave's block row by row, and transposed
        const int rb = wr * 32, cb = wc * 32, R = 2 * (th.q >> 1) + wr, C = 2 * (th.q & 1) + wc;
        auto threshold = [&](double v[16]) -> double {   // ||block||^2, -1 if dropped
            double ss = 0.0;
            bool nz = false;
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                if (th.elem && fabs(v[m]) < th.tau) v[m] = 0.0;
                nz = nz || v[m] != 0.0;
                ss += v[m] * v[m];
            }
            ss = wred_sum(ss);
            if (th.elem ? __any(nz) : ss >= th.tau * th.tau) return ss;
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = 0.0;
            return -1.0;
        };
        const int r0 = lane >> 5, c = lane & 31;   // element m of lane l is (r0 + 2 m, c)
        double v[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) v[m] = sm.e.ax[rb + r0 + 2 * m][cb + c];
        const double ss = threshold(v);
        if (lane == 0) th.blk[4 * R + C] = ss;
#pragma unroll
        for (int m = 0; m < 16; ++m) Xn[(size_t)(i0 + rb + r0 + 2 * m) * ld + j0 + cb + c] = v[m];
        if (th.diag && R == C) {
            double t = 0.0;
#pragma unroll
            for (int m = 0; m < 16; ++m)
                if (r0 + 2 * m == c) t += v[m];
            t = wred_sum(t);
            if (lane == 0) th.tr[R] = t;   // 0 if dropped
        }
        if (mirror) {
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = sm.e.ax[rb + c][cb + r0 + 2 * m];
            if (th.diag) {
                // a block of the diagonal tile's lower half: its own sum
                const double st2 = threshold(v);
                if (lane == 0) th.blk[4 * C + R] = st2;
            } else {
#pragma unroll
                for (int m = 0; m < 16; ++m)
                    if (th.elem ? fabs(v[m]) < th.tau : ss == -1.0) v[m] = 0.0;
            }
#pragma unroll
            for (int m = 0; m < 16; ++m) Xn[(size_t)(j0 + cb + r0 + 2 * m) * ld + i0 + rb + c] = v[m];
        }
        if (tid == 0)
            part[slot] = (mirror ? 2.0 : 1.0) *
                         ((sm.e.red[2][0] + sm.e.red[2][1]) + (sm.e.red[2][2] + sm.e.red[2][3]));
        return;
    }
    // row maxima: four lanes per row, 16 columns each; column maxima the same
    // way off the diagonal (a diagonal tile is symmetric)
    {
        const int q = tid & 3, l = tid >> 2;
        double m = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) m = fmax(m, sm.e.ax[l][q + 4 * k]);
        m = fmax(m, __shfl_xor(m, 1, 64));
        m = fmax(m, __shfl_xor(m, 2, 64));
        if (q == 0) atomicMax(rmax_next + i0 + l, (unsigned long long)__double_as_longlong(m));
        if (mirror) {
            double c = 0.0;
            const int col = tid & 63, r0 = (tid >> 6) * 16;
#pragma unroll
            for (int k = 0; k < 16; ++k) c = fmax(c, sm.e.ax[r0 + k][col]);
            atomicMax(rmax_next + j0 + col, (unsigned long long)__double_as_longlong(c));
        }
    }
    if (tid == 0) {
        const int t = slot;
        const double wgt = mirror ? 2.0 : 1.0;
        part[3 * t + 0] = (sm.e.red[0][0] + sm.e.red[0][1]) + (sm.e.red[0][2] + sm.e.red[0][3]);
        part[3 * t + 1] = wgt * ((sm.e.red[1][0] + sm.e.red[1][1]) + (sm.e.red[1][2] + sm.e.red[1][3]));
        part[3 * t + 2] = wgt * ((sm.e.red[2][0] + sm.e.red[2][1]) + (sm.e.red[2][2] + sm.e.red[2][3]));
    }
}

template <int S, int NL>
__global__ __launch_bounds__(256, 2) void k_gemm_int8x_t64(double* __restrict__ buf0, double* __restrict__ buf1,
                                                           int ld, const State* __restrict__ st,
                                                           const int8_t* __restrict__ digits,
                                                           const double* __restrict__ scale,
                                                           double* __restrict__ part,
                                                           unsigned long long* __restrict__ rmax, int tile_group) {
    if (st->done || st->phase != 1) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem64<S>& sm = *reinterpret_cast<I8Smem64<S>*>(smem_raw);
    int bi, bj;
    tile_of_block(blockIdx.x, ld / QT, tile_group, bi, bj);
    int8x_tile64<S, NL>(buf0, buf1, ld, st, digits, scale, part, bi, bj, sm, rmax + (size_t)(1 - st->cur) * ld,
                        tri_index(bi, bj, ld / QT));
}

// The 128 x 128 tiles of a last round that would leave at least half of the CUs
// idle (visiting positions t_full .. T - 1), as four 64 x 64 tiles each: sub-tile
// 0 takes the tile's partial slot, the others slots from T on; the one below
// the diagonal of a diagonal tile has none of the sums.  Against K chunks with
// a sum and an epilogue launch behind them, per product with its encode (4
// planes, 5 levels): N = 4096 (16 tiles left of 528) 413 -> 394 us, 4224 (33 of
// 561) 438 -> 408.
template <int S, int NL>
__global__ __launch_bounds__(256, 2) void k_gemm_int8x_left(double* __restrict__ buf0, double* __restrict__ buf1,
                                                            int ld, const State* __restrict__ st,
                                                            const int8_t* __restrict__ digits,
                                                            const double* __restrict__ scale,
                                                            double* __restrict__ part,
                                                            unsigned long long* __restrict__ rmax, int tile_group,
                                                            int t_full) {
    if (st->done || st->phase != 1) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem64<S>& sm = *reinterpret_cast<I8Smem64<S>*>(smem_raw);
    const int nt = ld / QB, p = blockIdx.x >> 2, sub = blockIdx.x & 3;
    int bi, bj;
    order_tile(t_full + p, nt, tile_group, bi, bj);
    const int slot = sub == 0 ? tri_index(bi, bj, nt) : nt * (nt + 1) / 2 + 3 * p + sub - 1;
    if (bi == bj && sub == 2) {
        if (threadIdx.x < 3) part[3 * slot + threadIdx.x] = 0.0;
        return;
    }
    int8x_tile64<S, NL>(buf0, buf1, ld, st, digits, scale, part, 2 * bi + (sub >> 1), 2 * bj + (sub & 1), sm,
                        rmax + (size_t)(1 - st->cur) * ld, slot);
}

// order_tile with one step per super-tile row instead of one per super-tile
// (the list kernel maps every tile of the triangle): the same tile for
// every position.
__device__ __forceinline__ void order_tile_rows(int t, int nt, int G, int& bi, int& bj) {
    if (G <= 0 || G > nt) G = nt;
    int I = 0, gi = min(G, nt);
    for (;;) {
        gi = min(G, nt - I * G);
        const int row = gi * (gi + 1) / 2 + gi * (nt - I * G - gi);
        if (t < row || I * G + gi >= nt) break;
        t -= row;
        ++I;
    }
    const int d = gi * (gi + 1) / 2;
    if (t < d) {
        int li = 0, off = 0;
        while (t >= off + (gi - li)) { off += gi - li; ++li; }
        bi = I * G + li;
        bj = I * G + li + (t - off);
        return;
    }
    t -= d;
    const int J = I + 1 + t / (gi * G);
    t -= (J - I - 1) * gi * G;
    const int gj = min(G, nt - J * G);
    bi = I * G + t / gj;
    bj = J * G + t % gj;
}

// ---- thresholded products driven by a work list (int8 from the first product on)
//
// Zero-tile flags tz (one row of T upper tiles per X buffer, kept with the
// threshold pass; a flagged tile is zero whatever its memory holds): a tile
// whose K range is empty and whose X_n tile is all zero has X_{n+1} = 0 there
// under either branch.  k_tile_list visits the tiles in the product's G x G
// super-tile order; such a tile gets its flag and zero partials, every other
// tile is listed for the product.  The list holds (bi << 15) | bj; list_ctr[0]
// counts entries (both counters cleared by the encode), list_ctr[1] hands them
// out in list order, so whatever the order the work is balanced, and
// concurrent workgroups work on nearby tiles that share row panels.  Also
// empties the ranges and masks env_next, which the threshold pass behind the
// product fills (nobody reads them in between).  The first product of a banded
// N = 16384, which stored zeros to 2 GB of the other buffer: 485 -> 96 us.
__global__ __launch_bounds__(256) void k_tile_list(const State* __restrict__ st, const int* __restrict__ env,
                                                   int* __restrict__ env_next, int* __restrict__ tz, int nt,
                                                   int tile_group, double* __restrict__ part, int* __restrict__ list,
                                                   int* __restrict__ list_ctr) {
    if (st->done || st->phase != 1) return;
    const int T = nt * (nt + 1) / 2;
    const int pos = blockIdx.x * 256 + threadIdx.x;
    for (int p = pos; p < nt * mask_words(nt * QB); p += gridDim.x * 256) {
        if (p < nt) {
            env_next[2 * p] = 0x7fffffff;
            env_next[2 * p + 1] = -1;
        }
        env_mask(env_next, nt)[p] = 0ull;
    }
    if (st->full_fill) return;
    bool listed = false;
    int item = 0;
    if (pos < T) {
        int bi, bj;
        order_tile_rows(pos, nt, tile_group, bi, bj);
        const int t = tri_index(bi, bj, nt);
        // no 32-column block set in both panels' masks: the product tile is zero
        const unsigned long long* mk = env_mask(env, nt);
        const int W = mask_words(nt * QB), nbk = nt * QB / QK;
        const bool k_empty = next_common_block(mk + (size_t)bi * W, mk + (size_t)bj * W, 0, nbk) >= nbk;
        if (k_empty && tz[(size_t)st->cur * T + t] != 0) {
            part[3 * t + 0] = 0.0;
            part[3 * t + 1] = 0.0;
            part[3 * t + 2] = 0.0;
            tz[(size_t)(1 - st->cur) * T + t] = 1;
        } else {
            listed = true;
            item = (bi << 15) | bj;
        }
    }
    // one atomic per wave
    const unsigned long long m = __ballot(listed);
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(&list_ctr[0], __popcll(m));
    base = __shfl(base, 0, 64);
    if (listed) list[base + __popcll(m & ((1ull << lane) - 1ull))] = item;
}

// One workgroup per CU takes list entries until none is left (every
// workgroup leaves once the shared counter passes the entry count).
template <int S, int NL>
__global__ __launch_bounds__(512) void k_gemm_int8x_list(double* __restrict__ buf0, double* __restrict__ buf1,
                                                         int ld, const State* __restrict__ st,
                                                         const int8_t* __restrict__ digits,
                                                         const double* __restrict__ scale,
                                                         double* __restrict__ part, const int* __restrict__ env,
                                                         const int* __restrict__ tz, const int* __restrict__ list,
                                                         int* __restrict__ list_ctr) {
    if (st->done || st->phase != 1 || st->full_fill) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem<S>& sm = *reinterpret_cast<I8Smem<S>*>(smem_raw);
    // the entry index is passed through the first word of the staging ring,
    // which no tile uses between the barriers around it (the ring fills the
    // 160 KiB of LDS; a separate shared variable would not fit)
    volatile int& s_k = *reinterpret_cast<int*>(smem_raw);
    const int nt = ld / QB, T = nt * (nt + 1) / 2;
    const int n = list_ctr[0];
    for (;;) {
        if (threadIdx.x == 0) s_k = atomicAdd(&list_ctr[1], 1);
        __syncthreads();
        const int k = s_k;
        __syncthreads();
        if (k >= n) break;
        const int it = list[k];
        const int bi = it >> 15, bj = it & 0x7fff;
        if (tz[(size_t)st->cur * T + tri_index(bi, bj, nt)]) {
            // the epilogue reads X_n: store the zeros the flag stands for (a
            // test per element would keep its loads from being in flight together)
            double* __restrict__ Xc = st->cur ? buf1 : buf0;
            for (int e = threadIdx.x; e < QB * QB / 2; e += 512)
                *reinterpret_cast<double2*>(Xc + (size_t)(bi * QB + e / (QB / 2)) * ld + bj * QB + 2 * (e % (QB / 2))) =
                    make_double2(0.0, 0.0);
            __syncthreads();
        }
        int8x_tile<S, NL, true, false>(buf0, buf1, ld, st, digits, scale, part, bi, bj, sm, env, nullptr);
        __syncthreads();
    }
}

// The same on 64 x 64 tiles, four per entry (the one below the diagonal of a
// diagonal tile is left out), for lists whose tiles have short K ranges: two
// workgroups share a CU, so one's X_n tile, mirrored stores and masks pass
// under the other's products, and a wave's block is the threshold's, which is
// applied before X_{n+1} is stored.  A whole number of workgroups per XCD,
// those of XCD x take every per-th tile of its run of the list.  Banded N =
// 16384 (875 entries of 8 stages), product and threshold: 228 + 58 us on 128 x
// 128 tiles, 130 + 58 on these with a threshold pass of its own, 123 + 5 now
// (k_tile_finish); the matrix instructions alone would be 66.
// Per listed tile t: idempotency partials idem4[4 t + q], block sums blk[16 t]
// and traces trd[4 bi].
struct List64 {
    double tau;
    int elem;
    double* idem4;
    double* blk;
    double* trd;
};

template <int S, int NL>
__global__ __launch_bounds__(256, 2) void k_gemm_int8x_list64(double* __restrict__ buf0, double* __restrict__ buf1,
                                                              int ld, const State* __restrict__ st,
                                                              const int8_t* __restrict__ digits,
                                                              const double* __restrict__ scale, List64 a,
                                                              const int* __restrict__ env,
                                                              const int* __restrict__ tz,
                                                              const int* __restrict__ list,
                                                              const int* __restrict__ list_ctr) {
    if (st->done || st->phase != 1 || st->full_fill) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem64<S>& sm = *reinterpret_cast<I8Smem64<S>*>(smem_raw);
    const int nt = ld / QB, T = nt * (nt + 1) / 2;
    const int n = 4 * list_ctr[0];
    const unsigned long long* __restrict__ mk = env_mask(env, nt);
    const int W = mask_words(ld);
    const int x = blockIdx.x % kXcds, per = gridDim.x / kXcds;
    const int end = (int)((long long)n * (x + 1) / kXcds);
    for (int k = (int)((long long)n * x / kXcds) + blockIdx.x / kXcds; k < end; k += per) {
        const int it = list[k >> 2], q = k & 3;
        const int bi = it >> 15, bj = it & 0x7fff;
        const int t = tri_index(bi, bj, nt);
        if (bi == bj && q == 2) {
            if (threadIdx.x == 0) a.idem4[4 * t + q] = 0.0;
            continue;
        }
        const Thr64 th = {mk + (size_t)bi * W, mk + (size_t)bj * W, a.tau, a.elem, a.blk + (size_t)16 * t,
                          a.trd + 4 * bi, q, bi == bj, tz[(size_t)st->cur * T + t] != 0};
        int8x_tile64<S, NL, true>(buf0, buf1, ld, st, digits, scale, a.idem4, 2 * bi + (q >> 1), 2 * bj + (q & 1), sm,
                                  nullptr, 4 * t + q, th);
        __syncthreads();
    }
}

// What the threshold pass leaves behind beside X, from the block sums of the
// 64 x 64 tiles: the tile's partials and flag, its panels' ranges and masks,
// and the kept count (of the nb x nb blocks without the padding).  One thread
// per listed tile; the same sums in the same order as threshold_tile.
__global__ __launch_bounds__(64) void k_tile_finish(State* __restrict__ st, int nt, int nb, List64 a,
                                                    double* __restrict__ part, int* __restrict__ env, int* __restrict__ tz,
                                                    const int* __restrict__ list, const int* __restrict__ list_ctr) {
    if (st->done || st->phase != 1 || st->full_fill) return;
    const int T = nt * (nt + 1) / 2, n = list_ctr[0];
    const int W = mask_words(nt * QB);
    int* __restrict__ tzn = tz + (size_t)(1 - st->cur) * T;
    unsigned long long* __restrict__ mk = env_mask(env, nt);
    int kept = 0;
    for (int k = blockIdx.x * 64 + threadIdx.x; k < n; k += gridDim.x * 64) {
        const int bi = list[k] >> 15, bj = list[k] & 0x7fff, t = tri_index(bi, bj, nt);
        const bool mirror = bi != bj;
        double f[4];
        int bits = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f[r] = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double ss = a.blk[(size_t)16 * t + 4 * r + c];
                if (ss != -1.0) {
                    f[r] += ss;
                    bits |= 1 << (4 * r + c);
                }
            }
        }
        const double* __restrict__ tr = a.trd + 4 * bi;
        const double* __restrict__ id = a.idem4 + 4 * t;
        part[3 * t + 0] = mirror ? 0.0 : (tr[0] + tr[1]) + (tr[2] + tr[3]);
        part[3 * t + 1] = (mirror ? 2.0 : 1.0) * ((f[0] + f[1]) + (f[2] + f[3]));
        part[3 * t + 2] = (id[0] + id[1]) + (id[2] + id[3]);
        tzn[t] = bits == 0 ? 1 : 0;
        if (bits == 0) continue;
        // of the padding's blocks, zero and below tau, none counts (nor is one
        // kept, unless tau^2 rounds to zero)
        const int in_r = (1 << 4 * min(4, nb - 4 * bi)) - 1, in_c = 0x1111 * ((1 << min(4, nb - 4 * bj)) - 1);
        kept += (mirror ? 2 : 1) * __popc(bits & in_r & in_c);
        // kept column sub-blocks of panel bi, row sub-blocks of panel bj
        const int cols = (bits | bits >> 4 | bits >> 8 | bits >> 12) & 15;
        int rows = 0;
        for (int r = 0; r < 4; ++r) rows |= ((bits >> (4 * r) & 15) != 0 ? 1 : 0) << r;
        atomicMin(&env[2 * bi], 4 * bj + __ffs(cols) - 1);
        atomicMax(&env[2 * bi + 1], 4 * bj + 31 - __clz(cols));
        atomicMin(&env[2 * bj], 4 * bi + __ffs(rows) - 1);
        atomicMax(&env[2 * bj + 1], 4 * bi + 31 - __clz(rows));
        atomicOr(&mk[(size_t)bi * W + ((4 * bj) >> 6)], (unsigned long long)cols << ((4 * bj) & 63));
        if (mirror) atomicOr(&mk[(size_t)bj * W + ((4 * bi) >> 6)], (unsigned long long)rows << ((4 * bi) & 63));
    }
    for (int o = 32; o > 0; o >>= 1) kept += __shfl_xor(kept, o, 64);
    if (threadIdx.x == 0 && kept) atomicAdd(&st->kept, (unsigned long long)kept);
}

// Epilogue of the split tiles: workgroup p takes the summed chunks of the
// tile at visiting position t_full + p and applies the update.
template <int S, int NL, bool UPPER, int C = 0>
__global__ __launch_bounds__(512) void k_gemm_int8x_tail(double* __restrict__ buf0, double* __restrict__ buf1,
                                                         int ld, const State* __restrict__ st,
                                                         const int8_t* __restrict__ digits,
                                                         const double* __restrict__ scale,
                                                         double* __restrict__ part,
                                                         unsigned long long* __restrict__ rmax, int tile_group,
                                                         int t_full, int nsplit, int* __restrict__ chunk_acc,
                                                         int when_full) {
    if (st->done || st->phase != 1 || (when_full && !st->full_fill)) return;
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem<S, C>& sm = *reinterpret_cast<I8Smem<S, C>*>(smem_raw);
    int bi, bj;
    order_tile(t_full + blockIdx.x, ld / QB, tile_group, bi, bj);
    // k_chunk_sum has added the tile's chunks into its first one
    int8x_tile<S, NL, false, UPPER, C>(buf0, buf1, ld, st, digits, scale, part, bi, bj, sm, nullptr,
                                    UPPER ? rmax + (size_t)(1 - st->cur) * ld : nullptr, 2, 0, -1,
                                    chunk_acc + (size_t)blockIdx.x * nsplit * (NL * 2 * 16 * 512), 1);
}

// The int32 accumulators of the nsplit K chunks of each split tile, added
// into the tile's first chunk (exact: every partial sum over a range of K is
// bounded like the whole sum).  kChunkSumParts workgroups per tile, each over
// an equal share of the tile's NL x 2 x 16 x 512 accumulators, so the sums
// are read by many CUs at once instead of by the tile's one tail workgroup.
constexpr int kChunkSumParts = 8;
template <int NL>
__global__ __launch_bounds__(256) void k_chunk_sum(int* __restrict__ chunk_acc, int nsplit,
                                                   const State* __restrict__ st, int when_full) {
    if (st->done || st->phase != 1 || (when_full && !st->full_fill)) return;
    constexpr int CH4 = NL * 2 * 16 * 512 / 4;          // int4 per chunk
    constexpr int PER = CH4 / kChunkSumParts;
    static_assert(CH4 % kChunkSumParts == 0, "chunk must split evenly");
    const int tile = blockIdx.x / kChunkSumParts, share = blockIdx.x % kChunkSumParts;
    int4* __restrict__ base = reinterpret_cast<int4*>(chunk_acc) + (size_t)tile * nsplit * CH4;
    for (int e = share * PER + threadIdx.x; e < (share + 1) * PER; e += 256) {
        int4 s = base[e];
        for (int ch = 1; ch < nsplit; ++ch) {
            const int4 v = base[(size_t)ch * CH4 + e];
            s.x += v.x;
            s.y += v.y;
            s.z += v.z;
            s.w += v.w;
        }
        base[e] = s;
    }
}

// Grouped: every upper-triangular 64 x 64 tile of every system in the group,
// upper-only.  A fixed grid (so the launch can be captured once and replayed),
// a whole number of workgroups per XCD (they are dealt to the XCDs
// round-robin): those of XCD x take every per-th tile of its run, whose tiles
// share row panels in its L2 and come in order of falling size.  Two
// workgroups share a CU, so one's waits for digits that just left another L2,
// its X_n tile and its row maxima pass under the other's products: with one
// workgroup of a 128 x 128 tile per CU (57 % of the wave cycles were waits) a
// burst of 24 requests of N = 148-2048 took 50 ms, upper-only 46-48, on these
// tiles 37.  Handing tiles out by an atomic counter instead of the fixed
// stride cost 5-15 ms of it.
template <int S, int NL>
__global__ __launch_bounds__(256, 2) void k_gemm_int8x_grouped(const GroupDesc* __restrict__ g) {
    extern __shared__ __align__(16) int8_t smem_raw[];
    I8Smem64<S>& sm = *reinterpret_cast<I8Smem64<S>*>(smem_raw);
    const int x = blockIdx.x % kXcds, per = gridDim.x / kXcds, end = g->xcd_off[x + 1];
    for (int item = g->xcd_off[x] + blockIdx.x / kXcds; item < end; item += per) {
        const int s = group_find(g->tile_off, g->nsys, item);
        const SysView& v = g->sys[s];
        if (v.st->done || v.st->phase != 1) continue;
        int bi, bj;
        order_tile(item - g->tile_off[s], v.ld / QT, 16, bi, bj);
        int8x_tile64<S, NL>(v.buf0, v.buf1, v.ld, v.st, v.digits, v.scale, v.part, bi, bj, sm,
                            v.rmax + (size_t)(1 - v.st->cur) * v.ld, tri_index(bi, bj, v.ld / QT));
        __syncthreads();
    }
}

// Compute units of the current device (cached per device; callers may be on
// several threads).
int device_cus() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Tiles of a dense product's last round that are handed out in pieces: when they
// would leave at least half of the CUs idle and a tile's K loop covers at least
// 4096 columns (shorter tiles cost less than what the pieces add).
static int left_tiles(const SplitScratch& s, int ld) {
    const int nt = ld / QB, cus = device_cus(), r = nt * (nt + 1) / 2 % cus;
    return s.tail_split != 0 && ld / QK >= 128 && 2 * r <= cus ? r : 0;
}

// Whether they are 64 x 64 pieces (upper-only products): up to four rounds of
// tiles.  Beyond, the chip is at its power limit and the pieces' operand
// traffic costs what their balance gives (N = 8192: 0.6 % slower than chunks).
static bool left_in_pieces(int ld) { return tri_tiles(ld / QB) < 4 * device_cus(); }

template <int S, int NL>
static hipError_t launch_left(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                              hipStream_t stream, int r) {
    const size_t lds = sizeof(I8Smem64<S>);
    static std::atomic<unsigned long long> attr_done{0};
    hipError_t e = once_per_device(attr_done, [&] {
        return hipFuncSetAttribute((const void*)k_gemm_int8x_left<S, NL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_gemm_int8x_left<S, NL>), dim3(4 * r), dim3(256), lds, stream, buf0, buf1, ld, st, s.digits,
                       s.scale, part, s.rmax, s.tile_group, tri_tiles(ld / QB) - r);
    return hipGetLastError();
}

template <int S, int NL, bool THR, bool UPPER, int C = 0>
static hipError_t launch_tile_kernel(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                                     hipStream_t stream, const int* env, int when_full = 0) {
    const int nt = ld / QB;
    const int T = nt * (nt + 1) / 2;
    const size_t lds = sizeof(I8Smem<S, C>);
    static std::atomic<unsigned long long> attr_done{0};
    hipError_t e = once_per_device(attr_done, [&] {
        hipError_t r = hipFuncSetAttribute((const void*)k_gemm_int8x<S, NL, THR, UPPER, C>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (r == hipSuccess && !THR)
            r = hipFuncSetAttribute((const void*)k_gemm_int8x_tail<S, NL, UPPER, C>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        return r;
    });
    if (e != hipSuccess) return e;
    // The left tiles: 64 x 64 pieces, else nsplit <= 8 chunks along K.
    int t_full = T, nsplit = 1;
    const int r = THR ? 0 : left_tiles(s, ld);
    const bool pieces = UPPER && r > 0 && left_in_pieces(ld);
    if (pieces) {
        t_full = T - r;
    } else if (r > 0 && s.tail_acc) {
        nsplit = std::min(8, device_cus() / r);
        if (nsplit >= 2 && (size_t)r * nsplit * NL * 2 * 16 * 512 * sizeof(int) <= s.tail_bytes) t_full = T - r;
        else nsplit = 1;
    }
    const int grid = t_full + (pieces ? 0 : (T - t_full) * nsplit);
    hipLaunchKernelGGL((k_gemm_int8x<S, NL, THR, UPPER, C>), dim3(grid), dim3(512), lds, stream, buf0, buf1, ld, st,
                       s.digits, s.scale, part, env, s.rmax, s.tile_group, t_full, nsplit, s.tail_acc, when_full);
    if (pieces) return launch_left<S, NL>(s, buf0, buf1, ld, st, part, stream, r);
    if (t_full < T) {
        hipLaunchKernelGGL(k_chunk_sum<NL>, dim3((T - t_full) * kChunkSumParts), dim3(256), 0, stream, s.tail_acc,
                           nsplit, st, when_full);
        hipLaunchKernelGGL((k_gemm_int8x_tail<S, NL, UPPER, C>), dim3(T - t_full), dim3(512), lds, stream, buf0, buf1, ld,
                           st, s.digits, s.scale, part, s.rmax, s.tile_group, t_full, nsplit, s.tail_acc, when_full);
    }
    return hipGetLastError();
}

template <int S, int NL>
static hipError_t launch_list_kernel(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                                     hipStream_t stream, const int* env) {
    const int nt = ld / QB;
    const int T = nt * (nt + 1) / 2;
    static std::atomic<unsigned long long> attr_done{0};
    hipError_t e = once_per_device(attr_done, [&] {
        hipError_t r = hipFuncSetAttribute((const void*)k_gemm_int8x_list<S, NL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(I8Smem<S>));
        if (r == hipSuccess)
            r = hipFuncSetAttribute((const void*)k_gemm_int8x_list64<S, NL>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(I8Smem64<S>));
        return r;
    });
    if (e != hipSuccess) return e;
    int* list = s.tz + (size_t)2 * T;
    int* ctr = list + T;
    hipLaunchKernelGGL(k_tile_list, dim3((T + 255) / 256), dim3(256), 0, stream, st, env, s.env_next, s.tz, nt,
                       s.tile_group, part, list, ctr);
    if (s.list64) {
        const int grid = std::max(2 * device_cus() / kXcds, 1) * kXcds;
        // 20 doubles per tile and 4 per diagonal one, where the dense kernel keeps its K chunks
        double* a0 = reinterpret_cast<double*>(s.tail_acc);
        if (((size_t)20 * T + 4 * nt) * sizeof(double) > s.tail_bytes) return hipErrorInvalidValue;
        const List64 a = {s.tau, s.elem, a0, a0 + (size_t)4 * T, a0 + (size_t)20 * T};
        hipLaunchKernelGGL((k_gemm_int8x_list64<S, NL>), dim3(grid), dim3(256), sizeof(I8Smem64<S>), stream, buf0,
                           buf1, ld, st, s.digits, s.scale, a, env, s.tz, list, ctr);
        hipLaunchKernelGGL(k_tile_finish, dim3(std::min((T + 63) / 64, device_cus())), dim3(64), 0, stream, st, nt,
                           s.nb, a, part, s.env_next, s.tz, list, ctr);
    } else {
        const int grid = std::min(T, device_cus());
        hipLaunchKernelGGL((k_gemm_int8x_list<S, NL>), dim3(grid), dim3(512), sizeof(I8Smem<S>), stream, buf0, buf1,
                           ld, st, s.digits, s.scale, part, env, s.tz, list, ctr);
    }
    return hipGetLastError();
}

// Dense products of which size run 64 x 64 tiles: those for which the model
// below makes them faster, in us per product.  A round of 128 x 128 tiles over
// the CUs takes 17 + 0.032 K (81 us at N = 2048, one round; 232 at 3072, two);
// the 64 x 64 tiles share CUs and follow their number, 10 + 4.8e-5 T K (174 us
// measured at N = 3072, 170 modelled; 113 against 101 at 2560, which stays on
// 128).  From ld = 4096 on the 128 x 128 kernel splits its last round and is
// never behind (N = 5600: 832 against 935 us).  The model is of four planes and
// five levels and holds the sizes for every recipe: whole solves per product,
// 128 x 128 tiles throughout against this rule, N = 720 / 2048 / 2304 / 3072 /
// 3328: three planes, four levels 42 -> 21, 74 -> 67, 81 -> 76, 182 -> 138, 198
// -> 178 us; five planes 54 -> 26, 104 -> 102, 116 -> 115, 282 -> 223, 305 ->
// 278; six 81 -> 31, 169 -> 130, 191 -> 146, 467 -> 297, 503 -> 372.  Sizes
// between these would gain too with six planes or six levels, not with fewer.
static bool use_tile64(int ld) {
    if (ld >= 4096) return false;
    const int n128 = ld / QB, n64 = ld / QT, cus = device_cus();
    const int T128 = n128 * (n128 + 1) / 2, T64 = n64 * (n64 + 1) / 2;
    const double t128 = ((T128 + cus - 1) / cus) * (17.0 + 0.032 * ld);
    const double t64 = 10.0 + 4.8e-5 * (256.0 / cus) * T64 * ld;
    return t64 < t128;
}

int int8x_folded_slots(int ld) {
    const int T = tri_tiles(ld / QT);
    return use_tile64(ld) && T <= kFoldSlots ? T : 0;
}

template <int S, int NL>
static hipError_t launch_t64(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                             hipStream_t stream) {
    const int nt = ld / QT, T = nt * (nt + 1) / 2;
    const size_t lds = sizeof(I8Smem64<S>);
    static std::atomic<unsigned long long> attr_done{0};
    hipError_t e = once_per_device(attr_done, [&] {
        return hipFuncSetAttribute((const void*)k_gemm_int8x_t64<S, NL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_gemm_int8x_t64<S, NL>), dim3(T), dim3(256), lds, stream, buf0, buf1, ld, st, s.digits,
                       s.scale, part, s.rmax, 2 * s.tile_group);
    return hipGetLastError();
}

template <int S, int NL>
static hipError_t run_int8x(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                            hipStream_t stream, const int* env) {
    if (env && s.tz) {
        // thresholded: the work-list product, and with the dense switch the
        // dense tile kernel over every upper tile (rows encoded whole); of
        // the two, the first runs while State::full_fill is clear, the second
        // while it is set.  The same tiles get the same integer sums either way.
        hipError_t e = launch_list_kernel<S, NL>(s, buf0, buf1, ld, st, part, stream, env);
        if (e == hipSuccess && s.dense_switch)
            e = launch_tile_kernel<S, NL, false, false>(s, buf0, buf1, ld, st, part, stream, nullptr, 1);
        return e;
    }
    if (env) return launch_tile_kernel<S, NL, true, false>(s, buf0, buf1, ld, st, part, stream, env);
    if (s.upper && s.tile64 && use_tile64(ld)) return launch_t64<S, NL>(s, buf0, buf1, ld, st, part, stream);
    // dense products: the stage configuration chosen by the autotuner
    if constexpr (i8_cfg_ok(S, 2)) {
        if (s.stage_cfg == 2)
            return s.upper ? launch_tile_kernel<S, NL, false, true, 2>(s, buf0, buf1, ld, st, part, stream, nullptr)
                           : launch_tile_kernel<S, NL, false, false, 2>(s, buf0, buf1, ld, st, part, stream, nullptr);
    }
    if (s.stage_cfg == 1)
        return s.upper ? launch_tile_kernel<S, NL, false, true, 1>(s, buf0, buf1, ld, st, part, stream, nullptr)
                       : launch_tile_kernel<S, NL, false, false, 1>(s, buf0, buf1, ld, st, part, stream, nullptr);
    if (s.upper) return launch_tile_kernel<S, NL, false, true>(s, buf0, buf1, ld, st, part, stream, nullptr);
    return launch_tile_kernel<S, NL, false, false>(s, buf0, buf1, ld, st, part, stream, nullptr);
}

// Eight columns j .. j + 7 of a row into its digit blocks.
template <int S>
__device__ __forceinline__ void store_digits8(const double4& a, const double4& b, double inv, int W, size_t rowblk,
                                              int r32, int j, int8_t* __restrict__ digits, size_t plane) {
    double y[8] = {a.x * inv, a.y * inv, a.z * inv, a.w * inv, b.x * inv, b.y * inv, b.z * inv, b.w * inv};
    const size_t off = (rowblk + (j >> 5)) * 1024 + r32 * 32 + 16 * (((j >> 4) & 1) ^ dswz(r32)) + (j & 15);
    unsigned long long packed[S];
    pack_digits8<S>(y, W, packed);
#pragma unroll
    for (int t = 0; t < S; ++t) *reinterpret_cast<unsigned long long*>(digits + t * plane + off) = packed[t];
}
__device__ __forceinline__ double abs_max8(const double4& a, const double4& b) {
    return fmax(fmax(fmax(fabs(a.x), fabs(a.y)), fmax(fabs(a.z), fabs(a.w))),
                fmax(fmax(fabs(b.x), fabs(b.y)), fmax(fabs(b.z), fabs(b.w))));
}

// Thresholded X: one wave per padded row, over the columns of its row panel's
// range of nonzero 32-column blocks only, rounded out to whole K stages the
// way the product rounds its K range (no product reads digits outside it);
// blocks without a nonzero are zeros, read or not.  Same digits as encode_row.
// A panel with no nonzero block is read by no product.  Ranges of up to 2048
// columns are held in registers between the maximum and the digits (one read of
// X instead of two): N = 16384 banded, 65 -> 51 us a product.  With tz (the work-list
// path) tiles flagged zero may hold anything: the masks leave them out here,
// and before the dense tile kernel, which reads every X_n tile, zeros are
// stored.  Also clears the work list's two counters.
template <int S>
__global__ __launch_bounds__(256) void k_encode_int8_env(double* __restrict__ buf0, double* __restrict__ buf1, int ld,
                                                         const State* __restrict__ st,
                                                         int8_t* __restrict__ digits,
                                                         double* __restrict__ scale, const int* __restrict__ env,
                                                         const int* __restrict__ tz, int* __restrict__ list_ctr) {
    if (st->done || st->phase != 1) return;
    if (list_ctr && blockIdx.x == 0 && threadIdx.x < 2) list_ctr[threadIdx.x] = 0;
    constexpr int KS = I8Stage<S>::KS;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nt = ld / QB, p = i / QB;
    double* __restrict__ X = st->cur ? buf1 : buf0;
    if (st->full_fill) {   // the dense tile kernel reads every K block and X_n tile
        if (tz) {
            const int* __restrict__ f = tz + (size_t)st->cur * (nt * (nt + 1) / 2);
            for (int q = 0; q < nt; ++q)
                if (f[tri_index(min(p, q), max(p, q), nt)])
                    *reinterpret_cast<double2*>(X + (size_t)i * ld + q * QB + 2 * lane) = make_double2(0.0, 0.0);
            // encode_row below reads columns other lanes of this wave stored
            __threadfence_block();
        }
        encode_row<S>(X, ld, i, lane, digits, scale, 0, ld);
        return;
    }
    const int lo = env[2 * p], hi = env[2 * p + 1];
    if (lo > hi) {
        if (lane == 0) scale[i] = 1.0;
        return;
    }
    const int c0 = (lo / KS) * KS * 32, c1 = min(ld, (hi / KS + 1) * KS * 32);
    const unsigned long long* __restrict__ mk = env_mask(env, nt) + (size_t)p * mask_words(ld);
    const double4 z4 = make_double4(0.0, 0.0, 0.0, 0.0);
    const double* __restrict__ row = X + (size_t)i * ld;
    const int W = digit_bits(ld, S);
    const size_t plane = (size_t)ld * ld, rowblk = (size_t)(i >> 5) * (ld >> 5);
    const int r32 = i & 31;
    auto kept = [&](int j) { return j < c1 && (mk[j >> 11] >> ((j >> 5) & 63) & 1ull); };
    auto load = [&](int j, double4& a, double4& b) {
        a = b = z4;
        if (kept(j)) {
            a = *reinterpret_cast<const double4*>(row + j);
            b = *reinterpret_cast<const double4*>(row + j + 4);
        }
    };
    double m = 0.0, sc;
    if (c1 - c0 <= 2048) {
        double4 a[4], b[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) load(c0 + 8 * lane + 512 * c, a[c], b[c]);
#pragma unroll
        for (int c = 0; c < 4; ++c) m = fmax(m, abs_max8(a[c], b[c]));
        const double inv = row_scale(wred_max(m), &sc);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = c0 + 8 * lane + 512 * c;
            if (j < c1) store_digits8<S>(a[c], b[c], inv, W, rowblk, r32, j, digits, plane);
        }
    } else {
        double4 a, b;
        for (int j = c0 + 8 * lane; j < c1; j += 512) {
            load(j, a, b);
            m = fmax(m, abs_max8(a, b));
        }
        const double inv = row_scale(wred_max(m), &sc);
        for (int j = c0 + 8 * lane; j < c1; j += 512) {
            load(j, a, b);
            store_digits8<S>(a, b, inv, W, rowblk, r32, j, digits, plane);
        }
    }
    if (lane == 0) scale[i] = sc;
}

template <int S>
static hipError_t run_encode(SplitScratch& s, const double* buf0, const double* buf1, int ld, State* st,
                             hipStream_t stream, const FoldArgs* f) {
    if (s.env) {
        const int nt = ld / QB;
        hipLaunchKernelGGL(k_encode_int8_env<S>, dim3(ld / 4), dim3(256), 0, stream, const_cast<double*>(buf0),
                           const_cast<double*>(buf1), ld, st, s.digits, s.scale, s.env, s.tz,
                           s.tz ? s.tz + (size_t)3 * tri_tiles(nt) : nullptr);
        return hipGetLastError();
    }
    if (s.upper) {
        const int nb = ld / 32;
        const dim3 grid(nb * (nb + 1) / 2);
        if (f)
            hipLaunchKernelGGL((k_encode_int8_upper<S, true>), grid, dim3(256), 0, stream, buf0, buf1, ld, st, s.digits,
                               s.scale, s.rmax, *f);
        else
            hipLaunchKernelGGL((k_encode_int8_upper<S, false>), grid, dim3(256), 0, stream, buf0, buf1, ld, st, s.digits,
                               s.scale, s.rmax, FoldArgs{});
    } else if (ld <= 2048 * ENC_CH)
        hipLaunchKernelGGL(k_encode_int8_reg<S>, dim3(ld), dim3(256), 0, stream, buf0, buf1, ld, st, s.digits,
                           s.scale);
    else
        hipLaunchKernelGGL(k_encode_int8<S>, dim3(ld / 4), dim3(256), 0, stream, buf0, buf1, ld, st, s.digits,
                           s.scale);
    return hipGetLastError();
}

template <int S, int NL>
static hipError_t run_grouped(const GroupDesc* g, hipStream_t stream) {
    const size_t lds = sizeof(I8Smem64<S>);
    static std::atomic<unsigned long long> attr_done{0};
    hipError_t e = once_per_device(attr_done, [&] {
        return hipFuncSetAttribute((const void*)k_gemm_int8x_grouped<S, NL>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_encode_int8_grouped<S>, dim3(2048), dim3(256), 0, stream, g);
    const int grid = std::max(2 * device_cus() / kXcds, 1) * kXcds;
    hipLaunchKernelGGL((k_gemm_int8x_grouped<S, NL>), dim3(grid), dim3(256), lds, stream, g);
    return hipGetLastError();
}

hipError_t launch_int8x_grouped(int slices, int levels, const GroupDesc* g, hipStream_t stream) {
    const bool next = levels == slices + 1;
    if (!next && levels != slices) return hipErrorInvalidValue;
    switch (slices) {
        case 2: return next ? run_grouped<2, 3>(g, stream) : run_grouped<2, 2>(g, stream);
        case 3: return next ? run_grouped<3, 4>(g, stream) : run_grouped<3, 3>(g, stream);
        case 4: return next ? run_grouped<4, 5>(g, stream) : run_grouped<4, 4>(g, stream);
        case 5: return next ? run_grouped<5, 6>(g, stream) : run_grouped<5, 5>(g, stream);
        case 6: return next ? hipErrorInvalidValue : run_grouped<6, 6>(g, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_int8x_encode(SplitScratch& s, const double* buf0, const double* buf1, int ld, State* st,
                               hipStream_t stream, const FoldArgs* f) {
    switch (s.slices) {
        case 2: return run_encode<2>(s, buf0, buf1, ld, st, stream, f);
        case 3: return run_encode<3>(s, buf0, buf1, ld, st, stream, f);
        case 4: return run_encode<4>(s, buf0, buf1, ld, st, stream, f);
        case 5: return run_encode<5>(s, buf0, buf1, ld, st, stream, f);
        case 6: return run_encode<6>(s, buf0, buf1, ld, st, stream, f);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_int8x_gemm(SplitScratch& s, double* buf0, double* buf1, int ld, State* st, double* part,
                             int* nslots, hipStream_t stream, const int* env) {
    const bool small = s.upper && s.tile64 && !env && use_tile64(ld);
    *nslots = tri_tiles(ld / (small ? QT : QB)) + (s.upper && !env && !small && left_in_pieces(ld) ? 3 * left_tiles(s, ld) : 0);
    const bool next = s.levels == s.slices + 1;
    if (!next && s.levels != s.slices) return hipErrorInvalidValue;
    switch (s.slices) {
        case 2: return next ? run_int8x<2, 3>(s, buf0, buf1, ld, st, part, stream, env)
                            : run_int8x<2, 2>(s, buf0, buf1, ld, st, part, stream, env);
        case 3: return next ? run_int8x<3, 4>(s, buf0, buf1, ld, st, part, stream, env)
                            : run_int8x<3, 3>(s, buf0, buf1, ld, st, part, stream, env);
        case 4: return next ? run_int8x<4, 5>(s, buf0, buf1, ld, st, part, stream, env)
                            : run_int8x<4, 4>(s, buf0, buf1, ld, st, part, stream, env);
        case 5: return next ? run_int8x<5, 6>(s, buf0, buf1, ld, st, part, stream, env)
                            : run_int8x<5, 5>(s, buf0, buf1, ld, st, part, stream, env);
        case 6: return next ? hipErrorInvalidValue : run_int8x<6, 6>(s, buf0, buf1, ld, st, part, stream, env);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sp2
