// K loop of the small FP64 products: the 32 x 32 block of A^T B at rows i0,
// columns j0, summed over the 4-deep K steps [s0, s1), by one wave with four
// v_mfma_f64_16x16x4f64 per step and operands loaded straight from global
// memory (both matrices stay in L2 or the last-level cache at these sizes).
//
// A lane loads two neighbouring columns of an operand at once (16 bytes):
// MFMA block m of the tile holds the columns 2 c + m, so the permutation costs
// nothing and a step is two loads instead of four.  The loads of four steps
// are issued while the four before them are multiplied: 16 MFMAs of 64 cycles
// cover the latency of a load that misses L2, where a loop that loads and
// multiplies the same steps waits for each.
#pragma once
#include <hip/hip_runtime.h>

namespace sp2 {

typedef double d4s __attribute__((ext_vector_type(4)));
constexpr int kSmallTile = 32;
constexpr int kSmallWideLd = 512;   // 8 waves per tile up to here, then 4

// EDGE: N need not be a multiple of 32; elements outside N x N read as zero.
// VEC: rows are 16-byte aligned (leading dimension even, bases aligned).
template <bool EDGE, bool VEC>
__device__ __forceinline__ double2 small_load(const double* __restrict__ M, int ldm, int N, int k, int col) {
    const double* p = M + (size_t)k * ldm + col;
    if (!EDGE) return *reinterpret_cast<const double2*>(p);
    double2 v = make_double2(0.0, 0.0);
    if (k < N && col < N) {
        if (VEC) return *reinterpret_cast<const double2*>(p);   // N even: both columns are inside
        v.x = p[0];
        if (col + 1 < N) v.y = p[1];
    }
    return v;
}

template <bool EDGE, bool VEC>
__device__ __forceinline__ void small_mma(const double* __restrict__ A, const double* __restrict__ B, int ldm, int N,
                                          int i0, int j0, int s0, int s1, d4s (&acc)[2][2]) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63;
    const int ci = i0 + 2 * (lane & 15), cj = j0 + 2 * (lane & 15), kr = lane >> 4;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = d4s{0.0, 0.0, 0.0, 0.0};
    if (s0 >= s1) return;
    double2 a[2][U], b[2][U];
    // steps past the end reload the last one and are not multiplied
    auto load = [&](int p, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 4 * min(s + u, s1 - 1) + kr;
            a[p][u] = small_load<EDGE, VEC>(A, ldm, N, k, ci);
            b[p][u] = small_load<EDGE, VEC>(B, ldm, N, k, cj);
        }
    };
    auto mul = [&](int p, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + u >= s1) break;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const double av = m ? a[p][u].y : a[p][u].x;
                acc[m][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b[p][u].x, acc[m][0], 0, 0, 0);
                acc[m][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, b[p][u].y, acc[m][1], 0, 0, 0);
            }
        }
    };
    load(0, s0);
    for (int s = s0; s < s1; s += 2 * U) {
        if (s + U < s1) load(1, s + U);
        mul(0, s);
        if (s + 2 * U < s1) load(0, s + 2 * U);
        if (s + U < s1) mul(1, s + U);
    }
}

// A wave's partial tile to LDS, rows of 33 doubles.
__device__ __forceinline__ void small_store(double* red, const d4s (&acc)[2][2]) {
    const int lane = threadIdx.x & 63;
    // v_mfma_f64_16x16x4f64 result: lane l, element r is row (l >> 4) + 4 r, column l & 15 of block (m, n)
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[(2 * ((lane >> 4) + 4 * r) + m) * (kSmallTile + 1) + 2 * (lane & 15) + n] = acc[m][n][r];
}

}  // namespace sp2
