// Chebyshev polynomials of a symmetric matrix for the finite-temperature
// functions: the elementwise passes and reductions around the FP64 products.
//
// The moments Tr T_k, k < m, come from about 2 sqrt(m) products instead of m / 2: with
// T_1 .. T_s stored and the multiples T_s, T_2s, .. formed one after another,
// T_(qs+j) = 2 T_qs T_j - T_|qs-j| makes every moment a trace of a product,
//     Tr T_(qs+j) = 2 <T_qs, T_j> - Tr T_|qs-j|,
// i.e. a sum over elements.  The dot kernel reads a multiple once for all s
// of its sums.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "cheb_internal.h"
#include "sp2_internal.h"

namespace sp2 {

namespace {

constexpr int CT = 32;   // tile of the elementwise passes over the upper triangle

__device__ __forceinline__ double wsum_c(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// T1 from the symmetric part of H (H itself where it is exactly symmetric; the
// check lets 1e-12 max|H| pass): the sums of a few polynomials read T1 directly,
// without a product that would make the result exactly symmetric.  One
// workgroup per pair of 32 x 32 tiles (bi, bj), (bj, bi), transposed through LDS.
__global__ __launch_bounds__(256) void k_cheb_scale(const double* __restrict__ H, int N, double c, double inv_w,
                                                    double* __restrict__ T1) {
    __shared__ double A[CT][CT + 1], B[CT][CT + 1];
    const int nt = (N + CT - 1) / CT;
    int bi, bj;
    order_tile(blockIdx.x, nt, 0, bi, bj);
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    for (int r = y; r < CT; r += 8) {
        const int i = bi * CT + r, j = bj * CT + x, it = bj * CT + r, jt = bi * CT + x;
        A[r][x] = i < N && j < N ? H[(size_t)i * N + j] : 0.0;
        B[r][x] = it < N && jt < N ? H[(size_t)it * N + jt] : 0.0;
    }
    __syncthreads();
    for (int r = y; r < CT; r += 8) {
        const int i = bi * CT + r, j = bj * CT + x, it = bj * CT + r, jt = bi * CT + x;
        if (i < N && j < N)
            T1[(size_t)i * N + j] = (i == j ? A[r][x] - c : 0.5 * (A[r][x] + B[x][r])) * inv_w;
        if (bi != bj && it < N && jt < N) T1[(size_t)it * N + jt] = 0.5 * (A[x][r] + B[r][x]) * inv_w;
    }
}

__global__ __launch_bounds__(256) void k_cheb_traces(const double* __restrict__ T, int N, double* __restrict__ out) {
    __shared__ double sw[4];
    const double* M = T + (size_t)blockIdx.x * N * N;
    double v = 0.0;
    for (int i = threadIdx.x; i < N; i += 256) v += M[(size_t)i * N + i];
    v = wsum_c(v);
    if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = (sw[0] + sw[1]) + (sw[2] + sw[3]);
}

// Workgroups stride over the 32 x 32 tiles of the upper triangle (off-diagonal
// ones count twice: half the reads of a pass over the whole matrices); each
// thread keeps the sums of NG multiples in registers, so two multiples share
// one read of the S - 1 matrices.  HBM (or last-level cache) bound:
// (S - 1 + NG) N^2 / 2 doubles read.  S is a template argument: with a run-time
// bound on j the loads waited for one another (S = 32, N = 500: 46 us for one
// multiple, 24 for two now; N = 2048: 204, and 122 for two, 4.7 TB/s).  ROWS: row
// y of the grid takes the sums j = y S .. y S + S - 1 of s = gridDim.y S.
template <int S, int NG, bool ROWS>
__global__ __launch_bounds__(256) void k_cheb_dots(const double* __restrict__ G0, const double* __restrict__ G1,
                                                   const double* __restrict__ T, int N, double* __restrict__ part) {
    const int nt = (N + CT - 1) / CT, ntiles = nt * (nt + 1) / 2;
    const size_t n2 = (size_t)N * N;
    const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    const int j0 = ROWS ? blockIdx.y * S : 0, s = ROWS ? gridDim.y * S : S;
    double acc[NG][S];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int j = 0; j < S; ++j) acc[g][j] = 0.0;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int bi, bj;
        order_tile(t, nt, 0, bi, bj);
        const double wgt = bi == bj ? 1.0 : 2.0;
        const int gj = bj * CT + c;
        for (int q = 0; q < 4; ++q) {
            const int gi = bi * CT + r0 + 8 * q;
            if (gi >= N || gj >= N) continue;
            const size_t e = (size_t)gi * N + gj;
            double v[S], g[NG];
#pragma unroll
            for (int j = ROWS ? 0 : 1; j < S; ++j)
                if (j > 0 || j0 > 0) v[j] = T[(size_t)(j0 + j - 1) * n2 + e];
            g[0] = wgt * G0[e];
            if (NG > 1) g[NG - 1] = wgt * G1[e];
#pragma unroll
            for (int k = 0; k < NG; ++k) {
                if (ROWS && j0 > 0) acc[k][0] += g[k] * v[0];
                else if (gi == gj) acc[k][0] += g[k];
#pragma unroll
                for (int j = 1; j < S; ++j) acc[k][j] += g[k] * v[j];
            }
        }
    }
    __shared__ double sw[4][NG * S];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NG; ++k)
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const double v = wsum_c(acc[k][j]);
            if (lane == 0) sw[w][k * S + j] = v;
        }
    __syncthreads();
    if (threadIdx.x < NG * S)
        part[(size_t)(ROWS ? threadIdx.x / S * s + j0 + threadIdx.x % S : threadIdx.x) * gridDim.x + blockIdx.x] =
            (sw[0][threadIdx.x] + sw[1][threadIdx.x]) + (sw[2][threadIdx.x] + sw[3][threadIdx.x]);
}

// HBM (or last-level cache) bound: (S + 1) N^2 / 2 doubles read and written
// (S = 32, N = 2048: 109 us, 5.1 TB/s).
template <int S>
__global__ __launch_bounds__(256) void k_cheb_combine(const double* __restrict__ T, int N, ChebCoef b,
                                                      const double* V, double* C, int full) {
    const int nt = (N + CT - 1) / CT;
    const size_t n2 = (size_t)N * N;
    const int t = blockIdx.x, c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    int bi, bj;
    if (full) {
        bi = t / nt;
        bj = t % nt;
    } else {
        order_tile(t, nt, 0, bi, bj);
    }
    const int gj = bj * CT + c;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int gi = bi * CT + r0 + 8 * q;
        if (gi >= N || gj >= N) continue;
        const size_t e = (size_t)gi * N + gj;
        double x[S], v = gi == gj ? b.b[0] : 0.0;
#pragma unroll
        for (int j = 1; j < S; ++j) x[j] = T[(size_t)(j - 1) * n2 + e];
        if (V) v -= V[e];
#pragma unroll
        for (int j = 1; j < S; ++j) v += b.b[j] * x[j];
        C[e] = v;
    }
}

__global__ __launch_bounds__(256) void k_cheb_sums(const double* __restrict__ part, int nblk,
                                                   double* __restrict__ out) {
    __shared__ double sw[4];
    double v = 0.0;
    for (int b = threadIdx.x; b < nblk; b += 256) v += part[(size_t)blockIdx.x * nblk + b];
    v = wsum_c(v);
    if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = (sw[0] + sw[1]) + (sw[2] + sw[3]);
}

// In-place radix-2 FFT, sum_j x_j e^(-2 pi i k j / n), n = re.size() a power of two.
void fft(std::vector<double>& re, std::vector<double>& im) {
    const size_t n = re.size();
    for (size_t i = 1, j = 0; i < n; ++i) {
        size_t bit = n >> 1;
        for (; j & bit; bit >>= 1) j ^= bit;
        j ^= bit;
        if (i < j) {
            std::swap(re[i], re[j]);
            std::swap(im[i], im[j]);
        }
    }
    std::vector<double> cs(n / 2), sn(n / 2);
    for (size_t k = 0; k < n / 2; ++k) {
        cs[k] = std::cos(2.0 * M_PI * (double)k / (double)n);
        sn[k] = -std::sin(2.0 * M_PI * (double)k / (double)n);
    }
    for (size_t len = 2; len <= n; len <<= 1) {
        const size_t half = len / 2, step = n / len;
        for (size_t i = 0; i < n; i += len)
            for (size_t k = 0; k < half; ++k) {
                const double wr = cs[k * step], wi = sn[k * step];
                const double xr = re[i + half + k], xi = im[i + half + k];
                const double vr = xr * wr - xi * wi, vi = xr * wi + xi * wr;
                re[i + half + k] = re[i + k] - vr;
                im[i + half + k] = im[i + k] - vi;
                re[i + k] += vr;
                im[i + k] += vi;
            }
    }
}

}  // namespace

std::vector<double> cheb_nodes(int M) {
    std::vector<double> x(M);
    for (int j = 0; j < M; ++j) x[j] = std::cos(M_PI * (j + 0.5) / M);
    return x;
}

// Re[e^(-i pi k / 2M) sum_j g_j e^(-2 pi i k j / 2M)]: one FFT of g padded to 2 M.
void cheb_coefficients(const std::vector<double>& g, std::vector<double>& a) {
    const size_t M = g.size();
    std::vector<double> re(2 * M, 0.0), im(2 * M, 0.0);
    std::copy(g.begin(), g.end(), re.begin());
    fft(re, im);
    a.resize(M);
    for (size_t k = 0; k < M; ++k) {
        const double t = M_PI * (double)k / (2.0 * (double)M);
        a[k] = (re[k] * std::cos(t) + im[k] * std::sin(t)) * 2.0 / (double)M;
    }
}

// Re sum_k (c_k e^(i pi k / 2M)) e^(2 pi i k j / 2M), c_0 halved: the conjugate of
// an FFT of the conjugates, padded to 2 M.
void cheb_weights(const std::vector<double>& mu, int M, std::vector<double>& W) {
    std::vector<double> re(2 * (size_t)M, 0.0), im(2 * (size_t)M, 0.0);
    for (size_t k = 0; k < mu.size() && k < (size_t)M; ++k) {
        const double t = M_PI * (double)k / (2.0 * M), c = (k == 0 ? 0.5 : 1.0) * mu[k];
        re[k] = c * std::cos(t);
        im[k] = -c * std::sin(t);
    }
    fft(re, im);
    W.resize(M);
    for (int j = 0; j < M; ++j) W[j] = re[j] * 2.0 / M;
}

// From the highest block down, T_(qs+j) = 2 T_qs T_j - T_(qs-j).
void cheb_blocks(const std::vector<double>& c, int s, int Q, std::vector<std::vector<double>>& b) {
    std::vector<double> a(c);
    a.resize((size_t)(Q + 1) * s, 0.0);
    b.assign(Q + 1, std::vector<double>(s, 0.0));
    for (int q = Q; q >= 0; --q) {
        b[q][0] = a[(size_t)q * s];
        for (int j = 1; j < s; ++j) {
            const double v = a[(size_t)q * s + j];
            if (q == 0) {
                b[0][j] = v;
            } else {
                b[q][j] = 2.0 * v;
                a[(size_t)q * s - j] -= v;
            }
        }
    }
}

hipError_t launch_cheb_scale(const double* H, int N, double c, double inv_w, double* T1, hipStream_t s) {
    hipLaunchKernelGGL(k_cheb_scale, dim3(tri_tiles((N + CT - 1) / CT)), dim3(256), 0, s, H, N, c, inv_w, T1);
    return hipGetLastError();
}
hipError_t launch_cheb_traces(const double* T, int N, int s, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_cheb_traces, dim3(s), dim3(256), 0, st, T, N, out);
    return hipGetLastError();
}
int cheb_dot_blocks(int N) {
    const int nt = (N + CT - 1) / CT;
    return std::min(tri_tiles(nt), kChebBlocks);
}
// f with the template argument S = s for the counts that cheb_round makes.
template <typename F>
static hipError_t with_stored(int s, F f) {
    switch (s) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 16: return f(std::integral_constant<int, 16>{});
        case 20: return f(std::integral_constant<int, 20>{});
        case 24: return f(std::integral_constant<int, 24>{});
        case 28: return f(std::integral_constant<int, 28>{});
        case 32: return f(std::integral_constant<int, 32>{});
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cheb_dots(const double* G0, const double* G1, const double* T, int N, int s, double* part,
                            hipStream_t st) {
    // Few tiles (up to N = 992) leave CUs idle, and a workgroup's time is the
    // chain of its NG s wave sums: the sums are dealt over rows of the grid, four
    // each.  s = 32, two multiples, N = 500: 24 -> 13 us; N = 1020 level.
    const int nblk = cheb_dot_blocks(N);
    if (nblk < 2 * device_cus() && s % 4 == 0 && s > 4) {
        const dim3 grid(nblk, s / 4);
        if (G1) hipLaunchKernelGGL((k_cheb_dots<4, 2, true>), grid, dim3(256), 0, st, G0, G1, T, N, part);
        else hipLaunchKernelGGL((k_cheb_dots<4, 1, true>), grid, dim3(256), 0, st, G0, G1, T, N, part);
        return hipGetLastError();
    }
    const dim3 grid(nblk);
    return with_stored(s, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        if (G1) hipLaunchKernelGGL((k_cheb_dots<S, 2, false>), grid, dim3(256), 0, st, G0, G1, T, N, part);
        else hipLaunchKernelGGL((k_cheb_dots<S, 1, false>), grid, dim3(256), 0, st, G0, G1, T, N, part);
        return hipGetLastError();
    });
}
hipError_t launch_cheb_combine(const double* T, int N, int s, const ChebCoef& b, const double* V, double* C, bool full,
                               hipStream_t st) {
    const int nt = (N + CT - 1) / CT, f = full ? 1 : 0;
    const dim3 grid(full ? nt * nt : tri_tiles(nt));
    return with_stored(s, [&](auto sc) {
        constexpr int S = decltype(sc)::value;
        hipLaunchKernelGGL(k_cheb_combine<S>, grid, dim3(256), 0, st, T, N, b, V, C, f);
        return hipGetLastError();
    });
}
hipError_t launch_cheb_sums(const double* part, int nblk, int nslots, double* out, hipStream_t st) {
    if (nslots < 1) return hipSuccess;
    hipLaunchKernelGGL(k_cheb_sums, dim3(nslots), dim3(256), 0, st, part, nblk, out);
    return hipGetLastError();
}

}  // namespace sp2
