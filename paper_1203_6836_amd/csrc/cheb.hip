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

#include "cheb_internal.h"
#include "sp2_internal.h"

namespace sp2 {

namespace {

constexpr int CT = 32;   // tile of the elementwise passes over the upper triangle

__device__ __forceinline__ double wsum_c(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__global__ __launch_bounds__(256) void k_cheb_scale(const double* __restrict__ H, int N, double c, double inv_w,
                                                    double* __restrict__ T1) {
    const size_t n2 = (size_t)N * N;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n2; e += (size_t)gridDim.x * 256)
        T1[e] = (H[e] - (e / N == e % N ? c : 0.0)) * inv_w;
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
// thread keeps the s sums in registers.  HBM (or last-level cache) bound:
// (s + 1) N^2 / 2 doubles read.  SM: s rounded up to 8, 16 or 32.
template <int SM>
__global__ __launch_bounds__(256) void k_cheb_dots(const double* __restrict__ G, const double* __restrict__ T, int N,
                                                   int s, double* __restrict__ part) {
    const int nt = (N + CT - 1) / CT, ntiles = nt * (nt + 1) / 2;
    const size_t n2 = (size_t)N * N;
    const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    double acc[SM];
#pragma unroll
    for (int j = 0; j < SM; ++j) acc[j] = 0.0;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int bi, bj;
        order_tile(t, nt, 0, bi, bj);
        const double wgt = bi == bj ? 1.0 : 2.0;
        const int gj = bj * CT + c;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int gi = bi * CT + r0 + 8 * q;
            if (gi >= N || gj >= N) continue;
            const size_t e = (size_t)gi * N + gj;
            const double g = wgt * G[e];
            if (gi == gj) acc[0] += g;
#pragma unroll
            for (int j = 1; j < SM; ++j)
                if (j < s) acc[j] += g * T[(size_t)(j - 1) * n2 + e];
        }
    }
    __shared__ double sw[4][SM];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < SM; ++j) {
        const double v = wsum_c(acc[j]);
        if (lane == 0) sw[w][j] = v;
    }
    __syncthreads();
    if (threadIdx.x < s)
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] =
            (sw[0][threadIdx.x] + sw[1][threadIdx.x]) + (sw[2][threadIdx.x] + sw[3][threadIdx.x]);
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

static int grid_elem(int N) {
    const size_t g = ((size_t)N * N + 255) / 256;
    return (int)(g < 4096 ? g : 4096);
}

hipError_t launch_cheb_scale(const double* H, int N, double c, double inv_w, double* T1, hipStream_t s) {
    hipLaunchKernelGGL(k_cheb_scale, dim3(grid_elem(N)), dim3(256), 0, s, H, N, c, inv_w, T1);
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
hipError_t launch_cheb_dots(const double* G, const double* T, int N, int s, double* part, hipStream_t st) {
    if (s < 1 || s > kChebMaxS) return hipErrorInvalidValue;
    const int nblk = cheb_dot_blocks(N);
    if (s <= 8) hipLaunchKernelGGL(k_cheb_dots<8>, dim3(nblk), dim3(256), 0, st, G, T, N, s, part);
    else if (s <= 16) hipLaunchKernelGGL(k_cheb_dots<16>, dim3(nblk), dim3(256), 0, st, G, T, N, s, part);
    else hipLaunchKernelGGL(k_cheb_dots<32>, dim3(nblk), dim3(256), 0, st, G, T, N, s, part);
    return hipGetLastError();
}
hipError_t launch_cheb_sums(const double* part, int nblk, int nslots, double* out, hipStream_t st) {
    if (nslots < 1) return hipSuccess;
    hipLaunchKernelGGL(k_cheb_sums, dim3(nslots), dim3(256), 0, st, part, nblk, out);
    return hipGetLastError();
}

}  // namespace sp2
