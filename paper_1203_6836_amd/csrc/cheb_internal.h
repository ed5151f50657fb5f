// Internal declarations of the Chebyshev expansions of the finite-temperature
// functions: polynomials of Ht = (H - c I) / w, whose spectrum lies in [-1, 1].
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

namespace sp2 {

constexpr int kChebMaxS = 32;       // most stored polynomials T_1 .. T_s
constexpr int kChebBlocks = 1024;   // most workgroups (and partials per sum) of the dot kernel

// T1 = (H - c I) * inv_w.
hipError_t launch_cheb_scale(const double* H, int N, double c, double inv_w, double* T1, hipStream_t s);
// out[j - 1] = Tr T_j of the s matrices T (T_j at T + (j - 1) N^2).
hipError_t launch_cheb_traces(const double* T, int N, int s, double* out, hipStream_t st);
// Partials of Tr G and of <G, T_j> = sum_e G_e T_j,e, j = 1 .. s - 1, for
// symmetric matrices: part[j * nblk + b], nblk = cheb_dot_blocks(N) (slot 0 the trace).
int cheb_dot_blocks(int N);
hipError_t launch_cheb_dots(const double* G, const double* T, int N, int s, double* part, hipStream_t st);
// out[k] = sum of part[k * nblk .. +nblk) in fixed order, k < nslots.
hipError_t launch_cheb_sums(const double* part, int nblk, int nslots, double* out, hipStream_t st);

// Host side.
// a_k = (2 / M) sum_j g_j cos(k theta_j), theta_j = pi (j + 1/2) / M, k < M = g.size()
// (a power of two): the coefficients of sum_k' a_k T_k interpolating g at the
// Chebyshev-Gauss nodes cos theta_j (a_0 counts half).
void cheb_coefficients(const std::vector<double>& g, std::vector<double>& a);
// Nodes cos theta_j.
std::vector<double> cheb_nodes(int M);

}  // namespace sp2
