// Internal declarations of the Chebyshev expansions of the finite-temperature
// functions: polynomials of Ht = (H - c I) / w, whose spectrum lies in [-1, 1].
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "cheb_plan.h"

namespace sp2 {

constexpr int kChebBlocks = 1024;   // most workgroups (and partials per sum) of the dot kernel

// T1 = ((H + H^T) / 2 - c I) * inv_w, exactly symmetric.
hipError_t launch_cheb_scale(const double* H, int N, double c, double inv_w, double* T1, hipStream_t s);
// out[j - 1] = Tr T_j of the s matrices T (T_j at T + (j - 1) N^2).
hipError_t launch_cheb_traces(const double* T, int N, int s, double* out, hipStream_t st);
// Partials of Tr G and of <G, T_j> = sum_e G_e T_j,e, j = 1 .. s - 1, for the
// symmetric matrices G = G0 and, if not null, G1: part[(g s + j) * nblk + b],
// nblk = cheb_dot_blocks(N) (j = 0 the trace).
int cheb_dot_blocks(int N);
hipError_t launch_cheb_dots(const double* G0, const double* G1, const double* T, int N, int s, double* part,
                            hipStream_t st);
// out[k] = sum of part[k * nblk .. +nblk) in fixed order, k < nslots.
hipError_t launch_cheb_sums(const double* part, int nblk, int nslots, double* out, hipStream_t st);
// C = sum_j b_j T_j (T_0 = I, 1 <= j < s) - V over the tiles on and above the
// diagonal (V may be null, and may be C), or over the whole matrix (full).
struct ChebCoef {
    double b[kChebMaxS];
};
hipError_t launch_cheb_combine(const double* T, int N, int s, const ChebCoef& b, const double* V, double* C, bool full,
                               hipStream_t st);

// Host side.
// a_k = (2 / M) sum_j g_j cos(k theta_j), theta_j = pi (j + 1/2) / M, k < M = g.size()
// (a power of two): the coefficients of sum_k' a_k T_k interpolating g at the
// Chebyshev-Gauss nodes cos theta_j (a_0 counts half).
void cheb_coefficients(const std::vector<double>& g, std::vector<double>& a);
// sum_j f_j W_j = sum_k' a_k mu_k for the moments mu (at most M of them) and
// every f on the M nodes with coefficients a: W_j = (2 / M) sum_k' mu_k cos(k theta_j).
void cheb_weights(const std::vector<double>& mu, int M, std::vector<double>& W);
// b[q][j], q <= Q, j < s, with sum_k c_k T_k = sum_q (sum_j b[q][j] T_j) T_qs
// (c taken as zero beyond its length).
void cheb_blocks(const std::vector<double>& c, int s, int Q, std::vector<std::vector<double>>& b);
// Nodes cos theta_j.
std::vector<double> cheb_nodes(int M);

}  // namespace sp2
