// How many polynomials and multiples a Chebyshev expansion stores and forms
// (host only).
#pragma once
#include <algorithm>
#include <cmath>

namespace sp2 {

constexpr int kChebMaxS = 32;                      // most stored polynomials T_1 .. T_s
constexpr double kChebBytes = 32.0 * 1073741824.0;   // most bytes of work matrices beyond five

// The number of stored polynomials the kernels are built for, at most s: 1, 2,
// 4, 8, 12, .. 32.
inline int cheb_round(int s) { return s <= 1 ? 1 : s <= 3 ? 2 : s <= 7 ? 4 : std::min(s / 4 * 4, kChebMaxS); }

// Stored polynomials for m coefficients of an N x N matrix: about sqrt(m), s + 2
// matrices within kChebBytes or five of them.
inline int cheb_stored(int N, int m) {
    const double fit = std::max(5.0, std::floor(kChebBytes / (8.0 * N * N))) - 2.0;
    return cheb_round((int)std::min({std::ceil(std::sqrt((double)m)), fit, (double)kChebMaxS}));
}

// Multiples T_s, T_2s, .. that the coefficients k < m need.
inline int cheb_multiples(int m, int s) { return std::max((m + s - 1) / s - 1, 0); }

}  // namespace sp2
