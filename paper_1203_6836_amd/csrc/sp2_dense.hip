// Dense SP2 kernels for gfx950: spectral bounds, X_0, the FP64-MFMA
// symmetric product with the fused purification update, the single-workgroup
// control step, and small observables (Mulliken charges, traces).
//
// SP2 (second-order spectral projection, Linear scaling section) builds the
// zero-temperature density matrix theta(mu0 I - H) as a sequence of squarings
// X <- X^2 or X <- 2X - X^2 starting from X_0 = (eps_max I - H)/(eps_max - eps_min).
//
// Layout: the library keeps X in two padded ld x ld row-major FP64 buffers
// (ld = N rounded up to 128, zero outside the N x N corner) used ping-pong;
// the zero padding makes every tile of the product full, with no bounds
// checks in the inner loop, and does not change X^2, traces or norms.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fold.h"
#include "small_f64.h"
#include "sp2_internal.h"

namespace sp2 {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_min(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Deterministic fixed-order block sum of per-thread values (blockDim 256).
__device__ double block_sum256(double v, double* sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    double r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return r;
}

// The same over NW waves (sums in wave order).
template <int NW>
__device__ __forceinline__ double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    double r = sh[0];
#pragma unroll
    for (int k = 1; k < NW; ++k) r += sh[k];
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------- bounds
// One wave per row i: lo_i = H_ii - sum_{j != i} |H_ij|, hi_i = H_ii + same.
// Each 256-thread workgroup covers 4 rows and writes (min lo, max hi).  With
// hz (k_check_h) the runs of 64 columns whose two blocks hold no nonzero are
// left out; the same sums in the same order (N = 16384 banded: 356 -> 17 us).
template <bool HZ>
__global__ __launch_bounds__(256) void k_gershgorin(const double* __restrict__ H, int N,
                                                     double* __restrict__ part,
                                                     const unsigned* __restrict__ hz) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + w;
    double lo = 1.0e300, hi = -1.0e300;
    if (i < N) {
        const double* row = H + (size_t)i * N;
        double s = 0.0;
        if constexpr (HZ) {
            const int nb = (N + 31) / 32;
            const unsigned* __restrict__ f = hz + (size_t)(i >> 5) * nb;
            for (int b0 = 0; b0 < nb; b0 += 128) {
                const int b = b0 + 2 * lane;
                unsigned long long m = __ballot((b < nb && f[b] != 0u) || (b + 1 < nb && f[b + 1] != 0u));
                for (; m; m &= m - 1) {
                    const int j = b0 * 32 + __builtin_ctzll(m) * 64 + lane;
                    if (j < N) s += fabs(row[j]);
                }
            }
        } else {
            for (int j = lane; j < N; j += 64) s += fabs(row[j]);
        }
        s = wave_sum(s);
        const double d = row[i];
        const double r = s - fabs(d);
        lo = d - r;
        hi = d + r;
    }
    __shared__ double sl[4], sh[4];
    if (lane == 0) { sl[w] = lo; sh[w] = hi; }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x + 0] = fmin(fmin(sl[0], sl[1]), fmin(sl[2], sl[3]));
        part[2 * blockIdx.x + 1] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    }
}

// H check: every 32 x 32 tile (bi, bj), bi <= bj, of the upper triangle is
// compared with the transpose of tile (bj, bi) through LDS; a fixed grid of
// workgroups strides over the tiles and keeps running maxima.  HZ: also records
// which 32 x 32 blocks hold a nonzero (or a NaN), hz[br nb + bc] != 0 with one
// byte per wave, for the passes over H behind it.
template <bool HZ>
__global__ __launch_bounds__(256) void k_check_h(const double* __restrict__ H, int N,
                                                 double* __restrict__ out, unsigned char* __restrict__ hz) {
    __shared__ double A[32][33], B[32][33];
    const int nb = (N + 31) / 32;
    const long long T = (long long)nb * (nb + 1) / 2;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
    double dmax = 0.0, amax = 0.0;
    bool bad = false;
    for (long long t = blockIdx.x; t < T; t += gridDim.x) {
        // row bi of the upper triangle starts at bi nb - bi (bi - 1) / 2
        int bi = (int)((2.0 * nb + 1.0 - sqrt((2.0 * nb + 1.0) * (2.0 * nb + 1.0) - 8.0 * (double)t)) / 2.0);
        bi = max(0, min(bi, nb - 1));
        while (bi > 0 && (long long)bi * nb - (long long)bi * (bi - 1) / 2 > t) --bi;
        while (bi + 1 < nb && (long long)(bi + 1) * nb - (long long)(bi + 1) * bi / 2 <= t) ++bi;
        const int bj = bi + (int)(t - ((long long)bi * nb - (long long)bi * (bi - 1) / 2));
        __syncthreads();
        for (int r = ty; r < 32; r += 8) {
            const int i = bi * 32 + r, j = bj * 32 + tx;      // tile (bi, bj)
            const int i2 = bj * 32 + r, j2 = bi * 32 + tx;    // tile (bj, bi)
            A[r][tx] = (i < N && j < N) ? H[(size_t)i * N + j] : 0.0;
            B[r][tx] = (i2 < N && j2 < N) ? H[(size_t)i2 * N + j2] : 0.0;
        }
        __syncthreads();
        bool na = false, nbz = false;
        for (int r = ty; r < 32; r += 8) {
            const double a = A[r][tx], b = B[tx][r];          // H_ij and H_ji
            if constexpr (HZ) {
                na = na || a != 0.0;
                nbz = nbz || b != 0.0;
            }
            if (!isfinite(a) || !isfinite(b)) bad = true;
            else {
                dmax = fmax(dmax, fabs(a - b));
                amax = fmax(amax, fabs(a));
            }
        }
        if constexpr (HZ) {
            const unsigned char fa = __any(na) ? 1 : 0, fb = __any(nbz) ? 1 : 0;
            if ((threadIdx.x & 63) == 0) {
                hz[4 * ((size_t)bi * nb + bj) + (threadIdx.x >> 6)] = fa;
                hz[4 * ((size_t)bj * nb + bi) + (threadIdx.x >> 6)] = fb;
            }
        }
    }
    dmax = wave_max(bad ? INFINITY : dmax);
    amax = wave_max(amax);
    __shared__ double sd[4], sa[4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sd[w] = dmax; sa[w] = amax; }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[2 * blockIdx.x + 0] = fmax(fmax(sd[0], sd[1]), fmax(sd[2], sd[3]));
        out[2 * blockIdx.x + 1] = fmax(fmax(sa[0], sa[1]), fmax(sa[2], sa[3]));
    }
}

__global__ __launch_bounds__(256) void k_bounds(const double* __restrict__ part, int nslots,
                                                const double* __restrict__ chk, int nchk,
                                                State* __restrict__ st) {
    double lo = 1.0e300, hi = -1.0e300, dmax = 0.0, amax = 0.0;
    for (int k = threadIdx.x; k < nslots; k += 256) {
        lo = fmin(lo, part[2 * k]);
        hi = fmax(hi, part[2 * k + 1]);
    }
    for (int k = threadIdx.x; k < nchk; k += 256) {
        dmax = fmax(dmax, chk[2 * k]);
        amax = fmax(amax, chk[2 * k + 1]);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    dmax = wave_max(dmax);
    amax = wave_max(amax);
    __shared__ double sl[4], sh[4], sd[4], sa[4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sl[w] = lo; sh[w] = hi; sd[w] = dmax; sa[w] = amax; }
    __syncthreads();
    if (threadIdx.x == 0) {
        st->eps_min = fmin(fmin(sl[0], sl[1]), fmin(sl[2], sl[3]));
        st->eps_max = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
        const double d = fmax(fmax(sd[0], sd[1]), fmax(sd[2], sd[3]));
        const double m = fmax(fmax(sa[0], sa[1]), fmax(sa[2], sa[3]));
        st->t1 = st->t2 = 0.0;
        st->fill_min = 1.0;
        st->fill_max = 0.0;
        st->bits[0] = st->bits[1] = 0ull;
        st->iter = 0;
        st->branch = 0;
        st->done = 0;
        st->cur = 0;
        st->result = 0;
        st->phase = 0;
        st->fp64_products = 0;
        st->head_switch = -1;
        st->tail_left = 0;
        st->full_fill = 0;
        st->kept = 0ull;
        if (!(d <= kSymTol * m)) st->done = 5;                          // also catches NaN / inf
        else if (!(st->eps_max > st->eps_min)) st->done = 4;            // H = c I: no gap anywhere
    }
    for (int k = threadIdx.x; k < kMaxIter; k += 256) {
        st->idem[k] = 0.0;
        st->fill[k] = 0.0f;
    }
}

// ------------------------------------------------------------------ X_0
// One wave per padded row.  Writes X_0 = (eps_max I - H)/(eps_max - eps_min)
// in the N x N corner and zeros elsewhere; per-workgroup partials
// (Tr X_0, ||X_0||_F^2, 0) into part[3 * block]; with rmax non-null also the
// row maxima max_j |X_0 ij| (as bit patterns) for the upper-only int8 path.
__global__ __launch_bounds__(256) void k_init(const double* __restrict__ H, int N, int ld,
                                              double* __restrict__ X, const State* __restrict__ st,
                                              double* __restrict__ part, unsigned long long* __restrict__ rmax) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + w;            // < ld by construction of the grid
    const double emax = st->eps_max;
    const double inv = 1.0 / (st->eps_max - st->eps_min);
    double tr = 0.0, fro = 0.0, mx = 0.0;
    double* xrow = X + (size_t)i * ld;
    if (i < N) {
        const double* hrow = H + (size_t)i * N;
        for (int j = lane; j < ld; j += 64) {
            double x = 0.0;
            if (j < N) {
                x = ((j == i ? emax : 0.0) - hrow[j]) * inv;
                if (j == i) tr += x;
            }
            xrow[j] = x;
            fro += x * x;
            mx = fmax(mx, fabs(x));
        }
    } else {
        for (int j = lane; j < ld; j += 64) xrow[j] = 0.0;
    }
    if (rmax) {
        mx = wave_max(mx);
        if (lane == 0) rmax[i] = (unsigned long long)__double_as_longlong(mx);
    }
    __shared__ double sh[4];
    const double btr = block_sum256(tr, sh);
    const double bfr = block_sum256(fro, sh);
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x + 0] = btr;
        part[3 * blockIdx.x + 1] = bfr;
        part[3 * blockIdx.x + 2] = 0.0;
    }
}

// --------------------------------------------------------------- control
// Fixed-order reduction of nslots x 3 partials (trace, ||X||^2, ||P - X||^2).
template <int NW>
__device__ void reduce3(const double* __restrict__ part, int nslots, double out[3]) {
    double a = 0.0, b = 0.0, c = 0.0;
    for (int k = threadIdx.x; k < nslots; k += 64 * NW) {
        a += part[3 * k];
        b += part[3 * k + 1];
        c += part[3 * k + 2];
    }
    __shared__ double sh[NW];
    if constexpr (NW == 4) {
        out[0] = block_sum256(a, sh);
        out[1] = block_sum256(b, sh);
        out[2] = block_sum256(c, sh);
    } else {
        out[0] = block_sum<NW>(a, sh);
        out[1] = block_sum<NW>(b, sh);
        out[2] = block_sum<NW>(c, sh);
    }
}

__global__ __launch_bounds__(256) void k_ctrl_init(const double* __restrict__ part, int nslots,
                                                   State* __restrict__ st, CtrlArgs a) {
    double r[3];
    reduce3<4>(part, nslots, r);
    if (threadIdx.x == 0) {
        (void)take_fill(st, a);
        st->t1 = r[0];
        st->t2 = r[1];
        const int b = choose_branch(r[0], r[1], a.n_occ);
        st->branch = b;
        set_bit(st, 0, b);
        // phase 0: FP64 products; 1: the reduced-precision (int8 or BF16)
        // products; 2: FP32 products (mixed 3 throughout)
        st->phase = a.mixed == 3 ? 2 : ((a.mixed != 0 && a.fp64_head == 0) ? 1 : 0);
        if (st->phase == 1) st->head_switch = 0;
    }
}

template <int NW>
__device__ __forceinline__ void ctrl_step_body(const double* __restrict__ part, int nslots, State* __restrict__ st,
                                               const CtrlArgs& a) {
    if (st->done) return;
    double r[3];
    reduce3<NW>(part, nslots, r);
    if (threadIdx.x == 0) ctrl_apply(r, st, a);
}

// Control step after product g - 1; writes the progress word (progress_word)
// to host memory.  One workgroup adds all the partials, so its time is a chain
// of loads: 4 waves up to 2048 triples (4.6-7.5 us), 16 beyond (N = 16384, 8256
// triples: 15.2 us on 4 waves, 9.5 on 16).
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_ctrl_step(const double* __restrict__ part, int nslots,
                                                       State* __restrict__ st, CtrlArgs a, int* __restrict__ progress,
                                                       int g) {
    ctrl_step_body<NW>(part, nslots, st, a);
    if (threadIdx.x == 0)
        __hip_atomic_store(progress,
                           progress_word(g, st->done, a.total_blocks > 0.0 ? (double)st->fill[g - 1] : 0.0),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One workgroup per system of a grouped launch.
__global__ __launch_bounds__(256) void k_ctrl_step_grouped(const GroupDesc* __restrict__ g) {
    const int s = blockIdx.x;
    if (s >= g->nsys) return;
    const SysView& v = g->sys[s];
    ctrl_step_body<4>(v.part, g->tile_off[s + 1] - g->tile_off[s], v.st, v.ctrl);
}

// ------------------------------------------------- FP64 symmetric product
// P = X X for symmetric X: P_ij = sum_k X_ki X_kj, so both MFMA operands are
// read as contiguous row segments of X (rows k, columns i or j), and only
// tiles with bi <= bj are computed; each is written to (bi,bj) and mirrored.
// Tile 128 x 128, 4 waves in a 2 x 2 arrangement, each wave 64 x 64 as 4 x 4
// blocks of v_mfma_f64_16x16x4f64.  K staged through LDS 16 at a time with
// register prefetch of the next stage (double-buffered LDS).
// Fused epilogue: X_{n+1} = P (branch 0) or 2 X_n - P (branch 1), written to
// the other buffer; per-tile partials Tr X_{n+1}, ||X_{n+1}||_F^2,
// ||P - X_n||_F^2 (off-diagonal tiles count twice) into part[3 * tile].
constexpr int GB = 128;   // tile
constexpr int GK = 16;    // k per stage
constexpr int GS = GB;      // LDS row stride (doubles)
constexpr int F64_NST = 2;  // LDS stages (double buffer: 2 stages x 2 operands x 16 KiB)

// Tile id t -> (bi, bj), bi <= bj, row-major over the upper triangle.
__device__ __forceinline__ void tri_coords(int t, int nt, int& bi, int& bj) {
    int i = 0, off = 0;
    while (t >= off + (nt - i)) { off += nt - i; ++i; }
    bi = i;
    bj = i + (t - off);
}

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of tile ids so tiles sharing row panels share an L2.
__device__ __forceinline__ int xcd_remap(int w, int T) {
    const int q = T >> 3, r = T & 7;
    const int x = w & 7, k = w >> 3;
    return x * q + (x < r ? x : r) + k;
}

// One 128 x 128 output tile (bi, bj); all 256 threads take part.  kmode 0:
// the whole tile; kmode 1: only K stages [kc0, kc1), whose accumulators are
// stored to chunk (one chunk of a tile split along K); kmode 2: no K loop,
// the accumulators are the sum of the nchunks chunks at chunk, added in
// chunk order, then the epilogue.  Chunk layout: d4 [16 blocks][256
// threads] (accumulator block m * 4 + n of each thread), 128 KiB.
template <bool THR>
__device__ __forceinline__ void f64_tile(double* __restrict__ buf0, double* __restrict__ buf1, int ld,
                                         const State* __restrict__ st, double* __restrict__ part,
                                         const int* __restrict__ env, int bi, int bj, int kmode, int kc0,
                                         int kc1, double* __restrict__ chunk, int nchunks) {
    const int nt = ld / GB;
    const int t = tri_index(bi, bj, nt);
    const double* __restrict__ Xc = st->cur ? buf1 : buf0;
    double* __restrict__ Xn = st->cur ? buf0 : buf1;
    const int i0 = bi * GB, j0 = bj * GB;

    // LDS double buffer; each operand row of a stage is one contiguous 1 KiB
    // row segment of X
    __shared__ double As[F64_NST][GK][GS];
    __shared__ double Bs[F64_NST][GK][GS];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wi = w >> 1, wj = w & 1;

    // global -> register staging: 4 double2 per operand per thread (loads
    // straight into LDS were measured slower for FP64)
    const int lrow = tid >> 6;           // + 4*s
    const int lcol = 2 * (tid & 63);
    double2 ra[4], rb[4];
    auto gload = [&](int k0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const size_t off = (size_t)(k0 + lrow + 4 * s) * ld;
            ra[s] = *reinterpret_cast<const double2*>(Xc + off + i0 + lcol);
            rb[s] = *reinterpret_cast<const double2*>(Xc + off + j0 + lcol);
        }
    };
    auto sstore = [&](int stg) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            As[stg][lrow + 4 * s][lcol] = ra[s].x;
            As[stg][lrow + 4 * s][lcol + 1] = ra[s].y;
            Bs[stg][lrow + 4 * s][lcol] = rb[s].x;
            Bs[stg][lrow + 4 * s][lcol + 1] = rb[s].y;
        }
    };

    d4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};

    // K stages: all of them (or the chunk [kc0, kc1)), or for a thresholded X
    // the 16-wide stages of the 32-column blocks set in both row panels'
    // block masks (elsewhere one of the two operands is zero, so skipping
    // those stages leaves every sum bitwise unchanged)
    int ks = 0, ke = ld / GK;
    if (kc1 >= 0) {
        ks = kc0;
        ke = kc1;
    }
    if (kmode == 2) ke = ks;                   // accumulators come from the chunks
    const int nbk = ld / 32;
    unsigned long long mword = 0ull;
    if (THR) {
        const unsigned long long* mk = env_mask(env, nt);
        mword = common_mask_word(mk + (size_t)bi * mask_words(ld), mk + (size_t)bj * mask_words(ld), nbk);
    }
    auto next_stage = [&](int s) -> int {      // first working stage >= s, or ke
        if (!THR || s >= ke) return s;
        const int b = next_block_in_wave(mword, s >> 1, nbk);
        return b >= nbk ? ke : max(s, 2 * b);
    };
    auto compute = [&](int stg) {
#pragma unroll
        for (int k4 = 0; k4 < GK / 4; ++k4) {
            const int kr = k4 * 4 + (lane >> 4);
            double av[4], bv[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) av[m] = As[stg][kr][wi * 64 + m * 16 + (lane & 15)];
#pragma unroll
            for (int n = 0; n < 4; ++n) bv[n] = Bs[stg][kr][wj * 64 + n * 16 + (lane & 15)];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[m], bv[n], acc[m][n], 0, 0, 0);
        }
    };
    int kt = next_stage(ks);
    if (kt < ke) {
        gload(kt * GK);
        sstore(0);
        __syncthreads();
        int stg = 0;
        while (kt < ke) {
            const int kn = next_stage(kt + 1);
            if (kn < ke) gload(kn * GK);
            compute(stg);
            if (kn < ke) sstore(stg ^ 1);
            __syncthreads();
            stg ^= 1;
            kt = kn;
        }
    }

    if (kmode == 1) {
        d4* out = reinterpret_cast<d4*>(chunk);
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int n = 0; n < 4; ++n) out[(m * 4 + n) * 256 + tid] = acc[m][n];
        return;
    }
    if (kmode == 2) {
        for (int ch = 0; ch < nchunks; ++ch) {
            const d4* in = reinterpret_cast<const d4*>(chunk + (size_t)ch * kF64Chunk);
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 4; ++n) acc[m][n] += in[(m * 4 + n) * 256 + tid];
        }
    }

    // fused SP2 update + partials
    const int br = st->branch;
    const bool mirror = bi != bj;
    double tr = 0.0, fro = 0.0, idm = 0.0;
    // one straight-line body per mirrored flag: it is uniform, and branching
    // on it per element keeps many values live across blocks
    auto epilogue = [&](auto mirc) {
        constexpr bool MIR = decltype(mirc)::value;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const int gj = j0 + wj * 64 + n * 16 + (lane & 15);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // v_mfma_f64_16x16x4f64 result: lane l, element r is row (l >> 4) + 4 r, column l & 15
                    const int gi = i0 + wi * 64 + m * 16 + (lane >> 4) + 4 * r;
                    const double p = acc[m][n][r];
                    const double x = Xc[(size_t)gi * ld + gj];
                    const double xn = br ? 2.0 * x - p : p;
                    Xn[(size_t)gi * ld + gj] = xn;
                    if constexpr (MIR) Xn[(size_t)gj * ld + gi] = xn;
                    tr += gi == gj ? xn : 0.0;
                    fro += xn * xn;
                    idm += (p - x) * (p - x);
                }
            }
        }
    };
    if (mirror) epilogue(std::true_type{});
    else epilogue(std::false_type{});
    const double wgt = mirror ? 2.0 : 1.0;
    __shared__ double sh[4];
    const double btr = block_sum256(tr, sh);
    const double bfr = block_sum256(fro, sh);
    const double bid = block_sum256(idm, sh);
    if (tid == 0) {
        part[3 * t + 0] = btr;
        part[3 * t + 1] = wgt * bfr;
        part[3 * t + 2] = wgt * bid;
    }
}

// At most 256 registers per lane: the accumulators then stay in VGPR form
// (with the whole register file the compiler splits them between VGPRs and
// AGPRs and copies them across on every K stage) and two workgroups fit on
// a CU (LDS 64 KiB each), so one hides the other's barriers and epilogue.
// Workgroups [0, t_full): whole tiles at visiting positions [0, t_full),
// dealt over the XCDs.  Workgroups from t_full on: the tiles at positions
// t_full, t_full + 1, ... (the last, partly filled wave of a launch), each
// split into nsplit chunks of the K loop whose accumulators go to chunk;
// k_gemm_f64_tail finishes them.
template <bool THR>
__global__ __launch_bounds__(256, 2) void k_gemm_f64(double* __restrict__ buf0,
                                                     double* __restrict__ buf1, int ld,
                                                     const State* __restrict__ st,
                                                     double* __restrict__ part,
                                                     const int* __restrict__ env, int tile_group, int t_full,
                                                     int nsplit, double* __restrict__ chunk) {
    if (st->done || st->phase != 0) return;
    const int nt = ld / GB, w = blockIdx.x;
    int pos, kmode = 0, kc0 = 0, kc1 = -1;
    double* cacc = nullptr;
    if (w < t_full) {
        pos = xcd_deal(w, t_full);
    } else {
        const int j = w - t_full, p = j / nsplit, ch = j - p * nsplit, nk = ld / GK;
        pos = t_full + p;
        kmode = 1;
        kc0 = ch * nk / nsplit;
        kc1 = (ch + 1) * nk / nsplit;
        cacc = chunk + (size_t)j * kF64Chunk;
    }
    int bi, bj;
    order_tile(pos, nt, tile_group, bi, bj);
    f64_tile<THR>(buf0, buf1, ld, st, part, env, bi, bj, kmode, kc0, kc1, cacc, 0);
}

// Small products (ld <= kSmallMaxLd): the 128 x 128 tiles occupy a part of the
// CUs, or leave a round nearly empty, and splitting them along K adds a second
// launch that reads the chunks back.  Instead one workgroup of NW waves per 32 x 32
// upper tile (T = nt(nt+1)/2, nt = ld / 32): each wave multiplies its share of
// the K range with operands loaded straight into registers, the partial tiles
// are added in LDS in wave order, and the fused update and the partials
// follow as in the large kernel (one slot per 32 x 32 tile).  With the
// pipelined K loop of small_f64.h and the tile of X_n loaded beside it a
// product takes 6.6 us at N = 256 (9.1 before), 9.5 at 512 (14.7), 33.7 at
// 1024 (48.4), 75 at 1536 (149; 100 on 128 x 128 tiles), 169 at 2048 (282;
// 200).  At N = 1024 and above the matrix cores are busy 45-70 % of it; 64 x 32
// tiles (a quarter less L2 traffic, half the waves) took 175 us at 2048.
template <int NW, bool FOLD>
__global__ __launch_bounds__(64 * NW) void k_gemm_f64_small(double* __restrict__ buf0, double* __restrict__ buf1,
                                                            int ld, const State* __restrict__ st,
                                                            double* __restrict__ part, FoldArgs f) {
    constexpr int PER = kSmallTile * kSmallTile / (64 * NW);
    __shared__ double red[NW][kSmallTile][kSmallTile + 1];
    __shared__ double sh[NW];
    __shared__ FoldShared fsh;
    if (!FOLD && (st->done || st->phase != 0)) return;
    const int cur = FOLD ? f.g & 1 : st->cur;
    FoldPart fp;
    if (FOLD) fp.load(f);
    const double* __restrict__ Xc = cur ? buf1 : buf0;
    double* __restrict__ Xn = cur ? buf0 : buf1;
    const int nts = ld / kSmallTile;
    int bi, bj;
    tile_of_block(blockIdx.x, nts, 16, bi, bj);
    const int t = tri_index(bi, bj, nts), i0 = bi * kSmallTile, j0 = bj * kSmallTile;
    const int tid = threadIdx.x, w = tid >> 6;
    double x[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = tid + 64 * NW * q;
        x[q] = Xc[(size_t)(i0 + (e >> 5)) * ld + j0 + (e & 31)];
    }
    const int nk = ld / 4;
    d4s acc[2][2];
    small_mma<false, true>(Xc, Xc, ld, ld, i0, j0, w * nk / NW, (w + 1) * nk / NW, acc);
    small_store(&red[w][0][0], acc);
    int done = 0, br;
    if (FOLD) {
        fold_decide<true>(f, fp, fsh, &done, &br);   // its barriers cover red
        if (done) return;
        if (f.g == 0) __syncthreads();
    } else {
        br = st->branch;
        __syncthreads();
    }
    double tr = 0.0, fro = 0.0, idm = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = tid + 64 * NW * q, r = e >> 5, c = e & 31;
        const int gi = i0 + r, gj = j0 + c;
        if (gi > gj) continue;
        double p = red[0][r][c];
#pragma unroll
        for (int v = 1; v < NW; ++v) p += red[v][r][c];
        const double xn = br ? 2.0 * x[q] - p : p;
        const double wgt = gi == gj ? 1.0 : 2.0;   // the mirrored element's share
        Xn[(size_t)gi * ld + gj] = xn;
        if (gi != gj) Xn[(size_t)gj * ld + gi] = xn;
        tr += gi == gj ? xn : 0.0;
        fro += wgt * xn * xn;
        idm += wgt * (p - x[q]) * (p - x[q]);
    }
    const double btr = block_sum<NW>(tr, sh);
    const double bfr = block_sum<NW>(fro, sh);
    const double bid = block_sum<NW>(idm, sh);
    if (tid == 0) {
        part[3 * t + 0] = btr;
        part[3 * t + 1] = bfr;
        part[3 * t + 2] = bid;
    }
}

// Epilogue of the split tiles: workgroup p sums the nsplit chunks of the tile
// at visiting position t_full + p and applies the update.
__global__ __launch_bounds__(256, 2) void k_gemm_f64_tail(double* __restrict__ buf0, double* __restrict__ buf1,
                                                          int ld, const State* __restrict__ st,
                                                          double* __restrict__ part, int tile_group, int t_full,
                                                          int nsplit, double* __restrict__ chunk) {
    if (st->done || st->phase != 0) return;
    const int nt = ld / GB, p = blockIdx.x;
    int bi, bj;
    order_tile(t_full + p, nt, tile_group, bi, bj);
    f64_tile<false>(buf0, buf1, ld, st, part, nullptr, bi, bj, 2, 0, -1, chunk + (size_t)p * nsplit * kF64Chunk,
                    nsplit);
}

// ---------------------------------------------------------------- finalize
__global__ __launch_bounds__(256) void k_finalize(const double* __restrict__ buf0,
                                                  const double* __restrict__ buf1, int ld, int N,
                                                  double* __restrict__ D,
                                                  const State* __restrict__ st) {
    const double* X = st->result ? buf1 : buf0;
    const size_t total = (size_t)N * N;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
        const size_t i = e / N, j = e - i * N;
        D[e] = X[i * ld + j];
    }
}

// D of a thresholded int8 solve: one workgroup per 128 x 128 tile, a tile
// flagged all zero (tz, per X buffer and upper tile) written without a read.
// VEC (N even, D 16-byte aligned): two columns per store.  N = 16384 banded:
// 918 -> 444 us for 2.1 GB of D.
template <bool VEC>
__global__ __launch_bounds__(256) void k_finalize_tiles(const double* __restrict__ buf0,
                                                        const double* __restrict__ buf1, int ld, int N,
                                                        double* __restrict__ D, const State* __restrict__ st,
                                                        const int* __restrict__ tz) {
    const int nt = ld / kTile, bi = blockIdx.y, bj = blockIdx.x;
    const double* __restrict__ X = st->result ? buf1 : buf0;
    const bool zero = tz[(size_t)st->result * (nt * (nt + 1) / 2) + tri_index(min(bi, bj), max(bi, bj), nt)] != 0;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if constexpr (VEC) {
        const int j = bj * kTile + 2 * lane;
        if (j >= N) return;
        const int i1 = min(N, (bi + 1) * kTile);
#pragma unroll 8
        for (int i = bi * kTile + w; i < i1; i += 4) {
            double2 v = make_double2(0.0, 0.0);
            if (!zero) v = *reinterpret_cast<const double2*>(X + (size_t)i * ld + j);
            *reinterpret_cast<double2*>(D + (size_t)i * N + j) = v;
        }
    } else {
        const int i1 = min(N, (bi + 1) * kTile);
        for (int i = bi * kTile + w; i < i1; i += 4)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = bj * kTile + 64 * h + lane;
                if (j < N) D[(size_t)i * N + j] = zero ? 0.0 : X[(size_t)i * ld + j];
            }
    }
}

// D from an X whose upper triangle (32 x 32 blocks I <= J) is valid: each
// workgroup copies block (I, J) and its transpose (through LDS) to D.
__global__ __launch_bounds__(256) void k_finalize_upper(const double* __restrict__ buf0,
                                                        const double* __restrict__ buf1, int ld, int N,
                                                        double* __restrict__ D,
                                                        const State* __restrict__ st) {
    const double* X = st->result ? buf1 : buf0;
    const int nb = (N + 31) / 32;
    const int t = blockIdx.x;
    int I = (int)((2.0 * nb + 1.0 - sqrt((2.0 * nb + 1.0) * (2.0 * nb + 1.0) - 8.0 * (double)t)) / 2.0);
    I = max(0, min(I, nb - 1));
    while (I > 0 && I * nb - I * (I - 1) / 2 > t) --I;
    while (I + 1 < nb && (I + 1) * nb - (I + 1) * I / 2 <= t) ++I;
    const int J = I + (t - (I * nb - I * (I - 1) / 2));
    __shared__ double T[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int r = ty; r < 32; r += 8) {
        const int i = I * 32 + r, j = J * 32 + tx;      // i, j < ld: X is padded with zeros
        const double x = X[(size_t)i * ld + j];
        T[r][tx] = x;
        if (i < N && j < N) D[(size_t)i * N + j] = x;
    }
    if (I == J) return;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int i = J * 32 + r, j = I * 32 + tx;
        if (i < N && j < N) D[(size_t)i * N + j] = T[tx][r];
    }
}

// Symmetric test operand for timing (the autotuner): X_ij = X_ji in (-1/2, 1/2)
// from an integer hash of (min(i, j), max(i, j)), so that products switch as
// many bits (and draw as much power) as on real data.
__global__ __launch_bounds__(256) void k_fill_test_matrix(double* __restrict__ X, int ld) {
    const size_t total = (size_t)ld * ld;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
        const unsigned i = (unsigned)(e / ld), j = (unsigned)(e % ld);
        unsigned h = (i < j ? i : j) * 0x9E3779B1u ^ (i < j ? j : i) * 0x85EBCA77u;
        h ^= h >> 15;
        h *= 0x2C1B3C6Du;
        h ^= h >> 12;
        X[e] = (double)(h >> 8) / 16777216.0 - 0.5;
    }
}

// ------------------------------------------------------------ observables
__global__ __launch_bounds__(256) void k_mulliken(const double* __restrict__ D, int n_atoms,
                                                  double z, double* __restrict__ q) {
    const int a = blockIdx.x * 256 + threadIdx.x;
    if (a >= n_atoms) return;
    const size_t N = 4 * (size_t)n_atoms;
    double s = 0.0;
    for (int k = 0; k < 4; ++k) {
        const size_t o = 4 * (size_t)a + k;
        s += D[o * N + o];
    }
    q[a] = 2.0 * s - z;
}

// sum_e A[e] B[e] with a fixed grid of 512 workgroups, then a one-workgroup
// fixed-order reduction into *out (device).
// Partial sums of sum_e A_e B_e, one per workgroup, in a fixed order;
// 16-byte loads when both operands are 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(256) void k_dot_part(const double* __restrict__ A,
                                                  const double* __restrict__ B, size_t n,
                                                  double* __restrict__ part) {
    double s = 0.0;
    const size_t stride = (size_t)kDotBlocks * 256;
    if (VEC) {
        const double2* __restrict__ A2 = reinterpret_cast<const double2*>(A);
        const double2* __restrict__ B2 = reinterpret_cast<const double2*>(B);
        for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n / 2; e += stride) {
            const double2 a = A2[e], b = B2[e];
            s += a.x * b.x;
            s += a.y * b.y;
        }
        if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) s += A[n - 1] * B[n - 1];
    } else {
        for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += stride) s += A[e] * B[e];
    }
    __shared__ double sh[4];
    const double b = block_sum256(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}
__global__ __launch_bounds__(256) void k_dot_final(const double* __restrict__ part, int nslots,
                                                   double* __restrict__ out) {
    double s = 0.0;
    for (int k = threadIdx.x; k < nslots; k += 256) s += part[k];
    __shared__ double sh[4];
    const double b = block_sum256(s, sh);
    if (threadIdx.x == 0) *out = b;
}

// ---------------------------------------------------------------- launchers
hipError_t launch_gershgorin(const double* H, int N, double* part, int* nslots, hipStream_t s, const unsigned* hz) {
    const int g = (N + 3) / 4;
    *nslots = g;
    if (hz) hipLaunchKernelGGL(k_gershgorin<true>, dim3(g), dim3(256), 0, s, H, N, part, hz);
    else hipLaunchKernelGGL(k_gershgorin<false>, dim3(g), dim3(256), 0, s, H, N, part, nullptr);
    return hipGetLastError();
}
hipError_t launch_check_h(const double* H, int N, double* out, int* nout, hipStream_t s, unsigned* hz) {
    const long long nb = (N + 31) / 32;
    const int g = (int)std::min<long long>(nb * (nb + 1) / 2, kCheckGrid);
    *nout = g;
    if (hz)
        hipLaunchKernelGGL(k_check_h<true>, dim3(g), dim3(256), 0, s, H, N, out, reinterpret_cast<unsigned char*>(hz));
    else
        hipLaunchKernelGGL(k_check_h<false>, dim3(g), dim3(256), 0, s, H, N, out, nullptr);
    return hipGetLastError();
}
hipError_t launch_bounds(const double* part, int nslots, const double* chk, int nchk, State* st, hipStream_t s) {
    hipLaunchKernelGGL(k_bounds, dim3(1), dim3(256), 0, s, part, nslots, chk, nchk, st);
    return hipGetLastError();
}
hipError_t launch_init(const double* H, int N, int ld, double* X0, State* st, double* part,
                       int* nslots, hipStream_t s, unsigned long long* rmax0) {
    const int g = ld / 4;
    *nslots = g;
    hipLaunchKernelGGL(k_init, dim3(g), dim3(256), 0, s, H, N, ld, X0, st, part, rmax0);
    return hipGetLastError();
}
hipError_t launch_ctrl_init(const double* part, int nslots, State* st, CtrlArgs a, hipStream_t s) {
    hipLaunchKernelGGL(k_ctrl_init, dim3(1), dim3(256), 0, s, part, nslots, st, a);
    return hipGetLastError();
}
hipError_t launch_ctrl_step(const double* part, int nslots, State* st, CtrlArgs a, int* progress, int g,
                            hipStream_t s) {
    if (nslots <= 2048)
        hipLaunchKernelGGL(k_ctrl_step<4>, dim3(1), dim3(256), 0, s, part, nslots, st, a, progress, g);
    else
        hipLaunchKernelGGL(k_ctrl_step<16>, dim3(1), dim3(1024), 0, s, part, nslots, st, a, progress, g);
    return hipGetLastError();
}
hipError_t launch_ctrl_step_grouped(const GroupDesc* g, hipStream_t s) {
    hipLaunchKernelGGL(k_ctrl_step_grouped, dim3(kMaxGroup), dim3(256), 0, s, g);
    return hipGetLastError();
}
bool small_f64_tile(int ld) {
    if (ld >= 4096) return false;
    const int cus = device_cus(), rounds = (tri_tiles(ld / GB) + cus - 1) / cus;
    return 1.82e-8 * (256.0 / cus) * ld * ld < 0.13 * rounds;
}
hipError_t launch_gemm_f64_folded(double* buf0, double* buf1, int ld, const FoldArgs& f, double* part_out,
                                  hipStream_t s) {
    const int T = tri_tiles(ld / kSmallTile);
    if (ld <= kSmallWideLd)
        hipLaunchKernelGGL((k_gemm_f64_small<8, true>), dim3(T), dim3(512), 0, s, buf0, buf1, ld, f.in, part_out, f);
    else
        hipLaunchKernelGGL((k_gemm_f64_small<4, true>), dim3(T), dim3(256), 0, s, buf0, buf1, ld, f.in, part_out, f);
    return hipGetLastError();
}
hipError_t launch_gemm_f64(double* buf0, double* buf1, int ld, State* st, double* part,
                           int* nslots, hipStream_t s, const int* env, int tile_group, double* tail_buf,
                           size_t tail_bytes, int split_cap, bool small_ok) {
    if (small_ok && !env && ld <= kSmallMaxLd) {
        const int T = tri_tiles(ld / kSmallTile);
        *nslots = T;
        if (ld <= kSmallWideLd)
            hipLaunchKernelGGL((k_gemm_f64_small<8, false>), dim3(T), dim3(512), 0, s, buf0, buf1, ld, st, part, FoldArgs{});
        else
            hipLaunchKernelGGL((k_gemm_f64_small<4, false>), dim3(T), dim3(256), 0, s, buf0, buf1, ld, st, part, FoldArgs{});
        return hipGetLastError();
    }
    const int nt = ld / GB;
    const int T = tri_tiles(nt);
    *nslots = T;
    // Tiles of a last wave that would leave at least half of the workgroup
    // slots (two per CU) idle are split along K into nsplit <= 16 chunks,
    // when a tile's K loop covers at least 4096 columns.  A smaller product
    // whose tiles fill at most half of the slots is latency-bound (each
    // workgroup walks its K stages one after another): all of its tiles are
    // split.  The chunk count balances the stages a chunk walks (~2.8 us
    // each) against the chunks the tail kernel reads back one after another
    // (~2 us each): about sqrt(1.4 nk), at most split_cap and no more than fit.
    int t_full = T, nsplit = 1;
    if (!env && tail_buf) {
        const int slots = 2 * device_cus();
        const int nk = ld / GK;
        int r = 0;
        if (nk >= 256) {
            r = T % slots;
            if (r > 0 && 2 * r <= slots) nsplit = std::min(split_cap, slots / r);
        } else if (2 * T <= slots) {
            r = T;
            nsplit = std::min({split_cap, slots / T, nk, (int)std::lround(std::sqrt(1.4 * nk))});
        }
        if (nsplit >= 2 && (size_t)r * nsplit * kF64Chunk * sizeof(double) <= tail_bytes) t_full = T - r;
        else nsplit = 1;
    }
    const int grid = t_full + (T - t_full) * nsplit;
    if (env)
        hipLaunchKernelGGL(k_gemm_f64<true>, dim3(grid), dim3(256), 0, s, buf0, buf1, ld, st, part, env, tile_group,
                           t_full, nsplit, tail_buf);
    else
        hipLaunchKernelGGL(k_gemm_f64<false>, dim3(grid), dim3(256), 0, s, buf0, buf1, ld, st, part, env,
                           tile_group, t_full, nsplit, tail_buf);
    if (t_full < T)
        hipLaunchKernelGGL(k_gemm_f64_tail, dim3(T - t_full), dim3(256), 0, s, buf0, buf1, ld, st, part, tile_group,
                           t_full, nsplit, tail_buf);
    return hipGetLastError();
}
hipError_t launch_finalize(const double* buf0, const double* buf1, int ld, int N, double* D,
                           const State* st, hipStream_t s) {
    size_t total = (size_t)N * N;
    int g = (int)((total + 255) / 256);
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_finalize, dim3(g), dim3(256), 0, s, buf0, buf1, ld, N, D, st);
    return hipGetLastError();
}
hipError_t launch_finalize_tiles(const double* buf0, const double* buf1, int ld, int N, double* D, const State* st,
                                 const int* tz, hipStream_t s) {
    const dim3 grid(ld / kTile, ld / kTile);
    if (N % 2 == 0 && reinterpret_cast<uintptr_t>(D) % 16 == 0)
        hipLaunchKernelGGL(k_finalize_tiles<true>, grid, dim3(256), 0, s, buf0, buf1, ld, N, D, st, tz);
    else
        hipLaunchKernelGGL(k_finalize_tiles<false>, grid, dim3(256), 0, s, buf0, buf1, ld, N, D, st, tz);
    return hipGetLastError();
}
hipError_t launch_finalize_upper(const double* buf0, const double* buf1, int ld, int N, double* D,
                                 const State* st, hipStream_t s) {
    const int nb = (N + 31) / 32;
    hipLaunchKernelGGL(k_finalize_upper, dim3(nb * (nb + 1) / 2), dim3(256), 0, s, buf0, buf1, ld, N, D, st);
    return hipGetLastError();
}
hipError_t launch_fill_test_matrix(double* X, int ld, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_test_matrix, dim3(2048), dim3(256), 0, s, X, ld);
    return hipGetLastError();
}
hipError_t launch_mulliken(const double* D, int n_atoms, double z, double* q, hipStream_t s) {
    hipLaunchKernelGGL(k_mulliken, dim3((n_atoms + 255) / 256), dim3(256), 0, s, D, n_atoms, z, q);
    return hipGetLastError();
}
hipError_t launch_dot(const double* A, const double* B, size_t n, double* part, int* nslots,
                      double* out, hipStream_t s) {
    *nslots = kDotBlocks;
    if ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) % 16 == 0)
        hipLaunchKernelGGL(k_dot_part<true>, dim3(kDotBlocks), dim3(256), 0, s, A, B, n, part);
    else
        hipLaunchKernelGGL(k_dot_part<false>, dim3(kDotBlocks), dim3(256), 0, s, A, B, n, part);
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(256), 0, s, part, kDotBlocks, out);
    return hipGetLastError();
}

}  // namespace sp2
