// Device side of the folded control step (FoldArgs).
#pragma once
#include "sp2_internal.h"

namespace sp2 {

// Branch rule: X^2 if its trace is at least as close to n_occ as that of
// 2X - X^2 (Tr X^2 = t2, Tr(2X - X^2) = 2 t1 - t2).
__device__ __forceinline__ int choose_branch(double t1, double t2, double nocc) {
    return fabs(t2 - nocc) <= fabs(2.0 * t1 - t2 - nocc) ? 0 : 1;
}

__device__ __forceinline__ void set_bit(State* st, int n, int b) {
    if (n < 128 && b) st->bits[n >> 6] |= (1ull << (n & 63));
}
__device__ __forceinline__ void clear_bit(State* st, int n) {
    if (n < 128) st->bits[n >> 6] &= ~(1ull << (n & 63));
}

// Kept-block fraction of the threshold pass that just ran (if any).
__device__ __forceinline__ double take_fill(State* st, const CtrlArgs& a) {
    if (a.total_blocks <= 0.0) return -1.0;
    const double f = (double)st->kept / a.total_blocks;
    st->kept = 0ull;
    st->full_fill = f >= a.dense_fill ? 1 : 0;
    st->fill_min = fmin(st->fill_min, f);
    st->fill_max = fmax(st->fill_max, f);
    return f;
}

// After product n: the partials hold Tr X_{n+1}, ||X_{n+1}||_F^2 and
// ||X_n^2 - X_n||_F^2.  Stop rules: e_n < idem_tol (converged, D = X_n);
// n >= 4, e_n >= r e_{n-2}, e_n < stall_tol (stalled at the floor of the
// idempotency error, D = X_n; r = 1, or 1/2 with a threshold, whose floor
// keeps creeping down); n + 1 == max_iter (not converged).  Otherwise X_{n+1} becomes
// current and the next branch is chosen from its traces.
__device__ __forceinline__ void ctrl_apply(const double r[3], State* st, const CtrlArgs& a) {
    const int n = st->iter;
    const double e = sqrt(r[2]);
    st->idem[n] = e;
    const double f = take_fill(st, a);
    if (f >= 0.0) st->fill[n] = (float)f;
    st->iter = n + 1;
    if (st->phase == 0) st->fp64_products += 1;   // FP64 products (the whole solve, or the head)
    const bool stall = n >= 4 && e >= a.stall_ratio * st->idem[n - 2] && e < a.stall_tol;
    // BF16X2 runs its own schedule: a stall of the BF16 stage starts a fixed
    // FP32 tail instead of stopping
    // a projector whose trace is not n_occ could not pick the occupied set:
    // the Fermi level is degenerate (done = 4)
    const int gap_or = fabs(st->t1 - a.n_occ) > 0.5 ? 4 : 0;
    if (e < a.idem_tol || (stall && a.mixed != 2)) {
        st->done = gap_or ? gap_or : ((e < a.idem_tol) ? 1 : 2);
        st->result = st->cur;
        clear_bit(st, n);
        return;
    }
    if (n + 1 >= a.max_iter) {
        st->done = (a.max_iter >= kGapMinIter && e >= kGapIdem) ? 4 : 3;
        st->result = 1 - st->cur;
        return;
    }
    if (a.mixed == 2 && st->phase == 2) {
        // tail product: its update X_{n+1} is applied; after fp32_tail of them, stop
        st->tail_left -= 1;
        if (st->tail_left <= 0) {
            st->done = fabs(r[0] - a.n_occ) > 0.5 ? 4 : 2;
            st->result = 1 - st->cur;
            st->t1 = r[0];
            st->t2 = r[1];
            return;
        }
    }
    if (a.mixed == 2 && st->phase == 1 && stall) {
        if (a.fp32_tail <= 0) {
            st->done = gap_or ? gap_or : 2;
            st->result = st->cur;
            clear_bit(st, n);
            return;
        }
        st->phase = 2;
        st->tail_left = a.fp32_tail;
        st->head_switch = n + 1;
    }
    st->cur = 1 - st->cur;
    st->t1 = r[0];
    st->t2 = r[1];
    const int b = choose_branch(r[0], r[1], a.n_occ);
    st->branch = b;
    set_bit(st, n + 1, b);
    if (a.mixed != 0 && st->phase == 0 && n + 1 >= a.fp64_head && a.fp64_head >= 0) {
        st->phase = 1;
        st->head_switch = n + 1;
    }
}

// What a workgroup has of the partials before its own work: one triple per
// thread of the first 256, in flight while it loads and multiplies.
struct FoldPart {
    double v[3];
    double e2;              // e_(g-3)
    int done, branch;       // of the state before the result
    __device__ __forceinline__ void load(const FoldArgs& f) {
        static_assert(kFoldSlots <= 256, "one triple per thread");
        done = f.in->done;
        branch = f.in->branch;
        e2 = f.g >= 3 ? f.in->idem[f.g - 3] : 0.0;
        const bool in = f.g > 0 && (int)threadIdx.x < f.nslots;
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] = in ? f.part[3 * threadIdx.x + q] : 0.0;
    }
};

struct FoldShared {
    double s[3][4];
    int dec[2];
};

__device__ __forceinline__ double fold_wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// All threads of the workgroup (at least 256): done and, with BRANCH, branch of
// product g, the same in every workgroup; workgroup 0 writes f.out and
// f.progress.  The sums are those of the control kernel (256 threads, then
// waves 0..3); without BRANCH only workgroup 0 needs the two traces.
template <bool BRANCH>
__device__ __forceinline__ void fold_decide(const FoldArgs& f, const FoldPart& p, FoldShared& sh, int* done,
                                            int* branch) {
    const int tid = threadIdx.x, w = tid >> 6;
    const bool writer = blockIdx.x == 0;
    if (f.g == 0) {
        *done = p.done;
        *branch = p.branch;
        return;
    }
    if (writer) {
        const int* src = reinterpret_cast<const int*>(f.in);
        int* dst = reinterpret_cast<int*>(f.out);
        for (int k = tid; k < (int)(sizeof(State) / sizeof(int)); k += blockDim.x) dst[k] = src[k];
    }
    if (w < 4) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (q < 2 && !BRANCH && !writer) continue;
            const double v = fold_wave_sum(p.v[q]);
            if ((tid & 63) == 0) sh.s[q][w] = v;
        }
    }
    __syncthreads();
    if (tid == 0) {
        double r[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) r[q] = (sh.s[q][0] + sh.s[q][1]) + (sh.s[q][2] + sh.s[q][3]);
        int d = p.done, b = p.branch;
        if (!d) {
            // the decision of ctrl_apply for FP64 and int8 products (no tail, no threshold)
            const int n = f.g - 1;
            const double e = sqrt(r[2]);
            const bool stall = n >= 4 && e >= f.ctrl.stall_ratio * p.e2 && e < f.ctrl.stall_tol;
            d = (e < f.ctrl.idem_tol || stall || n + 1 >= f.ctrl.max_iter) ? 1 : 0;
            if (BRANCH) b = choose_branch(r[0], r[1], f.ctrl.n_occ);
        }
        sh.dec[0] = d;
        sh.dec[1] = b;
        if (writer) {
            if (!p.done) ctrl_apply(r, f.out, f.ctrl);
            __hip_atomic_store(f.progress, progress_word(f.g, f.out->done, 0.0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __syncthreads();
    *done = sh.dec[0];
    *branch = sh.dec[1];
}

}  // namespace sp2
