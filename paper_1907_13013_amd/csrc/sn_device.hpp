// Device helpers shared by the FP64 kernels: launches timed by their own
// dispatch stamps, convergence gating, the iteration-relative fields of
// batched launches, and the stopping-test reduction.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "sn_kernels.hpp"

namespace snfpsa {

typedef double d4 __attribute__((ext_vector_type(4)));

// Kernel launch, timed by its own dispatch timestamps when a timer is set.
#define LAUNCH(id, t, kernel, grid, block, shm, st, ...)                                       \
    do {                                                                                       \
        hipEvent_t ev0_ = nullptr, ev1_ = nullptr;                                             \
        if ((t) && (t)->events((id), &ev0_, &ev1_))                                            \
            hipExtLaunchKernelGGL(kernel, grid, block, shm, st, ev0_, ev1_, 0, __VA_ARGS__);   \
        else                                                                                   \
            hipLaunchKernelGGL(kernel, grid, block, shm, st, __VA_ARGS__);                     \
    } while (0)

__device__ __forceinline__ bool skipped(const SkipTest &t) {
    if (!t.prev) return false;
    const double d = __longlong_as_double((long long)*t.prev);
    return d <= t.tol || !isfinite(d);
}

// Iteration-relative fields of a batched launch's descriptor (see
// MultiEntry): iteration m reads buffer (m - 1) & 1 and writes buffer m & 1
// of the slab's iterates, offset by the entry's rows.
__device__ __forceinline__ double *iter_buf(const IterPatch &p, int k) { return ((k & 1) ? p.phiB : p.phiA) + p.off; }
__device__ __forceinline__ unsigned long long *iter_slot(const IterPatch &p, int m) {
    return p.hist + hist_row(m) * (size_t)p.hist_stride;
}
__device__ __forceinline__ void patch_skip(SkipTest &sk, const IterPatch &p, int m) {
    if (p.flags & PATCH_SKIP) sk.prev = m > 1 ? iter_slot(p, m - 1) : nullptr;
}
__device__ __forceinline__ void apply_patch(SweepArgs &s, const IterPatch &p, int m) {
    patch_skip(s.skip, p, m);
    if (p.flags & PATCH_SRC_CUR) s.src_phi = iter_buf(p, m - 1);
    if (p.flags & PATCH_MOM_NXT) s.mom_out = iter_buf(p, m);
    if (p.flags & PATCH_MOM_STOP) {
        s.mom_ref = iter_buf(p, m - 1);
        s.mom_slot = iter_slot(p, m);
    }
}
__device__ __forceinline__ void apply_patch(GemmArgs &g, const IterPatch &p, int m) {
    patch_skip(g.skip, p, m);
    if (p.flags & PATCH_A1_CUR) g.A1 = iter_buf(p, m - 1);
    if (p.flags & PATCH_A1SUB_CUR) g.A1sub = iter_buf(p, m - 1);
    if (p.flags & PATCH_C_NXT) g.C = iter_buf(p, m);
    if (p.flags & PATCH_STOP) {
        g.stop_ref = iter_buf(p, m - 1);
        g.stop_slot = iter_slot(p, m);
    }
}
__device__ __forceinline__ void apply_patch(FPArgs &f, const IterPatch &p, int m) { patch_skip(f.skip, p, m); }
__device__ __forceinline__ void apply_patch(StopArgs &a, const IterPatch &p, int m) {
    patch_skip(a.skip, p, m);
    if (p.flags & PATCH_STOPTEST) {
        a.a = iter_buf(p, m);
        a.b = iter_buf(p, m - 1);
        a.slot = iter_slot(p, m);
    }
}

// ---------------------------------------------------------------------------
// Stopping test (eq:iterate) reduction shared by the stand-alone kernel and
// the fused GEMM epilogue: each block folds its maximum of |x - y| into the
// iteration's slot as the IEEE bit pattern of a non-negative double (ordered
// like unsigned integers; NaN sorts above +Inf, so a NaN anywhere surfaces
// as NaN).  The test itself is applied by the next iteration's kernels and
// by the host.  Called by all threads of the block.
// ---------------------------------------------------------------------------
__device__ inline void stop_block_reduce(unsigned long long m, unsigned long long *slot) {
    __shared__ unsigned long long red[16];
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(m, off, 64);
        m = o > m ? o : m;
    }
    const int nw = (blockDim.x + 63) / 64;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < nw; ++i) m = red[i] > m ? red[i] : m;
        atomicMax(slot, m);
    }
}

__device__ __forceinline__ unsigned long long absdiff_bits(double x, double y) {
    return (unsigned long long)__double_as_longlong(fabs(x - y));
}

}  // namespace snfpsa
