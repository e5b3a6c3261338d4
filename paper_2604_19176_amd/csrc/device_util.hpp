// device_util.hpp -- device helpers shared by the kernels' translation units.
#pragma once

#include "fft.hpp"
#include "pat_internal.hpp"

namespace pat {

// XCD-aware work mapping.  The hardware hands workgroup w to XCD (w mod 8);
// remap so that XCD x owns the contiguous item range [start(x), start(x+1))
// of the U work items (instance-major), keeping one instance's intermediates
// in one XCD's L2.  Returns -1 for the padding workgroups of the last round.
__device__ __forceinline__ int xcd_item(int w, int U)
{
    const int x = w % kXcds, q = w / kXcds;
    const int Q = U / kXcds, Rm = U - Q * kXcds;
    const int cnt = Q + (x < Rm ? 1 : 0);
    if (q >= cnt) return -1;
    return x * Q + min(x, Rm) + q;
}

// The 8 taps of the ES kernel phi(t) = exp(beta (sqrt(1 - (2t/w)^2) - 1)) at
// t = frac + 3 - d (d = 0..7, frac in [0, 1]): z = t / 4 lies in [-1, 1] also
// when rounded, so 1 - z^2, rounded once, is never negative; the hardware square
// root and base-2 exponential (about 1 ulp each) are used directly, since the
// argument of the exponential lies in [-beta log2(e), 0].  The same routine
// serves the interpolation and the spread, which keeps them exact transposes.
__device__ __forceinline__ void es_weights8(float frac, float (&w)[8])
{
    constexpr float kb = (float)(kEsBeta * 1.4426950408889634);  // beta log2(e)
    const float z0 = frac * 0.25f;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const float z = z0 + 0.25f * (float)(3 - d);
        w[d] = __builtin_amdgcn_exp2f(fmaf(kb, __builtin_amdgcn_sqrtf(fmaf(-z, z, 1.0f)), -kb));
    }
}

__device__ __forceinline__ int fbits(float v) { return __float_as_int(v); }

// Sum of v[0..n) in an order fixed by n alone (64 strided partial sums, then a
// fixed shuffle tree): the same bits for every workgroup size.  Must be
// reached by all threads of the first wave; the total is returned to lane 0.
__device__ __forceinline__ float wave0_fixed_sum(const float* __restrict__ v, int n)
{
    float s = 0.f;
    for (int t = threadIdx.x; t < n; t += 64) s += v[t];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    return s;
}

// st(t, ld(t)) for t < count by the workgroup (t = t0 + threadIdx.x + j blockDim.x,
// U values of t per thread and chunk).  A chunk issues all of a thread's loads
// before its first store, and no load sits under a divergent branch (indices
// past the end are clamped to count - 1 and their values dropped), so a chunk
// waits for one memory latency instead of one per element.
template <int U, class Ld, class St>
__device__ __forceinline__ void fill_batched(int count, Ld ld, St st)
{
    const int tid = threadIdx.x, bd = blockDim.x;
    for (int t0 = 0; t0 < count; t0 += U * bd) {
        decltype(ld(0)) v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = ld(min(t0 + tid + j * bd, count - 1));
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int t = t0 + tid + j * bd;
            if (t < count) st(t, v[j]);
        }
    }
}

struct IdxVal {
    int i;
    float2 v;
};

struct IdxF {
    int i;
    float v;
};

// ---------------------------------------------------------------------------
// Launch wrappers.  Single-plan kernels: `batch` instances of one plan with
// instance workspaces `wsp.stride` bytes apart.  Batch kernels (suffix _b):
// one launch covers every instance of a heterogeneous batch; the workgroup's
// work item is located in the per-stage prefix table and the instance's plan
// is read from the device table.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int batch_find(const int* __restrict__ base, int count, int item)
{
    int lo = 0, hi = count;  // base[lo] <= item < base[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (base[mid] <= item) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Locates the workgroup's instance and local tile for stage `st`; false for padding workgroups.
__device__ __forceinline__ bool batch_item(const BatchDev& bt, int st, int& inst, int& tile)
{
    const int* base = bt.base + st * (bt.count + 1);
    const int item = xcd_item(blockIdx.x, base[bt.count]);
    if (item < 0) return false;
    inst = batch_find(base, bt.count, item);
    tile = item - base[inst];
    return true;
}

}  // namespace pat
