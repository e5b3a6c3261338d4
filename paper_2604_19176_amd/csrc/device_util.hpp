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

// The ES kernel phi(t) = exp(beta (sqrt(1 - (t/4)^2) - 1)), beta = kEsBeta, at tap
// distances t = 3.5 - d + g, |g| <= 1/2, for d = 0 .. 3: polynomials of degree 8 in
// g, the Chebyshev least-squares fit in FP64 on [-1/2, 1/2] (coefficients of g^0 ..
// g^8), within 7.1e-9 of phi.  With the coefficients rounded to float the polynomials
// are within 3.5e-9, 3.4e-9, 1.3e-8 and 3.8e-8 (d = 0 .. 3) of it; these are parts of
// the largest tap, 1, not of the outermost one, which runs from 1.0e-8 to 2.0e-3.
static_assert(kEsBeta == 2.30 * 8, "kEsPoly is fitted to this beta");
constexpr float kEsPoly[4][9] = {
    {7.54424545e-05f, -0.000627239817f, 0.00222511124f, -0.00440370012f, 0.00529891253f, -0.00388452341f, 0.00149517192f, 3.90759233e-05f, -0.000277026353f},
    {0.0176590905f, -0.0650374591f, 0.0984192193f, -0.0738898143f, 0.0213647485f, 0.00744818663f, -0.00755627872f, 0.0010998128f, 0.000726180093f},
    {0.261128277f, -0.485905409f, 0.263611913f, 0.0497403592f, -0.095805265f, 0.0164990574f, 0.0136794029f, -0.00462838635f, -0.000992656103f},
    {0.865614235f, -0.501662731f, -0.364257514f, 0.251083404f, 0.0691484809f, -0.0597133376f, -0.00761750108f, 0.00851049926f, 0.00049085723f},
};

// The 8 taps of the ES kernel for a point at fraction frac in [0, 1] of its cell:
// w[d] = phi(frac + 3 - d).  Taps d and 7 - d are P_d(g) and P_d(-g), g = frac - 1/2,
// so the even and odd parts are summed once for both: 40 multiply-adds for 8
// taps.  (A square root and an exponential per tap took 44 issue cycles each
// against 20 here, with ten times the error: 1.5e-6 of the largest tap against
// 1.0e-7.)  The same routine serves the interpolation and the spread, which
// keeps them exact transposes.
__device__ __forceinline__ void es_weights8(float frac, float (&w)[8])
{
    const float g = frac - 0.5f, g2 = g * g;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const float (&c)[9] = kEsPoly[d];
        const float even = fmaf(fmaf(fmaf(fmaf(c[8], g2, c[6]), g2, c[4]), g2, c[2]), g2, c[0]);
        const float odd = fmaf(fmaf(fmaf(c[7], g2, c[5]), g2, c[3]), g2, c[1]);
        w[d] = fmaf(g, odd, even);
        w[7 - d] = fmaf(-g, odd, even);
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
