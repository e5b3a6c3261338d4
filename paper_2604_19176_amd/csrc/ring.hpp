// ring.hpp -- what the forward and the adjoint ring kernels (ring_fwd.hip, ring_adj.hip) share.
#pragma once

#include "cfft.hpp"
#include "device_util.hpp"
#include "fft.hpp"
#include "pat_internal.hpp"

namespace pat {

// ---------------------------------------------------------------------------
// Ring kernels.  One workgroup handles RT consecutive radial frequencies
// (rings) of one instance, one ring after another:
//   forward: the ring's interpolated half-plane values (k_gather), completion
//            F(l + Npsi/2) = conj F(l), angular FFT,
//            a_k = c_k e^{i k theta_0} i^k J_k(lam_n R) W_n F_k / Npsi (k <= K_n),
//            synthesis over detectors h(d) = Re sum_k a_k e^{i k d dtheta}
//            (one inverse FFT of length P after folding k mod P when
//            dtheta = 2 pi / P, else Bluestein with two FFTs of length L),
//            -> hT[n][d]  (real; the cosine transform over n follows)
//   adjoint: the exact transpose, ending with the Hermitian fold -> H,
//            stored in band order for the spread, which applies the conjugate
//            half-pixel phase as it stages each point from a band-order table
//            (scattered writes here, contiguous reads there: reading
//            H through each band-order point's ring index instead makes every
//            wave-load of the spread touch tens of cache lines per instance,
//            which costs the spread more than the scatter costs here).
// ---------------------------------------------------------------------------

// Unpack one bin of a real length-2H DFT from Z = FFT_H(z), z(t) = q(2t) + i q(2t+1):
//   Q_k = (Z_k + conj Z_{H-k}) / 2 - (i/2) w_{2H}^k (Z_k - conj Z_{H-k}),  0 <= k < H.
__device__ __forceinline__ float2 real_unpack(const float2* Z, int H, int k, float2 wk)
{
    const float2 zk = Z[k];
    const float2 zc = cconj(Z[k == 0 ? 0 : H - k]);
    const float2 sm = cadd(zk, zc), df = csub(zk, zc);
    const float2 t = cmul(wk, df);
    return make_float2(0.5f * (sm.x + t.y), 0.5f * (sm.y - t.x));
}

// Layout of the ring kernels' dynamic LDS (float2 slots, ring_lds_slots):
// sa (ring FFT; the half-length synthesis buffer sc shares it), sy
// (synthesis), and the two-level twiddles of lengths Npsi(n) (twN) and S
// (twA) used outside the transforms.  The transforms read their per-pass
// twiddles, and the mode loops the ring's coefficients, from global memory
// (tables shared by all instances of a plan, cache resident): small LDS per
// ring keeps many rings resident per CU, and nothing is held in registers
// across a transform.
struct RingLds {
    float2 *sa, *sc, *sy, *twN, *twA;
};

__device__ __forceinline__ RingLds ring_lds(float2* sm, const PlanDev& d)
{
    RingLds r;
    const int Pmax = d.npsi_max / 2;
    const int S = d.syn_len;
    const int B1 = max(Pmax, d.syn_half ? S / 2 : 0);
    const int B2 = max(S, Pmax);
    r.sa = sm;
    r.sc = sm;
    r.sy = sm + B1;
    r.twN = r.sy + B2;
    r.twA = r.twN + ring_tw_slots(d.npsi_max);
    return r;
}

// ---------------------------------------------------------------------------
// Ring kernels with compile-time transforms (plans with ring_spec: a uniform
// arc whose pitch is 2 pi s / P with P even, modes folded mod P, every length
// with a cfft.hpp plan).  The same operator as ring_fwd_tile /
// ring_adj_tile; lanes 0..63 of wave 0 do all the work in one LDS buffer of
// max(Npsi_max, P) / 2 complex values:
//   forward: head<Pn> (packed ring -> ring transform -> modes times their
//            coefficients, folded, straight into the half-length synthesis
//            input), synthesis transform (length P/2), tail (detectors);
//   adjoint: head (detectors -> synthesis transform), tail<Pn> (mode
//            coefficients straight into the half-length input of the ring's
//            inverse transform, transform, band-order stores).
// Each mode is evaluated once: the synthesis input at s and P/2 - s (forward),
// or the ring input at u and Pn - u (adjoint), need the same modes, so one
// lane computes both.  Twiddles come from the plan's FP64-computed tables.
// ---------------------------------------------------------------------------
struct RingSpecArgs {
    int off, Kn;
    const float2* __restrict__ cf;   // ring coefficients coef_k, k <= K_n
    const float2* __restrict__ ctwR; // ring transform table
    const float2* __restrict__ uw;   // w_{2 Pn}^k, k = 0..Pn
};

__device__ __forceinline__ RingSpecArgs ring_spec_args(const PlanDev& d, int n)
{
    RingSpecArgs a;
    a.off = d.ring_off[n];
    a.Kn = d.ring_K[n];
    a.cf = d.coef + d.ring_joff[n];
    a.ctwR = d.ctw + d.ring_ctw[n];
    a.uw = d.ctw + d.ring_uw[n];
    return a;
}

// Ring kernels: at most kRingMaxThreads threads (one wave for most rings).  Both
// are held to 128 VGPRs (four waves per SIMD), where the per-instance kernels
// do not spill: they are latency bound, so resident waves count more than the
// extra registers an unconstrained schedule would take.
// Ring tile order: a ring's work grows with n, so the largest rings go first
// and a launch ends on small ones.  The XCD ranges stay instance-major (an
// instance's data in one L2).  RING_MAJOR (used when every XCD owns whole
// instances, batch a multiple of 8): an XCD's tiles run ring-major across its
// instances (largest ring of each instance, then the next); else instance by
// instance.  Measured at 256^2, batch 64: the forward ring kernel is fastest
// instance by instance (a ring's polar values follow the previous ring's), the
// adjoint ring-major.
template <bool RING_MAJOR>
__device__ __forceinline__ bool ring_item(int w, int ntile, int batch, int& b, int& t)
{
    const int item = xcd_item(w, ntile * batch);
    if (item < 0) return false;
    if (RING_MAJOR && batch % kXcds == 0) {
        const int per = batch / kXcds;  // instances per XCD
        const int x = item / (per * ntile), q = item - x * per * ntile;
        const int tr = q / per;
        b = x * per + (q - tr * per);
        t = ntile - 1 - tr;
    } else {
        b = item / ntile;
        t = ntile - 1 - (item - b * ntile);
    }
    return true;
}

}  // namespace pat
