// ring_fwd.hip -- forward ring kernels and their launches (ring.hpp).
#include "ring.hpp"

namespace pat {

__device__ __forceinline__ void ring_fwd_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RT,
                                              float2* sm)
{
    const float2* __restrict__ Fp = (const float2*)(wb + L.polar);
    float* hT = (float*)(wb + L.hdet);  // [nlam][D]
    const int D = d.D, S = d.syn_len;
    const int tid = threadIdx.x, bd = blockDim.x;
    const RingLds R = ring_lds(sm, d);
    const int n0 = tile * RT;
    const int nr = min(RT, d.nlam - n0);
    // synthesis: fold with even P -> transform of P/2 + twiddles of P (twA); else transform of S
    const TwLds twA = d.syn_dense ? TwLds{R.twA, R.twA, 0} : tw_lds_build(R.twA, d.ffts[d.fft_syn], d.tw);
    const FftDev& fS = d.ffts[d.fft_synh];
    const float2* __restrict__ tbS = d.tw + fS.tb;
    for (int r = 0; r < nr; ++r) {
        const int n = n0 + r;
        const int off = d.ring_off[n], P = d.ring_off[n + 1] - off;
        const int Kn = d.ring_K[n];
        const float2* __restrict__ cf = d.coef + d.ring_joff[n];
        float* hn = hT + (size_t)n * D;
        const FftDev& fR = d.ffts[d.ring_fft[n]];
        const float2* __restrict__ tbR = d.tw + fR.tb;
        const FftDev& fN = d.ffts[d.ring_twn[n]];
        // the ring's inputs, all loads in flight together: twiddles w_{2P}^k (twN)
        // and the polar values, packed as follows:
        // q(m) = Re F + Im F (m < P), Re F - Im F (m >= P) is real; z(t) = q(2t) + i q(2t+1)
        const TwFetch twf = tw_lds_fetch(fN, d.tw);
        fill_batched<kRingFillUnroll>(
            P,
            [&](int t) {
                float qv[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int m = 2 * t + u;
                    const bool lo = m < P;
                    const float2 F = Fp[off + (lo ? m : m - P)];
                    qv[u] = lo ? F.x + F.y : F.x - F.y;
                }
                return make_float2(qv[0], qv[1]);
            },
            [&](int t, float2 v) { R.sa[t] = v; });
        const TwLds twN = tw_lds_store(R.twN, fN, d.tw, twf);
        __syncthreads();
        fft_lds<false, kRingFftMaxButterflies>(R.sa, P, 1, fR, tbR);
        if (d.syn_dense) {
            // explicit detector angles: the mode coefficients a_k go to the workspace;
            // the dense product with the cos/sin table synthesises the detectors
            float2* am = (float2*)(wb + L.modes) + (size_t)n * d.Kp;
            fill_batched<kRingFillUnroll>(
                Kn + 1, [&](int k) { return cmul(cf[k], real_unpack(R.sa, P, k, twN(k))); },
                [&](int k, float2 v) { am[k] = v; });
            __syncthreads();
            continue;
        }
        // y = the a_k = coef_k Q_k (Q: the real length-2P transform of q) folded
        // mod Pf (fold) or zero-padded to S (chirp-z), summed in order of k: pass
        // 0 writes k < Pf, each further pass adds the next Pf modes
        const int Pf = d.fold_P ? d.fold_P : S;
        for (int q = tid; q < Pf; q += bd)
            if (q > Kn) R.sy[q] = make_float2(0.f, 0.f);
        for (int base = 0; base <= Kn; base += Pf) {
            if (base) __syncthreads();
            fill_batched<kRingFillUnroll>(
                min(Kn + 1 - base, Pf),
                [&](int t) {
                    const int k = base + t;
                    const float2 a = cmul(cf[k], real_unpack(R.sa, P, k, twN(k)));
                    return base ? cadd(R.sy[t], a) : a;
                },
                [&](int t, float2 v) { R.sy[t] = v; });
        }
        __syncthreads();
        if (d.fold_P) {
            if (d.syn_half) {
                // Re(IFFT_P(y)) as a half-length inverse FFT of the Hermitian part
                const int H2 = Pf / 2;
                fill_batched<kRingFillUnroll>(
                    H2,
                    [&](int sidx) {
                        const int s1 = sidx, s2 = sidx + H2;
                        const float2 y1 = R.sy[s1], y1c = cconj(R.sy[s1 == 0 ? 0 : Pf - s1]);
                        const float2 y2 = R.sy[s2], y2c = cconj(R.sy[Pf - s2]);
                        const float2 h1 = cscale(cadd(y1, y1c), 0.5f), h2 = cscale(cadd(y2, y2c), 0.5f);
                        const float2 E = cadd(h1, h2);
                        const float2 O = cmulc(csub(h1, h2), twA(sidx));  // times e^{+2 pi i s / P}
                        return make_float2(E.x - O.y, E.y + O.x);         // E + i O
                    },
                    [&](int sidx, float2 v) { R.sc[sidx] = v; });
                __syncthreads();
                fft_lds<true, kRingFftMaxButterflies>(R.sc, H2, 1, fS, tbS);
                // detector q is point s q of the P-point grid
                fill_batched<kRingFillUnroll>(
                    D,
                    [&](int q) {
                        const int j = q * d.fold_s;
                        const float2 z = R.sc[j >> 1];
                        return (j & 1) ? z.y : z.x;
                    },
                    [&](int q, float v) { hn[q] = v; });
            } else {
                fft_lds<true, kRingFftMaxButterflies>(R.sy, Pf, 1, fS, tbS);
                fill_batched<kRingFillUnroll>(
                    D, [&](int q) { return R.sy[q * d.fold_s].x; }, [&](int q, float v) { hn[q] = v; });
            }
        } else {
            fft_lds<false, kRingFftMaxButterflies>(R.sy, S, 1, fS, tbS);
            for (int q = tid; q < S; q += bd) R.sy[q] = cmul(R.sy[q], d.czt_vhat[q]);
            __syncthreads();
            fft_lds<true, kRingFftMaxButterflies>(R.sy, S, 1, fS, tbS);
            for (int q = tid; q < D; q += bd) {
                const float2 v = R.sy[q], w = d.czt_post[q];
                hn[q] = w.x * v.x - w.y * v.y;
            }
        }
        __syncthreads();
    }
}

// E + i O of the real-output half-length synthesis at index s (0 <= s <= P/2)
// from y_s, y_{P-s}, y_{s+P/2}, y_{P/2-s} (y_q = a_q, q <= K_n; 0 above)
__device__ __forceinline__ float2 syn_prologue(float2 y1, float2 y1m, float2 y2, float2 y2m, float2 w)
{
    const float2 h1 = cscale(cadd(y1, cconj(y1m)), 0.5f), h2 = cscale(cadd(y2, cconj(y2m)), 0.5f);
    const float2 E = cadd(h1, h2);
    const float2 O = cmulc(csub(h1, h2), w);  // times e^{+2 pi i s / P}
    return make_float2(E.x - O.y, E.y + O.x);
}

// The modes a_k of a ring of Pn values, in buf.
template <int Pn, int T>
__device__ __forceinline__ void ring_fwd_spec_head(const float2* __restrict__ Fp, const RingSpecArgs& a, float2* buf)
{
    const int lane = threadIdx.x;
    const bool act = lane < T;
    // the ring's half-plane values packed as the real sequence q(m) = Re F + Im F
    // (m < Pn), Re F - Im F (m >= Pn), z(t) = q(2t) + i q(2t + 1)
    if (act) {
        constexpr int RND = (Pn + T - 1) / T;
        float2 v[RND];
#pragma unroll
        for (int i = 0; i < RND; ++i) {
            const int t = min(lane + i * T, Pn - 1);
            const int m0 = 2 * t, m1 = 2 * t + 1;
            const float2 F0 = Fp[a.off + (m0 < Pn ? m0 : m0 - Pn)];
            const float2 F1 = Fp[a.off + (m1 < Pn ? m1 : m1 - Pn)];
            v[i] = make_float2(m0 < Pn ? F0.x + F0.y : F0.x - F0.y, m1 < Pn ? F1.x + F1.y : F1.x - F1.y);
        }
#pragma unroll
        for (int i = 0; i < RND; ++i) {
            const int t = lane + i * T;
            if (Pn % T == 0 || t < Pn) buf[t] = v[i];
        }
    }
    __syncthreads();
    cfft<Pn, false, cfft_wg_lanes(Pn, T)>(buf, a.ctwR, lane, lane < cfft_wg_lanes(Pn, T));
    // a_k = coef_k Q_k for k <= K_n (zero above), in place of Z: the pair (k, Pn - k)
    // shares sm = Z_k + conj Z_{Pn-k}, df = Z_k - conj Z_{Pn-k} and t = w_{2Pn}^k df,
    //   Q_k = sm/2 - (i/2) t,  Q_{Pn-k} = conj(sm)/2 - (i/2) conj(t)
    // (w_{2Pn}^{Pn-k} = -conj w_{2Pn}^k)
    // (each lane reads and writes only its own pair's two slots)
    if (act) {
        constexpr int PAIRS = Pn / 2 + 1;  // k = 0 .. Pn/2
#pragma unroll
        for (int i = 0; i < (PAIRS + T - 1) / T; ++i) {
            const int k0 = lane + i * T;
            const int k = min(k0, PAIRS - 1);
            const int kc = k == 0 ? 0 : Pn - k;
            const float2 zk = buf[k];
            const float2 zc = cconj(buf[kc]);
            const float2 sm = cadd(zk, zc), df = csub(zk, zc);
            const float2 t = cmul(a.uw[k], df);
            const float2 Q1 = make_float2(0.5f * (sm.x + t.y), 0.5f * (sm.y - t.x));
            const float2 Q2 = make_float2(0.5f * (sm.x - t.y), 0.5f * (-sm.y - t.x));
            const float2 c1 = a.cf[min(k, a.Kn)], c2 = a.cf[min(kc, a.Kn)];
            const float2 v1 = k <= a.Kn ? cmul(c1, Q1) : make_float2(0.f, 0.f);
            const float2 v2 = kc <= a.Kn ? cmul(c2, Q2) : make_float2(0.f, 0.f);
            if (PAIRS % T == 0 || k0 < PAIRS) {
                buf[k] = v1;
                if (k != 0 && 2 * k != Pn) buf[kc] = v2;
            }
        }
    }
    __syncthreads();
}

// Folds the Pn modes in buf into the synthesis input, in their place (held in
// registers across the barrier): one buffer of max(Npsi_max / 2, P / 2) values per
// ring keeps twice as many rings resident.  SHM: longest half-length synthesis of
// the length group.  Outside the dispatch on the ring's length: with a copy per
// length the translation unit took 18 minutes to compile.
template <int T, int SHM>
__device__ __forceinline__ void ring_fwd_spec_fold(const PlanDev& d, int Pn, float2* buf)
{
    const int lane = threadIdx.x;
    const bool act = lane < T;
    const int Pf = d.fold_P, SH = Pf >> 1;
    // y_q = sum of a_k over k = q mod Pf, k < Pn (a_k = 0 above K_n), in increasing k
    auto mode = [&](int q) {
        float2 y = q < Pn ? buf[q] : make_float2(0.f, 0.f);
#pragma unroll 1
        for (int k = q + Pf; k < Pn; k += Pf) y = cadd(y, buf[k]);
        return y;
    };
    const float2* __restrict__ sw = d.ctw + d.syn_sw;
    const int items = (SH + 1) >> 1;
    constexpr int NI = (SHM / 2 + T - 1) / T;
    float2 oa[NI], ob[NI];  // inputs s and SH - s (s = 0: 0 and SH / 2)
    if (act) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int s = lane + i * T;
            if (s >= items) continue;
            if (s == 0) {
                const float2 y0 = mode(0), yh = mode(SH), yq = mode(SH >> 1), y3 = mode(SH + (SH >> 1));
                oa[i] = syn_prologue(y0, y0, yh, yh, sw[0]);
                ob[i] = syn_prologue(yq, y3, y3, yq, sw[SH >> 1]);
            } else {
                const float2 ya = mode(s), yb = mode(Pf - s), yc = mode(s + SH), yd = mode(SH - s);
                oa[i] = syn_prologue(ya, yb, yc, yd, sw[s]);
                ob[i] = syn_prologue(yd, yc, yb, ya, sw[SH - s]);
            }
        }
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int s = lane + i * T;
            if (s >= items) continue;
            buf[s] = oa[i];
            if (s != 0) buf[SH - s] = ob[i];
            else if ((SH & 1) == 0) buf[SH >> 1] = ob[i];
        }
    }
    __syncthreads();
}

template <int T>
__device__ __forceinline__ void ring_fwd_spec_tail(const PlanDev& d, const float2* buf, float* hn)
{
    const int lane = threadIdx.x;
    if (lane < T) {
        // detector q is point s q of the P-point grid: Re part at even, Im at odd points
        for (int q0 = 0; q0 < d.D; q0 += 4 * T) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = min(q0 + lane + u * T, d.D - 1);
                const int j = q * d.fold_s;
                const float2 z = buf[j >> 1];
                v[u] = (j & 1) ? z.y : z.x;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = q0 + lane + u * T;
                if (q < d.D) hn[q] = v[u];
            }
        }
    }
    __syncthreads();
}

template <int G, int W>
__device__ __forceinline__ void ring_fwd_spec_tile(const PlanDev& d, const WsLayout& L, char* wb, int n, float2* buf)
{
    // one ring per workgroup: a loop over rings would keep every length's
    // synthesis twiddles live across it
    const float2* __restrict__ Fp = (const float2*)(wb + L.polar);
    float* hT = (float*)(wb + L.hdet);  // [nlam][D]
    const RingSpecArgs a = ring_spec_args(d, n);
    const int Pn = d.ring_off[n + 1] - a.off;
    constexpr int T = ring_spec_threads(G, W), SHM = ring_spec_max(G);
    switch (Pn) {
#define PAT_RING_FWD_HEAD(LEN) \
    case LEN: ring_fwd_spec_head<LEN, T>(Fp, a, buf); break;
        PAT_CFFT_LENGTHS_LO(PAT_RING_FWD_HEAD)
        default:
            if constexpr (G >= 1) {
                switch (Pn) {
                    PAT_CFFT_LENGTHS_HI(PAT_RING_FWD_HEAD)
                    default:
                        if constexpr (G >= 2) {
                            switch (Pn) {
                                PAT_CFFT_LENGTHS_HI2(PAT_RING_FWD_HEAD)
                                default: break;
                            }
                        }
                        break;
                }
            }
            break;
#undef PAT_RING_FWD_HEAD
    }
    ring_fwd_spec_fold<T, SHM>(d, Pn, buf);
    cfft_run_wg<true, G, T>(buf, d.fold_P >> 1, d.ctw + d.syn_ctw);
    ring_fwd_spec_tail<T>(d, buf, hT + (size_t)n * d.D);
}

__global__ __launch_bounds__(kRingMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_fwd(PlanDev d, WsLayout L, InstPtrs wsp, int RT, int batch)
{
    extern __shared__ float2 sm[];
    int b, t;
    if (!ring_item<false>(blockIdx.x, (d.nlam + RT - 1) / RT, batch, b, t)) return;
    ring_fwd_tile(d, L, wsp.ws + (size_t)b * wsp.stride, t, RT, sm);
}

__global__ __launch_bounds__(kRingMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_fwd_b(BatchDev bt, char* ws)
{
    extern __shared__ float2 sm[];
    int i, tile;
    if (!batch_item(bt, kStRing, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    if (d.ring_spec && d.ring_spec_grp == 2) ring_fwd_spec_tile<2, 1>(d, I.L, ws + I.ws_off, tile, sm);
    else if (d.ring_spec) ring_fwd_spec_tile<1, 1>(d, I.L, ws + I.ws_off, tile, sm);
    else ring_fwd_tile(d, I.L, ws + I.ws_off, tile, I.ring_rt, sm);
}

// Ring kernels of plans with compile-time transforms: one ring per workgroup
// of ring_spec_threads(G, W) threads, largest rings first.  Length group G
// (cfft.hpp): 0 up to kCfftSplit, 1 up to 1024 (one wave), 2 up to 2048 (two
// waves); W waves per ring in the one-wave groups (the same arithmetic on
// more lanes: small batches, where a ring's chain of phases is the critical
// path).
template <int G, int W>
__global__ __launch_bounds__(ring_spec_threads(G, W)) void k_ring_fwd_spec(PlanDev d, WsLayout L, InstPtrs wsp, int batch)
{
    extern __shared__ float2 sm[];
    int b, n;
    if (!ring_item<false>(blockIdx.x, d.nlam, batch, b, n)) return;
    ring_fwd_spec_tile<G, W>(d, L, wsp.ws + (size_t)b * wsp.stride, n, sm);
}

// The ring kernel of a call on `batch` instances of one plan.
void ring_fwd_launch(const pat_plan* p, const InstPtrs& wsp, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int rt = d.ring_spec ? 1 : p->cfg.ring_rt;  // compile-time ring kernels: one ring per workgroup
    const dim3 grid(xcd_grid((d.nlam + rt - 1) / rt * batch)), blk(p->thr_ring);
    if (d.ring_spec && d.ring_spec_grp == 2)
        hipLaunchKernelGGL((k_ring_fwd_spec<2, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec && d.ring_spec_grp == 1)
        hipLaunchKernelGGL((k_ring_fwd_spec<1, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec && p->thr_ring == ring_spec_threads(0, 2))
        hipLaunchKernelGGL((k_ring_fwd_spec<0, 2>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec)
        hipLaunchKernelGGL((k_ring_fwd_spec<0, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else hipLaunchKernelGGL(k_ring_fwd, grid, blk, p->lds_ring, st, d, p->ws, wsp, p->cfg.ring_rt, batch);
}

// Heterogeneous batches whose instances all have compile-time transforms: one
// ring per workgroup of the largest instance's length group, without the
// run-time form's registers and workgroup size.
template <int G>
__global__ __launch_bounds__(ring_spec_threads(G)) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_fwd_spec_b(BatchDev bt, char* ws)
{
    extern __shared__ float2 sm[];
    int i, tile;
    if (!batch_item(bt, kStRing, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    ring_fwd_spec_tile<G, 1>(d, I.L, ws + I.ws_off, d.nlam - 1 - tile, sm);  // largest rings first
}

// The ring kernel of a heterogeneous batch of `items` work items.
void ring_fwd_b_launch(const BatchDev& bt, char* ws, int items, unsigned threads, size_t lds, int spec_grp, hipStream_t st)
{
    const dim3 grid(xcd_grid(items));
    if (spec_grp == 0) hipLaunchKernelGGL(k_ring_fwd_spec_b<0>, grid, dim3(ring_spec_threads(0)), lds, st, bt, ws);
    else if (spec_grp == 1) hipLaunchKernelGGL(k_ring_fwd_spec_b<1>, grid, dim3(ring_spec_threads(1)), lds, st, bt, ws);
    else if (spec_grp == 2) hipLaunchKernelGGL(k_ring_fwd_spec_b<2>, grid, dim3(ring_spec_threads(2)), lds, st, bt, ws);
    else hipLaunchKernelGGL(k_ring_fwd_b, grid, dim3(threads), lds, st, bt, ws);
}

}  // namespace pat
