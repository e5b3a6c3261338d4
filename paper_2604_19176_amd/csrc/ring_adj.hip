// ring_adj.hip -- adjoint ring kernels and their launches (ring.hpp).
#include "ring.hpp"

namespace pat {

// Value at point j of the P-point angular grid of the detector values placed
// at points s q (q < D), zero elsewhere.
__device__ __forceinline__ float grid_det(const float* hn, int j, int s, float rcp_s, int D)
{
    int q = j, rem = 0;
    if (s != 1) fdivmod(j, s, rcp_s, q, rem);
    const float v = hn[min(q, D - 1)];  // unconditional load (batched by the caller), value selected
    return (rem == 0 && q < D) ? v : 0.f;
}

__device__ __forceinline__ void ring_adj_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RT,
                                              float2* sm)
{
    const float* hT = (const float*)(wb + L.hdet);  // [nlam][D]
    float2* Hb = (float2*)(wb + L.polar);
    const int D = d.D, S = d.syn_len;
    const int tid = threadIdx.x, bd = blockDim.x;
    const RingLds R = ring_lds(sm, d);
    const int n0 = tile * RT;
    const int nr = min(RT, d.nlam - n0);
    const bool half = d.fold_P && d.syn_half;
    const float rcp_s = 1.0f / (float)max(d.fold_s, 1);
    const float rcp_P = __builtin_amdgcn_rcpf((float)max(d.fold_P, 1));  // fdivmod makes k mod P exact
    // the mode values Q~ go to qb, the Hermitian-part input of the ring's inverse FFT to eb
    float2* const qb = half ? R.sy : R.sa;
    float2* const eb = half ? R.sa : R.sy;
    const TwLds twA = d.syn_dense ? TwLds{R.twA, R.twA, 0} : tw_lds_build(R.twA, d.ffts[d.fft_syn], d.tw);
    const FftDev& fS = d.ffts[d.fft_synh];
    const float2* __restrict__ tbS = d.tw + fS.tb;
    for (int r = 0; r < nr; ++r) {
        const int n = n0 + r;
        const int off = d.ring_off[n], P = d.ring_off[n + 1] - off;
        const int Kn = d.ring_K[n];
        const float2* __restrict__ cf = d.coef + d.ring_joff[n];
        const float* hn = hT + (size_t)n * D;
        // explicit detector angles: y~_k from the dense product (workspace), no transform
        const float2* __restrict__ am = (const float2*)(wb + L.modes) + (size_t)n * d.Kp;
        const FftDev& fR = d.ffts[d.ring_fft[n]];
        const float2* __restrict__ tbR = d.tw + fR.tb;
        const FftDev& fN = d.ffts[d.ring_twn[n]];
        const TwFetch twf = tw_lds_fetch(fN, d.tw);
        // the ring's inputs, all loads in flight together: twiddles (twN) and the
        // detector values zero-padded to the synthesis length; then y~ = their
        // FFT.  Explicit angles: Q~ directly.
        if (d.syn_dense) {
            fill_batched<kRingFillUnroll>(
                Kn + 1, [&](int k) { return cmulc(am[k], cf[k]); }, [&](int k, float2 v) { qb[k] = v; });
            tw_lds_store(R.twN, fN, d.tw, twf);
        } else if (half) {
            const int H2 = d.fold_P / 2;
            fill_batched<kRingFillUnroll>(
                H2,
                [&](int t) {
                    return make_float2(grid_det(hn, 2 * t, d.fold_s, rcp_s, D), grid_det(hn, 2 * t + 1, d.fold_s, rcp_s, D));
                },
                [&](int t, float2 v) { R.sc[t] = v; });
            tw_lds_store(R.twN, fN, d.tw, twf);
            __syncthreads();
            fft_lds<false, kRingFftMaxButterflies>(R.sc, H2, 1, fS, tbS);
        } else if (d.fold_P) {
            fill_batched<kRingFillUnroll>(
                S, [&](int t) { return make_float2(grid_det(hn, t, d.fold_s, rcp_s, D), 0.f); },
                [&](int t, float2 v) { R.sy[t] = v; });
            tw_lds_store(R.twN, fN, d.tw, twf);
            __syncthreads();
            fft_lds<false, kRingFftMaxButterflies>(R.sy, S, 1, fS, tbS);
        } else {
            fill_batched<kRingFillUnroll>(
                S,
                [&](int q) {
                    const int qc = min(q, D - 1);
                    const float2 v = cmulc(make_float2(hn[qc], 0.f), d.czt_post[qc]);
                    return q < D ? v : make_float2(0.f, 0.f);
                },
                [&](int q, float2 v) { R.sy[q] = v; });
            tw_lds_store(R.twN, fN, d.tw, twf);
            __syncthreads();
            fft_lds<false, kRingFftMaxButterflies>(R.sy, S, 1, fS, tbS);
            for (int q = tid; q < S; q += bd) R.sy[q] = cmulc(R.sy[q], d.czt_vhat[q]);
            __syncthreads();
            fft_lds<true, kRingFftMaxButterflies>(R.sy, S, 1, fS, tbS);
        }
        const TwLds twN{R.twN, R.twN + 64, 0};
        // y~ at synthesis index sidx (0 <= sidx < S)
        auto ytil = [&](int sidx) {
            if (!half) return R.sy[sidx];
            const int Pf = d.fold_P, H2 = Pf / 2;
            if (sidx == H2) return make_float2(R.sc[0].x - R.sc[0].y, 0.f);
            const bool hi = sidx > H2;
            const int s0 = hi ? Pf - sidx : sidx;
            const float2 v = real_unpack(R.sc, H2, s0, twA(s0));
            return hi ? cconj(v) : v;
        };
        // Q~_k = conj(coef_k) y~_{k mod Pf}
        if (!d.syn_dense) {
            fill_batched<kRingFillUnroll>(
                Kn + 1,
                [&](int k) {
                    int sidx = k, fq;
                    if (d.fold_P) fdivmod(k, d.fold_P, rcp_P, fq, sidx);
                    return cmulc(ytil(sidx), cf[k]);
                },
                [&](int k, float2 v) { qb[k] = v; });
        }
        __syncthreads();
        // Re(IFFT_{2P}(Q~)) as a half-length inverse FFT: E + i O from the
        // Hermitian part of Q~ (which vanishes above K_n < P).
        // Q~_h[s] = Q~[s]/2 (0 < s <= K), Re Q~[0] (s = 0); Q~_h[s + P] = conj Q~[P - s]/2 (P - s <= K).
        fill_batched<kRingFillUnroll>(
            P,
            [&](int sidx) {
                // reads clamped into qb[0 .. Kn], values outside the mode range dropped
                const float2 q1 = qb[min(sidx, Kn)], q2 = qb[min(P - sidx, Kn)];
                const float2 zero = make_float2(0.f, 0.f);
                const float2 a = sidx == 0 ? make_float2(q1.x, 0.f) : (sidx <= Kn ? cscale(q1, 0.5f) : zero);
                const float2 c = (sidx != 0 && P - sidx <= Kn) ? cscale(cconj(q2), 0.5f) : zero;
                const float2 E = cadd(a, c);
                const float2 O = cmulc(csub(a, c), twN(sidx));
                return make_float2(E.x - O.y, E.y + O.x);
            },
            [&](int sidx, float2 v) { eb[sidx] = v; });
        __syncthreads();
        fft_lds<true, kRingFftMaxButterflies>(eb, P, 1, fR, tbR);
        // q~(m): m = 2t -> Re z_t, m = 2t + 1 -> Im z_t;  F~_h(l) = (q~(l) + q~(l+P)) + i (q~(l) - q~(l+P))
        fill_batched<kRingFillUnroll>(
            P,
            [&](int l) {
                const float2 z1 = eb[l >> 1];
                const float a = (l & 1) ? z1.y : z1.x;
                const int m = l + P;
                const float2 z2 = eb[m >> 1];
                const float c = (m & 1) ? z2.y : z2.x;
                const float2 Fh = make_float2(a + c, a - c);
                return IdxVal{d.band_of[off + l], Fh};
            },
            [&](int, IdxVal iv) { Hb[iv.i] = iv.v; });
        __syncthreads();
    }
}

template <int T>
__device__ __forceinline__ void ring_adj_spec_head(const PlanDev& d, const float* __restrict__ hn, float2* buf)
{
    const int lane = threadIdx.x;
    const int SH = d.fold_P >> 1, fs = d.fold_s, D = d.D;
    // the detector values at points s q of the P-point grid (zero between), packed
    // as z(t) = h(2t) + i h(2t + 1)
    if (lane < T) {
        const float rcp_s = __builtin_amdgcn_rcpf((float)fs);
        for (int t0 = 0; t0 < SH; t0 += 2 * T) {
            float2 v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = min(t0 + lane + u * T, SH - 1);
                float h[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int j = 2 * t + e;
                    int q = j, rem = 0;
                    if (fs != 1) fdivmod(j, fs, rcp_s, q, rem);
                    const float x = hn[min(q, D - 1)];
                    h[e] = (rem == 0 && q < D) ? x : 0.f;
                }
                v[u] = make_float2(h[0], h[1]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int t = t0 + lane + u * T;
                if (t < SH) buf[t] = v[u];
            }
        }
    }
    __syncthreads();
}

// The ring transform's input takes the place of the synthesis values in buf
// (held in registers across the barrier), as in the forward kernel.
template <int Pn, int T>
__device__ __forceinline__ void ring_adj_spec_tail(const PlanDev& d, const RingSpecArgs& a, float2* buf, float2* Hb)
{
    const int lane = threadIdx.x;
    const bool act = lane < T;
    const int Pf = d.fold_P, SH = Pf >> 1;
    const float2* __restrict__ sw = d.ctw + d.syn_sw;
    // the ring points' band-order slots, for the stores at the end: loaded now,
    // in flight during the transforms
    constexpr int RO = (Pn + T - 1) / T;
    int slot[RO];
#pragma unroll
    for (int i = 0; i < RO; ++i) slot[i] = d.band_of[a.off + min(lane + i * T, Pn - 1)];
    // y~ at synthesis index q (0 <= q <= P/2) from the half-length transform Z,
    // in place of Z (slot P/2 after it): the pair (s, SH - s) shares
    // sm = Z_s + conj Z_{SH-s}, df = Z_s - conj Z_{SH-s}, t = w_P^s df,
    //   y~_s = sm/2 - (i/2) t,  y~_{SH-s} = conj(sm)/2 - (i/2) conj(t),
    // and y~_{SH} = Re Z_0 - Im Z_0; above P/2, y~_{P-q} = conj y~_q
    // (each lane reads and writes only its own pair's slots)
    float2* ys = buf;
    if (act) {
        const int PAIRS = SH / 2 + 1;  // s = 0 .. SH/2
        for (int s = lane; s < PAIRS; s += T) {
            const int sc = s == 0 ? 0 : SH - s;
            const float2 zk = ys[s];
            const float2 zc = cconj(ys[sc]);
            const float2 sm = cadd(zk, zc), df = csub(zk, zc);
            const float2 t = cmul(sw[s], df);
            ys[s] = make_float2(0.5f * (sm.x + t.y), 0.5f * (sm.y - t.x));
            if (s == 0) ys[SH] = make_float2(zc.x + zc.y, 0.f);
            else if (2 * s != SH) ys[sc] = make_float2(0.5f * (sm.x - t.y), 0.5f * (-sm.y - t.x));
        }
    }
    __syncthreads();
    // Q~_k = conj(coef_k) y~_{k mod P} for k <= K_n (0 above)
    auto qmode = [&](int k) {
        const int kc = min(k, a.Kn);
        int kf = kc;  // synthesis index k mod Pf
        while (kf >= Pf) kf -= Pf;
        const bool hi = kf > SH;
        const float2 y0 = ys[hi ? Pf - kf : kf];
        const float2 v = cmulc(hi ? cconj(y0) : y0, a.cf[kc]);
        return k <= a.Kn ? v : make_float2(0.f, 0.f);
    };
    // input of the ring's half-length inverse transform at u: E + i O from the
    // Hermitian part of Q~ (q1 = Q~_u, q2 = Q~_{Pn-u})
    auto herm = [&](int u, float2 q1, float2 q2) {
        const float2 zero = make_float2(0.f, 0.f);
        const float2 av = u == 0 ? make_float2(q1.x, 0.f) : cscale(q1, 0.5f);
        const float2 cv = u == 0 ? zero : cscale(cconj(q2), 0.5f);
        const float2 E = cadd(av, cv);
        const float2 O = cmulc(csub(av, cv), a.uw[u]);
        return make_float2(E.x - O.y, E.y + O.x);
    };
    // item u < (Pn + 1)/2 writes slots u and Pn - u; item 0 writes slot 0 and,
    // for even Pn, slot Pn/2 (one path for every lane: no branch on u, the
    // loads of all rounds can be issued together)
    constexpr int items = (Pn + 1) / 2, NI = (items + T - 1) / T;
    float2 ha[NI], hb[NI];
    if (act) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int u = min(lane + i * T, items - 1);
            const int u2 = u == 0 ? ((Pn & 1) == 0 ? Pn / 2 : 0) : Pn - u;  // the second slot
            const float2 qa = qmode(u), qb = qmode(u2);
            ha[i] = herm(u, qa, qb);
            hb[i] = herm(u2, qb, u == 0 ? qb : qa);
        }
    }
    __syncthreads();
    if (act) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int u = lane + i * T;
            const int u2 = u == 0 ? ((Pn & 1) == 0 ? Pn / 2 : 0) : Pn - u;
            if (items % T == 0 || u < items) {
                buf[u] = ha[i];
                if (u2 != 0) buf[u2] = hb[i];
            }
        }
    }
    __syncthreads();
    cfft<Pn, true, cfft_wg_lanes(Pn, T)>(buf, a.ctwR, lane, lane < cfft_wg_lanes(Pn, T));
    // q~(m): m = 2t -> Re z_t, m = 2t + 1 -> Im z_t;  F~_h(l) = (q~(l) + q~(l+Pn)) + i (q~(l) - q~(l+Pn)),
    // stored in band order (the spread applies the conjugate half-pixel phase)
    if (act) {
#pragma unroll
        for (int i = 0; i < RO; ++i) {
            const int l0 = lane + i * T;
            const int l = min(l0, Pn - 1);
            const float2 z1 = buf[l >> 1];
            const float av = (l & 1) ? z1.y : z1.x;
            const int m = l + Pn;
            const float2 z2 = buf[m >> 1];
            const float cv = (m & 1) ? z2.y : z2.x;
            const float2 Fh = make_float2(av + cv, av - cv);
            if (Pn % T == 0 || l0 < Pn) Hb[slot[i]] = Fh;
        }
    }
    __syncthreads();
}

template <int G, int W>
__device__ __forceinline__ void ring_adj_spec_tile(const PlanDev& d, const WsLayout& L, char* wb, int n, float2* buf)
{
    const float* hT = (const float*)(wb + L.hdet);  // [nlam][D]
    float2* Hb = (float2*)(wb + L.polar);
    constexpr int T = ring_spec_threads(G, W);
    ring_adj_spec_head<T>(d, hT + (size_t)n * d.D, buf);
    cfft_run_wg<false, G, T>(buf, d.fold_P >> 1, d.ctw + d.syn_ctw);
    const RingSpecArgs a = ring_spec_args(d, n);
    const int Pn = d.ring_off[n + 1] - a.off;
    switch (Pn) {
#define PAT_RING_ADJ_TAIL(LEN) \
    case LEN: ring_adj_spec_tail<LEN, T>(d, a, buf, Hb); break;
        PAT_CFFT_LENGTHS_LO(PAT_RING_ADJ_TAIL)
        default:
            if constexpr (G >= 1) {
                switch (Pn) {
                    PAT_CFFT_LENGTHS_HI(PAT_RING_ADJ_TAIL)
                    default:
                        if constexpr (G >= 2) {
                            switch (Pn) {
                                PAT_CFFT_LENGTHS_HI2(PAT_RING_ADJ_TAIL)
                                default: break;
                            }
                        }
                        break;
                }
            }
            break;
#undef PAT_RING_ADJ_TAIL
    }
}

template <int G, int W>
__global__ __launch_bounds__(ring_spec_threads(G, W)) void k_ring_adj_spec(PlanDev d, WsLayout L, InstPtrs wsp, int batch)
{
    extern __shared__ float2 sm[];
    int b, n;
    if (!ring_item<true>(blockIdx.x, d.nlam, batch, b, n)) return;
    ring_adj_spec_tile<G, W>(d, L, wsp.ws + (size_t)b * wsp.stride, n, sm);
}

__global__ __launch_bounds__(kRingMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_adj(PlanDev d, WsLayout L, InstPtrs wsp, int RT, int batch)
{
    extern __shared__ float2 sm[];
    int b, t;
    if (!ring_item<true>(blockIdx.x, (d.nlam + RT - 1) / RT, batch, b, t)) return;
    ring_adj_tile(d, L, wsp.ws + (size_t)b * wsp.stride, t, RT, sm);
}

__global__ __launch_bounds__(kRingMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_adj_b(BatchDev bt, char* ws)
{
    extern __shared__ float2 sm[];
    int i, tile;
    if (!batch_item(bt, kStRing, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    if (d.ring_spec && d.ring_spec_grp == 2) ring_adj_spec_tile<2, 1>(d, I.L, ws + I.ws_off, tile, sm);
    else if (d.ring_spec) ring_adj_spec_tile<1, 1>(d, I.L, ws + I.ws_off, tile, sm);
    else ring_adj_tile(d, I.L, ws + I.ws_off, tile, I.ring_rt, sm);
}

// The ring kernel of a call on `batch` instances of one plan.
void ring_adj_launch(const pat_plan* p, const InstPtrs& wsp, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int rt = d.ring_spec ? 1 : p->cfg.ring_rt;  // compile-time ring kernels: one ring per workgroup
    const dim3 grid(xcd_grid((d.nlam + rt - 1) / rt * batch)), blk(p->thr_ring);
    if (d.ring_spec && d.ring_spec_grp == 2)
        hipLaunchKernelGGL((k_ring_adj_spec<2, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec && d.ring_spec_grp == 1)
        hipLaunchKernelGGL((k_ring_adj_spec<1, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec && p->thr_ring == ring_spec_threads(0, 2))
        hipLaunchKernelGGL((k_ring_adj_spec<0, 2>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else if (d.ring_spec)
        hipLaunchKernelGGL((k_ring_adj_spec<0, 1>), grid, blk, p->lds_ring, st, d, p->ws, wsp, batch);
    else hipLaunchKernelGGL(k_ring_adj, grid, blk, p->lds_ring, st, d, p->ws, wsp, p->cfg.ring_rt, batch);
}

// Heterogeneous batches whose instances all have compile-time transforms: one
// ring per workgroup of the largest instance's length group, without the
// run-time form's registers and workgroup size.
template <int G>
__global__ __launch_bounds__(ring_spec_threads(G)) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_adj_spec_b(BatchDev bt, char* ws)
{
    extern __shared__ float2 sm[];
    int i, tile;
    if (!batch_item(bt, kStRing, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    ring_adj_spec_tile<G, 1>(d, I.L, ws + I.ws_off, d.nlam - 1 - tile, sm);  // largest rings first
}

// The ring kernel of a heterogeneous batch of `items` work items.
void ring_adj_b_launch(const BatchDev& bt, char* ws, int items, unsigned threads, size_t lds, int spec_grp, hipStream_t st)
{
    const dim3 grid(xcd_grid(items));
    if (spec_grp == 0) hipLaunchKernelGGL(k_ring_adj_spec_b<0>, grid, dim3(ring_spec_threads(0)), lds, st, bt, ws);
    else if (spec_grp == 1) hipLaunchKernelGGL(k_ring_adj_spec_b<1>, grid, dim3(ring_spec_threads(1)), lds, st, bt, ws);
    else if (spec_grp == 2) hipLaunchKernelGGL(k_ring_adj_spec_b<2>, grid, dim3(ring_spec_threads(2)), lds, st, bt, ws);
    else hipLaunchKernelGGL(k_ring_adj_b, grid, dim3(threads), lds, st, bt, ws);
}

}  // namespace pat
