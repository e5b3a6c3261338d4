// grid_adj.hip -- adjoint 2D-FFT passes: kernels and their launches.
#include "fft.hpp"
#include "grid.hpp"

namespace pat {

// ---------------------------------------------------------------------------
// adjoint: row pass (inverse FFT along x, crop to the N image columns)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void rowpass_adj_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RPB,
                                                 float2* sm)
{
    const int N = d.N, Ng = d.Ng;
    float2* X1 = (float2*)(wb + L.x1);
    const int r0 = tile * RPB;
    const int nr = min(RPB, d.Hy - r0);
    const float2* tb = fft_twiddles_to_lds(sm + RPB * Ng, d.ffts[d.fft_grid], d.tw);
    for (int rr = 0; rr < nr; ++rr) {
        const GridRow g = grid_row(d, L, wb, r0 + rr);
        float2* dst = sm + (size_t)rr * Ng;
        fill_batched<4>(Ng, [&](int c) { return grid_row_at(g, Ng, c); }, [&](int c, float2 v) { dst[c] = v; });
    }
    __syncthreads();
    fft_lds<true>(sm, Ng, nr, d.ffts[d.fft_grid], tb);
    const float rcpN = 1.0f / (float)N;
    fill_batched<4>(
        nr * N,
        [&](int e) {
            int rr, j;
            fdivmod(e, N, rcpN, rr, j);
            int pos = j - N / 2;
            if (pos < 0) pos += Ng;
            return sm[rr * Ng + pos];
        },
        [&](int e, float2 v) { X1[(size_t)r0 * N + e] = v; });
}

// ---------------------------------------------------------------------------
// adjoint: column pass (Hermitian symmetrisation, inverse FFT along y, real
// parts of two columns packed as one complex transform, crop, deapodise, mask)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void colpass_adj_tile(const PlanDev& d, const WsLayout& L, char* wb, float* __restrict__ fb,
                                                 int tile, int NP, int n_sum, float2* sm, float* gsum_s)
{
    const int N = d.N, Ng = d.Ng, CT = 2 * NP;
    const float2* X1 = (const float2*)(wb + L.x1);
    const float* red = (const float*)(wb + L.red);
    if (threadIdx.x < 64) {
        const float s = wave0_fixed_sum(red, n_sum);
        if (threadIdx.x == 0) *gsum_s = s;
    }
    const int j0 = tile * CT;
    const int top = Ng / 2 + 4;
    const float2* tb = fft_twiddles_to_lds(sm + NP * Ng, d.ffts[d.fft_grid], d.tw);
    // column pair p at residue q: batched loads with rows and columns clamped
    // into the stored range, values outside it selected as zero
    const float rcpNg = 1.0f / (float)Ng;
    fill_batched<4>(
        NP * Ng,
        [&](int e) {
            int p, q;
            fdivmod(e, Ng, rcpNg, p, q);
            const int ja = j0 + 2 * p, jb = ja + 1;
            // stored row of residue q and of -q (or -1 if not stored)
            const int rq = q <= top ? q + 4 : (q >= Ng - 4 ? q - Ng + 4 : -1);
            const int qn = q == 0 ? 0 : Ng - q;
            const int rn = qn <= top ? qn + 4 : (qn >= Ng - 4 ? qn - Ng + 4 : -1);
            const int rqc = max(rq, 0), rnc = max(rn, 0), jac = min(ja, N - 1), jbc = min(jb, N - 1);
            const float2 z0 = make_float2(0.f, 0.f);
            const float2 la = X1[(size_t)rqc * N + jac], lna = X1[(size_t)rnc * N + jac];
            const float2 lb = X1[(size_t)rqc * N + jbc], lnb = X1[(size_t)rnc * N + jbc];
            const float2 ua = (ja < N && rq >= 0) ? la : z0, una = (ja < N && rn >= 0) ? lna : z0;
            const float2 ub = (jb < N && rq >= 0) ? lb : z0, unb = (jb < N && rn >= 0) ? lnb : z0;
            // z = (ua + conj una)/2 + i (ub + conj unb)/2
            const float2 ha = make_float2(0.5f * (ua.x + una.x), 0.5f * (ua.y - una.y));
            const float2 hb = make_float2(0.5f * (ub.x + unb.x), 0.5f * (ub.y - unb.y));
            return make_float2(ha.x - hb.y, ha.y + hb.x);
        },
        [&](int e, float2 v) { sm[e] = v; });
    __syncthreads();
    fft_lds<true>(sm, Ng, NP, d.ffts[d.fft_grid], tb);
    const float kt = d.kappa * d.h2 * *gsum_s;
    const float rcpCT = 1.0f / (float)CT;
    fill_batched<4>(
        N * CT,
        [&](int e) {
            int i, jj;
            fdivmod(e, CT, rcpCT, i, jj);
            const int j = j0 + jj, jc = min(j, N - 1);
            int pos = i - N / 2;
            if (pos < 0) pos += Ng;
            const float2 z = sm[(jj >> 1) * Ng + pos];
            const float c = (jj & 1) ? z.y : z.x;
            const int2 mr = d.mask_rows[i];
            const float di = d.deap[i], dj = d.deap[jc];
            const float v = (j >= mr.x && j < mr.y) ? di * dj * c + kt : 0.f;
            return IdxF{j < N ? i * N + j : -1, v};
        },
        [&](int, IdxF iv) {
            if (iv.i >= 0) fb[iv.i] = iv.v;
        });
}

__global__ __launch_bounds__(1024) void k_rowpass_adj(PlanDev d, WsLayout L, InstPtrs wsp, int RPB)
{
    extern __shared__ float2 sm[];
    rowpass_adj_tile(d, L, wsp.ws + (size_t)blockIdx.y * wsp.stride, blockIdx.x, RPB, sm);
}

__global__ __launch_bounds__(1024) void k_colpass_adj(PlanDev d, WsLayout L, InstPtrs wsp, float* __restrict__ f,
                                                     int NP, int n_sum)
{
    extern __shared__ float2 sm[];
    __shared__ float gsum_s;
    const int b = blockIdx.y;
    colpass_adj_tile(d, L, wsp.ws + (size_t)b * wsp.stride, f + (size_t)b * d.N * d.N, blockIdx.x, NP, n_sum, sm,
                     &gsum_s);
}

// Compile-time grid sides: XCD-contiguous, instance-major tiles, so that an
// instance's X1 and G stay in one XCD's L2 from pass to pass.
template <int NG>
__global__ __launch_bounds__(1024) void k_colpass_adj_spec(PlanDev d, WsLayout L, InstPtrs wsp, float* __restrict__ f,
                                                           int NP, int vec, int ntile, int batch)
{
    extern __shared__ __align__(16) float2 smc[];
    __shared__ float gsum_s;
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    colpass_adj_spec<NG>(d, L, wsp.ws + (size_t)b * wsp.stride, f + (size_t)b * d.N * d.N, item - b * ntile, NP, d.D, vec,
                         smc, &gsum_s);
}

template <int NG>
__global__ __launch_bounds__(1024) void k_rowpass_adj_spec(PlanDev d, WsLayout L, InstPtrs wsp, int RPB, int ntile, int batch)
{
    extern __shared__ __align__(16) float2 smc[];
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    rowpass_adj_spec<NG>(d, L, wsp.ws + (size_t)b * wsp.stride, item - b * ntile, RPB, smc);
}

// Heterogeneous batches.  HI: lengths above 1024 too (kept apart for their registers).
template <bool HI>
__global__ __launch_bounds__(1024) void k_colpass_adj_b(BatchDev bt, char* ws, float* const* __restrict__ fout)
{
    extern __shared__ __align__(16) float2 smc[];
    __shared__ float gsum_s;
    int i, tile;
    if (!batch_item(bt, kStCol, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    float* f = fout[i];
    char* wb = ws + I.ws_off;
    if (!d.grid_spec) {
        colpass_adj_tile(d, I.L, wb, f, tile, I.col_np, d.D, smc, &gsum_s);
        return;
    }
    const bool vec = (d.N & 1) == 0 && ((uintptr_t)f & 7) == 0;
    switch (d.Ng) {
#define PAT_CASE(NG) case NG: colpass_adj_spec<NG>(d, I.L, wb, f, tile, I.col_np, d.D, vec, smc, &gsum_s); break;
        PAT_GRID_LENGTHS_LO(PAT_CASE)
        default:
            if constexpr (HI) {
                switch (d.Ng) {
                    PAT_GRID_LENGTHS_HI(PAT_CASE)
                    default: break;
                }
            }
            break;
#undef PAT_CASE
    }
}

template <bool HI>
__global__ __launch_bounds__(1024) void k_rowpass_adj_b(BatchDev bt, char* ws)
{
    extern __shared__ __align__(16) float2 smc[];
    int i, tile;
    if (!batch_item(bt, kStRow, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    char* wb = ws + I.ws_off;
    if (!d.grid_spec) {
        rowpass_adj_tile(d, I.L, wb, tile, I.row_rpb, smc);
        return;
    }
    switch (d.Ng) {
#define PAT_CASE(NG) case NG: rowpass_adj_spec<NG>(d, I.L, wb, tile, I.row_rpb, smc); break;
        PAT_GRID_LENGTHS_LO(PAT_CASE)
        default:
            if constexpr (HI) {
                switch (d.Ng) {
                    PAT_GRID_LENGTHS_HI(PAT_CASE)
                    default: break;
                }
            }
            break;
#undef PAT_CASE
    }
}

void colpass_adj_launch(const pat_plan* p, const InstPtrs& wsp, float* f, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int np = p->np_col, nt = p->n_col_tiles;
    if (!d.grid_spec) {
        hipLaunchKernelGGL(k_colpass_adj, dim3(nt, batch), dim3(p->thr_col), p->lds_col, st, d, p->ws, wsp, f, np, d.D);
        return;
    }
    const int vec = (d.N & 1) == 0 && ((uintptr_t)f & 7) == 0;
    const dim3 grid(xcd_grid(nt * batch)), blk(p->thr_col);
    switch (d.Ng) {
#define PAT_CASE(NG) \
    case NG: hipLaunchKernelGGL(k_colpass_adj_spec<NG>, grid, blk, p->lds_col, st, d, p->ws, wsp, f, np, vec, nt, batch); break;
        PAT_GRID_LENGTHS(PAT_CASE)
#undef PAT_CASE
        default: break;
    }
}

void rowpass_adj_launch(const pat_plan* p, const InstPtrs& wsp, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int rpb = p->np_row, nt = (d.Hy + rpb - 1) / rpb;
    if (!d.grid_spec) {
        hipLaunchKernelGGL(k_rowpass_adj, dim3(nt, batch), dim3(p->thr_row), p->lds_row, st, d, p->ws, wsp, rpb);
        return;
    }
    const dim3 grid(xcd_grid(nt * batch)), blk(p->thr_row);
    switch (d.Ng) {
#define PAT_CASE(NG) \
    case NG: hipLaunchKernelGGL(k_rowpass_adj_spec<NG>, grid, blk, p->lds_row, st, d, p->ws, wsp, rpb, nt, batch); break;
        PAT_GRID_LENGTHS(PAT_CASE)
#undef PAT_CASE
        default: break;
    }
}

void colpass_adj_b_launch(const BatchDev& bt, char* ws, float* const* f, int items, unsigned thr, size_t lds, bool hi,
                          hipStream_t st)
{
    if (hi) hipLaunchKernelGGL(k_colpass_adj_b<true>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws, f);
    else hipLaunchKernelGGL(k_colpass_adj_b<false>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws, f);
}

void rowpass_adj_b_launch(const BatchDev& bt, char* ws, int items, unsigned thr, size_t lds, bool hi, hipStream_t st)
{
    if (hi) hipLaunchKernelGGL(k_rowpass_adj_b<true>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws);
    else hipLaunchKernelGGL(k_rowpass_adj_b<false>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws);
}

}  // namespace pat
