// grid_fwd.hip -- forward 2D-FFT passes: kernels and their launches.
#include "fft.hpp"
#include "grid.hpp"

namespace pat {

// Row / sample classes of the endpoint-term sums; red_s[1024] holds
// kSumClasses x the columns of a tile, so tiles have at most 32 (col_np <= 16).
constexpr int kSumClasses = 32;

// ---------------------------------------------------------------------------
// 2D-FFT passes of run-time grid sides (those without a compile-time form, grid.hpp)
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// forward: column pass (FFT along y of real columns, packed in pairs)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void colpass_fwd_tile(const PlanDev& d, const WsLayout& L, const float* __restrict__ fb,
                                                 char* wb, int tile, int NP, float2* sm, float* red_s)
{
    const int N = d.N, Ng = d.Ng, CT = 2 * NP;
    float2* X1 = (float2*)(wb + L.x1);
    float* red = (float*)(wb + L.red);
    const int j0 = tile * CT;
    const float2* tb = fft_twiddles_to_lds(sm + NP * Ng, d.ffts[d.fft_grid], d.tw);
    for (int e = threadIdx.x; e < NP * Ng; e += blockDim.x) sm[e] = make_float2(0.f, 0.f);
    __syncthreads();
    // the tile's columns, masked and deapodised, at rows centred in the padded
    // column (batched, branch-free loads; columns past N read as zero).
    // Endpoint term: h^2 times the masked sum of each column, rows in
    // kSumClasses classes (row i in class i mod kSumClasses), each summed in
    // order, then the classes in order (independent of the workgroup size and
    // of the tiling).  With kSumClasses x CT threads each thread's elements are
    // one column's rows of one class, in order: the class sums are taken from
    // the values loaded here; else a second loop reads the columns again.
    const float rcpCT = 1.0f / (float)CT;
    const bool own_class = (int)blockDim.x == kSumClasses * CT;
    float csum = 0.f;
    struct Elt {
        int i;
        float v, raw;
        bool in;
    };
    fill_batched<4>(
        N * CT,
        [&](int e) {
            int i, jj;
            fdivmod(e, CT, rcpCT, i, jj);
            const int j = j0 + jj, jc = min(j, N - 1);
            const int2 mr = d.mask_rows[i];
            const float fv = fb[(size_t)i * N + jc], di = d.deap[i], dj = d.deap[jc];
            const bool in = j < N && j >= mr.x && j < mr.y;
            const float v = in ? fv * di * dj : 0.f;
            int pos = i - N / 2;
            if (pos < 0) pos += Ng;
            return Elt{2 * ((jj >> 1) * Ng + pos) + (jj & 1), v, fv, in};
        },
        [&](int, Elt el) {
            ((float*)sm)[el.i] = el.v;
            csum = el.in ? csum + el.raw : csum;
        });
    if (own_class) red_s[threadIdx.x] = csum;  // class threadIdx.x / CT, column threadIdx.x % CT
    for (int t = threadIdx.x; !own_class && t < kSumClasses * CT; t += blockDim.x) {
        const int jj = t % CT, c = t / CT, j = j0 + jj, jc = min(j, N - 1);
        float sc = 0.f;
        for (int i0 = c; i0 < N; i0 += 4 * kSumClasses) {
            float v[4];
            bool in[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * kSumClasses, ic = min(i, N - 1);
                const int2 mr = d.mask_rows[ic];
                v[u] = fb[(size_t)ic * N + jc];
                in[u] = i < N && j < N && j >= mr.x && j < mr.y;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) sc = in[u] ? sc + v[u] : sc;
        }
        red_s[t] = sc;
    }
    __syncthreads();
    if ((int)threadIdx.x < CT && j0 + (int)threadIdx.x < N) {
        float sc = 0.f;
        for (int c = 0; c < kSumClasses; ++c) sc += red_s[c * CT + threadIdx.x];
        red[j0 + threadIdx.x] = sc * d.h2;
    }
    __syncthreads();
    fft_lds<false>(sm, Ng, NP, d.ffts[d.fft_grid], tb);
    fill_batched<4>(
        d.Hy * CT,
        [&](int e) {
            int r, jj;
            fdivmod(e, CT, rcpCT, r, jj);
            const int j = j0 + jj;
            const int m = r - 4;
            const int ip = m < 0 ? m + Ng : m;
            const int in = m > 0 ? Ng - m : -m;
            const float2 zp = sm[(jj >> 1) * Ng + ip], zn = sm[(jj >> 1) * Ng + in];
            // even column: (Z(m) + conj Z(-m)) / 2; odd: (Z(m) - conj Z(-m)) / (2i)
            const float2 o = (jj & 1) == 0 ? make_float2(0.5f * (zp.x + zn.x), 0.5f * (zp.y - zn.y))
                                           : make_float2(0.5f * (zp.y + zn.y), -0.5f * (zp.x - zn.x));
            return IdxVal{j < N ? r * N + j : -1, o};
        },
        [&](int, IdxVal iv) {
            if (iv.i >= 0) X1[iv.i] = iv.v;
        });
}

// ---------------------------------------------------------------------------
// forward: row pass (FFT along x)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void rowpass_fwd_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RPB,
                                                 float2* sm)
{
    const int N = d.N, Ng = d.Ng;
    const float2* X1 = (const float2*)(wb + L.x1);
    float2* G = (float2*)(wb + L.grid);
    const int r0 = tile * RPB;
    const int nr = min(RPB, d.Hy - r0);
    const float2* tb = fft_twiddles_to_lds(sm + RPB * Ng, d.ffts[d.fft_grid], d.tw);
    for (int e = threadIdx.x; e < nr * Ng; e += blockDim.x) sm[e] = make_float2(0.f, 0.f);
    __syncthreads();
    const float rcpN = 1.0f / (float)N;
    fill_batched<4>(
        nr * N,
        [&](int e) {
            int rr, j;
            fdivmod(e, N, rcpN, rr, j);
            int pos = j - N / 2;
            if (pos < 0) pos += Ng;
            return IdxVal{rr * Ng + pos, X1[(size_t)(r0 + rr) * N + j]};
        },
        [&](int, IdxVal iv) { sm[iv.i] = iv.v; });
    __syncthreads();
    fft_lds<false>(sm, Ng, nr, d.ffts[d.fft_grid], tb);
    fill_batched<4>(
        nr * Ng, [&](int e) { return sm[e]; }, [&](int e, float2 v) { G[(size_t)r0 * Ng + e] = v; });
}

__global__ __launch_bounds__(1024) void k_colpass_fwd(PlanDev d, WsLayout L, const float* __restrict__ f,
                                                     InstPtrs wsp, int NP)
{
    extern __shared__ float2 sm[];
    __shared__ float red_s[1024];
    const int b = blockIdx.y;
    colpass_fwd_tile(d, L, f + (size_t)b * d.N * d.N, wsp.ws + (size_t)b * wsp.stride, blockIdx.x, NP, sm, red_s);
}

__global__ __launch_bounds__(1024) void k_rowpass_fwd(PlanDev d, WsLayout L, InstPtrs wsp, int RPB)
{
    extern __shared__ float2 sm[];
    rowpass_fwd_tile(d, L, wsp.ws + (size_t)blockIdx.y * wsp.stride, blockIdx.x, RPB, sm);
}

// Compile-time grid sides: XCD-contiguous, instance-major tiles, so that an
// instance's X1 and G stay in one XCD's L2 from pass to pass.
template <int NG>
__global__ __launch_bounds__(1024) void k_colpass_fwd_spec(PlanDev d, WsLayout L, const float* __restrict__ f, InstPtrs wsp,
                                                           int NP, int vec, int ntile, int batch)
{
    extern __shared__ __align__(16) float2 smc[];
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    colpass_fwd_spec<NG>(d, L, f + (size_t)b * d.N * d.N, wsp.ws + (size_t)b * wsp.stride, item - b * ntile, NP, vec, smc);
}

template <int NG>
__global__ __launch_bounds__(1024) void k_rowpass_fwd_spec(PlanDev d, WsLayout L, InstPtrs wsp, int RPB, int ntile, int batch)
{
    extern __shared__ __align__(16) float2 smc[];
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    rowpass_fwd_spec<NG>(d, L, wsp.ws + (size_t)b * wsp.stride, item - b * ntile, RPB, smc);
}

// Heterogeneous batches.  HI: lengths above 1024 too (kept apart for their registers).
template <bool HI>
__global__ __launch_bounds__(1024) void k_colpass_fwd_b(BatchDev bt, const float* const* __restrict__ fin, char* ws)
{
    extern __shared__ __align__(16) float2 smc[];
    __shared__ float red_s[1024];
    int i, tile;
    if (!batch_item(bt, kStCol, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    const float* f = fin[i];
    char* wb = ws + I.ws_off;
    if (!d.grid_spec) {
        colpass_fwd_tile(d, I.L, f, wb, tile, I.col_np, smc, red_s);
        return;
    }
    const bool vec = (d.N & 1) == 0 && ((uintptr_t)f & 7) == 0;
    switch (d.Ng) {
#define PAT_CASE(NG) case NG: colpass_fwd_spec<NG>(d, I.L, f, wb, tile, I.col_np, vec, smc); break;
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
__global__ __launch_bounds__(1024) void k_rowpass_fwd_b(BatchDev bt, char* ws)
{
    extern __shared__ __align__(16) float2 smc[];
    int i, tile;
    if (!batch_item(bt, kStRow, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    char* wb = ws + I.ws_off;
    if (!d.grid_spec) {
        rowpass_fwd_tile(d, I.L, wb, tile, I.row_rpb, smc);
        return;
    }
    switch (d.Ng) {
#define PAT_CASE(NG) case NG: rowpass_fwd_spec<NG>(d, I.L, wb, tile, I.row_rpb, smc); break;
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

void colpass_fwd_launch(const pat_plan* p, const float* f, const InstPtrs& wsp, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int np = p->np_col, nt = p->n_col_tiles;
    if (!d.grid_spec) {
        hipLaunchKernelGGL(k_colpass_fwd, dim3(nt, batch), dim3(p->thr_col), p->lds_col, st, d, p->ws, f, wsp, np);
        return;
    }
    const int vec = (d.N & 1) == 0 && ((uintptr_t)f & 7) == 0;
    const dim3 grid(xcd_grid(nt * batch)), blk(p->thr_col);
    switch (d.Ng) {
#define PAT_CASE(NG) \
    case NG: hipLaunchKernelGGL(k_colpass_fwd_spec<NG>, grid, blk, p->lds_col, st, d, p->ws, f, wsp, np, vec, nt, batch); break;
        PAT_GRID_LENGTHS(PAT_CASE)
#undef PAT_CASE
        default: break;
    }
}

void rowpass_fwd_launch(const pat_plan* p, const InstPtrs& wsp, int batch, hipStream_t st)
{
    const PlanDev& d = p->dev;
    const int rpb = p->np_row, nt = (d.Hy + rpb - 1) / rpb;
    if (!d.grid_spec) {
        hipLaunchKernelGGL(k_rowpass_fwd, dim3(nt, batch), dim3(p->thr_row), p->lds_row, st, d, p->ws, wsp, rpb);
        return;
    }
    const dim3 grid(xcd_grid(nt * batch)), blk(p->thr_row);
    switch (d.Ng) {
#define PAT_CASE(NG) \
    case NG: hipLaunchKernelGGL(k_rowpass_fwd_spec<NG>, grid, blk, p->lds_row, st, d, p->ws, wsp, rpb, nt, batch); break;
        PAT_GRID_LENGTHS(PAT_CASE)
#undef PAT_CASE
        default: break;
    }
}

void colpass_fwd_b_launch(const BatchDev& bt, const float* const* f, char* ws, int items, unsigned thr, size_t lds, bool hi,
                          hipStream_t st)
{
    if (hi) hipLaunchKernelGGL(k_colpass_fwd_b<true>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, f, ws);
    else hipLaunchKernelGGL(k_colpass_fwd_b<false>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, f, ws);
}

void rowpass_fwd_b_launch(const BatchDev& bt, char* ws, int items, unsigned thr, size_t lds, bool hi, hipStream_t st)
{
    if (hi) hipLaunchKernelGGL(k_rowpass_fwd_b<true>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws);
    else hipLaunchKernelGGL(k_rowpass_fwd_b<false>, dim3(xcd_grid(items)), dim3(thr), lds, st, bt, ws);
}

}  // namespace pat
