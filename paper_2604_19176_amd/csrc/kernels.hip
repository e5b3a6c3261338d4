// kernels.hip -- gfx950 kernels of the PAT operator pair.
//
// Forward A (steps of the discrete operator; layouts per instance, row-major):
//   colpass_fwd : f [N][N] -> mask, deapodise, zero-pad to Ng, FFT along y of
//                 column pairs packed as complex -> X1 [Hy][N] (rows m_y = -4..Ng/2+4)
//                 + per-column sums of h^2 m f (endpoint term)
//   rowpass_fwd : X1 -> FFT along x -> G [Hy][Ng]  (oversampled half spectrum)
//   gather      : ES interpolation of G at the half-plane polar points, times
//                 the half-pixel phase -> F [npts] in ring order
//   ring_fwd    : per radial frequency n: angular FFT of the ring (completed by
//                 conjugate symmetry), weights c_k i^k J_k(lam_n R) W_n / Npsi(n),
//                 synthesis over the detector angles (one FFT after folding
//                 k mod P, or Bluestein) -> hT [nlam][D]
//   syn_dense   : explicit detector angles only: the synthesis as a matrix-core
//                 product of the ring's mode coefficients with a cos/sin table
//   dct         : per detector: g(d, j) = sum_n hT[n][d] cos(pi n j / M) via one
//                 complex FFT of length 2M for two detectors, + kappa * mass -> g [D][T]
// Adjoint A* runs the exact transposes in reverse (dct, ring_adj or
// syn_dense adjoint + ring_adj, spread (which applies the conjugate half-pixel
// phase as it stages each point), rowpass_adj, colpass_adj).  No
// floating-point atomics anywhere: every sum has a fixed order, so results are
// bitwise repeatable.
#include "cfft.hpp"
#include "device_util.hpp"
#include "fft.hpp"
#include "pat_internal.hpp"

namespace pat {


// Deterministic block sum (fixed tree); every thread gets the total.
__device__ float block_sum(float v, float* scratch)
{
    const int tid = threadIdx.x;
    scratch[tid] = v;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if (s < (int)blockDim.x && tid < s && tid + s < (int)blockDim.x) scratch[tid] += scratch[tid + s];
        __syncthreads();
    }
    float r = scratch[0];
    __syncthreads();
    return r;
}

// Sum of term(e) (float or float2), e < n, over the workgroup's threads, each in order
// (eight terms' loads in flight: one workgroup reduces an image, so it is bound by
// their latency)
template <class Term>
__device__ __forceinline__ auto strided_sum(long n, Term term)
{
    using V = decltype(term(0L));
    V acc{};
    const long bd = blockDim.x;
    long e = threadIdx.x;
    for (; e + 7 * bd < n; e += 8 * bd) {
        V v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = term(e + u * bd);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; e < n; e += bd) acc += term(e);
    return acc;
}

// Row / sample classes of the endpoint-term sums; red_s[1024] holds
// kSumClasses x (columns or detectors of a tile), so tiles have at most 32 of
// either (col_np, dct_dp <= 16).
constexpr int kSumClasses = 32;

// ---------------------------------------------------------------------------
// forward: ES interpolation of the half spectrum at the half-plane polar
// points.  Points are visited in band order (sorted by footprint base row r0,
// then base column bx); a tile is TH bands x CB columns: the points with r0
// in [R0, R0 + TH) and bx in [C0, C0 + CB).  The tile's whole window of the
// spectrum (rows R0 .. R0 + TH + 6, columns C0 .. C0 + CB + 6, wrapping
// around the periodic grid) is loaded into LDS once; then each band is
// handled by kGatherThreads / TH threads, one point per thread at a time.
// Output: the polar value times the half-pixel phase, stored in ring order
// (the ring-order index is the y field of the point's band-order geometry).
// ---------------------------------------------------------------------------
// IB instances of one plan share a tile (wbs[b], b < nb; b >= nb is padding):
// one window per instance, the ES weights and indexing of each point once.
template <int IB, int CB>
__device__ __forceinline__ void gather_tile(const PlanDev& d, const WsLayout& L, char* const (&wbs)[IB], int nb,
                                            int tile, int TH, float2* win)
{
    constexpr int W = CB + 7;  // compile-time row stride: the 64 taps are immediate offsets
    const int Ng = d.Ng, NB = d.NB, Hy = d.Hy;
    const int R = TH + 7, RW = R * W;
    const int ncb = (Ng + CB - 1) / CB;
    const int rbk = tile / ncb, cbk = tile - rbk * ncb;
    const int C0 = cbk * CB, R0 = rbk * TH;
    const int cend = min(C0 + CB, Ng);
    const int nbands = min(TH, NB - R0);
    int* seg_lo = (int*)(win + IB * RW);
    int* seg_hi = seg_lo + TH;
#pragma unroll
    for (int b = 0; b < IB; ++b) {
        if (b >= nb) break;
        const float2* __restrict__ G = (const float2*)(wbs[b] + L.grid);
        float2* wn = win + b * RW;
        // window rows R0 .. R0 + TH + 6 (zero past the stored rows), columns
        // C0 .. C0 + CB + 6 wrapped mod Ng (C0 + CB + 6 < 2 Ng)
        fill_batched<4>(
            RW,
            [&](int e) {
                const int rr = e / W, cc = e - rr * W;
                const int r = R0 + rr;
                int c = C0 + cc;
                c = c >= Ng ? c - Ng : c;
                const float2 v = G[(size_t)min(r, Hy - 1) * Ng + c];
                return r < Hy ? v : make_float2(0.f, 0.f);
            },
            [&](int e, float2 v) { wn[e] = v; });
    }
    if ((int)threadIdx.x < nbands) {
        const int* bp = d.band_ptr + (size_t)(R0 + threadIdx.x) * (Ng + 1);
        seg_lo[threadIdx.x] = bp[C0];
        seg_hi[threadIdx.x] = bp[cend];
    }
    __syncthreads();
    const int Q = kGatherThreads / TH;  // threads per band
    const int bnd = threadIdx.x / Q, u = threadIdx.x - bnd * Q;
    if (bnd >= nbands) return;          // no barrier follows
    const int hi = seg_hi[bnd];
    // the next point's geometry is loaded while the current one is interpolated
    // (index clamped to the segment's last point, or to point 0 for an empty
    // segment at the start: always a valid point)
    const int slast = max(hi - 1, 0);
    int s = seg_lo[bnd] + u;
    float4 ngq = d.bpt_geo[min(s, slast)];
    float2 nph = d.bpt_phase[min(s, slast)];
    for (; s < hi; s += Q) {
        const float4 gq = ngq;
        const float2 ph = nph;
        const int ri = fbits(gq.y);  // ring-order index of the point
        const int sn = min(s + Q, slast);
        ngq = d.bpt_geo[sn];
        nph = d.bpt_phase[sn];
        const int c0 = fbits(gq.x) - C0;
        float wx[8], wy[8];
        es_weights8(gq.z, wx);
        es_weights8(gq.w, wy);
#pragma unroll
        for (int b = 0; b < IB; ++b) {
            if (b >= nb) break;
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int dy = 0; dy < 8; ++dy) {
                const float2* row = win + b * RW + (bnd + dy) * W + c0;
                float2 ra = make_float2(0.f, 0.f);
#pragma unroll
                for (int dx = 0; dx < 8; ++dx) {
                    const float2 gv = row[dx];
                    ra.x = fmaf(wx[dx], gv.x, ra.x);
                    ra.y = fmaf(wx[dx], gv.y, ra.y);
                }
                acc.x = fmaf(wy[dy], ra.x, acc.x);
                acc.y = fmaf(wy[dy], ra.y, acc.y);
            }
            ((float2*)(wbs[b] + L.polar))[ri] = cmul(acc, ph);
        }
    }
}

// ---------------------------------------------------------------------------
// Explicit detector angles: the angular synthesis h(n, d) = Re sum_k a_k(n)
// e^{ik theta_d} (eq. (2)) as a dense product on the matrix cores,
//   forward  H[n][d] = sum_{j < 2(K_n + 1)} A[n][j] S[j][d],
//   adjoint  A[n][j] = sum_d H[n][d] S[j][d],
// with A the mode coefficients (re, im interleaved: [nlam][2(K+1)] floats) and
// S the FP64-computed table S[2k] = cos(k theta_d), S[2k+1] = -sin(k theta_d).
// 64 x 64 output tiles, four waves of 32 x 32 each (v_mfma_f32_32x32x2f32:
// lane i holds A[i % 32][i / 32] and B[i / 32][i % 32]; accumulator r holds
// D[8 (r / 4) + 4 (i / 32) + r % 4][i % 32]); the contraction runs in chunks of
// 32 staged in LDS.  Rows are rings: a tile stops at 2 (K_n + 1) of its last
// ring (K_n grows with n), and A's entries beyond a ring's own cut-off are
// read as zero, so the product skips the modes a ring does not have.
// ---------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kSynTile = 64;     // output tile side
constexpr int kSynChunk = 32;    // contraction chunk
constexpr int kSynThreads = 256; // four waves
constexpr int kSynLd = kSynChunk + 4;                    // LDS row stride (floats) of the operand fragments
constexpr int kSynPer = kSynTile * kSynChunk / kSynThreads;  // fragment elements fetched per thread
constexpr int kSynRows = kSynThreads / kSynChunk;        // rows one fetch step covers

// Operand fragments of a chunk in LDS, [64 tile rows / columns][kSynLd]: the
// element of contraction index k (0 .. kSynChunk-1) sits in slot
// (k & 1) * kSynChunk/2 + k / 2, so that the values lane group h = lane / 32
// feeds to the MFMAs of a chunk (k = 2 i + h) are contiguous: 128-bit LDS reads.
__device__ __forceinline__ int syn_slot(int k) { return (k & 1) * (kSynChunk / 2) + (k >> 1); }

__device__ __forceinline__ void syn_mfma_chunk(const float (*Ap)[kSynLd], const float (*Bp)[kSynLd], int wm, int wn,
                                               int lane, f32x16& acc)
{
    constexpr int NV = kSynChunk / 8;  // float4 per operand and lane
    const int h = lane >> 5, rr = lane & 31;
    const float4* ar = (const float4*)&Ap[wm + rr][h * (kSynChunk / 2)];
    const float4* br = (const float4*)&Bp[wn + rr][h * (kSynChunk / 2)];
    float4 a4[NV], b4[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        a4[i] = ar[i];
        b4[i] = br[i];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[i].x, b4[i].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[i].y, b4[i].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[i].z, b4[i].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[i].w, b4[i].w, acc, 0, 0, 0);
    }
}

// Forward: each chunk, thread t holds kSynPer values of the mode block
// (ring r = t / kSynChunk + kSynRows i, index c = t % kSynChunk) and kSynPer of
// the table block (k = t / 64 + 4 i, detector c = t % 64); the next chunk is fetched into
// registers while the matrix cores work on the current one.  Loads go to
// clamped in-bounds addresses without branches and masked entries are zeroed
// afterwards, so all 16 loads of a chunk are in flight together.
__device__ __forceinline__ void syn_dense_fwd_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile)
{
    __shared__ __align__(16) float Ap[kSynTile][kSynLd];  // [ring][slot]
    __shared__ __align__(16) float Bp[kSynTile][kSynLd];  // [detector][slot]
    const int J = 2 * d.Kp, D = d.D, NL = d.nlam;
    const int tq = (D + kSynTile - 1) / kSynTile;
    const int n0 = (tile / tq) * kSynTile, q0 = (tile % tq) * kSynTile;
    const float* __restrict__ A = (const float*)(wb + L.modes);
    const float* __restrict__ S = d.syn_tab;
    float* __restrict__ H = (float*)(wb + L.hdet);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    const int jmax = 2 * (d.ring_K[min(n0 + kSynTile - 1, NL - 1)] + 1);
    const int nch = (jmax + kSynChunk - 1) / kSynChunk;
    // this thread's rings: row offsets and mode limits 2 (K_n + 1) (0 past nlam)
    int aoff[kSynPer], jlim[kSynPer];
#pragma unroll
    for (int i = 0; i < kSynPer; ++i) {
        const int n = n0 + tid / kSynChunk + kSynRows * i;
        const int nc = min(n, NL - 1);
        aoff[i] = nc * J;
        jlim[i] = n < NL ? 2 * (d.ring_K[nc] + 1) : 0;
    }
    const int ca = tid % kSynChunk, cb = tid & 63;
    const int q = q0 + cb, qc = min(q, D - 1);
    float ra[kSynPer], rb[kSynPer];
    auto fetch = [&](int j0) {
        const int j = j0 + ca, jc = min(j, J - 1);
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            ra[i] = A[aoff[i] + jc];
            const int jb = j0 + (tid >> 6) + 4 * i;
            rb[i] = S[(size_t)min(jb, J - 1) * D + qc];
        }
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            if (j >= jlim[i]) ra[i] = 0.f;
            if (j0 + (tid >> 6) + 4 * i >= J || q >= D) rb[i] = 0.f;
        }
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    if (nch > 0) fetch(0);
    for (int ch = 0; ch < nch; ++ch) {
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            Ap[tid / kSynChunk + kSynRows * i][syn_slot(ca)] = ra[i];
            Bp[cb][syn_slot((tid >> 6) + 4 * i)] = rb[i];
        }
        __syncthreads();
        if (ch + 1 < nch) fetch((ch + 1) * kSynChunk);
        syn_mfma_chunk(Ap, Bp, wm, wn, lane, acc);
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int n = n0 + wm + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), qq = q0 + wn + (lane & 31);
        if (n < NL && qq < D) H[(size_t)n * D + qq] = acc[r];
    }
}

// Adjoint: both operands are read along the detector index (row
// r = t / kSynChunk + kSynRows i, detector c = t % kSynChunk), with the same
// branch-free clamped loads.
__device__ __forceinline__ void syn_dense_adj_tile(const PlanDev& d, const WsLayout& L, char* wb, int tile)
{
    __shared__ __align__(16) float Ap[kSynTile][kSynLd];  // [ring][slot]
    __shared__ __align__(16) float Bp[kSynTile][kSynLd];  // [table row j][slot]
    const int J = 2 * d.Kp, D = d.D, NL = d.nlam;
    const int tj = (J + kSynTile - 1) / kSynTile;
    const int n0 = (tile / tj) * kSynTile, j0 = (tile % tj) * kSynTile;
    // rows j >= 2 (K_n + 1) of every ring of the tile are never read: skip the tile
    if (j0 >= 2 * (d.ring_K[min(n0 + kSynTile - 1, NL - 1)] + 1)) return;
    const float* __restrict__ H = (const float*)(wb + L.hdet);
    const float* __restrict__ S = d.syn_tab;
    float* __restrict__ A = (float*)(wb + L.modes);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    const int nch = (D + kSynChunk - 1) / kSynChunk;
    const int ca = tid % kSynChunk, r0 = tid / kSynChunk;
    int hoff[kSynPer], soff[kSynPer];
    unsigned okh = 0, oks = 0;  // row i inside nlam / inside the table
#pragma unroll
    for (int i = 0; i < kSynPer; ++i) {
        const int n = n0 + r0 + kSynRows * i, j = j0 + r0 + kSynRows * i;
        hoff[i] = min(n, NL - 1) * D;
        soff[i] = min(j, J - 1) * D;
        okh |= (n < NL ? 1u : 0u) << i;
        oks |= (j < J ? 1u : 0u) << i;
    }
    float ra[kSynPer], rb[kSynPer];
    auto fetch = [&](int c0) {
        const int qv = c0 + ca, qc = min(qv, D - 1);
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            ra[i] = H[hoff[i] + qc];
            rb[i] = S[soff[i] + qc];
        }
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            if (qv >= D || !((okh >> i) & 1u)) ra[i] = 0.f;
            if (qv >= D || !((oks >> i) & 1u)) rb[i] = 0.f;
        }
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    fetch(0);
    for (int ch = 0; ch < nch; ++ch) {
#pragma unroll
        for (int i = 0; i < kSynPer; ++i) {
            Ap[r0 + kSynRows * i][syn_slot(ca)] = ra[i];
            Bp[r0 + kSynRows * i][syn_slot(ca)] = rb[i];
        }
        __syncthreads();
        if (ch + 1 < nch) fetch((ch + 1) * kSynChunk);
        syn_mfma_chunk(Ap, Bp, wm, wn, lane, acc);
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int n = n0 + wm + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), j = j0 + wn + (lane & 31);
        if (n < NL && j < J) A[(size_t)n * J + j] = acc[r];
    }
}

// ---------------------------------------------------------------------------
// Cosine transform over radial frequencies, per detector, two detectors packed
// as the real and imaginary parts of one complex sequence (the transform is
// real):  out(q) = sum_p in(p) cos(pi p q / M) = (X[q] + X[2M - q]) / 2 with
// X = FFT_2M of the zero-padded input (p, q >= 1).
//   forward: hT [nlam][D] -> g [D][T] (+ kappa * mass)
//   adjoint: g [D][T] -> hT [nlam][D] (+ per-detector sums of g)
// ---------------------------------------------------------------------------
// gout / gin point at this instance's [D][T] data.
__device__ __forceinline__ void dct_tile(const PlanDev& d, const WsLayout& L, char* wb, float* __restrict__ gout,
                                         const float* __restrict__ gin, int tile, int DP, int adj, int n_mass,
                                         float2* sm, float* red_s, float* mass_s)
{
    const int twoM = 2 * d.M, D = d.D, T = d.T, NL = d.nlam;
    float* hT = (float*)(wb + L.hdet);
    float* red = (float*)(wb + L.red);
    const int p0 = tile * DP;                        // first detector pair
    const int np = min(DP, (D + 1) / 2 - p0);
    const int nin = adj ? T : NL;
    const int nout = adj ? NL : T;
    if (!adj && threadIdx.x < 64) {
        const float m = wave0_fixed_sum(red, n_mass);
        if (threadIdx.x == 0) *mass_s = m;
    }
    const float2* tb = fft_twiddles_to_lds(sm + DP * twoM, d.ffts[d.fft_dct], d.tw);
    for (int e = threadIdx.x; e < np * twoM; e += blockDim.x) sm[e] = make_float2(0.f, 0.f);
    __syncthreads();
    // input pairs (detector d0 real, d0 + 1 imaginary) at sm[p][q + 1]; the loads
    // of a thread are batched (fill_batched), the partner of the last odd detector is 0
    if (adj) {  // g [D][T]: contiguous along t
        const float rcp = 1.0f / (float)nin;
        fill_batched<4>(
            np * nin,
            [&](int e) {
                int p, q;
                fdivmod(e, nin, rcp, p, q);
                const int d0 = 2 * (p0 + p);
                const float re = gin[(size_t)d0 * T + q];
                const float im = gin[(size_t)min(d0 + 1, D - 1) * T + q];
                return IdxVal{p * twoM + q + 1, make_float2(re, d0 + 1 < D ? im : 0.f)};
            },
            [&](int, IdxVal iv) { sm[iv.i] = iv.v; });
    } else {    // hT [nlam][D]: the tile's detectors are contiguous within a row
        const float rcp = 1.0f / (float)np;
        fill_batched<4>(
            np * nin,
            [&](int e) {
                int q, p;
                fdivmod(e, np, rcp, q, p);
                const int d0 = 2 * (p0 + p);
                const float* row = hT + (size_t)q * D;
                const float re = row[d0];
                const float im = row[min(d0 + 1, D - 1)];
                return IdxVal{p * twoM + q + 1, make_float2(re, d0 + 1 < D ? im : 0.f)};
            },
            [&](int, IdxVal iv) { sm[iv.i] = iv.v; });
    }
    if (adj) {
        // data sum of each detector of the tile (from the copy in LDS): samples in
        // kSumClasses classes, each summed in order, then the classes in order
        __syncthreads();
        const int nd = 2 * np;
        for (int t = threadIdx.x; t < kSumClasses * nd; t += blockDim.x) {
            const int c = t % kSumClasses, dd = t / kSumClasses, dg = 2 * p0 + dd;
            const float2* col = sm + (dd >> 1) * twoM + 1;
            float sc = 0.f;
            if (dg < D) {
                if (dd & 1)
                    for (int q = c; q < T; q += kSumClasses) sc += col[q].y;
                else
                    for (int q = c; q < T; q += kSumClasses) sc += col[q].x;
            }
            red_s[t] = sc;
        }
        __syncthreads();
        if ((int)threadIdx.x < nd && 2 * p0 + (int)threadIdx.x < D) {
            float sc = 0.f;
            for (int c = 0; c < kSumClasses; ++c) sc += red_s[threadIdx.x * kSumClasses + c];
            red[2 * p0 + threadIdx.x] = sc;
        }
    }
    __syncthreads();
    fft_lds<false>(sm, twoM, np, d.ffts[d.fft_dct], tb);
    const float add = adj ? 0.f : d.kappa * *mass_s;
    // outputs X[q + 1] + X[2M - q - 1] (halved) of each pair; the LDS reads of a
    // thread are batched ahead of its stores
    if (adj) {  // -> hT [nlam][D]
        const float rcp = 1.0f / (float)np;
        fill_batched<4>(
            np * nout,
            [&](int e) {
                int q, p;
                fdivmod(e, np, rcp, q, p);
                const float2 a = sm[p * twoM + q + 1], c = sm[p * twoM + twoM - q - 1];
                return make_float2(0.5f * (a.x + c.x), 0.5f * (a.y + c.y));
            },
            [&](int e, float2 v) {
                int q, p;
                fdivmod(e, np, rcp, q, p);
                const int d0 = 2 * (p0 + p);
                float* row = hT + (size_t)q * D;
                row[d0] = v.x;
                if (d0 + 1 < D) row[d0 + 1] = v.y;
            });
    } else {    // -> g [D][T]
        const float rcp = 1.0f / (float)nout;
        fill_batched<4>(
            np * nout,
            [&](int e) {
                int p, q;
                fdivmod(e, nout, rcp, p, q);
                const float2 a = sm[p * twoM + q + 1], c = sm[p * twoM + twoM - q - 1];
                return make_float2(0.5f * (a.x + c.x) + add, 0.5f * (a.y + c.y) + add);
            },
            [&](int e, float2 v) {
                int p, q;
                fdivmod(e, nout, rcp, p, q);
                const int d0 = 2 * (p0 + p);
                gout[(size_t)d0 * T + q] = v.x;
                if (d0 + 1 < D) gout[(size_t)(d0 + 1) * T + q] = v.y;
            });
    }
}

// ---------------------------------------------------------------------------
// The cosine transform with a compile-time length N2 = 2M (plans with
// dct_spec): the same transform as dct_tile, one detector pair per sequence
// of cfft_lanes(N2) lanes, DP pairs per workgroup.  The first pass (Ns = 1,
// no twiddles) takes its inputs straight from memory, so the zero padding is
// never stored, and blocks of it are never read.  The adjoint writes hT row
// by row, the workgroup's pairs side by side.  The adjoint's per-detector data
// sums are taken from the first pass's inputs, lane by lane in order, across
// each wave's lanes by a fixed tree, then over the pair's waves in order (the
// partial sums cross the barrier that precedes the second pass): one order
// for every launch shape.
// ---------------------------------------------------------------------------
template <int N2>
__device__ __forceinline__ void dct_spec_tile(const PlanDev& d, const WsLayout& L, char* wb, float* __restrict__ gout,
                                              const float* __restrict__ gin, int tile, int DP, int adj, int n_mass,
                                              float2* sm, float* red_s, float* mass_s)
{
    constexpr int T = cfft_lanes(N2);
    constexpr CPlan P = CPlanOf<N2>::p;
    constexpr int R0 = P.rad[0], NB0 = N2 / R0, RND0 = (NB0 + T - 1) / T;
    const int D = d.D, TT = d.T, NL = d.nlam;
    float* hT = (float*)(wb + L.hdet);
    float* red = (float*)(wb + L.red);
    const int npair = (D + 1) / 2;
    const int p0 = tile * DP;               // the workgroup's first pair
    const int npw = min(DP, npair - p0);    // and its number of pairs
    const int sq = threadIdx.x / T, lane = threadIdx.x - sq * T;
    const bool active = sq < npw;
    const int d0 = 2 * min(p0 + sq, npair - 1);
    const int d1 = d0 + 1 < D ? d0 + 1 : d0;  // the partner of the last odd detector reads d0, weighted 0
    const float w1 = d0 + 1 < D ? 1.f : 0.f;
    // D even: every pair's two values sit at an 8-byte aligned address of each row
    const bool pair2 = (D & 1) == 0;
    constexpr int NP2 = cfft_padded_len(N2);  // LDS slots per pair (padded sequence)
    float2* x = sm + (size_t)min(sq, DP - 1) * NP2;
    const float2* __restrict__ tw = d.ctw + d.dct_ctw;
    if (!adj && threadIdx.x < 64) {
        const float m = wave0_fixed_sum(red, n_mass);
        if (threadIdx.x == 0) *mass_s = m;
    }
    const int nin = adj ? TT : NL;
    // input position pos (1..nin) of the pair: g(d, pos-1) (adjoint) or
    // hT[pos-1][d] (forward); zero elsewhere
    auto inp = [&](int pos) {
        const int q = min(max(pos - 1, 0), nin - 1);
        float re, im;
        if (adj) {
            re = gin[(size_t)d0 * TT + q];
            im = gin[(size_t)d1 * TT + q];
        } else if (pair2) {  // the pair's two values are adjacent in the row: one 8-byte load
            const float2 v = *(const float2*)(hT + (size_t)q * D + d0);
            re = v.x;
            im = v.y;
        } else {
            const float* row = hT + (size_t)q * D;
            re = row[d0];
            im = row[d1];
        }
        const bool in = pos >= 1 && pos <= nin;
        return make_float2(in ? re : 0.f, in ? w1 * im : 0.f);
    };
    // first pass (Ns = 1, no twiddles), fed from the inputs; inputs past
    // position nin are the zero padding: a whole block of them needs no load.
    // The adjoint's lanes sum the pair's data (for the endpoint term's
    // transpose) from the same values.
    float s0 = 0.f, s1 = 0.f;
    float2 v[RND0][R0];
    // the second pass's twiddles, in flight with the inputs
    PassTw<N2, P.rad[1], P.ns[1], T> tw1;
    pass_tw_load<N2, P.rad[1], P.ns[1], P.twoff[1], T>(tw1, tw, active, lane);
    if (active) {
#pragma unroll
        for (int i = 0; i < RND0; ++i) {
            const int j0 = lane + i * T;
            const bool own = NB0 % T == 0 || i + 1 < RND0 || j0 < NB0;
            // the last round's idle lanes work on the last butterfly (results dropped)
            const int j = own ? j0 : NB0 - 1;
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                v[i][r] = (r * NB0 <= nin) ? inp(j + r * NB0) : make_float2(0.f, 0.f);
                if (adj && own) {
                    s0 += v[i][r].x;
                    s1 += v[i][r].y;
                }
            }
            butterfly<R0, false>(v[i]);
        }
    }
    if (active) {
#pragma unroll
        for (int i = 0; i < RND0; ++i) {
            const int j = lane + i * T;
            if (NB0 % T == 0 || i + 1 < RND0 || j < NB0) {
#pragma unroll
                for (int r = 0; r < R0; ++r) x[cfft_slot<true>(j * R0 + r)] = v[i][r];
            }
        }
    }
    if (adj) {  // each wave's share of the sums, across its lanes by a fixed tree
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            s0 += __shfl_down(s0, o, 64);
            s1 += __shfl_down(s1, o, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            red_s[2 * (threadIdx.x >> 6)] = s0;
            red_s[2 * (threadIdx.x >> 6) + 1] = s1;
        }
    }
    __syncthreads();
    if (adj && active && lane == 0) {  // the pair's waves in order
        const int w0 = threadIdx.x >> 6;
        float t0 = 0.f, t1 = 0.f;
#pragma unroll
        for (int k = 0; k < T / 64; ++k) {
            t0 += red_s[2 * (w0 + k)];
            t1 += red_s[2 * (w0 + k) + 1];
        }
        red[d0] = t0;
        if (d0 + 1 < D) red[d0 + 1] = t1;
    }
    cfft_passes_tw<N2, false, 1, true, T>(x, tw, active, lane, tw1);
    if (adj) {
        // -> hT [nlam][D]: row by row, the workgroup's pairs side by side
        const float rcp = 1.0f / (float)npw;
        fill_batched<4>(
            NL * npw,
            [&](int e) {
                int q, p;
                fdivmod(e, npw, rcp, q, p);
                const float2 a = sm[p * NP2 + cfft_slot<true>(q + 1)], c = sm[p * NP2 + cfft_slot<true>(N2 - q - 1)];
                return make_float2(0.5f * (a.x + c.x), 0.5f * (a.y + c.y));
            },
            [&](int e, float2 o) {
                int q, p;
                fdivmod(e, npw, rcp, q, p);
                const int a = 2 * (p0 + p);
                float* row = hT + (size_t)q * D;
                if (pair2) {
                    *(float2*)(row + a) = o;
                } else {
                    row[a] = o.x;
                    if (a + 1 < D) row[a + 1] = o.y;
                }
            });
        return;
    }
    if (!active) return;  // no barrier follows
    const float add = d.kappa * *mass_s;
    // -> g [D][T]: contiguous along t
    for (int q0 = 0; q0 < TT; q0 += 2 * T) {
        float2 o[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = min(q0 + lane + u * T, TT - 1);
            const float2 a = x[cfft_slot<true>(q + 1)], c = x[cfft_slot<true>(N2 - q - 1)];
            o[u] = make_float2(0.5f * (a.x + c.x) + add, 0.5f * (a.y + c.y) + add);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = q0 + lane + u * T;
            if (q < TT) {
                gout[(size_t)d0 * TT + q] = o[u].x;
                if (d0 + 1 < D) gout[(size_t)(d0 + 1) * TT + q] = o[u].y;
            }
        }
    }
}

// Lengths 2M with a compile-time cosine transform
#define PAT_DCT_LENGTHS(X) X(256) X(512) X(1024) X(2048) X(4096) X(8192)

__device__ __forceinline__ void dct_run(const PlanDev& d, const WsLayout& L, char* wb, float* __restrict__ gout,
                                        const float* __restrict__ gin, int tile, int DP, int adj, int n_mass,
                                        float2* sm, float* red_s, float* mass_s)
{
    switch (2 * d.M) {
#define PAT_DCT_CASE(N2) \
    case N2: dct_spec_tile<N2>(d, L, wb, gout, gin, tile, DP, adj, n_mass, sm, red_s, mass_s); break;
        PAT_DCT_LENGTHS(PAT_DCT_CASE)
#undef PAT_DCT_CASE
        default: break;
    }
}

// ---------------------------------------------------------------------------
// adjoint: deterministic spread of the polar half-plane values onto G~ [Hy][Ng]
// One lane owns one column; bands (footprint base rows) are swept in order and
// an 8-row register window accumulates; band points are staged in LDS with
// their ES weights.  Every output is a fixed-order sum.  The next band's
// ranges and first points are fetched into registers while the current band
// is processed.
// ---------------------------------------------------------------------------
struct BandMeta {
    int aLo, nA, bLo, ntot, lo, hi;
};

// A band's row of the band CSR as the spread tile at columns [C0, C0 + CB)
// needs it: v[k] = band_ptr[rb][col] for col = C0 - 7 + k (k = 0 .. CB + 8),
// wrapped to col + Ng below 0 and clamped to Ng above, and v[CB + 9] =
// band_ptr[rb][Ng].  Each thread fetches entries tid and tid + CB.
__device__ __forceinline__ void band_row_fetch(const PlanDev& d, int rb, int C0, int CB, int (&v)[2])
{
    const int Ng = d.Ng;
    const int* bp = d.band_ptr + (size_t)rb * (Ng + 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = threadIdx.x + i * CB;
        v[i] = 0;
        if (k < CB + 10) {
            const int col = C0 - 7 + k;
            v[i] = k == CB + 9 ? bp[Ng] : bp[col < 0 ? col + Ng : min(col, Ng)];
        }
    }
}

__device__ __forceinline__ void band_row_store(int* row, int CB, const int (&v)[2])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = threadIdx.x + i * CB;
        if (k < CB + 10) row[k] = v[i];
    }
}

// Staged-index ranges of a band from its CSR row in LDS: the wrapped segment
// (columns Ng-7 .. Ng-1, only for the tile at column 0) comes first, then the
// columns C0-7 .. C0+CB-1; lane's visit range is its footprint columns mx-7 .. mx.
__device__ __forceinline__ BandMeta band_meta(const int* row, int Ng, int C0, int CB, bool active)
{
    const int lo_col = C0 - 7;
    const int khi = min(C0 + CB, Ng) - lo_col;
    BandMeta m;
    m.aLo = lo_col < 0 ? row[0] : 0;
    const int aHi = lo_col < 0 ? row[CB + 9] : 0;
    m.bLo = row[lo_col < 0 ? -lo_col : 0];
    m.nA = aHi - m.aLo;
    m.ntot = m.nA + (row[khi] - m.bLo);
    m.lo = m.hi = 0;
    if (active) {
        const int t = threadIdx.x;
        m.lo = (lo_col + t < 0) ? (row[t] - m.aLo) : (m.nA + row[t] - m.bLo);
        m.hi = m.nA + row[t + 8] - m.bLo;
    }
    return m;
}

__device__ __forceinline__ int band_slot(const BandMeta& m, int idx)
{
    return idx < m.nA ? m.aLo + idx : m.bLo + (idx - m.nA);
}

// LDS of the spread (spread_lds_words): column-major so that lanes reading
// neighbouring points hit distinct banks.
template <int IB>
struct SpreadLds {
    float* wx;
    float* wy;
    int* bx;
    float2* h;
};

// staged value: the point's H times the conjugate half-pixel phase ph
template <int IB, int CAP>
__device__ __forceinline__ void spread_stage(const SpreadLds<IB>& S, int e, float4 gq, int bx_rel,
                                             const float2 (&h)[IB], float2 ph)
{
    float w[8];
    es_weights8(gq.z, w);
#pragma unroll
    for (int k = 0; k < 8; ++k) S.wx[k * CAP + e] = w[k];
    es_weights8(gq.w, w);
#pragma unroll
    for (int k = 0; k < 8; ++k) S.wy[k * CAP + e] = w[k];
    S.bx[e] = bx_rel;
    // explicit roundings: the same product in every instantiation of the tile
#pragma unroll
    for (int b = 0; b < IB; ++b)
        S.h[b * CAP + e] = make_float2(fmaf(h[b].x, ph.x, __fmul_rn(h[b].y, ph.y)),
                                       fmaf(h[b].y, ph.x, -__fmul_rn(h[b].x, ph.y)));
}

template <int IB, int CAP>
__device__ __forceinline__ void spread_visit(const SpreadLds<IB>& S, int s0, int s1, int c0, int lane7,
                                             float2 (&acc)[IB][8])
{
    if constexpr (IB == 1) {
        // one instance (small batches, where a tile's wave is often alone on
        // its SIMD): the LDS reads of the next point, and the column of the
        // one after, are issued before the current point's products (the same
        // products in the same order)
        if (s0 >= s1) return;
        const int last = s1 - 1 - c0;
        int e = s0 - c0;
        float w = S.wx[(lane7 - S.bx[e]) * CAP + e];
        float wy[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) wy[k] = S.wy[k * CAP + e];
        float2 hv = S.h[e];
        int bxn = S.bx[min(e + 1, last)];
        for (int s = s0; s < s1; ++s) {
            const int en = min(e + 1, last);
            const int bx2 = S.bx[min(e + 2, last)];
            const float wn = S.wx[(lane7 - bxn) * CAP + en];
            float wyn[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) wyn[k] = S.wy[k * CAP + en];
            const float2 hn = S.h[en];
            const float2 t = cscale(hv, w);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                acc[0][k].x = fmaf(wy[k], t.x, acc[0][k].x);
                acc[0][k].y = fmaf(wy[k], t.y, acc[0][k].y);
            }
            w = wn;
            hv = hn;
#pragma unroll
            for (int k = 0; k < 8; ++k) wy[k] = wyn[k];
            bxn = bx2;
            e = en;
        }
        return;
    }
    for (int s = s0; s < s1; ++s) {
        const int e = s - c0;
        const int dx = lane7 - S.bx[e];
        const float w = S.wx[dx * CAP + e];
        float wy[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) wy[k] = S.wy[k * CAP + e];
#pragma unroll
        for (int b = 0; b < IB; ++b) {
            const float2 t = cscale(S.h[b * CAP + e], w);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                acc[b][k].x = fmaf(wy[k], t.x, acc[b][k].x);
                acc[b][k].y = fmaf(wy[k], t.y, acc[b][k].y);
            }
        }
    }
}

// One tile of the spread for IB instances of one plan (wbs[b], b < nb, are the
// instance workspaces; instances b >= nb are padding and neither read nor
// written).  The workgroup has CB threads, one per column; CAP = 2 CB points
// are staged per chunk.  Work row wr (d.spr_row[wr]) sweeps a run of bands:
// a whole row tile rt, bands [8 rt, 8 rt + 8), writes their grid rows and
// leaves its partial sums for the 7 rows after its last band in the tail
// region unless it is the last row tile (the adjoint row pass adds them to the
// next tile's first rows); a run of a split row tile writes every row it
// touches, partial, to its rows of the slab region.  CB is a compile-time
// constant so that every LDS access of the inner loops is an immediate offset
// from one base address.
template <int IB, int CB>
__device__ __forceinline__ void spread_tile(const PlanDev& d, const WsLayout& L, char* const (&wbs)[IB], int nb,
                                            int tile, float* sf)
{
    constexpr int CAP = 2 * CB;
    const int Ng = d.Ng, NB = d.NB;
    const int ncb = (Ng + CB - 1) / CB;
    const int wr = tile / ncb, cb_ = tile - wr * ncb;
    const int4 run = d.spr_row[wr];
    const int band_lo = run.x, band_hi = run.y, rt = run.w;
    const bool to_slab = run.z >= 0;
    // the work row's output rows, from its first band on: grid or slab rows
    const float2* __restrict__ H[IB];
    float2* Ob[IB];
#pragma unroll
    for (int b = 0; b < IB; ++b) {
        H[b] = (const float2*)(wbs[b] + L.polar);
        Ob[b] = to_slab ? (float2*)(wbs[b] + L.slab) + (size_t)run.z * Ng : (float2*)(wbs[b] + L.grid) + (size_t)band_lo * Ng;
    }
    SpreadLds<IB> S;
    S.wx = sf;
    S.wy = sf + 8 * CAP;
    S.bx = (int*)(sf + 16 * CAP);
    S.h = (float2*)(sf + 17 * CAP);  // CAP is even: 8-byte aligned
    int* rows = (int*)(sf + (size_t)CAP * (17 + 2 * IB));  // [3][CB + 10]
    const int C0 = cb_ * CB;
    const int mx = C0 + threadIdx.x;
    const int lane7 = threadIdx.x + 7;
    const bool active = mx < Ng;
    float2 acc[IB][8];
#pragma unroll
    for (int b = 0; b < IB; ++b)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[b][k] = make_float2(0.f, 0.f);
    const int e0 = threadIdx.x, e1 = threadIdx.x + CB;
    // tile-relative footprint column of a staged point: the wrapped segment
    // (columns Ng-7 .. Ng-1 seen from a tile at column 0) is shifted by -Ng
    auto rel = [&](const BandMeta& m, int idx, float4 gq) {
        return fbits(gq.x) - (idx < m.nA ? Ng : 0) - C0 + 7;
    };
    // a point's geometry, half-pixel phase and values (the phase is applied
    // when the point is staged, so that the loads stay in flight until then)
    auto fetch = [&](const BandMeta& m, int idx, float4& gq, float2& ph, float2 (&h)[IB]) {
        const int sl = band_slot(m, idx);
        gq = d.bpt_geo[sl];
        ph = d.bpt_phase[sl];
#pragma unroll
        for (int b = 0; b < IB; ++b) h[b] = b < nb ? H[b][sl] : make_float2(0.f, 0.f);
    };
    // band_lo <= band_hi always (plan.hip, spread_runs)
    // Pipeline over bands (three LDS slots of CSR rows, slot of band r = (r - band_lo) % 3):
    // in the step of band rb, the CSR row of band rb+2 (fetched in the previous
    // step) is stored, the row of band rb+3 and the points of band rb+1 are
    // fetched, and band rb (points fetched in the previous step) is staged and
    // visited.  Every global load is first waited for one step after it is issued.
    // With one instance (small batches, registers to spare) the points are
    // fetched two bands ahead instead (a second register set holds band rb+1):
    // the band's CSR row is in LDS after the barrier of the step that stores it.
    constexpr bool AHEAD2 = IB == 1;
    auto slot = [&](int r) { return rows + ((r - band_lo) % 3) * (CB + 10); };
    BandMeta nm, qm;
    float4 ng0 = make_float4(0.f, 0.f, 0.f, 0.f), ng1 = ng0, qg0 = ng0, qg1 = ng0;
    float2 np0 = make_float2(0.f, 0.f), np1 = np0, qp0 = np0, qp1 = np0;
    float2 nh0[IB], nh1[IB], qh0[IB], qh1[IB];
#pragma unroll
    for (int b = 0; b < IB; ++b) nh0[b] = nh1[b] = qh0[b] = qh1[b] = make_float2(0.f, 0.f);
    int rv[2] = {0, 0};  // CSR row in flight (band rb + 2 at the top of the step of band rb)
    {
        int v[2];
        band_row_fetch(d, band_lo, C0, CB, v);
        band_row_store(slot(band_lo), CB, v);
        if (band_lo + 1 <= band_hi) {
            band_row_fetch(d, band_lo + 1, C0, CB, v);
            band_row_store(slot(band_lo + 1), CB, v);
        }
        if (band_lo + 2 <= band_hi) band_row_fetch(d, band_lo + 2, C0, CB, rv);
    }
    __syncthreads();
    nm = band_meta(slot(band_lo), Ng, C0, CB, active);
    if (e0 < nm.ntot) fetch(nm, e0, ng0, np0, nh0);
    if (e1 < nm.ntot) fetch(nm, e1, ng1, np1, nh1);
    if (AHEAD2 && band_lo + 1 <= band_hi) {
        qm = band_meta(slot(band_lo + 1), Ng, C0, CB, active);
        if (e0 < qm.ntot) fetch(qm, e0, qg0, qp0, qh0);
        if (e1 < qm.ntot) fetch(qm, e1, qg1, qp1, qh1);
    }
    for (int rb = band_lo; rb <= band_hi; ++rb) {
        // slot of band rb+2 last held band rb-1, whose row was read two steps ago
        if (rb + 2 <= band_hi) band_row_store(slot(rb + 2), CB, rv);
        const BandMeta m = nm;
        const float4 g0 = ng0, g1 = ng1;
        const float2 p0 = np0, p1 = np1;
        float2 h0[IB], h1[IB];
#pragma unroll
        for (int b = 0; b < IB; ++b) { h0[b] = nh0[b]; h1[b] = nh1[b]; }
        // chunk 0 from registers
        if (e0 < m.ntot) spread_stage<IB, CAP>(S, e0, g0, rel(m, e0, g0), h0, p0);
        if (e1 < m.ntot) spread_stage<IB, CAP>(S, e1, g1, rel(m, e1, g1), h1, p1);
        __syncthreads();
        if constexpr (AHEAD2) {
            if (rb + 2 <= band_hi) {  // band rb+2: its CSR row was stored at the top of this step
                nm = band_meta(slot(rb + 2), Ng, C0, CB, active);
                if (e0 < nm.ntot) fetch(nm, e0, ng0, np0, nh0);
                if (e1 < nm.ntot) fetch(nm, e1, ng1, np1, nh1);
            }
        } else if (rb < band_hi) {  // band rb+1: its CSR row was stored one step ago
            nm = band_meta(slot(rb + 1), Ng, C0, CB, active);
            if (e0 < nm.ntot) fetch(nm, e0, ng0, np0, nh0);
            if (e1 < nm.ntot) fetch(nm, e1, ng1, np1, nh1);
        }
        if (rb + 3 <= band_hi) band_row_fetch(d, rb + 3, C0, CB, rv);
        spread_visit<IB, CAP>(S, m.lo, min(m.hi, CAP), 0, lane7, acc);
        __syncthreads();
        // further chunks (dense bands only)
        for (int c0 = CAP; c0 < m.ntot; c0 += CAP) {
            const int cn = min(CAP, m.ntot - c0);
            for (int e = threadIdx.x; e < cn; e += CB) {
                float4 gq;
                float2 ph, hh[IB];
                fetch(m, c0 + e, gq, ph, hh);
                spread_stage<IB, CAP>(S, e, gq, rel(m, c0 + e, gq), hh, ph);
            }
            __syncthreads();
            spread_visit<IB, CAP>(S, max(m.lo, c0), min(m.hi, c0 + cn), c0, lane7, acc);
            __syncthreads();
        }
        // row rb has all of this work row's contributions
        if (active) {
#pragma unroll
            for (int b = 0; b < IB; ++b)
                if (b < nb) Ob[b][(size_t)(rb - band_lo) * Ng + mx] = acc[b][0];
        }
#pragma unroll
        for (int b = 0; b < IB; ++b) {
#pragma unroll
            for (int k = 0; k < 7; ++k) acc[b][k] = acc[b][k + 1];
            acc[b][7] = make_float2(0.f, 0.f);
        }
        if constexpr (AHEAD2) {  // the set of band rb+1 is staged next; band rb+2's waits
            const BandMeta tm = nm;
            nm = qm;
            qm = tm;
            const float4 t0 = ng0, t1 = ng1;
            ng0 = qg0; ng1 = qg1; qg0 = t0; qg1 = t1;
            const float2 u0 = np0, u1 = np1;
            np0 = qp0; np1 = qp1; qp0 = u0; qp1 = u1;
#pragma unroll
            for (int b = 0; b < IB; ++b) {
                const float2 a0 = nh0[b], a1 = nh1[b];
                nh0[b] = qh0[b]; nh1[b] = qh1[b]; qh0[b] = a0; qh1[b] = a1;
            }
        }
    }
    // the 7 rows after the last band: complete after the plan's last band (grid
    // rows NB .. Hy - 1), partial sums for the tail region after a whole row
    // tile's, slab rows after a run's
    const bool own = to_slab || band_hi == NB - 1;
    if (active) {
#pragma unroll
        for (int k = 0; k < 7; ++k) {
#pragma unroll
            for (int b = 0; b < IB; ++b) {
                if (b >= nb) continue;
                if (own) Ob[b][(size_t)(band_hi - band_lo + 1 + k) * Ng + mx] = acc[b][k];
                else ((float2*)(wbs[b] + L.tail))[((size_t)rt * 7 + k) * Ng + mx] = acc[b][k];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// adjoint: the spread of small launches (plans with spr_small), on the matrix
// cores.  A point of band r0 (footprint base row) adds wy[dy] wx[dx] h to the
// 8 x 8 cells at rows r0 + dy and columns bx + dx, so over a band 16 columns
// and the band's 8 rows take the product
//   out[(dy, re/im)][column] = sum_p (wy[p][dy] h[p].re/im) wx[p][column],
// a 16 x 16 output with the points as the contraction (v_mfma_f32_16x16x4f32,
// four points at a time; wx is zero outside a point's footprint).
//
// A workgroup owns a row tile (kSpreadTh bands) x 16 columns, each of its
// kSprWaves waves kSprBands of the bands.  A wave stages up to 64 points at a time
// in LDS, one per lane (16 ES weights, the value times the conjugate half-pixel
// phase), the next points' loads in flight.  Accumulator rows are used
// cyclically (row r in slot r mod 8): a finished row leaves its slot to the row
// eight further on.  At the end the waves' parts are added in wave order in LDS;
// the rows go where the row tile's go in spread_tile (grid and tail region), and
// every sum has a fixed order, the same for every launch shape and batch.
//
// Bound by the latency of a wave's chain (CSR bounds, points, staging, matrix
// instructions): 16 columns x 2 bands per wave give 16 times as many, 8 times
// shorter chains as one lane per column x 8 bands.  For large launches the
// lane-per-column form does less work: a point's 8 columns fill about a third
// of the matrix operand, and float32 matrix and vector instructions share the
// SIMD's issue.  256^2, one image: 12 us against 33; 32^2: 10 against 62; 256^2,
// batch 64: 136 against 108.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Orders a wave's LDS writes before its later reads by other lanes (LDS
// operations of a wave complete in order; this keeps the compiler's order).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

static_assert(kSprBands == 2, "a wave's first row is done after its first band");

template <int IB>
__device__ __forceinline__ void spread_small_tile(const PlanDev& d, const WsLayout& L, char* wb0, size_t stride, int nb,
                                                  int tile, float* lds)
{
    constexpr int NR = kSprBands + 7;  // grid rows a wave's bands reach
    const int Ng = d.Ng, NB = d.NB;
    const int ncg = (Ng + kSprCols - 1) / kSprCols;
    const int rt = tile / ncg, C0 = (tile - rt * ncg) * kSprCols;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16 = lane & 15, kq = lane >> 4;
    float* wls = lds + w * spread_wave_words(IB);
    float* swx = wls;                               // [64][kSprWx]: the 8 x weights, then a zero
    float* swy = swx + 64 * kSprWx;                 // [64][8]
    float* sh = swy + 64 * 8;                       // [64][re, im][IB]
    int* sbx = (int*)(sh + 64 * 2 * IB);            // [64] footprint column, relative to the tile
    const float2* H[IB];
#pragma unroll
    for (int b = 0; b < IB; ++b) H[b] = (const float2*)(wb0 + (size_t)min(b, nb - 1) * stride + L.polar);
    // the bands' points as one list: footprint columns C0 - 7 .. C0 + 15, the
    // wrapped ones (columns Ng - 7 .. Ng - 1 seen from the tile at column 0)
    // first; each band's part is padded to whole groups of four
    int ra[kSprBands], na[kSprBands], rb[kSprBands], n[kSprBands], at[kSprBands + 1];
    at[0] = 0;
#pragma unroll
    for (int q = 0; q < kSprBands; ++q) {
        const int band = rt * kSpreadTh + w * kSprBands + q;
        const bool ok = band < NB;
        const int* bp = d.band_ptr + (size_t)min(band, NB - 1) * (Ng + 1);
        rb[q] = bp[max(C0 - 7, 0)];
        const int n2 = bp[min(C0 + kSprCols, Ng)] - rb[q];
        ra[q] = C0 == 0 ? bp[Ng - 7] : 0;
        na[q] = ok && C0 == 0 ? bp[Ng] - ra[q] : 0;
        n[q] = ok ? na[q] + n2 : 0;
        at[q + 1] = at[q] + ((n[q] + 3) & ~3);
    }
    const int tot = at[kSprBands];
    f32x4 acc[IB];
    float2 done[IB];  // the wave's first row, complete after its first band (lanes kq = 0)
#pragma unroll
    for (int b = 0; b < IB; ++b) {
        acc[b] = (f32x4)(0.f);
        done[b] = make_float2(0.f, 0.f);
    }
    swx[lane * kSprWx + 8] = 0.f;
    // a lane's point: entry e of the list (past a band's points: a zero value)
    float4 gq;
    float2 ph, h[IB];
    int bxr;
    auto fetch = [&](int e) {
        const int q = e >= at[1];
        const int i = e - (q ? at[1] : 0), na_ = q ? na[1] : na[0];
        const bool ok = i < (q ? n[1] : n[0]);
        const int sl = ok ? (i < na_ ? (q ? ra[1] : ra[0]) + i : (q ? rb[1] : rb[0]) + (i - na_)) : 0;
        gq = d.bpt_geo[sl];
        ph = d.bpt_phase[sl];
#pragma unroll
        for (int b = 0; b < IB; ++b) {
            const float2 v = H[b][sl];
            h[b] = ok ? v : make_float2(0.f, 0.f);
        }
        bxr = (i < na_ ? Ng : 0) + C0;
    };
    auto stage = [&]() {
        float wv[8];
        es_weights8(gq.z, wv);
        float4* px = (float4*)(swx + lane * kSprWx);
        px[0] = make_float4(wv[0], wv[1], wv[2], wv[3]);
        px[1] = make_float4(wv[4], wv[5], wv[6], wv[7]);
        es_weights8(gq.w, wv);
        float4* py = (float4*)(swy + lane * 8);
        py[0] = make_float4(wv[0], wv[1], wv[2], wv[3]);
        py[1] = make_float4(wv[4], wv[5], wv[6], wv[7]);
        sbx[lane] = fbits(gq.x) - bxr;
        // explicit roundings: the same product for every IB
#pragma unroll
        for (int b = 0; b < IB; ++b) {
            sh[(lane * 2) * IB + b] = fmaf(h[b].x, ph.x, __fmul_rn(h[b].y, ph.y));
            sh[(lane * 2 + 1) * IB + b] = fmaf(h[b].y, ph.x, -__fmul_rn(h[b].x, ph.y));
        }
    };
    // the staged points p0 .. p1 - 1 (whole groups of four) of a band; dy: the tap of the lane's row
    auto feed = [&](int p0, int p1, int dy) {
        for (int c = p0; c < p1; c += 4) {
            const int p = c + kq;
            const float wx = swx[p * kSprWx + (int)min((unsigned)(n16 - sbx[p]), 8u)], wy = swy[p * 8 + dy];
            const float* hp = sh + (p * 2 + (n16 & 1)) * IB;
#pragma unroll
            for (int b = 0; b < IB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wy * hp[b], wx, acc[b], 0, 0, 0);
        }
    };
    if (tot > 0) fetch(lane);
    bool second = false;
    for (int base = 0; base < tot; base += 64) {
        const int bend = min(base + 64, tot);
        stage();
        wave_lds_fence();
        if (base + 64 < tot) fetch(base + 64 + lane);
        const int mid = min(max(at[1], base), bend);
        feed(0, mid - base, n16 >> 1);
        if (!second && at[1] <= bend) {
            second = true;
#pragma unroll
            for (int b = 0; b < IB; ++b) {
                done[b] = make_float2(acc[b][0], acc[b][1]);
                if (kq == 0) acc[b][0] = acc[b][1] = 0.f;
            }
        }
        feed(mid - base, bend - base, ((n16 >> 1) - 1) & 7);
        wave_lds_fence();
    }
    // the wave's rows to LDS [IB][NR][16] (its staging area is free), then their sum over the waves
    float2* ob = (float2*)wls;
#pragma unroll
    for (int b = 0; b < IB; ++b) {
        if (kq == 0) ob[b * NR * kSprCols + n16] = done[b];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int slot = 2 * kq + r;  // slot 0 holds row 8
            ob[(b * NR + (slot ? slot : 8)) * kSprCols + n16] = make_float2(acc[b][2 * r], acc[b][2 * r + 1]);
        }
    }
    __syncthreads();
    constexpr int ROWS = kSpreadTh + 7;
    const bool last = (rt + 1) * kSpreadTh >= NB;
    for (int t = threadIdx.x; t < nb * ROWS * kSprCols; t += kSprWaves * 64) {
        const int b = t / (ROWS * kSprCols), e = t - b * (ROWS * kSprCols), row = e / kSprCols, col = e % kSprCols;
        float2 sum = make_float2(0.f, 0.f);
#pragma unroll
        for (int v = 0; v < kSprWaves; ++v) {
            const int r = row - v * kSprBands;
            const float2* src = (const float2*)(lds + v * spread_wave_words(IB));
            const float2 x = src[(b * NR + min(max(r, 0), NR - 1)) * kSprCols + col];
            if (r >= 0 && r < NR) sum = cadd(sum, x);
        }
        const int gr = rt * kSpreadTh + row;
        if (C0 + col >= Ng) continue;
        char* wb = wb0 + (size_t)b * stride;
        if (row < kSpreadTh || last) {
            if (gr < d.Hy) ((float2*)(wb + L.grid))[(size_t)gr * Ng + C0 + col] = sum;
        } else {
            ((float2*)(wb + L.tail))[((size_t)rt * 7 + row - kSpreadTh) * Ng + C0 + col] = sum;
        }
    }
}

template <int IB, int CB>
__global__ __launch_bounds__(kGatherThreads) void k_gather(PlanDev d, WsLayout L, InstPtrs wsp, int TH, int batch)
{
    extern __shared__ float2 win[];
    const int per = ((d.Ng + CB - 1) / CB) * ((d.NB + TH - 1) / TH);
    const int ngroups = (batch + IB - 1) / IB;
    const int item = xcd_item(blockIdx.x, per * ngroups);
    if (item < 0) return;
    const int g = item / per;
    const int b0 = g * IB, nb = min(IB, batch - b0);
    char* wbs[IB];
#pragma unroll
    for (int b = 0; b < IB; ++b) wbs[b] = wsp.ws + (size_t)(b0 + (b < nb ? b : 0)) * wsp.stride;
    gather_tile<IB, CB>(d, L, wbs, nb, item - g * per, TH, win);
}

// CB is the batch-wide tile width (the instance table carries TH).
template <int CB>
__global__ __launch_bounds__(kGatherThreads) void k_gather_b(BatchDev bt, char* ws)
{
    extern __shared__ float2 win[];
    int i, tile;
    if (!batch_item(bt, kStGather, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    char* const wbs[1] = {ws + I.ws_off};
    gather_tile<1, CB>(d, I.L, wbs, 1, tile, I.gat_th, win);
}

// Dense synthesis (explicit detector angles): `ntile` tiles per instance,
// instance-major and XCD-contiguous, so one instance's mode coefficients stay
// in one XCD's L2 while all its tiles read them; the _b forms take their
// instance and tile from the batch tables.
__global__ __launch_bounds__(kSynThreads) void k_syn_dense_fwd(PlanDev d, WsLayout L, InstPtrs wsp, int ntile,
                                                               int batch)
{
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    syn_dense_fwd_tile(d, L, wsp.ws + (size_t)b * wsp.stride, item - b * ntile);
}

__global__ __launch_bounds__(kSynThreads) void k_syn_dense_adj(PlanDev d, WsLayout L, InstPtrs wsp, int ntile,
                                                               int batch)
{
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    syn_dense_adj_tile(d, L, wsp.ws + (size_t)b * wsp.stride, item - b * ntile);
}

__global__ __launch_bounds__(kSynThreads) void k_syn_dense_fwd_b(BatchDev bt, char* ws)
{
    int i, tile;
    if (!batch_item(bt, kStSynFwd, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    syn_dense_fwd_tile(d, I.L, ws + I.ws_off, tile);
}

__global__ __launch_bounds__(kSynThreads) void k_syn_dense_adj_b(BatchDev bt, char* ws)
{
    int i, tile;
    if (!batch_item(bt, kStSynAdj, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    syn_dense_adj_tile(d, I.L, ws + I.ws_off, tile);
}

__global__ __launch_bounds__(1024) void k_dct_det(PlanDev d, WsLayout L, InstPtrs wsp, float* __restrict__ gout,
                                                  const float* __restrict__ gin, int DP, int adj, int n_mass, int batch)
{
    extern __shared__ float2 sm[];
    __shared__ float red_s[1024];
    __shared__ float mass_s;
    const int ntile = ((d.D + 1) / 2 + DP - 1) / DP;
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    const size_t go = (size_t)b * d.D * d.T;
    dct_tile(d, L, wsp.ws + (size_t)b * wsp.stride, adj ? nullptr : gout + go, adj ? gin + go : nullptr,
             item - b * ntile, DP, adj, n_mass, sm, red_s, &mass_s);
}

template <int N2>
__global__ __launch_bounds__(1024) void k_dct_spec(PlanDev d, WsLayout L, InstPtrs wsp, float* __restrict__ gout,
                                                   const float* __restrict__ gin, int DP, int adj, int n_mass, int batch)
{
    extern __shared__ float2 sm[];
    __shared__ float red_s[32];  // two per wave
    __shared__ float mass_s;
    const int ntile = ((d.D + 1) / 2 + DP - 1) / DP;
    const int item = xcd_item(blockIdx.x, ntile * batch);
    if (item < 0) return;
    const int b = item / ntile;
    const size_t go = (size_t)b * d.D * d.T;
    dct_spec_tile<N2>(d, L, wsp.ws + (size_t)b * wsp.stride, adj ? nullptr : gout + go, adj ? gin + go : nullptr,
                      item - b * ntile, DP, adj, n_mass, sm, red_s, &mass_s);
}

// adj = 0: out[i] receives the data of instance i; adj = 1: in[i] is read.
__global__ __launch_bounds__(1024) void k_dct_det_b(BatchDev bt, char* ws, float* const* __restrict__ out,
                                                    const float* const* __restrict__ in, int adj)
{
    extern __shared__ float2 sm[];
    __shared__ float red_s[1024];
    __shared__ float mass_s;
    int i, tile;
    if (!batch_item(bt, kStDct, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    if (d.dct_spec)
        dct_run(d, I.L, ws + I.ws_off, adj ? nullptr : out[i], adj ? in[i] : nullptr, tile, I.dct_dp, adj, d.N, sm,
                red_s, &mass_s);
    else
        dct_tile(d, I.L, ws + I.ws_off, adj ? nullptr : out[i], adj ? in[i] : nullptr, tile, I.dct_dp, adj, d.N, sm,
                 red_s, &mass_s);
}

// IB instances per workgroup: instances g*IB .. g*IB + IB - 1 of the batch; CB threads.
// At IB = 4 the register budget is held to three waves per SIMD (168 VGPRs;
// the kernel needs 170 unconstrained).
template <int IB, int CB>
__global__ __launch_bounds__(CB) __attribute__((amdgpu_waves_per_eu(IB == 4 ? 3 : 1))) void k_spread(PlanDev d, WsLayout L, InstPtrs wsp, int batch)
{
    extern __shared__ float sf[];
    const int per = ((d.Ng + CB - 1) / CB) * d.spr_rows;
    const int ngroups = (batch + IB - 1) / IB;
    const int item = xcd_item(blockIdx.x, per * ngroups);
    if (item < 0) return;
    const int g = item / per;
    const int b0 = g * IB, nb = min(IB, batch - b0);
    char* wbs[IB];
#pragma unroll
    for (int b = 0; b < IB; ++b) wbs[b] = wsp.ws + (size_t)(b0 + (b < nb ? b : 0)) * wsp.stride;
    spread_tile<IB, CB>(d, L, wbs, nb, item - g * per, sf);
}

template <int IB>
__global__ __launch_bounds__(kSprWaves * 64) void k_spread_small(PlanDev d, WsLayout L, InstPtrs wsp, int batch)
{
    extern __shared__ __align__(16) float sfs[];
    const int per = spread_small_tiles(d.Ng, d.NB);
    const int ngroups = (batch + IB - 1) / IB;
    const int item = xcd_item(blockIdx.x, per * ngroups);
    if (item < 0) return;
    const int g = item / per;
    const int b0 = g * IB, nb = min(IB, batch - b0);
    spread_small_tile<IB>(d, L, wsp.ws + (size_t)b0 * wsp.stride, wsp.stride, nb, item - g * per, sfs);
}

__global__ __launch_bounds__(kSprWaves * 64) void k_spread_small_b(BatchDev bt, char* ws)
{
    extern __shared__ __align__(16) float sfs[];
    int i, tile;
    if (!batch_item(bt, kStSpreadSmall, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    spread_small_tile<1>(d, I.L, ws + I.ws_off, 0, 1, tile, sfs);
}

template <int CB>
__global__ __launch_bounds__(CB) void k_spread_b(BatchDev bt, char* ws)
{
    extern __shared__ float sf[];
    int i, tile;
    if (!batch_item(bt, kStSpread, i, tile)) return;
    const BatchInst& I = bt.inst[i];
    const PlanDev d = I.d;
    char* const wbs[1] = {ws + I.ws_off};
    spread_tile<1, CB>(d, I.L, wbs, 1, tile, sf);
}

// ---------------------------------------------------------------------------
// total variation (smoothed, isotropic, forward differences, Neumann boundary)
// ---------------------------------------------------------------------------
// A wave takes 62 columns (and one beside them on either side) and ROWS rows: its
// loads come first, neighbours' values and quotients from the lanes beside and the
// row above, so that a pixel's root and divisions are done 1 + 1 / ROWS times (three
// times with a pixel per lane).  Large launches are bound by them: four rows; small
// ones by the chain of one wave: one row.  us at 1 / 2 / 4 rows (a pixel per lane):
// 256^2 2.4 / 2.6 / 3.0 (2.6), batch 4 3.1 / 3.1 / 3.4 (3.1), batch 8 4.1 / 3.8 / 4.0
// (4.1), batch 16 6.2 / 5.5 / 5.3 (6.0); 1024^2 batch 8 29 / 23 / 21 (40).
constexpr int kTvCols = 62;
__host__ __device__ constexpr int tv_grad_rows(long pixels) { return pixels < 1L << 18 ? 1 : pixels < 1L << 20 ? 2 : 4; }
template <int ROWS>
__global__ __launch_bounds__(256) void k_tv_grad(const float* __restrict__ f, float* __restrict__ grad, int n,
                                                 float eps2)
{
    const int b = blockIdx.z, lane = threadIdx.x & 63;
    const int j = blockIdx.x * kTvCols + lane - 1;
    const int i0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * ROWS;
    if (i0 >= n) return;
    const float* fb = f + (size_t)b * n * n;
    float* gb = grad + (size_t)b * n * n;
    const int jc = min(max(j, 0), n - 1);
    float c[ROWS + 2];  // rows i0 - 1 .. i0 + ROWS
#pragma unroll
    for (int r = 0; r < ROWS + 2; ++r) c[r] = fb[(size_t)min(max(i0 - 1 + r, 0), n - 1) * n + jc];
    const bool out = lane > 0 && lane <= kTvCols && j < n;
    float up = 0.f;  // dy / s of the row above
#pragma unroll
    for (int r = 0; r <= ROWS; ++r) {
        const int i = i0 - 1 + r;
        const float right = __shfl_down(c[r], 1, 64);
        const float dx = j + 1 < n ? right - c[r] : 0.f;
        const float dy = i + 1 < n ? c[r + 1] - c[r] : 0.f;
        const float s = sqrtf(dx * dx + dy * dy + eps2);
        if (r > 0) {
            const float left = __shfl_up(dx / s, 1, 64);
            float gval = -(dx + dy) / s;
            if (j > 0) gval += left;
            if (i > 0) gval += up;
            if (out && i < n) gb[(size_t)i * n + j] = gval;
        }
        up = dy / s;
    }
}

// One workgroup per image: a wave takes RW rows and CW groups of 64 columns at a
// time, so that the latency of its loads, which bounds it, is paid once for them:
// four rows and 128 columns; images of up to 64 columns two rows and 64, which
// leaves fewer waves and lanes idle (32^2 2.9 us, 2.9 in four rows with half the
// lanes; 64^2 3.5 / 3.8; 200^2 13 us, 20 with a pixel per lane and a division each).
template <int RW, int CW>
__global__ __launch_bounds__(1024) void k_tv_value(const float* __restrict__ f, float* __restrict__ tv, int n,
                                                   float eps2)
{
    __shared__ float red_s[1024];
    const int b = blockIdx.x;
    const float* fb = f + (size_t)b * n * n;
    const int lane = threadIdx.x & 63;
    const int nx = (n + 64 * CW - 1) / (64 * CW), items = nx * ((n + RW - 1) / RW);
    float acc = 0.f;
    for (int it = threadIdx.x >> 6; it < items; it += 16) {
        const int q = it / nx, i = RW * q, j0 = (it - q * nx) * (64 * CW) + lane;
        float c[RW + 1][CW], r[RW][CW];
#pragma unroll
        for (int u = 0; u <= RW; ++u) {
            const float* row = fb + (size_t)min(i + u, n - 1) * n;
#pragma unroll
            for (int v = 0; v < CW; ++v) {
                const int j = j0 + 64 * v;
                c[u][v] = row[min(j, n - 1)];
                if (u < RW) r[u][v] = row[min(j + 1, n - 1)];
            }
        }
#pragma unroll
        for (int u = 0; u < RW; ++u)
#pragma unroll
            for (int v = 0; v < CW; ++v) {
                const float dx = j0 + 64 * v + 1 < n ? r[u][v] - c[u][v] : 0.f;
                const float dy = i + u + 1 < n ? c[u + 1][v] - c[u][v] : 0.f;
                const float m = sqrtf(dx * dx + dy * dy + eps2);
                acc += j0 + 64 * v < n && i + u < n ? m : 0.f;
            }
    }
    const float tot = block_sum(acc, red_s);
    if (threadIdx.x == 0) tv[b] = tot;
}

__global__ __launch_bounds__(256) void k_pgd_update(float* __restrict__ f, const float* __restrict__ adj,
                                                    const float* __restrict__ tvg, long count, float tau,
                                                    float lam)
{
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < count; e += (long)gridDim.x * blockDim.x) {
        float gr = adj[e];
        if (tvg) gr += lam * tvg[e];
        const float v = f[e] - tau * gr;
        f[e] = v > 0.f ? v : 0.f;
    }
}

__global__ __launch_bounds__(256) void k_residual(float* __restrict__ g, const float* __restrict__ gm, long count)
{
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < count; e += (long)gridDim.x * blockDim.x)
        g[e] = g[e] - gm[e];
}

__global__ __launch_bounds__(1024) void k_half_sq(const float* __restrict__ g, float* __restrict__ sq, long per)
{
    __shared__ float red_s[1024];
    const int b = blockIdx.x;
    const float* gb = g + (size_t)b * per;
    const float tot = block_sum(strided_sum(per, [&](long e) { return gb[e] * gb[e]; }), red_s);
    if (threadIdx.x == 0) sq[b] = 0.5f * tot;
}

// ---------------------------------------------------------------------------
// primal-dual TV iteration (the paper's TV baseline): dual steps for the data
// term and the isotropic TV term, primal step with the f >= 0 projection and
// the extrapolation fbar = 2 f' - f, and the relative-change norms
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pd_dual_data(float* __restrict__ y1, const float* __restrict__ ax,
                                                      const float* __restrict__ g, long count, float sigma,
                                                      float inv1s)
{
    for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < count; e += (long)gridDim.x * blockDim.x)
        y1[e] = (y1[e] + sigma * (ax[e] - g[e])) * inv1s;
}

// Columns of a workgroup's tile (256 / W rows of W) in the two kernels below.  Rows of
// 64 are whole cache lines of every array: the primal step's choice for images wider
// than a tile of 16 (us, rows of 64 / 16: 16^2 2.28 / 2.13, 32^2 2.31 / 2.45, 256^2
// batch 8 3.6 / 4.6).  The dual step reads one row below its own: tiles of 16 rows keep
// it in L1 where images are wide, launches small and rows start on 64-byte lines (256^2
// batch 8 3.5 / 3.4, 512^2 2.86 / 2.75, batch 4 4.9 / 4.8, but batch 8 7.3 / 11.0; 64^2
// 2.24 / 2.32, 300^2 batch 2 3.4 / 3.6).
__host__ inline int pd_primal_cols(int n) { return n <= 16 ? 16 : 64; }
__host__ inline int pd_dual_cols(int n, int batch)
{
    return n <= 16 || (n >= 256 && n % 16 == 0 && (long)n * n * batch <= 1L << 20) ? 16 : 64;
}

// y2 [batch][n][n] float2 (x and y components), xbar [batch][n][n]
template <int W>
__global__ __launch_bounds__(256) void k_pd_dual_tv(float2* __restrict__ y2, const float* __restrict__ xbar, int n,
                                                    float sigma, float alpha)
{
    const int b = blockIdx.z;
    const int j = blockIdx.x * W + threadIdx.x % W;
    const int i = blockIdx.y * (256 / W) + threadIdx.x / W;
    if (i >= n || j >= n) return;
    const float* xb = xbar + (size_t)b * n * n;
    const size_t e = (size_t)b * n * n + (size_t)i * n + j;
    const float c = xb[(size_t)i * n + j];
    const float dx = (j + 1 < n) ? xb[(size_t)i * n + j + 1] - c : 0.f;
    const float dy = (i + 1 < n) ? xb[(size_t)(i + 1) * n + j] - c : 0.f;
    float2 v = y2[e];
    v.x += sigma * dx;
    v.y += sigma * dy;
    const float m = sqrtf(v.x * v.x + v.y * v.y);
    const float sc = m > alpha ? alpha / m : 1.f;  // projection onto |v| <= alpha
    y2[e] = make_float2(v.x * sc, v.y * sc);
}

// f' = max(f - tau (aty + grad* y2), 0); xbar = 2 f' - f; f = f'
template <int W>
__global__ __launch_bounds__(256) void k_pd_primal(float* __restrict__ f, float* __restrict__ xbar,
                                                   const float* __restrict__ aty, const float2* __restrict__ y2,
                                                   int n, float tau)
{
    const int b = blockIdx.z;
    const int j = blockIdx.x * W + threadIdx.x % W;
    const int i = blockIdx.y * (256 / W) + threadIdx.x / W;
    if (i >= n || j >= n) return;
    const size_t base = (size_t)b * n * n;
    const size_t e = base + (size_t)i * n + j;
    // (grad* y2)_ij: the x component enters at (i, j) with -1 (j < n-1) and at (i, j+1) with +1,
    // the y component at (i, j) with -1 (i < n-1) and at (i+1, j) with +1
    const float2 p = y2[e];
    float gs = 0.f;
    if (j + 1 < n) gs -= p.x;
    if (j > 0) gs += y2[e - 1].x;
    if (i + 1 < n) gs -= p.y;
    if (i > 0) gs += y2[e - n].y;
    const float old = f[e];
    const float fn = fmaxf(old - tau * (aty[e] + gs), 0.f);
    f[e] = fn;
    xbar[e] = 2.f * fn - old;
}

// out[b] = (sum (xbar - f)^2, sum f^2) over instance b (after k_pd_primal,
// xbar - f = f' - f_old): one workgroup per instance, fixed-order sums
__global__ __launch_bounds__(1024) void k_pd_change(const float* __restrict__ f, const float* __restrict__ xbar,
                                                    float* __restrict__ out, long per)
{
    __shared__ float red_s[1024];
    const int b = blockIdx.x;
    const float* fb = f + (size_t)b * per;
    const float* xb = xbar + (size_t)b * per;
    // both sums in one sweep: 64^2 3.7 us, 200^2 6.3, 1024^2 85 (4.1, 8.3 and 126 with a sweep each)
    const float2 acc = strided_sum(per, [&](long e) {
        const float v = fb[e], dlt = xb[e] - v;
        return make_float2(dlt * dlt, v * v);
    });
    const float td = block_sum(acc.x, red_s);
    const float tf = block_sum(acc.y, red_s);
    if (threadIdx.x == 0) {
        out[2 * b] = td;
        out[2 * b + 1] = tf;
    }
}


// ---------------------------------------------------------------------------
// CGLS pieces (one workgroup per instance for the norms: fixed-order sums)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_cg_norm2(const float* __restrict__ x, float* __restrict__ out, long per)
{
    __shared__ float red_s[1024];
    const int b = blockIdx.x;
    const float* xb = x + (size_t)b * per;
    const float t = block_sum(strided_sum(per, [&](long e) { return xb[e] * xb[e]; }), red_s);
    if (threadIdx.x == 0) out[b] = t;
}

__global__ void k_cg_step_fr(float* __restrict__ f, const float* __restrict__ p, long nf, float* __restrict__ r,
                             const float* __restrict__ q, long nr, const float* __restrict__ gamma,
                             const float* __restrict__ qq)
{
    const int b = blockIdx.y;
    const float den = qq[b];
    const float alpha = den > 0.f ? gamma[b] / den : 0.f;
    const long stride = (long)gridDim.x * blockDim.x;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < nf; e += stride)
        f[(size_t)b * nf + e] += alpha * p[(size_t)b * nf + e];
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < nr; e += stride)
        r[(size_t)b * nr + e] -= alpha * q[(size_t)b * nr + e];
}

__global__ void k_cg_step_p(float* __restrict__ p, const float* __restrict__ s, long n,
                            const float* __restrict__ gamma_new, const float* __restrict__ gamma)
{
    const int b = blockIdx.y;
    const float den = gamma[b];
    const float beta = den > 0.f ? gamma_new[b] / den : 0.f;
    const long stride = (long)gridDim.x * blockDim.x;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride)
        p[(size_t)b * n + e] = s[(size_t)b * n + e] + beta * p[(size_t)b * n + e];
}


// ---------------------------------------------------------------------------
// Streaming copies: the bandwidth yardstick the roofline figures are quoted
// against, and the known-size traffic that calibrates the byte counters.
// k_stream_copy: dst = src over n4 16-byte elements, four loads in flight per
// thread before its stores.  k_scatter_copy: dst[perm[i]] = src[i] over
// 8-byte elements (the scattered-store pattern of the ring adjoint's
// band-order output).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_stream_copy(const float4* __restrict__ src, float4* __restrict__ dst,
                                                     long n4)
{
    const long stride = (long)gridDim.x * 1024;
    for (long base = (long)blockIdx.x * 1024 + threadIdx.x; base < n4; base += stride) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long e = base + u * 256;
            v[u] = src[e < n4 ? e : n4 - 1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long e = base + u * 256;
            if (e < n4) dst[e] = v[u];
        }
    }
}

__global__ __launch_bounds__(256) void k_scatter_copy(const float2* __restrict__ src, float2* __restrict__ dst,
                                                      const int* __restrict__ perm, long n)
{
    const long stride = (long)gridDim.x * 256;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += stride) dst[perm[e]] = src[e];
}

}  // namespace pat
