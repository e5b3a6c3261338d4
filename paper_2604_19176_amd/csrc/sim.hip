// sim.hip -- FFT wave-propagation data simulator (gfx950 kernels and host plan).
//
// The simulation study (Sec. 2.4.1) computes its data on a finer Cartesian grid
// with an FFT-based wave propagation method.  For a constant speed of sound the
// field is p(t) = IFFT2[F cos(c|k|t)], F = FFT2 of the zero-padded fine image on
// a periodic box wide enough that no wave wraps around to a detector by the
// last sample (box rule and sampling in pat.h).
//
// Per run: F is computed once (the image rows, then every column of the box;
// rows outside the image are zero).  The data then come in pairs of time
// samples (t_a, t_b): both fields are real, so one complex inverse transform of
// F (cos(c|k|t_a) + i cos(c|k|t_b)) gives p(t_a) + i p(t_b).  Per chunk of
// pairs: the inverse transform along y with the spectrum modulated as it is
// loaded (the phase c|k|t / 2 pi reduced mod 1 in FP64, then cos(2 pi x) in
// FP32), keeping only the box rows the detectors' stencils read; the inverse
// transform along x of those rows; the Keys samples at the detectors.
#include "../../include/pat.h"
#include "cfft.hpp"
#include "device_util.hpp"
#include "fft.hpp"
#include "pat_internal.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

namespace pat {

struct SimDev {
    int Ns, M, off;         // fine grid side, box side, box index of the image's first row / column
    int D, T;               // detectors, time samples
    int rlo, nrow;          // box rows [rlo, rlo + nrow) read by the detectors' stencils
    int CT, RPB;            // columns per column-transform workgroup, rows per row-transform workgroup
    float a_hi, a_lo;       // alpha = c dt / (M h) as an unevaluated FP32 sum (FP64 on the host): the
                            // phase c |k| j dt / (2 pi) = j alpha sqrt(mx^2 + my^2)
    const int2* mask_rows;  // [Ns]: image row i keeps columns jlo <= j < jhi (support disc)
    const int2* dix;        // [D]: box cell (x, y) of each detector's stencil sample at offset 0
    const float2* dfr;      // [D]: its fractional offsets (FP64-computed)
    const float2* tw;       // twiddle table of the length-M transform
    FftDev fm;              // the length-M transform
};

// Compile-time box sides (cfft.hpp): only the box rows some stencil reads are kept.
// Apart from SimDev, whose further 40 bytes of kernel arguments cost the run-time
// forms of a 64^2 box 4 % (207 against 199 us at 512 samples).
struct SimSpecDev {
    int nkeep;              // their number
    const int* keep;        // [M]: index of a box row among them, or -1
    const int* ent_ptr;     // [nkeep + 1]: the stencil rows that lie in each kept row
    const int2* ent;        // (detector, stencil row 0 .. 3)
    const float2* ctw;      // the length-M transform's table
};

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// FFT along x of RPB image rows (masked, zero-padded into box columns) -> W [Ns][M]
__global__ __launch_bounds__(1024) void k_sim_rows_fwd(SimDev s, const float* __restrict__ f, float2* __restrict__ W)
{
    extern __shared__ float2 sm[];
    const int M = s.M, Ns = s.Ns, RPB = s.RPB;
    const int r0 = blockIdx.x * RPB, nr = min(RPB, Ns - r0);
    const float2* tb = fft_twiddles_to_lds(sm + RPB * M, s.fm, s.tw);
    for (int e = threadIdx.x; e < RPB * M; e += blockDim.x) sm[e] = make_float2(0.f, 0.f);
    __syncthreads();
    for (int e = threadIdx.x; e < nr * Ns; e += blockDim.x) {
        const int rr = e / Ns, j = e - rr * Ns, i = r0 + rr;
        const int2 mr = s.mask_rows[i];
        const float v = (j >= mr.x && j < mr.y) ? f[(size_t)i * Ns + j] : 0.f;
        sm[rr * M + s.off + j] = make_float2(v, 0.f);
    }
    __syncthreads();
    fft_lds<false>(sm, M, RPB, s.fm, tb);
    for (int e = threadIdx.x; e < nr * M; e += blockDim.x) W[(size_t)r0 * M + e] = sm[e];
}

// FFT along y of CT box columns (rows outside the image are zero) -> F [M][M]
__global__ __launch_bounds__(1024) void k_sim_cols_fwd(SimDev s, const float2* __restrict__ W, float2* __restrict__ F)
{
    extern __shared__ float2 sm[];
    const int M = s.M, CT = s.CT;
    const int c0 = blockIdx.x * CT, nc = min(CT, M - c0);
    const float2* tb = fft_twiddles_to_lds(sm + CT * M, s.fm, s.tw);
    for (int e = threadIdx.x; e < M * CT; e += blockDim.x) {
        const int r = e / CT, cc = e - r * CT;
        const int ri = r - s.off;
        float2 v = make_float2(0.f, 0.f);
        if (cc < nc && ri >= 0 && ri < s.Ns) v = W[(size_t)ri * M + c0 + cc];
        sm[cc * M + r] = v;
    }
    __syncthreads();
    fft_lds<false>(sm, M, CT, s.fm, tb);
    for (int e = threadIdx.x; e < M * CT; e += blockDim.x) {
        const int r = e / CT, cc = e - r * CT;
        if (cc < nc) F[(size_t)r * M + c0 + cc] = sm[cc * M + r];
    }
}

// The phase j alpha sqrt(mx^2 + my^2) reduced mod 1, in FP32 arithmetic with
// error-free products (each quantity an unevaluated sum of two floats, as in
// double-float arithmetic): q = mx^2 + my^2 is exact (q_hi + q_lo), the
// square root is refined by one Newton step on its exact FMA residual, and
// the products alpha s and j u are split exactly by FMA, so the fraction
// returned is correct to about 2^-24 (a few cycles of phase would otherwise
// lose their fraction's accuracy in FP32).
__device__ __forceinline__ float sim_phase_frac(int mx, int my, int j, float a_hi, float a_lo)
{
    const unsigned q = (unsigned)(mx * mx + my * my);
    const float q_hi = (float)q;
    const float q_lo = (float)(int)(q - (unsigned)q_hi);  // exact: |q - q_hi| < 2^3 for q < 2^27
    const float s = sqrtf(q_hi);
    const float e = fmaf(-s, s, q_hi) + q_lo;             // q - s^2
    const float sc = q == 0u ? 0.f : e * __builtin_amdgcn_rcpf(2.f * s);
    // u = alpha (s + sc) = u_hi + u_lo
    const float p = a_hi * s;
    const float pe = fmaf(a_hi, s, -p);
    const float t = pe + fmaf(a_hi, sc, a_lo * s);
    const float u_hi = p + t;
    const float u_lo = t - (u_hi - p);
    // x = j u = P + L
    const float J = (float)j;
    const float P = J * u_hi;
    const float L = fmaf(J, u_hi, -P) + J * u_lo;
    float x = (P - floorf(P)) + L;
    x -= floorf(x);
    return x;
}

// Pair p of the chunk (time indices ja = 2 (pair0 + p) + 1, jb = ja + 1): the
// inverse FFT along y of CT columns of F (cos(c|k|t_a) + i cos(c|k|t_b)),
// rows [rlo, rlo + nrow) -> Wt [chunk][nrow][M]
__global__ __launch_bounds__(1024) void k_sim_cols_inv(SimDev s, const float2* __restrict__ F, float2* __restrict__ Wt,
                                                       int pair0)
{
    extern __shared__ float2 sm[];
    const int M = s.M, CT = s.CT, p = blockIdx.y;
    const int c0 = blockIdx.x * CT, nc = min(CT, M - c0);
    const int ja = 2 * (pair0 + p) + 1, jb = ja + 1;
    const bool has_b = jb <= s.T;
    const float2* tb = fft_twiddles_to_lds(sm + CT * M, s.fm, s.tw);
    for (int e = threadIdx.x; e < M * CT; e += blockDim.x) {
        const int r = e / CT, cc = e - r * CT, c = c0 + min(cc, nc - 1);
        const float2 z = F[(size_t)r * M + c];
        const int mx = c < M / 2 ? c : c - M, my = r < M / 2 ? r : r - M;
        const float xa = sim_phase_frac(mx, my, ja, s.a_hi, s.a_lo);
        const float xb = sim_phase_frac(mx, my, jb, s.a_hi, s.a_lo);
        const float ca = cospif(2.0f * xa), cb = has_b ? cospif(2.0f * xb) : 0.f;
        sm[cc * M + r] = make_float2(z.x * ca - z.y * cb, z.y * ca + z.x * cb);
    }
    __syncthreads();
    fft_lds<true>(sm, M, CT, s.fm, tb);
    float2* out = Wt + (size_t)p * s.nrow * M;
    for (int e = threadIdx.x; e < s.nrow * CT; e += blockDim.x) {
        const int rr = e / CT, cc = e - rr * CT;
        if (cc < nc) out[(size_t)rr * M + c0 + cc] = sm[cc * M + s.rlo + rr];
    }
}

// inverse FFT along x of RPB rows of pair p's band, in place
__global__ __launch_bounds__(1024) void k_sim_rows_inv(SimDev s, float2* __restrict__ Wt)
{
    extern __shared__ float2 sm[];
    const int M = s.M, RPB = s.RPB, p = blockIdx.y;
    const int r0 = blockIdx.x * RPB, nr = min(RPB, s.nrow - r0);
    float2* base = Wt + ((size_t)p * s.nrow + r0) * M;
    const float2* tb = fft_twiddles_to_lds(sm + RPB * M, s.fm, s.tw);
    for (int e = threadIdx.x; e < RPB * M; e += blockDim.x) sm[e] = e < nr * M ? base[e] : make_float2(0.f, 0.f);
    __syncthreads();
    fft_lds<true>(sm, M, RPB, s.fm, tb);
    for (int e = threadIdx.x; e < nr * M; e += blockDim.x) base[e] = sm[e];
}

// ---------------------------------------------------------------------------
// Compile-time box sides M (the even 2^a 3^b of 216 .. 2048).  Bound by VALU work per
// box cell and pair of samples (the phase, its cosine, the transform); at a 1152^2
// box, per 16 pairs, the run-time forms below take 149 us (columns) and 52 us
// (rows), these 95 and 41; the arithmetic alone would take half of the 95:
//   - rows r and M - r of a column share |k| and so the cosines, which are computed
//     once and handed over in LDS;
//   - cos(2 pi x) = sin(2 pi (|x - 1/2| - 1/4)) by one odd polynomial;
//   - memory goes straight into the first pass and out of the last one;
//   - only the rows some stencil reads leave the column transforms, and the row
//     transforms keep just their samples (x weights applied), not the rows.
// Smaller boxes take the run-time forms: with 16 values per lane a box column is
// 3 to 12 lanes, so a launch is few waves with long chains, where the run-time
// forms spread it over 32 lanes a column.  Whole calls, run-time / compile-time in us,
// at 64, 128 and 512 samples (16, 64, 256 detectors): side 64 34 / 41, 57 / 73, 199 / 277;
// 144 47 / 51, 82 / 90, 283 / 327; 192 51 / 51, 89 / 91, 310 / 329; 216 55 / 53, 97 / 94,
// 335 / 337; 256 56 / 51, 100 / 92, 351 / 328; 432 95 / 66, 173 / 125, 639 / 501.
// Sequences of kSimNP neighbouring columns (or rows) are interleaved over the
// workgroup's threads, sim_lanes(M) lanes each (16 values per lane and pass).
// ---------------------------------------------------------------------------
constexpr int kSimNP = 8;
__host__ __device__ constexpr int sim_lanes(int m) { return (m + 15) / 16; }
constexpr int sim_threads(int m) { return (kSimNP * sim_lanes(m) + 63) / 64 * 64; }
#define PAT_SIM_LENGTHS(X) \
    X(216) X(256) X(288) X(324) X(384) X(432) X(486) X(512) X(576) X(648) X(768) X(864) X(972) X(1024) PAT_GRID_LENGTHS_HI(X)
constexpr bool sim_len_ok(int m)
{
#define PAT_CASE(LEN) if (m == LEN) return true;
    PAT_SIM_LENGTHS(PAT_CASE)
#undef PAT_CASE
    return false;
}

// alpha sqrt(q) as u_hi + u_lo for q = mx^2 + my^2 (exact in two floats); see sim_phase_frac
__device__ __forceinline__ float2 sim_phase_rate(int mx, int my, float a_hi, float a_lo)
{
    const unsigned q = (unsigned)(mx * mx + my * my);
    const float q_hi = (float)q;
    const float q_lo = (float)(int)(q - (unsigned)q_hi);
    const float s = __builtin_amdgcn_sqrtf(q_hi);
    const float e = fmaf(-s, s, q_hi) + q_lo;
    const float sc = q == 0u ? 0.f : e * __builtin_amdgcn_rcpf(2.f * s);
    const float p = a_hi * s;
    const float t = fmaf(a_hi, s, -p) + fmaf(a_hi, sc, a_lo * s);
    const float u_hi = p + t;
    return make_float2(u_hi, t - (u_hi - p));
}

// cos(2 pi j (u_hi + u_lo)): the product split exactly, its fraction, and the
// Taylor polynomial of sin(2 pi u) on |u| <= 1/4 (degree 13: 7e-10)
__device__ __forceinline__ float sim_cos(float J, float2 u)
{
    const float P = J * u.x;
    const float L = fmaf(J, u.x, -P) + J * u.y;
    const float x = __builtin_amdgcn_fractf(__builtin_amdgcn_fractf(P) + L);
    const float v = fabsf(x - 0.5f) - 0.25f, w = v * v;
    constexpr double t = 6.283185307179586476925;
    constexpr double t3 = t * t * t, t5 = t3 * t * t, t7 = t5 * t * t, t9 = t7 * t * t, t11 = t9 * t * t, t13 = t11 * t * t;
    float r = (float)(t13 / 6227020800.0);
    r = fmaf(r, w, (float)(-t11 / 39916800.0));
    r = fmaf(r, w, (float)(t9 / 362880.0));
    r = fmaf(r, w, (float)(-t7 / 5040.0));
    r = fmaf(r, w, (float)(t5 / 120.0));
    r = fmaf(r, w, (float)(-t3 / 6.0));
    // the leading term with 2 pi in two floats: its rounding would show in every value
    constexpr float th = (float)t, tl = (float)(t - (double)(float)t);
    return fmaf(th, v, fmaf(tl, v, r * w * v));
}

// Pair p of the chunk: the inverse FFT along y of F (cos(c|k|t_a) + i cos(c|k|t_b))
// -> kept rows Wt [chunk][nkeep][M].  Column tile by column tile, its pairs in
// turn, tiles contiguous per XCD: a tile's 64 bytes of F's rows stay cached from
// pair to pair, and the two tiles of a 128-byte line share an L2.
template <int M>
__global__ __launch_bounds__(sim_threads(M)) void k_sim_cols_inv_spec(SimDev s, SimSpecDev sp, const float2* __restrict__ F,
                                                                      float2* __restrict__ Wt, int pair0, int npairs)
{
    extern __shared__ __align__(16) float2 sm[];
    constexpr int T = sim_lanes(M), LD = grid_col_ld(M);
    using Fst = cfft_first<M, T>;
    constexpr int RH = (Fst::R + 1) / 2;  // inputs r < RH of a lane: rows up to the middle
    const int item = xcd_item(blockIdx.x, (M + kSimNP - 1) / kSimNP * npairs);
    if (item < 0) return;
    const int tile = item / npairs, p = item - tile * npairs;
    const int lane = threadIdx.x / kSimNP, sq = threadIdx.x % kSimNP;
    const int c = tile * kSimNP + sq, mx = c < M / 2 ? c : c - M;
    const bool on = lane < T && c < M;
    const int ja = 2 * (pair0 + p) + 1;
    const bool has_b = ja + 1 <= s.T;
    float2* x = sm + sq * LD;
    float2* out = Wt + (size_t)p * sp.nkeep * M + c;
    auto cosines = [&](int row) {  // rows up to M / 2
        const float2 u = sim_phase_rate(mx, row, s.a_hi, s.a_lo);
        return make_float2(sim_cos((float)ja, u), has_b ? sim_cos((float)(ja + 1), u) : 0.f);
    };
    // rows r and M - r share their cosines: the lower half is computed and
    // handed over in LDS, ahead of the transform
    float2 cs[Fst::RND][Fst::R];
    if (on) {
#pragma unroll
        for (int i = 0; i < Fst::RND; ++i)
#pragma unroll
            for (int r = 0; r < RH; ++r) {
                const int row = Fst::pos(lane, i, r);
                cs[i][r] = cosines(row <= M / 2 ? row : M - row);
                x[cfft_slot<true>(row)] = cs[i][r];
            }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int i = 0; i < Fst::RND; ++i)
#pragma unroll
            for (int r = RH; r < Fst::R; ++r) {
                const int row = Fst::pos(lane, i, r);
                cs[i][r] = 2 * row == M ? cosines(row) : x[cfft_slot<true>(M - row)];
            }
    }
    __syncthreads();
    cfft_stream<M, true, T, SyncWg, false>(
        x, sp.ctw, on, lane,
        [&](float2 (&v)[Fst::RND][Fst::R]) {
#pragma unroll
            for (int i = 0; i < Fst::RND; ++i)
#pragma unroll
                for (int r = 0; r < Fst::R; ++r) v[i][r] = F[(size_t)Fst::pos(lane, i, r) * M + c];
#pragma unroll
            for (int i = 0; i < Fst::RND; ++i)
#pragma unroll
                for (int r = 0; r < Fst::R; ++r) {
                    const float2 z = v[i][r], k = cs[i][r];
                    v[i][r] = make_float2(z.x * k.x - z.y * k.y, z.y * k.x + z.x * k.y);
                }
        },
        [&](int pos, float2 z) {
            const int row = sp.keep[pos];
            if (row >= 0) out[(size_t)row * M] = z;
        });
}

// Keys cubic convolution weight (a = -1/2) at distance t (0 <= t < 2)
__device__ __forceinline__ float keys_w(float t)
{
    constexpr float a = -0.5f;
    return t <= 1.f ? ((a + 2.f) * t - (a + 3.f)) * t * t + 1.f : ((a * t - 5.f * a) * t + 8.f * a) * t - 4.f * a;
}

// Inverse FFT along x of kept rows; their stencil rows' samples -> S [chunk][D][4]
template <int M>
__global__ __launch_bounds__(sim_threads(M)) void k_sim_rows_inv_spec(SimDev s, SimSpecDev sp, const float2* __restrict__ Wt,
                                                                      float2* __restrict__ S)
{
    extern __shared__ __align__(16) float2 sm[];
    constexpr int T = sim_lanes(M), LD = grid_col_ld(M);
    using Fst = cfft_first<M, T>;
    const int p = blockIdx.y, lane = threadIdx.x / kSimNP, sq = threadIdx.x % kSimNP;
    const int r0 = blockIdx.x * kSimNP, row = r0 + sq;
    const float2* src = Wt + ((size_t)p * sp.nkeep + min(row, sp.nkeep - 1)) * M;
    float2* x = sm + sq * LD;
    cfft_stream<M, true, T, SyncWg, true>(
        x, sp.ctw, lane < T && row < sp.nkeep, lane,
        [&](float2 (&v)[Fst::RND][Fst::R]) {
#pragma unroll
            for (int i = 0; i < Fst::RND; ++i)
#pragma unroll
                for (int r = 0; r < Fst::R; ++r) v[i][r] = src[Fst::pos(lane, i, r)];
        },
        [&](int pos, float2 z) { x[cfft_slot<true>(pos)] = z; });
    for (int k = 0; k < kSimNP && r0 + k < sp.nkeep; ++k)
        for (int e = sp.ent_ptr[r0 + k] + threadIdx.x; e < sp.ent_ptr[r0 + k + 1]; e += blockDim.x) {
            const int2 en = sp.ent[e];
            const int ix = s.dix[en.x].x;
            const float fx = s.dfr[en.x].x;
            const float wx[4] = {keys_w(1.f + fx), keys_w(fx), keys_w(1.f - fx), keys_w(2.f - fx)};
            const float2* rowp = sm + k * LD;
            float2 ra = make_float2(0.f, 0.f);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float2 v = rowp[cfft_slot<true>(ix - 1 + b)];
                ra.x = fmaf(wx[b], v.x, ra.x);
                ra.y = fmaf(wx[b], v.y, ra.y);
            }
            S[((size_t)p * s.D + en.x) * 4 + en.y] = ra;
        }
}

// The stencil rows' sum at each detector: thread (d, p) -> g[d][ja - 1] and g[d][jb - 1]
__global__ __launch_bounds__(256) void k_sim_combine(SimDev s, const float2* __restrict__ S, float* __restrict__ g, int pair0,
                                                     int npairs)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= s.D * npairs) return;
    const int d = t / npairs, p = t - d * npairs;
    const int ja = 2 * (pair0 + p) + 1, jb = ja + 1;
    const float fy = s.dfr[d].y;
    const float wy[4] = {keys_w(1.f + fy), keys_w(fy), keys_w(1.f - fy), keys_w(2.f - fy)};
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float2 ra = S[((size_t)p * s.D + d) * 4 + a];
        acc.x = fmaf(wy[a], ra.x, acc.x);
        acc.y = fmaf(wy[a], ra.y, acc.y);
    }
    const float scale = 1.0f / ((float)s.M * (float)s.M);
    g[(size_t)d * s.T + ja - 1] = acc.x * scale;
    if (jb <= s.T) g[(size_t)d * s.T + jb - 1] = acc.y * scale;
}

// ---------------------------------------------------------------------------
// Run-time box sides (below 216 and above 2048)
// ---------------------------------------------------------------------------
// Samples at the detectors: thread (d, p) -> g[d][ja - 1] and g[d][jb - 1]
__global__ __launch_bounds__(256) void k_sim_sample(SimDev s, const float2* __restrict__ Wt, float* __restrict__ g,
                                                    int pair0, int npairs)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= s.D * npairs) return;
    const int p = t / s.D, d = t - p * s.D;
    const int ja = 2 * (pair0 + p) + 1, jb = ja + 1;
    const int2 ix = s.dix[d];
    const float2 fr = s.dfr[d];
    const float wx[4] = {keys_w(1.f + fr.x), keys_w(fr.x), keys_w(1.f - fr.x), keys_w(2.f - fr.x)};
    const float wy[4] = {keys_w(1.f + fr.y), keys_w(fr.y), keys_w(1.f - fr.y), keys_w(2.f - fr.y)};
    const float2* base = Wt + (size_t)p * s.nrow * s.M;
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float2* row = base + (size_t)(ix.y - 1 + a - s.rlo) * s.M + (ix.x - 1);
        float2 ra = make_float2(0.f, 0.f);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            ra.x = fmaf(wx[b], row[b].x, ra.x);
            ra.y = fmaf(wx[b], row[b].y, ra.y);
        }
        acc.x = fmaf(wy[a], ra.x, acc.x);
        acc.y = fmaf(wy[a], ra.y, acc.y);
    }
    const float scale = 1.0f / ((float)s.M * (float)s.M);
    g[(size_t)d * s.T + ja - 1] = acc.x * scale;
    if (jb <= s.T) g[(size_t)d * s.T + jb - 1] = acc.y * scale;
}

}  // namespace pat

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------

using pat::SimDev;

struct pat_sim {
    SimDev dev;
    pat::SimSpecDev sp;
    void* table_mem;
    int device;
    int thr_col, thr_row;       // workgroup sizes of the column and row transforms
    size_t lds_col, lds_row;    // their dynamic LDS
    int npairs, chunk;          // time-sample pairs, pairs per chunk
    size_t off_F, off_W, off_Wt, off_S, ws_bytes;
    int spec;                   // compile-time box side
};

namespace {

constexpr int kSimMaxBox = 8192;
constexpr int kSimChunk = 16;
constexpr size_t kSimLdsMax = 160 * 1024;

long smooth_2a3b(long m)
{
    long best = -1;
    for (long p2 = 1; p2 < 2 * m + 2; p2 *= 2)
        for (long p = p2; p < 2 * m + 2; p *= 3)
            if (p >= m && (best < 0 || p < best)) best = p;
    return best;
}

// box side per the rule in pat.h
long sim_box_side(int ns, double det_r, double support_r, double c, double t_last)
{
    const double h = 2.0 / ns;
    const double half = std::max((det_r + support_r + c * t_last) / 2.0, det_r + 3.0 * h) + h;
    long m = std::max((long)std::ceil(2.0 * half / h), (long)ns);
    for (;;) {
        m = smooth_2a3b(m);
        if (m % 2 == 0) return m;
        ++m;
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

extern "C" int pat_sim_create(const pat_plan_desc* desc, pat_sim** out)
{
    if (!desc || !out) return PAT_ERR_ARG;
    const int Ns = desc->n, D = desc->n_det, T = desc->n_t;
    if (Ns < 8 || D < 1 || T < 1 || !(desc->dt > 0.0) || !(desc->c > 0.0) || !(desc->det_r > 0.0) ||
        !(desc->support_r > 0.0))
        return PAT_ERR_ARG;
    const double h = 2.0 / Ns;
    const long Ml = sim_box_side(Ns, desc->det_r, desc->support_r, desc->c, T * desc->dt);
    if (Ml > kSimMaxBox) return PAT_ERR_UNSUPPORTED;
    const int M = (int)Ml;

    pat_sim* s = new (std::nothrow) pat_sim;
    if (!s) return PAT_ERR_ALLOC;
    std::memset(s, 0, sizeof(*s));
    SimDev& d = s->dev;
    d.Ns = Ns;
    d.M = M;
    d.off = (M - Ns) / 2;
    d.D = D;
    d.T = T;
    {
        const double alpha = desc->c * desc->dt / (M * h);
        d.a_hi = (float)alpha;
        d.a_lo = (float)(alpha - (double)d.a_hi);
    }

    // support mask per image row (FP64, as the reference decides it)
    std::vector<int2> mrows(Ns);
    for (int i = 0; i < Ns; ++i) {
        const double y = -1.0 + (i + 0.5) * h;
        int lo = Ns, hi = 0;
        for (int j = 0; j < Ns; ++j) {
            const double x = -1.0 + (j + 0.5) * h;
            if (x * x + y * y < desc->support_r * desc->support_r) {
                lo = std::min(lo, j);
                hi = j + 1;
            }
        }
        mrows[i] = make_int2(lo < hi ? lo : 0, lo < hi ? hi : 0);
    }
    // detectors: stencil cells and fractional offsets in box index units
    std::vector<int2> dix(D);
    std::vector<float2> dfr(D);
    int ylo = M, yhi = -1;
    for (int q = 0; q < D; ++q) {
        const double th = desc->det_theta ? desc->det_theta[q]
                                          : desc->arc_center - desc->arc_span / 2 + (q + 0.5) * desc->arc_span / D;
        // relative to the image's centre: the box's for even Ns, half a cell before it for odd
        const double gx = desc->det_r * std::cos(th) / h + d.off + Ns / 2.0 - 0.5;
        const double gy = desc->det_r * std::sin(th) / h + d.off + Ns / 2.0 - 0.5;
        const int ix = (int)std::floor(gx), iy = (int)std::floor(gy);
        if (ix - 1 < 0 || ix + 2 >= M || iy - 1 < 0 || iy + 2 >= M) {
            delete s;
            return PAT_ERR_UNSUPPORTED;
        }
        dix[q] = make_int2(ix, iy);
        dfr[q] = make_float2((float)(gx - ix), (float)(gy - iy));
        ylo = std::min(ylo, iy - 1);
        yhi = std::max(yhi, iy + 3);
    }
    d.rlo = ylo;
    d.nrow = yhi - ylo;

    std::vector<float2> tw;
    const int tps = pat::fixed_fft_for(M, &d.fm, tw);
    if (!tps) {
        delete s;
        return PAT_ERR_UNSUPPORTED;
    }
    // workgroup shapes: the most columns / rows per workgroup (8, 4, 2, 1) whose
    // threads and LDS fit
    auto shape = [&](int& n_out, int& thr_out, size_t& lds_out) {
        for (int n = 8; n >= 1; n /= 2) {
            const int thr = pat::fft_workgroup_threads(n, d.fm);
            const size_t lds = sizeof(float2) * ((size_t)n * M + (size_t)d.fm.ntb);
            if (thr <= 1024 && lds <= kSimLdsMax / 2) {
                n_out = n;
                thr_out = thr;
                lds_out = lds;
                return true;
            }
        }
        return false;
    };
    if (!shape(d.CT, s->thr_col, s->lds_col) || !shape(d.RPB, s->thr_row, s->lds_row)) {
        delete s;
        return PAT_ERR_UNSUPPORTED;
    }

    // compile-time box sides: the kept rows, the stencil rows in each, the transform's table
    s->spec = pat::sim_len_ok(M);
    std::vector<int> keep(M, -1), eptr;
    std::vector<int2> ent;
    std::vector<float2> ctw;
    if (s->spec) {
        std::vector<std::vector<int2>> in_row(M);
        for (int q = 0; q < D; ++q)
            for (int a = 0; a < 4; ++a) in_row[dix[q].y - 1 + a].push_back(make_int2(q, a));
        for (int r = 0; r < M; ++r) {
            if (in_row[r].empty()) continue;
            keep[r] = s->sp.nkeep++;
            eptr.push_back((int)ent.size());
            ent.insert(ent.end(), in_row[r].begin(), in_row[r].end());
        }
        eptr.push_back((int)ent.size());
        const pat::CPlan cp = pat::make_cplan(M);
        ctw.resize(cp.twoff[cp.np]);
        for (int st = 0; st < cp.np; ++st)
            for (int k = 0; cp.ns[st] > 1 && k < cp.ns[st]; ++k)
                for (int r = 1; r < cp.rad[st]; ++r) {
                    const double a = -2.0 * 3.14159265358979323846 * (double)(k * r) / (double)(cp.ns[st] * cp.rad[st]);
                    ctw[cp.twoff[st] + k * (cp.rad[st] - 1) + r - 1] = make_float2((float)std::cos(a), (float)std::sin(a));
                }
    }

    // device tables
    size_t o_mask = 0, o_dix = align256(o_mask + sizeof(int2) * Ns), o_dfr = align256(o_dix + sizeof(int2) * D),
           o_tw = align256(o_dfr + sizeof(float2) * D), o_keep = align256(o_tw + sizeof(float2) * tw.size()),
           o_eptr = align256(o_keep + sizeof(int) * keep.size()), o_ent = align256(o_eptr + sizeof(int) * eptr.size()),
           o_ctw = align256(o_ent + sizeof(int2) * ent.size()), bytes = o_ctw + sizeof(float2) * ctw.size();
    std::vector<unsigned char> host(bytes, 0);
    std::memcpy(host.data() + o_mask, mrows.data(), sizeof(int2) * Ns);
    std::memcpy(host.data() + o_dix, dix.data(), sizeof(int2) * D);
    std::memcpy(host.data() + o_dfr, dfr.data(), sizeof(float2) * D);
    std::memcpy(host.data() + o_tw, tw.data(), sizeof(float2) * tw.size());
    std::memcpy(host.data() + o_keep, keep.data(), sizeof(int) * keep.size());
    if (s->spec) {
        std::memcpy(host.data() + o_eptr, eptr.data(), sizeof(int) * eptr.size());
        std::memcpy(host.data() + o_ent, ent.data(), sizeof(int2) * ent.size());
        std::memcpy(host.data() + o_ctw, ctw.data(), sizeof(float2) * ctw.size());
    }
    if (hipGetDevice(&s->device) != hipSuccess) {
        delete s;
        return PAT_ERR_HIP;
    }
    if (hipMalloc(&s->table_mem, bytes) != hipSuccess) {
        delete s;
        return PAT_ERR_ALLOC;
    }
    if (hipMemcpy(s->table_mem, host.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(s->table_mem);
        delete s;
        return PAT_ERR_HIP;
    }
    char* base = (char*)s->table_mem;
    d.mask_rows = (const int2*)(base + o_mask);
    d.dix = (const int2*)(base + o_dix);
    d.dfr = (const float2*)(base + o_dfr);
    d.tw = (const float2*)(base + o_tw);
    s->sp.keep = (const int*)(base + o_keep);
    s->sp.ent_ptr = (const int*)(base + o_eptr);
    s->sp.ent = (const int2*)(base + o_ent);
    s->sp.ctw = (const float2*)(base + o_ctw);

    // workspace: F [M][M], W [Ns][M], Wt [chunk][nrow][M]
    s->npairs = (T + 1) / 2;
    s->chunk = std::min(s->npairs, kSimChunk);
    s->off_F = 0;
    s->off_W = align256(sizeof(float2) * (size_t)M * M);
    s->off_Wt = s->off_W + align256(sizeof(float2) * (size_t)Ns * M);
    s->ws_bytes = s->off_Wt + align256(sizeof(float2) * (size_t)s->chunk * d.nrow * M);
    // compile-time box sides: the stencil rows' samples [chunk][D][4], over W
    // (read before the first of them is written) where they fit
    const size_t s_bytes = align256(sizeof(float2) * 4 * (size_t)s->chunk * D);
    s->off_S = s->off_W;
    if (s->spec && s_bytes > s->off_Wt - s->off_W) {
        s->off_S = s->ws_bytes;
        s->ws_bytes += s_bytes;
    }
    *out = s;
    return PAT_OK;
}

extern "C" int pat_sim_query(const pat_sim* s, int* box_side, size_t* workspace_bytes)
{
    if (!s) return PAT_ERR_ARG;
    if (box_side) *box_side = s->dev.M;
    if (workspace_bytes) *workspace_bytes = s->ws_bytes;
    return PAT_OK;
}

extern "C" int pat_sim_run(const pat_sim* s, const float* f, float* g, void* ws, size_t ws_bytes, void* stream)
{
    if (!s || !f || !g) return PAT_ERR_ARG;
    if (!ws || ws_bytes < s->ws_bytes) return PAT_ERR_WORKSPACE;
    const SimDev& d = s->dev;
    hipStream_t st = (hipStream_t)stream;
    char* w = (char*)ws;
    float2* F = (float2*)(w + s->off_F);
    float2* W = (float2*)(w + s->off_W);
    float2* Wt = (float2*)(w + s->off_Wt);
    hipLaunchKernelGGL(pat::k_sim_rows_fwd, dim3((d.Ns + d.RPB - 1) / d.RPB), dim3(s->thr_row), s->lds_row, st, d, f,
                       W);
    if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
    hipLaunchKernelGGL(pat::k_sim_cols_fwd, dim3((d.M + d.CT - 1) / d.CT), dim3(s->thr_col), s->lds_col, st, d,
                       (const float2*)W, F);
    if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
    float2* Sd = (float2*)(w + s->off_S);
    for (int p0 = 0; p0 < s->npairs; p0 += s->chunk) {
        const int np = std::min(s->chunk, s->npairs - p0);
        if (s->spec) {
            const dim3 gc(pat::xcd_grid((d.M + pat::kSimNP - 1) / pat::kSimNP * np)), gr((s->sp.nkeep + pat::kSimNP - 1) / pat::kSimNP, np);
            switch (d.M) {
#define PAT_CASE(LEN)                                                                                                 \
    case LEN: {                                                                                                       \
        const size_t lds = sizeof(float2) * (size_t)pat::kSimNP * pat::grid_col_ld(LEN);                               \
        hipLaunchKernelGGL(pat::k_sim_cols_inv_spec<LEN>, gc, dim3(pat::sim_threads(LEN)), lds, st, d, s->sp, (const float2*)F, Wt, p0, np); \
        hipLaunchKernelGGL(pat::k_sim_rows_inv_spec<LEN>, gr, dim3(pat::sim_threads(LEN)), lds, st, d, s->sp, (const float2*)Wt, Sd);    \
        break;                                                                                                        \
    }
                PAT_SIM_LENGTHS(PAT_CASE)
#undef PAT_CASE
                default: break;
            }
            if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
            hipLaunchKernelGGL(pat::k_sim_combine, dim3((d.D * np + 255) / 256), dim3(256), 0, st, d, (const float2*)Sd, g,
                               p0, np);
            if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
            continue;
        }
        hipLaunchKernelGGL(pat::k_sim_cols_inv, dim3((d.M + d.CT - 1) / d.CT, np), dim3(s->thr_col), s->lds_col, st, d,
                           (const float2*)F, Wt, p0);
        if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
        hipLaunchKernelGGL(pat::k_sim_rows_inv, dim3((d.nrow + d.RPB - 1) / d.RPB, np), dim3(s->thr_row), s->lds_row,
                           st, d, Wt);
        if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
        hipLaunchKernelGGL(pat::k_sim_sample, dim3((d.D * np + 255) / 256), dim3(256), 0, st, d, (const float2*)Wt, g,
                           p0, np);
        if (hipGetLastError() != hipSuccess) return PAT_ERR_HIP;
    }
    return PAT_OK;
}

extern "C" void pat_sim_destroy(pat_sim* s)
{
    if (!s) return;
    if (s->table_mem) {
        int cur = 0;
        if (hipGetDevice(&cur) != hipSuccess) cur = s->device;
        (void)hipSetDevice(s->device);
        (void)hipFree(s->table_mem);
        (void)hipSetDevice(cur);
    }
    delete s;
}
