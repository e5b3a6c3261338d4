// grid.hpp -- the 2D transform's passes with a compile-time grid side NG (plans
// with grid_spec): column passes (FFT along y of real columns, packed in pairs)
// and row passes (FFT along x), forward and adjoint.
//
// Memory goes straight into the transform's first pass and out of its last one
// (cfft_stream), so LDS only carries the exchanges between passes, zero padding
// is neither stored nor read and cropped outputs are never formed.
//   rows: one sequence per wave(s), lanes along the row: 512-byte accesses;
//         waves of one-wave lengths run independently of each other;
//   columns: sequence s of a workgroup's NP pairs is transformed by the threads
//         t = s mod NP, so that neighbouring threads read and write neighbouring
//         columns of a row (8 NP bytes of f, 16 NP of X1).
#pragma once

#include "cfft.hpp"
#include "device_util.hpp"
#include "pat_internal.hpp"

#include <type_traits>

namespace pat {

// Image index of padded position pos (centred: image index i sits at i - N/2 mod
// NG), or a value outside 0 .. N - 1 where the position is padding.
template <int NG>
__device__ __forceinline__ int grid_image_index(int pos, int N)
{
    return pos < NG / 2 ? pos + N / 2 : pos - NG + N / 2;
}

// No image index among positions [lo, lo + n)
template <int NG>
__device__ __forceinline__ bool grid_all_padding(int lo, int n, int N)
{
    return lo >= N - N / 2 && lo + n <= NG - N / 2;
}

// forward: mask, deapodise, zero-pad, FFT along y of column pairs -> X1 [Hy][N]
// (rows m_y = -4 .. NG/2 + 4), and the per-column sums of h^2 m f.  vec: f's rows
// allow 8-byte loads of a pair (N even, f 8-byte aligned).
template <int NG>
__device__ __forceinline__ void colpass_fwd_spec(const PlanDev& d, const WsLayout& L, const float* __restrict__ fb,
                                                 char* wb, int tile, int NP, bool vec, float2* sm)
{
    constexpr int T = cfft_lanes(NG), LD = grid_col_ld(NG);
    using F = cfft_first<NG, T>;
    const int N = d.N;
    float2* __restrict__ X1 = (float2*)(wb + L.x1);
    float* red = (float*)(wb + L.red);
    const int lane = threadIdx.x / NP, s = threadIdx.x - lane * NP;
    const int c0 = 2 * (tile * NP + s);  // the pair's first column
    const bool active = lane < T && c0 < N, odd = c0 + 1 < N;
    float2* x = sm + (size_t)s * LD;
    float* red_s = (float*)(sm + (size_t)NP * LD);  // [T][2 NP] lane sums, [kColSumGroups][2 NP] group sums
    const int c1 = odd ? c0 + 1 : c0;
    const float d0 = active ? d.deap[c0] : 0.f, d1 = active && odd ? d.deap[c1] : 0.f;
    cfft_stream<NG, false, T, SyncWg, true>(
        x, d.ctw + d.grid_ctw, active, lane,
        [&](float2 (&v)[F::RND][F::R]) {
            float2 raw[F::RND][F::R];
            int2 mr[F::RND][F::R];
            float dy[F::RND][F::R];
#pragma unroll
            for (int i = 0; i < F::RND; ++i)
#pragma unroll
                for (int r = 0; r < F::R; ++r) {
                    if (grid_all_padding<NG>(r * F::NB, F::NB, N)) continue;
                    const int row = min(max(grid_image_index<NG>(F::pos(lane, i, r), N), 0), N - 1);
                    const float* p = fb + (size_t)row * N;
                    raw[i][r] = vec ? *(const float2*)(p + c0) : make_float2(p[c0], p[c1]);
                    mr[i][r] = d.mask_rows[row];
                    dy[i][r] = d.deap[row];
                }
            float2 sum = make_float2(0.f, 0.f);
#pragma unroll
            for (int i = 0; i < F::RND; ++i)
#pragma unroll
                for (int r = 0; r < F::R; ++r) {
                    v[i][r] = make_float2(0.f, 0.f);
                    if (grid_all_padding<NG>(r * F::NB, F::NB, N)) continue;
                    const int row = grid_image_index<NG>(F::pos(lane, i, r), N);
                    const bool in = row >= 0 && row < N;
                    const bool i0 = in && c0 >= mr[i][r].x && c0 < mr[i][r].y;
                    const bool i1 = in && odd && c1 >= mr[i][r].x && c1 < mr[i][r].y;
                    v[i][r] = make_float2(i0 ? raw[i][r].x * dy[i][r] * d0 : 0.f, i1 ? raw[i][r].y * dy[i][r] * d1 : 0.f);
                    const bool own = F::own(lane, i);
                    sum.x = own && i0 ? sum.x + raw[i][r].x : sum.x;
                    sum.y = own && i1 ? sum.y + raw[i][r].y : sum.y;
                }
            red_s[(lane * NP + s) * 2] = sum.x;
            red_s[(lane * NP + s) * 2 + 1] = sum.y;
        },
        [&](int pos, float2 z) { x[cfft_slot<true>(pos)] = z; });
    // rows m = -4 .. NG/2 + 4 of the two columns: (Z(m) + conj Z(-m)) / 2 and (Z(m) - conj Z(-m)) / (2i)
    if (active) {
        const bool pair16 = (N & 1) == 0;
        for (int r = lane; r < NG / 2 + 9; r += T) {
            const int m = r - 4, ip = m < 0 ? m + NG : m, in = m > 0 ? NG - m : -m;
            const float2 zp = x[cfft_slot<true>(ip)], zn = x[cfft_slot<true>(in)];
            const float2 a = make_float2(0.5f * (zp.x + zn.x), 0.5f * (zp.y - zn.y));
            const float2 b = make_float2(0.5f * (zp.y + zn.y), -0.5f * (zp.x - zn.x));
            float2* o = X1 + (size_t)r * N + c0;
            if (pair16) {
                *(float4*)o = make_float4(a.x, a.y, b.x, b.y);
            } else {
                o[0] = a;
                if (odd) o[1] = b;
            }
        }
    }
    // the columns' sums: lanes g, g + kColSumGroups, ... of each column, then the groups in order
    const int CT = 2 * NP;
    float* grp = red_s + T * CT;
    for (int u = threadIdx.x; u < kColSumGroups * CT; u += blockDim.x) {
        const int c = u % CT, g = u / CT;
        float a = 0.f;
        if (2 * tile * NP + c < N)
            for (int l = g; l < T; l += kColSumGroups) a += red_s[l * CT + c];
        grp[u] = a;
    }
    __syncthreads();
    if ((int)threadIdx.x < CT && 2 * tile * NP + (int)threadIdx.x < N) {
        float a = 0.f;
#pragma unroll
        for (int g = 0; g < kColSumGroups; ++g) a += grp[g * CT + threadIdx.x];
        red[2 * tile * NP + threadIdx.x] = a * d.h2;
    }
}

// adjoint: Hermitian symmetrisation, inverse FFT along y of column pairs, crop,
// deapodise, mask, plus the endpoint term's constant.  vec: as above, for f's stores.
template <int NG>
__device__ __forceinline__ void colpass_adj_spec(const PlanDev& d, const WsLayout& L, char* wb, float* __restrict__ fb,
                                                 int tile, int NP, int n_sum, bool vec, float2* sm, float* gsum_s)
{
    constexpr int T = cfft_lanes(NG), LD = grid_col_ld(NG);
    using F = cfft_first<NG, T>;
    const int N = d.N;
    const float2* __restrict__ X1 = (const float2*)(wb + L.x1);
    const float* red = (const float*)(wb + L.red);
    if (threadIdx.x < 64) {
        const float a = wave0_fixed_sum(red, n_sum);
        if (threadIdx.x == 0) *gsum_s = a;  // read after the transform's barriers
    }
    const int lane = threadIdx.x / NP, s = threadIdx.x - lane * NP;
    const int c0 = 2 * (tile * NP + s);
    const bool active = lane < T && c0 < N, odd = c0 + 1 < N, pair16 = (N & 1) == 0;
    const int c1 = odd ? c0 + 1 : c0;
    const float d0 = active ? d.deap[c0] : 0.f, d1 = active ? d.deap[c1] : 0.f;
    auto row_pair = [&](int row) {  // X1's two values, the second 0 past the last column
        const float2* p = X1 + (size_t)row * N;
        if (pair16) return *(const float4*)(p + c0);
        const float2 a = p[c0], b = p[c1];
        return make_float4(a.x, a.y, odd ? b.x : 0.f, odd ? b.y : 0.f);
    };
    constexpr int top = NG / 2 + 4;
    cfft_stream<NG, true, T, SyncWg, false>(
        sm + (size_t)s * LD, d.ctw + d.grid_ctw, active, lane,
        [&](float2 (&v)[F::RND][F::R]) {
            // z(q) = (ua(q) + conj ua(-q)) / 2 + i (ub(q) + conj ub(-q)) / 2 with u stored for
            // residues -4 .. NG/2 + 4: one of q, -q is, and near 0 and NG/2 both
            float4 u[F::RND][F::R];
#pragma unroll
            for (int i = 0; i < F::RND; ++i)
#pragma unroll
                for (int r = 0; r < F::R; ++r) {
                    const int q = F::pos(lane, i, r);
                    u[i][r] = row_pair(q <= top ? q + 4 : NG - q + 4);
                }
#pragma unroll
            for (int i = 0; i < F::RND; ++i)
#pragma unroll
                for (int r = 0; r < F::R; ++r) {
                    const int q = F::pos(lane, i, r);
                    float4 w = u[i][r];
                    if (q > top) { w.y = -w.y; w.w = -w.w; }
                    // the other of q, -q, where it is stored too
                    const int qn = q == 0 ? 0 : NG - q;
                    const bool nq = q <= top ? (qn <= top || qn >= NG - 4) : q >= NG - 4;
                    if (nq) {
                        const bool up = q <= top;  // the other is -q (conjugated), or q itself stored below 0
                        const float4 t = row_pair(up ? (qn <= top ? qn + 4 : qn - NG + 4) : q - NG + 4);
                        w.x += t.x;
                        w.z += t.z;
                        w.y += up ? -t.y : t.y;
                        w.w += up ? -t.w : t.w;
                    }
                    v[i][r] = make_float2(0.5f * w.x - 0.5f * w.w, 0.5f * w.y + 0.5f * w.z);
                }
        },
        [&](int pos, float2 z) {
            const int row = grid_image_index<NG>(pos, N);
            if (row < 0 || row >= N) return;
            const int2 mr = d.mask_rows[row];
            const float dy = d.deap[row], kt = d.kappa * d.h2 * *gsum_s;
            const float a = c0 >= mr.x && c0 < mr.y ? dy * d0 * z.x + kt : 0.f;
            const float b = c1 >= mr.x && c1 < mr.y ? dy * d1 * z.y + kt : 0.f;
            float* o = fb + (size_t)row * N + c0;
            if (vec) {
                *(float2*)o = make_float2(a, b);
            } else {
                o[0] = a;
                if (odd) o[1] = b;
            }
        });
}

// forward: zero-pad, FFT along x of RPB rows -> G [Hy][NG]
template <int NG>
__device__ __forceinline__ void rowpass_fwd_spec(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RPB, float2* sm)
{
    constexpr int T = cfft_lanes(NG), LD = cfft_padded_len(NG);
    using F = cfft_first<NG, T>;
    using Sync = std::conditional_t<T == 64, SyncWave, SyncWg>;
    const int N = d.N, sq = threadIdx.x / T, lane = threadIdx.x - sq * T, row = tile * RPB + sq;
    const bool active = sq < RPB && row < d.Hy;
    const float2* __restrict__ src = (const float2*)(wb + L.x1) + (size_t)min(row, d.Hy - 1) * N;
    float2* __restrict__ dst = (float2*)(wb + L.grid) + (size_t)row * NG;
    cfft_stream<NG, false, T, Sync, false>(
        sm + (size_t)min(sq, RPB - 1) * LD, d.ctw + d.grid_ctw, active, lane,
        [&](float2 (&v)[F::RND][F::R]) {
#pragma unroll
            for (int i = 0; i < F::RND; ++i)
#pragma unroll
                for (int r = 0; r < F::R; ++r) {
                    v[i][r] = make_float2(0.f, 0.f);
                    if (grid_all_padding<NG>(r * F::NB, F::NB, N)) continue;
                    const int c = grid_image_index<NG>(F::pos(lane, i, r), N);
                    const float2 u = src[min(max(c, 0), N - 1)];
                    if (c >= 0 && c < N) v[i][r] = u;
                }
        },
        [&](int pos, float2 z) { dst[pos] = z; });
}

// First and last run of a spread row tile split 2^lg ways (lg >= 1) that reach
// relative row x (0 .. 14): run j covers x when j w <= x <= j w + w + 6, w = 8 / 2^lg.
__device__ __forceinline__ int2 split_runs_at(int lg, int x)
{
    const int w = kSpreadTh >> lg, a = x - w - 6;
    return make_int2(a > 0 ? (a + w - 1) >> (3 - lg) : 0, min((1 << lg) - 1, x >> (3 - lg)));
}

// Where the adjoint row pass finds grid row r = 8 q + k: row tile q's part (its
// grid row, or, if the tile was split into S runs, the slab rows of the runs that
// reach relative row k) and, for q >= 1, k < 7 and 8 q < NB (a spread row tile q
// exists), row tile q - 1's part at relative row k + 8 (its tail row, or its runs'
// slab rows).  Run j of a tile split S ways (w = 8 / S bands) holds relative rows
// j w .. j w + w + 6 at slab rows s0 + 7 j + (relative row).  The terms are added
// in one order: (the tile's part, its runs in order) + (the previous tile's part,
// its runs in order).
struct GridRow {
    const float2 *o, *t;  // the two parts' first rows (t: o where there is none)
    int no, nt;           // their numbers of rows, 7 Ng apart
};

__device__ __forceinline__ GridRow grid_row(const PlanDev& d, const WsLayout& L, const char* wb, int r)
{
    static_assert(kSpreadTh == 8, "row tiles by shifting");
    const size_t Ng = d.Ng;
    const float2* Gt = (const float2*)(wb + L.grid);
    const float2* Tl = (const float2*)(wb + L.tail);
    const float2* Sl = (const float2*)(wb + L.slab);
    const int q = r >> 3, k = r & 7;
    const bool tail = q >= 1 && k < 7 && 8 * q < d.NB;
    const unsigned eo = d.spr_head[q], et = tail ? d.spr_head[q - 1] : 0u;  // log2 of the runs, first slab row
    GridRow g{Gt + (size_t)r * Ng, nullptr, 1, tail ? 1 : 0};
    if (eo & 15u) {
        g.no = split_runs_at(eo & 15u, k).y + 1;
        g.o = Sl + (size_t)((eo >> 4) + k) * Ng;
    }
    g.t = tail ? Tl + ((size_t)(q - 1) * 7 + k) * Ng : g.o;
    if (et & 15u) {
        const int2 j = split_runs_at(et & 15u, k + 8);
        g.nt = j.y - j.x + 1;
        g.t = Sl + (size_t)((et >> 4) + 7 * j.x + k + 8) * Ng;
    }
    return g;
}

__device__ __forceinline__ float2 grid_row_at(const GridRow& g, int Ng, int c)
{
    float2 o = g.o[c];
    for (int j = 1; j < g.no; ++j) o = cadd(o, g.o[(size_t)(7 * j) * Ng + c]);
    if (!g.nt) return o;
    float2 t = g.t[c];
    for (int j = 1; j < g.nt; ++j) t = cadd(t, g.t[(size_t)(7 * j) * Ng + c]);
    return cadd(o, t);
}

// adjoint: complete the spread's rows, inverse FFT along x, crop -> X1 [Hy][N]
template <int NG>
__device__ __forceinline__ void rowpass_adj_spec(const PlanDev& d, const WsLayout& L, char* wb, int tile, int RPB, float2* sm)
{
    constexpr int T = cfft_lanes(NG), LD = cfft_padded_len(NG);
    using F = cfft_first<NG, T>;
    using Sync = std::conditional_t<T == 64, SyncWave, SyncWg>;
    const int N = d.N, sq = __builtin_amdgcn_readfirstlane(threadIdx.x / T), lane = threadIdx.x - sq * T;
    const int row = tile * RPB + sq;
    const bool active = sq < RPB && row < d.Hy;
    const GridRow g = grid_row(d, L, wb, min(row, d.Hy - 1));
    float2* __restrict__ dst = (float2*)(wb + L.x1) + (size_t)row * N;
    cfft_stream<NG, true, T, Sync, false>(
        sm + (size_t)min(sq, RPB - 1) * LD, d.ctw + d.grid_ctw, active, lane,
        [&](float2 (&v)[F::RND][F::R]) {
            if (g.no == 1 && g.nt <= 1) {  // uniform over the sequence: whole tiles
                float2 t[F::RND][F::R];
#pragma unroll
                for (int i = 0; i < F::RND; ++i)
#pragma unroll
                    for (int r = 0; r < F::R; ++r) {
                        v[i][r] = g.o[F::pos(lane, i, r)];
                        if (g.nt) t[i][r] = g.t[F::pos(lane, i, r)];
                    }
                if (g.nt) {
#pragma unroll
                    for (int i = 0; i < F::RND; ++i)
#pragma unroll
                        for (int r = 0; r < F::R; ++r) v[i][r] = cadd(v[i][r], t[i][r]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < F::RND; ++i)
#pragma unroll
                    for (int r = 0; r < F::R; ++r) v[i][r] = grid_row_at(g, NG, F::pos(lane, i, r));
            }
        },
        [&](int pos, float2 z) {
            const int c = grid_image_index<NG>(pos, N);
            if (c >= 0 && c < N) dst[c] = z;
        });
}

}  // namespace pat
