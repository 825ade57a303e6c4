// Gain-calibration loss and its gradient with respect to the complex gains.
// Sec. "Calibration Pipeline": per-channel amplitude and phase calibration of
// the XX and YY visibilities against a point-source sky model; read here as
// the least-squares loss
//
//   R_ab = V_ab - g_a M_ab conj(g_b),   L = sum_{a,b} |R_ab|^2
//   grad_a = dL/dRe g_a + i dL/dIm g_a = -2 sum_b [R_ab conj(M_ab) + conj(R_ba) M_ba] g_b
//
// With V and M stored as lower triangles (upper = conjugate), R is Hermitian
// off the diagonal and, for t_ab = R_ab conj(M_ab),
//   grad_a = -4 [ sum_{b<a} t_ab g_b + sum_{c>a} conj(t_ca) g_c + Re(t_aa) g_a ].
// Every stored element therefore feeds one row sum (antenna a) and one
// column sum (antenna b).
//
// Weighted form (Sec. "Real-time Flagging, Calibration and Imaging": the
// calibration works on the flagged visibilities, re-weighted for lost data):
// L = sum_{a,b} w_ab |R_ab|^2 with a real weight w_ab = w_ba per stored
// baseline and polarisation (0 where flagged), and t_ab = w_ab R_ab conj(M_ab).
//
// Pass 1: one workgroup per 64 x 64 antenna tile of the lower triangle and
// channel, both polarisations.  Each thread owns 4 rows x 4 columns;
// the residual is formed in float32 with error-free product and sum
// transformations, so that R keeps full float32 relative accuracy even when
// V and G M G^H cancel to a few percent.  Row sums (over the 16 lanes
// of a row) and column sums (over lanes, then LDS across the waves) are
// accumulated in float64 and written to the workspace; the tile's loss is a
// float32 tree sum.
// Pass 2: one thread per antenna adds its row and column partials over the
// tiles in a fixed order (float64) and writes -4 x the sum; the first block
// of each (channel, polarisation) adds the tile losses in a fixed order.
// No atomics: the result is bitwise reproducible.
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "afc_internal.h"

// The error-free transformations below need every product and sum rounded
// on its own: this file is compiled with -ffp-contract=off (the fma in
// two_prod is explicit), and the pragma keeps the intent visible.
#pragma clang fp contract(off)

namespace afc {
namespace {

constexpr int kTileA = 64;      // antennas per tile side
constexpr int kThreads = 256;   // 4 waves: rows r, r+4, ...

struct ff {
    float hi, lo;
};
__device__ __forceinline__ ff two_prod(float a, float b) {
    const float p = __fmul_rn(a, b);
    return {p, fmaf(a, b, -p)};
}
__device__ __forceinline__ ff two_sum(float a, float b) {
    const float s = __fadd_rn(a, b);
    const float bb = __fsub_rn(s, a);
    const float e = __fadd_rn(__fsub_rn(a, __fsub_rn(s, bb)), __fsub_rn(b, bb));
    return {s, e};
}
// a*b + c*d as hi + lo
__device__ __forceinline__ ff dot2(float a, float b, float c, float d) {
    const ff p = two_prod(a, b), q = two_prod(c, d);
    const ff s = two_sum(p.hi, q.hi);
    return {s.hi, __fadd_rn(s.lo, __fadd_rn(p.lo, q.lo))};
}

// R = V - g_a M conj(g_b), each component rounded once to float32.
__device__ __forceinline__ float2 residual(float2 v, float2 m, float2 ga, float2 gb) {
    // q = g_a conj(g_b)
    const ff qr = dot2(ga.x, gb.x, ga.y, gb.y);
    const ff qi = dot2(ga.y, gb.x, -ga.x, gb.y);
    // w = q M
    ff wr = dot2(qr.hi, m.x, -qi.hi, m.y);
    ff wi = dot2(qr.hi, m.y, qi.hi, m.x);
    wr.lo = __fadd_rn(wr.lo, __fsub_rn(__fmul_rn(qr.lo, m.x), __fmul_rn(qi.lo, m.y)));
    wi.lo = __fadd_rn(wi.lo, __fadd_rn(__fmul_rn(qr.lo, m.y), __fmul_rn(qi.lo, m.x)));
    // R = V - w
    const ff rr = two_sum(v.x, -wr.hi);
    const ff ri = two_sum(v.y, -wi.hi);
    return make_float2(__fadd_rn(rr.hi, __fsub_rn(rr.lo, wr.lo)), __fadd_rn(ri.hi, __fsub_rn(ri.lo, wi.lo)));
}

// v plus the lane's partner's value, the partner at (lane xor OFF) or, for OFF
// = 4 and 8, one that holds the same value after the sums over OFF = 1, 2 (4):
// the butterfly sums over rows of 16 lanes without LDS traffic (a shuffle is
// two ds_bpermute per double).  16 and 32: the row and half exchanges.
template <int OFF>
__device__ __forceinline__ int lane_partner(int v) {
    if constexpr (OFF == 1) return __builtin_amdgcn_mov_dpp(v, 1 | (0 << 2) | (3 << 4) | (2 << 6), 0xF, 0xF, false);
    else if constexpr (OFF == 2) return __builtin_amdgcn_mov_dpp(v, 2 | (3 << 2) | (0 << 4) | (1 << 6), 0xF, 0xF, false);
    else if constexpr (OFF == 4) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    else return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false);                           // row_mirror
}
template <int OFF>
__device__ __forceinline__ double partner_sum(double v) {
    const long long u = __double_as_longlong(v);
    const int lo = (int)u, hi = (int)(u >> 32);
    if constexpr (OFF <= 8) {
        const int plo = lane_partner<OFF>(lo), phi = lane_partner<OFF>(hi);
        return v + __longlong_as_double(((long long)phi << 32) | (unsigned)plo);
    } else {
        // rows 0 and 2 (half 0) of both results hold the one row of the pair,
        // the other result the other: their sum is the pair's in every lane
        unsigned l0, l1, h0, h1;
        if constexpr (OFF == 16) {
            const auto a = __builtin_amdgcn_permlane16_swap((unsigned)lo, (unsigned)lo, false, false);
            const auto b = __builtin_amdgcn_permlane16_swap((unsigned)hi, (unsigned)hi, false, false);
            l0 = a[0], l1 = a[1], h0 = b[0], h1 = b[1];
        } else {
            const auto a = __builtin_amdgcn_permlane32_swap((unsigned)lo, (unsigned)lo, false, false);
            const auto b = __builtin_amdgcn_permlane32_swap((unsigned)hi, (unsigned)hi, false, false);
            l0 = a[0], l1 = a[1], h0 = b[0], h1 = b[1];
        }
        return __longlong_as_double(((long long)h0 << 32) | l0) + __longlong_as_double(((long long)h1 << 32) | l1);
    }
}
__device__ __forceinline__ double row_sum16(double v) {
    return partner_sum<8>(partner_sum<4>(partner_sum<2>(partner_sum<1>(v))));
}

__device__ __forceinline__ float wave_sumf(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ void tile_rc(int t, int& ti, int& tj) {
    int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > t) --r;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    ti = r;
    tj = t - r * (r + 1) / 2;
}

// workspace layout: rowpart, colpart double2 [P][2][n_tiles][64]; loss float
// [P][2][n_tiles]; the solver's rowd, cold double [P][2][n_tiles][64]
//
// Thread (r4, c4) of the tile owns rows 4 r4 .. 4 r4 + 3 and columns c4,
// c4 + 16, c4 + 32, c4 + 48 for both polarisations (a load of 16 lanes
// covers 16 consecutive baselines): a row's 16 column threads are 16
// consecutive lanes (xor-shuffle sum in 4 steps), a column's 16 row threads
// are 4 per wave (2 steps) times 4 waves (LDS).
// kRec: the 32-byte records of V and M are at 16-byte aligned addresses: each element is read as two 16-byte halves,
// (XX, XY) and (YX, YY), which the hardware fetches whole anyway (6% faster
// than two 8-byte loads).
// kW: weighted loss sum_{a,b} w_ab |R_ab|^2 with w from the visibility
// flags fl (uint8 [P][Nbl][2], nonzero = weight 0) and the weights wt (float
// [P][Nbl][2]; either may be NULL): every per-element term (loss, the
// gradient's t = w R conj(M), the solver's w |M|^2) is scaled by w.

__device__ __forceinline__ double norm2(float2 g) { return (double)g.x * g.x + (double)g.y * g.y; }

// One element a >= b: its terms of row a, column b and the loss.  kInner: the
// tile lies off the diagonal (a != b).
template <bool kDiag, bool kInner>
__device__ __forceinline__ void cal_element(float2 v, float2 mm, float wq, float2 ga, float2 gb, double ga2, double gb2,
                                            bool same, double* row, double* col, float& lsum) {
    const float2 R = residual(v, mm, ga, gb);
    if constexpr (!kDiag) {
        const float r2 = wq * (R.x * R.x + R.y * R.y);
        lsum += !kInner && same ? r2 : 2.0f * r2;
    }
    // t = w R conj(M); on the diagonal Re(t) only
    const float tr = wq * (R.x * mm.x + R.y * mm.y);
    const float ti = wq * (R.y * mm.x - R.x * mm.y);
    const float tm = !kInner && same ? 0.0f : ti;
    // row a: t g_b
    row[0] += (double)(tr * gb.x - tm * gb.y);
    row[1] += (double)(tr * gb.y + tm * gb.x);
    if (kInner || !same) {                                     // column b: conj(t) g_a
        col[0] += (double)(tr * ga.x + tm * ga.y);
        col[1] += (double)(tr * ga.y - tm * ga.x);
    }
    if constexpr (kDiag) {
        // |M|^2 |g_b|^2 to row a; |M|^2 |g_a|^2 to column b off the diagonal
        const double m2 = (double)wq * ((double)mm.x * mm.x + (double)mm.y * mm.y);
        row[2] += m2 * gb2;
        if (kInner || !same) col[2] += m2 * ga2;
    }
}

// weights (XX, YY) of the element at index i of the weight arrays
__device__ __forceinline__ float2 element_weight(const uint8_t* fl, const float* wt, int64_t i) {
    const unsigned short fp = fl ? *reinterpret_cast<const unsigned short*>(fl + i) : (unsigned short)0;
    const float2 wp = wt ? *reinterpret_cast<const float2*>(wt + i) : make_float2(1.0f, 1.0f);
    return make_float2((fp & 0xFF) ? 0.0f : wp.x, (fp >> 8) ? 0.0f : wp.y);
}

template <bool kRec, bool kW>
__global__ __launch_bounds__(kThreads) void cal_tiles_kernel(int Na, int P, int n_tiles,
                                                             const float2* __restrict__ V,
                                                             const float2* __restrict__ M, const float2* __restrict__ g,
                                                             double2* __restrict__ rowpart, double2* __restrict__ colpart,
                                                             float* __restrict__ losspart,
                                                             const uint8_t* __restrict__ fl,
                                                             const float* __restrict__ wt) {
    constexpr int NV = 2;                                     // re, im
    __shared__ double col_lds[4][kTileA][2][NV];
    __shared__ float loss_lds[4][2];
    const int t = blockIdx.x, ch = blockIdx.y;
    int ti, tj;
    tile_rc(t, ti, tj);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c4 = tid & 15, r4 = tid >> 4;
    // per-channel bases; element offsets within a channel fit 32 bits (at most
    // 8.4 million baselines of 32 bytes)
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    const float2* Vc = V + (int64_t)ch * nbl * 4;
    const float2* Mc = M + (int64_t)ch * nbl * 4;
    const uint8_t* flc = kW && fl ? fl + (int64_t)ch * nbl * 2 : nullptr;
    const float* wtc = kW && wt ? wt + (int64_t)ch * nbl * 2 : nullptr;
    const float2* gc = g + (int64_t)ch * Na * 2;              // [a][2]

    float2 gb[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int b = tj * kTileA + c4 + 16 * q;
#pragma unroll
        for (int p = 0; p < 2; ++p) gb[q][p] = b < Na ? gc[b * 2 + p] : make_float2(0.0f, 0.0f);
    }
    double col[4][2][NV];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < NV; ++k) col[q][p][k] = 0.0;
    float lsum[2] = {0.0f, 0.0f};
    const int64_t slot0 = ((int64_t)(ch * 2) * n_tiles + t) * kTileA;            // pol 0
    const int64_t slot1 = ((int64_t)(ch * 2 + 1) * n_tiles + t) * kTileA;        // pol 1

#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 4 * r4 + i;
        const int a = ti * kTileA + r;
        float2 ga[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) ga[p] = a < Na ? gc[a * 2 + p] : make_float2(0.0f, 0.0f);
        double row[2][NV];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < NV; ++k) row[p][k] = 0.0;
        // all loads of the row first (clamped to element 0 where the
        // element is outside the triangle; such elements contribute nothing)
        float2 vv[4][2], mv[4][2], ww[4];
        bool ok[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int b = tj * kTileA + c4 + 16 * q;
            ok[q] = a < Na && b < Na && b <= a;
            const unsigned el = ok[q] ? (unsigned)a * (unsigned)(a + 1) / 2u + (unsigned)b : 0u;
            ww[q] = make_float2(1.0f, 1.0f);
            if constexpr (kW) ww[q] = element_weight(flc, wtc, (int64_t)el * 2);
            if constexpr (kRec) {
                const char* ve = reinterpret_cast<const char*>(Vc) + el * 32u;
                const char* me = reinterpret_cast<const char*>(Mc) + el * 32u;
                const float4 v0 = *reinterpret_cast<const float4*>(ve), v1 = *reinterpret_cast<const float4*>(ve + 16);
                const float4 m0 = *reinterpret_cast<const float4*>(me), m1 = *reinterpret_cast<const float4*>(me + 16);
                vv[q][0] = make_float2(v0.x, v0.y);
                vv[q][1] = make_float2(v1.z, v1.w);
                mv[q][0] = make_float2(m0.x, m0.y);
                mv[q][1] = make_float2(m1.z, m1.w);
            } else {
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    vv[q][p] = Vc[el * 4u + 3 * p];
                    mv[q][p] = Mc[el * 4u + 3 * p];
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool same = a == tj * kTileA + c4 + 16 * q;
            if (ok[q]) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    cal_element<false, false>(vv[q][p], mv[q][p], p ? ww[q].y : ww[q].x, ga[p], gb[q][p], 0.0, 0.0, same,
                                              row[p], col[q][p], lsum[p]);
            }
        }
        // row sums over the 16 column threads (consecutive lanes)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < NV; ++k) row[p][k] = row_sum16(row[p][k]);
        if (c4 == 0) {
            rowpart[slot0 + r] = make_double2(row[0][0], row[0][1]);
            rowpart[slot1 + r] = make_double2(row[1][0], row[1][1]);
        }
    }
    // column sums: the 4 row threads of this wave, then the 4 waves
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int k = 0; k < NV; ++k) col[q][p][k] = partner_sum<32>(partner_sum<16>(col[q][p][k]));
    if (lane < 16) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int k = 0; k < NV; ++k) col_lds[wv][c4 + 16 * q][p][k] = col[q][p][k];
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const float l = wave_sumf(lsum[p]);
        if (lane == 0) loss_lds[wv][p] = l;
    }
    __syncthreads();
    if (tid < 2 * kTileA) {
        const int c = tid & (kTileA - 1), p = tid / kTileA;
        const int64_t slot = p ? slot1 : slot0;
        double s[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k)
            s[k] = (col_lds[0][c][p][k] + col_lds[1][c][p][k]) + (col_lds[2][c][p][k] + col_lds[3][c][p][k]);
        colpart[slot + c] = make_double2(s[0], s[1]);
    }
    if (tid < 2) {
        const int p = tid;
        losspart[(int64_t)(ch * 2 + p) * n_tiles + t] = (loss_lds[0][p] + loss_lds[1][p]) + (loss_lds[2][p] + loss_lds[3][p]);
    }
}

// Model of an element for the solver: a flagged element's becomes zero, which
// makes each of its terms zero as a weight of zero does, and the steps then
// read no flags (NaN for a model that is not finite, whose terms times zero are
// NaN).  The zero is -0 + 0 i, which no other element keeps: its weight is
// ignored by it, whatever the weight array holds.  (Reading the flags in every
// step instead: 576 antennas x 64 channels, 20 steps, 2.42 -> 3.03 ms.)
__device__ __forceinline__ float2 solver_model(float2 m, bool flagged) {
    if (!flagged) return make_float2(m.x + 0.0f, m.y);         // (-0 + 0 = 0)
    return fabsf(m.x) < INFINITY && fabsf(m.y) < INFINITY ? make_float2(-0.0f, 0.0f) : make_float2(NAN, NAN);
}
__device__ __forceinline__ float solver_weight(float w, float2 m) {
    return __float_as_uint(m.x) == 0x80000000u ? 0.0f : w;
}

// Tile pass of a solver step: one workgroup per 64 x 64 tile, channel and
// polarisation, on the compact copies of V and M ([P][2][Nbl], flags applied;
// kW: weights wt as well), threads and sums as in cal_tiles_kernel, with the third sum D_a = sum_b w |M_ab|^2
// |g_b|^2 over the full Hermitian matrix (the diagonal of the Gauss-Newton
// normal matrix of the row-wise least-squares problem).  It is bound by its
// vector instructions (the residual's error-free transformations are about
// half of them), so it leaves out the loss, forms |g|^2 once per row and
// column and tests the triangle and the array's edge only in tiles that meet
// them; one polarisation at a time, because the sums of two take the
// registers of a wave per SIMD.
template <bool kW>
__global__ __launch_bounds__(kThreads) void cal_solve_tiles_kernel(int Na, int P, int nT, const float2* __restrict__ V,
                                                                   const float2* __restrict__ M,
                                                                   const float2* __restrict__ g,
                                                                   double2* __restrict__ rowpart,
                                                                   double2* __restrict__ colpart,
                                                                   double* __restrict__ rowd, double* __restrict__ cold,
                                                                   const float* __restrict__ wt, int reverse) {
    __shared__ double col_lds[4][kTileA][3];
    // Whole tiles first, then the array's last rows, then the diagonal (5/8 of
    // the elements): the launch is one to two rounds of workgroups, and the
    // short ones even out its end.  Every second step takes them in the opposite
    // order, on the same XCD (workgroup id modulo 8): what the caches still hold
    // from the end of a step is then the first to be read of the next instead
    // of being pushed out first.  (Together 1043 -> 1009 us for the solve of 288
    // antennas x 64 channels with flagging, 3.15 -> 2.99 ms at 576.)
    const int n8 = (int)gridDim.x >> 3, id8 = (int)blockIdx.x >> 3;
    const int id = reverse && id8 < n8 ? ((n8 - 1 - id8) << 3) | (int)(blockIdx.x & 7) : (int)blockIdx.x;
    const int P2 = 2 * P, k = id / P2, ch = id % P2 >> 1, pol = id & 1;
    const int n_whole = (nT - 1) * (nT - 2) / 2;
    int ti, tj;
    if (k < n_whole) {
        tile_rc(k, ti, tj);
        ++ti;
    } else if (k < n_whole + nT - 1) {
        ti = nT - 1;
        tj = k - n_whole;
    } else {
        ti = tj = k - n_whole - (nT - 1);
    }
    const int t = ti * (ti + 1) / 2 + tj, n_tiles = nT * (nT + 1) / 2;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c4 = tid & 15, r4 = tid >> 4;
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    const float2* Vc = V + (int64_t)(2 * ch + pol) * nbl;
    const float2* Mc = M + (int64_t)(2 * ch + pol) * nbl;
    const float* wtc = kW ? wt + (int64_t)ch * nbl * 2 + pol : nullptr;
    const float2* gc = g + (int64_t)ch * Na * 2 + pol;        // [a][2]
    float2 gb[4];
    double gb2[4], col[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int b = tj * kTileA + c4 + 16 * q;
        gb[q] = b < Na ? gc[b * 2] : make_float2(0.0f, 0.0f);
        gb2[q] = norm2(gb[q]);
#pragma unroll
        for (int k = 0; k < 3; ++k) col[q][k] = 0.0;
    }
    const int64_t slot = ((int64_t)(ch * 2 + pol) * n_tiles + t) * kTileA;
    auto rows = [&](auto inner_tag) {
        constexpr bool kInner = decltype(inner_tag)::value;   // off the diagonal, all rows below Na
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * r4 + i;
            const int a = ti * kTileA + r;
            const float2 ga = kInner || a < Na ? gc[a * 2] : make_float2(0.0f, 0.0f);
            const double ga2 = norm2(ga);
            double row[3] = {0.0, 0.0, 0.0};
            float2 vv[4], mv[4];
            float ww[4];
            bool ok[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = tj * kTileA + c4 + 16 * q;
                ok[q] = kInner || (a < Na && b < Na && b <= a);
                const unsigned el = ok[q] ? (unsigned)a * (unsigned)(a + 1) / 2u + (unsigned)b : 0u;
                ww[q] = 1.0f;
                vv[q] = Vc[el];
                mv[q] = Mc[el];
                if constexpr (kW) ww[q] = solver_weight(wtc[el * 2u], mv[q]);
            }
            float unused = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (ok[q])
                    cal_element<true, kInner>(vv[q], mv[q], ww[q], ga, gb[q], ga2, gb2[q],
                                              a == tj * kTileA + c4 + 16 * q, row, col[q], unused);
#pragma unroll
            for (int k = 0; k < 3; ++k) row[k] = row_sum16(row[k]);
            if (c4 == 0) {
                rowpart[slot + r] = make_double2(row[0], row[1]);
                rowd[slot + r] = row[2];
            }
        }
    };
    if (ti != tj && (ti + 1) * kTileA <= Na) rows(std::true_type{});
    else rows(std::false_type{});
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double c = partner_sum<32>(partner_sum<16>(col[q][k]));
            if (lane < 16) col_lds[wv][c4 + 16 * q][k] = c;
        }
    __syncthreads();
    if (tid < kTileA) {
        double s[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            s[k] = (col_lds[0][tid][k] + col_lds[1][tid][k]) + (col_lds[2][tid][k] + col_lds[3][tid][k]);
        colpart[slot + tid] = make_double2(s[0], s[1]);
        cold[slot + tid] = s[2];
    }
}

__global__ __launch_bounds__(256) void cal_reduce_kernel(int Na, int P, int nT, int n_tiles,
                                                         const double2* __restrict__ rowpart,
                                                         const double2* __restrict__ colpart,
                                                         const float* __restrict__ losspart, double* __restrict__ loss,
                                                         float2* __restrict__ grad) {
    const int ch = blockIdx.y, pol = blockIdx.z;
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t base = (int64_t)(ch * 2 + pol) * n_tiles;
    if (grad && a < Na) {
        const int ta = a / kTileA, ra = a % kTileA;
        double sr = 0.0, si = 0.0;
        for (int tj = 0; tj <= ta; ++tj) {                   // row a: tiles (ta, tj)
            const double2 v = rowpart[(base + ta * (ta + 1) / 2 + tj) * kTileA + ra];
            sr += v.x;
            si += v.y;
        }
        for (int ti = ta; ti < nT; ++ti) {                   // column a: tiles (ti, ta)
            const double2 v = colpart[(base + ti * (ti + 1) / 2 + ta) * kTileA + ra];
            sr += v.x;
            si += v.y;
        }
        grad[((int64_t)ch * Na + a) * 2 + pol] = make_float2((float)(-4.0 * sr), (float)(-4.0 * si));
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        float s = 0.0f;
        for (int t = 0; t < n_tiles; ++t) s += losspart[base + t];
        loss[ch * 2 + pol] = (double)s;
    }
}

int n_tiles_side(int Na) { return (int)ceil_div(Na, kTileA); }

// Remove the common phase of each (channel, polarisation): g_a conj(g_0) / |g_0|.
__device__ __forceinline__ float2 referenced(float2 ga, float2 g0) {
    const double m = sqrt((double)g0.x * g0.x + (double)g0.y * g0.y);
    if (!(m > 0.0)) return ga;
    const double cr = g0.x / m, ci = -(double)g0.y / m;
    return make_float2((float)(ga.x * cr - ga.y * ci), (float)(ga.x * ci + ga.y * cr));
}

// New gain of an antenna from its sums: g - grad / (4 D), which with grad =
// -4 (sum_b V_ab conj(z_ab) - g_a D_a), z_ab = M_ab conj(g_b), is the
// alternating least-squares update sum_b V_ab conj(z_ab) / D_a of each gain
// with all others fixed; on every second iteration the new gain is averaged
// with the previous one.
__device__ __forceinline__ float2 new_gain(float2 gc, double sr, double si, double d, bool average) {
    const float gx = (float)(-4.0 * sr), gy = (float)(-4.0 * si);
    double nr = gc.x, ni = gc.y;
    if (d > 0.0) {
        nr = (double)gc.x - (double)gx / (4.0 * d);
        ni = (double)gc.y - (double)gy / (4.0 * d);
    }
    if (average) {
        nr = 0.5 * (nr + (double)gc.x);
        ni = 0.5 * (ni + (double)gc.y);
    }
    return make_float2((float)nr, (float)ni);
}

// One solver step: the tile partials of every (channel, antenna, polarisation)
// summed in a fixed order and the gain updated, in one kernel (a reduction and
// an update kernel took 6.2 and 4.7 us at 288 antennas x 64 channels).
__global__ __launch_bounds__(64) void cal_step_kernel(int Na, int nT, int n_tiles, const double2* __restrict__ rowpart,
                                                      const double2* __restrict__ colpart,
                                                      const double* __restrict__ rowd, const double* __restrict__ cold,
                                                      const float2* __restrict__ g, float2* __restrict__ g_next,
                                                      int average) {
    const int ch = blockIdx.y, pol = blockIdx.z, ta = blockIdx.x, ra = threadIdx.x;
    const int a = ta * kTileA + ra;
    if (a >= Na) return;
    const int64_t base = (int64_t)(ch * 2 + pol) * n_tiles;
    double sr = 0.0, si = 0.0, sd = 0.0;
#pragma unroll 4
    for (int k = 0; k <= nT; ++k) {
        // row a: tiles (ta, 0 .. ta), then column a: tiles (ta .. nT - 1, ta)
        const bool in_row = k <= ta;
        const int ti = in_row ? ta : k - 1, tj = in_row ? k : ta;
        const int64_t e = (base + ti * (ti + 1) / 2 + tj) * kTileA + ra;
        const double2 v = in_row ? rowpart[e] : colpart[e];
        sr += v.x;
        si += v.y;
        sd += in_row ? rowd[e] : cold[e];
    }
    const int64_t e = ((int64_t)ch * Na + a) * 2 + pol;
    g_next[e] = new_gain(g[e], sr, si, sd, average != 0);
}

// The whole solve of one (channel, polarisation) of at most 128 antennas in
// one workgroup, its tiles' elements held in registers (four waves per tile):
// on small arrays a solve was bound by its launches (94 of them for 30
// iterations).  Sums and their order are those of the tile and step kernels,
// so the gains are the same.
template <bool kW>
__global__ __launch_bounds__(3 * kThreads) void cal_solve_small_kernel(int Na, int n_iter, const float2* __restrict__ V,
                                                                       const float2* __restrict__ M,
                                                                       float2* __restrict__ g,
                                                                       const uint8_t* __restrict__ fl,
                                                                       const float* __restrict__ wt) {
    __shared__ double row_lds[3][kTileA][3], col_lds[3][4][kTileA][3];
    __shared__ float2 gl[2 * kTileA];
    const int ch = blockIdx.x, pol = blockIdx.y;
    const int tid = threadIdx.x, t = tid >> 8, lane = tid & 63, wv = (tid >> 6) & 3;
    const int ti = t == 0 ? 0 : 1, tj = t == 2 ? 1 : 0;        // tiles (0, 0), (1, 0), (1, 1)
    const int nT = blockDim.x > kThreads ? 2 : 1;
    const int c4 = tid & 15, r4 = (tid & 255) >> 4;
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    const float2* Vc = V + (int64_t)ch * nbl * 4 + 3 * pol;
    const float2* Mc = M + (int64_t)ch * nbl * 4 + 3 * pol;
    float2* gc = g + (int64_t)ch * Na * 2 + pol;
    float2 vv[4][4], mv[4][4];
    float ww[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int a = ti * kTileA + 4 * r4 + i, b = tj * kTileA + c4 + 16 * q;
            const bool ok = a < Na && b <= a;
            const int64_t el = ok ? (int64_t)a * (a + 1) / 2 + b : 0;
            vv[i][q] = Vc[el * 4];
            const int64_t wi = ((int64_t)ch * nbl + el) * 2 + pol;
            mv[i][q] = solver_model(Mc[el * 4], fl && fl[wi]);
            ww[i][q] = kW ? solver_weight(wt[wi], mv[i][q]) : 1.0f;
        }
    if (tid < 2 * kTileA) gl[tid] = tid < Na ? gc[(int64_t)tid * 2] : make_float2(0.0f, 0.0f);
    __syncthreads();
    for (int it = 1; it <= n_iter; ++it) {
        float2 gb[4];
        double gb2[4], col[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            gb[q] = gl[tj * kTileA + c4 + 16 * q];
            gb2[q] = norm2(gb[q]);
#pragma unroll
            for (int k = 0; k < 3; ++k) col[q][k] = 0.0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int a = ti * kTileA + 4 * r4 + i;
            const float2 ga = gl[a];
            const double ga2 = norm2(ga);
            double row[3] = {0.0, 0.0, 0.0};
            float unused = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = tj * kTileA + c4 + 16 * q;
                if (a < Na && b <= a)
                    cal_element<true, false>(vv[i][q], mv[i][q], ww[i][q], ga, gb[q], ga2, gb2[q], a == b, row, col[q],
                                             unused);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) row[k] = row_sum16(row[k]);
            if (c4 == 0) {
#pragma unroll
                for (int k = 0; k < 3; ++k) row_lds[t][4 * r4 + i][k] = row[k];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double c = partner_sum<32>(partner_sum<16>(col[q][k]));
                if (lane < 16) col_lds[t][wv][c4 + 16 * q][k] = c;
            }
        __syncthreads();
        if (tid < Na) {
            const int ta = tid / kTileA, ra = tid % kTileA;
            double s[3] = {0.0, 0.0, 0.0};
            for (int k = 0; k <= nT; ++k) {                    // as in cal_step_kernel
                const bool in_row = k <= ta;
                const int si = in_row ? ta : k - 1, sj = in_row ? k : ta, st = si * (si + 1) / 2 + sj;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    s[c] += in_row ? row_lds[st][ra][c]
                                   : (col_lds[st][0][ra][c] + col_lds[st][1][ra][c]) +
                                         (col_lds[st][2][ra][c] + col_lds[st][3][ra][c]);
            }
            gl[tid] = new_gain(gl[tid], s[0], s[1], s[2], it % 2 == 0);
        }
        __syncthreads();
    }
    if (tid < Na) gc[(int64_t)tid * 2] = referenced(gl[tid], gl[0]);
}

__global__ void cal_reference_kernel(int Na, int P, const float2* __restrict__ g, float2* __restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= P * Na * 2) return;
    const int pol = e & 1, ch = e / (2 * Na);
    out[e] = referenced(g[e], g[(int64_t)ch * Na * 2 + pol]);
}

// XX and YY of V and M from [P][Nbl][2][2] into [P][2][Nbl] (one thread per
// channel and baseline), the model zero where flagged (fl or NULL)
__global__ void cal_compact_kernel(int64_t total, int64_t nbl, const float2* __restrict__ V,
                                   const float2* __restrict__ M, const uint8_t* __restrict__ fl,
                                   float2* __restrict__ Vc, float2* __restrict__ Mc) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int64_t ch = e / nbl, bl = e - ch * nbl;
    const float2 xx = M[4 * e], yy = M[4 * e + 3];
    const unsigned short f = fl ? *reinterpret_cast<const unsigned short*>(fl + 2 * e) : (unsigned short)0;
    Vc[2 * ch * nbl + bl] = V[4 * e];                           // XX
    Vc[(2 * ch + 1) * nbl + bl] = V[4 * e + 3];                 // YY
    Mc[2 * ch * nbl + bl] = solver_model(xx, (f & 0xFF) != 0);
    Mc[(2 * ch + 1) * nbl + bl] = solver_model(yy, (f >> 8) != 0);
}

}  // namespace

size_t cal_workspace_bytes(int Na, int P) {
    const int nT = n_tiles_side(Na);
    const size_t n_tiles = (size_t)nT * (nT + 1) / 2;
    return (size_t)P * 2 * n_tiles * (2 * kTileA * sizeof(double2) + sizeof(float)) + 256;
}

// row and column partials of D, two gain buffers, and what callers' workspaces
// have held besides (D, the gradient and the per-iteration loss; the size an
// entry point asks for is part of its interface), rounded up to 256 B
static size_t solver_bytes(int Na, int P) {
    const int nT = n_tiles_side(Na);
    const size_t n_tiles = (size_t)nT * (nT + 1) / 2;
    const size_t n_g = (size_t)P * Na * 2;
    const size_t b = (size_t)P * 2 * n_tiles * kTileA * 2 * sizeof(double) + n_g * (sizeof(double) + 3 * sizeof(float2))
                     + (size_t)P * 2 * sizeof(double);
    return (b + 255) & ~(size_t)255;
}

size_t cal_solve_workspace_bytes(int Na, int P) {
    const size_t nbl = (size_t)Na * (Na + 1) / 2;
    // gradient workspace (rounded up to 256 B), the solver's, and the compact
    // XX / YY copies of V and M
    return ((cal_workspace_bytes(Na, P) + 255) & ~(size_t)255) + solver_bytes(Na, P) + 2 * (size_t)P * 2 * nbl * sizeof(float2);
}

hipError_t launch_calibrate_solve(int Na, int P, const float2* V, const float2* M, float2* g, int n_iter,
                                  double* loss, void* ws, hipStream_t stream, const uint8_t* fl, const float* wt) {
    const int nT = n_tiles_side(Na);
    const int n_tiles = nT * (nT + 1) / 2;
    hipError_t e;
    if (nT <= 2) {
        const dim3 grid((unsigned)P, 2), block((unsigned)(n_tiles * kThreads));
        if (wt)
            hipLaunchKernelGGL(cal_solve_small_kernel<true>, grid, block, 0, stream, Na, n_iter, V, M, g, fl, wt);
        else
            hipLaunchKernelGGL(cal_solve_small_kernel<false>, grid, block, 0, stream, Na, n_iter, V, M, g, fl, wt);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        return loss ? launch_calibrate(Na, P, V, M, g, loss, nullptr, ws, stream, fl, wt) : hipSuccess;
    }
    const size_t n_g = (size_t)P * Na * 2;
    char* w = reinterpret_cast<char*>(ws);
    double2* rowpart = reinterpret_cast<double2*>(w);
    double2* colpart = rowpart + (size_t)P * 2 * n_tiles * kTileA;
    char* w2 = w + ((cal_workspace_bytes(Na, P) + 255) & ~(size_t)255);
    double* rowd = reinterpret_cast<double*>(w2);
    double* cold = rowd + (size_t)P * 2 * n_tiles * kTileA;
    float2* ga = reinterpret_cast<float2*>(cold + (size_t)P * 2 * n_tiles * kTileA);
    float2* gb = ga + n_g;
    // compact XX / YY copies of V and M: every iteration reads only what it
    // uses, contiguously
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    float2* Vc = reinterpret_cast<float2*>(w2 + solver_bytes(Na, P));
    float2* Mc = Vc + (size_t)P * 2 * nbl;
    if (n_iter > 0) {
        const int64_t total = (int64_t)P * nbl;
        hipLaunchKernelGGL(cal_compact_kernel, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, stream, total, nbl,
                           V, M, fl, Vc, Mc);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const float2* gc = g;                                     // the first iteration reads the caller's gains
    if (n_iter == 0) {                                        // (the referencing reads all of them while it writes g)
        e = hipMemcpyAsync(ga, g, n_g * sizeof(float2), hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return e;
        gc = ga;
    }
    for (int it = 1; it <= n_iter; ++it) {
        const dim3 grid((unsigned)(n_tiles * P * 2));
        if (wt)
            hipLaunchKernelGGL(cal_solve_tiles_kernel<true>, grid, dim3(kThreads), 0, stream, Na, P, nT, Vc, Mc, gc,
                               rowpart, colpart, rowd, cold, wt, it % 2 == 0);
        else
            hipLaunchKernelGGL(cal_solve_tiles_kernel<false>, grid, dim3(kThreads), 0, stream, Na, P, nT, Vc, Mc, gc,
                               rowpart, colpart, rowd, cold, nullptr, it % 2 == 0);
        hipLaunchKernelGGL(cal_step_kernel, dim3((unsigned)nT, P, 2), dim3(kTileA), 0, stream, Na, nT, n_tiles, rowpart,
                           colpart, rowd, cold, gc, ga, (int)(it % 2 == 0));
        gc = ga;
        std::swap(ga, gb);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(cal_reference_kernel, dim3((unsigned)ceil_div((int64_t)n_g, 256)), dim3(256), 0, stream, Na, P,
                       gc, g);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (loss) return launch_calibrate(Na, P, V, M, g, loss, nullptr, ws, stream, fl, wt);
    return hipSuccess;
}

// Scratch of the allocation-free gradient entry point: the per-tile partial
// sums (every element read is written earlier in the same call, so nothing
// has to start at zero).  Each GPU the library runs on holds its own copy
// until the process ends.  Host code never passes `cal_scratch` itself to a
// kernel (on the host it names a stand-in, not the device address): it uses
// the address hipGetSymbolAddress returns for the current device.
__device__ __align__(256) unsigned char cal_scratch[kCalScratchBytes];

hipError_t cal_scratch_address(void** out) {
    static std::mutex mu;
    static std::vector<void*> ptrs;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    if ((int)ptrs.size() <= dev) ptrs.resize(dev + 1, nullptr);
    if (!ptrs[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(cal_scratch));
        if (e != hipSuccess) return e;
        ptrs[dev] = p;
    }
    *out = ptrs[dev];
    return hipSuccess;
}

hipError_t launch_calibrate(int Na, int P, const float2* V, const float2* M, const float2* g, double* loss,
                            float2* grad, void* ws, hipStream_t stream, const uint8_t* fl, const float* wt) {
    const int nT = n_tiles_side(Na);
    const int n_tiles = nT * (nT + 1) / 2;
    char* w = reinterpret_cast<char*>(ws);
    double2* rowpart = reinterpret_cast<double2*>(w);
    double2* colpart = rowpart + (size_t)P * 2 * n_tiles * kTileA;
    float* losspart = reinterpret_cast<float*>(colpart + (size_t)P * 2 * n_tiles * kTileA);
    const bool aligned16 = (reinterpret_cast<uintptr_t>(V) | reinterpret_cast<uintptr_t>(M)) % 16 == 0;
    const bool weighted = fl || wt;
#define AFC_CAL_TILES(REC, W)                                                                                    \
    hipLaunchKernelGGL((cal_tiles_kernel<REC, W>), dim3(n_tiles, P), dim3(kThreads), 0, stream, Na, P, n_tiles, V, \
                       M, g, rowpart, colpart, losspart, fl, wt)
    if (aligned16) {
        if (weighted) AFC_CAL_TILES(true, true);
        else AFC_CAL_TILES(true, false);
    } else {
        if (weighted) AFC_CAL_TILES(false, true);
        else AFC_CAL_TILES(false, false);
    }
#undef AFC_CAL_TILES
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(cal_reduce_kernel, dim3((unsigned)ceil_div(Na, 256), P, 2), dim3(256), 0, stream, Na, P, nT,
                       n_tiles, rowpart, colpart, losspart, loss, grad);
    return hipGetLastError();
}

}  // namespace afc
