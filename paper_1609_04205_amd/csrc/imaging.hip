// Gridding and imaging (Sec. "Imaging Pipeline": the calibrated
// visibilities of several subbands are gridded onto one grid with bilinear
// interpolation, which integrates them spectrally, and the grid is Fourier
// transformed into the snapshot image).
//
// Gridding, per cross-correlation a > c of subband b and channel k with
// weight w > 0: I = (XX + YY) / 2 at u = (x_a - x_c) nu / c, v = (y_a - y_c)
// nu / c; (pu, pv) = (u, v) / du + N/2, i0 = floor(pu), fu = pu - i0;
// w I goes to the four cells around (pu, pv) with bilinear weights and
// w conj(I) to the mirrored cells (N - j, N - i) (the point -u, -v).  A
// visibility is gridded only if all eight cells are inside the grid.
//
//  * grid_estimate_kernel: the sum of 2 w (|Re I| + |Im I|) over a sample of
//    the gridded visibilities (every 64th group of 4 baselines on large arrays,
//    all of them on small ones), reduced in a fixed order: an estimate of a
//    bound on any cell, from which the fixed-point scale is taken.
//  * grid_kernel: one workgroup per (subband, part of its channels, pair of
//    48-antenna blocks), one thread per baseline at a time.  Across a subband
//    a baseline's uv point moves by a small fraction of its length, so the
//    thread accumulates the four cells around it in registers (float64) and
//    only adds them when the point enters another cell and at the end: to a 64
//    x 64-cell window in LDS around the blocks' mean separation (added to the
//    grid once per workgroup), or to the grid.  The grid accumulates in 64-bit
//    fixed point: integer atomics make the result independent of the order of
//    the additions, so the grid is bitwise reproducible.  The same pass sums
//    the bound itself and the normalisation.
//  * grid_check_kernel: the totals; should the bound exceed what the scale
//    allows (a sample that missed most of the power) or the scale resolve it
//    to fewer than 60 bits (a sample that met nothing, or an outlier), it sets
//    the exact scale and a flag, and a second clearing and gridding, which
//    otherwise end at once, replace the grid.
//  * imaging: (-1)^(p+q) modulation, FFT of the rows with the transpose in its
//    store, row FFT again, and (-1)^(i+j) Re(.) / norm with the transpose back.
#include <algorithm>
#include <type_traits>

#include "afc_internal.h"

namespace afc {
namespace {

constexpr double kC = 299792458.0;

struct GridArgs {
    const float2* vis;            // [B][64][Nbl][2][2]
    const int32_t* weights;       // [B][Nbl] or nullptr
    const double* pos;            // [Na][2]
    const double* freq;           // [B][64]
    int Na, B, N;
    double per_hz;                // cells per metre and Hz: 1 / (c du)
    double inv_du;
};

// scale of the fixed-point grid, and whether the estimated one did not do
struct Scale {
    double scale;
    int redo, pad;
};

__device__ __forceinline__ void pair_of(int64_t t, int& a, int& c) {
    // t-th cross-correlation in lower-triangle order (a > c): a(a-1)/2 + c
    int x = (int)((sqrt(8.0 * (double)t + 1.0) + 1.0) * 0.5);
    while ((int64_t)x * (x - 1) / 2 > t) --x;
    while ((int64_t)(x + 1) * x / 2 <= t) ++x;
    a = x;
    c = (int)(t - (int64_t)x * (x - 1) / 2);
}

// Grid position of a baseline (dx, dy) at frequency nu: the cell below it, the
// fractions, and whether all eight cells it touches lie inside the grid.  The
// position takes one product with 1 / (c du) instead of a division per
// coordinate; within 1e-9 cells of the grid's edge, where its last bit decides
// on a visibility (regular layouts put points exactly there), it is formed as
// dx nu / c / du.
struct Cell {
    int i, j;
    double fu, fv;
    bool ok;
};
__device__ __forceinline__ Cell cell_of(const GridArgs& g, double dx, double dy, double nu) {
    const double s = nu * g.per_hz, x = dx * s, y = dy * s, edge = 0.5 * g.N - 1.0;
    double pu = x + 0.5 * g.N, pv = y + 0.5 * g.N;
    Cell c;
    c.ok = fabs(x) < edge - 1e-9 && fabs(y) < edge - 1e-9;
    if (!c.ok && fabs(x) < edge + 1e-9 && fabs(y) < edge + 1e-9) {
        pu = dx * nu / kC * g.inv_du + 0.5 * g.N;
        pv = dy * nu / kC * g.inv_du + 0.5 * g.N;
        c.ok = floor(pu) >= 1.0 && floor(pv) >= 1.0 && floor(pu) <= g.N - 2.0 && floor(pv) <= g.N - 2.0;
    }
    const double i0 = floor(pu), j0 = floor(pv);
    c.i = c.ok ? (int)i0 : 0;
    c.j = c.ok ? (int)j0 : 0;
    c.fu = pu - i0;
    c.fv = pv - j0;
    return c;
}

// XX and YY of channels k0 .. k0 + kBatch - 1 of one baseline, all loaded
// before the first is used
constexpr int kBatch = 8;
struct Batch {
    float2 xx[kBatch], yy[kBatch];
};
__device__ __forceinline__ Batch load_batch(const float2* __restrict__ v, int64_t ch_stride, int k0) {
    Batch t;
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
        t.xx[e] = v[(k0 + e) * ch_stride];
        t.yy[e] = v[(k0 + e) * ch_stride + 3];
    }
    return t;
}

// sums of 2 w (|Re I| + |Im I|) and 2 w
struct Sums {
    double a, w;
};
// sums over the workgroup (NT threads), tree-reduced in a fixed order; the
// result in thread 0
template <int NT>
__device__ __forceinline__ Sums block_sums(Sums s, Sums* lds) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s.a += __shfl_xor(s.a, off, 64);
        s.w += __shfl_xor(s.w, off, 64);
    }
    if ((tid & 63) == 0) lds[tid >> 6] = s;
    __syncthreads();
    if (tid == 0)
        for (int v = 1; v < NT / 64; ++v) {
            s.a += lds[v].a;
            s.w += lds[v].w;
        }
    return s;
}

// Sample of the bound and clearing of the grid.  The sample: of every `stride`
// groups of 4 consecutive baselines (4 records share a 128-byte line), all
// subbands in line, one group; a thread takes 8 channels of a baseline.
__global__ __launch_bounds__(256) void grid_estimate_kernel(GridArgs g, int64_t n_cross, int64_t n_sample, int stride,
                                                            Sums* __restrict__ part,
                                                            unsigned long long* __restrict__ grid, int64_t n_words) {
    __shared__ Sums red[4];
    Sums sum{0.0, 0.0};
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, n_thr = (int64_t)gridDim.x * 256;
    for (int64_t t = t0; t < n_sample * (kP / kBatch); t += n_thr) {
        const int k0 = (int)(t / n_sample) * kBatch;
        const int64_t q = t % n_sample, e = q / 4 * 4 * stride + q % 4;
        if (e >= n_cross * g.B) continue;
        const int b = (int)(e / n_cross);
        int a, c;
        pair_of(e % n_cross, a, c);
        const double dx = g.pos[a * 2] - g.pos[c * 2], dy = g.pos[a * 2 + 1] - g.pos[c * 2 + 1];
        const int64_t nbl = (int64_t)g.Na * (g.Na + 1) / 2, bl = (int64_t)a * (a + 1) / 2 + c;
        const double w = g.weights ? (double)g.weights[(int64_t)b * nbl + bl] : 1.0;
        if (w <= 0.0) continue;
        const Batch t8 = load_batch(g.vis + ((int64_t)b * kP * nbl + bl) * 4, nbl * 4, k0);
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            if (!cell_of(g, dx, dy, g.freq[b * kP + k0 + k]).ok) continue;
            sum.a += 2.0 * w * (fabs(0.5 * ((double)t8.xx[k].x + (double)t8.yy[k].x)) +
                                fabs(0.5 * ((double)t8.xx[k].y + (double)t8.yy[k].y)));
        }
    }
    sum = block_sums<256>(sum, red);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
    for (int64_t i = t0; i < n_words; i += n_thr) grid[i] = 0ull;
}

// totals of n_part partial sums in a fixed order (a workgroup of NT threads;
// the result in thread 0)
template <int NT>
__device__ __forceinline__ Sums total_sums(const Sums* __restrict__ part, int n_part, Sums* lds) {
    Sums s{0.0, 0.0};
    for (int i = threadIdx.x; i < n_part; i += NT) {
        s.a += part[i].a;
        s.w += part[i].w;
    }
    return block_sums<NT>(s, lds);
}

// scale = 2^k that takes the exact bound to 2^60 .. 2^61, the estimated one to
// 2^60.5 .. 2^61.5
__device__ __forceinline__ double scale_for(double bound, bool exact) {
    int e = 0;
    const double m = frexp(bound > 0.0 ? bound : 1.0, &e);
    return ldexp(1.0, 61 - e + (!exact && m < 0.70710678118654752440 ? 1 : 0));
}

// Totals of the gridding pass: the normalisation, whether the scale from the
// sample (sampled) took the bound to 2^60 .. 2^63, so that every cell fits 63
// bits and none is held in fewer than with the exact bound, and else the scale
// for a second pass and the grid cleared for it.  The estimate may thus be 0.36
// to 1.4 of the bound; a sample that meets no visibility says nothing about
// it.  Every workgroup adds up the totals for itself, which
// saves a launch (this and the scale in the gridding kernel: 150 antennas x 3
// subbands on 1024^2 75.6 -> 70.6 us, 576 x 8 on 2048^2 702 -> 697).
__global__ __launch_bounds__(256) void grid_check_kernel(const Sums* __restrict__ part, int n_part, bool sampled,
                                                         Scale* __restrict__ scale, double* __restrict__ norm,
                                                         unsigned long long* __restrict__ grid, int64_t n_words) {
    __shared__ Sums red[4];
    __shared__ int redo;
    const Sums s = total_sums<256>(part, n_part, red);
    if (threadIdx.x == 0) {
        Scale next{scale[0].scale, 0, 0};
        const double t = s.a * next.scale;                    // (zero: every cell is; NaN: as with the exact bound)
        if (sampled && t != 0.0 && !(t >= 0x1p60 && t < 0x1.f8p62)) next = Scale{scale_for(s.a, true), 1, 0};
        redo = next.redo;
        if (blockIdx.x == 0) {
            norm[0] = s.w;
            scale[1] = next;
        }
    }
    __syncthreads();
    if (!redo) return;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_words; i += (int64_t)gridDim.x * 256) grid[i] = 0ull;
}

// Gridding work: one workgroup per (subband, pair of 48-antenna blocks; a
// block is one station of the array), so that the baselines of a workgroup
// land in a compact patch of the uv plane.  Cells inside a 64 x 64 window
// around the blocks' mean separation are summed in LDS (64-bit fixed point,
// the same integers as the grid's atomics) and added to the grid once per
// workgroup with their mirrors; cells outside the window (other layouts, a
// patch larger than the window) go to the grid directly.  Integer sums: the
// grid is the same whatever the routing.
constexpr int kGB = 48;                      // antennas per block
constexpr int kGW = 64;                      // LDS window side, cells
constexpr int kGThreads = 1024;

// (a sum that is zero, of flagged data say, adds nothing)
__device__ __forceinline__ void add_fixed(unsigned long long* cell, double v, double scale) {
    if (v != 0.0) atomicAdd(cell, (unsigned long long)llrint(v * scale));
}

// One baseline a > c of subband b, channels k_begin .. k_end - 1: its
// contributions are summed in registers (float64) while its point stays in one
// cell, and the four corners flushed to the LDS window or the grid when it
// leaves the cell and at the end; `sum` takes the bound and the weights.
// (Across a subband a point moves by 0.3% of
// its baseline's length, a cell or two at most; a 3 x 3 window of corners,
// flushed less often, cost three times the vector instructions per visibility.)
__device__ __forceinline__ void grid_baseline(const GridArgs& g, int b, int a, int c, int k_begin, int k_end, double scale,
                                              unsigned long long* __restrict__ grid, unsigned long long* win,
                                              int i0w, int j0w, Sums& sum) {
    const double dx = g.pos[a * 2] - g.pos[c * 2], dy = g.pos[a * 2 + 1] - g.pos[c * 2 + 1];
    const int64_t nbl = (int64_t)g.Na * (g.Na + 1) / 2, bl = (int64_t)a * (a + 1) / 2 + c;
    const double w = g.weights ? (double)g.weights[(int64_t)b * nbl + bl] : 1.0;
    if (w <= 0.0) return;
    const int N = g.N;
    const float2* v = g.vis + ((int64_t)b * kP * nbl + bl) * 4;
    double wr[2][2], wi[2][2];
    int ai = 0, aj = 0;                                       // (0 is no cell of a gridded visibility)
    auto flush = [&]() {
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int i = ai + x, j = aj + y;
                const unsigned li = (unsigned)(i - i0w), lj = (unsigned)(j - j0w);
                if (li < (unsigned)kGW && lj < (unsigned)kGW) {
                    unsigned long long* l = win + (lj * kGW + li) * 2;
                    add_fixed(l, wr[y][x], scale);
                    add_fixed(l + 1, wi[y][x], scale);
                } else {
                    // cells of gridded visibilities: 1 <= i, j <= N-1, mirrors likewise
                    unsigned long long* d = grid + ((int64_t)j * N + i) * 2;
                    unsigned long long* m = grid + ((int64_t)(N - j) * N + (N - i)) * 2;
                    add_fixed(d, wr[y][x], scale);
                    add_fixed(d + 1, wi[y][x], scale);
                    add_fixed(m, wr[y][x], scale);
                    add_fixed(m + 1, -wi[y][x], scale);
                }
            }
    };
    for (int k0 = k_begin; k0 < k_end; k0 += kBatch) {
        const Batch t = load_batch(v, nbl * 4, k0);
#pragma unroll
        for (int e = 0; e < kBatch; ++e) {
            const Cell p = cell_of(g, dx, dy, g.freq[b * kP + k0 + e]);
            if (!p.ok) continue;
            if (p.i != ai || p.j != aj) {
                if (ai) flush();
                ai = p.i;
                aj = p.j;
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x) wr[y][x] = wi[y][x] = 0.0;
            }
            const double re = 0.5 * w * ((double)t.xx[e].x + (double)t.yy[e].x);
            const double im = 0.5 * w * ((double)t.xx[e].y + (double)t.yy[e].y);
            sum.a += 2.0 * (fabs(re) + fabs(im));
            sum.w += 2.0 * w;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const double wy = y ? p.fv : 1.0 - p.fv;
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const double f = (x ? p.fu : 1.0 - p.fu) * wy;
                    wr[y][x] += f * re;
                    wi[y][x] += f * im;
                }
            }
        }
    }
    if (ai) flush();
}

// The scale: from the n_est partial sums of the estimate, which every workgroup
// adds up for itself (2 per thread, no launch of their own; without a sample,
// stride 1, it is the bound); the second pass (repeat) takes scale_p[1].
__global__ __launch_bounds__(kGThreads) void grid_kernel(GridArgs g, const Sums* __restrict__ est, int n_est, int stride,
                                                         Scale* __restrict__ scale_p,
                                                         unsigned long long* __restrict__ grid, int n_split,
                                                         Sums* __restrict__ part, int repeat) {
    __shared__ unsigned long long win[kGW * kGW * 2];
    __shared__ double msum[2], shared_scale;
    __shared__ Sums red[kGThreads / 64];
    if (repeat && !scale_p[1].redo) return;
    const int b = blockIdx.y / n_split;
    const int k_begin = blockIdx.y % n_split * (kP / n_split), k_end = k_begin + kP / n_split;
    int ba, bc;                                               // block pair ba >= bc
    {
        const int t = blockIdx.x;
        int r = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while (r * (r + 1) / 2 > t) --r;
        while ((r + 1) * (r + 2) / 2 <= t) ++r;
        ba = r;
        bc = t - r * (r + 1) / 2;
    }
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int a0 = ba * kGB, c0 = bc * kGB;
    const int nA = min(kGB, g.Na - a0), nC = min(kGB, g.Na - c0);
    for (int e = tid; e < kGW * kGW * 2; e += kGThreads) win[e] = 0ull;
    // window origin: the mean separation of the two blocks at the subband's
    // middle channel (wave 0 sums the positions)
    if (wv == 0) {
        double sx = 0.0, sy = 0.0, tx = 0.0, ty = 0.0;
        if (lane < nA) {
            sx = g.pos[(a0 + lane) * 2];
            sy = g.pos[(a0 + lane) * 2 + 1];
        }
        if (lane < nC) {
            tx = g.pos[(c0 + lane) * 2];
            ty = g.pos[(c0 + lane) * 2 + 1];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            sx += __shfl_xor(sx, off, 64);
            sy += __shfl_xor(sy, off, 64);
            tx += __shfl_xor(tx, off, 64);
            ty += __shfl_xor(ty, off, 64);
        }
        if (lane == 0) {
            msum[0] = sx / nA - tx / nC;
            msum[1] = sy / nA - ty / nC;
        }
    }
    if (!repeat) {
        const Sums s = total_sums<kGThreads>(est, n_est, red);
        if (tid == 0) {
            shared_scale = scale_for(s.a * stride, stride == 1);
            if (blockIdx.x == 0 && blockIdx.y == 0) scale_p[0] = Scale{shared_scale, 0, 0};
        }
    } else if (tid == 0) {
        shared_scale = scale_p[1].scale;
    }
    __syncthreads();
    const double nu = g.freq[b * kP + kP / 2];
    const double ur = msum[0] * nu * g.per_hz + 0.5 * g.N;
    const double vr = msum[1] * nu * g.per_hz + 0.5 * g.N;
    const int i0w = (int)floor(ur) - kGW / 2, j0w = (int)floor(vr) - kGW / 2;
    const double scale = shared_scale;
    Sums sum{0.0, 0.0};

    const int n_bl = ba == bc ? nA * (nA - 1) / 2 : nA * nC;
    for (int q = tid; q < n_bl; q += kGThreads) {
        int a, c;
        if (ba == bc) {
            pair_of(q, a, c);
            a += a0;
            c += c0;
        } else {
            a = a0 + q / nC;
            c = c0 + q % nC;
        }
        grid_baseline(g, b, a, c, k_begin, k_end, scale, grid, win, i0w, j0w, sum);
    }
    sum = block_sums<kGThreads>(sum, red);                    // (its barrier also completes the window)
    if (tid == 0 && !repeat) part[blockIdx.y * gridDim.x + blockIdx.x] = sum;
    const int N = g.N;
    for (int e = tid; e < kGW * kGW; e += kGThreads) {
        const long long re = (long long)win[e * 2], im = (long long)win[e * 2 + 1];
        if (re == 0 && im == 0) continue;
        // nonzero cells are cells of gridded visibilities: 1 <= i, j <= N-1
        const int i = i0w + e % kGW, j = j0w + e / kGW;
        unsigned long long* d = grid + ((int64_t)j * N + i) * 2;
        unsigned long long* m = grid + ((int64_t)(N - j) * N + (N - i)) * 2;
        if (re != 0) {
            atomicAdd(d, (unsigned long long)re);
            atomicAdd(m, (unsigned long long)re);
        }
        if (im != 0) {
            atomicAdd(d + 1, (unsigned long long)im);
            atomicAdd(m + 1, (unsigned long long)(-im));
        }
    }
}

// fixed point -> float2 grid (un-normalised), as the gridding's output
__global__ void grid_to_float_kernel(const unsigned long long* __restrict__ grid, const Scale* __restrict__ scale_p,
                                     float2* __restrict__ out, int64_t n) {
    const double inv = 1.0 / scale_p->scale;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const long long re = (long long)grid[i * 2], im = (long long)grid[i * 2 + 1];
        out[i] = make_float2((float)((double)re * inv), (float)((double)im * inv));
    }
}

// ---------------------------------------------------------------- FFT
__device__ __forceinline__ float2 cmulf(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }         // -i a

// R-point DFT in place, natural order, R = 2, 4 or 8
template <int R>
__device__ __forceinline__ void dft(float2 (&x)[R]) {
    if constexpr (R == 2) {
        const float2 t = x[0];
        x[0] = cadd(t, x[1]);
        x[1] = csub(t, x[1]);
    } else if constexpr (R == 4) {
        const float2 a = cadd(x[0], x[2]), b = csub(x[0], x[2]), c = cadd(x[1], x[3]), d = mul_mi(csub(x[1], x[3]));
        x[0] = cadd(a, c);
        x[1] = cadd(b, d);
        x[2] = csub(a, c);
        x[3] = csub(b, d);
    } else {
        constexpr float r2 = 0.70710678118654752440f;   // sqrt(1/2)
        float2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        dft<4>(e);
        dft<4>(o);
        o[1] = make_float2(r2 * (o[1].x + o[1].y), r2 * (o[1].y - o[1].x));
        o[2] = mul_mi(o[2]);
        o[3] = make_float2(r2 * (o[3].y - o[3].x), -r2 * (o[3].x + o[3].y));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = cadd(e[k], o[k]);
            x[k + 4] = csub(e[k], o[k]);
        }
    }
}

// Rows per workgroup of the N-point transform: enough that the transposed
// store writes 64 bytes (2048 points; 156 KB of LDS) and a workgroup has at
// least one wave, few enough that 256 workgroups result where N allows.
template <int N>
constexpr int fft_rows() { return N >= 4096 ? 2 : N >= 2048 ? 8 : N >= 512 ? 4 : N >= 128 ? 1024 / N : 32; }
constexpr int kFftPer = 16;                      // points per thread

// Forward DFT of rows, X[k] = sum_n x[n] exp(-2 pi i n k / N), with the
// transpose fused into the store: out[k][row].  Stockham passes of radix 8
// (the last 4 or 2) over registers and one LDS buffer: with sub-DFTs of size
// ns done, butterfly j takes x[j + r N / R], rotates it by exp(-2 pi i r (j mod
// ns) / (R ns)) and writes its outputs to (j / ns) R ns + j mod ns + r ns.
// kFirst: input the gridding's grid, modulated by (-1)^(row + column), output
// float2; otherwise output float, (-1)^(row + k) Re(.) / norm.  Bound by the
// memory traffic and by latency: 2048^2 takes 44 us for both transforms (five
// passes over 32 MB); radix-2 passes, twiddles, transposes and a copy in
// launches of their own took 111 us.
template <int N, bool kFirst>
__global__ __launch_bounds__(fft_rows<N>() * N / kFftPer) void fft_kernel(const float2* __restrict__ in,
                                                                          void* __restrict__ out,
                                                                          const double* __restrict__ norm_p) {
    constexpr int kRows = fft_rows<N>(), kThr = kRows * N / kFftPer;
    // one element of padding per 8, so that butterflies' stores (8 elements
    // apart) meet all banks; rows 8 elements apart, for the transposed reads
    constexpr int kRS = N + N / 8 + 8;
    __shared__ float2 buf[kRows * kRS];
    __shared__ float2 tw[N / 2];
    const int tid = threadIdx.x;
    // rows of one XCD are neighbours, whose stores share lines
    const int per = gridDim.x / 8;
    const int w = per ? (int)((blockIdx.x & 7) * per + (blockIdx.x >> 3)) : (int)blockIdx.x;
    const int row0 = w * kRows;
    auto at = [](int row, int i) { return row * kRS + i + (i >> 3); };
    for (int m = tid; m < N / 2; m += kThr) {
        double sn, cs;
        sincospi(-2.0 * (double)m / (double)N, &sn, &cs);
        tw[m] = make_float2((float)cs, (float)sn);
    }
    auto pass = [&](auto r_tag, int ns, bool first) {
        constexpr int R = decltype(r_tag)::value, kB = kFftPer / R;
        float2 v[kB][R];
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int id = tid + b * kThr, row = id / (N / R), j = id % (N / R);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = j + r * (N / R);
                if (first) {
                    float2 x = in[(int64_t)(row0 + row) * N + i];
                    if (kFirst && ((row0 + row + i) & 1)) x = make_float2(-x.x, -x.y);
                    v[b][r] = x;
                } else {
                    v[b][r] = buf[at(row, i)];
                }
            }
        }
        __syncthreads();                                      // all reads done (and, first, the twiddles written)
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int id = tid + b * kThr, row = id / (N / R), j = id % (N / R), k = j & (ns - 1);
            if (!first) {
                const int step = k * (N / R / ns);
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    const int m = r * step;                   // below N
                    const float2 t = tw[m & (N / 2 - 1)];
                    v[b][r] = cmulf(v[b][r], m & (N / 2) ? make_float2(-t.x, -t.y) : t);
                }
            }
            dft<R>(v[b]);
            const int o = (j - k) * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r) buf[at(row, o + r * ns)] = v[b][r];
        }
        __syncthreads();
    };
    constexpr int kLog = __builtin_ctz(N);
    using R8 = std::integral_constant<int, 8>;
    pass(R8{}, 1, true);
    int ns = 8;
#pragma unroll
    for (int p = 1; p < kLog / 3; ++p, ns *= 8) pass(R8{}, ns, false);
    if constexpr (kLog % 3 == 1) pass(std::integral_constant<int, 2>{}, ns, false);
    if constexpr (kLog % 3 == 2) pass(std::integral_constant<int, 4>{}, ns, false);
    float inv = 1.0f;
    if constexpr (!kFirst) {
        const double nv = norm_p[0];
        inv = (float)(1.0 / (nv > 0.0 ? nv : 1.0));
    }
#pragma unroll
    for (int e = 0; e < kFftPer; ++e) {
        const int id = tid + e * kThr, row = id % kRows, k = id / kRows;
        const float2 v = buf[at(row, k)];
        const int64_t o = (int64_t)k * N + row0 + row;
        if constexpr (kFirst) {
            reinterpret_cast<float2*>(out)[o] = v;
        } else {
            const float f = v.x * inv;
            reinterpret_cast<float*>(out)[o] = ((k + row0 + row) & 1) ? -f : f;
        }
    }
}

template <int N>
hipError_t launch_fft2(const float2* grid, const double* norm, float* image, float2* plane, hipStream_t stream) {
    constexpr int kRows = fft_rows<N>(), kThr = kRows * N / kFftPer;
    static_assert(N % kRows == 0 && kThr >= 64 && kThr <= 1024, "rows per workgroup");
    hipLaunchKernelGGL((fft_kernel<N, true>), dim3(N / kRows), dim3(kThr), 0, stream, grid, (void*)plane, nullptr);
    hipLaunchKernelGGL((fft_kernel<N, false>), dim3(N / kRows), dim3(kThr), 0, stream, plane, (void*)image, norm);
    return hipGetLastError();
}

}  // namespace

size_t imaging_workspace_bytes(int Na, int B, int N) {
    const int64_t n_cross = (int64_t)Na * (Na - 1) / 2;
    const int64_t n_part = ceil_div(std::max<int64_t>(1, n_cross * B), 256);
    return (size_t)N * N * 16                      // fixed-point grid
           + (size_t)N * N * 8                     // the imager's plane
           + (size_t)N * N * 8 + (size_t)N / 2 * 8 // partial sums of the gridding, and room that callers' workspaces
                                                   // have held besides (the size is part of the interface)
           + (size_t)n_part * 16 + 64;             // partial sums, two scales
}

hipError_t launch_grid(const float2* vis, const int32_t* weights, const double* pos, const double* freq, int Na, int B,
                       int N, double du, float2* grid_out, double* norm, void* ws, hipStream_t stream) {
    const int64_t n_cross = (int64_t)Na * (Na - 1) / 2;
    const int64_t n_thr = std::max<int64_t>(1, n_cross * B);
    const int64_t n_part = ceil_div(n_thr, 256);              // pairs of doubles the workspace holds
    char* w = reinterpret_cast<char*>(ws);
    unsigned long long* fixed = reinterpret_cast<unsigned long long*>(w);
    // partial sums: behind the imager's plane (an image may be formed from the
    // last grid in the same workspace meanwhile) and in the workspace's tail
    Sums* est = reinterpret_cast<Sums*>(w + (size_t)N * N * 24);
    Sums* tail = reinterpret_cast<Sums*>(w + (size_t)N * N * 32 + (size_t)N / 2 * 8);
    Scale* scale = reinterpret_cast<Scale*>(tail + n_part);
    GridArgs g{vis, weights, pos, freq, Na, B, N, 1.0 / (kC * du), 1.0 / du};
    const int64_t n_words = (int64_t)N * N * 2;
    // 1 in 64 of the baselines (times subbands), from 2^19 of them on, of the
    // fewer at least 2^13, below 2^14 all.  At 576 antennas x 8 subbands the
    // sample's scattered lines and the clearing take 30 us; 1 in 32 48 us, 1 in
    // 128 23 us.
    const int stride = (int)std::min<int64_t>(64, std::max<int64_t>(1, n_thr >> 13));
    const int64_t n_sample = ceil_div(n_thr, 4 * stride) * 4;
    // workgroups: enough to clear the grid as well; their partial sums take the
    // first half of the room behind the plane
    const int64_t half = (int64_t)N * N / 4;
    const int n_est = (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n_sample * (kP / kBatch), 256), n_words / 1024),
                                             std::min<int64_t>(half, 2048));
    hipLaunchKernelGGL(grid_estimate_kernel, dim3(n_est), dim3(256), 0, stream, g, n_cross, n_sample, stride, est, fixed,
                       n_words);
    const int n_blk = (int)ceil_div(Na, kGB);
    // Channels of a subband in 1, 2 or 4 workgroups: two workgroups run on a
    // CU at a time, and 1.5 rounds of them or more even out (576 antennas x 8
    // subbands 624 workgroups 709 us, 1248 630 us; 96 x 8 24 and 96 workgroups
    // 146 and 81 us for the whole gridding); every part adds its window to the
    // grid, so no more parts than that.
    const int64_t n_pair = (int64_t)n_blk * (n_blk + 1) / 2;
    // (the sums of the parts lie in the tail of the workspace, or, more than it
    // holds, in the second half of the room behind the plane, 256 or more:
    // without a split at most one per subband, that is)
    const int64_t cap = std::max<int64_t>(n_part, half);
    int n_split = 1;
    while (n_split < 4 && n_pair * B * n_split < 768 && n_pair * B * n_split * 2 <= cap) n_split *= 2;
    const int64_t n_wg = n_pair * B * n_split;
    Sums* part = n_wg <= n_part ? tail : est + half;
    const dim3 grid((unsigned)n_pair, (unsigned)(B * n_split));
    hipLaunchKernelGGL(grid_kernel, grid, dim3(kGThreads), 0, stream, g, est, n_est, stride, scale, fixed, n_split,
                       part, 0);
    // (without a sample the bound is the estimate: no second pass, nothing to clear)
    hipLaunchKernelGGL(grid_check_kernel, dim3(stride > 1 ? 512 : 1), dim3(256), 0, stream, part, (int)n_wg, stride > 1,
                       scale, norm, fixed, n_words);
    if (stride > 1)
        hipLaunchKernelGGL(grid_kernel, grid, dim3(kGThreads), 0, stream, g, est, n_est, stride, scale, fixed, n_split,
                           part, 1);
    hipLaunchKernelGGL(grid_to_float_kernel, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)N * N, 256), 4096)),
                       dim3(256), 0, stream, fixed, scale + 1, grid_out, (int64_t)N * N);
    return hipGetLastError();
}

hipError_t launch_image(const float2* grid, const double* norm, float* image, int N, void* ws, hipStream_t stream) {
    float2* plane = reinterpret_cast<float2*>(reinterpret_cast<char*>(ws) + (size_t)N * N * 16);
    switch (N) {
        case 32: return launch_fft2<32>(grid, norm, image, plane, stream);
        case 64: return launch_fft2<64>(grid, norm, image, plane, stream);
        case 128: return launch_fft2<128>(grid, norm, image, plane, stream);
        case 256: return launch_fft2<256>(grid, norm, image, plane, stream);
        case 512: return launch_fft2<512>(grid, norm, image, plane, stream);
        case 1024: return launch_fft2<1024>(grid, norm, image, plane, stream);
        case 2048: return launch_fft2<2048>(grid, norm, image, plane, stream);
        case 4096: return launch_fft2<4096>(grid, norm, image, plane, stream);
        default: return hipErrorInvalidValue;                 // refused by the entry point
    }
}

}  // namespace afc
