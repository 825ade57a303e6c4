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
//    the gridded visibilities (every 32nd group of 4 baselines on large arrays,
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
//  * grid_verify_kernel: the totals; should the bound exceed what the scale
//    allows (a sample that missed most of the power), it sets the exact scale
//    and a flag, and a second clearing and gridding, which otherwise end at
//    once, replace the grid.
//  * imaging: (-1)^(p+q) modulation, radix-2 Stockham FFT of each row in LDS,
//    transpose, row FFT again, and (-1)^(i+j) Re(.) / norm with the
//    transpose back.
#include <algorithm>

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
};

// scale of the fixed-point grid, and whether the estimated one was too large
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
// fractions, and whether all eight cells it touches lie inside the grid.
struct Cell {
    int i, j;
    double fu, fv;
    bool ok;
};
__device__ __forceinline__ Cell cell_of(const GridArgs& g, double dx, double dy, double nu) {
    const double s = nu * g.per_hz;
    const double pu = dx * s + 0.5 * g.N, pv = dy * s + 0.5 * g.N;
    const double i0 = floor(pu), j0 = floor(pv);
    Cell c;
    c.ok = i0 >= 1.0 && j0 >= 1.0 && i0 <= g.N - 2.0 && j0 <= g.N - 2.0;
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

// totals of n_part partial sums in a fixed order (one workgroup)
__device__ __forceinline__ Sums total_sums(const Sums* __restrict__ part, int n_part, Sums* lds) {
    Sums s{0.0, 0.0};
    for (int i = threadIdx.x; i < n_part; i += 256) {
        s.a += part[i].a;
        s.w += part[i].w;
    }
    return block_sums<256>(s, lds);
}

// scale = 2^(bits - e) with bound < 2^e
__device__ __forceinline__ double scale_for(double bound, int bits) {
    int e = 0;
    frexp(bound > 0.0 ? bound : 1.0, &e);
    return ldexp(1.0, bits - e);
}

// Scale from the estimate: with a sample, 2^60 for the estimated bound, so that
// the bound may be seven times the estimate; without (stride 1), 2^61.
__global__ __launch_bounds__(256) void grid_scale_kernel(const Sums* __restrict__ part, int n_part, int stride,
                                                         Scale* __restrict__ scale) {
    __shared__ Sums red[4];
    const Sums s = total_sums(part, n_part, red);
    if (threadIdx.x == 0) *scale = Scale{scale_for(s.a * stride, stride > 1 ? 60 : 61), 0, 0};
}

// Totals of the gridding pass: the normalisation, and whether every cell must
// fit 63 bits at the scale used.
__global__ __launch_bounds__(256) void grid_verify_kernel(const Sums* __restrict__ part, int n_part,
                                                          Scale* __restrict__ scale, double* __restrict__ norm) {
    __shared__ Sums red[4];
    const Sums s = total_sums(part, n_part, red);
    if (threadIdx.x == 0) {
        norm[0] = s.w;
        if (s.a * scale->scale >= 0x1.f8p62) *scale = Scale{scale_for(s.a, 61), 1, 0};
    }
}

// clears the grid if the pass has to be repeated
__global__ void grid_clear_kernel(unsigned long long* __restrict__ p, int64_t n, const Scale* __restrict__ scale) {
    if (!scale->redo) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
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

__global__ __launch_bounds__(kGThreads) void grid_kernel(GridArgs g, const Scale* __restrict__ scale_p,
                                                         unsigned long long* __restrict__ grid, int n_split,
                                                         Sums* __restrict__ part, int repeat) {
    __shared__ unsigned long long win[kGW * kGW * 2];
    __shared__ double msum[2];
    __shared__ Sums red[kGThreads / 64];
    if (repeat && !scale_p->redo) return;
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
    __syncthreads();
    const double nu = g.freq[b * kP + kP / 2];
    const double ur = msum[0] * nu * g.per_hz + 0.5 * g.N;
    const double vr = msum[1] * nu * g.per_hz + 0.5 * g.N;
    const int i0w = (int)floor(ur) - kGW / 2, j0w = (int)floor(vr) - kGW / 2;
    const double scale = scale_p->scale;
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

__global__ void twiddle_kernel(float2* __restrict__ tw, int N) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= N / 2) return;
    const double ang = -2.0 * 3.14159265358979323846 * (double)m / (double)N;
    tw[m] = make_float2((float)cos(ang), (float)sin(ang));
}

// Forward DFT of each row of `data` (N points, N a power of two) in place:
// X[k] = sum_n x[n] exp(-2 pi i k n / N).  Radix-2 Stockham: with sub-DFTs
// of size ns done, butterfly j (< N/2) takes x[j] and x[j + N/2], rotates
// the second by exp(-2 pi i (j mod ns) / (2 ns)) and writes the sum and the
// difference to positions (j / ns) 2 ns + j mod ns and that + ns.
// Optional (-1)^(row + column) modulation on load.
__global__ __launch_bounds__(256) void fft_rows_kernel(float2* __restrict__ data, const float2* __restrict__ tw,
                                                       int N, int log2N, int modulate) {
    extern __shared__ float2 buf[];
    float2* x = buf;
    float2* y = buf + N;
    const int row = blockIdx.x;
    float2* r = data + (int64_t)row * N;
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        float2 v = r[i];
        if (modulate && ((row + i) & 1)) v = make_float2(-v.x, -v.y);
        x[i] = v;
    }
    __syncthreads();
    const int half = N / 2;
    for (int l = 0; l < log2N; ++l) {
        const int ns = 1 << l;
        for (int j = threadIdx.x; j < half; j += blockDim.x) {
            const int k = j & (ns - 1);
            const float2 a = x[j];
            const float2 b = cmulf(x[j + half], tw[k << (log2N - 1 - l)]);
            const int o = ((j >> l) << (l + 1)) + k;
            y[o] = make_float2(a.x + b.x, a.y + b.y);
            y[o + ns] = make_float2(a.x - b.x, a.y - b.y);
        }
        __syncthreads();
        float2* t = x;
        x = y;
        y = t;
    }
    for (int i = threadIdx.x; i < N; i += blockDim.x) r[i] = x[i];
}

// out[c][r] = in[r][c] for an N x N float2 matrix; 32 x 32 tiles via LDS.
// finalize: out is float, (-1)^(r+c) Re(in[r][c]) / norm.
template <bool kFinal>
__global__ __launch_bounds__(256) void transpose_kernel(const float2* __restrict__ in, void* __restrict__ out, int N,
                                                        const double* __restrict__ norm_p) {
    __shared__ float2 tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8
    for (int y = ty; y < 32; y += 8) tile[y][tx] = in[(int64_t)(by + y) * N + bx + tx];
    __syncthreads();
    if constexpr (kFinal) {
        const double nv = norm_p[0];
        const float inv = (float)(1.0 / (nv > 0.0 ? nv : 1.0));
        float* o = reinterpret_cast<float*>(out);
        for (int y = ty; y < 32; y += 8) {
            const int orow = bx + y, ocol = by + tx;                   // element in[ocol][orow]
            const float v = tile[tx][y].x * inv;
            o[(int64_t)orow * N + ocol] = ((orow + ocol) & 1) ? -v : v;
        }
    } else {
        float2* o = reinterpret_cast<float2*>(out);
        for (int y = ty; y < 32; y += 8) o[(int64_t)(bx + y) * N + by + tx] = tile[tx][y];
    }
}

}  // namespace

size_t imaging_workspace_bytes(int Na, int B, int N) {
    const int64_t n_cross = (int64_t)Na * (Na - 1) / 2;
    const int64_t n_part = ceil_div(std::max<int64_t>(1, n_cross * B), 256);
    return (size_t)N * N * 16                      // fixed-point grid
           + (size_t)N * N * 8 * 2                 // two float2 planes
           + (size_t)N / 2 * 8                     // twiddles
           + (size_t)n_part * 16 + 64;             // partial sums, scale
}

hipError_t launch_grid(const float2* vis, const int32_t* weights, const double* pos, const double* freq, int Na, int B,
                       int N, double du, float2* grid_out, double* norm, void* ws, hipStream_t stream) {
    const int64_t n_cross = (int64_t)Na * (Na - 1) / 2;
    const int64_t n_thr = std::max<int64_t>(1, n_cross * B);
    const int64_t n_part = ceil_div(n_thr, 256);              // pairs of doubles the workspace holds
    char* w = reinterpret_cast<char*>(ws);
    unsigned long long* fixed = reinterpret_cast<unsigned long long*>(w);
    char* planes = w + (size_t)N * N * 16;                    // the imager's, free here
    Sums* tail = reinterpret_cast<Sums*>(planes + (size_t)N * N * 16 + (size_t)N / 2 * 8);
    Scale* scale = reinterpret_cast<Scale*>(tail + n_part);
    GridArgs g{vis, weights, pos, freq, Na, B, N, 1.0 / (kC * du)};
    const int64_t n_words = (int64_t)N * N * 2;
    // A sample of 1 in 32 costs 3% of a pass over the visibilities; below 2^19
    // baselines (times subbands) it thins out, below 2^15 all are taken.
    const int stride = (int)std::min<int64_t>(32, std::max<int64_t>(1, n_thr >> 14));
    const int64_t n_sample = ceil_div(n_thr, 4 * stride) * 4;
    // workgroups: enough to clear the grid as well; their partial sums lie in
    // the planes (read before the gridding pass writes its own there)
    const int n_est = (int)std::min<int64_t>(std::max<int64_t>(ceil_div(n_sample * (kP / kBatch), 256), n_words / 1024),
                                             std::min<int64_t>((int64_t)N * N, 4096));
    Sums* est = reinterpret_cast<Sums*>(planes);
    hipLaunchKernelGGL(grid_estimate_kernel, dim3(n_est), dim3(256), 0, stream, g, n_cross, n_sample, stride, est, fixed,
                       n_words);
    hipLaunchKernelGGL(grid_scale_kernel, dim3(1), dim3(256), 0, stream, est, n_est, stride, scale);
    const int n_blk = (int)ceil_div(Na, kGB);
    // Channels of a subband in 1, 2 or 4 workgroups: two workgroups run on a
    // CU at a time, and 1.5 rounds of them or more even out (576 antennas x 8
    // subbands 624 workgroups 709 us, 1248 630 us; 96 x 8 24 and 96 workgroups
    // 146 and 81 us for the whole gridding); every part adds its window to the
    // grid, so no more parts than that.
    const int64_t n_pair = (int64_t)n_blk * (n_blk + 1) / 2;
    const int64_t cap = std::max<int64_t>(n_part, (int64_t)N * N);
    int n_split = 1;
    while (n_split < 4 && n_pair * B * n_split < 768 && n_pair * B * n_split * 2 <= cap) n_split *= 2;
    const int64_t n_wg = n_pair * B * n_split;
    Sums* part = n_wg <= n_part ? tail : reinterpret_cast<Sums*>(planes);
    const dim3 grid((unsigned)n_pair, (unsigned)(B * n_split));
    const dim3 cgrid((unsigned)std::min<int64_t>(ceil_div(n_words, 256), 4096));
    hipLaunchKernelGGL(grid_kernel, grid, dim3(kGThreads), 0, stream, g, scale, fixed, n_split, part, 0);
    hipLaunchKernelGGL(grid_verify_kernel, dim3(1), dim3(256), 0, stream, part, (int)n_wg, scale, norm);
    if (stride > 1) {
        hipLaunchKernelGGL(grid_clear_kernel, cgrid, dim3(256), 0, stream, fixed, n_words, scale);
        hipLaunchKernelGGL(grid_kernel, grid, dim3(kGThreads), 0, stream, g, scale, fixed, n_split, part, 1);
    }
    hipLaunchKernelGGL(grid_to_float_kernel, dim3((unsigned)std::min<int64_t>(ceil_div((int64_t)N * N, 256), 4096)),
                       dim3(256), 0, stream, fixed, scale, grid_out, (int64_t)N * N);
    return hipGetLastError();
}

hipError_t launch_image(const float2* grid, const double* norm, float* image, int N, void* ws, hipStream_t stream) {
    int log2N = 0;
    while ((1 << log2N) < N) ++log2N;
    char* w = reinterpret_cast<char*>(ws);
    float2* a = reinterpret_cast<float2*>(w + (size_t)N * N * 16);
    float2* b = a + (size_t)N * N;
    float2* tw = b + (size_t)N * N;
    hipLaunchKernelGGL(twiddle_kernel, dim3((unsigned)ceil_div(N / 2, 256)), dim3(256), 0, stream, tw, N);
    hipError_t e = hipMemcpyAsync(a, grid, (size_t)N * N * sizeof(float2), hipMemcpyDeviceToDevice, stream);
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)2 * N * sizeof(float2);
    const dim3 tgrid((unsigned)(N / 32), (unsigned)(N / 32));
    hipLaunchKernelGGL(fft_rows_kernel, dim3(N), dim3(256), lds, stream, a, tw, N, log2N, 1);
    hipLaunchKernelGGL(transpose_kernel<false>, tgrid, dim3(256), 0, stream, a, b, N, norm);
    hipLaunchKernelGGL(fft_rows_kernel, dim3(N), dim3(256), lds, stream, b, tw, N, log2N, 0);
    hipLaunchKernelGGL(transpose_kernel<true>, tgrid, dim3(256), 0, stream, b, image, N, norm);
    return hipGetLastError();
}

}  // namespace afc
