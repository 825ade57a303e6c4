// Real-time flagging by sigma clipping (Sec. "Calibration Pipeline",
// flagging: visibility amplitudes are clipped against a threshold above the
// locally computed RMS, first across the visibilities of a channel, then
// across the channels of each visibility), on the XX and YY correlations.
//
//   stage 1, per (channel, pol):  RMS^2 = mean over cross-correlations of
//            |V|^2; flag |V|^2 > k^2 RMS^2
//   stage 2, per (baseline, pol): RMS^2 = mean over the channels not flagged
//            in stage 1; flag the channels with |V|^2 > k^2 RMS^2
// Autocorrelations are neither used nor flagged.  |V|^2 is formed in float64
// (exact products of the float32 components); every sum runs in a fixed
// order, so the flags are reproducible.
#include "afc_internal.h"

namespace afc {
namespace {

constexpr int kClipChunk = 4096;   // baselines per partial sum of stage 1
constexpr int kClipBl = 64;         // baselines per workgroup of the flagging pass
constexpr int kClipG = 8;           // channel groups per workgroup of the flagging pass
constexpr int kClipHeld = 8;        // channels a thread can hold: 64 channels in all

// whether bl = a(a+1)/2 + b has a = b, bl = a(a+3)/2 (bl < 2^23: 4096 antennas;
// the float32 root is within one of a)
__device__ __forceinline__ bool is_auto(int bl) {
    const int r = (int)((sqrtf(8.0f * (float)bl + 9.0f) - 3.0f) * 0.5f);
    bool hit = false;
#pragma unroll
    for (int d = -1; d <= 1; ++d) hit = hit || (r + d >= 0 && (r + d) * (r + d + 3) / 2 == bl);
    return hit;
}

__device__ __forceinline__ double abs2(float2 v) { return (double)v.x * v.x + (double)v.y * v.y; }

__global__ __launch_bounds__(256) void clip_partial_kernel(int nbl, const float2* __restrict__ V,
                                                           double* __restrict__ part, int n_chunks) {
    __shared__ double red[2][256];
    const int c = blockIdx.x, ch = blockIdx.y, tid = threadIdx.x;
    const int bl0 = c * kClipChunk, bl1 = min(nbl, bl0 + kClipChunk);
    const float2* v = V + (int64_t)ch * nbl * 4;
    double xx = 0.0, yy = 0.0;
#pragma unroll 4
    for (int bl = bl0 + tid; bl < bl1; bl += 256) {
        const float2 x = v[(int64_t)bl * 4], y = v[(int64_t)bl * 4 + 3];
        if (!is_auto(bl)) {
            xx += abs2(x);
            yy += abs2(y);
        }
    }
    red[0][tid] = xx;
    red[1][tid] = yy;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
            red[0][tid] += red[0][tid + s];
            red[1][tid] += red[1][tid + s];
        }
        __syncthreads();
    }
    if (tid < 2) part[(int64_t)(ch * 2 + tid) * n_chunks + c] = red[tid][0];
}

__global__ void clip_mean_kernel(int P, int n_chunks, int64_t n_cross, const double* __restrict__ part,
                                 double* __restrict__ mean) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= P * 2) return;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < n_chunks; ++c) s += part[(int64_t)e * n_chunks + c];
    mean[e] = n_cross > 0 ? s / (double)n_cross : 0.0;
}

// Both stages for 64 baselines: thread (baseline, group g) takes the channels
// g, g + 8, ..., both polarisations; stage 1 as they are read, the baseline's
// mean over the channels that pass it by a sum over the groups, stage 2 and the
// flags.  kHeld (up to 64 channels): the |V|^2 stay in registers, so that V is
// read once (a flag pass, and one thread per baseline and polarisation that
// read V and the flags twice, took 14 + 60 us at 288 antennas x 64 channels
// against 25 us); otherwise V is read again for stage 2.
template <bool kHeld>
__global__ __launch_bounds__(kClipBl* kClipG) void clip_flags_kernel(int P, int nbl, const float2* __restrict__ V,
                                                                     const double* __restrict__ mean, double k2,
                                                                     uint8_t* __restrict__ flags) {
    __shared__ double sum[kClipG][2][kClipBl];
    __shared__ int cnt[kClipG][2][kClipBl];
    const int lane = threadIdx.x % kClipBl, g = threadIdx.x / kClipBl;
    const int bl = blockIdx.x * kClipBl + lane;
    const bool live = bl < nbl;
    const float2* v = V + (int64_t)(live ? bl : 0) * 4;
    const int64_t ch_stride = (int64_t)nbl * 4;
    uint8_t* f = flags + (int64_t)bl * 2;
    const bool au = is_auto(bl);
    double s[2] = {0.0, 0.0};
    int n[2] = {0, 0};
    // stage 1 of one channel
    auto first = [&](int ch, double (&a2)[2], bool (&hit)[2]) {
        a2[0] = abs2(v[ch * ch_stride]);
        a2[1] = abs2(v[ch * ch_stride + 3]);
#pragma unroll
        for (int p = 0; p < 2; ++p) hit[p] = !au && a2[p] > k2 * mean[ch * 2 + p];
    };
    auto store = [&](int ch, bool x, bool y) {
        if (live) {
            f[(int64_t)ch * nbl * 2] = x ? 1 : 0;
            f[(int64_t)ch * nbl * 2 + 1] = y ? 1 : 0;
        }
    };
    double a2[kHeld ? kClipHeld : 1][2];
    bool hit[kHeld ? kClipHeld : 1][2];
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kClipHeld; ++c) first(min(g + c * kClipG, P - 1), a2[c], hit[c]);
    }
    auto add = [&](const double (&a)[2], const bool (&h)[2]) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
            if (!h[p]) {
                s[p] += a[p];
                ++n[p];
            }
    };
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kClipHeld; ++c)
            if (g + c * kClipG < P) add(a2[c], hit[c]);
    } else {
        for (int ch = g; ch < P; ch += kClipG) {
            first(ch, a2[0], hit[0]);
            add(a2[0], hit[0]);
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        sum[g][p][lane] = s[p];
        cnt[g][p][lane] = n[p];
    }
    __syncthreads();
    double limit[2];
    bool any[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        double t = 0.0;
        int m = 0;
#pragma unroll
        for (int q = 0; q < kClipG; ++q) {
            t += sum[q][p][lane];
            m += cnt[q][p][lane];
        }
        any[p] = !au && m > 0;
        limit[p] = any[p] ? k2 * (t / (double)m) : 0.0;
    }
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kClipHeld; ++c)
            if (g + c * kClipG < P)
                store(g + c * kClipG, hit[c][0] || (any[0] && a2[c][0] > limit[0]),
                      hit[c][1] || (any[1] && a2[c][1] > limit[1]));
    } else {
        for (int ch = g; ch < P; ch += kClipG) {
            first(ch, a2[0], hit[0]);
            store(ch, hit[0][0] || (any[0] && a2[0][0] > limit[0]), hit[0][1] || (any[1] && a2[0][1] > limit[1]));
        }
    }
}

__global__ void apply_flags_kernel(int64_t n, const uint8_t* __restrict__ flags, float2* __restrict__ V,
                                   float2* __restrict__ M) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
#pragma unroll
    for (int pol = 0; pol < 2; ++pol)
        if (flags[e * 2 + pol]) {
            if (V) V[e * 4 + pol * 3] = make_float2(0.0f, 0.0f);
            if (M) M[e * 4 + pol * 3] = make_float2(0.0f, 0.0f);
        }
}

int clip_chunks(int64_t nbl) { return (int)ceil_div(nbl, kClipChunk); }

}  // namespace

size_t sigma_clip_workspace_bytes(int Na, int P) {
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    return ((size_t)P * 2 * clip_chunks(nbl) + (size_t)P * 2) * sizeof(double);
}

hipError_t launch_sigma_clip(int Na, int P, const float2* V, float k, uint8_t* flags, void* ws, hipStream_t stream) {
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    const int nc = clip_chunks(nbl);
    double* part = reinterpret_cast<double*>(ws);
    double* mean = part + (size_t)P * 2 * nc;
    const double k2 = (double)k * (double)k;
    hipLaunchKernelGGL(clip_partial_kernel, dim3(nc, P), dim3(256), 0, stream, (int)nbl, V, part, nc);
    hipLaunchKernelGGL(clip_mean_kernel, dim3((unsigned)ceil_div(P * 2, 64)), dim3(64), 0, stream, P, nc,
                       nbl - Na, part, mean);
    const dim3 grid((unsigned)ceil_div(nbl, kClipBl)), block(kClipBl * kClipG);
    if (P <= kClipG * kClipHeld)
        hipLaunchKernelGGL(clip_flags_kernel<true>, grid, block, 0, stream, P, (int)nbl, V, mean, k2, flags);
    else
        hipLaunchKernelGGL(clip_flags_kernel<false>, grid, block, 0, stream, P, (int)nbl, V, mean, k2, flags);
    return hipGetLastError();
}

hipError_t launch_apply_vis_flags(int Na, int P, const uint8_t* flags, float2* V, float2* M, hipStream_t stream) {
    const int64_t n = (int64_t)P * Na * (Na + 1) / 2;
    hipLaunchKernelGGL(apply_flags_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, stream, n, flags, V, M);
    return hipGetLastError();
}

}  // namespace afc
