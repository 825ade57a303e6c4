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
constexpr int kClipThreads = 512;   // of the flagging pass

// whether bl = a(a+1)/2 + b has a = b, bl = a(a+3)/2 (bl < 4096 * 4097 / 2; the
// float32 root is within one of a)
__device__ __forceinline__ bool is_auto(int bl) {
    const int r = (int)((sqrtf(8.0f * (float)bl + 9.0f) - 3.0f) * 0.5f);
    bool hit = false;
#pragma unroll
    for (int d = -1; d <= 1; ++d) hit = hit || (r + d >= 0 && (r + d) * (r + d + 3) / 2 == bl);
    return hit;
}

__device__ __forceinline__ double abs2(float2 v) { return (double)v.x * v.x + (double)v.y * v.y; }

// Partial sums of stage 1: a workgroup per chunk and channel.  kAll: all loads
// of a thread in flight (baselines past the last repeat it and are not added).
template <bool kAll>
__global__ __launch_bounds__(256) void clip_partial_kernel(int nbl, const float2* __restrict__ V,
                                                           double* __restrict__ part, int n_chunks) {
    __shared__ double red[2][256];
    const int c = blockIdx.x, ch = blockIdx.y, tid = threadIdx.x;
    const int bl0 = c * kClipChunk, bl1 = min(nbl, bl0 + kClipChunk);
    const float2* v = V + (int64_t)ch * nbl * 4;
    double xx = 0.0, yy = 0.0;
    auto add = [&](int bl, float2 x, float2 y) {
        if (!is_auto(bl)) {
            xx += abs2(x);
            yy += abs2(y);
        }
    };
    if constexpr (kAll) {
        constexpr int kPer = kClipChunk / 256;
        float2 x[kPer], y[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t bl = min(bl0 + k * 256 + tid, bl1 - 1);
            x[k] = v[bl * 4];
            y[k] = v[bl * 4 + 3];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (bl0 + k * 256 + tid < bl1) add(bl0 + k * 256 + tid, x[k], y[k]);
    } else {
#pragma unroll 4
        for (int bl = bl0 + tid; bl < bl1; bl += 256) add(bl, v[(int64_t)bl * 4], v[(int64_t)bl * 4 + 3]);
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

// Both stages for kBl baselines: thread (baseline, group g of kG) takes the
// channels g, g + kG, ..., both polarisations; stage 1 as they are read, the
// baseline's mean over the channels that pass it by a sum over the groups, stage
// 2 and the flags.  kH: channels a thread holds, so that V is read once (a flag
// pass, and one thread per baseline and polarisation that read V and the flags
// twice, took 14 + 60 us at 288 antennas x 64 channels against 25 us); 0: V is
// read again for stage 2.
template <int kG, int kH>
__global__ __launch_bounds__(kClipThreads) void clip_flags_kernel(int P, int nbl, const float2* __restrict__ V,
                                                                  const double* __restrict__ mean, double k2,
                                                                  uint8_t* __restrict__ flags) {
    constexpr int kBl = kClipThreads / kG;
    constexpr bool kHeld = kH > 0;
    __shared__ double sum[kG][2][kBl];
    __shared__ int cnt[kG][2][kBl];
    const int lane = threadIdx.x % kBl, g = threadIdx.x / kBl;
    const int bl = blockIdx.x * kBl + lane;
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
    double a2[kHeld ? kH : 1][2];
    bool hit[kHeld ? kH : 1][2];
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kH; ++c) first(min(g + c * kG, P - 1), a2[c], hit[c]);
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
        for (int c = 0; c < kH; ++c)
            if (g + c * kG < P) add(a2[c], hit[c]);
    } else {
        for (int ch = g; ch < P; ch += kG) {
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
        for (int q = 0; q < kG; ++q) {
            t += sum[q][p][lane];
            m += cnt[q][p][lane];
        }
        any[p] = !au && m > 0;
        limit[p] = any[p] ? k2 * (t / (double)m) : 0.0;
    }
    if constexpr (kHeld) {
#pragma unroll
        for (int c = 0; c < kH; ++c)
            if (g + c * kG < P)
                store(g + c * kG, hit[c][0] || (any[0] && a2[c][0] > limit[0]),
                      hit[c][1] || (any[1] && a2[c][1] > limit[1]));
    } else {
        for (int ch = g; ch < P; ch += kG) {
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
    // A workgroup or two per CU: a thread's 16 loads all in flight (1000 antennas
    // x 4 channels, 492 workgroups, 36 us for all three launches); more of them
    // hide the latency of four at a time and fit a CU then (576 x 16, 656
    // workgroups: 38.5 us with all, 37.0 with four); nor does a chunk of less
    // than half its size gain.
    if ((int64_t)nc * P <= 512 && nbl > 2048)
        hipLaunchKernelGGL(clip_partial_kernel<true>, dim3(nc, P), dim3(256), 0, stream, (int)nbl, V, part, nc);
    else
        hipLaunchKernelGGL(clip_partial_kernel<false>, dim3(nc, P), dim3(256), 0, stream, (int)nbl, V, part, nc);
    hipLaunchKernelGGL(clip_mean_kernel, dim3((unsigned)ceil_div(P * 2, 64)), dim3(64), 0, stream, P, nc,
                       nbl - Na, part, mean);
    // groups and held channels by the number of channels: with eight and eight
    // for any up to 64, few channels were read several times over (1500 antennas
    // x 2 channels 169 us for all three launches, 42 now; a pass per stage 83)
#define AFC_CLIP(G, H)                                                                                          \
    hipLaunchKernelGGL((clip_flags_kernel<G, H>), dim3((unsigned)ceil_div(nbl, kClipThreads / (G))),            \
                       dim3(kClipThreads), 0, stream, P, (int)nbl, V, mean, k2, flags)
    if (P == 1) AFC_CLIP(1, 1);
    else if (P == 2) AFC_CLIP(2, 1);
    else if (P <= 4) AFC_CLIP(4, 1);
    else if (P <= 8) AFC_CLIP(8, 1);
    else if (P <= 16) AFC_CLIP(8, 2);
    else if (P <= 32) AFC_CLIP(8, 4);
    else if (P <= 64) AFC_CLIP(8, 8);
    else AFC_CLIP(8, 0);
#undef AFC_CLIP
    return hipGetLastError();
}

hipError_t launch_apply_vis_flags(int Na, int P, const uint8_t* flags, float2* V, float2* M, hipStream_t stream) {
    const int64_t n = (int64_t)P * Na * (Na + 1) / 2;
    hipLaunchKernelGGL(apply_flags_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, stream, n, flags, V, M);
    return hipGetLastError();
}

}  // namespace afc
