// Lost packets and the weighting matrix (Sec. "CPU Data Collation": the
// correlator handles lost UDP packets and produces a weighting matrix with
// the visibilities; Sec. "Calibration Pipeline": the visibilities are
// re-weighted for the lost data).
//
// A spectrum of antenna a is valid iff every input sample of its FIR window
// (spectrum s reads samples s*Ps .. (s+T)*Ps - 1) arrived.  Invalid spectra
// are zeroed in the channelised array, so that the X-engine's sums run over
// the spectra valid for both antennas of a baseline, and the weight of a
// baseline is the number of those spectra.
//
//   validity_kernel   packet flags -> bit masks [B][ceil(S/32)][Na]
//   zero_kernel       zero the channelised samples of invalid spectra
//   weights_kernel    W[b][bl(a,c)] = popcount of (v_a & v_c) over s < S_b
//   normalise_kernel  V / W per baseline, float2 out
#include <type_traits>

#include "afc_internal.h"

namespace afc {
namespace {

// One thread = one antenna and one word of 32 spectra; threads of a block
// take consecutive antennas, so the packet flags of one packet row and the
// output words are read and written contiguously.  Losses are rare: the flags
// of kFlags packets are loaded together and looked at one by one only if one of
// them is zero: 576 antennas x 4 subbands x 12264 packets take 25 us (122 us
// with the window of a lost packet by 64-bit division, 183 us with one load at
// a time as well).
constexpr int kFlags = 16;
__global__ void validity_kernel(const uint8_t* __restrict__ pkt, uint32_t* __restrict__ v, int Na, int S,
                                int Wd, int64_t n_pk, int Q, int log2Ps) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const int wd = blockIdx.y;
    const int b = blockIdx.z;
    if (a >= Na) return;
    const int s0 = wd * 32;
    const int n = min(32, S - s0);
    uint32_t bits = n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u);
    // packets touched by the windows of spectra s0 .. s0+n-1
    // (samples fit 32 bits: a subband's input is below 2^31 values)
    const int64_t k_lo = ((unsigned)s0 << log2Ps) / (unsigned)Q;
    const int64_t k_hi = (((unsigned)(s0 + n - 1 + kT) << log2Ps) - 1u) / (unsigned)Q;
    const uint8_t* pb = pkt + (int64_t)b * n_pk * Na + a;
    // clears the spectra whose window [s Ps, (s+T) Ps - 1] meets packet k,
    // samples [k Q, (k+1) Q - 1]: floor(k Q / Ps) - T + 1 to floor(((k+1) Q - 1)
    // / Ps) (Ps is a power of two)
    auto lost = [&](int64_t k) {
        const int lo = (int)max(((k * Q) >> log2Ps) - kT + 1 - s0, (int64_t)0);
        const int hi = (int)min((((k + 1) * Q - 1) >> log2Ps) - s0, (int64_t)(n - 1));
        if (lo <= hi) bits &= ~((0xFFFFFFFFu << lo) & (0xFFFFFFFFu >> (31 - hi)));
    };
    int64_t k = k_lo;
    for (; bits != 0 && k + kFlags <= min(k_hi + 1, n_pk); k += kFlags) {
        uint8_t f[kFlags];
#pragma unroll
        for (int e = 0; e < kFlags; ++e) f[e] = pb[(k + e) * Na];
        bool all = true;
#pragma unroll
        for (int e = 0; e < kFlags; ++e) all = all && f[e] != 0;
        if (!all) {
#pragma unroll
            for (int e = 0; e < kFlags; ++e)
                if (f[e] == 0) lost(k + e);
        }
    }
    // the rest, and all of it where packets are long, four at a time (one by one
    // is a chain of loads); packets past the last are lost
    const int64_t last = min(k_hi, n_pk - 1);
    for (; bits != 0 && k <= k_hi; k += 4) {
        uint8_t f[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = pb[min(k + e, last) * Na];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k + e <= k_hi && (k + e >= n_pk || f[e] == 0)) lost(k + e);
    }
    v[((int64_t)b * Wd + wd) * Na + a] = bits;
}

// A workgroup looks at four words of 32 spectra of 64 antennas, a word per
// wave; losses are rare, and it ends there if it has none.  Else the waves share
// the channels and take the four words one after the other, an antenna per lane:
// zeros over both receivers, 8, 2 or 1 spectra at a time (kWide: z is 16-byte
// aligned, and with it every block).  kSplit workgroups share the channels of
// the words, four or, on small launches, eight or 16: losses are bursts of whole
// stations or a dead one, the work of few words.  576 antennas x 4 subbands, int8: 3.6 us
// without a loss, 48 us with bursts (0.6% of the packets) and a dead station; a
// thread per antenna and word that took all channels, spectrum by spectrum, 2.8
// and 363 us, a thread for every eight of the channels 5.9 and 56 us (16 subbands
// 8.6 and 160 us; 4.9 and 786, 18 and 156).  Where nearly every group of words has
// a loss, single packets at random, the words in a row cost instead: 576 x 1, 0.6%
// 17.9 us, the thread per eight channels 15.5.
constexpr int kZeroWords = 4;
template <typename SampleT, bool kWide, int kSplit>
__global__ __launch_bounds__(64 * kZeroWords) void zero_kernel(const uint32_t* __restrict__ v, SampleT* __restrict__ z,
                                                               int Na, int S, int Wd, int Sb) {
    constexpr int kCh = kP / kSplit / kZeroWords;             // channels of a thread
    __shared__ uint32_t words[kZeroWords][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int a = blockIdx.x * 64 + lane, wd0 = blockIdx.y * kZeroWords, b = blockIdx.z / kSplit;
    uint32_t own = 0u;
    if (a < Na && wd0 + wv < Wd) {
        const int n = min(32, S - (wd0 + wv) * 32);
        const uint32_t all = n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u);
        own = ~v[((int64_t)b * Wd + wd0 + wv) * Na + a] & all;
    }
    words[wv][lane] = own;
    if (!__syncthreads_or(own != 0)) return;
    const int N = 2 * Na;
    const int64_t ch_stride = (int64_t)Sb * N * kSBlk;
    SampleT* zb = z + ((int64_t)b * kP + (blockIdx.z % kSplit * kZeroWords + wv) * kCh) * ch_stride;
    // zeros of 2^E samples at p of both receivers in every channel of the thread
    auto put = [&](SampleT* p, auto e_tag) {
        constexpr size_t kRun = sizeof(SampleT) << decltype(e_tag)::value;
        struct alignas(kRun < 16 ? kRun : 16) Run {
            SampleT s[1 << decltype(e_tag)::value];
        };
#pragma unroll
        for (int k = 0; k < kCh; ++k) {
            *reinterpret_cast<Run*>(p + k * ch_stride) = Run{};
            *reinterpret_cast<Run*>(p + k * ch_stride + kSBlk) = Run{};
        }
    };
    for (int e = 0; e < 4 * kZeroWords; ++e) {                // blocks of 8 spectra
        const unsigned m8 = (words[e >> 2][lane] >> (8 * (e & 3))) & 0xFFu;
        if (m8 == 0) continue;
        SampleT* p = zb + ((int64_t)(wd0 * 4 + e) * N + 2 * a) * kSBlk;
        if (kWide && m8 == 0xFFu) {
            put(p, std::integral_constant<int, 3>{});
            continue;
        }
        for (int h = 0; h < 4; ++h) {                         // pairs of spectra
            const unsigned u = (m8 >> (2 * h)) & 3u;
            if (kWide && u == 3u) {
                put(p + 2 * h, std::integral_constant<int, 1>{});
            } else {
                if (u & 1u) put(p + 2 * h, std::integral_constant<int, 0>{});
                if (u & 2u) put(p + 2 * h + 1, std::integral_constant<int, 0>{});
            }
        }
    }
}

struct WeightArgs {
    const uint32_t* v;
    const uint8_t* flags;
    int32_t* W;
    int Na, Wd, n_tiles;
    int S[AFC_MAX_SUBBANDS];
};

constexpr int kWT = 32;          // antennas per tile side
constexpr int kWChunk = 128;     // words of 32 spectra staged per pass

// One workgroup (256 threads) = one 32 x 32 tile (a-tile >= c-tile) of one
// subband; each thread sums four (a, c) pairs, masks staged in LDS.
__global__ __launch_bounds__(256) void weights_kernel(WeightArgs w) {
    __shared__ uint32_t la[kWChunk][kWT], lc[kWChunk][kWT];
    const int b = blockIdx.y;
    // tile pair from the linear index: ta >= tc
    int t = blockIdx.x, ta = 0;
    while (t > ta) { t -= ta + 1; ++ta; }
    const int tc = t;
    const int Na = w.Na, Wd = w.Wd, S = w.S[b];
    const int tid = threadIdx.x;
    const int ci = tid & 15, ai = tid >> 4;
    int cnt[2][2] = {{0, 0}, {0, 0}};
    const uint32_t* vb = w.v + (int64_t)b * Wd * Na;
    for (int w0 = 0; w0 < Wd; w0 += kWChunk) {
        const int nw = min(kWChunk, Wd - w0);
        for (int e = tid; e < nw * kWT; e += 256) {
            const int wd = e / kWT, j = e % kWT;
            const int s0 = (w0 + wd) * 32;
            // spectra >= S of this subband do not count
            const int n = max(0, min(32, S - s0));
            const uint32_t m = n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u);
            const int a = ta * kWT + j, c = tc * kWT + j;
            la[wd][j] = a < Na ? vb[(int64_t)(w0 + wd) * Na + a] & m : 0u;
            lc[wd][j] = c < Na ? vb[(int64_t)(w0 + wd) * Na + c] & m : 0u;
        }
        __syncthreads();
        for (int wd = 0; wd < nw; ++wd) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    cnt[x][y] += __popc(la[wd][ai + 16 * x] & lc[wd][ci + 16 * y]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int a = ta * kWT + ai + 16 * x, c = tc * kWT + ci + 16 * y;
            if (a >= Na || c > a) continue;
            const bool flagged = w.flags && (w.flags[(int64_t)b * Na + a] || w.flags[(int64_t)b * Na + c]);
            w.W[(int64_t)b * ((int64_t)Na * (Na + 1) / 2) + (int64_t)a * (a + 1) / 2 + c] = flagged ? 0 : cnt[x][y];
        }
}

// out = vis / W per baseline (0 where W = 0); one thread = one baseline's
// 2 x 2 block of one channel; blockIdx.y = subband * P + channel, so the
// indices need no 64-bit division.  Every byte is touched once: loads and
// stores are non-temporal.
typedef int nv4i __attribute__((ext_vector_type(4)));
typedef float nv4f __attribute__((ext_vector_type(4)));

template <bool kInt>
__global__ void normalise_kernel(const void* __restrict__ vis, const int32_t* __restrict__ W,
                                 float2* __restrict__ out, int nbl, int P) {
    const int bl = blockIdx.x * blockDim.x + threadIdx.x;
    if (bl >= nbl) return;
    const int slice = blockIdx.y;                           // subband * P + channel
    const int64_t e = (int64_t)slice * nbl + bl;
    const int32_t wt = W[(int64_t)(slice / P) * nbl + bl];
    float2 r[4];
    if constexpr (kInt) {
        const nv4i* src = reinterpret_cast<const nv4i*>(vis) + e * 2;
        const nv4i u0 = __builtin_nontemporal_load(src), u1 = __builtin_nontemporal_load(src + 1);
        const int vv[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            r[j] = wt > 0 ? make_float2((float)((double)vv[2 * j] / wt), (float)((double)vv[2 * j + 1] / wt))
                          : make_float2(0.0f, 0.0f);
    } else {
        const nv4f* src = reinterpret_cast<const nv4f*>(vis) + e * 2;
        const nv4f f0 = __builtin_nontemporal_load(src), f1 = __builtin_nontemporal_load(src + 1);
        const float vv[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
        const float fw = (float)wt;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            r[j] = wt > 0 ? make_float2(vv[2 * j] / fw, vv[2 * j + 1] / fw) : make_float2(0.0f, 0.0f);
    }
    nv4f* dst = reinterpret_cast<nv4f*>(out) + e * 2;
    __builtin_nontemporal_store(nv4f{r[0].x, r[0].y, r[1].x, r[1].y}, dst);
    __builtin_nontemporal_store(nv4f{r[2].x, r[2].y, r[3].x, r[3].y}, dst + 1);
}

struct alignas(4) Half2Raw { uint16_t x, y; };
struct alignas(2) I8x2 { int8_t x, y; };

}  // namespace

hipError_t launch_validity(const uint8_t* pkt, uint32_t* v, int B, int Na, int S, int64_t n_pk, int Q, int Ps,
                           hipStream_t stream) {
    const int Wd = (int)ceil_div(S, 32);
    const dim3 grid((unsigned)ceil_div(Na, 256), (unsigned)Wd, (unsigned)B);
    hipLaunchKernelGGL(validity_kernel, grid, dim3(256), 0, stream, pkt, v, Na, S, Wd, n_pk, Q,
                       Ps == kP ? 6 : 8);
    return hipGetLastError();
}

hipError_t launch_zero_invalid(const uint32_t* v, void* z, afc_dtype dt, int B, int Na, int S, hipStream_t stream) {
    const int Wd = (int)ceil_div(S, 32);
    const int Sb = (int)ceil_div(S, kSBlk);
    const bool wide = reinterpret_cast<uintptr_t>(z) % 16 == 0;
    const int64_t n_wg = ceil_div(Na, 64) * ceil_div(Wd, kZeroWords) * B;
    const int split = n_wg * 16 <= 2048 ? 16 : n_wg * 8 <= 2048 ? 8 : 4;
    const dim3 grid((unsigned)ceil_div(Na, 64), (unsigned)ceil_div(Wd, kZeroWords), (unsigned)(B * split));
#define AFC_ZERO_N(T, W, N)                                                                                     \
    hipLaunchKernelGGL((zero_kernel<T, W, N>), grid, dim3(64 * kZeroWords), 0, stream, v, reinterpret_cast<T*>(z), Na, \
                       S, Wd, Sb)
#define AFC_ZERO_W(T, W)                                                                                        \
    if (split == 16) AFC_ZERO_N(T, W, 16);                                                                      \
    else if (split == 8) AFC_ZERO_N(T, W, 8);                                                                   \
    else AFC_ZERO_N(T, W, 4);
#define AFC_ZERO(T)                                                                                             \
    if (wide) { AFC_ZERO_W(T, true) } else { AFC_ZERO_W(T, false) }
    switch (dt) {
        case AFC_F32: AFC_ZERO(float2) break;
        case AFC_F16: AFC_ZERO(Half2Raw) break;
        default: AFC_ZERO(I8x2) break;
    }
#undef AFC_ZERO_N
#undef AFC_ZERO_W
#undef AFC_ZERO
    return hipGetLastError();
}

hipError_t launch_validity_weights(const uint32_t* v, const uint8_t* flags, int32_t* W, int B, int Na, int S,
                                   const int32_t* S_host, hipStream_t stream) {
    WeightArgs w{};
    w.v = v;
    w.flags = flags;
    w.W = W;
    w.Na = Na;
    w.Wd = (int)ceil_div(S, 32);
    const int nt = (int)ceil_div(Na, kWT);
    w.n_tiles = nt;
    for (int b = 0; b < B; ++b) w.S[b] = S_host ? S_host[b] : S;
    const dim3 grid((unsigned)(nt * (nt + 1) / 2), (unsigned)B);
    hipLaunchKernelGGL(weights_kernel, grid, dim3(256), 0, stream, w);
    return hipGetLastError();
}

hipError_t launch_normalise(const void* vis, bool is_int, const int32_t* W, void* out, int B, int Na,
                            hipStream_t stream) {
    const int64_t nbl = (int64_t)Na * (Na + 1) / 2;
    if (nbl > (1 << 30) || (int64_t)B * kP > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)ceil_div(nbl, 256), (unsigned)(B * kP));
    if (is_int)
        hipLaunchKernelGGL(normalise_kernel<true>, grid, dim3(256), 0, stream, vis, W,
                           reinterpret_cast<float2*>(out), (int)nbl, kP);
    else
        hipLaunchKernelGGL(normalise_kernel<false>, grid, dim3(256), 0, stream, vis, W,
                           reinterpret_cast<float2*>(out), (int)nbl, kP);
    return hipGetLastError();
}

}  // namespace afc
