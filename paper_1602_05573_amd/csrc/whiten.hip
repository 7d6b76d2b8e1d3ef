// Whitening front end: the filter bank's input is whitened strain; this is
// the step that makes it from raw detector data (the paper's SPIIR section
// takes noisy detector data as input, "SPIIR method"). Frames of N samples at
// hop H = N/2 with a periodic Hann window w[t] = sin^2(pi t / N):
//   PSD estimate : S[f] = mean over frames of |DFT(w . s_k)[f]|^2 / sum_t w[t]^2, f = 0..N/2
//   whitening    : y_k = IDFT(DFT(w . x_k) / sqrt(S)), overlap-added at hop H
// The stream is whitened with a delay of H samples (H zeros precede it).
//
// Two neighbouring frames share one complex transform (the earlier one in the
// real part, the later one in the imaginary part): 1 / sqrt(S) is real and
// even, so whitening acts on both parts alone, and the hop that the two frames
// overlap in is the sum of one half of each, so a hop is written by the one
// group of threads that transforms its two frames and no frame output goes
// through memory. The first hop takes the stored half of the frame before the
// call instead of that frame, and one more group transforms the last frame
// alone for the half that the next call takes: neither depends on samples
// outside its frames, and the stored half keeps the PSD it was made with.
//
// What bounds it is the latency of one transform on one compute unit (4,096
// samples are 3 workgroups): FP32 issue of the butterflies and the exchanges
// through LDS. Hence radix 8 with 8 elements per thread (3 exchanges each way
// at N = 4,096, where radix 4 had 12 passes through LDS and two more for the
// bit reversal), the frequencies left in digit-reversed order between the two
// transforms (1 / sqrt(S) is stored in that order), and every twiddle factor
// loaded once into registers, from tables in the order of use, and used by
// both transforms. A call of 4,096 samples at N = 4,096: one launch of 6.5 us,
// where one real frame per workgroup, radix 4 over bit-reversed input and a
// launch for the overlap-add took 16.8 + 3.3 us; 262,144 samples after a PSD of
// 131,072: 108 -> 22 us.
#include "spiir_internal.h"

#include <algorithm>

namespace spiir {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {   // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// a * (-i) forward, a * i inverse
template <bool INV>
__device__ __forceinline__ float2 rot90(float2 a) {
    return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// Frequency digits: position p of the transformed frame holds frequency f when
// the base-8 digits of f, lowest first, are those of p, highest first (the last
// digit has the remaining 1 to 3 bits).
__device__ __forceinline__ int pos_of(int f, int logn) {
    int p = 0, left = logn;
    while (left > 3) {
        left -= 3;
        p |= (f & 7) << left;
        f >>= 3;
    }
    return p | f;
}

// LDS position of frame element p: bits 3-7 are XORed into bits 0-4, so that
// the strided accesses of every pass (elements 1, 8 and 64 apart over the lanes)
// take the 32 pairs of banks once per half wave. Linear over bits: a sum of
// parts with disjoint bits maps to the XOR of their images.
__device__ __forceinline__ constexpr int sw(int p) { return p ^ ((p >> 3) & 31); }

template <bool INV>
__device__ __forceinline__ void dft4(float2 &c0, float2 &c1, float2 &c2, float2 &c3) {
    const float2 s0 = cadd(c0, c2), s1 = csub(c0, c2), s2 = cadd(c1, c3), s3 = rot90<INV>(csub(c1, c3));
    c0 = cadd(s0, s2);
    c1 = cadd(s1, s3);
    c2 = csub(s0, s2);
    c3 = csub(s1, s3);
}

template <bool INV>
__device__ __forceinline__ void dft8(float2 (&v)[8]) {
    constexpr float r = 0.70710678118654752440f;
    float2 a0 = cadd(v[0], v[4]), a1 = cadd(v[1], v[5]), a2 = cadd(v[2], v[6]), a3 = cadd(v[3], v[7]);
    float2 b0 = csub(v[0], v[4]), b1 = csub(v[1], v[5]), b2 = csub(v[2], v[6]), b3 = csub(v[3], v[7]);
    // times exp(-+ i pi k / 4)
    const float2 q1 = rot90<INV>(b1), q3 = rot90<INV>(b3);
    b1 = make_float2((b1.x + q1.x) * r, (b1.y + q1.y) * r);
    b2 = rot90<INV>(b2);
    b3 = make_float2((q3.x - b3.x) * r, (q3.y - b3.y) * r);
    dft4<INV>(a0, a1, a2, a3);
    dft4<INV>(b0, b1, b2, b3);
    v[0] = a0;
    v[1] = b0;
    v[2] = a1;
    v[3] = b1;
    v[4] = a2;
    v[5] = b2;
    v[6] = a3;
    v[7] = b3;
}

// N-point transform of one group of N/8 threads, 8 elements each. Pass s of
// the kPasses radix-8 passes takes blocks of N >> 3s elements; the last pass
// takes each thread's 8 consecutive elements in transforms of kLast.
template <int LOGN>
struct Fft {
    static constexpr int N = 1 << LOGN;
    static constexpr int T = N / 8;
    static constexpr int kPasses = (LOGN + 2) / 3 - 1;
    static constexpr int kLast = N >> (3 * kPasses);
    static constexpr int kGroup = T < 64 ? 64 : T;   // threads per workgroup

    float2 v[8];
    float2 w[kPasses][7];

    static constexpr int span(int s) { return N >> (3 * (s + 1)); }
    static __device__ __forceinline__ int base(int s, int t) {
        const int m = span(s);
        return (t / m) * (8 * m) + (t & (m - 1));
    }
    // table of pass s: exp(-2 pi i q pos / (8 span)), q = 1..7 by pos
    __device__ __forceinline__ void twiddles(const float2 *__restrict__ tw, int t) {
#pragma unroll
        for (int s = 0; s < kPasses; ++s) {
            const int m = span(s);
#pragma unroll
            for (int q = 1; q < 8; ++q) w[s][q - 1] = tw[(q - 1) * m + (t & (m - 1))];
            tw += 7 * m;
        }
    }
    __device__ __forceinline__ void put(float2 *buf, int b, int m) {
        b = sw(b);
#pragma unroll
        for (int k = 0; k < 8; ++k) buf[b ^ sw(k * m)] = v[k];
    }
    __device__ __forceinline__ void get(const float2 *buf, int b, int m) {
        b = sw(b);
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = buf[b ^ sw(k * m)];
    }
    template <bool INV>
    __device__ __forceinline__ void last() {
        if constexpr (kLast == 8) {
            dft8<INV>(v);
        } else if constexpr (kLast == 4) {
            dft4<INV>(v[0], v[1], v[2], v[3]);
            dft4<INV>(v[4], v[5], v[6], v[7]);
        } else {
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
                const float2 u = v[k];
                v[k] = cadd(u, v[k + 1]);
                v[k + 1] = csub(u, v[k + 1]);
            }
        }
    }
    // v[k] = element t + k T in; position 8 t + k out. Each pass stores where it
    // loaded, so one barrier per exchange is enough.
    __device__ __forceinline__ void forward(float2 *buf, int t) {
#pragma unroll
        for (int s = 0; s < kPasses; ++s) {
            dft8<false>(v);
#pragma unroll
            for (int q = 1; q < 8; ++q) v[q] = cmul(v[q], w[s][q - 1]);
            put(buf, base(s, t), span(s));
            __syncthreads();
            if (s + 1 < kPasses)
                get(buf, base(s + 1, t), span(s + 1));
            else
                get(buf, 8 * t, 1);
        }
        last<false>();
    }
    // the transposed steps: position 8 t + k in, element t + k T out
    __device__ __forceinline__ void inverse(float2 *buf, int t) {
        last<true>();
        put(buf, 8 * t, 1);
#pragma unroll
        for (int s = kPasses - 1; s >= 0; --s) {
            __syncthreads();
            get(buf, base(s, t), span(s));
#pragma unroll
            for (int q = 1; q < 8; ++q) v[q] = cmulc(v[q], w[s][q - 1]);
            dft8<true>(v);
            if (s > 0) put(buf, base(s, t), span(s));
        }
    }
};

// Hop j = 0..nf (group j of the grid; nf is the stored half for the next call).
// Half frame b of the stream is hist for b = 0 and x + (b - 1) H after it;
// frame j has the half frames j and j + 1.
template <int LOGN>
__global__ void __launch_bounds__(Fft<LOGN>::kGroup)
    wh_hops_kernel(const float *__restrict__ hist, const float *__restrict__ x, int64_t nf,
                   const float *__restrict__ wtab, const float2 *__restrict__ tw, const float *__restrict__ inv,
                   const float *__restrict__ pend, float *__restrict__ pend_new, float *__restrict__ hist_new,
                   float *__restrict__ out) {
    using F = Fft<LOGN>;
    constexpr int T = F::T, H = F::N / 2, kPer = F::kGroup / T;
    __shared__ float2 lds[F::kGroup * 8];
    const int t = threadIdx.x & (T - 1);
    float2 *buf = lds + (threadIdx.x / T) * F::N;
    const int64_t j = (int64_t)blockIdx.x * kPer + threadIdx.x / T;
    const bool live = j <= nf, prev = live && j > 0, next = j < nf;
    // half frames j - 1, j, j + 1
    const float *h0 = j <= 1 ? hist : x + (j - 2) * H, *h1 = j == 0 ? hist : x + (j - 1) * H, *h2 = x + j * H;
    F f;
    float s[12];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        s[k] = prev ? h0[t + k * T] : 0.f;
        s[4 + k] = live ? h1[t + k * T] : 0.f;
        s[8 + k] = next ? h2[t + k * T] : 0.f;
    }
    float win[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) win[k] = wtab[t + k * T];
    f.twiddles(tw, t);
    const float4 i0 = *reinterpret_cast<const float4 *>(inv + 8 * t);
    const float4 i1 = *reinterpret_cast<const float4 *>(inv + 8 * t + 4);
#pragma unroll
    for (int k = 0; k < 8; ++k)
        f.v[k] = make_float2(prev ? win[k] * s[k] : 0.f, next ? win[k] * s[4 + k] : 0.f);
    f.forward(buf, t);
    const float g[8] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) f.v[k] = make_float2(f.v[k].x * g[k], f.v[k].y * g[k]);
    f.inverse(buf, t);
    constexpr float scale = 1.0f / (float)F::N;
    if (!live) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = t + k * T;
        const float before = prev ? f.v[k + 4].x * scale : pend[i];
        if (next) {
            out[j * H + i] = f.v[k].y * scale + before;
        } else {
            pend_new[i] = before;
            hist_new[i] = s[4 + k];
        }
    }
}

// Power of the training frames 2j and 2j + 1 in one transform Z of the two:
// |X_2j[f]|^2 + |X_2j+1[f]|^2 = (|Z[f]|^2 + |Z[N - f]|^2) / 2, f = 0..H.
template <int LOGN>
__global__ void __launch_bounds__(Fft<LOGN>::kGroup)
    wh_power_kernel(const float *__restrict__ x, int64_t frames, const float *__restrict__ wtab,
                    const float2 *__restrict__ tw, float *__restrict__ pw) {
    using F = Fft<LOGN>;
    constexpr int T = F::T, H = F::N / 2, kPer = F::kGroup / T;
    __shared__ float2 lds[F::kGroup * 8];
    const int t = threadIdx.x & (T - 1);
    float2 *buf = lds + (threadIdx.x / T) * F::N;
    const int64_t j = (int64_t)blockIdx.x * kPer + threadIdx.x / T;
    const bool first = 2 * j < frames, second = 2 * j + 1 < frames;
    const float *h = x + 2 * j * H;
    F f;
    float s[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) s[k] = (k < 8 ? first : second) ? h[t + k * T] : 0.f;
    float win[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) win[k] = wtab[t + k * T];
    f.twiddles(tw, t);
#pragma unroll
    for (int k = 0; k < 8; ++k) f.v[k] = make_float2(win[k] * s[k], second ? win[k] * s[4 + k] : 0.f);
    f.forward(buf, t);
    f.put(buf, 8 * t, 1);
    __syncthreads();
    if (!first) return;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int q = t + k * T;
        if (q > H) break;
        const float2 a = buf[sw(pos_of(q, LOGN))], b = buf[sw(pos_of((F::N - q) & (F::N - 1), LOGN))];
        pw[j * (H + 1) + q] = (float)(0.5 * ((double)a.x * a.x + (double)a.y * a.y + (double)b.x * b.x +
                                             (double)b.y * b.y));
    }
}

__device__ __forceinline__ void put_inv(double v, int f, int logn, float *inv) {
    const float s = v > 0.0 ? (float)(1.0 / sqrt(v)) : 0.0f;
    inv[pos_of(f, logn)] = s;
    inv[pos_of(((1 << logn) - f) & ((1 << logn) - 1), logn)] = s;
}

// S[f] = sum_j pw[j][f] / (frames * wsum2) in FP64 over the rows of the frame
// pairs; inv[position of f and of N - f] = 1 / sqrt(S[f]), 0 where S <= 0. A
// workgroup takes 32 frequencies and every thread every 8th row: with one
// thread per frequency the serial loads of 63 rows took 17 us; 2.9 us now.
__global__ void __launch_bounds__(kThreads)
    wh_psd_reduce_kernel(const float *__restrict__ pw, int64_t rows, int64_t frames, int logn, double wsum2,
                         double *__restrict__ S, float *__restrict__ inv) {
    const int H = 1 << (logn - 1);
    const int f = blockIdx.x * 32 + (threadIdx.x & 31);
    const int r = threadIdx.x >> 5;
    __shared__ double part[8][32];
    double acc = 0.0;
    if (f <= H) {
#pragma unroll 4
        for (int64_t j = r; j < rows; j += 8) acc += (double)pw[j * (H + 1) + f];
    }
    part[r][threadIdx.x & 31] = acc;
    __syncthreads();
    if (r > 0 || f > H) return;
    acc = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += part[q][threadIdx.x];
    const double v = acc / ((double)frames * wsum2);
    S[f] = v;
    put_inv(v, f, logn, inv);
}

// inv from a given S (host-set PSD).
__global__ void wh_inv_kernel(const double *__restrict__ S, int logn, float *__restrict__ inv) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f <= 1 << (logn - 1)) put_inv(S[f], f, logn, inv);
}

__global__ void wh_copy_kernel(const float *a, float *b, int64_t n, const float *c, float *d, int64_t m) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = a[i];
    if (i < m) d[i] = c[i];
}

template <int LOGN>
hipError_t hops(const WhitenHops &a, hipStream_t st) {
    using F = Fft<LOGN>;
    constexpr int per = F::kGroup / F::T;
    hipLaunchKernelGGL(wh_hops_kernel<LOGN>, dim3((unsigned)(a.nf / per + 1)), dim3(F::kGroup), 0, st, a.hist, a.x,
                       a.nf, a.wtab, a.tw, a.inv, a.pend, a.pend_new, a.hist_new, a.out);
    return hipGetLastError();
}

template <int LOGN>
hipError_t power(const float *x, int64_t frames, const float *wtab, const float2 *tw, float *pw, hipStream_t st) {
    using F = Fft<LOGN>;
    constexpr int per = F::kGroup / F::T;
    const int64_t pairs = (frames + 1) / 2;
    hipLaunchKernelGGL(wh_power_kernel<LOGN>, dim3((unsigned)((pairs + per - 1) / per)), dim3(F::kGroup), 0, st, x,
                       frames, wtab, tw, pw);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_wh_hops(const WhitenHops &a, int logn, hipStream_t st) {
    if (a.nf <= 0) return hipSuccess;
    switch (logn) {
        case 4: return hops<4>(a, st);
        case 5: return hops<5>(a, st);
        case 6: return hops<6>(a, st);
        case 7: return hops<7>(a, st);
        case 8: return hops<8>(a, st);
        case 9: return hops<9>(a, st);
        case 10: return hops<10>(a, st);
        case 11: return hops<11>(a, st);
        case 12: return hops<12>(a, st);
        case 13: return hops<13>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_wh_power(const float *x, int64_t frames, const float *wtab, const float2 *tw, int logn, float *pw,
                           hipStream_t st) {
    if (frames <= 0) return hipSuccess;
    switch (logn) {
        case 4: return power<4>(x, frames, wtab, tw, pw, st);
        case 5: return power<5>(x, frames, wtab, tw, pw, st);
        case 6: return power<6>(x, frames, wtab, tw, pw, st);
        case 7: return power<7>(x, frames, wtab, tw, pw, st);
        case 8: return power<8>(x, frames, wtab, tw, pw, st);
        case 9: return power<9>(x, frames, wtab, tw, pw, st);
        case 10: return power<10>(x, frames, wtab, tw, pw, st);
        case 11: return power<11>(x, frames, wtab, tw, pw, st);
        case 12: return power<12>(x, frames, wtab, tw, pw, st);
        case 13: return power<13>(x, frames, wtab, tw, pw, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_wh_psd_reduce(const float *pw, int64_t frames, int logn, double wsum2, double *S, float *inv,
                                hipStream_t st) {
    const int H = 1 << (logn - 1);
    hipLaunchKernelGGL(wh_psd_reduce_kernel, dim3((unsigned)(H / 32 + 1)), dim3(kThreads), 0, st, pw,
                       (frames + 1) / 2, frames, logn, wsum2, S, inv);
    return hipGetLastError();
}

hipError_t launch_wh_inv(const double *S, int logn, float *inv, hipStream_t st) {
    const int H = 1 << (logn - 1);
    hipLaunchKernelGGL(wh_inv_kernel, dim3((unsigned)(H / kThreads + 1)), dim3(kThreads), 0, st, S, logn, inv);
    return hipGetLastError();
}

hipError_t launch_wh_copy(const float *a, float *b, int64_t n, const float *c, float *d, int64_t m, hipStream_t st) {
    const int64_t most = std::max(n, m);
    if (most <= 0) return hipSuccess;
    hipLaunchKernelGGL(wh_copy_kernel, dim3((unsigned)((most + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, a, b,
                       n, c, d, m);
    return hipGetLastError();
}

}  // namespace spiir
