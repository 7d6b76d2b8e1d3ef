// Multi-rate filter bank: the resampling and recombination around the
// per-level filter banks. The paper remarks that a slowly evolving chirp lets
// both the data and the templates run at a lower sampling rate (Sect.
// "Multimessenger astronomy"); this library's reading:
//   x_r[q]  = sum_i h[i] x_{r-1}[2q + 1 - i]                 (decimation, causal FIR)
//   z_r     = level-r template sums of filters run on x_r      (ordinary bank, z mode)
//   w_R     = z_R,  w_r[p] = z_r[p] + sum_q g[p - 2q] w_{r+1}[q]   (interpolation, causal FIR)
//   z       = w_0, then |z|^2 and the per-sample max / argmax over templates.
// All kernels here are streaming: each level keeps the last samples of its
// resampling input as history, so consecutive calls continue one stream.
#include "spiir_internal.h"

#include <algorithm>

namespace spiir {
namespace {

constexpr int kThreads = 256;

int64_t nblk(int64_t n, int64_t b) { return (n + b - 1) / b; }

// dst[q] = sum_i h[i] v(2q + 1 - i) for q < n_src / 2, with v(m) = src[m] for
// m >= 0 and hist[lh - 1 + m] (the previous lh - 1 samples) for m < 0. Block 0
// also writes the next call's history (the last lh - 1 samples of v) to
// hist_new, a different buffer than hist.
__global__ __launch_bounds__(kThreads) void mr_decimate_kernel(const float *__restrict__ src, int64_t n_src,
                                                               const float *__restrict__ hist,
                                                               float *__restrict__ hist_new,
                                                               const float *__restrict__ h, int lh,
                                                               float *__restrict__ dst) {
    const int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t nq = n_src / 2;
    if (q < nq) {
        float acc = 0.0f;
        for (int i = 0; i < lh; ++i) {
            const int64_t m = 2 * q + 1 - i;
            const float v = m >= 0 ? src[m] : hist[lh - 1 + m];
            acc = fmaf(h[i], v, acc);
        }
        dst[q] = acc;
    }
    if (blockIdx.x == 0 && threadIdx.x < lh - 1) {
        const int64_t m = n_src - (lh - 1) + threadIdx.x;
        hist_new[threadIdx.x] = m >= 0 ? src[m] : hist[lh - 1 + m];
    }
}

constexpr int kMaxTaps = 64;
typedef float f4v __attribute__((ext_vector_type(4)));

// Output pairs (2m, 2m + 1) read the same W samples:
// out(2m) += sum_k g[2k] W(m - k), out(2m + 1) += sum_k g[2k + 1] W(m - k),
// with s[sb + m[u] - k] the staged W(m - k). Each of the NU pairs of a lane
// accumulates its taps in ascending order, as the plain per-output sum does,
// so both forms give the same values. Two tap pairs per step: their taps are
// one 16-byte read and their samples neighbours.
template <int NU>
__device__ __forceinline__ void interp_pairs(const float2 *s, int sb, const float *sg, int lg, const int *m,
                                             float2 *ev, float2 *od) {
    const int kp = lg >> 1;   // whole (even, odd) tap pairs
    int k = 0;
    for (; k + 2 <= kp; k += 2) {
        const f4v g = *reinterpret_cast<const f4v *>(sg + 2 * k);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const float2 *p = s + (sb + m[u] - k - 1);
            const float2 x = p[1], y = p[0];
            ev[u].x = fmaf(g.x, x.x, ev[u].x);
            ev[u].y = fmaf(g.x, x.y, ev[u].y);
            od[u].x = fmaf(g.y, x.x, od[u].x);
            od[u].y = fmaf(g.y, x.y, od[u].y);
            ev[u].x = fmaf(g.z, y.x, ev[u].x);
            ev[u].y = fmaf(g.z, y.y, ev[u].y);
            od[u].x = fmaf(g.w, y.x, od[u].x);
            od[u].y = fmaf(g.w, y.y, od[u].y);
        }
    }
    if (k < kp) {
        const float ge = sg[2 * k], go = sg[2 * k + 1];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const float2 x = s[sb + m[u] - k];
            ev[u].x = fmaf(ge, x.x, ev[u].x);
            ev[u].y = fmaf(ge, x.y, ev[u].y);
            od[u].x = fmaf(go, x.x, od[u].x);
            od[u].y = fmaf(go, x.y, od[u].y);
        }
    }
    if (lg & 1) {   // an odd tap count's last even tap
        const float ge = sg[2 * kp];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const float2 x = s[sb + m[u] - kp];
            ev[u].x = fmaf(ge, x.x, ev[u].x);
            ev[u].y = fmaf(ge, x.y, ev[u].y);
        }
    }
}

// Every decimation level of a piece in one launch. A workgroup takes slice
// samples of the input and forms its part of every level, each level's samples
// kept in LDS as the input of the next; what the taps reach before its part is
// formed again by the workgroup itself (22 * 15 samples of the input for 24
// taps and 4 levels). Taps are added in the same order as in
// mr_decimate_kernel, so the values are those of the per-level launches; so are
// the histories, which the last workgroup writes to hist_new. Bound by latency:
// one workgroup for the whole piece took 8 us for 4,096 samples and 22 us for
// 16,384 (24 taps, 4 levels), slices of 512 take 5 us for both.
constexpr int kPyrThreads = 512;
constexpr int kPyrSlice = 512;

// Samples of level r that a slice's part of the levels above reaches back to
// before its own part.
int pyr_reach(int r, int top, int lh) {
    int reach = 0;
    for (int q = top - 1; q >= r; --q) reach = std::max(0, 2 * reach + lh - 2);
    return reach;
}

// acc = sum_{i < lh} h[i] v(m0 - i), v(m0 - i) = s[-i], taps ascending.
__device__ __forceinline__ float fir_down(const float *sh, const float *s, int lh) {
    float acc = 0.0f;
    int i = 0;
    for (; i + 8 <= lh; i += 8) {
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = fmaf(sh[i + u], s[-(i + u)], acc);
    }
    for (; i < lh; ++i) acc = fmaf(sh[i], s[-i], acc);
    return acc;
}

__global__ __launch_bounds__(kPyrThreads) void mr_pyramid_kernel(const float *__restrict__ x, int n, int top,
                                                                 MrPyramid pm, const float *__restrict__ h, int lh,
                                                                 int slice, int cap0) {
    // dynamic LDS: [cap0] levels r < top with r even, then those with r odd
    extern __shared__ float pbuf[];
    __shared__ float sh[kMaxTaps];
    __shared__ int slo[kMaxLevels];   // first sample of each level in LDS (below 0: history)
    const int hl = lh - 1;
    const int first = (int)blockIdx.x * slice, end = min(n, first + slice);
    if (threadIdx.x == 0) {
        int lo = first >> top;
        for (int r = top - 1; r >= 0; --r) {
            lo = min(first >> r, 2 * max(lo, 0) + 1 - hl);
            slo[r] = lo;
        }
    }
    if (threadIdx.x < lh) sh[threadIdx.x] = h[threadIdx.x];
    __syncthreads();
    for (int m = slo[0] + (int)threadIdx.x; m < end; m += kPyrThreads)
        pbuf[m - slo[0]] = m >= 0 ? x[m] : pm.hist[1][hl + m];
    for (int r = 1; r <= top; ++r) {
        __syncthreads();
        const float *lsrc = pbuf + ((r - 1) & 1) * cap0;   // sample m of level r - 1: lsrc[m - lo]
        float *ldst = pbuf + (r & 1) * cap0;
        const int lo = slo[r - 1], own = first >> r, qe = end >> r, q0 = r < top ? slo[r] : own;
        for (int q = q0 + (int)threadIdx.x; q < qe; q += kPyrThreads) {
            float acc;
            if (q >= 0) {
                acc = fir_down(sh, lsrc + (2 * q + 1 - lo), lh);
                if (q >= own) pm.dst[r][q] = acc;
            } else {
                acc = pm.hist[r + 1][hl + q];
            }
            if (r < top) ldst[q - q0] = acc;
        }
        if (end == n)
            for (int i = threadIdx.x; i < hl; i += kPyrThreads) pm.hist_new[r][i] = lsrc[(n >> (r - 1)) - hl + i - lo];
    }
}

// Interpolation of every level back to the full rate, fused with the output:
//   W_top = z_top,  W_r(q) = Z_r(q) + sum_{i < lg, q - i even} g[i] W_{r+1}((q - i) / 2)  (r = top - 1 .. 0)
// with Z_r(q) = z[r][zrow[r][j]][q] (0 where the level or the row has no
// filters) and W_r(q) for -hh <= q < 0 taken from the previous call's history
// whist[r][j][hh + q]. Block = one chunk of kKeyChunk template rows x one
// tile of kTile full-rate samples, one wave per row. For the tile each wave
// forms, from the top level down, the window of every level that the tile's
// outputs depend on (level r + 1's window covers the taps of level r's,
// recomputed where tiles overlap) in two LDS buffers used in turn, then
// writes the full-rate z of the tile (Z mode) or its |z|^2 to LDS, from which
// every sample's largest key (|z|^2 bits << 32 | ~j) over the chunk's rows is
// formed (keys mode; plain LDS reads, no atomics). Outputs pair
// up (2m, 2m + 1), which read the same W samples with the even and the odd
// taps; each output adds its taps in ascending order onto Z_r, as the plain
// per-output sum does. The last tile writes every level's next history (the
// last hh samples of W_r) to whist_new.
//
// Bound by LDS reads and FP32 issue about equally (1,024 templates, 5 levels,
// 4,096 samples, 24 taps: 33.5 MB written at 1.7 TB/s in 20 us; 25 us before).
// Hence two tap pairs per step, as many pairs per lane as the level's window
// has, one 16-byte store and load per pair, every level's z loaded while the
// level above is formed, and no barrier between levels, whose windows belong
// to one wave.
constexpr int kKeyChunk = 16;
constexpr int kChainThreads = kKeyChunk * 64;
constexpr int kTile = 512;
// pairs per lane of a level's window: at most (kTile + kMaxTaps + 1) / 2 + 1 samples at
// level 1 and fewer above, from an odd index on
constexpr int kWinPairs = ((kTile + kMaxTaps + 1) / 2 + 3 + 127) / 128;
constexpr int kChainLdsMax = 60 * 1024;   // dynamic LDS of mr_chain_kernel (static part: 384 bytes)

__device__ __forceinline__ int floor_half(int v) { return v >= 0 ? v / 2 : -((-v + 1) / 2); }

// Pairs (2m, 2m + 1) of a level's z for m = m0 + 64 u + lane, 0 from n on or
// without a row. A row starts at a multiple of its stride in its buffer, so an
// even stride makes every pair one aligned 16-byte load.
template <int NU>
__device__ __forceinline__ void load_pairs(const float2 *zj, int64_t ld, int m0, int lane, int n, float2 (&ev)[NU],
                                           float2 (&od)[NU]) {
#pragma unroll
    for (int u = 0; u < NU; ++u) ev[u] = od[u] = make_float2(0.0f, 0.0f);
    if (!zj) return;
    const bool pairs = (ld & 1) == 0;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int q = 2 * (m0 + u * 64 + lane);
        if (pairs && q + 1 < n) {
            const f4v z = *reinterpret_cast<const f4v *>(zj + q);
            ev[u] = make_float2(z.x, z.y);
            od[u] = make_float2(z.z, z.w);
        } else {
            if (q < n) ev[u] = zj[q];
            if (q + 1 < n) od[u] = zj[q + 1];
        }
    }
}

// Indices inside a piece fit int32 (a piece has at most max_block samples).
template <bool KEYS>
__global__ __launch_bounds__(kChainThreads, 8) void mr_chain_kernel(MrChain c, int top, int hh,
                                                                 const float *__restrict__ g, int lg, int n_out,
                                                                 int T, int capA, int capB, uint64_t *__restrict__ keys,
                                                                 int64_t ld_keys, float2 *__restrict__ out,
                                                                 int64_t ld_out, int tiles) {
    extern __shared__ __align__(16) float2 wbuf[];   // per wave: capA then capB samples
    __shared__ __align__(16) float sg[kMaxTaps];
    __shared__ int slo[kMaxLevels], shi[kMaxLevels];
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int chunk = (int)blockIdx.x / tiles;
    const int tile = (int)blockIdx.x % tiles;
    const bool last = tile == tiles - 1;
    const int p0 = tile * kTile;
    const int j = chunk * kKeyChunk + wv;
    const bool live = j < T;
    float2 *bufA = wbuf + wv * (capA + capB);
    float2 *bufB = bufA + capA;
    if (threadIdx.x == 0) {
        // windows: level 0 = the tile; level r covers the taps of level r - 1's
        // computed part (its non-negative indices; the rest is history)
        slo[0] = p0;
        shi[0] = min(p0 + kTile, n_out) - 1;
        for (int r = 1; r <= top; ++r) {
            const int a = r == 1 ? slo[0] : max(slo[r - 1], 0);
            slo[r] = floor_half(a - lg + 1);
            shi[r] = shi[r - 1] / 2;
        }
    }
    if (threadIdx.x < lg) sg[threadIdx.x] = g[threadIdx.x];
    __syncthreads();
    // the rows of every level in one load, lane = level
    int rows = -1;
    if (live && lane <= top && c.z[lane]) rows = c.zrow[lane][j];
    auto zrow_of = [&](int r) -> const float2 * {
        const int zr = __builtin_amdgcn_readlane(rows, r);
        return zr >= 0 ? c.z[r] + (int64_t)zr * c.ld_z[r] : nullptr;
    };
    auto even = [](int lo) { return lo & ~1; };   // windows begin at an even index
    auto write_hist = [&](int r, const float2 *win) {
        // the last hh samples of W_r lie inside the last tile's window of level r
        if (live && last && lane < hh) c.whist_new[r][j * hh + lane] = win[(n_out >> r) - hh + lane - even(slo[r])];
    };
    // a level's z, loaded while the level above is formed; pair m0 + 64 u + lane
    constexpr int NU = kTile / 2 / 64;
    static_assert(kWinPairs == 3 && kWinPairs <= NU, "a level's window in one load");
    float2 ev[NU], od[NU];
    auto load = [&](int r) {
        load_pairs<NU>(zrow_of(r), c.ld_z[r], max(slo[r], 0) / 2, lane, min(n_out >> r, shi[r] + 1), ev, od);
    };
    load(top);
    for (int r = top; r >= 1; --r) {
        float2 *win = (r & 1) ? bufA : bufB;
        const float2 *src = (r & 1) ? bufB : bufA;   // W_{r+1}
        const int lo = slo[r], lb = even(lo), qa = max(lo, 0), mlo = qa / 2, np = shi[r] / 2 - mlo + 1;
        float2 e[kWinPairs], o[kWinPairs];
        int mw[kWinPairs];
#pragma unroll
        for (int u = 0; u < kWinPairs; ++u) {
            e[u] = ev[u];
            o[u] = od[u];
            mw[u] = min(u * 64 + lane, np - 1);   // past the window: a repeat, not written
        }
        load(r - 1);
        if (live) {
            for (int q = lo + lane; q < qa; q += 64) win[q - lb] = c.whist[r][j * hh + hh + q];
            if (r < top) {
                const int sb = mlo - even(slo[r + 1]);
                if (np > 128)
                    interp_pairs<3>(src, sb, sg, lg, mw, e, o);
                else if (np > 64)
                    interp_pairs<2>(src, sb, sg, lg, mw, e, o);
                else
                    interp_pairs<1>(src, sb, sg, lg, mw, e, o);
            }
            // whole pairs: what one holds outside the window is not read
            f4v *w4 = reinterpret_cast<f4v *>(win + (2 * mlo - lb));
#pragma unroll
            for (int u = 0; u < kWinPairs; ++u)
                if (u * 64 + lane < np) w4[u * 64 + lane] = f4v{e[u].x, e[u].y, o[u].x, o[u].y};
        }
        // the buffers are the wave's own: its reads follow its writes in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        write_hist(r, win);
    }
    int m[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) m[u] = u * 64 + lane;   // tile offsets 2m, 2m + 1
    if (live) {
        if (top > 0) interp_pairs<NU>(bufA, p0 / 2 - even(slo[1]), sg, lg, m, ev, od);
        if (!KEYS) {
            float2 *oj = out + j * ld_out + p0;
            if (((uintptr_t)oj & 15) == 0 && p0 + kTile <= n_out) {
                f4v *o4 = reinterpret_cast<f4v *>(oj);
#pragma unroll
                for (int u = 0; u < NU; ++u) o4[m[u]] = f4v{ev[u].x, ev[u].y, od[u].x, od[u].y};
            } else {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int p = p0 + 2 * m[u];
                    if (p < n_out) oj[2 * m[u]] = ev[u];
                    if (p + 1 < n_out) oj[2 * m[u] + 1] = od[u];
                }
            }
        }
    }
    if (KEYS) {
        // |z|^2 of each row into its wave's first buffer (free once every wave
        // has read W_1), then per sample the largest key over the chunk's rows
        __syncthreads();
        float *sq = reinterpret_cast<float *>(bufA);
        if (live) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int t = 2 * (u * 64 + lane);
                *reinterpret_cast<float2 *>(sq + t) = make_float2(ev[u].x * ev[u].x + ev[u].y * ev[u].y,
                                                                  od[u].x * od[u].x + od[u].y * od[u].y);
            }
        }
        __syncthreads();
        const int nlive = min(kKeyChunk, T - chunk * kKeyChunk);
        const int wstride = (capA + capB) * 2;   // floats between the waves' buffers
        const float *sq0 = reinterpret_cast<const float *>(wbuf);
        for (int t = threadIdx.x; t < kTile; t += kChainThreads) {
            const int p = p0 + t;
            if (p >= n_out) continue;
            unsigned long long best = 0ull;
            for (int w = 0; w < nlive; ++w) {
                const unsigned long long key = ((unsigned long long)__float_as_uint(sq0[w * wstride + t]) << 32) |
                                               (unsigned long long)(0xFFFFFFFFu - (uint32_t)(chunk * kKeyChunk + w));
                best = key > best ? key : best;
            }
            keys[chunk * ld_keys + p] = best;
        }
    }
}

// The replayed piece's max / argmax out of the graph's buffers, one launch
// for both arrays.
__global__ __launch_bounds__(kThreads) void mr_copy_out_kernel(float *__restrict__ mx, const float *__restrict__ mxo,
                                                               int32_t *__restrict__ am,
                                                               const int32_t *__restrict__ amo, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) {
        mx[i] = mxo[i];
        am[i] = amo[i];
    }
}

}  // namespace

hipError_t launch_mr_copy_out(float *mx, const float *mxo, int32_t *am, const int32_t *amo, int64_t n,
                              hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(mr_copy_out_kernel, dim3((unsigned)nblk(n, kThreads)), dim3(kThreads), 0, st, mx, mxo, am, amo,
                       n);
    return hipGetLastError();
}

hipError_t launch_mr_decimate(const float *src, int64_t n_src, const float *hist, float *hist_new,
                              const float *h, int lh, float *dst, hipStream_t st) {
    const int64_t nq = n_src / 2;
    const int64_t blocks = std::max<int64_t>(1, nblk(nq, kThreads));
    hipLaunchKernelGGL(mr_decimate_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, st, src, n_src, hist,
                       hist_new, h, lh, dst);
    return hipGetLastError();
}

void mr_chain_caps(int top, int lg, int *capA, int *capB) {
    // window lengths: level 1 at most (kTile + lg + 1) / 2, level r at most
    // (len_{r-1} + lg + 1) / 2 + 1; odd levels share buffer A, even ones B
    int cap = kTile;
    *capA = kTile / 2;   // at least the tile's |z|^2 (kTile floats) for the keys
    *capB = 0;
    for (int r = 1; r <= top; ++r) {
        cap = (cap + lg + 1) / 2 + 1;
        int &slot = (r & 1) ? *capA : *capB;
        slot = std::max(slot, (cap + 3) & ~1);   // from an even index to an odd one
    }
}

size_t mr_chain_lds(int top, int lg) {
    int capA = 0, capB = 0;
    mr_chain_caps(top, lg, &capA, &capB);
    return (size_t)kKeyChunk * (size_t)(capA + capB) * sizeof(float2);
}

hipError_t launch_mr_chain(const MrChain &c, int top, int hh, const float *g, int lg, int64_t n_out, int T,
                           uint64_t *keys, int64_t ld_keys, float2 *out, int64_t ld_out, hipStream_t st) {
    if (n_out <= 0) return hipSuccess;
    int capA = 0, capB = 0;
    mr_chain_caps(top, lg, &capA, &capB);
    const size_t lds = mr_chain_lds(top, lg);
    // at most 60,416 bytes (64 taps), within the default 64 KB with the static part
    if (lds > (size_t)kChainLdsMax) return hipErrorInvalidValue;
    if (n_out > INT32_MAX - kTile) return hipErrorInvalidValue;   // tile-local indices are int32
    const int tiles = (int)nblk(n_out, kTile);
    const unsigned grid = (unsigned)(tiles * mr_key_chunks(T));
    const int n = (int)n_out;
    if (keys)
        hipLaunchKernelGGL(mr_chain_kernel<true>, dim3(grid), dim3(kChainThreads), lds, st, c, top, hh, g, lg, n, T,
                           capA, capB, keys, ld_keys, out, ld_out, tiles);
    else
        hipLaunchKernelGGL(mr_chain_kernel<false>, dim3(grid), dim3(kChainThreads), lds, st, c, top, hh, g, lg, n, T,
                           capA, capB, keys, ld_keys, out, ld_out, tiles);
    return hipGetLastError();
}

size_t mr_pyramid_lds(int top, int lh) {
    const int cap0 = kPyrSlice + pyr_reach(0, top, lh), cap1 = top >= 2 ? kPyrSlice / 2 + pyr_reach(1, top, lh) : 0;
    return (size_t)(cap0 + cap1) * sizeof(float);
}

hipError_t launch_mr_pyramid(const float *x, int64_t n, int top, const MrPyramid &pm, const float *h, int lh,
                             hipStream_t st) {
    if (n <= 0 || n > INT32_MAX - kPyrSlice || n % (1 << top)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mr_pyramid_kernel, dim3((unsigned)nblk(n, kPyrSlice)), dim3(kPyrThreads),
                       mr_pyramid_lds(top, lh), st, x, (int)n, top, pm, h, lh, kPyrSlice,
                       kPyrSlice + pyr_reach(0, top, lh));
    return hipGetLastError();
}

int mr_key_chunks(int T) { return (T + kKeyChunk - 1) / kKeyChunk; }

}  // namespace spiir
