// Device kernels of libspiir (gfx950 / CDNA4).
//
// Forward path (Sect. "GPU accelerated SPIIR method", subsection "Optimized
// GPU implementation of SPIIR"): the per-template parameter arrays are loaded
// with coalesced accesses, each filter's output lives in registers across
// iterations, the strain window shared by all filters is staged once per
// workgroup, and the per-template sum of filter outputs is a parallel
// reduction. The MI355X mapping:
//   * one workgroup = up to 8 waves = a packed set of whole templates;
//     every lane holds FL filters of one template in registers;
//   * the delayed strain window x[m - d] of a whole block lives in LDS and is
//     read with immediate offsets (no address arithmetic in the hot loop);
//   * the recursion runs in blocks of 4 steps in a frame that does not rotate;
//   * the template sum is done per tile of 8 time steps: an in-lane sum over
//     the lane's FL filters and a wave-local LDS transpose into sums of 16-lane
//     rows, which all waves add up per template once per 64 steps;
//   * every L samples each filter's carried state gets its FP64 correction
//     (chunked time scan: the chunk-end state is a^L times the chunk-start
//     state plus the in-chunk response);
//   * epilogues: per-template SNR rows, z rows, or a fused per-sample
//     max/argmax encoded as a 64-bit key (SNR bits << 32 | ~template).
#include <hip/hip_ext.h>

#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "spiir_internal.h"

namespace spiir {

namespace {

__device__ __forceinline__ double2 cmul64(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ double2 cpow64(double2 a, int e) {
    double2 r = make_double2(1.0, 0.0);
    while (e > 0) {
        if (e & 1) r = cmul64(r, a);
        a = cmul64(a, a);
        e >>= 1;
    }
    return r;
}

__device__ __forceinline__ float dpp_swap_pairs(float v) {
    // quad_perm [1,0,3,2]: the value of lane ^ 1
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));
}

__device__ __forceinline__ int64_t slot_index(int g, int wpg, int wave, int f, int fl, int lane) {
    return ((int64_t)(g * wpg + wave) * fl + f) * 64 + lane;
}

// Four floats at a 4-byte aligned address (global loads accept this alignment).
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// The recursion y[t] = a y[t-1] + b x[t] in blocks of kRot steps. Inside a
// block the state is kept in a frame that does not rotate: S is y scaled to
// the block's last step, so each input is only added,
//     S <- S + c_j x[j],  c_j = a^(3-j) b     (the block's first step also
//     S <- a^4 S),        y[j] = v_j S,  v_j = a^-(3-j)  (v_3 = 1),
// and the template sum takes v_j S by multiply-adds into the sum. Per update
// that is 6.5 VALU operations with the in-lane sum, against 8 for turning y by
// a every step and adding it (the kernels are bound by VALU issue); the carried
// state also meets one rounded power a^4 per four steps instead of four rounded
// a. On the 1,024-template bank: see the forward kernel's comment.
constexpr int kRot = 4;
// Below this |a| the inverse powers could leave the FP32 range for small
// inputs (|v_0| = |a|^-3; a = 0 is allowed): a wave that holds such a filter
// runs the plain recursion for all of its filters.
constexpr double kRotMin = 0.1;

struct RotCoeffs {
    float2 a4, c[kRot], v[kRot - 1];
};

__device__ __forceinline__ float2 f32c(double2 z) { return make_float2((float)z.x, (float)z.y); }
__device__ __forceinline__ double2 f64c(float2 z) { return make_double2((double)z.x, (double)z.y); }

// FP64 powers, rounded once. |a| < kRotMin: zeros (never used, see above).
__device__ __forceinline__ RotCoeffs rot_coeffs(double2 a, float2 b) {
    RotCoeffs r;
    const double n2 = a.x * a.x + a.y * a.y;
    const bool ok = n2 >= kRotMin * kRotMin;
    const double q = ok ? 1.0 / n2 : 0.0;
    const double2 a2 = cmul64(a, a), b64 = f64c(b), inv = make_double2(a.x * q, -a.y * q), inv2 = cmul64(inv, inv);
    r.a4 = f32c(cmul64(a2, a2));
    r.c[0] = f32c(cmul64(cmul64(a2, a), b64));
    r.c[1] = f32c(cmul64(a2, b64));
    r.c[2] = f32c(cmul64(a, b64));
    r.c[3] = b;
    r.v[0] = f32c(cmul64(inv2, inv));
    r.v[1] = f32c(inv2);
    r.v[2] = f32c(inv);
    return r;
}

// v[j] by value (a choice between the elements' addresses would put the array in memory).
__device__ __forceinline__ float2 rot_v(const float2 (&v)[kRot - 1], int j) {
    const float v0x = v[0].x, v0y = v[0].y, v1x = v[1].x, v1y = v[1].y, v2x = v[2].x, v2y = v[2].y;
    return make_float2(j == 0 ? +v0x : j == 1 ? +v1x : +v2x, j == 0 ? +v0y : j == 1 ? +v1y : +v2y);
}

// What the FP32 recursion above multiplies a carried state by over len steps.
__device__ __forceinline__ double2 rot_pow(float2 a4, const float2 (&v)[kRot - 1], int len) {
    double2 r = cpow64(f64c(a4), len / kRot);
    const int rem = len % kRot;
    if (rem) r = cmul64(r, cmul64(f64c(a4), f64c(rot_v(v, rem - 1))));
    return r;
}

// Per-lane register state of FL filter slots. Plain waves (see kRotMin) hold a
// in a4 and b in c[3].
template <int FL>
struct Lane {
    float2 a4[FL], c[FL][kRot], v[FL][kRot - 1];
    int xo[FL];
    float yr[FL], yi[FL];     // running state (FP32): S inside a block, y between blocks
    float y0r[FL], y0i[FL];   // state at the chunk start (hi part)
    float l0r[FL], l0i[FL];   // low part of the chunk-start carry
    unsigned flags;           // bit f: slot f carries in FP64 (hybrid mode)
    int64_t slot0;            // slot of filter f is slot0 + 64 f
    __device__ __forceinline__ int64_t slot(int f) const { return slot0 + 64 * f; }
};

// x values of a lane's filters, RING rows of one step each, read RING / 2 steps
// ahead of their use: one block in the full pass on an LDS window (a block's
// arithmetic covers the LDS latency), one tile in the state pass (a third of
// the arithmetic) and where the window stays in global memory (VEC).
template <bool SUM, bool VEC>
struct Ring {
    static constexpr int value = VEC || !SUM ? 2 * kFwdTile : kFwdTile;
};

// x[m - d] of every filter for one block of steps, t0 .. t0 + kRot - 1, into
// rows k .. of xv. The window is padded by one tile, so reads past the
// sub-block end stay inside it (their values are never used). The scheduling
// barrier keeps the LDS reads here: left alone, the compiler sinks them to
// just before their use to save registers and every step then waits for the
// LDS. Window in global memory: one 16-byte load.
template <int FL, int ROWS, bool VEC>
__device__ __forceinline__ void load_block(float (&xv)[ROWS][FL], const float *xw, const Lane<FL> &s, int t0, int k) {
    static_assert(kRot == 4, "one 16-byte load per block");
#pragma unroll
    for (int f = 0; f < FL; ++f) {
        const float *xp = xw + (s.xo[f] + t0);
        if (VEC) {
            const f4u q = *reinterpret_cast<const f4u *>(xp);
            xv[k][f] = q.x;
            xv[k + 1][f] = q.y;
            xv[k + 2][f] = q.z;
            xv[k + 3][f] = q.w;
        } else {
#pragma unroll
            for (int t = 0; t < kRot; ++t) xv[k + t][f] = xp[t];
        }
    }
    if (!VEC) __builtin_amdgcn_sched_barrier(0);
}

// One tile of kFwdTile steps: FL filter updates per step and per lane, the lane's
// partial template sum of every step written to the wave's LDS tile
// [kFwdTile][64] (SUM; without it only the states advance). Rows BASE .. of xv
// hold the tile's x, or its first block in a ring of one tile; the rows that
// follow in the ring are read here (AHEAD; without it xv arrives complete).
// Tiles start on a block of kRot steps; a partial tile (not FULL) leaves y.
template <int FL, int ROWS, bool FULL, bool SUM, bool PLAIN, bool VEC, bool AHEAD, int BASE>
__device__ __forceinline__ void compute_tile(Lane<FL> &s, float (&xv)[ROWS][FL], const float *xw, int t0, int steps,
                                             float2 *wt, int lane) {
    constexpr int kLast = kRot - 1;
    static_assert(kFwdTile == 2 * kRot, "ring of two blocks / two tiles");
#pragma unroll
    for (int t = 0; t < kFwdTile; ++t) {
        if (AHEAD && t % kRot == 0) {
            const int u = t + ROWS / 2;   // step whose x is read now
            load_block<FL, ROWS, VEC>(xv, xw, s, t0 + u, (BASE + u) % ROWS);
        }
        if (!FULL && t >= steps) continue;  // uniform; keeps every index static
        const int j = t % kRot;
        float pr = 0.f, pi = 0.f;
#pragma unroll
        for (int f = 0; f < FL; ++f) {
            const float x = xv[BASE + t][f];
            float nr, ni;
            if (PLAIN || j == 0) {
                const float2 m = s.a4[f], c = s.c[f][PLAIN ? kLast : 0];
                nr = fmaf(-m.y, s.yi[f], fmaf(m.x, s.yr[f], c.x * x));
                ni = fmaf(m.y, s.yr[f], fmaf(m.x, s.yi[f], c.y * x));
            } else {
                nr = fmaf(s.c[f][j].x, x, s.yr[f]);
                ni = fmaf(s.c[f][j].y, x, s.yi[f]);
            }
            s.yr[f] = nr;
            s.yi[f] = ni;
            if (!SUM) continue;
            if (PLAIN || j == kLast) {
                pr = f == 0 ? nr : pr + nr;
                pi = f == 0 ? ni : pi + ni;
            } else {
                const float2 v = s.v[f][j < kLast ? j : 0];
                pr = fmaf(-v.y, ni, f == 0 ? v.x * nr : fmaf(v.x, nr, pr));
                pi = fmaf(v.y, nr, f == 0 ? v.x * ni : fmaf(v.x, ni, pi));
            }
        }
        if (SUM) wt[t * 64 + lane] = make_float2(pr, pi);
    }
    if (!FULL && !PLAIN && steps % kRot) {   // S of an unfinished block -> y
#pragma unroll
        for (int f = 0; f < FL; ++f) {
            const float2 v = rot_v(s.v[f], steps % kRot - 1);
            const float yr = fmaf(-v.y, s.yi[f], v.x * s.yr[f]);
            s.yi[f] = fmaf(v.y, s.yr[f], v.x * s.yi[f]);
            s.yr[f] = yr;
        }
    }
}

// A tile outside the ring: waves that run the plain recursion, the last tile
// of a pass that ends inside it, a tile without a partner in a ring of two.
template <int FL, bool SUM, bool VEC>
__device__ __forceinline__ void lone_tile(Lane<FL> &s, const float *xw, int t0, int steps, float2 *wt, int lane,
                                          bool plain) {
    float xv[kFwdTile][FL];
    load_block<FL, kFwdTile, VEC>(xv, xw, s, t0, 0);
    load_block<FL, kFwdTile, VEC>(xv, xw, s, t0 + kRot, kRot);
    if (plain && steps == kFwdTile)
        compute_tile<FL, kFwdTile, true, SUM, true, VEC, false, 0>(s, xv, xw, t0, steps, wt, lane);
    else if (plain)
        compute_tile<FL, kFwdTile, false, SUM, true, VEC, false, 0>(s, xv, xw, t0, steps, wt, lane);
    else
        compute_tile<FL, kFwdTile, false, SUM, false, VEC, false, 0>(s, xv, xw, t0, steps, wt, lane);
}

template <int FL, bool SUM, bool VEC>
__device__ __forceinline__ void fill_ring(const Lane<FL> &s, float (&xv)[Ring<SUM, VEC>::value][FL], const float *xw,
                                          int t0) {
    constexpr int RING = Ring<SUM, VEC>::value;
    load_block<FL, RING, VEC>(xv, xw, s, t0, 0);
    if (RING > kFwdTile) load_block<FL, RING, VEC>(xv, xw, s, t0 + kRot, kRot);
}

// Tiles of steps [t0, t1) of a sub-block, each followed by post(its first step,
// its steps). The ring holds the x that the first tile expects on entry and the
// next tile's at the end (refilled after lone tiles).
template <int FL, bool SUM, bool VEC, class Post>
__device__ __forceinline__ void run_tiles(Lane<FL> &s, float (&xv)[Ring<SUM, VEC>::value][FL], const float *xw, int t0,
                                          int t1, float2 *wt, int lane, bool plain, Post post) {
    constexpr int RING = Ring<SUM, VEC>::value;
    if (!plain) {
        for (; t0 + RING <= t1; t0 += RING) {
            compute_tile<FL, RING, true, SUM, false, VEC, true, 0>(s, xv, xw, t0, kFwdTile, wt, lane);
            post(t0, kFwdTile);
            if (RING > kFwdTile) {
                constexpr int kOdd = RING > kFwdTile ? kFwdTile : 0;
                compute_tile<FL, RING, true, SUM, false, VEC, true, kOdd>(s, xv, xw, t0 + kFwdTile, kFwdTile, wt, lane);
                post(t0 + kFwdTile, kFwdTile);
            }
        }
        if (t0 >= t1) return;
    }
    for (; t0 < t1; t0 += kFwdTile) {
        const int steps = min(kFwdTile, t1 - t0);
        lone_tile<FL, SUM, VEC>(s, xw, t0, steps, wt, lane, plain);
        post(t0, steps);
    }
    if (!plain) fill_ring<FL, SUM, VEC>(s, xv, xw, t1);
}

// Row sums of a wave tile: wsum[t][4 * wave + r] = sum of the 16 lanes of row
// r at step t. Tile row k = 4 t + r is 128 bytes = four 32-byte units. Lanes
// 2p and 2p+1 read the two halves of one unit together (the LDS serves a
// ds_read_b128 per lane pair), and pair p walks its row's units in an order
// rotated by p / 2, so the 8 pairs served in one cycle hit distinct banks.
// Each lane sums its halves; one DPP swap adds the partner's half. The reads
// (row_reads) are issued right after the tile's writes - a wave's LDS
// operations take effect in order, so neither they nor the next tile's writes
// need a wait - and are added up after the next tile's recursion (row_add),
// which hides their latency.
struct RowReads {
    float4 v[4];
};

__device__ __forceinline__ RowReads row_reads(const float2 *wt, int lane) {
    const char *base = reinterpret_cast<const char *>(wt);
    const int p = lane >> 1, h = lane & 1;
    RowReads r;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = (i + (p >> 1)) & 3;
        r.v[i] = *reinterpret_cast<const float4 *>(base + p * 128 + (2 * q + h) * 16);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    return r;
}

__device__ __forceinline__ void row_add(const RowReads &r, float2 *wsum, int Rp, int wave, int lane) {
    const float sx = ((r.v[0].x + r.v[0].z) + (r.v[1].x + r.v[1].z)) +
                     ((r.v[2].x + r.v[2].z) + (r.v[3].x + r.v[3].z));
    const float sy = ((r.v[0].y + r.v[0].w) + (r.v[1].y + r.v[1].w)) +
                     ((r.v[2].y + r.v[2].w) + (r.v[3].y + r.v[3].w));
    const float ox = dpp_swap_pairs(sx), oy = dpp_swap_pairs(sy);
    const int k = lane >> 1;
    if ((lane & 1) == 0) wsum[(k >> 2) * Rp + wave * 4 + (k & 3)] = make_float2(sx + ox, sy + oy);
}

// xs[i] = src[off + i] (0 if ZERO) for i in [i0, i1), by the whole workgroup:
// a scalar head up to a 16-byte LDS boundary, then 16-byte global loads (4-byte
// aligned) with four per thread in flight and 16-byte LDS stores, then a scalar
// tail. Indices off + i are in range for every i in [i0, i1). Returns the
// largest magnitude that the thread saw.
template <bool ZERO>
__device__ __forceinline__ float stage_range(float *xs, const float *src, int64_t off, int i0, int i1) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int ia = min(i1, (i0 + 3) & ~3);
    float top = 0.f;
    for (int i = i0 + tid; i < ia; i += nt) {
        xs[i] = ZERO ? 0.f : src[off + i];
        if (!ZERO) top = fmaxf(top, fabsf(xs[i]));
    }
    const int nv = (i1 - ia) >> 2;
    for (int v0 = tid; v0 < nv; v0 += 4 * nt) {
        float4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + u * nt;
            q[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (!ZERO && v < nv) {
                const f4u w = *reinterpret_cast<const f4u *>(src + (off + ia + 4 * (int64_t)v));
                q[u] = make_float4(w.x, w.y, w.z, w.w);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + u * nt;
            if (v < nv) *reinterpret_cast<float4 *>(xs + ia + 4 * v) = q[u];
            if (!ZERO) {
                top = fmaxf(fmaxf(top, fabsf(q[u].x)), fabsf(q[u].y));
                top = fmaxf(fmaxf(top, fabsf(q[u].z)), fabsf(q[u].w));
            }
        }
    }
    for (int i = ia + 4 * nv + tid; i < i1; i += nt) {
        xs[i] = ZERO ? 0.f : src[off + i];
        if (!ZERO) top = fmaxf(top, fabsf(xs[i]));
    }
    return top;
}

// Template sum over its nr row sums of one step, in a fixed order.
__device__ __forceinline__ float2 sum_rows(const float2 *ws, int nr) {
    float zr = 0.f, zi = 0.f;
    int r = 0;
    for (; r + 4 <= nr; r += 4) {
        const float2 v0 = ws[r], v1 = ws[r + 1], v2 = ws[r + 2], v3 = ws[r + 3];
        zr += (v0.x + v1.x) + (v2.x + v3.x);
        zi += (v0.y + v1.y) + (v2.y + v3.y);
    }
    for (; r < nr; ++r) {
        zr += ws[r].x;
        zi += ws[r].y;
    }
    return make_float2(zr, zi);
}

// Chunk-end correction of the carried state (len = samples in the chunk).
template <int FL>
__device__ __forceinline__ void carry_correct(Lane<FL> &s, const SlotArrays &sa, int prec, bool plain,
                                              int len, int L) {
#pragma unroll
    for (int f = 0; f < FL; ++f) {
        float hr = s.yr[f], hi = s.yi[f], lr = 0.f, li = 0.f;
        if (prec != kPrecFp32) {
            double2 al, dl;
            if (len == L && !plain) {
                al = sa.aL[s.slot(f)];
                dl = sa.dL[s.slot(f)];
            } else {
                al = cpow64(sa.a64[s.slot(f)], len);
                const double2 ah = plain ? cpow64(f64c(s.a4[f]), len) : rot_pow(s.a4[f], s.v[f], len);
                dl = make_double2(al.x - ah.x, al.y - ah.y);
            }
            if (prec == kPrecFp64 || ((s.flags >> f) & 1u)) {
                // c_end = y_end + (a^l - what FP32 carried) * hi_start + a^l * lo_start, in FP64
                const double y0r = s.y0r[f], y0i = s.y0i[f], l0r = s.l0r[f], l0i = s.l0i[f];
                const double cr = (double)hr + (dl.x * y0r - dl.y * y0i) + (al.x * l0r - al.y * l0i);
                const double ci = (double)hi + (dl.x * y0i + dl.y * y0r) + (al.x * l0i + al.y * l0r);
                hr = (float)cr;
                hi = (float)ci;
                lr = (float)(cr - (double)hr);
                li = (float)(ci - (double)hi);
            } else {
                const float dr = (float)dl.x, di = (float)dl.y;
                hr = fmaf(dr, s.y0r[f], fmaf(-di, s.y0i[f], hr));
                hi = fmaf(dr, s.y0i[f], fmaf(di, s.y0r[f], hi));
            }
        }
        s.yr[f] = hr;
        s.yi[f] = hi;
        s.y0r[f] = hr;
        s.y0i[f] = hi;
        s.l0r[f] = lr;
        s.l0i[f] = li;
    }
}

// Time range and state routing of one workgroup item.
struct SegCtx {
    int64_t tb, tn;          // launch samples [tb, tb + tn)
    const float4 *st_in;     // initial state per slot (null: cold start), entry slot - in_off
    float4 *st_out;          // final state per slot (null: not stored), entry slot - out_off
    int64_t in_off, out_off;
    // seg > 0: the initial state is composed from the end states of the segments before it,
    // st_in[k * stride] for segment k (segment 0's from the carried state), each `len` samples
    int seg;
    int64_t stride, len;
};

// One step of the carry chain: c <- al c + e, e = hi + lo.
__device__ __forceinline__ void chain_step(double2 &c, double2 al, float4 e) {
    const double2 m = cmul64(al, c);
    c.x = m.x + ((double)e.x + (double)e.z);
    c.y = m.y + ((double)e.y + (double)e.w);
}

__device__ __forceinline__ float4 hi_lo(double2 c) {
    const float hr = (float)c.x, hi = (float)c.y;
    return make_float4(hr, hi, (float)(c.x - (double)hr), (float)(c.y - (double)hi));
}

// Up to this many segments every workgroup of the full pass composes its own
// start state (at most 15 reads per slot); beyond it a launch of its own does.
// The launch costs about 6 us with its gaps: 21.7 -> 15.1 us per 512-sample
// call of a 4 x 128-filter bank.
constexpr int kChainInline = 16;

// Coefficients and initial states of a lane's slots; true if the wave runs
// the plain recursion. The block powers are formed here in FP64 (full rate on
// this chip): 72 bytes of tables less to read per slot and launch.
template <int FL>
__device__ __forceinline__ bool load_lane(Lane<FL> &s, const FwdArgs &p, int g, int wave, int lane, bool ract,
                                          int xshift, const SegCtx &sc) {
    s.slot0 = slot_index(g, p.wpg, wave, 0, FL, lane);
    s.flags = 0u;
    double2 a[FL];
    float2 b[FL];
    bool small = false;
#pragma unroll
    for (int f = 0; f < FL; ++f) {
        a[f] = make_double2(0.0, 0.0);
        b[f] = make_float2(0.f, 0.f);
        s.xo[f] = 0;
        float4 st = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ract) {
            a[f] = p.s.a64[s.slot(f)];
            if (p.prec == kPrecFp32) a[f] = f64c(f32c(a[f]));
            b[f] = p.s.b32[s.slot(f)];
            s.xo[f] = p.s.xoff[s.slot(f)] - xshift;
            s.flags |= (unsigned)(p.s.flags[s.slot(f)] & 1) << f;
            if (sc.st_in && sc.seg <= 1) st = sc.st_in[s.slot(f) - sc.in_off];
            if (sc.seg > 1) {
                float4 e[kChainInline - 1];
#pragma unroll
                for (int k = 0; k < kChainInline - 1; ++k)
                    if (k < sc.seg) e[k] = sc.st_in[(int64_t)k * sc.stride + s.slot(f) - sc.in_off];
                const double2 al = cpow64(a[f], (int)sc.len);
                double2 c = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < kChainInline - 1; ++k)
                    if (k < sc.seg) chain_step(c, al, e[k]);
                st = hi_lo(c);
            }
        }
        s.yr[f] = s.y0r[f] = st.x;
        s.yi[f] = s.y0i[f] = st.y;
        s.l0r[f] = st.z;
        s.l0i[f] = st.w;
        // padding slots (a = b = 0) stay zero in either form
        const double n2 = a[f].x * a[f].x + a[f].y * a[f].y;
        small = small || (n2 < kRotMin * kRotMin && (n2 > 0.0 || b[f].x != 0.f || b[f].y != 0.f));
    }
    const bool plain = __ballot(small) != 0;
#pragma unroll
    for (int f = 0; f < FL; ++f) {
        const RotCoeffs r = rot_coeffs(a[f], b[f]);
        s.a4[f] = plain ? f32c(a[f]) : r.a4;
#pragma unroll
        for (int j = 0; j < kRot; ++j) s.c[f][j] = r.c[j];
#pragma unroll
        for (int j = 0; j < kRot - 1; ++j) s.v[f][j] = r.v[j];
    }
    return plain;
}

// An infinite sample makes S infinite in both parts, and the products v_j S are then NaN in
// the steps of its block where y is still infinite: a workgroup whose window holds one
// runs the plain recursion from that window on. Windows in LDS are looked over while they are
// staged, those in global memory while they are filled (one mark per kMarkSamples). That
// costs 6 us of the headline call's 450 (rows; the fused call is 5 us faster), nothing that
// shows in the time-split calls, 1 us of 31 with the window in global memory. A vote on the
// final states and a second run of the whole item cost 0.4 us per launch.
template <int FL>
__device__ __forceinline__ void to_plain(Lane<FL> &s, const FwdArgs &p, bool ract) {
#pragma unroll
    for (int f = 0; f < FL; ++f)
        if (ract) s.a4[f] = p.s.a32[s.slot(f)];   // c[3] is b in both forms
}

// Stages xs[i] = x[m0 + i], i in [0, gw + nbs), m0 = first sample - glo - gw;
// samples before x[0] come from the history. Sets *inf if one of them is infinite.
// The caller syncs around it.
__device__ __forceinline__ void stage_window(float *xs, const FwdArgs &p, int64_t xfirst, int glo, int gw, int nbs,
                                             int *inf) {
    const int cnt = gw + nbs;
    const int64_t m0 = xfirst - glo - gw;
    const int nneg = (int)min((int64_t)cnt, max((int64_t)0, -m0));
    // a band's window may reach past the largest delay (glo + gw > max_delay):
    // samples before the history (m < -max_delay) are read by no filter and
    // staged as zeros, so the history is only read at indices >= 0
    const int nz = (int)min((int64_t)nneg, max((int64_t)0, -(int64_t)p.dmax - m0));
    float top = 0.f;
    if (p.hist) {
        stage_range<true>(xs, nullptr, 0, 0, nz);
        top = stage_range<false>(xs, p.hist, p.dmax + m0, nz, nneg);
    } else {
        stage_range<true>(xs, nullptr, 0, 0, nneg);
    }
    top = fmaxf(top, stage_range<false>(xs, p.x, m0, nneg, cnt));
    if (top > FLT_MAX) *inf = 1;
}

// This lane's share of the same question for a window in global memory, from the marks
// that its fill left (one per kMarkSamples): two loads that nothing waits for before the
// coefficients are there, more only beyond 128 marks.
__device__ __forceinline__ int window_marked(const FwdArgs &p, int64_t xfirst, int nbs) {
    if (!p.xmark) return 0;
    const int64_t m0 = xfirst / kMarkSamples + (threadIdx.x & 63), m1 = (xfirst + p.dmax + nbs - 1) / kMarkSamples;
    const int a = p.xmark[min(m0, m1)], b = p.xmark[min(m0 + 64, m1)];
    if (xfirst / kMarkSamples + 128 > m1) return a | b;
    int more = 0;
    for (int64_t m = m0 + 128; m <= m1; m += 64) more |= p.xmark[m];
    return a | b | more;
}

__host__ __device__ __forceinline__ size_t window_bytes(int gw, int nb) {
    return (size_t)((gw + nb + kFwdTile + 3) & ~3) * 4;
}

// The whole forward pass of workgroup g over launch samples [sc.tb, sc.tb + sc.tn).
// The waves run tiles on their own and meet once per batch of sumb (64) steps,
// when every row sum of the batch is in LDS: then each wave takes some of the
// workgroup's templates, lane = step, adds their row sums and writes 64
// consecutive samples.
// Bound: VALU issue at 2 waves per SIMD (FL = 4: 230 registers), so a wave that
// waits is hardly covered. Per 4,096-sample call of the 1,024-template bank:
// 541 us with the rotating recursion (8 operations per update), a barrier per
// 16 steps and the template sums on the waves that hold a template's first row;
// 577 with blocks of 4 steps alone (its LDS reads were sunk to their use), 545
// with the reads pinned a block ahead, 507 with batches of 64 steps and the
// row-sum reads left in flight, 463 with a hot loop that no other case joins:
// 7.1 operations per update, 4.06e12 updates/s.
// PARTS: the bank has templates split over workgroups (rows with part >= 0);
// banks without them run the variant that has no part branch.
template <int FL, int MODE, bool XLDS, bool PARTS = false>
__device__ void fwd_group(const FwdArgs &p, int g, unsigned char *smem, const SegCtx &sc) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = p.wpg, R = 4 * W, Rp = R + 1;  // odd row stride of wsum: no bank aliasing over steps
    // LDS window: x[m - d] for the group's delays d in [glo, glo + gw]; slot offsets are
    // max_delay - d, so a lane's window offset is that minus (max_delay - glo - gw)
    const int glo = XLDS && p.group_lo ? p.group_lo[g] : 0;
    const int gw = XLDS ? p.band_w : p.dmax;
    const size_t win_bytes = XLDS ? window_bytes(gw, p.nb) : 0;
    float *xs = reinterpret_cast<float *>(smem);
    float2 *tiles = reinterpret_cast<float2 *>(smem + win_bytes);
    float2 *wt = tiles + wave * kFwdTile * 64;
    const int sb = p.sumb;
    float2 *wsum = tiles + W * kFwdTile * 64;   // [2][sb][Rp]
    unsigned long long *kmax = reinterpret_cast<unsigned long long *>(wsum + 2 * sb * Rp);  // [2][sb]

    const RowInfo ri = p.rows[(int64_t)g * R + wave * 4 + (lane >> 4)];
    const bool ract = ri.tpl >= 0 && (p.only_tpl < 0 || ri.tpl == p.only_tpl);
    const bool wact = __ballot(ract) != 0;
    // the workgroup's templates: lane i of every wave holds the first row of template i
    RowInfo it = {-1, 0, 0, -1};
    if (lane < R) it = p.rows[(int64_t)g * R + lane];
    unsigned long long first = __ballot(it.tpl >= 0 && it.r0 == lane && (p.only_tpl < 0 || it.tpl == p.only_tpl));
    const int ni = __popcll(first);
    {
        int from = lane;   // the lane holding the first row of template `lane`
        for (int i = 0; i < ni; ++i) {
            if (lane == i) from = __ffsll(first) - 1;
            first &= first - 1;
        }
        it = RowInfo{__shfl(it.tpl, from), __shfl(it.r0, from), __shfl(it.nr, from), __shfl(it.part, from)};
    }
    if (MODE == kModeKeys)
        for (int i = tid; i < 2 * sb; i += W * 64) kmax[i] = 0ull;

    __shared__ int inf;
    if (tid == 0) inf = 0;
    int marked = XLDS ? 0 : window_marked(p, p.xbase + sc.tb, (int)min((int64_t)p.nb, sc.tn));
    Lane<FL> s;
    bool plain = load_lane<FL>(s, p, g, wave, lane, ract, p.dmax - glo - gw, sc);
    const int64_t n = sc.tn;
    const int64_t xbase = p.xbase + sc.tb;

    int chunk_done = 0;   // samples of the current chunk so far
    int buf = 0, pend_steps = 0;
    int64_t pend_t = 0;
    float xv[Ring<true, !XLDS>::value][FL];
    RowReads rr;

    auto flush_keys = [&](int b) {   // the keys of the batch before the last barrier
        if (MODE == kModeKeys && wave == 0 && lane < pend_steps) {
            p.keys[(int64_t)g * p.ld + sc.tb + pend_t + lane] = kmax[b * sb + lane];
            kmax[b * sb + lane] = 0ull;
        }
    };
    // template sums and outputs of one batch: launch samples sc.tb + t + [0, steps)
    auto emit = [&](int64_t t, int steps) {
        unsigned long long best = 0ull;
        for (int i = wave; i < ni; i += W) {
            const int r0 = __builtin_amdgcn_readlane(it.r0, i), nr = __builtin_amdgcn_readlane(it.nr, i);
            const int tpl = __builtin_amdgcn_readlane(it.tpl, i), part = __builtin_amdgcn_readlane(it.part, i);
            if (lane >= steps) continue;
            const float2 z = sum_rows(wsum + (buf * sb + lane) * Rp + r0, nr);
            if (PARTS && part >= 0) {
                // one part of a template split over workgroups: its partial sum goes to the
                // part's row; the parts are added before the mode's output
                p.zpart[(int64_t)part * p.ld_part + sc.tb + t + lane] = z;
            } else if (MODE == kModeSnr) {
                p.snr[(int64_t)tpl * p.ld + p.obase + sc.tb + t + lane] = z.x * z.x + z.y * z.y;
            } else if (MODE == kModeZ) {
                p.z[(int64_t)tpl * p.ld + p.obase + sc.tb + t + lane] = z;
            } else {
                const float sn = z.x * z.x + z.y * z.y;
                const unsigned long long key = ((unsigned long long)__float_as_uint(sn) << 32) |
                                               (unsigned long long)(0xFFFFFFFFu - (uint32_t)tpl);
                best = key > best ? key : best;
            }
        }
        if (MODE == kModeKeys && best != 0ull) atomicMax(&kmax[buf * sb + lane], best);
    };

    // Sub-blocks from launch sample `from` on, up to the first whose window holds an infinite
    // sample; with COLD all of them, in the plain recursion, the first one's window being
    // staged. Two instances: one loop for both cost the headline call 2.5 %.
    auto sub_blocks = [&](auto cold, int64_t from) -> int64_t {
        constexpr bool COLD = decltype(cold)::value;
        for (int64_t s0 = from; s0 < n; s0 += p.nb) {
            const int nbs = (int)min((int64_t)p.nb, n - s0);
            const float *xw = XLDS ? xs : p.xwin + (xbase + s0);
            if (!COLD || s0 > from) {
                __syncthreads();
                if (XLDS) {
                    stage_window(xs, p, xbase + s0, glo, gw, nbs, &inf);
                    __syncthreads();
                } else if (s0 > 0) {
                    marked = window_marked(p, xbase + s0, nbs);
                }
            }
            // the same answer in every wave
            if (!COLD && (XLDS ? __builtin_amdgcn_readfirstlane(inf) != 0 : __ballot(marked != 0) != 0)) return s0;
            const bool pl = COLD || plain;
            if (wact && !pl) fill_ring<FL, true, !XLDS>(s, xv, xw, 0);

            for (int b0 = 0; b0 < nbs; b0 += sb) {
                const int bsteps = min(sb, nbs - b0);
                if (wact) {
                    float2 *ws = wsum + buf * sb * Rp;
                    run_tiles<FL, true, !XLDS>(s, xv, xw, b0, b0 + bsteps, wt, lane, pl, [&](int t0, int steps) {
                        if (t0 > b0) {
                            row_add(rr, ws, Rp, wave, lane);
                            ws += kFwdTile * Rp;
                        }
                        rr = row_reads(wt, lane);
                        chunk_done += steps;
                        if (chunk_done == p.L) {
                            carry_correct<FL>(s, p.s, p.prec, pl, p.L, p.L);
                            chunk_done = 0;
                        }
                    });
                    row_add(rr, ws, Rp, wave, lane);
                }
                __syncthreads();
                flush_keys(buf ^ 1);
                emit(s0 + b0, bsteps);
                pend_t = s0 + b0;
                pend_steps = bsteps;
                buf ^= 1;
            }
        }
        return n;
    };
    const int64_t from = sub_blocks(std::false_type(), 0);
    if (from < n) {
        to_plain<FL>(s, p, ract);
        plain = true;
        sub_blocks(std::true_type(), from);
    }
    if (wact && chunk_done) carry_correct<FL>(s, p.s, p.prec, plain, chunk_done, p.L);
    if (MODE == kModeKeys) {
        __syncthreads();
        flush_keys(buf ^ 1);
    }
    if (ract && sc.st_out) {
#pragma unroll
        for (int f = 0; f < FL; ++f)
            sc.st_out[s.slot(f) - sc.out_off] = make_float4(s.yr[f], s.yi[f], s.l0r[f], s.l0i[f]);
    }
}

// The states of workgroup g alone over launch samples [sc.tb, sc.tb + sc.tn):
// no template sums, no output rows, no barrier but the window's.
template <int FL, bool XLDS>
__device__ void state_group(const FwdArgs &p, int g, unsigned char *smem, const SegCtx &sc, float4 *st_copy) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int glo = XLDS && p.group_lo ? p.group_lo[g] : 0;
    const int gw = XLDS ? p.band_w : p.dmax;
    float *xs = reinterpret_cast<float *>(smem);
    const RowInfo ri = p.rows[(int64_t)g * 4 * p.wpg + wave * 4 + (lane >> 4)];
    const bool ract = ri.tpl >= 0 && (p.only_tpl < 0 || ri.tpl == p.only_tpl);
    const bool wact = __ballot(ract) != 0;
    __shared__ int inf;
    if (threadIdx.x == 0) inf = 0;
    int marked = XLDS ? 0 : window_marked(p, p.xbase + sc.tb, (int)min((int64_t)p.nb, sc.tn));
    Lane<FL> s;
    bool plain = load_lane<FL>(s, p, g, wave, lane, ract, p.dmax - glo - gw, sc);
    if (ract && st_copy) {
#pragma unroll
        for (int f = 0; f < FL; ++f)
            st_copy[s.slot(f) - sc.out_off] = make_float4(s.yr[f], s.yi[f], s.l0r[f], s.l0i[f]);
    }
    const int64_t n = sc.tn, xbase = p.xbase + sc.tb;
    int chunk_done = 0;
    float xv[Ring<false, !XLDS>::value][FL];
    auto sub_blocks = [&](auto cold, int64_t from) -> int64_t {   // as in fwd_group
        constexpr bool COLD = decltype(cold)::value;
        for (int64_t s0 = from; s0 < n; s0 += p.nb) {
            const int nbs = (int)min((int64_t)p.nb, n - s0);
            const float *xw = XLDS ? xs : p.xwin + (xbase + s0);
            if (!COLD || s0 > from) {
                if (XLDS) {
                    __syncthreads();
                    stage_window(xs, p, xbase + s0, glo, gw, nbs, &inf);
                    __syncthreads();
                } else if (s0 > 0) {
                    marked = window_marked(p, xbase + s0, nbs);
                }
            }
            if (!COLD && (XLDS ? __builtin_amdgcn_readfirstlane(inf) != 0 : __ballot(marked != 0) != 0)) return s0;
            const bool pl = COLD || plain;
            if (!wact) continue;
            if (!pl) fill_ring<FL, false, !XLDS>(s, xv, xw, 0);
            for (int t0 = 0; t0 < nbs;) {   // whole stretches up to a chunk end
                const int t1 = min(nbs, t0 + p.L - chunk_done);
                run_tiles<FL, false, !XLDS>(s, xv, xw, t0, t1, nullptr, lane, pl, [](int, int) {});
                chunk_done += t1 - t0;
                t0 = t1;
                if (chunk_done == p.L) {
                    carry_correct<FL>(s, p.s, p.prec, pl, p.L, p.L);
                    chunk_done = 0;
                }
            }
        }
        return n;
    };
    const int64_t from = sub_blocks(std::false_type(), 0);
    if (from < n) {
        to_plain<FL>(s, p, ract);
        plain = true;
        sub_blocks(std::true_type(), from);
    }
    if (wact && chunk_done) carry_correct<FL>(s, p.s, p.prec, plain, chunk_done, p.L);
    if (ract && sc.st_out) {
#pragma unroll
        for (int f = 0; f < FL; ++f)
            sc.st_out[s.slot(f) - sc.out_off] = make_float4(s.yr[f], s.yi[f], s.l0r[f], s.l0i[f]);
    }
}

__device__ __forceinline__ SegCtx whole_launch(const FwdArgs &p) {
    SegCtx sc;
    sc.tb = 0;
    sc.tn = p.n;
    sc.st_in = p.state;
    sc.st_out = p.state;
    sc.in_off = 0;
    sc.out_off = 0;
    sc.seg = 0;
    return sc;
}

__device__ __forceinline__ void hist_copy_at(const HistCopy &hc, int i) {
    const int64_t m = hc.n - hc.dmax + i;
    hc.new_h[i] = m >= 0 ? hc.x[m] : hc.old_h[hc.dmax + m];
}

// A streaming call's last launch also writes the next call's history (hc.dmax >
// 0); it reads old_h and x only, which the launch does not write.
__device__ __forceinline__ void hist_copy_part(const HistCopy &hc, int block, int blocks) {
    for (int i = block * blockDim.x + threadIdx.x; i < hc.dmax; i += blocks * blockDim.x) hist_copy_at(hc, i);
}

__device__ __forceinline__ void hist_copy_all(const HistCopy &hc) { hist_copy_part(hc, blockIdx.x, gridDim.x); }

template <int FL, int MODE, bool XLDS, bool PARTS>
__global__ void __launch_bounds__(512) fwd_kernel(FwdArgs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if constexpr (MODE != kModeKeys) hist_copy_all(p.hist_next);
    const SegCtx sc = whole_launch(p);
    fwd_group<FL, MODE, XLDS, PARTS>(p, p.gbase + blockIdx.x, smem, sc);
}

// Time split: the launch's samples in nseg segments that run in parallel.
// Every segment but the last is first run for its states alone (segment 0
// from the carried state, the others from rest), seg_chain_kernel composes the
// segments' true start states in FP64, and then every segment runs in full
// from its true start. The state pass costs 4.4 VALU operations per update (3 of them the
// recursion, the rest window reads, chunk ends and the start); the
// other way round (every segment in full from rest, then the free response of
// the true starts added to stored template sums) cost about 6.5 and wrote and
// read the sums. 64 x 1,000 filters, 16,384 samples, 16 segments: state pass
// 107 us + full pass 241 us, against 296 + 172 us.
__device__ __forceinline__ SegCtx segment(const FwdArgs &p, int seg) {
    SegCtx sc;
    sc.tb = (int64_t)seg * p.seg_len;
    sc.tn = min(p.seg_len, p.n - sc.tb);
    sc.st_in = nullptr;
    sc.st_out = nullptr;
    sc.in_off = p.seg_slot0;
    sc.out_off = 0;
    sc.seg = 0;
    sc.stride = p.seg_stride;
    sc.len = p.seg_len;
    return sc;
}

template <int FL, bool XLDS>
__device__ __forceinline__ void pre_item(const FwdArgs &p, unsigned bid, unsigned char *smem) {
    const int g = p.gbase + bid % p.groups, seg = bid / p.groups;
    SegCtx sc = segment(p, seg);
    if (seg == 0) {
        sc.st_in = p.state;
        sc.in_off = 0;
    }
    sc.st_out = p.seg_end + (int64_t)seg * p.seg_stride;
    sc.out_off = p.seg_slot0;
    // the full pass overwrites p.state while it runs: its segment 0 starts from this copy
    state_group<FL, XLDS>(p, g, smem, sc, seg == 0 && p.chain_inline ? p.seg_start : nullptr);
}

template <int FL, int MODE, bool XLDS, bool PARTS>
__device__ __forceinline__ void seg_item(const FwdArgs &p, unsigned bid, unsigned char *smem) {
    const int g = p.gbase + bid % p.groups, seg = bid / p.groups;
    SegCtx sc = segment(p, seg);
    if (sc.tn == p.n) {   // the one segment of a bank in a group
        sc.st_in = p.state;
    } else if (p.chain_inline && seg > 0) {
        sc.st_in = p.seg_end;
        sc.seg = seg;
    } else {
        sc.st_in = p.seg_start + (int64_t)seg * p.seg_stride;
    }
    if (sc.tb + sc.tn == p.n) sc.st_out = p.state;
    fwd_group<FL, MODE, XLDS, PARTS>(p, g, smem, sc);
}

template <int FL, bool XLDS>
__global__ void __launch_bounds__(512) fwd_pre_kernel(FwdArgs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    pre_item<FL, XLDS>(p, blockIdx.x, smem);
}

template <int FL, int MODE, bool XLDS, bool PARTS>
__global__ void __launch_bounds__(512) fwd_seg_kernel(FwdArgs p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (p.chain_inline) hist_copy_all(p.hist_next);
    seg_item<FL, MODE, XLDS, PARTS>(p, blockIdx.x, smem);
}

// True start states of one slot's segments: start[0] = the carried state, c_1 =
// e_0 (segment 0 ran from the carried state), c_{k+1} = a^seg_len c_k + e_k in
// FP64 (e_k: segment k's end state from rest; every segment but the last has
// seg_len samples). A block takes 64 slots; its four waves take a quarter each
// of up to 64 end states, compose it from rest, exchange the four results and
// write the states from the true start of their quarter: one read latency and
// half the dependent chain of a thread per slot (29.7 us for 64 segments).
__device__ __forceinline__ void chain_segments(const float4 *seg_end, float4 *seg_start, int64_t stride, int64_t sl,
                                               bool act, float4 state, double2 a, int nseg, int64_t seg_len) {
    __shared__ double2 loc[4][64];
    constexpr int kPer = 16;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const double2 al = cpow64(a, (int)seg_len);
    double2 c0 = make_double2(0.0, 0.0);   // true state before end state `base`
    if (act && q == 0) seg_start[sl] = state;
    for (int base = 0; base < nseg - 1; base += 4 * kPer) {
        const int ne = min(4 * kPer, nseg - 1 - base), per = (ne + 3) / 4;
        const int k0 = min(ne, q * per), cnt = min(ne, k0 + per) - k0;
        float4 e[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (act && u < cnt) e[u] = seg_end[(int64_t)(base + k0 + u) * stride + sl];
        double2 c = make_double2(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (act && u < cnt) chain_step(c, al, e[u]);
        __syncthreads();   // the exchange of the previous 64
        loc[q][lane] = c;
        __syncthreads();
        const double2 ap = cpow64(al, per);
        c = c0;
        for (int k = 0; k < 4; ++k) {   // quarters before a non-empty one hold `per` end states
            const double2 m = cmul64(ap, c0), t = loc[k][lane];
            c0 = make_double2(m.x + t.x, m.y + t.y);
            if (k + 1 == q) c = c0;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (act && u < cnt) {
                chain_step(c, al, e[u]);
                seg_start[(int64_t)(base + k0 + u + 1) * stride + sl] = hi_lo(c);
            }
    }
}

// What a carried state is multiplied by per sample in the chain: a, or the
// rounded coefficient in the all-FP32 mode.
__device__ __forceinline__ double2 chain_coeff(const FwdArgs &p, int64_t sl) {
    return p.prec == kPrecFp32 ? f64c(p.s.a32[sl]) : p.s.a64[sl];
}

// Time split, carry chain over slots [seg_slot0, seg_slot0 + seg_stride) of
// the segment buffers; with only_tpl >= 0 only that template's slots (the
// other slots' entries were not written by the state pass).
__device__ __forceinline__ void chain_item(const FwdArgs &p, int fl, int nseg, unsigned chain_blocks, unsigned bid) {
    if (bid >= chain_blocks) {   // the history copy (hist_next.dmax > 0), 256 samples per block
        const int i = (int)(bid - chain_blocks) * 256 + (int)threadIdx.x;
        if (i < p.hist_next.dmax) hist_copy_at(p.hist_next, i);
        return;
    }
    if (nseg < 2) return;
    const int64_t i = (int64_t)bid * 64 + (threadIdx.x & 63), sl = p.seg_slot0 + i;
    bool act = i < p.seg_stride;  // every slot, padding included (its states stay zero)
    if (act && p.only_tpl >= 0) {
        // slot = ((group * wpg + wave) * fl + f) * 64 + lane; row = 4 (group * wpg + wave) + lane / 16
        act = p.rows[((sl >> 6) / fl) * 4 + ((sl & 63) >> 4)].tpl == p.only_tpl;
    }
    float4 st = make_float4(0.f, 0.f, 0.f, 0.f);
    double2 a = make_double2(0.0, 0.0);
    if (act) {
        st = p.state[sl];
        a = chain_coeff(p, sl);
    }
    chain_segments(p.seg_end, p.seg_start, p.seg_stride, i, act, st, a, nseg, p.seg_len);
}

__global__ void __launch_bounds__(256) seg_chain_kernel(FwdArgs p, int fl, int nseg, unsigned chain_blocks) {
    chain_item(p, fl, nseg, chain_blocks, blockIdx.x);
}

// Several banks' time-split passes, one launch per pass for all of them: the
// workgroups [first[b], first[b + 1]) of a pass run bank b's items (its own
// strain, segments, state and output rows) exactly as the one-bank kernels do.
__device__ __forceinline__ int multi_bank(const int32_t *first, int count) {
    int b = 0;
    while (b + 1 < count && (int)blockIdx.x >= first[b + 1]) ++b;
    return b;
}

template <int FL>
__global__ void __launch_bounds__(512) fwd_pre_multi_kernel(MultiFwd m) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = multi_bank(m.pre_first, m.count);
    pre_item<FL, true>(m.a[b], blockIdx.x - (unsigned)m.pre_first[b], smem);
}

template <int FL, int MODE>
__global__ void __launch_bounds__(512) fwd_seg_multi_kernel(MultiFwd m) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = multi_bank(m.seg_first, m.count);
    if (m.a[b].chain_inline)
        hist_copy_part(m.a[b].hist_next, blockIdx.x - (unsigned)m.seg_first[b], m.seg_first[b + 1] - m.seg_first[b]);
    seg_item<FL, MODE, true, false>(m.a[b], blockIdx.x - (unsigned)m.seg_first[b], smem);
}

__global__ void __launch_bounds__(256) seg_chain_multi_kernel(MultiFwd m, int fl) {
    const int b = multi_bank(m.chain_first, m.count);
    chain_item(m.a[b], fl, m.nseg[b], (unsigned)m.chain_blocks[b], blockIdx.x - (unsigned)m.chain_first[b]);
}

// Persistent batch kernel: workgroups pop (stream, group) items until the list
// is exhausted; every item is one block of one stream for one group.
template <int FL>
__global__ void __launch_bounds__(512) batch_kernel(const BatchStream *streams, const int2 *items,
                                                    int nitems, int *counter, const int64_t *pos,
                                                    int block_len) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int item_s;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) item_s = atomicAdd(counter, 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(item_s);
        if (it >= nitems) break;
        const int2 item = items[it];
        const int sidx = __builtin_amdgcn_readfirstlane(item.x);
        const int g = __builtin_amdgcn_readfirstlane(item.y);
        const int64_t p0 = pos[sidx];
        const int64_t len = streams[sidx].len;
        if (p0 >= len) continue;
        FwdArgs a = streams[sidx].args;
        a.xbase = p0;
        a.n = min((int64_t)block_len, len - p0);
        a.ld = block_len;
        const SegCtx sc = whole_launch(a);
        fwd_group<FL, kModeKeys, true, false>(a, g, smem, sc);
    }
}

// Batch with each live stream's block cut into time segments (used while the
// live streams alone cannot fill the device). Items are (stream, group << 4 |
// segment), one workgroup each; items of ended streams or of segments past the
// block's end exit at once. Per-stream segment buffers hang off the stream's
// FwdArgs (seg_end, seg_start, seg_len).
__device__ __forceinline__ bool batch_item(const BatchStream *streams, const int2 *items, const int64_t *pos,
                                           int block_len, FwdArgs &a, int &g, int &seg) {
    const int2 item = items[blockIdx.x];
    const int sidx = __builtin_amdgcn_readfirstlane(item.x);
    g = __builtin_amdgcn_readfirstlane(item.y >> 4);
    seg = __builtin_amdgcn_readfirstlane(item.y & 15);
    const int64_t p0 = pos[sidx], len = streams[sidx].len;
    if (p0 >= len) return false;
    a = streams[sidx].args;
    a.xbase = p0;
    a.n = min((int64_t)block_len, len - p0);
    a.ld = block_len;
    a.gbase = 0;
    a.seg_slot0 = 0;
    a.seg_stride = a.nslots;
    return (int64_t)seg * a.seg_len < a.n;
}

template <int FL>
__global__ void __launch_bounds__(512) batch_pre_kernel(const BatchStream *streams, const int2 *items,
                                                        const int64_t *pos, int block_len) {
    extern __shared__ __align__(16) unsigned char smem[];
    FwdArgs a;
    int g, seg;
    if (!batch_item(streams, items, pos, block_len, a, g, seg)) return;
    if ((int64_t)(seg + 1) * a.seg_len >= a.n) return;   // the block's last segment needs no end state
    pre_item<FL, true>(a, (unsigned)(seg * a.groups + g), smem);
}

template <int FL>
__global__ void __launch_bounds__(512) batch_seg_kernel(const BatchStream *streams, const int2 *items,
                                                        const int64_t *pos, int block_len) {
    extern __shared__ __align__(16) unsigned char smem[];
    FwdArgs a;
    int g, seg;
    if (!batch_item(streams, items, pos, block_len, a, g, seg)) return;
    seg_item<FL, kModeKeys, true, false>(a, (unsigned)(seg * a.groups + g), smem);
}

// FP64 carry chain of every live stream (grid.y = stream): the same
// composition as seg_chain_kernel over the segments the block actually has.
__global__ void __launch_bounds__(256) batch_chain_kernel(const BatchStream *streams, const int64_t *pos,
                                                          int block_len) {
    const int sidx = blockIdx.y;
    const FwdArgs &a = streams[sidx].args;
    const int64_t sl = (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const int64_t p0 = pos[sidx], len = streams[sidx].len;
    if (p0 >= len || (int64_t)blockIdx.x * 64 >= a.nslots) return;
    const int64_t n = min((int64_t)block_len, len - p0);
    const int nv = (int)((n + a.seg_len - 1) / a.seg_len);
    const bool act = sl < a.nslots;   // whole waves: a bank's slot count is a multiple of 64
    float4 st = make_float4(0.f, 0.f, 0.f, 0.f);
    double2 av = make_double2(0.0, 0.0);
    if (act) {
        st = a.state[sl];
        av = chain_coeff(a, sl);
    }
    chain_segments(a.seg_end, a.seg_start, a.nslots, sl, act, st, av, nv, a.seg_len);
}

// Max over workgroup partial keys and the key rows of split templates: 16
// samples x 16 row slices per block. Blocks from key_blocks on write the
// history copy (hc.new_h set), 256 samples each.
__global__ void __launch_bounds__(256) finalize_keys_kernel(const uint64_t *keys, int groups, int64_t ld,
                                                            int64_t n, float *mx, int32_t *am, HistCopy hc,
                                                            unsigned key_blocks, SplitKeys sk) {
    if (blockIdx.x >= key_blocks) {   // uniform per block: no barrier below is reached
        const int i = (int)(blockIdx.x - key_blocks) * 256 + (int)threadIdx.x;
        if (i < hc.dmax) hist_copy_at(hc, i);
        return;
    }
    __shared__ uint64_t red[16][17];
    const int si = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int64_t i = (int64_t)blockIdx.x * 16 + si;
    uint64_t k = 0;
    if (i < n)
        for (int g = q; g < groups; g += 16) {
            const uint64_t v = keys[(int64_t)g * ld + i];
            k = v > k ? v : k;
        }
    if (i < n) {
#pragma unroll 4
        for (int r = q; r * kSplitSlice < sk.n_split; r += 16) {
            const uint64_t v = sk.rows[(int64_t)sk.split_off[r * kSplitSlice] * sk.ld + i];
            k = v > k ? v : k;
        }
    }
    red[q][si] = k;
    __syncthreads();
    if (q == 0 && i < n) {
        for (int r = 1; r < 16; ++r) k = red[r][si] > k ? red[r][si] : k;
        mx[i] = __uint_as_float((uint32_t)(k >> 32));
        am[i] = (int32_t)(0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull));
    }
}

// Templates split over workgroups: z_j = the sum of its parts' partial sums
// (in part order).
__device__ __forceinline__ float2 sum_parts(const float2 *zpart, int64_t ld_part, int q0, int q1, int64_t t) {
    float zr = 0.f, zi = 0.f;
#pragma unroll 4
    for (int q = q0; q < q1; ++q) {
        const float2 v = zpart[(int64_t)q * ld_part + t];
        zr += v.x;
        zi += v.y;
    }
    return make_float2(zr, zi);
}

// SNR or z rows of the split templates for samples [0, n) of a piece (grid.y over the
// templates: one block per template and 256 samples, since 64 blocks alone took
// 45 us for 256 templates of 16,384 samples).
__global__ void __launch_bounds__(256) combine_parts_kernel(const float2 *zpart, int64_t ld_part,
                                                            const int32_t *split_tpl, const int32_t *split_off,
                                                            int n_split, int64_t n, int mode, float *snr, float2 *z,
                                                            int64_t ld, int64_t obase) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    for (int i = blockIdx.y; i < n_split; i += gridDim.y) {
        const float2 v = sum_parts(zpart, ld_part, split_off[i], split_off[i + 1], t);
        const int64_t o = (int64_t)split_tpl[i] * ld + obase + t;
        if (mode == kModeSnr)
            snr[o] = v.x * v.x + v.y * v.y;
        else
            z[o] = v;
    }
}

// Per sample the largest key of each kSplitSlice split templates (grid.y over the slices),
// left in the place of the partial sums of the slice's first part: the same 8 bytes,
// read by the thread that writes them and by no other. A block takes 32 samples, a
// thread per template: bound by the latency of one template's offsets and sums.
// spiir_trigger_max of 64 / 4,096 samples of 1,400 banded templates (4 parts each): 1,407
// / 2,334 us with one grid row for all templates, 55 / 943 so (65 / 2,532
// without bands, the window in global memory); 200 templates, 64 samples: 205, 27 (23).
__global__ void __launch_bounds__(256) split_keys_kernel(float2 *zpart, int64_t ld_part, const int32_t *split_tpl,
                                                         const int32_t *split_off, int n_split, int64_t n) {
    constexpr int kCols = 256 / kSplitSlice;
    __shared__ uint64_t red[kSplitSlice][kCols + 1];
    const int c = threadIdx.x % kCols, r = threadIdx.x / kCols;
    const int64_t t = (int64_t)blockIdx.x * kCols + c;
    for (int i0 = blockIdx.y * kSplitSlice; i0 < n_split; i0 += gridDim.y * kSplitSlice) {
        const int i = i0 + r;
        uint64_t k = 0;
        if (i < n_split && t < n) {
            const float2 z = sum_parts(zpart, ld_part, split_off[i], split_off[i + 1], t);
            const float sn = z.x * z.x + z.y * z.y;
            k = ((uint64_t)__float_as_uint(sn) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)split_tpl[i]);
        }
        red[r][c] = k;
        __syncthreads();
        if (r == 0 && t < n) {
            for (int q = 1; q < kSplitSlice; ++q) k = red[q][c] > k ? red[q][c] : k;
            reinterpret_cast<uint64_t *>(zpart)[(int64_t)split_off[i0] * ld_part + t] = k;
        }
        __syncthreads();
    }
}

// a^L minus what the FP32 recursion multiplies a carried state by over a chunk.
__device__ __forceinline__ double2 chunk_drift(double2 a, float2 b, int L) {
    const RotCoeffs r = rot_coeffs(a, b);
    const double2 p = cpow64(a, L), q = rot_pow(r.a4, r.v, L);
    return make_double2(p.x - q.x, p.y - q.y);
}

__global__ void __launch_bounds__(256) chunk_drift_kernel(const double2 *a64, const float2 *b32, int64_t nslots,
                                                          int L, double2 *dL) {
    const int64_t sl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl < nslots) dL[sl] = chunk_drift(a64[sl], b32[sl], L);
}

// Slot arrays from caller-order FP64 coefficients on the device (fl32
// roundings, a^L and the chunk drift in FP64, the FP64-carry flag). Padding
// slots keep their zeros.
__global__ void __launch_bounds__(256) set_coeffs_kernel(const double2 *a, const double2 *b,
                                                         const int32_t *slot_filter, int64_t nslots, int L,
                                                         float2 *a32, float2 *b32, double2 *aL, double2 *dL,
                                                         double2 *a64, int32_t *flags) {
    const int64_t sl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= nslots) return;
    const int k = slot_filter[sl];
    if (k < 0) return;
    const double2 av = a[k], bv = b[k];
    const float2 af = make_float2((float)av.x, (float)av.y);
    a32[sl] = af;
    b32[sl] = make_float2((float)bv.x, (float)bv.y);
    aL[sl] = cpow64(av, L);
    dL[sl] = chunk_drift(av, b32[sl], L);
    a64[sl] = av;
    flags[sl] = hypot(av.x, av.y) > 1.0 - 1e-5 ? 1 : 0;
}

__global__ void rows_argmax_kernel(const float *snr, int T, int64_t ld, int64_t n, float *mx,
                                   int32_t *am) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float best = snr[i];
    int bj = 0;
    for (int j = 1; j < T; ++j) {
        const float v = snr[(int64_t)j * ld + i];
        if (v > best) {
            best = v;
            bj = j;
        }
    }
    mx[i] = best;
    am[i] = bj;
}

__global__ void hist_update_kernel(HistCopy hc) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < hc.dmax) hist_copy_at(hc, i);
}

// A block fills kMarkSamples samples and marks whether one of them is infinite.
__global__ void __launch_bounds__(kMarkSamples) window_fill_kernel(float *xwin, int32_t *mark, const float *hist,
                                                                   const float *x, int64_t n, int dmax) {
    __shared__ int inf;
    const int64_t i = (int64_t)blockIdx.x * kMarkSamples + threadIdx.x;
    float v = 0.f;
    if (i < n + dmax) {
        v = i < dmax ? (hist ? hist[i] : 0.f) : x[i - dmax];
        xwin[i] = v;
    }
    if (!mark) return;
    if (threadIdx.x == 0) inf = 0;
    __syncthreads();
    if (fabsf(v) > FLT_MAX) inf = 1;
    __syncthreads();
    if (threadIdx.x == 0) mark[blockIdx.x] = inf;
}

__global__ void fill_zero_kernel(uint32_t *p, int64_t words) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) p[i] = 0u;
}

__global__ void noise_fill_kernel(float *x, int64_t n, uint32_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // 64-bit mix (splitmix64 finaliser) of the index and seed -> uniform in [-1, 1)
    uint64_t z = (uint64_t)i + 0x9E3779B97F4A7C15ull * (uint64_t)(seed + 1);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    x[i] = (float)((int64_t)(z >> 40) - (1ll << 23)) * (1.0f / 8388608.0f);
}

// ---------------------------------------------------------------------------
// Adjoint. With lambda[m] = G[m] + conj(a) lambda[m+1] (lambda[n] = 0) the
// gradients of a real loss of z are
//     grad_b = sum_m lambda[m] x[m - d],
//     grad_a = sum_m lambda[m] conj(y[m - 1]).
// From a cold start y[m - 1] = sum_{k < m} a^(m-1-k) b x[k - d], so the second
// sum regroups exactly as
//     grad_a = conj(b) sum_k nu[k] x[k - d],
//     nu[k] = sum_{m > k} conj(a)^(m-1-k) lambda[m] = lambda[k+1] + conj(a) nu[k+1],
// a second reverse recursion driven by lambda. The backward therefore runs the
// pair (lambda, nu) from the end of the stream and never forms y: no forward
// recomputation and no stored filter states. Over s steps without input the
// pair moves by the Jordan block
//     lambda <- conj(a)^s lambda,   nu <- conj(a)^s nu + s conj(a)^(s-1) lambda.
// The pair recursion is linear, so the stream is cut into nseg segments of
// whole chunks: bwd_scan_kernel runs every segment but the first from a zero
// pair at its end (reading only G), and bwd_seg_kernel composes the segments
// after its own from the end in FP64 with the Jordan block, which gives the true
// pair entering its segment, and runs the segment from that pair with the
// gradient sums (FP32 within a chunk, FP64 across chunks). bwd_reduce_kernel
// adds the per-segment sums in FP64 in segment order and applies conj(b).
// Every L samples (a chunk) the pair carried into the chunk is corrected for
// the FP32 coefficient: lambda += conj(a^l - fl(a)^l) lambda_in,
// nu += conj(a^l - fl(a)^l) nu_in + l conj(a^(l-1) - fl(a)^(l-1)) lambda_in.
// ---------------------------------------------------------------------------


// v[t] = p[t] for t < ql, else 0; full runs use 16-byte loads (p is only
// 4-byte aligned, which global loads accept).
__device__ __forceinline__ void fetch_x(const float *p, int ql, float (&v)[kSub]) {
    if (ql == kSub) {
#pragma unroll
        for (int i = 0; i < kSub / 4; ++i) {
            const f4u q = *reinterpret_cast<const f4u *>(p + 4 * i);
            v[4 * i] = q.x;
            v[4 * i + 1] = q.y;
            v[4 * i + 2] = q.z;
            v[4 * i + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < kSub; ++t) v[t] = t < ql ? p[t] : 0.f;
    }
}

// G of one template for one sub-chunk when the address is the same for the
// whole wave: read through the constant address space, so the loads are
// scalar (one per wave, values in SGPRs) and never reach the texture path.
typedef const __attribute__((address_space(4))) float cfloat;

__device__ __forceinline__ void fetch_g_uniform(const float2 *p, int ql, float (&gr)[kSub], float (&gi)[kSub]) {
    cfloat *c = (cfloat *)p;
    if (ql == kSub) {
#pragma unroll
        for (int t = 0; t < kSub; ++t) {
            gr[t] = c[2 * t];
            gi[t] = c[2 * t + 1];
        }
    } else {
#pragma unroll
        for (int t = 0; t < kSub; ++t) {
            gr[t] = t < ql ? c[2 * t] : 0.f;
            gi[t] = t < ql ? c[2 * t + 1] : 0.f;
        }
    }
}

// A backward wave: the filters [k0, k1) of template tpl (at most 64, lane i
// takes filter k0 + i), so that G is the same for the whole wave.
struct BwdLane {
    int tpl;
    int64_t k0, k1, k;
};

__device__ __forceinline__ bool bwd_lane(const BwdArgs &p, BwdLane &bl) {
    const int w = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    if (w >= p.n_bwaves) return false;
    const int4 e = p.bwaves[w];
    bl.tpl = __builtin_amdgcn_readfirstlane(e.x);
    bl.k0 = (int64_t)(unsigned)__builtin_amdgcn_readfirstlane(e.y);
    bl.k1 = (int64_t)(unsigned)__builtin_amdgcn_readfirstlane(e.z);
    bl.k = bl.k0 + (threadIdx.x & 63);
    return bl.k < bl.k1;
}

// The carried-pair corrections of an l-step chunk (see above), FP32:
// d1 = conj(a^l - fl(a)^l), d2 = l conj(a^(l-1) - fl(a)^(l-1)).
struct PairDrift {
    float d1r, d1i, d2r, d2i;
};

__device__ __forceinline__ PairDrift pair_drift(const SlotArrays &s, int64_t slot, int l, float ar, float ai) {
    const double2 a = s.a64[slot];
    const double2 af = make_double2((double)ar, (double)ai);
    const double2 p1 = cpow64(a, l - 1), q1 = cpow64(af, l - 1);
    const double2 p = cmul64(p1, a), q = cmul64(q1, af);
    PairDrift d;
    d.d1r = (float)(p.x - q.x);
    d.d1i = (float)-(p.y - q.y);
    d.d2r = (float)((double)l * (p1.x - q1.x));
    d.d2i = (float)-((double)l * (p1.y - q1.y));
    return d;
}

// lambda += d1 lambda_in; nu += d1 nu_in + d2 lambda_in (complex products).
__device__ __forceinline__ void pair_correct(float &lr, float &li, float &vr, float &vi, const PairDrift &d,
                                             float l0r, float l0i, float v0r, float v0i) {
    lr = fmaf(d.d1r, l0r, fmaf(-d.d1i, l0i, lr));
    li = fmaf(d.d1r, l0i, fmaf(d.d1i, l0r, li));
    vr = fmaf(d.d1r, v0r, fmaf(-d.d1i, v0i, fmaf(d.d2r, l0r, fmaf(-d.d2i, l0i, vr))));
    vi = fmaf(d.d1r, v0i, fmaf(d.d1i, v0r, fmaf(d.d2r, l0i, fmaf(d.d2i, l0r, vi))));
}

// One sub-chunk of the pair recursion, last step first: on entry (l, v) =
// (lambda[m+1], nu[m+1]); each step forms nu[m] = lambda[m+1] + conj(a) nu[m+1]
// and lambda[m] = G[m] + conj(a) lambda[m+1] (FULL: all kSub steps).
template <int FL, bool FULL>
__device__ __forceinline__ void pair_steps(float (&lr)[FL], float (&li)[FL], float (&vr)[FL], float (&vi)[FL],
                                           const float (&ar)[FL], const float (&ai)[FL], const float (&gr)[kSub],
                                           const float (&gi)[kSub], int ql) {
#pragma unroll
    for (int t = kSub - 1; t >= 0; --t) {
        if (FULL || t < ql) {
#pragma unroll
            for (int f = 0; f < FL; ++f) {
                const float nvr = fmaf(ar[f], vr[f], fmaf(ai[f], vi[f], lr[f]));
                const float nvi = fmaf(ar[f], vi[f], fmaf(-ai[f], vr[f], li[f]));
                const float nlr = fmaf(ar[f], lr[f], fmaf(ai[f], li[f], gr[t]));
                const float nli = fmaf(ar[f], li[f], fmaf(-ai[f], lr[f], gi[t]));
                vr[f] = nvr;
                vi[f] = nvi;
                lr[f] = nlr;
                li[f] = nli;
            }
        }
    }
}

// The same steps with the gradient sums sb += lambda[m] x[m - d],
// sa += nu[m] x[m - d] for one filter.
template <bool FULL>
__device__ __forceinline__ void grad_steps(float &lr, float &li, float &vr, float &vi, float ar, float ai,
                                           const float (&xv)[kSub], const float (&gr)[kSub], const float (&gi)[kSub],
                                           float &sar, float &sai, float &sbr, float &sbi, int ql) {
#pragma unroll
    for (int t = kSub - 1; t >= 0; --t) {
        if (FULL || t < ql) {
            const float nvr = fmaf(ar, vr, fmaf(ai, vi, lr));
            const float nvi = fmaf(ar, vi, fmaf(-ai, vr, li));
            const float nlr = fmaf(ar, lr, fmaf(ai, li, gr[t]));
            const float nli = fmaf(ar, li, fmaf(-ai, lr, gi[t]));
            vr = nvr;
            vi = nvi;
            lr = nlr;
            li = nli;
            sbr = fmaf(lr, xv[t], sbr);
            sbi = fmaf(li, xv[t], sbi);
            sar = fmaf(vr, xv[t], sar);
            sai = fmaf(vi, xv[t], sai);
        }
    }
}

// Segment-local pair at the start of segment blockIdx.y + 1, from a zero pair
// at its end (reads only G, by scalar loads). One filter per lane, one
// template per wave; the G of the next sub-chunk is loaded while the current
// one is computed.
__global__ void __launch_bounds__(256) bwd_scan_kernel(BwdArgs p) {
    BwdLane bl;
    if (!bwd_lane(p, bl)) return;
    const int64_t slot = p.filter_slot[bl.k];
    const int tpl = bl.tpl;
    const int seg = blockIdx.y + 1;
    const int64_t n = p.n, nch = (n + p.L - 1) / p.L;
    const int64_t cs = (int64_t)seg * p.seg_chunks, ce = min(nch, cs + p.seg_chunks);
    const float2 *gz = p.gz + (int64_t)tpl * n;
    const float2 a = p.s.a32[slot];
    float ar[1] = {a.x}, ai[1] = {a.y};
    PairDrift dfull;
    if (p.prec != kPrecFp32) dfull = pair_drift(p.s, slot, p.L, ar[0], ai[0]);
    float lr[1] = {0.f}, li[1] = {0.f}, vr[1] = {0.f}, vi[1] = {0.f};
    float l0r = 0.f, l0i = 0.f, v0r = 0.f, v0i = 0.f;
    auto nq_of = [&](int64_t c) { return (int)((min((int64_t)p.L, n - c * p.L) + kSub - 1) / kSub); };
    auto fetch = [&](float (&gr)[kSub], float (&gi)[kSub], int64_t c, int q) {
        const int64_t m0 = c * p.L + (int64_t)q * kSub;
        const int ql = (int)min((int64_t)kSub, min((int64_t)p.L, n - c * p.L) - (int64_t)q * kSub);
        fetch_g_uniform(gz + m0, ql, gr, gi);
    };
    auto run = [&](const float (&gr)[kSub], const float (&gi)[kSub], int64_t c, int q) {
        const int l = (int)min((int64_t)p.L, n - c * p.L);
        const int ql = min(kSub, l - q * kSub);
        if (q == nq_of(c) - 1) {
            l0r = lr[0];
            l0i = li[0];
            v0r = vr[0];
            v0i = vi[0];
        }
        if (ql == kSub)
            pair_steps<1, true>(lr, li, vr, vi, ar, ai, gr, gi, ql);
        else
            pair_steps<1, false>(lr, li, vr, vi, ar, ai, gr, gi, ql);
        if (q == 0 && p.prec != kPrecFp32) {
            const PairDrift d = l == p.L ? dfull : pair_drift(p.s, slot, l, ar[0], ai[0]);
            pair_correct(lr[0], li[0], vr[0], vi[0], d, l0r, l0i, v0r, v0i);
        }
    };
    auto step_back = [&](int64_t &c, int &q) {
        if (q > 0) {
            --q;
        } else {
            --c;
            q = c >= cs ? nq_of(c) - 1 : 0;
        }
    };
    if (ce > cs) {
        float agr[kSub], agi[kSub], bgr[kSub], bgi[kSub];
        int64_t c = ce - 1;
        int q = nq_of(c) - 1;
        fetch(agr, agi, c, q);
        while (true) {
            int64_t cb = c;
            int qb = q;
            step_back(cb, qb);
            if (cb >= cs) fetch(bgr, bgi, cb, qb);
            run(agr, agi, c, q);
            if (cb < cs) break;
            c = cb;
            q = qb;
            int64_t ca = c;
            int qa = q;
            step_back(ca, qa);
            if (ca >= cs) fetch(agr, agi, ca, qa);
            run(bgr, bgi, c, q);
            if (ca < cs) break;
            c = ca;
            q = qa;
        }
    }
    p.pair_loc[(int64_t)seg * p.nslots + slot] = make_float4(lr[0], li[0], vr[0], vi[0]);
}

// True pair entering segment seg from the right: the later segments' local
// pairs composed from the last one on, pair <- pair_loc[s] + J^len pair with J
// the Jordan block of conj(a), in FP64 (with fl32(a) in the all-FP32 mode). Every
// segment composes its own, with the loads of 8 segments in flight, instead of
// a launch that wrote them all with a load and two powers of a per segment one
// after the other: 32 templates of 100 filters over 4,001 samples (16 segments)
// took 11.6 us there.
__device__ __forceinline__ float4 pair_entering(const BwdArgs &p, int64_t slot, int seg) {
    float4 in = make_float4(0.f, 0.f, 0.f, 0.f);   // of the last segment
    if (seg >= p.nseg - 1) return in;
    double2 a = p.s.a64[slot];
    if (p.prec == kPrecFp32) {
        const float2 a32 = p.s.a32[slot];
        a = make_double2((double)a32.x, (double)a32.y);
    }
    const int len = p.seg_chunks * p.L;   // of every segment but the last, which enters with a zero pair
    const double2 a1 = cpow64(a, len - 1), al = cmul64(a1, a);   // conj(a)^k = conj(a^k)
    const double sr = (double)len * a1.x, si = (double)len * a1.y;
    double lr = 0.0, li = 0.0, vr = 0.0, vi = 0.0;
    constexpr int kAhead = 8;
    for (int top = p.nseg - 1; top > seg; top -= kAhead) {
        float4 loc[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (top - u > seg) loc[u] = p.pair_loc[(int64_t)(top - u) * p.nslots + slot];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (top - u > seg) {
                const double nvr = (double)loc[u].z + (al.x * vr + al.y * vi) + (sr * lr + si * li);
                const double nvi = (double)loc[u].w + (al.x * vi - al.y * vr) + (sr * li - si * lr);
                const double nlr = (double)loc[u].x + al.x * lr + al.y * li;
                const double nli = (double)loc[u].y + al.x * li - al.y * lr;
                lr = nlr;
                li = nli;
                vr = nvr;
                vi = nvi;
            }
    }
    return make_float4((float)lr, (float)li, (float)vr, (float)vi);
}

// Strain and G of one sub-chunk of the backward.
struct SubBuf {
    float x[kSub], gr[kSub], gi[kSub];
};

// Full backward of segment blockIdx.y from its true incoming pair. One filter
// per lane; every wave holds filters of one template (G read by scalar loads).
// Sub-chunks are taken in reverse order through two register buffers: the
// next one is loaded while the current one is computed.
__global__ void __launch_bounds__(256) bwd_seg_kernel(BwdArgs p) {
    BwdLane bl;
    if (!bwd_lane(p, bl)) return;
    const int64_t slot = p.filter_slot[bl.k];
    const int tpl = bl.tpl;
    const int seg = blockIdx.y;
    const int64_t n = p.n, nch = (n + p.L - 1) / p.L;
    const int64_t cs = (int64_t)seg * p.seg_chunks, ce = min(nch, cs + p.seg_chunks);
    const float2 *gz = p.gz + (int64_t)tpl * n;
    const float2 a = p.s.a32[slot];
    const float ar = a.x, ai = a.y;
    const float *xw = p.xwin + p.s.xoff[slot];  // xw[m] = x[m - d]
    PairDrift dfull;
    if (p.prec != kPrecFp32) dfull = pair_drift(p.s, slot, p.L, ar, ai);
    double gar = 0.0, gai = 0.0, gbr = 0.0, gbi = 0.0;
    const float4 pin = pair_entering(p, slot, seg);
    float lr = pin.x, li = pin.y, vr = pin.z, vi = pin.w;   // the pair after the current chunk
    float l0r = 0.f, l0i = 0.f, v0r = 0.f, v0i = 0.f;       // the pair entering the current chunk
    float sar = 0.f, sai = 0.f, sbr = 0.f, sbi = 0.f;
    auto nq_of = [&](int64_t c) { return (int)((min((int64_t)p.L, n - c * p.L) + kSub - 1) / kSub); };
    auto fetch = [&](SubBuf &b, int64_t c, int q) {
        const int64_t m0 = c * p.L + (int64_t)q * kSub;
        const int ql = (int)min((int64_t)kSub, min((int64_t)p.L, n - c * p.L) - (int64_t)q * kSub);
        fetch_x(xw + m0, ql, b.x);
        fetch_g_uniform(gz + m0, ql, b.gr, b.gi);
    };
    // one sub-chunk: chunk bookkeeping at its first (q = last) and last (q = 0) sub-chunk
    auto run = [&](const SubBuf &b, int64_t c, int q) {
        const int l = (int)min((int64_t)p.L, n - c * p.L);
        const int ql = min(kSub, l - q * kSub);
        if (q == nq_of(c) - 1) {
            l0r = lr;
            l0i = li;
            v0r = vr;
            v0i = vi;
            sar = sai = sbr = sbi = 0.f;
        }
        if (ql == kSub)
            grad_steps<true>(lr, li, vr, vi, ar, ai, b.x, b.gr, b.gi, sar, sai, sbr, sbi, ql);
        else
            grad_steps<false>(lr, li, vr, vi, ar, ai, b.x, b.gr, b.gi, sar, sai, sbr, sbi, ql);
        if (q == 0) {
            if (p.prec != kPrecFp32) {
                const PairDrift d = l == p.L ? dfull : pair_drift(p.s, slot, l, ar, ai);
                pair_correct(lr, li, vr, vi, d, l0r, l0i, v0r, v0i);
            }
            gar += (double)sar;
            gai += (double)sai;
            gbr += (double)sbr;
            gbi += (double)sbi;
        }
    };
    // reverse enumeration of the segment's sub-chunks
    auto step_back = [&](int64_t &c, int &q) {
        if (q > 0) {
            --q;
        } else {
            --c;
            q = c >= cs ? nq_of(c) - 1 : 0;
        }
    };
    if (ce > cs) {
        SubBuf A, B;
        int64_t c = ce - 1;
        int q = nq_of(c) - 1;
        fetch(A, c, q);
        while (true) {
            int64_t cb = c;
            int qb = q;
            step_back(cb, qb);
            if (cb >= cs) fetch(B, cb, qb);
            run(A, c, q);
            if (cb < cs) break;
            c = cb;
            q = qb;
            int64_t ca = c;
            int qa = q;
            step_back(ca, qa);
            if (ca >= cs) fetch(A, ca, qa);
            run(B, c, q);
            if (ca < cs) break;
            c = ca;
            q = qa;
        }
    }
    p.gpart[((int64_t)seg * 2 + 0) * p.nslots + slot] = make_double2(gar, gai);
    p.gpart[((int64_t)seg * 2 + 1) * p.nslots + slot] = make_double2(gbr, gbi);
}

// Sum over segments in FP64, then grad_a = conj(fl32(b)) * sum nu x.
__global__ void __launch_bounds__(256) bwd_reduce_kernel(BwdArgs p) {
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= p.nslots) return;
    const int k = p.slot_filter[slot];
    if (k < 0) return;
    double gar = 0.0, gai = 0.0, gbr = 0.0, gbi = 0.0;
#pragma unroll 4
    for (int seg = 0; seg < p.nseg; ++seg) {
        const double2 ga = p.gpart[((int64_t)seg * 2 + 0) * p.nslots + slot];
        const double2 gb = p.gpart[((int64_t)seg * 2 + 1) * p.nslots + slot];
        gar += ga.x;
        gai += ga.y;
        gbr += gb.x;
        gbi += gb.y;
    }
    const float2 b = p.s.b32[slot];
    const double br = (double)b.x, bi = (double)b.y;
    p.grad_a[k] = make_float2((float)(br * gar + bi * gai), (float)(br * gai - bi * gar));
    p.grad_b[k] = make_float2((float)gbr, (float)gbi);
}

// Batch bookkeeping.
__global__ void __launch_bounds__(256) batch_finalize_kernel(const BatchStream *streams, const uint64_t *keys,
                                                             int64_t key_stride, const int64_t *pos,
                                                             int block_len) {
    __shared__ uint64_t red[16][17];
    const int sidx = blockIdx.y;
    const int si = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int64_t i = (int64_t)blockIdx.x * 16 + si;
    const int64_t p0 = pos[sidx];
    const int64_t len = streams[sidx].len;
    const bool live = p0 < len && i < min((int64_t)block_len, len - p0);
    const uint64_t *kk = keys + sidx * key_stride;
    const int groups = streams[sidx].groups;
    uint64_t k = 0;
    if (live)
        for (int g = q; g < groups; g += 16) {
            const uint64_t v = kk[(int64_t)g * block_len + i];
            k = v > k ? v : k;
        }
    red[q][si] = k;
    __syncthreads();
    if (q == 0 && live) {
        for (int r = 1; r < 16; ++r) k = red[r][si] > k ? red[r][si] : k;
        streams[sidx].max_out[p0 + i] = __uint_as_float((uint32_t)(k >> 32));
        streams[sidx].arg_out[p0 + i] = (int32_t)(0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull));
    }
}

__global__ void batch_advance_kernel(int64_t *pos, const BatchStream *streams, int nstreams,
                                     int *counter, int block_len) {
    const int i = threadIdx.x;
    if (i == 0) *counter = 0;
    if (i < nstreams) {
        const int64_t len = streams[i].len;
        pos[i] = min(len, pos[i] + (int64_t)block_len);
    }
}

template <int FL, int MODE, bool XLDS>
hipError_t launch_fwd_t(const FwdArgs &a, int groups, size_t lds, hipStream_t st, KernelEvents ev) {
    if (a.zpart)
        hipExtLaunchKernelGGL((fwd_kernel<FL, MODE, XLDS, true>), dim3(groups), dim3(a.wpg * 64), (uint32_t)lds,
                              st, ev.start, ev.stop, 0u, a);
    else
        hipExtLaunchKernelGGL((fwd_kernel<FL, MODE, XLDS, false>), dim3(groups), dim3(a.wpg * 64), (uint32_t)lds,
                              st, ev.start, ev.stop, 0u, a);
    return hipGetLastError();
}

template <int MODE, bool XLDS>
hipError_t launch_fwd_m(const FwdArgs &a, int fl, int groups, size_t lds, hipStream_t st, KernelEvents ev) {
    switch (fl) {
        case 1: return launch_fwd_t<1, MODE, XLDS>(a, groups, lds, st, ev);
        case 2: return launch_fwd_t<2, MODE, XLDS>(a, groups, lds, st, ev);
        case 3: return launch_fwd_t<3, MODE, XLDS>(a, groups, lds, st, ev);
        case 4: return launch_fwd_t<4, MODE, XLDS>(a, groups, lds, st, ev);
        default: return hipErrorInvalidValue;
    }
}

template <bool XLDS>
hipError_t launch_fwd_x(const FwdArgs &a, int mode, int fl, int groups, size_t lds, hipStream_t st,
                        KernelEvents ev) {
    switch (mode) {
        case kModeSnr: return launch_fwd_m<kModeSnr, XLDS>(a, fl, groups, lds, st, ev);
        case kModeKeys: return launch_fwd_m<kModeKeys, XLDS>(a, fl, groups, lds, st, ev);
        case kModeZ: return launch_fwd_m<kModeZ, XLDS>(a, fl, groups, lds, st, ev);
        default: return hipErrorInvalidValue;
    }
}

template <int FL, int MODE, bool XLDS>
hipError_t launch_split_t(const FwdArgs &a, int nseg, size_t lds, size_t lds_pre, hipStream_t st, KernelEvents ev) {
    hipExtLaunchKernelGGL((fwd_pre_kernel<FL, XLDS>), dim3(a.groups * (nseg - 1)), dim3(a.wpg * 64),
                          (uint32_t)lds_pre, st, ev.start, (hipEvent_t) nullptr, 0u, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!a.chain_inline) {
        const unsigned nb = (unsigned)((a.seg_stride + 63) / 64);
        const unsigned hb = a.hist_next.dmax > 0 ? (unsigned)((a.hist_next.dmax + 255) / 256) : 0u;
        hipLaunchKernelGGL(seg_chain_kernel, dim3(nb + hb), dim3(256), 0, st, a, FL, nseg, nb);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.zpart)
        hipExtLaunchKernelGGL((fwd_seg_kernel<FL, MODE, XLDS, true>), dim3(a.groups * nseg), dim3(a.wpg * 64),
                              (uint32_t)lds, st, (hipEvent_t) nullptr, ev.stop, 0u, a);
    else
        hipExtLaunchKernelGGL((fwd_seg_kernel<FL, MODE, XLDS, false>), dim3(a.groups * nseg), dim3(a.wpg * 64),
                              (uint32_t)lds, st, (hipEvent_t) nullptr, ev.stop, 0u, a);
    return hipGetLastError();
}

template <int MODE, bool XLDS>
hipError_t launch_split_m(const FwdArgs &a, int fl, int nseg, size_t lds, size_t ldp, hipStream_t st,
                          KernelEvents ev) {
    switch (fl) {
        case 1: return launch_split_t<1, MODE, XLDS>(a, nseg, lds, ldp, st, ev);
        case 2: return launch_split_t<2, MODE, XLDS>(a, nseg, lds, ldp, st, ev);
        case 3: return launch_split_t<3, MODE, XLDS>(a, nseg, lds, ldp, st, ev);
        case 4: return launch_split_t<4, MODE, XLDS>(a, nseg, lds, ldp, st, ev);
        default: return hipErrorInvalidValue;
    }
}

template <bool XLDS>
hipError_t launch_split_x(const FwdArgs &a, int mode, int fl, int nseg, size_t lds, size_t ldp, hipStream_t st,
                          KernelEvents ev) {
    if (mode == kModeSnr) return launch_split_m<kModeSnr, XLDS>(a, fl, nseg, lds, ldp, st, ev);
    if (mode == kModeKeys) return launch_split_m<kModeKeys, XLDS>(a, fl, nseg, lds, ldp, st, ev);
    if (mode == kModeZ) return launch_split_m<kModeZ, XLDS>(a, fl, nseg, lds, ldp, st, ev);
    return hipErrorInvalidValue;
}

template <int FL>
int occ_t(int wpg, size_t lds) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fwd_kernel<FL, kModeKeys, true, false>, wpg * 64, lds) !=
        hipSuccess)
        return 0;
    return nb;
}

inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_forward(const FwdArgs &a, int mode, int fl, bool x_in_lds, int groups, size_t lds, hipStream_t st,
                          KernelEvents ev) {
    if (groups <= 0) return hipSuccess;
    return x_in_lds ? launch_fwd_x<true>(a, mode, fl, groups, lds, st, ev)
                    : launch_fwd_x<false>(a, mode, fl, groups, lds, st, ev);
}

// The state pass needs the strain window only (so more workgroups share a compute unit).
size_t state_pass_lds(const FwdArgs &a, bool x_in_lds) { return x_in_lds ? window_bytes(a.band_w, a.nb) : 0; }

hipError_t launch_forward_split(const FwdArgs &args, int mode, int fl, bool x_in_lds, int nseg, size_t lds,
                                hipStream_t st, KernelEvents ev) {
    if (args.groups <= 0 || nseg < 2) return hipErrorInvalidValue;
    FwdArgs a = args;
    a.chain_inline = nseg <= kChainInline ? 1 : 0;
    const size_t lds_pre = state_pass_lds(a, x_in_lds);
    return x_in_lds ? launch_split_x<true>(a, mode, fl, nseg, lds, lds_pre, st, ev)
                    : launch_split_x<false>(a, mode, fl, nseg, lds, lds_pre, st, ev);
}

namespace {

template <int FL>
hipError_t launch_multi_t(const MultiFwd &args, int wpg, size_t lds, size_t lds_pre, hipStream_t st) {
    const int n = args.count;
    MultiFwd m = args;
    bool chain = false;
    for (int b = 0; b < n; ++b) {
        m.a[b].chain_inline = m.nseg[b] <= kChainInline ? 1 : 0;
        chain = chain || !m.a[b].chain_inline;
    }
    for (int b = 0; b < n && chain; ++b) m.a[b].chain_inline = 0;   // one bank too many: the launch serves all
    hipError_t e = hipSuccess;
    if (m.pre_first[n] > 0) {
        hipLaunchKernelGGL((fwd_pre_multi_kernel<FL>), dim3((unsigned)m.pre_first[n]), dim3(wpg * 64), lds_pre, st, m);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (chain) {
        hipLaunchKernelGGL(seg_chain_multi_kernel, dim3((unsigned)m.chain_first[n]), dim3(256), 0, st, m, FL);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((fwd_seg_multi_kernel<FL, kModeZ>), dim3((unsigned)m.seg_first[n]), dim3(wpg * 64), lds,
                       st, m);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_forward_split_multi(const MultiFwd &m, int fl, int wpg, size_t lds, hipStream_t st) {
    if (m.count < 1 || m.count > kMultiMax) return hipErrorInvalidValue;
    size_t lds_pre = 0;
    for (int b = 0; b < m.count; ++b) {
        const size_t l = state_pass_lds(m.a[b], true);
        lds_pre = l > lds_pre ? l : lds_pre;
    }
    switch (fl) {
        case 1: return launch_multi_t<1>(m, wpg, lds, lds_pre, st);
        case 2: return launch_multi_t<2>(m, wpg, lds, lds_pre, st);
        case 3: return launch_multi_t<3>(m, wpg, lds, lds_pre, st);
        case 4: return launch_multi_t<4>(m, wpg, lds, lds_pre, st);
        default: return hipErrorInvalidValue;
    }
}

int forward_occupancy(int fl, int wpg, size_t lds) {
    switch (fl) {
        case 1: return occ_t<1>(wpg, lds);
        case 2: return occ_t<2>(wpg, lds);
        case 3: return occ_t<3>(wpg, lds);
        case 4: return occ_t<4>(wpg, lds);
        default: return 0;
    }
}

namespace {

template <int FL>
int pre_occ_t(int wpg, size_t lds, bool x_in_lds) {
    int nb = 0;
    const hipError_t e = x_in_lds ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fwd_pre_kernel<FL, true>, wpg * 64, lds)
                                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fwd_pre_kernel<FL, false>, wpg * 64, lds);
    return e == hipSuccess ? nb : 0;
}

}  // namespace

int state_occupancy(int fl, int wpg, const FwdArgs &a, bool x_in_lds) {
    const size_t lds = state_pass_lds(a, x_in_lds);
    switch (fl) {
        case 1: return pre_occ_t<1>(wpg, lds, x_in_lds);
        case 2: return pre_occ_t<2>(wpg, lds, x_in_lds);
        case 3: return pre_occ_t<3>(wpg, lds, x_in_lds);
        case 4: return pre_occ_t<4>(wpg, lds, x_in_lds);
        default: return 0;
    }
}

hipError_t launch_finalize_keys(const uint64_t *keys, int groups, int64_t ld, int64_t n,
                                float *mx, int32_t *am, hipStream_t st, const HistCopy *hc, const SplitKeys &sk) {
    HistCopy h{nullptr, nullptr, nullptr, 0, 0};
    if (hc && hc->dmax > 0) h = *hc;
    const unsigned kb = n > 0 ? nblocks(n, 16) : 0u;
    const unsigned hb = h.dmax > 0 ? nblocks(h.dmax, 256) : 0u;
    if (kb + hb == 0) return hipSuccess;
    hipLaunchKernelGGL(finalize_keys_kernel, dim3(kb + hb), dim3(256), 0, st, keys, groups, ld, n, mx, am, h,
                       kb, sk);
    return hipGetLastError();
}

hipError_t launch_combine_parts(float2 *zpart, int64_t ld_part, const int32_t *split_tpl,
                                const int32_t *split_off, int n_split, int64_t n, int mode, float *snr, float2 *z,
                                int64_t ld, int64_t obase, hipStream_t st) {
    if (n <= 0 || n_split <= 0) return hipSuccess;
    const int rows = mode == kModeKeys ? (n_split + kSplitSlice - 1) / kSplitSlice : n_split;
    const unsigned gy = (unsigned)std::min(rows, 65535);
    if (mode == kModeKeys)
        hipLaunchKernelGGL(split_keys_kernel, dim3(nblocks(n, 256 / kSplitSlice), gy), dim3(256), 0, st, zpart, ld_part,
                           split_tpl, split_off, n_split, n);
    else
        hipLaunchKernelGGL(combine_parts_kernel, dim3(nblocks(n, 256), gy), dim3(256), 0, st, zpart, ld_part, split_tpl,
                           split_off, n_split, n, mode, snr, z, ld, obase);
    return hipGetLastError();
}

hipError_t launch_set_coeffs(const double *a, const double *b, const int32_t *slot_filter, int64_t nslots, int L,
                             float2 *a32, float2 *b32, double2 *aL, double2 *dL, double2 *a64, int32_t *flags,
                             hipStream_t st) {
    if (nslots <= 0) return hipSuccess;
    hipLaunchKernelGGL(set_coeffs_kernel, dim3(nblocks(nslots, 256)), dim3(256), 0, st,
                       reinterpret_cast<const double2 *>(a), reinterpret_cast<const double2 *>(b), slot_filter,
                       nslots, L, a32, b32, aL, dL, a64, flags);
    return hipGetLastError();
}

hipError_t launch_chunk_drift(const double2 *a64, const float2 *b32, int64_t nslots, int L, double2 *dL,
                              hipStream_t st) {
    if (nslots <= 0) return hipSuccess;
    hipLaunchKernelGGL(chunk_drift_kernel, dim3(nblocks(nslots, 256)), dim3(256), 0, st, a64, b32, nslots, L, dL);
    return hipGetLastError();
}

hipError_t launch_rows_argmax(const float *snr, int T, int64_t ld, int64_t n, float *mx,
                              int32_t *am, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(rows_argmax_kernel, dim3(nblocks(n, 256)), dim3(256), 0, st, snr, T, ld, n,
                       mx, am);
    return hipGetLastError();
}

hipError_t launch_hist_update(const float *old_h, float *new_h, const float *x, int64_t n,
                              int dmax, hipStream_t st) {
    if (dmax <= 0) return hipSuccess;
    const HistCopy hc{old_h, new_h, x, n, dmax};
    hipLaunchKernelGGL(hist_update_kernel, dim3(nblocks(dmax, 256)), dim3(256), 0, st, hc);
    return hipGetLastError();
}

hipError_t launch_window_fill(float *xwin, int32_t *mark, const float *hist, const float *x, int64_t n, int dmax,
                              hipStream_t st) {
    if (n + dmax <= 0) return hipSuccess;
    hipLaunchKernelGGL(window_fill_kernel, dim3(nblocks(n + dmax, kMarkSamples)), dim3(kMarkSamples), 0, st, xwin, mark,
                       hist, x, n, dmax);
    return hipGetLastError();
}

template <int FL>
int bocc_t(int wpg, size_t lds) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_kernel<FL>, wpg * 64, lds) != hipSuccess)
        return 0;
    return nb;
}

int batch_occupancy(int fl, int wpg, size_t lds) {
    switch (fl) {
        case 1: return bocc_t<1>(wpg, lds);
        case 2: return bocc_t<2>(wpg, lds);
        case 3: return bocc_t<3>(wpg, lds);
        case 4: return bocc_t<4>(wpg, lds);
        default: return 0;
    }
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t st) {
    const int64_t words = (int64_t)(bytes / 4);
    if (words <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(nblocks(words, 256)), dim3(256), 0, st,
                       static_cast<uint32_t *>(p), words);
    return hipGetLastError();
}

hipError_t launch_noise_fill(float *x, int64_t n, uint32_t seed, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(noise_fill_kernel, dim3(nblocks(n, 256)), dim3(256), 0, st, x, n, seed);
    return hipGetLastError();
}

hipError_t launch_backward_t(const BwdArgs &a, hipStream_t st) {
    if (a.nseg > 1) {
        hipLaunchKernelGGL(bwd_scan_kernel, dim3(nblocks(a.n_bwaves, 4), a.nseg - 1), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(bwd_seg_kernel, dim3(nblocks(a.n_bwaves, 4), a.nseg), dim3(256), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bwd_reduce_kernel, dim3(nblocks(a.nslots, 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_backward(const BwdArgs &a, hipStream_t st) {
    if (a.n_bwaves <= 0) return hipSuccess;
    if (a.nseg < 1 || a.nseg > 65535 || a.seg_chunks < 1) return hipErrorInvalidValue;
    return launch_backward_t(a, st);
}

template <int FL>
hipError_t launch_batch_t(const BatchStream *streams, const int2 *items, int nitems, int *counter,
                          const int64_t *pos, int block_len, int grid, int wpg, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL((batch_kernel<FL>), dim3(grid), dim3(wpg * 64), lds, st, streams, items, nitems,
                       counter, pos, block_len);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchStream *streams, const int2 *items, int nitems, int *counter,
                        const int64_t *pos, int block_len, int fl, int grid, int wpg, size_t lds,
                        hipStream_t st) {
    switch (fl) {
        case 1: return launch_batch_t<1>(streams, items, nitems, counter, pos, block_len, grid, wpg, lds, st);
        case 2: return launch_batch_t<2>(streams, items, nitems, counter, pos, block_len, grid, wpg, lds, st);
        case 3: return launch_batch_t<3>(streams, items, nitems, counter, pos, block_len, grid, wpg, lds, st);
        case 4: return launch_batch_t<4>(streams, items, nitems, counter, pos, block_len, grid, wpg, lds, st);
        default: return hipErrorInvalidValue;
    }
}

template <int FL>
hipError_t launch_batch_split_t(const BatchStream *streams, const int2 *pre_items, int n_pre_items,
                                const int2 *seg_items, int n_seg_items, const int64_t *pos, int block_len,
                                int nstreams, int64_t max_slots, int wpg, size_t lds, hipStream_t st) {
    hipError_t e = hipSuccess;
    if (n_pre_items > 0) {
        hipLaunchKernelGGL((batch_pre_kernel<FL>), dim3(n_pre_items), dim3(wpg * 64), lds, st, streams, pre_items,
                           pos, block_len);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(batch_chain_kernel, dim3(nblocks(max_slots, 64), nstreams), dim3(256), 0, st, streams, pos,
                       block_len);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((batch_seg_kernel<FL>), dim3(n_seg_items), dim3(wpg * 64), lds, st, streams, seg_items,
                       pos, block_len);
    return hipGetLastError();
}

hipError_t launch_batch_split(const BatchStream *streams, const int2 *pre_items, int n_pre_items,
                              const int2 *seg_items, int n_seg_items, const int64_t *pos, int block_len,
                              int nstreams, int64_t max_slots, int fl, int wpg, size_t lds,
                              hipStream_t st) {
#define SPIIR_SPLIT_ARGS streams, pre_items, n_pre_items, seg_items, n_seg_items, pos, block_len, nstreams, \
                         max_slots, wpg, lds, st
    switch (fl) {
        case 1: return launch_batch_split_t<1>(SPIIR_SPLIT_ARGS);
        case 2: return launch_batch_split_t<2>(SPIIR_SPLIT_ARGS);
        case 3: return launch_batch_split_t<3>(SPIIR_SPLIT_ARGS);
        case 4: return launch_batch_split_t<4>(SPIIR_SPLIT_ARGS);
        default: return hipErrorInvalidValue;
    }
#undef SPIIR_SPLIT_ARGS
}

hipError_t launch_batch_finalize(const BatchStream *streams, int nstreams, const uint64_t *keys,
                                 int64_t key_stride, const int64_t *pos, int block_len,
                                 int max_groups, hipStream_t st) {
    (void)max_groups;
    hipLaunchKernelGGL(batch_finalize_kernel, dim3(nblocks(block_len, 16), nstreams), dim3(256), 0,
                       st, streams, keys, key_stride, pos, block_len);
    return hipGetLastError();
}

hipError_t launch_batch_advance(int64_t *pos, const BatchStream *streams, int nstreams,
                                int *counter, int block_len, hipStream_t st) {
    hipLaunchKernelGGL(batch_advance_kernel, dim3(1), dim3(((nstreams + 63) / 64) * 64), 0, st, pos,
                       streams, nstreams, counter, block_len);
    return hipGetLastError();
}

int forward_max_threads() { return kMaxWaves * 64; }

}  // namespace spiir
