// Register-resident line scans for planes with H, W <= 64, read from memory
// step by step: the forwards of small_fwd_preferred (few planes, blocked planes,
// one channel a group), the backward of planes of a few pixels, and callers whose
// workspace holds neither scan_plane.hip's partial sums nor a round of
// scan_line.hip.
//
// One lane owns one position of a line (the perpendicular axis); a line of P
// positions occupies T lanes (T = 16, 32 or 64, T >= P) and a wave holds
// 64 / T lines, i.e. 64 / T channels.  The hidden state h stays in a VGPR for
// the whole scan; the tridiagonal step reads the two neighbours of the
// previous line with DPP lane shifts (Sec. 3, Eq. (gspn_recurrence)).
//
// Forward: a workgroup is 4 waves, one per scan direction, over the same
// 64 / T channels.  Each wave keeps its direction's contributions u_d * h_d in
// registers and the four are summed in direction-bit order through an fp32
// LDS plane, so y is stored once, in the storage type.
//
// Backward: a workgroup is up to 8 waves over `cw` channels of one weight
// group.  Every wave runs the directions one after another: a forward sweep
// that keeps the line states h_0..h_{L-1} in registers, then the reverse
// adjoint sweep.  dx accumulates in an fp32 LDS plane per channel; the weight
// gradient of each step is reduced over the workgroup's channels through LDS
// (all waves step in lock-step, one barrier per step) and written either as
// the final dw or, when a group spans several workgroups, as an fp32 partial
// that a second kernel sums in fixed order.
#include <algorithm>

#include "device.hpp"
#include "launch.hpp"

namespace gspn {

namespace {

template <int T, typename S>
__global__ __launch_bounds__(256) void fwd_small_kernel(
    const S *__restrict__ x, const S *__restrict__ w, const S *__restrict__ lam,
    const S *__restrict__ u, S *__restrict__ y, int mask, int B, int C, int G, int H, int W,
    int pm)
{
    constexpr int NL = 64 / T;        // lines (channels) per wave
    constexpr int PITCH = T + 1;      // odd LDS row pitch: column walks are conflict-free
    __shared__ float acc[NL * T * PITCH];

    const int d = threadIdx.x >> 6;   // this wave's direction index
    const int lane = threadIdx.x & 63;
    const int line = lane / T;
    const int j = lane % T;
    const int nblk = (C + NL - 1) / NL;
    const int b = blockIdx.x / nblk;
    const int c0 = (blockIdx.x % nblk) * NL;
    const int c = c0 + line;
    const bool cvalid = c < C;
    const int cc = cvalid ? c : C - 1;
    const int g = cc / (C / G);
    const int bit = 1 << d;
    const bool mine = (mask & bit) != 0;
    const int HW = H * W;
    const int P = line_len(d, H, W);
    const bool active = cvalid && j < P;
    const int jc = active ? j : 0;

    float yr[T];
    if (mine) {
        const Frame f = make_frame(d, jc, H, W, W, pm != 0);
        const int s = dir_slot(mask, bit);
        const S *xp = x + ((int64_t)b * C + cc) * HW;
        const int64_t pd = (((int64_t)s * B + b) * C + cc) * HW;
        const S *lp = lam + pd;
        const S *up = u + pd;
        const S *wp = w + (((int64_t)s * B + b) * G + g) * 3 * HW;
        const bool m0 = active && j > 0;
        const bool m2 = active && j + 1 < P;
        float h = 0.f;
        // Steps past the line's end (T > L) repeat its last step's reads and
        // leave results that the merge never reads: no branch per step, so
        // the compiler can issue the loads of later steps early.
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int ic = i < f.L ? i : f.L - 1;
            const int e = f.e0 + ic * f.es;      // pixel (x)
            const int q = f.lm(ic);              // per-direction planes (lam, u, w)
            float inj = load_f(lp + q) * load_f(xp + e);
            inj = active ? inj : 0.f;
            float hn = inj;
            if (i > 0) {
                float w0 = load_f(wp + q);
                float w1 = load_f(wp + HW + q);
                float w2 = load_f(wp + 2 * HW + q);
                w0 = m0 ? w0 : 0.f;
                w1 = active ? w1 : 0.f;
                w2 = m2 ? w2 : 0.f;
                const float hl = from_left<T>(h);
                const float hr = from_right<T>(h);
                hn = fmaf(w1, h, hn);
                hn = fmaf(w0, hl, hn);
                hn = fmaf(w2, hr, hn);
            }
            h = hn;
            yr[i] = load_f(up + q) * h;
        }
    }

    // Merge the directions in bit order: the first one present stores, the
    // others add.  One direction per phase, so every sum has a fixed order.
    float *a = acc + line * T * PITCH;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (d == p && mine && active) {
            const Frame fl = make_frame(d, jc, H, W, PITCH);
            const bool first = (mask & ((1 << p) - 1)) == 0;
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if (i < fl.L) {
                    const int e = fl.e0 + i * fl.es;
                    a[e] = first ? yr[i] : a[e] + yr[i];
                }
            }
        }
        __syncthreads();
    }

    const int nch = min(NL, C - c0);
    S *yb = y + ((int64_t)b * C + c0) * HW;
    for (int t = threadIdx.x; t < nch * HW; t += blockDim.x) {
        const int l = t / HW;
        const int rc = t - l * HW;
        const int r = rc / W;
        const int col = rc - r * W;
        store_f(yb + t, acc[(l * T + r) * PITCH + col]);
    }
}

template <int T, typename S>
__global__ __launch_bounds__(512) void bwd_small_kernel(
    const S *__restrict__ x, const S *__restrict__ w, const S *__restrict__ lam,
    const S *__restrict__ u, const S *__restrict__ dy, S *__restrict__ dx,
    S *__restrict__ dw, S *__restrict__ dlam, S *__restrict__ du, float *__restrict__ dwp,
    int mask, int B, int C, int G, int H, int W, int cw, int nchunk, int pm)
{
    constexpr int NL = 64 / T;
    extern __shared__ float smem[];
    const int pitch = W | 1;                  // odd pitch: column walks are conflict-free
    const int plane = H * pitch;
    float *X = smem;                          // [cw][H][pitch]   dx accumulators
    float *slots = smem + cw * plane;         // [2][cw][3][T]    per-step dw terms

    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int line = lane / T;
    const int j = lane % T;
    const int cpg = C / G;
    const int chunk = blockIdx.x % nchunk;
    const int bg = blockIdx.x / nchunk;
    const int g = bg % G;
    const int b = bg / G;
    const int cfirst = chunk * cw;            // first channel of this chunk, within the group
    const int nvalid = min(cw, cpg - cfirst);
    const int q = wave * NL + line;           // channel slot inside the workgroup
    const bool cvalid = q < nvalid;
    const int c = g * cpg + cfirst + (cvalid ? q : 0);
    const int HW = H * W;
    const int D = __popc(mask);
    const int dfirst = __ffs(mask) - 1;
    float *Xq = X + q * plane;
    const S *xp = x + ((int64_t)b * C + c) * HW;
    const S *dyp = dy + ((int64_t)b * C + c) * HW;

    for (int d = 0; d < 4; ++d) {
        const int bit = 1 << d;
        if (!(mask & bit))
            continue;
        const int s = dir_slot(mask, bit);
        const int L = scan_len(d, H, W);
        const int P = line_len(d, H, W);
        const bool active = cvalid && j < P;
        const int jc = active ? j : 0;
        const Frame f = make_frame(d, jc, H, W, W, pm != 0);
        const Frame fl = make_frame(d, jc, H, W, pitch);
        const int64_t pd = (((int64_t)s * B + b) * C + c) * HW;
        const S *lp = lam + pd;
        const S *up = u + pd;
        S *dlp = dlam + pd;
        S *dup = du + pd;
        const S *wp = w + (((int64_t)s * B + b) * G + g) * 3 * HW;
        const bool m0 = active && j > 0;
        const bool m2 = active && j + 1 < P;

        // Forward sweep: line states of this direction, kept in registers.
        float hist[T];
        float h = 0.f;
#pragma unroll
        for (int i = 0; i < T; ++i) {
            if (i < L) {
                const int e = f.e0 + i * f.es;   // pixel (x)
                const int q = f.lm(i);           // per-direction planes (lam, u, w)
                float inj = load_f(lp + q) * load_f(xp + e);
                inj = active ? inj : 0.f;
                float hn = inj;
                if (i > 0) {
                    float w0 = load_f(wp + q);
                    float w1 = load_f(wp + HW + q);
                    float w2 = load_f(wp + 2 * HW + q);
                    w0 = m0 ? w0 : 0.f;
                    w1 = active ? w1 : 0.f;
                    w2 = m2 ? w2 : 0.f;
                    const float hl = from_left<T>(h);
                    const float hr = from_right<T>(h);
                    hn = fmaf(w1, h, hn);
                    hn = fmaf(w0, hl, hn);
                    hn = fmaf(w2, hr, hn);
                }
                h = hn;
                hist[i] = h;
            }
        }

        // Reverse sweep: adjoint a_i from a_{i+1} through the transposed
        // tridiagonal step (the neighbours' taps of line i+1).
        float an = 0.f;
#pragma unroll
        for (int i = T - 1; i >= 0; --i) {
            if (i < L) {
                const int e = f.e0 + i * f.es;   // pixel (x, dy)
                const int qd = f.lm(i);          // per-direction planes (lam, u, w, dlam, du)
                const float dyv = load_f(dyp + e);
                float a = load_f(up + qd) * dyv;
                if (i + 1 < L) {
                    const int qn = f.lm(i + 1);
                    float w0 = load_f(wp + qn);
                    float w1 = load_f(wp + HW + qn);
                    float w2 = load_f(wp + 2 * HW + qn);
                    w0 = m0 ? w0 : 0.f;
                    w1 = active ? w1 : 0.f;
                    w2 = m2 ? w2 : 0.f;
                    // target j+1 reads this position through its tap 0,
                    // target j-1 through its tap 2.
                    const float q0 = from_right<T>(w0 * an);
                    const float q2 = from_left<T>(w2 * an);
                    a = fmaf(w1, an, a);
                    a += q0;
                    a += q2;
                }
                a = active ? a : 0.f;
                const float xv = load_f(xp + e);
                const float lv = load_f(lp + qd);
                if (active) {
                    store_f(dup + qd, dyv * hist[i]);
                    store_f(dlp + qd, a * xv);
                    const int ae = fl.e0 + i * fl.es;
                    Xq[ae] = (d == dfirst) ? a * lv : Xq[ae] + a * lv;
                }
                // weight-gradient terms of line i (zero on line 0 and on
                // taps that leave the grid)
                float t0 = 0.f, t1 = 0.f, t2 = 0.f;
                if (i > 0) {
                    const float hp = hist[i - 1];
                    const float hl = from_left<T>(hp);
                    const float hr = from_right<T>(hp);
                    t0 = m0 ? a * hl : 0.f;
                    t1 = active ? a * hp : 0.f;
                    t2 = m2 ? a * hr : 0.f;
                }
                float *sl = slots + ((i & 1) * cw + q) * 3 * T;
                sl[j] = t0;
                sl[T + j] = t1;
                sl[2 * T + j] = t2;
                __syncthreads();
                for (int t = threadIdx.x; t < 3 * P; t += blockDim.x) {
                    const int k = t / P;
                    const int jj = t - k * P;
                    const float *src = slots + (i & 1) * cw * 3 * T + k * T + jj;
                    float sum = 0.f;
                    for (int qq = 0; qq < nvalid; ++qq)
                        sum += src[qq * 3 * T];
                    const Frame ft = make_frame(d, jj, H, W, W, pm != 0);
                    const int et = k * HW + ft.lm(i);
                    const int64_t unit = ((int64_t)s * B + b) * G + g;
                    if (nchunk == 1)
                        store_f(dw + unit * 3 * HW + et, sum);
                    else
                        dwp[((int64_t)chunk * D * B * G + unit) * 3 * HW + et] = sum;
                }
                an = a;
            }
        }
        __syncthreads();   // slot buffers are reused by the next direction
    }

    // dx of this wave's channels
    const int nmine = max(0, min(NL, nvalid - wave * NL));
    S *dxb = dx + ((int64_t)b * C + g * cpg + cfirst + wave * NL) * HW;
    const float *Xw = X + wave * NL * plane;
    for (int t = lane; t < nmine * HW; t += 64) {
        const int l = t / HW;
        const int rc = t - l * HW;
        const int r = rc / W;
        const int col = rc - r * W;
        store_f(dxb + t, Xw[l * plane + r * pitch + col]);
    }
}

// dw = sum over chunks of the fp32 partials, in chunk order.
template <typename S>
__global__ __launch_bounds__(256) void dw_reduce_kernel(const float *__restrict__ dwp,
                                                        S *__restrict__ dw, int64_t n, int nchunk)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x) {
        float sum = 0.f;
        for (int k = 0; k < nchunk; ++k)
            sum += dwp[k * n + e];
        store_f(dw + e, sum);
    }
}

template <int T, typename S>
hipError_t fwd_small_t(const Problem &p, hipStream_t st)
{
    if (p.ws->counting)
        return hipSuccess;
    constexpr int NL = 64 / T;
    const int nblk = (p.C + NL - 1) / NL;
    const dim3 grid((unsigned)(p.B * nblk));
    hipLaunchKernelGGL((fwd_small_kernel<T, S>), grid, dim3(256), 0, st,
                       (const S *)p.x, (const S *)p.w, (const S *)p.lam, (const S *)p.u, (S *)p.y,
                       p.mask, p.B, p.C, p.G, p.H, p.W, p.layout);
    return hipGetLastError();
}

// The backward's split: `cw` channels a workgroup, `nchunk` workgroups a group.
struct BwdSplit {
    int cw, nchunk;                  // nchunk 0: no channel fits
    size_t per_ch;                   // LDS bytes a channel
};

BwdSplit bwd_split(const Problem &p, int T)
{
    const int NL = 64 / T, pitch = p.W | 1, cpg = p.C / p.G;
    BwdSplit q{0, 0, (size_t)p.H * pitch * 4 + 2 * 3 * T * 4};
    int cap = (int)((size_t)kLdsBytes / q.per_ch);
    cap = cap < 8 * NL ? cap : 8 * NL;
    cap = cap / NL * NL;
    if (cap < NL)
        return q;
    q.nchunk = (cpg + cap - 1) / cap;
    q.cw = (cpg + q.nchunk - 1) / q.nchunk;
    q.cw = (q.cw + NL - 1) / NL * NL;
    return q;
}

int64_t dw_elems(const Problem &p)
{
    return (int64_t)__builtin_popcount(p.mask) * p.B * p.G * 3 * p.H * p.W;
}

template <int T, typename S>
hipError_t bwd_small_t(const Problem &p, hipStream_t st)
{
    constexpr int NL = 64 / T;
    hipError_t e = hipSuccess;
    const BwdSplit q = bwd_split(p, T);
    const int cw = q.cw, nchunk = q.nchunk;
    if (nchunk == 0)
        return hipErrorInvalidConfiguration;
    const int nwaves = cw / NL;
    const size_t lds = (size_t)cw * q.per_ch;
    const int64_t ndw = dw_elems(p);

    float *dwp = nullptr;
    if (nchunk > 1) {
        e = p.ws->take((void **)&dwp, (size_t)nchunk * ndw * sizeof(float));
        if (e != hipSuccess)
            return e;
    }
    if (p.ws->counting)
        return hipSuccess;
    e = hipFuncSetAttribute((const void *)bwd_small_kernel<T, S>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    const dim3 grid((unsigned)(p.B * p.G * nchunk));
    hipLaunchKernelGGL((bwd_small_kernel<T, S>), grid, dim3(64 * nwaves), lds, st,
                       (const S *)p.x, (const S *)p.w, (const S *)p.lam, (const S *)p.u,
                       (const S *)p.dy, (S *)p.dx, (S *)p.dw, (S *)p.dlam, (S *)p.du, dwp,
                       p.mask, p.B, p.C, p.G, p.H, p.W, cw, nchunk, p.layout);
    e = hipGetLastError();
    if (e == hipSuccess && nchunk > 1) {
        int64_t blocks = (ndw + 255) / 256;
        blocks = blocks < 8192 ? blocks : 8192;
        hipLaunchKernelGGL((dw_reduce_kernel<S>), dim3((unsigned)blocks), dim3(256), 0, st,
                           (const float *)dwp, (S *)p.dw, ndw, nchunk);
        e = hipGetLastError();
    }
    return e;
}

template <int T>
hipError_t fwd_small_dt(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? fwd_small_t<T, float>(p, st) : fwd_small_t<T, bf16_t>(p, st);
}

template <int T>
hipError_t bwd_small_dt(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? bwd_small_t<T, float>(p, st) : bwd_small_t<T, bf16_t>(p, st);
}

int lanes_per_line(int H, int W)
{
    const int m = H > W ? H : W;
    return m <= 16 ? 16 : (m <= 32 ? 32 : 64);
}

}  // namespace

// Where the forward here is the fastest of the three that take any plane up to 64
// a side (times in us: small / plane / line).  It stages nothing and takes the
// directions side by side, so with few planes it is one scan's latency, and its
// loads are whole lines for vertical directions and blocked planes; pixel-major
// horizontal ones (`gather`) touch a line of memory per lane.  `w`: its
// workgroups, of one wave a direction.
//  * up to 16 a side plane wins once its workgroups fill the chip and a wave's
//    four channels are of one group: 13 x 13, four directions, G = C, w = 1024:
//    18 / 25 / 96; 4 channels a group, w = 512: 11 / 13 / 43, 1024: 18 / 14 / 71; 2
//    channels, w = 700: 14 / 14, 1100: 20 / 16; 15 x 15 blocked, 2, w = 5309: 84 /
//    117.  At G = C its loads of horizontal lines, 16 to a wave, stop being served
//    by the cache with many planes in flight (`many`): fp32 8 x 8 blocked, three
//    directions, w = 4920: 73 / 46, 10 x 10, four, 19710: 417 / 286; bf16 11 x 11,
//    four, 7104 and less: even, 28072: 423 / 316, but with rows of 16 bytes 9 x 8,
//    12632: 106 / 133, and blocked 9 x 9, 35073: 453 / 486;
//  * pixel-major with horizontal directions: few planes up to 40 a side, 28 x 28
//    bf16, B*C = 256: 14 / 27 / 16, 1024: 23 / 27 / 29, 12288: 208 / 87 / 249; fp32
//    1024: 39 / 31 / 28; 37 x 37 bf16 256: 20 / 27 / 21, 1024: 73 / 28 / 38.  One
//    direction alone gives the line family nothing to run side by side: 59 x 45
//    L2R, 142 planes bf16: 14 / 18 / 17, fp32: 21 / 21 / 19;
//  * otherwise up to 32 a side: vertical pixel-major bf16 until w = 900, or until
//    two directions are 1552 waves (25 x 25, two, w = 700: 11 / 14 / 19, 900: 13 /
//    14 / 23), and where plane holds under 8 channels a CU (31 x 31, 3 a group,
//    two, w = 2010: 30 / 52 / 36); fp32 until w = 900, where plane holds under 10
//    until 2000 (24 x 24, two, w = 816: 13 / 27 / 18, 2000: 27 / 33 / 29); blocked
//    until w = 850 (28 x 27, 12 a group, four, w = 750: 36 / 48 / 62, 1500: 63 / 52 /
//    95), and always where plane holds under 10 channels a CU, fp32 7 (31 x 31, 3 a
//    group, four, w = 2010: 80 / 182 / 144); both where one or two waves share large
//    planes' taps (28 x 28, 2 a group, two, w = 1920: pixel-major 27 / 40 / -,
//    blocked 45 / 68 / -);
//  * blocked up to 64, where line turns every plane around first: bf16 53 x 53,
//    three directions, w = 224: 22 / 71 / 53; 47 x 47, four, w = 2112: 134 / 161 /
//    131; planes that plane holds 6 or 8 of until w = 800 (44 x 28 L2R, 828: 24 /
//    15 / 27), large ones until 4000 (36 x 55, two directions, 1920: 76 / 74 / 69,
//    44 x 44, two, 6656: 243 / 189 / 194); of three or four directions 6 suffice
//    from 2400 with taps to share (33 x 42, four, 3 a group, 3072: 155 / 122 / 191,
//    38 x 38, 12 a group, 2016: 107 / 113 / 109).  fp32, whose planes are twice the bytes to turn, until one or two
//    directions are 1400 waves and more 2200 (55 x 55, four, w = 216: 42 / 140 / 68;
//    48 x 33, three, w = 1576: 118 / 182 / 165), but for large planes of several
//    channels a group (64 x 64, four, 12 a group, w = 36: 52 / 130 / 39) or of few
//    (56 x 56, four, 2: 46 / 98 / 33).
bool small_fwd_preferred(const Problem &p)
{
    const int T = lanes_per_line(p.H, p.W), cpg = p.C / p.G, HW = p.H * p.W;
    const bool f32 = p.dtype == 0, pm = p.layout == kPixelMajor;
    const int64_t w = ((int64_t)p.B * p.C * T + 63) / 64;
    const int D = __builtin_popcount(p.mask);
    const bool gather = pm && (p.mask & 12) != 0;
    if (w > kMaxThreads / 256)
        return false;
    if (T == 16) {
        const bool many = (p.mask & 12) != 0 && HW >= 40 && HW <= (f32 && !pm ? 100 : 180) &&
                          (f32 ? w >= 4900 : pm && p.W % 8 != 0 && w >= 12000);
        return w < 800 || (cpg == 1 ? !many : !pm && cpg < 4 && HW >= 190);
    }
    if (gather) {
        if (T == 64 && D == 1)
            return w <= (f32 ? 128 : 256);
        return p.H <= 40 && p.W <= 40 && w * (f32 ? 4 : 2) <= (T == 64 ? 512 : 1024);
    }
    if (T == 32) {
        const bool lone = cpg < 4 && HW >= 700;
        const int ch = plane_channels(p, false);
        if (pm)
            return f32 ? w < 900 || (w < 2000 && ch < 10)
                       : (w < 900 && w * D < 1552) || lone || ch < 8;
        return w < 850 || lone || ch < (f32 ? 7 : 10);
    }
    if (pm)
        return p.H <= 40 && p.W <= 40 && w * (f32 ? 4 : 2) <= 512;
    if (f32)
        return w * D < (D > 2 ? 2200 : 1400) && (D <= 2 || HW < 2400 || (cpg == 1 && w >= 100));
    return w < 800 || (HW >= 1800 && w < 4000) ||
           plane_channels(p, false) < (D > 2 && (w < 2400 || cpg < 3) ? 8 : 6);
}

// ... and the backward: planes of a few pixels, which plane's staging and
// barriers exceed, of groups whose channels a step here takes in turn (small /
// plane; line takes several times either): 1 x 1 T2B, B*C = 46326: 14 / 34, four
// directions 36 / 86; 1 x 8 T2B, 58448: 14 / 33; 5 x 2, four, 4524 of G = C: 28 /
// 38; 3 x 3, four, 2048, 4 a group: 17 / 18, 256, 32 a group: 30 / 22; 3 x 1 L2R
// and R2L, 19296, 32 a group: 11 / 25; 4 x 4, four, 512: 20 / 17; 1 x 8 L2R and
// R2L, 32: 34 / 16; 5 x 4 T2B, 2000: 8.1 / 8.1.
bool small_bwd_preferred(const Problem &p)
{
    const int HW = p.H * p.W, m = p.H > p.W ? p.H : p.W;
    const int steps = std::max((p.mask & 3) ? p.H : 0, (p.mask & 12) ? p.W : 0);
    const bool few = __builtin_popcount(p.mask) == 1 ? HW <= 20 && m <= 16 : HW < 12 && m <= 5;
    return few && (int64_t)(p.C / p.G) * steps <= 64;
}

// Bytes of the backward's partial sums.
int64_t small_bwd_bytes(const Problem &p)
{
    const int n = bwd_split(p, lanes_per_line(p.H, p.W)).nchunk;
    return n > 1 ? n * dw_elems(p) * (int64_t)sizeof(float) : 0;
}

hipError_t launch_fwd_small(const Problem &p, hipStream_t st)
{
    switch (lanes_per_line(p.H, p.W)) {
    case 16: return fwd_small_dt<16>(p, st);
    case 32: return fwd_small_dt<32>(p, st);
    default: return fwd_small_dt<64>(p, st);
    }
}

hipError_t launch_bwd_small(const Problem &p, hipStream_t st)
{
    switch (lanes_per_line(p.H, p.W)) {
    case 16: return bwd_small_dt<16>(p, st);
    case 32: return bwd_small_dt<32>(p, st);
    default: return bwd_small_dt<64>(p, st);
    }
}

}  // namespace gspn
