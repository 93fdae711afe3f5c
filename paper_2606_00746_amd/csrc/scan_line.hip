// Line scans of any storage type, layout and side up to kLineSide, as
// independent sweeps over lines in memory, for the planes that no on-chip
// family takes.
//
// The two recurrences of the backward do not depend on each other: the
// forward sweep makes h from lam, x and w, the reverse sweep the adjoint a
// from u, dy and w.  Every gradient is then local:
//   du = dy h,  dlam = a x,  dx = sum_d a_d lam_d,
//   dw_i[j,k] = sum_{c in group} a_i[j] h_{i-1}[j+k-1].
// So one launch runs both sweeps of every direction and channel, a wave
// each, and stores h and a as fp32 lines; a second takes tiles of pixels,
// reads h and a of every channel of a group and writes all gradients, the
// group's dw summed in registers.  A sweep carries one line in registers and
// no history, and there are 2 D B C waves of them instead of one workgroup
// per (direction, batch, group) taking the group's channels in turn.
//
// A wave owns a whole line, lane l the K adjacent positions K l .. K l + K-1
// (K = 1, 2 or 4 for lines of up to 64, 128, 256), so a step reads whole
// rows.  Horizontal directions read copies whose lines are rows
// (transpose_kernel: x, dy, lam, u and w turned around once); vertical
// pixel-major ones read the caller's planes in place; blocked planes, and
// lines shorter than K, are gathered into rows.  Copies and fp32 lines have a
// pitch of a multiple of 4 elements.
//
// The work is taken in rounds of whole weight groups whose workspace fits in
// kRoundBytes.
//
// 128 x 128, B = 2, C = 192, G = 6, four directions, bf16, training pair: 13315 us
// with one workgroup per (direction, batch, group), 341 us so.  Of that the sweeps
// take 48 us in the forward and 86 us in the backward (more than half of their wave
// time waits to issue, three waves a SIMD), the gradients 131 us (474 MB, 3.6 TB/s:
// each of their phases waits for its tile, two workgroups a CU), the turned copies
// 16 and 29 us, the merge 26 us.
#include <algorithm>

#include "cdna.hpp"
#include "device.hpp"
#include "launch.hpp"

namespace gspn {

namespace {

using namespace cdna;

constexpr int pad4(int v) { return (v + 3) & ~3; }

// One direction of a round.  lam, u, w: rows of `lp` elements, planes of
// lsz (lam, u; first plane of the round) and 3 lsz (w) elements; x, dy: rows
// of `xp` elements, planes of xsz; h, a: rows of `op` floats, planes of osz.
struct LineDir {
    const void *lam, *u, *w, *x, *dy;
    float *h, *a;
    int L, P, lp, xp, op;
    int64_t lsz, xsz, osz;
    bool rev;
};

struct SweepArgs {
    LineDir dir[4];
    int nd, np, cpg;      // directions, channel planes of the round, planes per group
};

// K adjacent stored elements of a row, from any element-aligned address.
template <typename S, int K>
struct Raw {
    static constexpr int NB = K * (int)sizeof(S);
    static constexpr int NW = NB < 4 ? 1 : NB / 4;
    uint32_t d[NW];
    __device__ __forceinline__ void load(const void *base, uint32_t off)
    {
        const char *p = static_cast<const char *>(base) + off;
        if constexpr (NB == 2) {
            d[0] = *reinterpret_cast<const uint16_t *>(p);
        } else if constexpr (NB == 4) {
            typedef uint32_t T __attribute__((aligned(2)));
            d[0] = *reinterpret_cast<const T *>(p);
        } else if constexpr (NB == 8) {
            typedef uint32_t T __attribute__((ext_vector_type(2), aligned(2)));
            const T v = *reinterpret_cast<const T *>(p);
            d[0] = v.x, d[1] = v.y;
        } else {
            typedef uint32_t T __attribute__((ext_vector_type(4), aligned(4)));
            const T v = *reinterpret_cast<const T *>(p);
            d[0] = v.x, d[1] = v.y, d[2] = v.z, d[3] = v.w;
        }
    }
    // Widened elements; the lane's first element sits r elements in (the last
    // lane of a line whose length is not a multiple of K reads from P - K).
    template <bool RAG>
    __device__ __forceinline__ void get(int r, float (&v)[K]) const
    {
        if constexpr (sizeof(S) == 4) {
            float f[K];
#pragma unroll
            for (int k = 0; k < K; ++k)
                f[k] = __uint_as_float(d[k]);
            if constexpr (RAG && K == 4) {
                if (r & 2)
                    f[0] = f[2], f[1] = f[3];
                if (r & 1)
                    f[0] = f[1], f[1] = f[2], f[2] = f[3];
            } else if constexpr (RAG && K == 2) {
                if (r & 1)
                    f[0] = f[1];
            }
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[k] = f[k];
        } else if constexpr (K == 1) {
            v[0] = bf_lo(d[0]);
        } else if constexpr (K == 2) {
            const uint32_t q = RAG ? d[0] >> (16 * r) : d[0];
            v[0] = bf_lo(q), v[1] = bf_hi(q);
        } else {
            uint64_t q = ((uint64_t)d[1] << 32) | d[0];
            if (RAG)
                q >>= 16 * r;
            const uint32_t lo = (uint32_t)q, hi = (uint32_t)(q >> 32);
            v[0] = bf_lo(lo), v[1] = bf_hi(lo), v[2] = bf_lo(hi), v[3] = bf_hi(hi);
        }
    }
};

// A step's store of K fp32 values.  The registers of a wide store have to keep
// their values for some cycles after it: the values stored stay alive until the
// next step's store (hold), which costs no wait states (16 of them behind each
// store: 48 x 80 bf16 C = 256 forward 32.3 -> 35.6 us).  The empty asm gives them
// registers of their own, which the state then lives in.
template <int K>
struct LineStore {
    typedef uint32_t V __attribute__((ext_vector_type(K)));
    V last = {};
    __device__ __forceinline__ void hold() const
    {
        if constexpr (K > 1)
            asm volatile("" : : "v"(last));
    }
    __device__ __forceinline__ void put(float *base, uint32_t off, float (&v)[K], bool on)
    {
        if constexpr (K > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                last[k] = __float_as_uint(v[k]);
            asm volatile("" : "+v"(last));
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[k] = __uint_as_float(last[k]);
        } else {
            last[0] = __float_as_uint(v[0]);
        }
        if (!on)
            return;
        *reinterpret_cast<V *>(reinterpret_cast<char *>(base) + off) = last;
    }
};

// One sweep of one (direction, channel): steps of the scan in order, or in
// reverse for the adjoint (ADJ).  s0, s1: the two streams whose product is
// injected (lam, x or u, dy).  U steps' loads are in flight while the U
// steps before them run.
template <typename S, int K, bool RAG, bool ADJ>
__device__ __forceinline__ void sweep(const LineDir &D, const S *s0, const S *s1, const S *w,
                                      float *out, int lane)
{
    using R = Raw<S, K>;
    constexpr int U = R::NW >= 4 ? 2 : (R::NW == 2 ? 4 : 8);
    const int L = D.L, P = D.P;
    const int p0 = K * lane;
    const int pc = p0 < P - K ? p0 : (P >= K ? P - K : 0);   // where the lane reads
    const int r = p0 - pc < K ? p0 - pc : 0;
    const uint32_t es = sizeof(S);
    bool on[K], on0[K], on2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        on[k] = p0 + k < P;
        on0[k] = on[k] && p0 + k > 0;
        on2[k] = p0 + k + 1 < P;
    }
    // storage line of the n-th step taken, and its offsets
    const bool down = D.rev != ADJ;
    auto line = [&](int n) { return down ? L - 1 - n : n; };
    const S *w1 = w + D.lsz, *w2 = w + 2 * D.lsz;
    struct Step {
        R a, b, t0, t1, t2;
    };
    auto fetch = [&](Step (&q)[U], int n0) {
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int n = n0 + t < L ? n0 + t : L - 1;
            const int l = line(n);
            const uint32_t ol = es * (uint32_t)(l * D.lp + pc), ox = es * (uint32_t)(l * D.xp + pc);
            q[t].a.load(s0, ol);
            q[t].b.load(s1, ox);
            q[t].t0.load(w, ol);
            q[t].t1.load(w1, ol);
            q[t].t2.load(w2, ol);
        }
    };
    LineStore<K> rows;
    float st[K], v0[K], v1[K], v2[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
        st[k] = v0[k] = v1[k] = v2[k] = 0.f;
    auto run = [&](const Step (&q)[U], int n0) {
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int n = n0 + t;
            if (n >= L)
                break;
            float a[K], b[K], inj[K], t0[K], t1[K], t2[K];
            q[t].a.template get<RAG>(r, a);
            q[t].b.template get<RAG>(r, b);
            q[t].t0.template get<RAG>(r, t0);
            q[t].t1.template get<RAG>(r, t1);
            q[t].t2.template get<RAG>(r, t2);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                inj[k] = on[k] ? a[k] * b[k] : 0.f;
                t0[k] = on0[k] ? t0[k] : 0.f;
                t1[k] = on[k] ? t1[k] : 0.f;
                t2[k] = on2[k] ? t2[k] : 0.f;
            }
            if (n == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    st[k] = inj[k];
            } else if constexpr (!ADJ) {
                // h_i[j] = w0 h[j-1] + w1 h[j] + w2 h[j+1] + lam x
                const float hl = from_left<64>(st[K - 1]), hr = from_right<64>(st[0]);
                float hn[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    hn[k] = fmaf(t1[k], st[k], inj[k]);
                    hn[k] = fmaf(t0[k], k > 0 ? st[k > 0 ? k - 1 : 0] : hl, hn[k]);
                    hn[k] = fmaf(t2[k], k + 1 < K ? st[k + 1 < K ? k + 1 : 0] : hr, hn[k]);
                }
#pragma unroll
                for (int k = 0; k < K; ++k)
                    st[k] = on[k] ? hn[k] : 0.f;
            } else {
                // a_i[j] = w1 a[j] + (w0 a)[j+1] + (w2 a)[j-1] + u dy, the taps
                // those of step i+1, read with the step before this one
                float q0[K], q2[K], an[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    q0[k] = v0[k] * st[k];
                    q2[k] = v2[k] * st[k];
                }
                const float ql = from_left<64>(q2[K - 1]), qr = from_right<64>(q0[0]);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    an[k] = fmaf(v1[k], st[k], inj[k]);
                    an[k] += k + 1 < K ? q0[k + 1 < K ? k + 1 : 0] : qr;
                    an[k] += k > 0 ? q2[k > 0 ? k - 1 : 0] : ql;
                    an[k] = on[k] ? an[k] : 0.f;
                }
#pragma unroll
                for (int k = 0; k < K; ++k)
                    st[k] = an[k];
            }
            if (ADJ) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    v0[k] = t0[k], v1[k] = t1[k], v2[k] = t2[k];
            }
            rows.hold();
            rows.put(out, 4u * (uint32_t)(line(n) * D.op + p0), st, p0 < D.op);
        }
    };
    Step qa[U], qb[U];
    fetch(qa, 0);
    for (int n0 = 0;;) {
        fetch(qb, n0 + U);
        run(qa, n0);
        n0 += U;
        if (n0 >= L)
            break;
        fetch(qa, n0 + U);
        run(qb, n0);
        n0 += U;
        if (n0 >= L)
            break;
    }
}

// Four waves of a workgroup: four consecutive channel planes of one direction
// and sweep.  Workgroups of one direction and sweep are consecutive, planes
// in order, so that a group's taps are read under one L2.
template <typename S, int K, bool RAG>
__global__ __launch_bounds__(256) void sweep_kernel(const SweepArgs A, int nblk, bool bwd)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int row = blk / nblk;                       // direction slot, sweep
    const int pl = 4 * (blk - row * nblk) + wave;     // channel plane of the round
    const int s = bwd ? row >> 1 : row;
    if (pl >= A.np)
        return;
    const LineDir &D = A.dir[s];
    const S *w = static_cast<const S *>(D.w) + (int64_t)(pl / A.cpg) * 3 * D.lsz;
    const int64_t ol = pl * D.lsz, ox = pl * D.xsz, oo = pl * D.osz;
    if (!(bwd && (row & 1)))
        sweep<S, K, RAG, false>(D, static_cast<const S *>(D.lam) + ol,
                                static_cast<const S *>(D.x) + ox, w, D.h + oo, lane);
    else
        sweep<S, K, RAG, true>(D, static_cast<const S *>(D.u) + ol,
                               static_cast<const S *>(D.dy) + ox, w, D.a + oo, lane);
}

// ---------------------------------------------------------------------------
// rows out of planes
// ---------------------------------------------------------------------------

// Planes to turn around: n planes of H x W at src -> W rows of `pitch`
// elements at dst.
struct Turn {
    const void *src;
    void *dst;
    int first;                   // first plane of this part in the launch
};
constexpr int kMaxTurns = 8;
struct TurnArgs {
    Turn t[kMaxTurns];
    int nt, H, W, pitch, tiles_c, tiles;
};

// One 64 x 64 tile of one plane per workgroup, through LDS.
template <typename S>
__global__ __launch_bounds__(256) void transpose_kernel(const TurnArgs A)
{
    __shared__ S tile[64][64 + (sizeof(S) == 4 ? 1 : 2)];
    const int pl = blockIdx.x / A.tiles, tl = blockIdx.x - pl * A.tiles;
    int k = 0;
    while (k + 1 < A.nt && pl >= A.t[k + 1].first)
        ++k;
    const int tr = tl / A.tiles_c, r0 = 64 * tr, c0 = 64 * (tl - tr * A.tiles_c);
    const int64_t i = pl - A.t[k].first;
    const S *src = static_cast<const S *>(A.t[k].src) + i * A.H * A.W;
    S *dst = static_cast<S *>(A.t[k].dst) + i * A.W * A.pitch;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    S v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = r0 + wave + 4 * q, c = c0 + lane;
        v[q] = r < A.H && c < A.W ? src[(int64_t)r * A.W + c] : S(0);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
        tile[wave + 4 * q][lane] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int c = c0 + wave + 4 * q, r = r0 + lane;
        if (c < A.W && r < A.pitch)
            dst[(int64_t)c * A.pitch + r] = tile[lane][wave + 4 * q];
    }
}

// Rows of `pitch` elements from n planes in either layout, element by element
// (blocked planes; lines shorter than a lane's positions).
template <typename S>
__global__ __launch_bounds__(256) void rows_kernel(const S *__restrict__ src, S *__restrict__ dst,
                                                   int64_t n, int L, int P, int W, int pitch,
                                                   int vert, int pm)
{
    const int per = L * pitch, HW = L * P;
    for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n * per;
         o += (int64_t)gridDim.x * blockDim.x) {
        const int64_t pl = o / per;
        const int e = (int)(o - pl * per);
        const int l = e / pitch, p = e - l * pitch;
        dst[o] = p < P ? src[pl * HW + dir_offset(pm != 0, vert != 0, l, p, L, P, W)] : S(0);
    }
}

// ---------------------------------------------------------------------------
// gradients (and the forward's merge) from the lines
// ---------------------------------------------------------------------------

constexpr int kTileR = 32, kTileC = 64;       // pixels of a tile
constexpr int kTileThreads = 512;             // 4 pixels each: 2 columns of 2 rows

struct GradArgs {
    const void *x, *dy, *lam, *u;             // caller's tensors, first plane of the round
    void *y, *dx, *dlam, *du;
    void *dw;                                 // caller's dw, first unit of the round
    float *part;                              // [chunk][slot][unit][3][HW], or null
    const float *h[4], *a[4];                 // per slot
    int opv, oph;                             // row pitch of h and a: vertical, horizontal
    int dirs[4];                              // direction index per slot
    int nd, mask, H, W, cpg, cc;              // cc: channels per chunk
    int64_t per_slot;                         // elements between slots of lam, u, dlam, du
    int64_t w_slot;                           // ... of dw
    int nu, nchunk, tiles_c, tiles, pm;
};

// Offset of an access that its descriptor's range check drops (a load then
// reads 0): every descriptor here covers at most one plane.
constexpr uint32_t kDrop = 0x80000000u;

// Two adjacent pixels of a row as stored, at byte offsets o and (odd rows) o1
// of a plane.  Rows of an even number of elements keep every pair aligned;
// with an odd width the two go separately.  Widened where they are used, so
// that the wait for the load stands there.
template <typename S>
struct Pair;
template <>
struct Pair<bf16_t> {
    uint32_t d;
    __device__ __forceinline__ void load(rsrc_t r, uint32_t o, uint32_t o1, bool odd)
    {
        d = odd ? ld16(r, o, 0) | (ld16(r, o1, 0) << 16) : ld32(r, o, 0);
    }
    __device__ __forceinline__ float get(int e) const { return e ? bf_hi(d) : bf_lo(d); }
    static __device__ __forceinline__ void store(const u32x4 &r, uint32_t o, uint32_t o1, bool odd,
                                                 float a, float b)
    {
        const uint32_t q = pack2(a, b);
        if (odd) {
            st16(r, o, 0, q);
            st16(r, o1, 0, q >> 16);
        } else {
            st32(r, o, 0, q);
        }
    }
};
template <>
struct Pair<float> {
    uint32_t d[2];
    __device__ __forceinline__ void load(rsrc_t r, uint32_t o, uint32_t o1, bool odd)
    {
        if (odd) {
            d[0] = ld32(r, o, 0);
            d[1] = ld32(r, o1, 0);
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
            d[0] = v[0], d[1] = v[1];
        }
    }
    __device__ __forceinline__ float get(int e) const { return __uint_as_float(d[e]); }
    static __device__ __forceinline__ void store(const u32x4 &r, uint32_t o, uint32_t o1, bool odd,
                                                 float a, float b)
    {
        if (odd) {
            st32(r, o, 0, __float_as_uint(a));
            st32(r, o1, 0, __float_as_uint(b));
        } else {
            st64_held(r, o, 0, __float_as_uint(a), __float_as_uint(b));
        }
    }
};

// A tile of one direction's fp32 lines in LDS, lines along the first index.
// Vertical directions: lines are rows, positions columns; horizontal ones the
// other way around.  h is held from one line before the tile's first (scans
// against the storage order: from its first) and from position -1 on, so that
// a thread's 2 x 2 pixels take aligned pairs of positions: position p of a at
// p, of h at p + 1.  The pitches (2 mod 32 in pairs) leave the line walk of
// the horizontal directions two lanes to a bank.
template <bool VERT>
struct TileShape {
    static constexpr int NL = VERT ? kTileR : kTileC, NP = VERT ? kTileC : kTileR;
    static constexpr int Q = NP / 4;                   // 16-byte pieces of a line
    static constexpr int PITCH = NP + 2;
    static constexpr int HL = NL + 1;                  // h lines
};
constexpr int kATile = 64 * 34 > 32 * 66 ? 64 * 34 : 32 * 66;
constexpr int kHTile = 65 * 34 > 33 * 66 ? 65 * 34 : 33 * 66;

// Byte offsets of what a thread loads of a tile in one orientation: its piece
// of a (and, a line earlier for scans in storage order, of h), its piece of
// h's last line, and one of h's halo positions.  What lies off the plane is
// out of the descriptor's range and reads as 0.
struct TileOff {
    uint32_t a, h1, e;
};

template <bool VERT>
__device__ __forceinline__ TileOff tile_off(int t, int l0, int p0, int P, int op)
{
    using T = TileShape<VERT>;
    const int ln = t / T::Q, q = t - ln * T::Q;
    TileOff o;
    o.a = p0 + 4 * q < op ? 4u * (uint32_t)((l0 + ln) * op + p0 + 4 * q) : kDrop;
    o.h1 = t < T::Q && p0 + 4 * t < op ? 4u * (uint32_t)((l0 + T::NL) * op + p0 + 4 * t) : kDrop;
    const int p = (t & 1) ? p0 + T::NP : p0 - 1;
    o.e = t < 2 * T::HL && p >= 0 && p < P ? 4u * (uint32_t)((l0 + (t >> 1)) * op + p) : kDrop;
    return o;
}

// The thread index as a value the compiler cannot see through: LDS addresses
// and blocked offsets derived from it are formed where they are used instead
// of being kept in registers over the channel loop (which spilled).
__device__ __forceinline__ int opaque(int t)
{
    asm volatile("" : "+v"(t));
    return t;
}

struct Fetch {
    uint4 a, h0, h1;
    uint32_t e;
};

// a, h: the plane's descriptors; back: bytes of a line where h starts one
// line earlier, else 0.
__device__ __forceinline__ void fetch_tile(Fetch &f, rsrc_t a, rsrc_t h, const TileOff &o,
                                           uint32_t back)
{
    f.a = ld128(a, o.a, 0);
    f.h0 = ld128(h, o.a - back, 0);
    f.h1 = ld128(h, o.h1 - back, 0);
    f.e = ld32(h, o.e - back, 0);
}

template <bool VERT>
__device__ __forceinline__ void put_tile(const Fetch &f, uint32_t *A, uint32_t *Hh, int t0)
{
    using T = TileShape<VERT>;
    const int t = opaque(t0);
    const int ln = t / T::Q, q = t - ln * T::Q;
    uint2 *pa = reinterpret_cast<uint2 *>(A + ln * T::PITCH + 4 * q);
    pa[0] = make_uint2(f.a.x, f.a.y);
    pa[1] = make_uint2(f.a.z, f.a.w);
    auto put = [](uint32_t *p, const uint4 &v) {
        p[0] = v.x;
        *reinterpret_cast<uint2 *>(p + 1) = make_uint2(v.y, v.z);
        p[3] = v.w;
    };
    put(Hh + ln * T::PITCH + 4 * q + 1, f.h0);
    if (t < T::Q)
        put(Hh + T::NL * T::PITCH + 4 * t + 1, f.h1);
    if (t < 2 * T::HL)
        Hh[(t >> 1) * T::PITCH + ((t & 1) ? T::NP + 1 : 0)] = f.e;
}

template <typename S>
struct GradState {
    Pair<S> x[2], g[2];                      // this channel's 2 x 2 pixels (rows, pairs)
    float dx[2][2];
    float dw[4][2][2][3];                    // the group's sums, per direction
    uint32_t o[2], o1[2];                    // byte offsets of the pixels' rows (kDrop: none)
};

// One direction of one channel.  Element (m, n) of the thread's block: line
// base + m, position base + n of the direction.
template <typename S, bool PM, int D>
__device__ __forceinline__ void grad_dir(const GradArgs &A, GradState<S> &G, const float *At,
                                         const float *Ht, int r0, int c0, int64_t pd, int t0,
                                         const Pair<S> (&lv)[2])
{
    constexpr bool VERT = D < 2, REV = D & 1;
    using T = TileShape<VERT>;
    const int H = A.H, W = A.W, L = VERT ? H : W, P = VERT ? W : H;
    const int t = opaque(t0);
    const int cx = 2 * (t & 31), ry = 2 * (t >> 5);
    const int ln = VERT ? ry : cx, ps = VERT ? cx : ry;
    auto pair = [](const float *p) { return *reinterpret_cast<const float2 *>(p); };
    const float2 a0 = pair(At + ln * T::PITCH + ps), a1 = pair(At + (ln + 1) * T::PITCH + ps);
    const float a[2][2] = {{a0.x, a0.y}, {a1.x, a1.y}};
    // three lines of h, in storage order: before (REV: after) the block's two
    float h[3][4];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float *p = Ht + (ln + m) * T::PITCH + ps;
        const float2 lo = pair(p), hi = pair(p + 2);
        h[m][0] = lo.x, h[m][1] = lo.y, h[m][2] = hi.x, h[m][3] = hi.y;
    }
    float dl[2][2], duv[2][2];               // by (row, column) of the block
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const int q = VERT ? m : n, e = VERT ? n : m;
            const float (&hc)[4] = h[REV ? m : m + 1], (&hb)[4] = h[REV ? m + 1 : m];
            dl[q][e] = a[m][n] * G.x[q].get(e);
            duv[q][e] = G.g[q].get(e) * hc[n + 1];
            G.dx[q][e] = fmaf(a[m][n], lv[q].get(e), G.dx[q][e]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                G.dw[D][q][e][k] = fmaf(a[m][n], hb[n + k], G.dw[D][q][e][k]);
        }
    const u32x4 rl = make_sdesc(static_cast<S *>(A.dlam) + pd, H * W * (uint32_t)sizeof(S));
    const u32x4 ru = make_sdesc(static_cast<S *>(A.du) + pd, H * W * (uint32_t)sizeof(S));
    if constexpr (PM) {
        const bool odd = W & 1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            Pair<S>::store(rl, G.o[q], G.o1[q], odd, dl[q][0], dl[q][1]);
            Pair<S>::store(ru, G.o[q], G.o1[q], odd, duv[q][0], duv[q][1]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = r0 + ry + q, c = c0 + cx + e;
                if (r < H && c < W) {
                    const int o = VERT ? lm_offset(r, c, L, P) : lm_offset(c, r, L, P);
                    store_f(static_cast<S *>(A.dlam) + pd + o, dl[q][e]);
                    store_f(static_cast<S *>(A.du) + pd + o, duv[q][e]);
                }
            }
    }
    step_fence();
}

// All gradients of one tile of pixels, one chunk of a group's channels.  The
// directions are taken in turn for every channel; the next direction's lines
// are loaded while the current one is used (two LDS buffers, one barrier a
// direction).  A thread owns 2 x 2 pixels, whose lines it reads from LDS as
// pairs in either orientation.
template <typename S, bool PM>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(4))) void grad_kernel(
    const GradArgs A)
{
    __shared__ float lds[2][kATile + kHTile];
    const int t = threadIdx.x;
    int idx = xcd_remap(blockIdx.x, gridDim.x);
    const int tl = idx % A.tiles;
    idx /= A.tiles;
    const int chunk = idx % A.nchunk, unit = idx / A.nchunk;
    const int tr = tl / A.tiles_c;
    const int r0 = kTileR * tr, c0 = kTileC * (tl - tr * A.tiles_c);
    const int H = A.H, W = A.W, HW = H * W;
    const uint32_t pbytes = (uint32_t)HW * (uint32_t)sizeof(S);
    const bool odd = W & 1;
    const int first = chunk * A.cc, nch = min(A.cc, A.cpg - first);
    const int pl0 = unit * A.cpg + first;              // first channel plane
    const int col = c0 + 2 * (t & 31), row = r0 + 2 * (t >> 5);
    const TileOff ov = tile_off<true>(t, r0, c0, W, A.opv);
    const TileOff oh = tile_off<false>(t, c0, r0, H, A.oph);
    GradState<S> G;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const bool live = row + q < H && col < W;
        G.o[q] = live ? (uint32_t)((row + q) * W + col) * (uint32_t)sizeof(S) : kDrop;
        G.o1[q] = live && col + 1 < W ? G.o[q] + (uint32_t)sizeof(S) : kDrop;
    }
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    G.dw[d][q][e][k] = 0.f;

    // the next direction's lines and lam, and the next channel's x and dy
    Fetch f;
    Pair<S> nl[2], nx[2], ng[2];
    auto fetch = [&](int ch, int s) {
        const int d = A.dirs[s];
        const int64_t pc = (int64_t)(pl0 + ch) * HW;
        const S *lam = static_cast<const S *>(A.lam) + s * A.per_slot + pc;
        if (s == 0) {
            const rsrc_t rx = make_rsrc(static_cast<const S *>(A.x) + pc, pbytes);
            const rsrc_t rg = make_rsrc(static_cast<const S *>(A.dy) + pc, pbytes);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                nx[q].load(rx, G.o[q], G.o1[q], odd);
                ng[q].load(rg, G.o[q], G.o1[q], odd);
            }
        }
        const bool vert = d < 2;
        const int op = vert ? A.opv : A.oph, L = vert ? H : W;
        const int64_t o = (int64_t)(pl0 + ch) * L * op;
        const rsrc_t ra = make_rsrc(A.a[s] + o, 4u * (uint32_t)(L * op));
        const rsrc_t rh = make_rsrc(A.h[s] + o, 4u * (uint32_t)(L * op));
        const uint32_t back = (d & 1) ? 0u : 4u * (uint32_t)op;
        if (vert)
            fetch_tile(f, ra, rh, ov, back);
        else
            fetch_tile(f, ra, rh, oh, back);
        const rsrc_t rl = make_rsrc(lam, pbytes);
        if constexpr (PM) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                nl[q].load(rl, G.o[q], G.o1[q], odd);
        } else {
            const int P = vert ? W : H, tt = opaque(t);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t oe[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int r = r0 + 2 * (tt >> 5) + q, c = c0 + 2 * (tt & 31) + e;
                    oe[e] = r < H && c < W ? (uint32_t)(vert ? lm_offset(r, c, L, P)
                                                             : lm_offset(c, r, L, P)) *
                                                 (uint32_t)sizeof(S)
                                           : kDrop;
                }
                nl[q].load(rl, oe[0], oe[1], true);
            }
        }
    };
    fetch(0, 0);
    int buf = 0;
    for (int ch = 0; ch < nch; ++ch) {
        const int64_t pc = (int64_t)(pl0 + ch) * HW;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            G.x[q] = nx[q];
            G.g[q] = ng[q];
            G.dx[q][0] = G.dx[q][1] = 0.f;
        }
        for (int s = 0; s < A.nd; ++s) {
            const int d = A.dirs[s];
            float *At = lds[buf], *Ht = lds[buf] + kATile;
            if (d < 2)
                put_tile<true>(f, reinterpret_cast<uint32_t *>(At), reinterpret_cast<uint32_t *>(Ht), t);
            else
                put_tile<false>(f, reinterpret_cast<uint32_t *>(At), reinterpret_cast<uint32_t *>(Ht), t);
            const int64_t pd = s * A.per_slot + pc;
            const Pair<S> lv[2] = {nl[0], nl[1]};
            if (s + 1 < A.nd)
                fetch(ch, s + 1);
            else if (ch + 1 < nch)
                fetch(ch + 1, 0);
            lds_barrier();
            if (d == 0)
                grad_dir<S, PM, 0>(A, G, At, Ht, r0, c0, pd, t, lv);
            else if (d == 1)
                grad_dir<S, PM, 1>(A, G, At, Ht, r0, c0, pd, t, lv);
            else if (d == 2)
                grad_dir<S, PM, 2>(A, G, At, Ht, r0, c0, pd, t, lv);
            else
                grad_dir<S, PM, 3>(A, G, At, Ht, r0, c0, pd, t, lv);
            buf ^= 1;
        }
        const u32x4 rdx = make_sdesc(static_cast<S *>(A.dx) + pc, pbytes);
#pragma unroll
        for (int q = 0; q < 2; ++q)
            Pair<S>::store(rdx, G.o[q], G.o1[q], odd, G.dx[q][0], G.dx[q][1]);
    }
    // the group's weight gradient: final, or this chunk's fp32 partial; taps
    // that the scan ignores are written as 0, whatever their sums hold
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!((A.mask >> d) & 1))
            continue;
        const int tt = opaque(t);
        const int s = dir_slot(A.mask, 1 << d);
        const int L = d < 2 ? H : W, P = d < 2 ? W : H;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int r = r0 + 2 * (tt >> 5) + q, c = c0 + 2 * (tt & 31) + e;
                if (r >= H || c >= W)
                    continue;
                const int l = d < 2 ? r : c, p = d < 2 ? c : r;
                const int o = dir_offset(PM, d < 2, l, p, L, P, W);
                const bool prev = (d & 1) ? l + 1 < L : l > 0;
                const bool on[3] = {prev && p > 0, prev, prev && p + 1 < P};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const float v = on[k] ? G.dw[d][q][e][k] : 0.f;
                    if (A.nchunk == 1)
                        store_f(static_cast<S *>(A.dw) + s * A.w_slot +
                                    ((int64_t)unit * 3 + k) * HW + o, v);
                    else
                        A.part[((((int64_t)chunk * A.nd + s) * A.nu + unit) * 3 + k) * HW + o] = v;
                }
            }
        step_fence();
    }
}

// dw = sum of the chunks' partials, in chunk order.
template <typename S>
__global__ __launch_bounds__(256) void dw_parts_kernel(const float *__restrict__ part,
                                                       S *__restrict__ dw, int64_t per, int nd,
                                                       int nchunk, int64_t w_slot)
{
    const int64_t n = per * nd;
    for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n;
         o += (int64_t)gridDim.x * blockDim.x) {
        float v = 0.f;
        for (int k = 0; k < nchunk; ++k)
            v += part[k * n + o];
        const int64_t s = o / per;
        store_f(dw + s * w_slot + (o - s * per), v);
    }
}

// y = sum_d u_d h_d over one tile of one channel plane: the vertical
// directions' lines are rows of the tile, the horizontal ones are turned
// around through LDS.
template <typename S, bool PM>
__global__ __launch_bounds__(kTileThreads) void merge_kernel(const GradArgs A)
{
    using T = TileShape<false>;
    __shared__ float lds[2][T::NL * T::PITCH];
    const int t = threadIdx.x;
    const int idx = xcd_remap(blockIdx.x, gridDim.x);
    const int pl = idx / A.tiles, tl = idx - pl * A.tiles;
    const int tr = tl / A.tiles_c;
    const int r0 = kTileR * tr, c0 = kTileC * (tl - tr * A.tiles_c);
    const int H = A.H, W = A.W, HW = H * W;
    const uint32_t pbytes = (uint32_t)HW * (uint32_t)sizeof(S);
    const bool odd = W & 1;
    const int cx = 2 * (t & 31), ry = 2 * (t >> 5), col = c0 + cx, row = r0 + ry;
    uint32_t o[2], o1[2], ov[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const bool live = row + q < H && col < W;
        o[q] = live ? (uint32_t)((row + q) * W + col) * (uint32_t)sizeof(S) : kDrop;
        o1[q] = live && col + 1 < W ? o[q] + (uint32_t)sizeof(S) : kDrop;
        ov[q] = live ? 4u * (uint32_t)((row + q) * A.opv + col) : kDrop;
    }
    const TileOff oh = tile_off<false>(t, c0, r0, H, A.oph);
    const int64_t pc = (int64_t)pl * HW;
    // every load first: u, the vertical lines of the block, the horizontal
    // lines' pieces
    Pair<S> uv[4][2];
    float2 hv[4][2];
    uint4 hp[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!((A.mask >> d) & 1))
            continue;
        const int s = dir_slot(A.mask, 1 << d);
        const int L = d < 2 ? H : W, P = d < 2 ? W : H, op = d < 2 ? A.opv : A.oph;
        const rsrc_t rh = make_rsrc(A.h[s] + (int64_t)pl * L * op, 4u * (uint32_t)(L * op));
        const rsrc_t ru = make_rsrc(static_cast<const S *>(A.u) + s * A.per_slot + pc, pbytes);
        if (d >= 2)
            hp[d] = ld128(rh, oh.a, 0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (d < 2) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rh, ov[q], 0, 0);
                hv[d][q] = make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
            }
            if constexpr (PM) {
                uv[d][q].load(ru, o[q], o1[q], odd);
            } else {
                uint32_t oe[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int r = row + q, c = col + e;
                    oe[e] = r < H && c < W ? (uint32_t)(d < 2 ? lm_offset(r, c, L, P)
                                                              : lm_offset(c, r, L, P)) *
                                                 (uint32_t)sizeof(S)
                                           : kDrop;
                }
                uv[d][q].load(ru, oe[0], oe[1], true);
            }
        }
    }
#pragma unroll
    for (int d = 2; d < 4; ++d) {
        if (!((A.mask >> d) & 1))
            continue;
        const int ln = t / T::Q, q = t - ln * T::Q;
        uint2 *p = reinterpret_cast<uint2 *>(lds[d - 2] + ln * T::PITCH + 4 * q);
        p[0] = make_uint2(hp[d].x, hp[d].y);
        p[1] = make_uint2(hp[d].z, hp[d].w);
    }
    lds_barrier();
    float y[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (!((A.mask >> d) & 1))
            continue;
        if (d >= 2) {
            const float2 c0v = *reinterpret_cast<const float2 *>(lds[d - 2] + cx * T::PITCH + ry);
            const float2 c1v = *reinterpret_cast<const float2 *>(lds[d - 2] + (cx + 1) * T::PITCH + ry);
            hv[d][0] = make_float2(c0v.x, c1v.x);
            hv[d][1] = make_float2(c0v.y, c1v.y);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            y[q][0] = add_nc(y[q][0], mul_nc(uv[d][q].get(0), hv[d][q].x));
            y[q][1] = add_nc(y[q][1], mul_nc(uv[d][q].get(1), hv[d][q].y));
        }
    }
    const u32x4 ry_ = make_sdesc(static_cast<S *>(A.y) + pc, pbytes);
#pragma unroll
    for (int q = 0; q < 2; ++q)
        Pair<S>::store(ry_, o[q], o1[q], odd, y[q][0], y[q][1]);
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------

// Workspace.  A round takes what its weight groups need, at most kRoundBytes,
// or one whole group, or the general family's need where these are more (a group
// is never cut: 256 x 256 bf16, C = 768, G = 1, backward: 2.2 GB).  Small rounds
// would leave h and a in the 256 MB Infinity Cache for the gradients, but fill the
// chip less: 128 x 128, B = 2, C = 192 in rounds of 160 MB 453 us, of 240 MB 389
// us, in one (277 MB) 381 us.  The size that the query gives is never below the
// general family's; a caller that hands in less than the query's size, but what the
// general family takes, gets smaller rounds, or the general family.
//
// Below kSmallBytes the query gives what the general family takes, no more, as it
// always has: callers hold workspaces of those sizes, and one byte less is refused
// there.  That is the only reason; the line family with a workspace of its own is
// the faster at nearly every size below (us, general / line: forward fp32 70 x 100,
// B*C = 3: 92 / 26; bf16 70 x 70, 8: 66 / 20, blocked 50 / 38; backward 70 x 70, 8
// of G = C: 179 / 32).  The line lies close above the sizes so held (168,000 and
// 672,000 bytes); from it on the gap is wider than a few hundred kilobytes are
// worth: backward 70 x 70, 8 in one group (0.94 MB): 1515 / 55; 80 x 80, 32 in one
// group, T2B (0.92 MB): 5438 / 29.
constexpr int64_t kRoundBytes = (int64_t)512 << 20;
constexpr int64_t kSmallBytes = (int64_t)704 << 10;
constexpr int64_t kPartPad = 64 * 256;           // alignment of a round's parts

// A small workspace cuts a call into rounds of a group or a few, each with its
// own launches and its own chain of steps.  They are taken where a round still
// has two waves a CU, or where there are so few of them that all planes at once in
// the general family, whose time is its steps, take longer: in the backward up to
// kFewRounds, or in proportion to the channels of a group, which the general
// backward takes in turn; in the forward one for so many steps (kRoundSteps: vertical
// pixel-major directions alone, which turn nothing around; pixel-major; blocked,
// where every tensor of a direction is a launch), a step counted by `load`, the time of
// all planes' general step over that of a few: it grows with their lines, horizontal
// ones, which it reads by columns, most.  us, rounds / general: T2B and B2T,
// 70 x 70, two rounds: 28 / 52, 114 x 114, three: 41 / 81, 21 x 137, two: 27 / 18;
// 62 x 88, two, four directions: 45 / 81, 22 x 145, four, R2L: 151 / 93; blocked 77
// x 77, 8, four directions: 159 / 60, 28 x 154, four: 230 / 97; 51 x 73, L2R, B*C =
// 1448, rounds below that: 144 / 633; blocked 114 x 114, both horizontal, 366: 176 / 248.
//
// The blocked forward, whose rounds have the most launches, and planes up to 64 a side,
// whose other families' backward is faster than the general one, ask for more waves (a workspace
// below the query's; us, rounds / the other family): blocked 35 x 149, four
// directions, three rounds of 1376: 393 / 277; backward 38 x 38, T2B and B2T, seven of
// 1088: 322 / 175, blocked eleven of 704: 847 / 180, 42 x 64, four directions, eleven of
// 1664: 1857 / 1032, but pixel-major ten of 1920: 859 / 1929, 63 x 63, three, ten of 672:
// 589 / 775; fp32 42 x 23, four, twelve of 2304: 2026 / 683, bf16 31 x 31, four: 1980 /
// 453.
constexpr int64_t kFullWaves = 512;
constexpr int64_t kFewRounds = 4;
constexpr int kRoundSteps[3] = {16, 38, 50};

// What a call of the general family takes; planes of at most 64 have other
// fallbacks, which take less.
int64_t general_bytes(const Problem &p, bool bwd)
{
    if (p.H <= kSmallSide && p.W <= kSmallSide)
        return 0;
    return bwd ? general_bwd_bytes(p) : general_fwd_bytes(p);
}

// The plan of a problem: what is copied into rows, and the sizes of a round.
struct LinePlan {
    int K, es, D, nh, cpg, Hp, Wp, nchunk, cc;
    bool rows_v, rows_x;             // vertical lam, u, w (and x, dy) gathered into rows
    int64_t units, ru;               // units (b, g), units per round
    int64_t plane_lines, plane_copies, unit_bytes;
    int64_t bytes;                   // workspace taken
    int64_t rounds;
    bool fits;                       // a round of one group fits
    bool worth;                      // its rounds are not too many
};

LinePlan line_plan(const Problem &p, bool bwd)
{
    LinePlan q;
    const int m = p.H > p.W ? p.H : p.W;
    q.K = m <= 64 ? 1 : (m <= 128 ? 2 : 4);
    q.es = p.dtype == 0 ? 4 : 2;
    q.D = __builtin_popcount(p.mask);
    q.nh = __builtin_popcount(p.mask & 12);
    q.cpg = p.C / p.G;
    q.Hp = pad4(p.H);
    q.Wp = pad4(p.W);
    const int nv = q.D - q.nh;
    q.rows_x = nv > 0 && p.W < q.K;
    q.rows_v = nv > 0 && (p.layout != kPixelMajor || q.rows_x);
    q.units = (int64_t)p.B * p.G;
    const int64_t vsz = (int64_t)p.H * q.Wp, hsz = (int64_t)p.W * q.Hp;
    // chunks of a group's channels in the gradient launch: 1.5 workgroups a
    // CU, at least 4 channels each (128 x 128, B = 2, C = 192, G = 6: 384
    // workgroups 381 us, 768 397 us for twice the partials, 192 430 us)
    const int tiles = ((p.H + kTileR - 1) / kTileR) * ((p.W + kTileC - 1) / kTileC);
    q.nchunk = 1;
    if (bwd)
        while (q.nchunk * q.units * tiles < 384 && (q.cpg + 2 * q.nchunk - 1) / (2 * q.nchunk) >= 4)
            q.nchunk *= 2;
    q.cc = (q.cpg + q.nchunk - 1) / q.nchunk;
    q.nchunk = (q.cpg + q.cc - 1) / q.cc;
    q.plane_lines = nv * vsz + q.nh * hsz;                                 // floats of h (or a)
    const int streams = bwd ? 2 : 1;                                       // lam, or lam and u
    q.plane_copies = streams * (q.nh * hsz + (q.rows_v ? nv * vsz : 0)) +
                     streams * ((q.nh ? hsz : 0) + (q.rows_x ? vsz : 0));
    const int64_t wcopies = 3 * (q.nh * hsz + (q.rows_v ? nv * vsz : 0));
    q.unit_bytes = q.cpg * (q.plane_lines * 4 * streams + q.plane_copies * q.es) + wcopies * q.es +
                   (q.nchunk > 1 ? (int64_t)q.nchunk * q.D * 3 * p.H * p.W * 4 : 0);
    const int64_t gen = general_bytes(p, bwd), one = q.unit_bytes + kPartPad;
    int64_t most = std::max({gen, kRoundBytes, one});
    const int64_t whole = most;
    if (p.ws_cap >= 0)
        most = std::min(most, p.ws_cap - (((int64_t)p.ws->used + 255) & ~(int64_t)255));
    else if (gen > 0 && gen < kSmallBytes && (bwd || !wide_supported(p)))
        most = gen;
    q.fits = one <= most && gen <= most;
    q.ru = std::max<int64_t>(1, std::min(q.units, (most - kPartPad) / q.unit_bytes));
    // (the merge has kTileThreads a tile of every plane, the other launches up to
    // twice that a plane)
    const int64_t max_planes = kMaxThreads / (2 * kTileThreads * tiles);
    q.fits = q.fits && q.cpg <= max_planes;
    q.ru = std::max<int64_t>(1, std::min(q.ru, max_planes / q.cpg));
    // rounds follow each other on the stream
    q.rounds = (q.units + q.ru - 1) / q.ru;
    const int64_t waves = q.ru * q.cpg * q.D * (bwd ? 2 : 1);
    const int steps = std::max(nv ? p.H : 0, q.nh ? p.W : 0);
    const bool blocked = p.layout != kPixelMajor;
    const int kind = blocked ? 2 : (q.nh || q.rows_x ? 1 : 0);
    int64_t full = kFullWaves;
    if (most < whole && m <= kSmallSide && bwd)
        full *= blocked || m <= 32 || p.dtype == 0 ? 8 : q.D <= 2 ? 4 : 1;
    else if (most < whole && blocked && !bwd)
        full *= 8;
    // the general forward's load and the line family's turned planes, in tenths of a step
    const int64_t planes = (int64_t)p.B * p.C, hl = planes * q.nh * p.H, vl = planes * nv * p.W;
    const int64_t by_load = blocked ? (4 * hl + vl) / 10000 : (5 * hl + vl) / 4600;
    const int64_t load = kind == 0 ? 10 : std::max<int64_t>(10, by_load);
    const int64_t turned = blocked ? planes * p.H * p.W * q.D / 9000 : 0;
    const int64_t few = std::max<int64_t>(kFewRounds, m <= kSmallSide ? 0 : (blocked ? 2 : 3) * q.cpg);
    q.worth = q.rounds == 1 || waves >= full ||
              (bwd ? q.rounds <= few : 10 * q.rounds * kRoundSteps[kind] + turned <= steps * load);
    q.bytes = std::max(gen, q.ru * q.unit_bytes + kPartPad);
    return q;
}

template <typename S, int K>
hipError_t launch_sweeps(const SweepArgs &a, bool rag, bool bwd, hipStream_t st)
{
    const int nblk = (a.np + 3) / 4;
    const dim3 grid((unsigned)(nblk * a.nd * (bwd ? 2 : 1)));
    if (rag)
        hipLaunchKernelGGL((sweep_kernel<S, K, true>), grid, dim3(256), 0, st, a, nblk, bwd);
    else
        hipLaunchKernelGGL((sweep_kernel<S, K, false>), grid, dim3(256), 0, st, a, nblk, bwd);
    return hipGetLastError();
}

unsigned blocks_for(int64_t n)
{
    const int64_t b = (n + 255) / 256;
    return (unsigned)(b < 8192 ? b : 8192);
}

template <typename S>
hipError_t line_t(const Problem &p, bool bwd, hipStream_t st)
{
    const LinePlan q = line_plan(p, bwd);
    const int H = p.H, W = p.W;
    const int64_t HW = (int64_t)H * W, BC = (int64_t)p.B * p.C, BG = (int64_t)p.B * p.G;
    const int64_t vsz = (int64_t)H * q.Wp, hsz = (int64_t)W * q.Hp;
    const int64_t rp = q.ru * q.cpg;                    // planes of a full round
    Workspace parts;                                    // of the block taken
    hipError_t e = p.ws->take((void **)&parts.base, (size_t)q.bytes);
    if (e != hipSuccess || p.ws->counting)
        return e;
    parts.size = (size_t)q.bytes;
    auto take = [&](int64_t elems, int es) -> void * {
        void *ptr = nullptr;
        if (e == hipSuccess && elems > 0)
            e = parts.take(&ptr, (size_t)(elems * es));
        return ptr;
    };
    // fp32 lines per slot, copies (lam, u, w of the copied slots; x, dy)
    float *hb[4] = {}, *ab[4] = {};
    S *lc[4] = {}, *uc[4] = {}, *wc[4] = {};
    int dirs[4], slot = 0;
    for (int d = 0; d < 4; ++d)
        if ((p.mask >> d) & 1)
            dirs[slot++] = d;
    for (int s = 0; s < q.D; ++s) {
        const bool vert = dirs[s] < 2;
        const int64_t sz = vert ? vsz : hsz;
        hb[s] = static_cast<float *>(take(rp * sz, 4));
        if (bwd)
            ab[s] = static_cast<float *>(take(rp * sz, 4));
        if (!vert || q.rows_v) {
            lc[s] = static_cast<S *>(take(rp * sz, q.es));
            if (bwd)
                uc[s] = static_cast<S *>(take(rp * sz, q.es));
            wc[s] = static_cast<S *>(take(q.ru * 3 * sz, q.es));
        }
    }
    S *xt = q.nh ? static_cast<S *>(take(rp * hsz, q.es)) : nullptr;
    S *gt = q.nh && bwd ? static_cast<S *>(take(rp * hsz, q.es)) : nullptr;
    S *xr = q.rows_x ? static_cast<S *>(take(rp * vsz, q.es)) : nullptr;
    S *gr = q.rows_x && bwd ? static_cast<S *>(take(rp * vsz, q.es)) : nullptr;
    float *part = nullptr;
    if (bwd && q.nchunk > 1)
        part = static_cast<float *>(take((int64_t)q.nchunk * q.D * q.ru * 3 * HW, 4));
    if (e != hipSuccess)
        return e;

    const bool pm = p.layout == kPixelMajor;
    const S *x = static_cast<const S *>(p.x), *dy = static_cast<const S *>(p.dy);
    const S *lam = static_cast<const S *>(p.lam), *u = static_cast<const S *>(p.u);
    const S *w = static_cast<const S *>(p.w);
    const int tiles_c = (W + kTileC - 1) / kTileC, tiles = ((H + kTileR - 1) / kTileR) * tiles_c;
    for (int64_t u0 = 0; u0 < q.units && e == hipSuccess; u0 += q.ru) {
        const int64_t nu = std::min(q.ru, q.units - u0), pl0 = u0 * q.cpg, np = nu * q.cpg;
        // --- rows
        TurnArgs t{};
        t.H = H, t.W = W, t.pitch = q.Hp;
        t.tiles_c = (W + 63) / 64;
        t.tiles = ((q.Hp + 63) / 64) * t.tiles_c;
        int64_t nturn = 0;
        auto flush = [&]() {
            if (t.nt == 0 || e != hipSuccess)
                return;
            hipLaunchKernelGGL((transpose_kernel<S>), dim3((unsigned)(nturn * t.tiles)), dim3(256),
                               0, st, t);
            e = hipGetLastError();
            t.nt = 0;
            nturn = 0;
        };
        auto turn = [&](const S *src, S *dst, int64_t n) {
            if (t.nt == kMaxTurns || (nturn + n) * t.tiles > 0x7fffffff)
                flush();
            t.t[t.nt++] = Turn{src, dst, (int)nturn};
            nturn += n;
        };
        auto rows = [&](const S *src, S *dst, int64_t n, bool vert, bool pmaj) {
            if (e != hipSuccess)
                return;
            const int L = vert ? H : W, P = vert ? W : H, pitch = vert ? q.Wp : q.Hp;
            hipLaunchKernelGGL((rows_kernel<S>), dim3(blocks_for(n * L * pitch)), dim3(256), 0, st,
                               src, dst, n, L, P, W, pitch, (int)vert, (int)pmaj);
            e = hipGetLastError();
        };
        if (q.nh) {
            turn(x + pl0 * HW, xt, np);
            if (bwd)
                turn(dy + pl0 * HW, gt, np);
        }
        if (q.rows_x) {
            rows(x + pl0 * HW, xr, np, true, true);
            if (bwd)
                rows(dy + pl0 * HW, gr, np, true, true);
        }
        for (int s = 0; s < q.D; ++s) {
            if (lc[s] == nullptr)
                continue;
            const bool vert = dirs[s] < 2;
            const S *sl = lam + (s * BC + pl0) * HW, *su = u + (s * BC + pl0) * HW;
            const S *sw = w + (s * BG + u0) * 3 * HW;
            if (pm && !vert) {
                turn(sl, lc[s], np);
                if (bwd)
                    turn(su, uc[s], np);
                turn(sw, wc[s], 3 * nu);
            } else {
                rows(sl, lc[s], np, vert, pm);
                if (bwd)
                    rows(su, uc[s], np, vert, pm);
                rows(sw, wc[s], 3 * nu, vert, pm);
            }
        }
        flush();
        if (e != hipSuccess)
            return e;
        // --- sweeps
        SweepArgs a{};
        a.nd = q.D, a.np = (int)np, a.cpg = q.cpg;
        GradArgs g{};
        bool rag = false;
        for (int s = 0; s < q.D; ++s) {
            const bool vert = dirs[s] < 2;
            LineDir &d = a.dir[s];
            d.L = vert ? H : W;
            d.P = vert ? W : H;
            d.op = vert ? q.Wp : q.Hp;
            d.osz = vert ? vsz : hsz;
            d.rev = dirs[s] & 1;
            const bool copied = lc[s] != nullptr;
            d.lam = copied ? lc[s] : lam + (s * BC + pl0) * HW;
            d.u = copied ? uc[s] : u + (s * BC + pl0) * HW;
            d.w = copied ? wc[s] : w + (s * BG + u0) * 3 * HW;
            d.lp = copied ? d.op : W;
            d.lsz = copied ? d.osz : HW;
            d.x = vert ? (q.rows_x ? xr : x + pl0 * HW) : xt;
            d.dy = vert ? (q.rows_x ? gr : dy + pl0 * HW) : gt;
            d.xp = vert && !q.rows_x ? W : d.op;
            d.xsz = vert && !q.rows_x ? HW : d.osz;
            d.h = hb[s];
            d.a = ab[s];
            g.h[s] = hb[s], g.a[s] = ab[s], g.dirs[s] = dirs[s];
            rag = rag || (d.P >= q.K && d.P % q.K != 0);
        }
        e = q.K == 1 ? launch_sweeps<S, 1>(a, false, bwd, st)
                     : (q.K == 2 ? launch_sweeps<S, 2>(a, rag, bwd, st)
                                 : launch_sweeps<S, 4>(a, rag, bwd, st));
        if (e != hipSuccess)
            return e;
        // --- gradients, or the merge
        g.x = x + pl0 * HW;
        g.lam = lam + pl0 * HW;
        g.u = u + pl0 * HW;
        g.opv = q.Wp, g.oph = q.Hp;
        g.nd = q.D, g.mask = p.mask, g.H = H, g.W = W, g.cpg = q.cpg, g.cc = q.cc;
        g.per_slot = BC * HW;
        g.w_slot = BG * 3 * HW;
        g.nu = (int)nu, g.nchunk = q.nchunk, g.tiles_c = tiles_c, g.tiles = tiles, g.pm = pm;
        if (!bwd) {
            g.y = static_cast<S *>(p.y) + pl0 * HW;
            const dim3 mgrid((unsigned)(np * tiles));
            if (pm)
                hipLaunchKernelGGL((merge_kernel<S, true>), mgrid, dim3(kTileThreads), 0, st, g);
            else
                hipLaunchKernelGGL((merge_kernel<S, false>), mgrid, dim3(kTileThreads), 0, st, g);
            e = hipGetLastError();
            continue;
        }
        g.dy = dy + pl0 * HW;
        g.dx = static_cast<S *>(p.dx) + pl0 * HW;
        g.dlam = static_cast<S *>(p.dlam) + pl0 * HW;
        g.du = static_cast<S *>(p.du) + pl0 * HW;
        g.dw = static_cast<S *>(p.dw) + u0 * 3 * HW;
        g.part = part;
        const dim3 ggrid((unsigned)(nu * q.nchunk * tiles));
        if (pm)
            hipLaunchKernelGGL((grad_kernel<S, true>), ggrid, dim3(kTileThreads), 0, st, g);
        else
            hipLaunchKernelGGL((grad_kernel<S, false>), ggrid, dim3(kTileThreads), 0, st, g);
        e = hipGetLastError();
        if (e == hipSuccess && q.nchunk > 1) {
            const int64_t per = nu * 3 * HW;
            hipLaunchKernelGGL((dw_parts_kernel<S>), dim3(blocks_for(per * q.D)), dim3(256), 0, st,
                               (const float *)part, static_cast<S *>(g.dw), per, q.D, q.nchunk,
                               g.w_slot);
            e = hipGetLastError();
        }
    }
    return e;
}

}  // namespace

// Blocked forwards that the general family does faster: its time is its steps, while
// the line family's launches turn every plane into rows first, and of few channels a
// group the taps as well (us, line / general):
//  * up to 16 steps always: 12 x 118, T2B and B2T, B*C = 64: 17 / 11; 16 x 68, 19: 18 / 14;
//  * both vertical directions: one or two channels a group until 44 steps, with few
//    planes 34 (19 x 158, 995: 85 / 48; 40 x 122, 928: 126 / 79; 44 x 134, 124: 42 / 39, but
//    44 x 90, 40: 25 / 31), more until 24 (20 x 132, 16 a group, 16: 20 / 18; 31 x 142, 4 a
//    group, 48: 24 / 24);
//  * one vertical direction, of one or two channels a group until 22 (22 x 121, 2 a
//    group, 1676: 51 / 45; 24 x 77, 24: 16 / 19; 4 a group, 20 x 183, 560: 31 / 32), of one
//    and 250 planes until 34 (27 x 158, 1120: 70 / 51; 34 x 73, 864: 50 / 48; 43 x 76, 736:
//    48 / 55);
//  * horizontal ones, whose lines of few positions the general family reads by lanes,
//    only up to 350 planes: both until 24 steps, 36 of one or two channels a group and
//    50 planes (169 x 23, 224: 45 / 30; 172 x 33, 100: 40 / 33; 126 x 33, 8: 25 / 33; 172 x
//    30, 704: 108 / 188); one until 19 (102 x 17, 862: 39 / 29, but 82 x 27, fp32, 2592: 128
//    / 265).
static bool few_steps(const Problem &p)
{
    const bool vert = (p.mask & 12) == 0, horiz = (p.mask & 3) == 0;
    const int steps = std::max((p.mask & 3) ? p.H : 0, (p.mask & 12) ? p.W : 0);
    if (steps <= 16)
        return true;
    if ((p.H > p.W ? p.H : p.W) <= kSmallSide || !(vert || horiz))
        return false;
    const bool two = (p.mask & (p.mask - 1)) != 0;
    const int64_t planes = (int64_t)p.B * p.C, cpg = p.C / p.G;
    if (vert)
        return two ? steps <= (cpg > 2 ? 24 : planes >= 50 ? 44 : 34)
                   : cpg <= 2 && steps <= (cpg == 1 && planes >= 250 ? 34 : 22);
    return two ? planes <= 350 && steps <= (cpg <= 2 && planes >= 50 ? 36 : 24)
               : planes <= 900 && cpg <= 2 && steps <= 19;
}

bool line_supported(const Problem &p, bool bwd)
{
    if (!bwd && p.layout != kPixelMajor && few_steps(p))
        return false;
    if ((p.H > p.W ? p.H : p.W) > kLineSide)
        return false;
    const LinePlan q = line_plan(p, bwd);
    return q.fits && q.worth;
}

// Whether the workspace holds a round of it at all.
bool line_fits(const Problem &p, bool bwd)
{
    return (p.H > p.W ? p.H : p.W) <= kLineSide && line_plan(p, bwd).fits;
}

// Pixel-major shapes that the wide family takes too (bf16, sides multiples of
// 8): with lines of at most 128 positions, or few planes, a wave per direction
// and plane beats a workgroup per plane (us, wide / line): 128 x 128, B*C =
// 384: 121 / 91, 2048: 583 / 481; 72 x 72, 2048: 295 / 213; 256 x 256, 8: 96 /
// 66, 64: 119 / 83; but 256: 240 / 251, 1024: 958 / 1024; 160 x 160, 1024: 407
// / 491 (4 positions a lane move more bytes than the wide family's rounds).  In a
// workspace that holds the wide family's only in one round: 160 x 184 T2B, B*C = 160,
// two: 49 / 80; 104 x 104, T2B and B2T, 96, two: 36 / 45.
bool line_fwd_preferred(const Problem &p)
{
    return p.layout == kPixelMajor && (p.ws_cap < 0 || line_plan(p, false).rounds == 1) &&
           ((p.H <= 128 && p.W <= 128) ||
            (int64_t)__builtin_popcount(p.mask) * p.B * p.C <= 512);
}

hipError_t launch_fwd_line(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? line_t<float>(p, false, st) : line_t<bf16_t>(p, false, st);
}

hipError_t launch_bwd_line(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? line_t<float>(p, true, st) : line_t<bf16_t>(p, true, st);
}

}  // namespace gspn
