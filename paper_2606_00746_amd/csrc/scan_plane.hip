// Line scans of planes with both sides at most 64, of any size, type and
// layout, with everything a workgroup's channels need in LDS.
//
// A workgroup takes up to 8 waves of channels of one weight group, T = 16, 32
// or 64 lanes a channel (lane j of them line position j), and runs the
// directions one after another.  In LDS are, per channel, one record per
// pixel -- x and dy, u and lam of the current direction (replaced by du and
// dlam as its sweep passes), the fp32 sum of dx or y -- and, once for the
// workgroup, the direction's taps in scan order with those that the scan
// ignores set to 0 and a line of zeros behind the last.  A record is an odd
// number of dwords and rows have an odd pitch, so row and column walks are
// free of bank conflicts and one address serves a step's whole record.
// Planes come and go as the dwords of the channels' contiguous stretch of
// memory, whatever its alignment (a lane's dword holds two bf16 records: six
// LDS dwords from lane to lane keep the copies' conflicts at two lanes a
// bank, where 16-byte pieces made it eight); the next direction's are loaded
// into registers while the current one runs.
//
// Idle lanes (no position, no channel) read records of zeros and the line of
// zero taps, and write nothing.
//
// Backward: a reverse sweep keeps the adjoint a_i in registers, a forward
// sweep recomputes h_i and forms every gradient; a_i and h_{i-1} of a batch
// of KB steps go to LDS slots, and after the batch's barrier each step's
// weight gradient is summed over the channels by one line of lanes.  A group
// of more channels than fit has its chunks' fp32 sums added by a second
// kernel in chunk order.
//
// Four directions, bf16, forward / backward in us, against the kernels that
// read every step's values from memory (scan_small.hip): 28 x 28, B = 64,
// C = 192, G = 16: 217 / 1196 -> 109 / 245; 37 x 37, B = 16, C = 384, G = 12:
// 392 / 1500 -> 93 / 238; 7 x 7, B = 32, C = 768, G = 24: 70 / 90 -> 26 / 60.
// LDS holds 6 to 8 waves a CU; at 37 x 37 the backward's time is about half
// issuing (20 vector instructions a step and sweep), a quarter the slots'
// sums and their barriers (without them 202 us), the rest the copies (about
// 25 us each way).  Measured on the way there (37 x 37 backward): copies in
// 16-byte pieces, eight lanes to a bank, 322 us, in dwords 296; double-buffered
// slots of 2 steps 296, one buffer of 4 steps and two barriers 265; addresses
// by multiply-adds on scalars instead of selects 238.
#include <algorithm>
#include <type_traits>

#include "cdna.hpp"
#include "device.hpp"
#include "launch.hpp"
#include "plane_lds.hpp"

namespace gspn {

namespace {

using namespace cdna;

struct PlaneArgs {
    const void *x, *w, *lam, *u, *dy;
    void *out, *dw, *dlam, *du;     // out: y or dx
    float *dwp;                     // [chunk][slot][b][g][3][HW] partials, or null
    int mask, B, C, G, H, W;
    int cw, nchunk, pm;             // channels per workgroup, chunks per group
    int Wp, RS;                     // record pitch of a row, dwords of a plane's records
    uint32_t mW;                    // ceil(2^32 / W) for even W, 0 for odd
    uint32_t mD;                    // ceil(2^32 / W), 0 for W = 1
    int o_w, o_sink, o_rec;         // dword offsets in LDS (the slots are at 0)
    Magic divChunk, divG;
};

// n contiguous elements from p on, as the dwords that cover them: sh elements
// of the first dword lie before p.  The descriptor ends with the dword of the
// last element; base addresses are multiples of 16, so no dword reaches
// outside the memory of the tensor's own dwords.
template <typename S>
struct Stretch {
    uint64_t base;
    int sh, n;
    __device__ __forceinline__ Stretch(const S *p, int count)
    {
        const uint64_t a = reinterpret_cast<uint64_t>(p);
        base = a & ~3ull;
        sh = (int)(a & 3) / (int)sizeof(S);
        n = count;
    }
    __device__ __forceinline__ int units() const
    {
        return n > 0 ? (sh + n + Rec<S>::E - 1) / Rec<S>::E : 0;
    }
    __device__ __forceinline__ rsrc_t rsrc() const
    {
        return make_rsrc(reinterpret_cast<const void *>(base), 4u * (uint32_t)units());
    }
    __device__ __forceinline__ u32x4 sdesc() const
    {
        return make_sdesc(reinterpret_cast<const void *>(base), 4u * (uint32_t)units());
    }
};

template <int T>
__device__ __forceinline__ float add_left(float acc, float v, float w)
{
    if constexpr (T == 16)
        return fmaf(w, from_left<16>(v), acc);
    else
        return fmac_left(acc, v, w);
}
template <int T>
__device__ __forceinline__ float add_right(float acc, float v, float w)
{
    if constexpr (T == 16)
        return fmaf(w, from_right<16>(v), acc);
    else
        return fmac_right(acc, v, w);
}

// One step's inputs as they are in LDS.
template <typename S>
struct In {
    uint32_t r[Rec<S>::N], w[Rec<S>::WN];
    __device__ __forceinline__ float x() const
    {
        if constexpr (sizeof(S) == 4)
            return __uint_as_float(r[0]);
        else
            return bf_lo(r[0]);
    }
    __device__ __forceinline__ float dy() const
    {
        if constexpr (sizeof(S) == 4)
            return __uint_as_float(r[1]);
        else
            return bf_hi(r[0]);
    }
    __device__ __forceinline__ float u() const
    {
        if constexpr (sizeof(S) == 4)
            return __uint_as_float(r[2]);
        else
            return bf_lo(r[1]);
    }
    __device__ __forceinline__ float lam() const
    {
        if constexpr (sizeof(S) == 4)
            return __uint_as_float(r[3]);
        else
            return bf_hi(r[1]);
    }
    __device__ __forceinline__ float sum() const { return __uint_as_float(r[Rec<S>::N - 1]); }
    __device__ __forceinline__ float tap(int k) const
    {
        if constexpr (sizeof(S) == 4)
            return __uint_as_float(w[k]);
        else
            return k == 0 ? bf_lo(w[0]) : (k == 1 ? bf_hi(w[0]) : bf_lo(w[1]));
    }
};

// LDS by byte address: the sweeps' addresses are kept as integers.
typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
__device__ __forceinline__ int lds_addr(const void *p)
{
    return (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ lds_u32_t *lds_ptr(int a)
{
    return (lds_u32_t *)(uintptr_t)(uint32_t)a;
}

constexpr int kUnits = 13;     // dwords of u and of lam per lane loaded a direction ahead
constexpr int kTaps = 3;       // pixels' taps per thread loaded a direction ahead

template <int NB, typename S, bool BWD, int KB>
__global__ __launch_bounds__(512, NB == 1 ? 4 : 2) void plane_kernel(const PlaneArgs A)
{
    using R = Rec<S>;
    constexpr int T = NB <= 2 ? 16 : (NB <= 4 ? 32 : 64);   // lanes of a channel
    constexpr int TS = 8 * NB;                              // steps unrolled
    constexpr int NL = 64 / T, N = R::N, WN = R::WN, E = R::E;
    extern __shared__ uint4 smem4[];
    uint32_t *lds = reinterpret_cast<uint32_t *>(smem4);
    const int lds0 = lds_addr(smem4);                // its LDS byte address

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwaves = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const int lane = threadIdx.x & 63, cl = lane / T, j = lane % T;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int bg = mdiv(blk, A.divChunk), chunk = blk - bg * A.nchunk;
    const int b = mdiv(bg, A.divG), g = bg - b * A.G;
    const int H = A.H, W = A.W, HW = H * W;
    const int cpg = mdiv(A.C, A.divG);
    const int cfirst = chunk * A.cw, nvalid = min(A.cw, cpg - cfirst);
    const int q0 = wave * NL, q = q0 + cl;               // channel slots of this wave, this lane
    const int nmine = max(0, min(NL, nvalid - q0));      // channels of this wave
    const int64_t pl0 = (int64_t)b * A.C + g * cpg + cfirst + (nmine > 0 ? q0 : 0);
    const int n = nmine * HW;                            // elements of this wave's stretch
    const int rec0 = plane_wave_rec0(A.o_rec, wave, NL, A.RS, N);   // this wave's records
    const bool pm = A.pm != 0;

    // the records of zeros, the line of zero taps, the slots of absent channels
    for (int t = threadIdx.x; t < 64 * N; t += blockDim.x)
        lds[A.o_sink + t] = 0u;
    for (int t = threadIdx.x; t < max(H, W) * WN; t += blockDim.x)
        lds[A.o_w + HW * WN + t] = 0u;
    const int nq = nwaves * NL, nqs = (nq + 3) & ~3;     // channel slots, rounded up
    if (BWD) {
        for (int t = threadIdx.x; t < KB * nqs * T * 2; t += blockDim.x)
            lds[t] = 0u;
        lds_barrier();
    }

    // lane and thread index as values made opaque once per direction: what the
    // copies derive from them is formed there instead of being kept in
    // registers over all directions
    int ln = lane, tid = (int)threadIdx.x;
    // the record of pixel e of the wave's stretch
    auto rec_of = [&](int e) { return rec0 + plane_rec(e, A.mW, N); };
    // ... and of element e of a blocked plane's stretch
    auto rec_of_blocked = [&](int e, bool vert, int L, int P) {
        int c = 0;
#pragma unroll
        for (int k = 1; k < NL; ++k)
            c += e >= k * HW ? 1 : 0;
        e -= c * HW;
        const int qb = e / (8 * P), rem = e - 8 * P * qb, nl = min(8, L - 8 * qb);
        const int p = rem / nl, l = 8 * qb + rem - p * nl;
        return rec0 + c * A.RS + N * (vert ? l * A.Wp + p : p * A.Wp + l);
    };
    // dwords k of this lane of two planes into the records (a pixel before or
    // behind the stretch goes to a spare record)
    auto put = [&](const Stretch<S> &s, int k, uint32_t va, uint32_t vb, bool xdy) {
        const int e0 = E * ln - s.sh;                // its first dword's first pixel
        auto write = [&](uint32_t *r) {
            if constexpr (sizeof(S) == 4) {
                r[xdy ? 0 : 2] = va;
                r[xdy ? 1 : 3] = vb;
                if (xdy)
                    r[N - 1] = 0u;
            } else {
                r[xdy ? 0 : 1] = __builtin_amdgcn_perm(vb, va, 0x05040100u);
                r[N + (xdy ? 0 : 1)] = __builtin_amdgcn_perm(vb, va, 0x07060302u);
                if (xdy)
                    r[N - 1] = r[2 * N - 1] = 0u;
            }
        };
        const int nu = s.units();
        if (64 * (k + 1) <= nu || ln + 64 * k < nu)
            write(A.mW == 0 ? lds + rec0 + N * e0 + N * E * 64 * k : lds + rec_of(e0 + E * 64 * k));
    };
    // two planes of the stretch, from dword k0 of a lane on
    auto copy = [&](const Stretch<S> &s, rsrc_t ra, rsrc_t rb, int k0, bool xdy) {
        const int nu = s.units();
        for (int k = k0; 64 * k < nu; k += 8) {
            uint32_t a[8], c[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                a[m] = ld32(ra, 4u * (uint32_t)(ln + 64 * (k + m)), 0);
                c[m] = xdy && !BWD ? 0u : ld32(rb, 4u * (uint32_t)(ln + 64 * (k + m)), 0);
            }
#pragma unroll
            for (int m = 0; m < 8; ++m)
                put(s, k + m, a[m], c[m], xdy);
        }
    };

    {
        const Stretch<S> sx(static_cast<const S *>(A.x) + pl0 * HW, n);
        const rsrc_t rx = sx.rsrc();
        copy(sx, rx, BWD ? Stretch<S>(static_cast<const S *>(A.dy) + pl0 * HW, n).rsrc() : rx, 0, true);
    }

    // u, lam and the taps of a direction: what is loaded ahead
    uint32_t pu[kUnits], pl[kUnits];
    uint32_t pw[kTaps][3];
    auto slot_of = [&](int d) { return __popc(A.mask & ((1 << d) - 1)); };
    auto lam_at = [&](int d) { return ((int64_t)slot_of(d) * A.B * A.C + pl0) * HW; };
    auto w_at = [&](int d) { return (((int64_t)slot_of(d) * A.B + b) * A.G + g) * 3 * HW; };
    auto ld_el = [](rsrc_t r, int e) {
        if constexpr (sizeof(S) == 4)
            return ld32(r, 4u * (uint32_t)e, 0);
        else
            return ld16(r, 2u * (uint32_t)e, 0);
    };
    auto ahead = [&](int d) {
        if (pm) {
            const rsrc_t ru = Stretch<S>(static_cast<const S *>(A.u) + lam_at(d), n).rsrc();
            const rsrc_t rl = Stretch<S>(static_cast<const S *>(A.lam) + lam_at(d), n).rsrc();
#pragma unroll
            for (int k = 0; k < kUnits; ++k) {
                pu[k] = ld32(ru, 4u * (uint32_t)(ln + 64 * k), 0);
                pl[k] = ld32(rl, 4u * (uint32_t)(ln + 64 * k), 0);
            }
        }
        const rsrc_t rw = make_rsrc(static_cast<const S *>(A.w) + w_at(d),
                                    3u * (uint32_t)HW * (uint32_t)sizeof(S));
#pragma unroll
        for (int m = 0; m < kTaps; ++m)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int e = tid + m * (int)blockDim.x;
                pw[m][k] = ld_el(rw, e < HW ? e + k * HW : 3 * HW);
            }
    };
    // taps of pixel (blocked: element) e into scan order
    auto put_taps = [&](int d, int e, const uint32_t (&t)[3]) {
        const bool vert = d < 2, rev = d & 1;
        const int L = vert ? H : W, P = vert ? W : H;
        int l, p;
        if (pm) {
            const int r = W > 1 ? (int)__umulhi((uint32_t)e, A.mD) : e, c = e - r * W;
            l = vert ? r : c, p = vert ? c : r;
        } else {
            const int qb = e / (8 * P), rem = e - 8 * P * qb, nl = min(8, L - 8 * qb);
            p = rem / nl;
            l = 8 * qb + rem - p * nl;
        }
        const int i = rev ? L - 1 - l : l;
        uint32_t *o = lds + A.o_w + WN * (i * P + p);
        const uint32_t t0 = i > 0 && p > 0 ? t[0] : 0u, t1 = i > 0 ? t[1] : 0u,
                       t2 = i > 0 && p + 1 < P ? t[2] : 0u;
        if constexpr (sizeof(S) == 4) {
            o[0] = t0, o[1] = t1, o[2] = t2;
        } else {
            o[0] = t0 | (t1 << 16), o[1] = t2;
        }
    };
    // a direction's u, lam and taps into LDS: what was loaded ahead, then the rest
    auto stage = [&](int d) {
        if (pm) {
            const Stretch<S> su(static_cast<const S *>(A.u) + lam_at(d), n);
            const int nu = su.units();
#pragma unroll
            for (int k = 0; k < kUnits; ++k)
                if (64 * k < nu)
                    put(su, k, pu[k], pl[k], false);
            if (64 * kUnits < nu)
                copy(su, su.rsrc(), Stretch<S>(static_cast<const S *>(A.lam) + lam_at(d), n).rsrc(),
                     kUnits, false);
        } else {
            const rsrc_t ru = make_rsrc(static_cast<const S *>(A.u) + lam_at(d), n * (uint32_t)sizeof(S));
            const rsrc_t rl = make_rsrc(static_cast<const S *>(A.lam) + lam_at(d), n * (uint32_t)sizeof(S));
            const int L = d < 2 ? H : W, P = d < 2 ? W : H;
            for (int e = ln; e < n; e += 64) {
                uint32_t *r = lds + rec_of_blocked(e, d < 2, L, P);
                const uint32_t a = ld_el(ru, e), c = ld_el(rl, e);
                if constexpr (sizeof(S) == 4)
                    r[2] = a, r[3] = c;
                else
                    r[1] = a | (c << 16);
            }
        }
#pragma unroll
        for (int m = 0; m < kTaps; ++m) {
            const int e = tid + m * (int)blockDim.x;
            if (e < HW)
                put_taps(d, e, pw[m]);
        }
        if (kTaps * (int)blockDim.x < HW) {
            const rsrc_t rw = make_rsrc(static_cast<const S *>(A.w) + w_at(d),
                                        3u * (uint32_t)HW * (uint32_t)sizeof(S));
            for (int e = tid + kTaps * (int)blockDim.x; e < HW; e += blockDim.x) {
                const uint32_t t[3] = {ld_el(rw, e), ld_el(rw, e + HW), ld_el(rw, e + 2 * HW)};
                put_taps(d, e, t);
            }
        }
    };
    // this wave's du and dlam (or, with `last`, its sums) out of the records
    auto flush = [&](const Stretch<S> &s, const u32x4 &ra, const u32x4 &rb, bool last) {
        const int nu = s.units();
        constexpr int M = 4;                         // dwords whose records are read together
        for (int k0 = 0; 64 * k0 < nu; k0 += M) {
            uint32_t va[M], vb[M];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const uint32_t *r = lds + rec_of(plane_flush_pixel(E * (ln + 64 * (k0 + m)) - s.sh, s.n));
                if constexpr (sizeof(S) == 4) {
                    va[m] = last ? r[N - 1] : r[2];
                    vb[m] = last ? 0u : r[3];
                } else if (last) {
                    va[m] = pack2(__uint_as_float(r[N - 1]), __uint_as_float(r[2 * N - 1]));
                    vb[m] = 0u;
                } else {
                    const uint32_t lo = r[1], hi = r[N + 1];
                    va[m] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
                    vb[m] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
                }
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int un = ln + 64 * (k0 + m), e0 = E * un - s.sh;
                const uint32_t o = 4u * (uint32_t)un;
                if constexpr (sizeof(S) == 4) {
                    st32(ra, o, 0, va[m]);           // (dropped by the descriptor's end)
                    if (!last)
                        st32(rb, o, 0, vb[m]);
                } else if (e0 >= 0 && e0 + 1 < s.n) {
                    st32(ra, o, 0, va[m]);
                    if (!last)
                        st32(rb, o, 0, vb[m]);
                } else if (un < nu) {
                    // one of the dword's two elements is the stretch's
                    const uint32_t hi = e0 < 0 ? 16u : 0u;
                    st16(ra, o + hi / 8, 0, va[m] >> hi);
                    if (!last)
                        st16(rb, o + hi / 8, 0, vb[m] >> hi);
                }
            }
        }
    };

    int d = __ffs(A.mask) - 1;
    ahead(d);
#pragma nounroll
    while (d < 4) {
        asm volatile("" : "+v"(ln), "+v"(tid));
        stage(d);
        lds_barrier();                               // the taps are in place
        int dn = d + 1;                              // the next direction
        while (dn < 4 && !((A.mask >> dn) & 1))
            ++dn;

        const bool vert = d < 2, rev = d & 1;
        const int L = vert ? H : W, P = vert ? W : H;
        const bool act = cl < nmine && j < P;
        const int sl = 4 * N * (vert ? A.Wp : 1), sp = 4 * N * (vert ? 1 : A.Wp);
        // byte addresses of step 0's record and taps, and bytes to the next
        // step's (idle lanes stay where they are)
        const int rb = lds0 + (act ? 4 * (rec0 + cl * A.RS) + j * sp + (rev ? (L - 1) * sl : 0)
                                   : 4 * (A.o_sink + N * lane));
        const int rs = act ? (rev ? -sl : sl) : 0;
        const int wb = lds0 + 4 * (A.o_w + (act ? WN * j : WN * HW));
        const int Ls = __builtin_amdgcn_readfirstlane(L);
        const int ws = act ? 4 * WN * P : 0;
        // base + v for steps below m: one multiply-add with the scalar sign of
        // i - m, where a select would take two instructions
        auto step_if = [](int i, int m, int v, int base) {
            const int f = (int)((uint32_t)(i - m) >> 31);
            int r;
            asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "s"(f), "v"(v), "v"(base));
            return r;
        };
        auto read = [&](In<S> &in, int ra, int wa) {
            const lds_u32_t *r = lds_ptr(ra), *w = lds_ptr(wa);
#pragma unroll
            for (int k = 0; k < N; ++k)
                in.r[k] = r[k];
#pragma unroll
            for (int k = 0; k < WN; ++k)
                in.w[k] = w[k];
        };

        float ahist[BWD ? TS : 1];
        if constexpr (BWD) {
            // a_i[j] = u dy + w1 a[j] + (w0 a)[j+1] + (w2 a)[j-1], taps of step
            // i+1.  Reads run a block of RB steps ahead; those of steps past the
            // line's end repeat its last step and are not used.
            constexpr int RB = 4;
            In<S> in[TS];
            float an = 0.f;
            int ra = rb + (L - 1) * rs, wa = wb + L * ws;
            auto block = [&](int bk) {
#pragma unroll
                for (int t = RB - 1; t >= 0; --t) {
                    const int i = RB * bk + t;
                    read(in[i], ra, wa);
                    ra = step_if(i, Ls, -rs, ra);
                    wa = step_if(i, Ls, -ws, wa);
                }
            };
            block(TS / RB - 1);
#pragma unroll
            for (int bk = TS / RB - 1; bk >= 0; --bk) {
                if (bk > 0)
                    block(bk > 0 ? bk - 1 : 0);
#pragma unroll
                for (int t = RB - 1; t >= 0; --t) {
                    const int i = RB * bk + t;
                    if (i < L) {
                        float a = in[i].u() * in[i].dy();
                        const float q0v = in[i].tap(0) * an, q2v = in[i].tap(2) * an;
                        a = fmaf(in[i].tap(1), an, a);
                        a += from_right<T>(q0v);
                        a += from_left<T>(q2v);
                        // (a zero tap times an infinite adjoint is a NaN: it
                        // stays out of the idle lanes, which hand it back)
                        a = act ? a : 0.f;
                        ahist[i] = a;
                        an = a;
                    }
                }
                step_fence();
            }
        }
        asm volatile("" : "+v"(ln), "+v"(tid));
        if (dn < 4)
            ahead(dn);

        // h_i, the gradients (or u h), the weight gradient's terms
        {
            In<S> in[TS];
            int adr[TS];
            float h = 0.f;
            float *slots = reinterpret_cast<float *>(lds);
            const int64_t unit = ((int64_t)slot_of(d) * A.B + b) * A.G + g;
            int ra = rb, wa = wb;
            auto block = [&](int bk) {
#pragma unroll
                for (int t = 0; t < KB; ++t) {
                    const int i = KB * bk + t;
                    read(in[i], ra, wa);
                    adr[i] = ra;
                    ra = step_if(i + 1, Ls, rs, ra);
                    wa = step_if(i + 1, Ls, ws, wa);
                }
            };
            block(0);
            const int64_t per = (int64_t)__popc(A.mask) * A.B * A.G;
            const u32x4 rdw =
                !BWD ? u32x4{}
                     : A.nchunk == 1 ? make_sdesc(static_cast<S *>(A.dw) + unit * 3 * HW,
                                                  3u * (uint32_t)HW * (uint32_t)sizeof(S))
                                     : make_sdesc(A.dwp + (chunk * per + unit) * 3 * HW,
                                                  12u * (uint32_t)HW);
#pragma unroll
            for (int bk = 0; bk < TS / KB; ++bk) {
                if (KB * bk >= L)
                    break;
                if (bk + 1 < TS / KB)
                    block(bk + 1 < TS / KB ? bk + 1 : 0);
#pragma unroll
                for (int t = 0; t < KB; ++t) {
                    const int i = KB * bk + t;
                    if (i < L) {
                        const float hp = h, xv = in[i].x(), lv = in[i].lam();
                        h = lv * xv;
                        h = fmaf(in[i].tap(1), hp, h);
                        h = add_left<T>(h, hp, in[i].tap(0));
                        h = add_right<T>(h, hp, in[i].tap(2));
                        lds_u32_t *r = lds_ptr(adr[i]);
                        if constexpr (BWD) {
                            const float a = ahist[i];
                            const float duv = in[i].dy() * h, dlv = a * xv;
                            const uint32_t sum = __float_as_uint(fmaf(a, lv, in[i].sum()));
                            slots[2 * ((t * nqs + q) * T + j)] = a;
                            slots[2 * ((t * nqs + q) * T + j) + 1] = hp;
                            if (act) {
                                if constexpr (sizeof(S) == 4) {
                                    r[2] = __float_as_uint(duv);
                                    r[3] = __float_as_uint(dlv);
                                } else {
                                    r[1] = pack2(duv, dlv);
                                }
                                r[N - 1] = sum;
                            }
                        } else {
                            if (act)
                                r[N - 1] = __float_as_uint(add_nc(in[i].sum(), mul_nc(in[i].u(), h)));
                        }
                    }
                }
                if constexpr (BWD) {
                    lds_barrier();
                    // the batch's weight gradients, a line of lanes for each step
                    for (int st = q; st - cl < KB; st += nq) {
                        const int i = KB * bk + st;
                        float d0 = 0.f, d1 = 0.f, d2 = 0.f;
                        const float *v = slots + 2 * (min(st, KB - 1) * nqs * T + j);
                        // (the pairs of several channels are loaded together)
                        constexpr int kMost = T == 32 ? 16 : 8;
                        for (int c0 = 0; c0 < nqs; c0 += kMost) {
                            float va[kMost], vh[kMost];
#pragma unroll
                            for (int c = 0; c < kMost; c += 4)
                                if (c0 + c < nqs) {
#pragma unroll
                                    for (int k = c; k < c + 4; ++k) {
                                        va[k] = v[2 * (c0 + k) * T];
                                        vh[k] = v[2 * (c0 + k) * T + 1];
                                    }
                                }
#pragma unroll
                            for (int c = 0; c < kMost; c += 4)
                                if (c0 + c < nqs) {
#pragma unroll
                                    for (int k = c; k < c + 4; ++k) {
                                        d0 = add_left<T>(d0, vh[k], va[k]);
                                        d1 = fmaf(va[k], vh[k], d1);
                                        d2 = add_right<T>(d2, vh[k], va[k]);
                                    }
                                }
                        }
                        // ignored taps get 0, whatever the lanes beside hold
                        const bool live = st < KB && i < L && j < P;
                        d0 = i > 0 && j > 0 ? d0 : 0.f;
                        d1 = i > 0 ? d1 : 0.f;
                        d2 = i > 0 && j + 1 < P ? d2 : 0.f;
                        const int l = rev ? L - 1 - i : i;
                        const int o = pm ? (vert ? l * W + j : j * W + l) : lm_offset(l, j, L, P);
                        if (A.nchunk == 1) {
                            const uint32_t ob = live ? (uint32_t)o * (uint32_t)sizeof(S) : 0x80000000u;
                            const uint32_t pb = (uint32_t)HW * (uint32_t)sizeof(S);
                            if constexpr (sizeof(S) == 4) {
                                st32(rdw, ob, 0, __float_as_uint(d0));
                                st32(rdw, ob, pb, __float_as_uint(d1));
                                st32(rdw, ob, 2 * pb, __float_as_uint(d2));
                            } else {
                                st16(rdw, ob, 0, pack1(d0));
                                st16(rdw, ob, pb, pack1(d1));
                                st16(rdw, ob, 2 * pb, pack1(d2));
                            }
                        } else {
                            const uint32_t ob = live ? 4u * (uint32_t)o : 0x80000000u;
                            const uint32_t pb = 4u * (uint32_t)HW;
                            st32(rdw, ob, 0, __float_as_uint(d0));
                            st32(rdw, ob, pb, __float_as_uint(d1));
                            st32(rdw, ob, 2 * pb, __float_as_uint(d2));
                        }
                    }
                    lds_barrier();               // the slots are free again
                } else {
                    step_fence();
                }
            }
        }
        if constexpr (BWD) {
            if (pm) {
                const Stretch<S> s(static_cast<S *>(A.du) + lam_at(d), n);
                flush(s, s.sdesc(),
                      Stretch<S>(static_cast<S *>(A.dlam) + lam_at(d), n).sdesc(), false);
            } else {
                S *du = static_cast<S *>(A.du) + lam_at(d), *dl = static_cast<S *>(A.dlam) + lam_at(d);
                for (int e = ln; e < n; e += 64) {
                    const uint32_t *r = lds + rec_of_blocked(e, vert, L, P);
                    if constexpr (sizeof(S) == 4) {
                        du[e] = __uint_as_float(r[2]);
                        dl[e] = __uint_as_float(r[3]);
                    } else {
                        du[e] = (bf16_t)r[1];
                        dl[e] = (bf16_t)(r[1] >> 16);
                    }
                }
            }
        } else {
            lds_barrier();                           // every wave is done with the taps
        }
        d = dn;
    }
    {
        const Stretch<S> s(static_cast<S *>(A.out) + pl0 * HW, n);
        const u32x4 ro = s.sdesc();
        flush(s, ro, ro, true);
    }
}

// dw = sum over chunks of the fp32 partials, in chunk order.
template <typename S>
__global__ __launch_bounds__(256) void plane_dw_kernel(const float *__restrict__ dwp,
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

PlanePlan plane_plan_of(const Problem &p, bool bwd)
{
    return plane_plan(p.H, p.W, p.C / p.G, p.dtype == 0, bwd);
}

template <int NB, typename S, bool BWD, int KB>
hipError_t plane_launch(const Problem &p, const PlanePlan &q, float *dwp, hipStream_t st)
{
    PlaneArgs a{};
    a.x = p.x, a.w = p.w, a.lam = p.lam, a.u = p.u, a.dy = p.dy;
    a.out = BWD ? p.dx : p.y;
    a.dw = p.dw, a.dlam = p.dlam, a.du = p.du;
    a.dwp = dwp;
    a.mask = p.mask, a.B = p.B, a.C = p.C, a.G = p.G, a.H = p.H, a.W = p.W;
    a.cw = q.cw, a.nchunk = q.nchunk, a.pm = p.layout == kPixelMajor;
    a.Wp = q.Wp, a.RS = q.RS;
    a.mW = q.mW;
    a.mD = p.W > 1 ? (uint32_t)((((uint64_t)1 << 32) + p.W - 1) / p.W) : 0u;
    a.o_w = q.o_w, a.o_sink = q.o_sink, a.o_rec = q.o_rec;
    a.divChunk = make_magic((uint32_t)q.nchunk);
    a.divG = make_magic((uint32_t)p.G);
    hipError_t e = hipFuncSetAttribute((const void *)plane_kernel<NB, S, BWD, KB>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)q.lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((plane_kernel<NB, S, BWD, KB>), dim3((unsigned)(p.B * p.G * q.nchunk)),
                       dim3(64 * q.nwaves), q.lds, st, a);
    return hipGetLastError();
}

template <typename S, bool BWD, int KB>
hipError_t plane_nb(const Problem &p, const PlanePlan &q, float *dwp, hipStream_t st)
{
    switch (q.NB) {
    case 1: return plane_launch<1, S, BWD, KB>(p, q, dwp, st);
    case 2: return plane_launch<2, S, BWD, KB>(p, q, dwp, st);
    case 3: return plane_launch<3, S, BWD, KB>(p, q, dwp, st);
    case 4: return plane_launch<4, S, BWD, KB>(p, q, dwp, st);
    case 5: return plane_launch<5, S, BWD, KB>(p, q, dwp, st);
    case 6: return plane_launch<6, S, BWD, KB>(p, q, dwp, st);
    case 7: return plane_launch<7, S, BWD, KB>(p, q, dwp, st);
    default: return plane_launch<8, S, BWD, KB>(p, q, dwp, st);
    }
}

template <typename S, bool BWD>
hipError_t plane_t(const Problem &p, hipStream_t st)
{
    const PlanePlan q = plane_plan_of(p, BWD);
    if (q.nchunk == 0)
        return hipErrorInvalidConfiguration;
    const int64_t ndw = (int64_t)__builtin_popcount(p.mask) * p.B * p.G * 3 * p.H * p.W;
    float *dwp = nullptr;
    hipError_t e = hipSuccess;
    if (BWD && q.nchunk > 1)
        e = p.ws->take((void **)&dwp, (size_t)(q.nchunk * ndw) * sizeof(float));
    if (e != hipSuccess || p.ws->counting)
        return e;
    e = q.KB == 4 || !BWD ? plane_nb<S, BWD, 4>(p, q, dwp, st) : plane_nb<S, BWD, BWD ? 8 : 4>(p, q, dwp, st);
    if (e == hipSuccess && BWD && q.nchunk > 1) {
        const int64_t blocks = std::min<int64_t>((ndw + 255) / 256, 8192);
        hipLaunchKernelGGL((plane_dw_kernel<S>), dim3((unsigned)blocks), dim3(256), 0, st,
                           (const float *)dwp, (S *)p.dw, ndw, q.nchunk);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

// Channels that a CU holds at once.
int plane_channels(const Problem &p, bool bwd)
{
    const PlanePlan q = plane_plan_of(p, bwd);
    if (q.nchunk == 0)
        return 0;
    return (int)((size_t)kLdsBytes / q.lds) * std::min(q.cw, q.nwaves * (64 / q.T));
}

// Whether the plane family is faster than the line family, both sides at most
// 64 (times in us, forward / backward; line: scan_line.hip; where neither is
// wanted: small_fwd_preferred, small_bwd_preferred):
//  * its time is that of the channels a CU holds: below 4 (waves of them in
//    the forward) the line family's traffic costs less: bf16 50 x 50, 4
//    channels, B*C = 3072: plane 136 / 317, line 135 / 406; 61 x 61, 2
//    channels: 464 / 1115 and 202 / 745; fp32 37 x 37, 4 channels, B*C = 6144:
//    222 / 467 and 265 / 905; fp32 40 x 56, 2 channels: 116 / 219 and 39 / 124.
//    A pixel-major forward with vertical directions, which line need not turn
//    around, is line's up to 6: 51 x 33, T2B and B2T, G = C, 1468 planes: 68 and
//    29; 41 x 41, four directions, G = C, 1216: 120 and 61; but not with shared
//    taps and many planes, where only the waves in flight count: four directions,
//    bf16 47 x 47, 30 a group, 8460: 310 and 384 (44 x 44, 8 a group, 2944: 112 and
//    101), fp32 41 x 41, 32 a group, 3072: 122 and 149, nor one direction in a
//    single round of workgroups: 45 x 45 T2B, 1024 in 256: 13 and 17 (42 x 40, 1056
//    in 264: 21 and 17); with vertical ones alone up to 32 a side, in
//    waves of two channels, up to 8: 31 x 31, 3 a group, 4020: 52 and 36; in
//    fp32 up to 10, until some 8000 channels: 24 x 24, 1632: 27 and 18;
//  * with few workgroups it is one workgroup's time, where the line family
//    takes the directions and both sweeps side by side: 45 x 45, B*C = 256:
//    38 / 104 and 27 / 85, B*C = 1024: 42 / 147 and 44 / 172; 28 x 28, B*C =
//    64: 30 / 70 and 24 / 52, B*C = 1024: 30 / 89 and 32 / 134; 33 x 51, G = C,
//    224 (forward): 41 and 27 (one horizontal direction alone leaves nothing to
//    run beside it: 42 x 35, 336 in 84 workgroups: 10 and 16).  Up to 16 x 16 it always wins, and in the
//    backward below 250 pixels: 11 x 22, 120, 8 a group: 32 and 44.
bool plane_preferred(const Problem &p, bool bwd)
{
    const PlanePlan q = plane_plan_of(p, bwd);
    if (q.nchunk == 0)
        return false;
    if (q.T == 16)
        return true;
    const int per_cu = (int)((size_t)kLdsBytes / q.lds);
    const int64_t wgs = (int64_t)p.B * p.G * q.nchunk;
    if (bwd)
        return (q.T == 32 && p.H * p.W < 250) || (plane_channels(p, true) >= 4 && wgs >= 32);
    const bool turned = p.layout != kPixelMajor || (p.mask & 12) != 0;
    if (q.T == 32) {
        const int ch = plane_channels(p, false);
        if (!turned)
            return wgs >= 64 && (ch >= 10 || (ch >= 8 && (p.dtype == 1 || (int64_t)p.B * p.C >= 8000)));
        return per_cu * q.nwaves >= 4 && wgs >= 64;
    }
    const bool horizontal = (p.mask & 3) == 0;
    const bool one = p.layout == kPixelMajor && horizontal && p.mask != 12;
    const int D = __builtin_popcount(p.mask);
    const bool shared = (D > 2 && p.C / p.G >= 4 && (int64_t)p.B * p.C >= (p.dtype == 0 ? 3000 : 3600)) ||
                        (D == 1 && wgs <= 256);
    return per_cu * q.nwaves >= (horizontal || p.layout != kPixelMajor || shared ? 4 : 6) &&
           wgs >= (one ? 28 : 128) && (horizontal || wgs * q.nwaves >= 600);
}

// Forwards that would be the line family's, without the workspace for it: plane
// against the small kernels, which both take none (us, small / plane: fp32 43 x 43,
// both horizontal, B*C = 1344: 274 / 50; bf16 36 x 56, T2B and B2T, 856: 34 / 18; 59 x
// 56, four, 49: 32 / 66, 59 x 59, both horizontal, 288: 144 / 71; fp32 62 x 62, four, one
// channel a CU, 508: 155 / 238; blocked fp32 33 x 62, 3 channels a CU, 768: 70 / 110).
bool plane_over_small(const Problem &p)
{
    const PlanePlan q = plane_plan_of(p, false);
    if (q.nchunk == 0)
        return false;
    const int64_t w = (int64_t)p.B * p.C * q.T / 64;
    const bool pm = p.layout == kPixelMajor;
    const int ch = plane_channels(p, false);
    return (w >= 400 && ch >= (pm ? 3 : 4)) ||
           (pm && ch >= 2 && w * __builtin_popcount(p.mask & 12) >= 500);
}

// Bytes of the backward's partial sums.
int64_t plane_bwd_bytes(const Problem &p)
{
    const PlanePlan q = plane_plan_of(p, true);
    return q.nchunk > 1 ? (int64_t)q.nchunk * __builtin_popcount(p.mask) * p.B * p.G * 3 * p.H *
                              p.W * (int64_t)sizeof(float)
                        : 0;
}

hipError_t launch_fwd_plane(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? plane_t<float, false>(p, st) : plane_t<bf16_t, false>(p, st);
}

hipError_t launch_bwd_plane(const Problem &p, hipStream_t st)
{
    return p.dtype == 0 ? plane_t<float, true>(p, st) : plane_t<bf16_t, true>(p, st);
}

}  // namespace gspn
