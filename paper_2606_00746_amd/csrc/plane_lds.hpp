// LDS layout of the plane family (scan_plane.hip): the sizes of its launches and
// the places of its records, by functions that the kernel and the host share.
#pragma once

#include <algorithm>

#include <stdint.h>

#include "device.hpp"
#include "launch.hpp"

namespace gspn {

// dwords of a pixel's record and of a tap entry
template <typename S>
struct Rec;
template <>
struct Rec<bf16_t> {
    static constexpr int N = 3;     // x | dy, u | lam, sum
    static constexpr int WN = 2;    // w0 | w1, w2
    static constexpr int E = 2;     // elements of a dword
};
template <>
struct Rec<float> {
    static constexpr int N = 5;     // x, dy, u, lam, sum
    static constexpr int WN = 3;    // w0, w1, w2
    static constexpr int E = 1;
};

// First dword of the records of a wave's channels: each wave's NL planes of RS
// dwords have a spare record before and one behind.
__host__ __device__ __forceinline__ int plane_wave_rec0(int o_rec, int wave, int NL, int RS, int N)
{
    return o_rec + wave * (NL * RS + 2 * N) + N;
}

// Dword offset (from there) of the record of pixel e of a wave's stretch:
// linear where rows are odd (mW = 0), else a record is left out behind each row
// (channels follow each other the same way).  With even rows planes begin at
// whole dwords, so a dword's two pixels lie in one row and their records side
// by side.
__host__ __device__ __forceinline__ int plane_rec(int e, uint32_t mW, int N)
{
    return N * (e + (int)(((uint64_t)(uint32_t)(e > 0 ? e : 0) * mW) >> 32));
}

// The pixel whose record, and the one after it, a lane reads to store the dword
// that starts with pixel e of a stretch of n: behind the stretch (values that
// are not stored) the last one, whose neighbour is the spare record.
__host__ __device__ __forceinline__ int plane_flush_pixel(int e, int n)
{
    return e < n - 1 ? e : n - 1;
}

struct PlanePlan {
    int NB, T, KB, cw, nwaves, nchunk, Wp, RS, o_w, o_sink, o_rec;
    uint32_t mW;             // ceil(2^32 / W) for even W, 0 for odd
    size_t lds;
};

inline PlanePlan plane_plan(int H, int W, int cpg, bool f32, bool bwd)
{
    const int N = f32 ? Rec<float>::N : Rec<bf16_t>::N;
    const int WN = f32 ? Rec<float>::WN : Rec<bf16_t>::WN;
    const int m = std::max(H, W), HW = H * W;
    PlanePlan q{};
    q.NB = (m + 7) / 8;
    q.T = m <= 16 ? 16 : (m <= 32 ? 32 : 64);
    q.Wp = W | 1;
    q.RS = H * q.Wp * N;
    q.mW = W % 2 == 0 ? (uint32_t)((((uint64_t)1 << 32) + W - 1) / W) : 0u;
    const int NL = 64 / q.T;
    auto layout = [&](PlanePlan &r, int kb, int nw) {
        const int slots = bwd ? kb * ((nw * NL + 3) & ~3) * q.T * 2 : 0;
        r.KB = kb;
        r.nwaves = nw;
        r.o_w = slots;
        r.o_sink = (r.o_w + (HW + m) * WN + 1) & ~1;
        r.o_rec = r.o_sink + 64 * N;
        r.lds = ((size_t)r.o_rec + (size_t)nw * (NL * q.RS + 2 * N)) * 4;
        return r.lds <= (size_t)kLdsBytes;
    };
    PlanePlan best = q;
    best.nchunk = 0;
    for (int kb : {8, 4}) {
        if (kb == 8 && q.T == 16)
            continue;
        PlanePlan r = q;
        int nw = std::min(8, (cpg + NL - 1) / NL);
        while (nw > 0 && !layout(r, kb, nw))
            --nw;
        if (nw == 0)
            continue;
        r.nchunk = (cpg + nw * NL - 1) / (nw * NL);
        r.cw = (cpg + r.nchunk - 1) / r.nchunk;
        layout(r, kb, (r.cw + NL - 1) / NL);
        // the larger batch where its steps have a line of lanes each
        if (best.nchunk == 0 || r.nchunk < best.nchunk ||
            (r.nchunk == best.nchunk && best.nwaves * NL < best.KB))
            best = r;
    }
    return best;
}

}  // namespace gspn
