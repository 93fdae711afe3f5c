// Every LDS access of the plane family's copies, for all sides up to 64, both
// types and passes and uneven group widths: the records that a wave's lanes
// write as the planes come in and read as they go out lie within the
// workgroup's allocation, and each wave's within its own part.
#include <cstdio>

#include "plane_lds.hpp"

using namespace gspn;

static long bad = 0;

template <typename S>
static void check(int H, int W, int cpg, bool bwd)
{
    constexpr int N = Rec<S>::N, WN = Rec<S>::WN, E = Rec<S>::E;
    const PlanePlan q = plane_plan(H, W, cpg, E == 1, bwd);
    if (q.nchunk == 0) {
        printf("%dx%d cpg %d: no plan\n", H, W, cpg);
        ++bad;
        return;
    }
    const int NL = 64 / q.T, HW = H * W, total = (int)(q.lds / 4), m = std::max(H, W);
    bool ok = q.lds <= (size_t)kLdsBytes && q.nwaves <= 8 && q.cw * q.nchunk >= cpg &&
              q.cw <= q.nwaves * NL && q.o_w + (HW + m) * WN <= q.o_sink &&
              q.o_sink + 64 * N <= q.o_rec &&
              (!bwd || q.KB * ((q.nwaves * NL + 3) & ~3) * q.T * 2 <= q.o_w);
    // the last wave with all of its channels (the addresses grow with both), and one channel
    for (int wave : {0, q.nwaves - 1})
        for (int nmine : {1, std::min(NL, q.cw - wave * NL)}) {
            if (nmine <= 0)
                continue;
            const int n = nmine * HW;
            const int lo = q.o_rec + wave * (NL * q.RS + 2 * N), hi = lo + NL * q.RS + 2 * N;
            ok = ok && hi <= total;
            for (int sh = 0; sh < (E == 2 && HW % 2 ? 2 : 1); ++sh) {
                const int nu = (sh + n + E - 1) / E;
                const int rec0 = plane_wave_rec0(q.o_rec, wave, NL, q.RS, N);
                for (int un = 0; un < (nu + 255) / 256 * 256; ++un) {
                    if (un == 1 && nu > 2)
                        un = nu - 2;      // in between the offsets only grow
                    const int e = E * un - sh;
                    // coming in: two pixels' records (bf16) or one
                    const int in = rec0 + plane_rec(e, q.mW, N);
                    if (un < nu)
                        ok = ok && in >= lo && in + E * N <= hi;
                    // going out, also by the lanes behind the stretch
                    const int out = rec0 + plane_rec(plane_flush_pixel(e, n), q.mW, N);
                    ok = ok && out >= lo && out + E * N <= hi && (un >= nu || out == in);
                }
            }
        }
    if (!ok && ++bad <= 10)
        printf("%dx%d cpg %d %s %s: outside its part of %d dwords\n", H, W, cpg,
               E == 1 ? "f32" : "bf16", bwd ? "backward" : "forward", total);
}

int main()
{
    for (int H = 1; H <= 64; ++H)
        for (int W = 1; W <= 64; ++W)
            for (int cpg : {1, 2, 3, 4, 5, 8, 9, 12, 31, 32, 33, 100})
                for (int bwd = 0; bwd < 2; ++bwd) {
                    check<bf16_t>(H, W, cpg, bwd != 0);
                    check<float>(H, W, cpg, bwd != 0);
                }
    printf(bad ? "%ld plans wrong\n" : "all plans clean\n", bad);
    return bad != 0;
}
