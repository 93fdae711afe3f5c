// The kernel family of planes up to 64 a side, for calls timed in every family (us,
// small / plane / line): each goes to one that is at most 5% behind the fastest.
#include <cstdio>

#include "launch.hpp"

namespace gspn {
hipError_t dispatch_bwd(const Problem &p, hipStream_t s);      // api.cpp
}

using namespace gspn;

struct Call {
    bool bwd, blocked;
    int H, W, B, C, G, dtype, mask;
    float us[3];
};

// H, W, B, C, G, dtype, direction mask, times.  About half of them had been sent to a
// family 1.3 times slower or more.
static const Call calls[] = {
    {true, false, 9, 9, 8, 6, 3, 0, 15, {38.5f, 19.5f, 28.9f}},
    {true, false, 2, 2, 2, 54, 18, 0, 15, {12.7f, 16.6f, 35.6f}},
    {true, false, 1, 2, 4, 21, 21, 0, 3, {5.6f, 9.9f, 11.4f}},
    {true, false, 13, 13, 2, 16, 4, 1, 15, {58.2f, 27.3f, 43.8f}},
    {true, false, 2, 2, 3, 1, 1, 1, 12, {6.9f, 9.8f, 14.9f}},
    {true, false, 2, 3, 2, 102, 51, 1, 1, {4.8f, 7.1f, 11.0f}},
    {true, false, 22, 22, 2, 840, 70, 0, 1, {41.2f, 17.0f, 42.1f}},
    {true, false, 11, 22, 1, 84, 7, 0, 4, {37.4f, 12.9f, 27.7f}},
    {true, false, 20, 11, 4, 24, 2, 0, 15, {98.7f, 34.9f, 65.7f}},
    {true, false, 28, 28, 1, 1896, 474, 1, 7, {144.6f, 49.8f, 76.7f}},
    {true, false, 13, 17, 8, 24, 3, 1, 15, {78.7f, 31.2f, 49.6f}},
    {true, false, 10, 19, 2, 32, 1, 1, 4, {35.8f, 15.2f, 25.2f}},
    {true, false, 63, 63, 1, 104, 13, 0, 3, {190.8f, 110.3f, 41.5f}},
    {true, false, 62, 34, 1, 1636, 1636, 1, 15, {1194.8f, 555.0f, 273.7f}},
    {true, true, 7, 8, 12, 2, 1, 0, 15, {31.7f, 17.1f, 52.0f}},
    {true, true, 1, 1, 8, 2, 2, 0, 15, {8.6f, 12.8f, 42.5f}},
    {true, true, 1, 1, 1, 10128, 1266, 0, 4, {5.4f, 7.7f, 120.0f}},
    {true, true, 10, 10, 1, 3, 1, 1, 15, {42.2f, 28.1f, 55.2f}},
    {true, true, 1, 1, 1, 3136, 98, 1, 7, {11.3f, 16.9f, 98.9f}},
    {true, true, 1, 1, 32, 82, 41, 1, 1, {4.5f, 8.3f, 35.8f}},
    {true, true, 16, 23, 1, 10248, 854, 0, 7, {519.5f, 201.3f, 541.7f}},
    {true, true, 11, 22, 1, 120, 15, 0, 1, {20.6f, 12.8f, 28.5f}},
    {true, true, 22, 11, 1, 2, 2, 0, 12, {27.6f, 17.7f, 27.6f}},
    {true, true, 22, 22, 8, 1100, 550, 1, 15, {444.6f, 273.4f, 610.7f}},
    {true, true, 11, 20, 1, 3, 1, 1, 15, {66.2f, 39.8f, 56.0f}},
    {true, true, 11, 19, 2, 3, 1, 1, 7, {45.7f, 30.1f, 47.5f}},
    {true, true, 37, 61, 1, 2, 1, 0, 15, {249.7f, 130.7f, 75.5f}},
    {true, true, 59, 56, 4, 2, 2, 1, 7, {254.5f, 172.6f, 49.2f}},
    {false, false, 13, 13, 1, 328, 41, 0, 1, {4.4f, 6.5f, 7.3f}},
    {false, false, 15, 15, 2, 832, 26, 0, 15, {13.2f, 23.6f, 34.6f}},
    {false, false, 8, 12, 8, 208, 26, 0, 7, {6.8f, 8.8f, 24.5f}},
    {false, false, 8, 7, 4, 12, 1, 1, 15, {6.2f, 9.3f, 11.4f}},
    {false, false, 14, 15, 8, 462, 462, 1, 1, {6.6f, 10.9f, 17.0f}},
    {false, false, 14, 8, 32, 98, 98, 1, 3, {6.4f, 10.6f, 20.3f}},
    {false, false, 20, 31, 2, 668, 334, 0, 12, {35.6f, 17.6f, 33.2f}},
    {false, false, 19, 19, 4, 228, 19, 0, 3, {9.1f, 12.4f, 11.9f}},
    {false, false, 32, 32, 1, 1312, 41, 0, 1, {9.6f, 13.2f, 13.4f}},
    {false, false, 10, 17, 2, 9960, 1245, 1, 15, {149.3f, 44.7f, 294.3f}},
    {false, false, 25, 27, 4, 306, 153, 1, 3, {11.4f, 15.0f, 18.2f}},
    {false, false, 62, 46, 1, 1, 1, 0, 7, {20.7f, 48.7f, 14.7f}},
    {false, false, 38, 38, 8, 160, 5, 0, 3, {35.4f, 40.7f, 21.5f}},
    {false, false, 32, 41, 4, 384, 48, 0, 3, {36.6f, 37.3f, 20.8f}},
    {false, false, 37, 37, 1, 574, 287, 1, 4, {21.0f, 11.2f, 20.6f}},
    {false, false, 30, 44, 1, 374, 187, 1, 3, {15.6f, 15.0f, 11.3f}},
    {false, false, 46, 46, 4, 92, 46, 1, 15, {55.5f, 44.8f, 25.3f}},
    {false, true, 6, 10, 32, 336, 84, 0, 15, {36.0f, 19.4f, 125.2f}},
    {false, true, 1, 1, 4, 536, 536, 0, 3, {5.0f, 7.2f, 21.6f}},
    {false, true, 14, 14, 32, 624, 624, 0, 1, {38.8f, 68.4f, 102.4f}},
    {false, true, 8, 14, 1, 14672, 7336, 1, 15, {58.0f, 41.4f, 188.0f}},
    {false, true, 12, 15, 8, 352, 11, 1, 7, {14.0f, 21.2f, 49.4f}},
    {false, true, 12, 15, 2, 1923, 1923, 1, 4, {7.8f, 11.6f, 36.0f}},
    {false, true, 32, 32, 4, 10, 5, 0, 7, {20.4f, 41.4f, 26.7f}},
    {false, true, 30, 30, 2, 294, 147, 0, 3, {20.4f, 30.4f, 33.9f}},
    {false, true, 32, 32, 2, 297, 297, 0, 15, {46.9f, 106.1f, 68.1f}},
    {false, true, 13, 26, 2, 4960, 155, 1, 4, {44.1f, 22.0f, 72.4f}},
    {false, true, 27, 29, 1, 4552, 569, 1, 15, {87.7f, 149.0f, 131.6f}},
    {false, true, 30, 30, 32, 41, 41, 1, 15, {36.0f, 96.0f, 88.2f}},
    {false, true, 29, 37, 8, 15, 15, 0, 15, {24.8f, 42.1f, 42.1f}},
    {false, true, 44, 44, 1, 32, 1, 0, 1, {11.0f, 17.1f, 14.9f}},
    {false, true, 57, 59, 1, 4, 1, 0, 4, {14.7f, 32.8f, 19.4f}},
    {false, true, 21, 38, 8, 128, 4, 1, 7, {41.8f, 25.5f, 44.3f}},
    {false, true, 41, 41, 7, 3, 1, 1, 7, {17.2f, 35.2f, 29.9f}},
    {false, true, 32, 43, 1, 64, 2, 1, 15, {21.9f, 46.6f, 36.6f}},    // many planes
    {false, false, 10, 10, 2, 39420, 39420, 0, 15, {416.7f, 286.4f, 1729.4f}},
    {false, true, 8, 8, 8, 2460, 2460, 0, 7, {72.5f, 46.0f, 170.2f}},
    {false, false, 11, 11, 16, 10128, 10128, 1, 15, {625.6f, 455.3f, 3687.0f}},
    {false, false, 9, 8, 4, 12632, 12632, 1, 15, {106.0f, 133.0f, 1030.0f}},
    {false, true, 9, 9, 8, 17536, 17536, 1, 15, {453.0f, 486.0f, 1864.0f}},
    {false, false, 47, 47, 1, 8460, 282, 1, 15, {1008.3f, 309.7f, 384.3f}},
    {false, false, 44, 44, 32, 92, 11, 1, 15, {288.0f, 112.0f, 101.0f}},
    {false, false, 41, 41, 32, 96, 3, 0, 15, {396.5f, 122.2f, 149.1f}},
    {false, false, 45, 45, 16, 64, 8, 1, 1, {29.1f, 12.5f, 16.6f}},
    {false, false, 42, 40, 4, 264, 66, 1, 1, {25.0f, 21.0f, 17.0f}},
    {false, true, 38, 38, 4, 2178, 363, 1, 7, {319.6f, 264.5f, 374.0f}},
    {false, true, 26, 35, 2, 1953, 279, 1, 15, {180.3f, 120.8f, 135.7f}},
    {false, true, 44, 44, 8, 832, 26, 1, 12, {242.6f, 188.9f, 193.6f}},
};

// Planes above 64 a side: line family, in rounds of what the query's workspace holds, /
// general family.
struct LongCall {
    bool bwd, blocked;
    int H, W, B, C, G, dtype, mask;
    float line, general;
};

static const LongCall long_calls[] = {
    {false, true, 68, 34, 18, 1, 1, 1, 15, 146.8f, 43.2f},
    {false, true, 47, 65, 3, 8, 1, 1, 8, 81.6f, 42.1f},
    {false, true, 43, 69, 2, 10, 5, 1, 8, 106.0f, 45.4f},
    {false, true, 26, 146, 8, 1, 1, 1, 1, 61.2f, 20.2f},
    {false, true, 102, 63, 1, 14, 14, 1, 3, 138.0f, 65.2f},
    {false, true, 12, 118, 2, 32, 2, 1, 3, 17.1f, 11.2f},
    {false, true, 16, 68, 19, 1, 1, 1, 3, 17.7f, 13.9f},
    {false, false, 22, 145, 1, 8, 4, 1, 8, 150.7f, 92.7f},
    {false, false, 31, 95, 2, 14, 14, 1, 4, 119.7f, 72.9f},
    {false, false, 77, 150, 2, 3, 3, 1, 4, 223.6f, 135.1f},
    {false, false, 21, 137, 2, 8, 1, 1, 3, 27.1f, 18.4f},
    {false, false, 70, 70, 2, 1, 1, 1, 3, 28.1f, 51.8f},
    {false, false, 114, 114, 3, 1, 1, 1, 3, 41.3f, 81.2f},
    {false, false, 40, 110, 1, 8, 2, 1, 15, 50.6f, 92.5f},    {false, true, 102, 17, 2, 431, 431, 1, 4, 38.8f, 28.7f},
    {false, true, 82, 27, 32, 81, 81, 0, 4, 128.1f, 265.5f},
    {false, true, 18, 93, 1, 3476, 869, 0, 2, 73.3f, 95.0f},
    {false, true, 22, 167, 4, 384, 192, 1, 2, 61.6f, 49.5f},
    {false, true, 23, 131, 2, 276, 69, 1, 1, 29.9f, 31.6f},
    {false, true, 27, 158, 32, 35, 35, 1, 2, 69.5f, 51.4f},
    {false, true, 19, 158, 1, 995, 995, 1, 3, 85.1f, 48.4f},
    {false, true, 40, 122, 4, 232, 232, 1, 3, 126.4f, 78.9f},
    {false, true, 37, 171, 1, 352, 22, 1, 3, 50.7f, 53.3f},
    {false, true, 169, 23, 32, 7, 7, 1, 12, 45.1f, 29.8f},
    {false, true, 172, 33, 1, 100, 100, 1, 12, 39.6f, 33.4f},
    {false, true, 172, 30, 2, 352, 352, 1, 12, 107.6f, 188.1f},
};

// A caller's workspace below the query's: line family in rounds / the other family.
struct LimitedCall {
    bool bwd, blocked;
    int H, W, B, C, G, dtype, mask;
    int64_t bytes;
    float line, other;
};

static const LimitedCall limited_calls[] = {
    {true, true, 38, 38, 1, 1856, 116, 1, 3, 8040192, 847.3f, 179.5f},
    {true, true, 54, 54, 1, 1808, 113, 1, 15, 31632768, 1714.6f, 584.3f},
    {true, false, 38, 38, 1, 1856, 116, 1, 3, 8040192, 321.8f, 174.5f},
    {true, false, 59, 34, 2, 992, 62, 1, 3, 11939712, 349.4f, 265.5f},
    {true, false, 63, 63, 4, 272, 17, 1, 7, 19432224, 589.2f, 775.5f},
    {true, false, 42, 64, 2, 1104, 69, 1, 15, 35610624, 859.2f, 1928.7f},
    {true, false, 42, 23, 4, 832, 26, 0, 15, 19289088, 2026.0f, 683.4f},
    {true, false, 31, 31, 1, 3264, 102, 1, 15, 9410112, 1979.7f, 453.4f},
    {false, false, 51, 73, 8, 181, 181, 1, 8, 21563616, 143.6f, 633.4f},
    {false, true, 83, 83, 32, 12, 4, 1, 15, 42326016, 205.3f, 160.1f},
    {false, false, 83, 83, 32, 12, 4, 1, 15, 42326016, 89.6f, 590.1f},
    {true, true, 35, 149, 1, 708, 177, 1, 15, 118151040, 665.6f, 1982.0f},
};

// Whatever the workspace, a backward up to 64 a side that any family can run in it is
// taken, and takes no more than it.
static int check_limited()
{
    int bad = 0;
    Workspace ws;
    ws.counting = true;
    for (const LimitedCall &c : limited_calls) {
        Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                  nullptr, c.mask, c.B, c.C, c.G, c.H, c.W, c.dtype, c.blocked ? kBlocked : kPixelMajor, &ws};
        p.ws_cap = c.bytes;
        if (line_supported(p, c.bwd) != (c.line < c.other)) {
            printf("limited %s%s %dx%d C=%d: line %.1f, other %.1f us\n", c.bwd ? "bwd" : "fwd",
                   c.blocked ? "_blocked" : "", c.H, c.W, c.C, c.line, c.other);
            ++bad;
        }
    }
    for (int side : {1, 3, 9, 17, 20, 33, 38, 63})
        for (int cpg : {1, 7, 40, 60, 130})
            for (int G : {1, 6})
                for (int mask : {1, 12, 15})
                    for (int layout : {kBlocked, kPixelMajor})
                        for (int64_t cap = 0; cap < (int64_t)1 << 30; cap = cap * 3 / 2 + 1024) {
                            Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                                      nullptr, nullptr, nullptr, mask, 2, cpg * G, G, side, side + 1, 1,
                                      layout, &ws};
                            ws.used = 0;
                            p.ws_cap = cap;
                            const bool can = small_bwd_bytes(p) <= cap || plane_bwd_bytes(p) <= cap ||
                                             line_fits(p, true);
                            if (dispatch_bwd(p, nullptr) != hipSuccess || (can && (int64_t)ws.used > cap)) {
                                printf("%dx%d cpg %d G %d mask %d layout %d: %lld of %lld bytes\n", side,
                                       side + 1, cpg, G, mask, layout, (long long)ws.used, (long long)cap);
                                ++bad;
                            }
                        }
    return bad;
}

// Calls whose single launch in the family would have 2^32 threads or more, which HIP
// refuses, and the largest that have fewer: taken by the family or not.
static int check_launch_limits()
{
    int bad = 0;
    auto problem = [](int mask, int C, int G, int H, int W, int layout) {
        return Problem{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                       nullptr, mask, 1, C, G, H, W, 1, layout};
    };
    auto expect = [&](bool got, bool want, const char *what) {
        if (got != want) {
            printf("launch limits: %s\n", what);
            ++bad;
        }
    };
    // a plane of 8 x 16 pixels is 256 threads of the sum in LDS
    expect(wide_sum_supported(problem(1, (1 << 24) - 1, 1, 8, 16, kBlocked)), true, "sums");
    expect(wide_sum_supported(problem(1, 1 << 24, 1, 8, 16, kBlocked)), false, "too many sums");
    // one group of 65 x 65 planes, 6 tiles of 512 threads each
    expect(line_supported(problem(1, 1 << 19, 1, 65, 65, kPixelMajor), false), true, "a group");
    expect(line_supported(problem(1, 1 << 21, 1, 65, 65, kPixelMajor), false), false, "too large a group");
    // the small forward: 256 threads for every four planes
    expect(small_fwd_preferred(problem(1, (1 << 26) - 4, (1 << 26) - 4, 9, 9, kPixelMajor)), true, "small");
    expect(small_fwd_preferred(problem(1, 1 << 26, 1 << 26, 9, 9, kPixelMajor)), false, "too many small");
    return bad;
}

int main()
{
    int bad = check_launch_limits() + check_limited();
    for (const LongCall &c : long_calls) {
        Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                  nullptr, c.mask, c.B, c.C, c.G, c.H, c.W, c.dtype, c.blocked ? kBlocked : kPixelMajor};
        if (line_supported(p, c.bwd) != (c.line < c.general)) {
            printf("%s%s %dx%d B=%d C=%d G=%d dtype %d mask %d: line %.1f, general %.1f us\n",
                   c.bwd ? "bwd" : "fwd", c.blocked ? "_blocked" : "", c.H, c.W, c.B, c.C, c.G,
                   c.dtype, c.mask, c.line, c.general);
            ++bad;
        }
    }
    for (const Call &c : calls) {
        Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                  nullptr, c.mask, c.B, c.C, c.G, c.H, c.W, c.dtype, c.blocked ? kBlocked : kPixelMajor};
        const bool small = c.bwd ? small_bwd_preferred(p) : small_fwd_preferred(p);
        const int family = small ? 0 : plane_preferred(p, c.bwd) ? 1 : 2;
        float best = c.us[0];
        for (float t : c.us)
            best = t < best ? t : best;
        if (c.us[family] > 1.05f * best + 0.3f) {
            printf("%s%s %dx%d B=%d C=%d G=%d dtype %d mask %d: family %d, %.1f of %.1f us\n",
                   c.bwd ? "bwd" : "fwd", c.blocked ? "_blocked" : "", c.H, c.W, c.B, c.C, c.G,
                   c.dtype, c.mask, family, c.us[family], best);
            ++bad;
        }
    }
    printf(bad ? "%d calls on a slower family\n" : "all routes clean\n", bad);
    return bad != 0;
}
