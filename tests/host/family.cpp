// The kernel family of calls given on stdin, one a line: name, B, C, G, H, W, dtype,
// direction mask, operation (fwd, bwd, fwd_blocked, bwd_blocked), with the workspace
// that the query gives.  Prints the name, the operation and the family.
#include <cstdio>
#include <cstring>

#include "launch.hpp"

using namespace gspn;

static const char *family(const Problem &p, bool bwd)
{
    if (med_supported(p))
        return "med";
    if (tiny_supported(p))
        return "tiny";
    if (!bwd && wide_sum_supported(p))
        return "sum";
    if (p.H <= kSmallSide && p.W <= kSmallSide) {
        if (bwd ? small_bwd_preferred(p) : small_fwd_preferred(p))
            return "small";
        if (plane_preferred(p, bwd))
            return "plane";
        return line_supported(p, bwd) ? "line" : bwd || plane_over_small(p) ? "plane" : "small";
    }
    const bool wide = !bwd && wide_supported(p);
    if ((!wide || line_fwd_preferred(p)) && line_supported(p, bwd))
        return "line";
    return wide ? "wide" : "general";
}

int main()
{
    char name[256], op[32];
    int B, C, G, H, W, dtype, mask;
    while (scanf("%255s %d %d %d %d %d %d %d %31s", name, &B, &C, &G, &H, &W, &dtype, &mask, op) == 9) {
        const Problem p{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                        nullptr, mask, B, C, G, H, W, dtype,
                        strstr(op, "blocked") ? kBlocked : kPixelMajor};
        printf("%s %s %s\n", name, op, family(p, strncmp(op, "bwd", 3) == 0));
    }
    return 0;
}
