// Host check: launch_tile refuses what it has no kernel or no tile for (nothing is launched here), and
// k_tile's LDS stays within the figures that its header states.
#include "lb_internal.h"

#include <stdio.h>

using namespace lbf;

int main()
{
    int bad = 0;
    const float field = 0;
    for (int precision : {0, 1, 2})
        for (int ns = -1; ns <= 8; ++ns)
            for (int ty = 0; ty <= 20; ++ty)
                for (int cn = 0; cn < 2; ++cn) {
                    const bool kernel = ns == 1 || ns == 2 || (ns == 4 && precision != 0 && !cn);
                    if (kernel && ty > 4 * (ns - 1) && ty <= 16) continue;   // would launch
                    TileLaunch a{};
                    a.ns = ns;
                    a.ty = ty;
                    a.xi = cn ? &field : nullptr;
                    if (launch_tile(precision, a, nullptr) != hipErrorInvalidValue && bad++ < 10)
                        printf("precision %d, %d steps, %d rows, correlated %d: not refused\n", precision, ns, ty, cn);
                }
    for (int ns : {1, 2, 4})
        if (tile_lds_bytes(2, ns, TILE_MAX_TY) > 36.65 * 1024 || tile_lds_bytes(0, ns, TILE_MAX_TY) > 73.3 * 1024) ++bad;
    printf("%d failures\n", bad);
    return bad != 0;
}
