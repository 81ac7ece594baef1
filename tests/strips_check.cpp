// Host check of the two-step kernel's strips (make_tiles2): for every width and workgroup size the strips
// store every column once, their count stays below 17/16 of the fewest possible, and the list fits its bound.
#include "lb_internal.h"

#include <stdio.h>

using namespace lbf;

int main()
{
    long long bad = 0;
    for (int elem : {4, 8})
        for (int bx = STEP2_MIN_BX; bx <= 512; bx += 64)
            for (int nx = 3, ny = STEP2_MIN_H; nx < 20000; nx += ny > STEP2_MIN_H ? (nx < 2100 ? 1 : 7) : 0,
                     ny = ny > STEP2_MIN_H ? STEP2_MIN_H : 1 << 15) {
                RepDesc d{};
                d.nx = nx;
                d.ny = ny;
                std::vector<Tile> tiles;
                std::vector<int32_t> wgs;
                make_tiles2({d}, elem, bx, ny, tiles, wgs);   // one band
                std::vector<int> x0;
                for (const Tile &t : tiles)
                    if (t.rep >= 0) x0.push_back(t.x0);
                const long long n = (long long)x0.size(), w = nx > bx ? step2_out(bx, elem, nx, ny) : nx;
                const long long fewest = nx > bx ? (nx + bx - 7) / (bx - 6) : 1;
                bool ok = w <= (nx > bx ? bx - 6 : nx) && n == (nx + w - 1) / w && (n == fewest || (16 * n < 17 * fewest && (long long)nx * ny >= 1 << 22)) &&
                          (long long)tiles.size() <= max_tiles2({nx}, {ny}) &&
                          (long long)wgs.size() - 1 == step2_workgroups({d}, elem, bx, ny);
                if (nx < 600 && ny == STEP2_MIN_H)   // several bands, several replicas
                    for (double h : {8.0, 11.0, 40.0}) {
                        RepDesc e = d, f = d;
                        e.ny = 8 + nx / 3;
                        f.nx = 3 + nx / 2;
                        f.ny = 129;
                        make_tiles2({d, e, f}, elem, bx, h, tiles, wgs);
                        ok = ok && (long long)wgs.size() - 1 == step2_workgroups({d, e, f}, elem, bx, h);
                    }
                std::vector<char> seen(nx, 0);
                for (int x : x0)
                    for (int c = x; c < x + w && c < nx; ++c) ok = ok && !seen[c]++;
                for (char c : seen) ok = ok && c;
                if (!ok && bad++ < 10) printf("elem %d bx %d nx %d: %lld strips of %lld (fewest %lld)\n", elem, bx, nx, n, w, fewest);
            }
    printf("%lld failures\n", bad);
    return bad != 0;
}
