// Host check of the S(k) kernels' dynamic LDS limits, which belong to the kernels and so to every handle of the
// process: with the limits set for handles in any order, the last setting covers the row and column blocks of every
// lattice the sampler takes.  hipFuncSetAttribute is this program's own and records the bytes.
#include "lb_fftcore.h"
#include "lb_internal.h"

#include <stdio.h>

#include <map>

using namespace lbf;

static std::map<const void *, int> limit;
extern "C" hipError_t hipFuncSetAttribute(const void *func, hipFuncAttribute, int value)
{
    limit[func] = value;
    return hipSuccess;
}

int main()
{
    int bad = 0;
    for (int precision : {0, 2}) {
        limit.clear();
        if (set_sk_lds_limits(precision) != hipSuccess || limit.size() < 5) return 2;
        long long least = 1ll << 40, most = 0;   // the columns' limit and the rows', which is no lower
        for (const auto &l : limit) {
            least = l.second < least ? l.second : least;
            most = l.second > most ? l.second : most;
        }
        const int e = sk_elem(precision);
        for (int nx = 4; nx <= SK_MAX; nx *= 2)
            for (int ny = 4; ny <= SK_MAX; ny *= 2)
                for (int other = nx; other <= SK_MAX; other *= 2) {   // the widest replica of the handle
                    const long long rows = e * lds_padded((long long)sk_modes_per_pass(precision, other) * ((nx > 1024 ? nx : 1024) / 2));
                    const int split = sk_split(precision, ny), cpb = sk_cols_per_block(precision, nx, ny);
                    const long long points = (long long)(cpb + (split == 1 && cpb > 1)) * (ny / split);
                    const long long cols = e * (precision == 0 ? lds_padded(points) : lds_padded16(points));
                    if ((rows > most || cols > least) && bad++ < 10) printf("precision %d %d x %d: rows %lld, columns %lld, limits %lld and %lld\n", precision, nx, ny, rows, cols, most, least);
                }
        if (most > 160 * 1024) ++bad;
    }
    printf("%d failures\n", bad);
    return bad != 0;
}
