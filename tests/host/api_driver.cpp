// Checks of the library's host side that need no device, run by
// tests/test_host_api.py: api_driver <check>.  Prints what failed and returns
// whether anything did.
#include <cstdio>
#include <cstring>
#include <set>

#include "fpts_internal.hpp"
#include "fpts_lpt.h"

namespace {

int failures = 0;

// A mesh handle with what the size calls read.
fpts_mesh shape(int D, int R, int N, int64_t nel, int NL, int max_cell)
{
    fpts_mesh m{};
    m.D = D;
    m.R = R;
    m.N = N;
    m.NP = R == 3 ? N * N * N : R == 2 ? N * N : N;
    m.nel = nel;
    m.NL = NL;
    m.max_cell = max_cell;
    m.cus = 256;
    return m;
}

typedef size_t (*SizeFn)(const fpts_mesh *, int64_t);
struct Size {
    const char *name;
    SizeFn fn;
};
const Size kSizes[] = {{"find", fpts_find_workspace_size},
                       {"eval", fpts_eval_workspace_size},
                       {"find_eval", fpts_find_eval_workspace_size},
                       {"lpt", fpts_lpt_workspace_size}};

// A workspace made for n points holds for fewer: none of the sizes decreases
// as n grows, whichever layouts lie between.
void sizes()
{
    const fpts_mesh meshes[] = {
        shape(3, 3, 8, 110592, 48, 20), shape(3, 3, 4, 64000, 40, 27),
        shape(3, 3, 4, 8000, 20, 27),   shape(3, 3, 6, 13824, 24, 30),
        shape(3, 3, 9, 1728, 12, 27),   shape(2, 2, 5, 256, 16, 9),
        shape(2, 2, 5, 505, 23, 9),     shape(2, 2, 6, 16384, 128, 9),
        shape(3, 2, 7, 6144, 19, 60),   shape(2, 1, 4, 1024, 32, 8),
        shape(2, 1, 4, 1u << 20, 1024, 6), shape(3, 3, 3, 1, 1, 1),
        shape(3, 3, 8, 4096, 300, 4)};
    std::set<int64_t> ns;
    for (int64_t n = 0; n < 20000; ++n) ns.insert(n);
    for (double x = 2e4; x < 5e7; x *= 1.003) ns.insert((int64_t)x);
    // where the tiles of the cell binning change their size, and the steps of
    // a histogram by one tile below
    for (int64_t items = 1; items <= 64; items *= 2)
        for (int64_t b : {int64_t(4096), 256 * items * 768, 256 * items, 128 * items * 8}) {
            for (int64_t k = -4100; k <= 4100; k += 41)
                if (b + k >= 0) ns.insert(b + k);
            for (int64_t k = -2; k <= 2; ++k) ns.insert(b + k);
        }
    for (const fpts_mesh &m : meshes)
        for (const Size &s : kSizes) {
            if (s.fn == fpts_lpt_workspace_size && m.R != m.D) continue;
            size_t most = 0;
            int64_t at = 0;
            int bad = 0;
            for (int64_t n : ns) {
                const size_t b = s.fn(&m, n);
                if (b < most && bad++ < 3)
                    std::printf("%s, D %d R %d N %d, %lld elements: %zu bytes for %lld points, "
                                "%zu for %lld\n",
                                s.name, m.D, m.R, m.N, (long long)m.nel, most, (long long)at, b,
                                (long long)n);
                if (b >= most) {
                    most = b;
                    at = n;
                }
            }
            failures += bad;
        }
}

}  // namespace

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "sizes")) sizes();
    else return 2;
    std::printf("%s: %d failures\n", what, failures);
    return failures != 0;
}
