// Checks of the library's host side that need no device, run by
// tests/test_host_api.py: api_driver <check>.  Prints what failed and returns
// whether anything did.  The HIP calls that a check reaches are defined here
// (the program's own definitions come before the runtime's) and touch no
// device: launches are noted, nothing runs.
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "fpts_internal.hpp"
#include "fpts_lpt.h"

struct Launch {
    const void *kernel;
    uint64_t blocks, threads;   // threads of a block
};
static std::vector<Launch> launches;
static int copies_back = 0;   // the copies to the host until one fails
static std::vector<double> first_back;   // what the first one brings

extern "C" {

hipError_t hipGetLastError() { return hipSuccess; }

static dim3 call_grid, call_block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t)
{
    call_grid = g;
    call_block = b;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s)
{
    *g = call_grid;
    *b = call_block;
    *shared = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *kernel, dim3 g, dim3 b, void **, size_t, hipStream_t)
{
    launches.push_back({kernel, (uint64_t)g.x * g.y * g.z, (uint64_t)b.x * b.y * b.z});
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t)
{
    // an address that nothing is read from
    *p = reinterpret_cast<void *>(uintptr_t(1) << 40);
    return hipSuccess;
}

hipError_t hipFree(void *) { return hipSuccess; }

hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

hipError_t hipMemcpyAsync(void *dst, const void *, size_t bytes, hipMemcpyKind kind, hipStream_t)
{
    if (kind != hipMemcpyDeviceToHost) return hipSuccess;
    if (copies_back-- <= 0) return hipErrorInvalidValue;
    if (!first_back.empty() && bytes % (first_back.size() * sizeof(double)) == 0) {
        const size_t w = first_back.size();
        for (size_t i = 0; i < bytes / sizeof(double); ++i)
            static_cast<double *>(dst)[i] = first_back[i % w];
        first_back.clear();
    }
    return hipSuccess;
}

}  // extern "C"

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

// What the calls asked for before their kernels kept records and spread
// counters: programs have budgets made for it (a server's pool, a buffer), so
// they must not ask for more, and fpts_eval must take that much.
struct Asked {
    int D, R, N;
    int64_t nel;
    int NL, max_cell;
    int64_t n;
    size_t bytes[4];   // find, eval, find_eval, lpt
};
const Asked kAsked[] = {
    {3, 3, 8, 110592, 48, 20, 1, {5807104, 1329152, 7136512, 5807616}},
    {3, 3, 8, 110592, 48, 20, 1000, {6158592, 1344512, 7527168, 6186752}},
    {3, 3, 8, 110592, 48, 20, 4096, {6932480, 1394176, 8424960, 7047168}},
    {3, 3, 8, 110592, 48, 20, 4097, {6938368, 1394944, 8431872, 7053568}},
    {3, 3, 8, 110592, 48, 20, 30000, {13263616, 1810432, 15794176, 14103808}},
    {3, 3, 8, 110592, 48, 20, 1000000, {236058624, 13833216, 273891840, 264058624}},
    {3, 3, 8, 110592, 48, 20, 6291455, {1444400384, 77661184, 1673056512, 1620561152}},
    {3, 3, 6, 13824, 24, 30, 1, {774400, 167936, 942592, 774912}},
    {3, 3, 6, 13824, 24, 30, 1000, {1125888, 183296, 1333248, 1154048}},
    {3, 3, 6, 13824, 24, 30, 4096, {1899776, 232960, 2231040, 2014464}},
    {3, 3, 6, 13824, 24, 30, 4097, {1905664, 233728, 2237952, 2020864}},
    {3, 3, 6, 13824, 24, 30, 30000, {7969536, 584448, 9274112, 8809728}},
    {3, 3, 6, 13824, 24, 30, 1000000, {229385216, 12284928, 265670144, 257385216}},
    {3, 3, 6, 13824, 24, 30, 6291455, {1437239552, 76112896, 1664347392, 1613400320}},
    {2, 2, 5, 256, 16, 9, 1, {60672, 5120, 66048, 61184}},
    {2, 2, 5, 256, 16, 9, 1000, {361216, 17664, 395008, 381440}},
    {2, 2, 5, 256, 16, 9, 4096, {960768, 54784, 1081088, 1042688}},
    {2, 2, 5, 256, 16, 9, 4097, {966656, 55552, 1088000, 1049088}},
    {2, 2, 5, 256, 16, 9, 30000, {5838336, 367360, 6685696, 6438400}},
    {2, 2, 5, 256, 16, 9, 1000000, {188441600, 12067840, 216509440, 208441600}},
    {2, 2, 5, 256, 16, 9, 6291455, {1184570624, 75895808, 1361129728, 1310399744}},
    {3, 2, 7, 6144, 19, 60, 1, {375552, 75776, 451584, 376064}},
    {3, 2, 7, 6144, 19, 60, 1000, {703232, 91136, 810496, 731392}},
    {3, 2, 7, 6144, 19, 60, 4096, {1402624, 140800, 1608960, 1517312}},
    {3, 2, 7, 6144, 19, 60, 4097, {1408512, 141568, 1615872, 1523712}},
    {3, 2, 7, 6144, 19, 60, 30000, {6730240, 461568, 7671808, 7570432}},
    {3, 2, 7, 6144, 19, 60, 1000000, {204859904, 12162048, 233021952, 232859904}},
    {3, 2, 7, 6144, 19, 60, 6291455, {1285686016, 75990016, 1462339328, 1461846784}},
    {2, 1, 4, 1024, 32, 8, 1, {92416, 14336, 107008, 92928}},
    {2, 1, 4, 1024, 32, 8, 1000, {557056, 29696, 594944, 577280}},
    {2, 1, 4, 1024, 32, 8, 4096, {1629184, 67072, 1729024, 1711104}},
    {2, 1, 4, 1024, 32, 8, 4097, {1634816, 67840, 1735680, 1717248}},
    {2, 1, 4, 1024, 32, 8, 30000, {10454528, 379648, 11074304, 11054592}},
    {2, 1, 4, 1024, 32, 8, 1000000, {340861184, 12080128, 360941312, 360861184}},
    {2, 1, 4, 1024, 32, 8, 6291455, {2143278592, 75908096, 2269518336, 2269107712}},
    {3, 1, 4, 700, 9, 12, 1, {74496, 9984, 84736, 75008}},
    {3, 1, 4, 700, 9, 12, 1000, {662528, 24320, 695040, 690688}},
    {3, 1, 4, 700, 9, 12, 4096, {2130688, 61184, 2224640, 2245376}},
    {3, 1, 4, 700, 9, 12, 4097, {2136320, 61952, 2231296, 2251520}},
    {3, 1, 4, 700, 9, 12, 30000, {14278912, 374016, 14893056, 15119104}},
    {3, 1, 4, 700, 9, 12, 1000000, {469088256, 12074496, 489162752, 497088256}},
    {3, 1, 4, 700, 9, 12, 6291455, {2950135040, 75902464, 3076369152, 3126295808}},
};

void budgets()
{
    for (const Asked &a : kAsked) {
        fpts_mesh m = shape(a.D, a.R, a.N, a.nel, a.NL, a.max_cell);
        for (int k = 0; k < 4; ++k) {
            if (kSizes[k].fn == fpts_lpt_workspace_size && a.R != a.D) continue;
            const size_t b = kSizes[k].fn(&m, a.n);
            int st = b <= a.bytes[k] ? FPTS_OK : FPTS_EINVAL;
            if (kSizes[k].fn == fpts_eval_workspace_size) {
                // no memory behind the addresses: nothing is launched
                void *p = reinterpret_cast<void *>(uintptr_t(1) << 40);
                st = fpts_eval(&m, a.n, (int32_t *)p, (int32_t *)p, (double *)p, 1, (double *)p,
                               (double *)p, p, a.bytes[k], nullptr);
            }
            if (st == FPTS_OK) continue;
            ++failures;
            std::printf("%s, D %d R %d N %d, %lld elements, %lld points: %zu bytes, had %zu\n",
                        kSizes[k].name, a.D, a.R, a.N, (long long)a.nel, (long long)a.n, b,
                        a.bytes[k]);
        }
    }
}

// The device setup's launches take fewer than 2^32 threads each, and enough
// together, for the most elements and cells that fpts_setup lets in.
void setup_launches(int64_t nel, int NL, int copies, uint64_t threads, uint64_t needed)
{
    fpts_mesh m = shape(2, 1, 2, nel, NL, 1);
    m.p.bbox_tol = 0.1;
    launches.clear();
    copies_back = copies;
    first_back = {0.0, 0.0, 1.0, 1.0};   // the union box
    (void)fpts::device_setup(&m, nullptr);
    uint64_t most = 0;
    for (const Launch &l : launches) {
        if (l.blocks * l.threads >= (uint64_t(1) << 32) || l.blocks > INT32_MAX) {
            ++failures;
            std::printf("%lld elements, %d^2 cells: a launch of %llu blocks of %llu threads\n",
                        (long long)nel, NL, (unsigned long long)l.blocks,
                        (unsigned long long)l.threads);
        }
        uint64_t sum = 0;   // of this kernel's launches
        for (const Launch &k : launches)
            if (k.kernel == l.kernel) sum += k.blocks * k.threads;
        if (l.threads == threads) most = sum > most ? sum : most;
    }
    if (most < needed) {
        ++failures;
        std::printf("%lld elements, %d^2 cells: %llu threads of %llu needed\n", (long long)nel, NL,
                    (unsigned long long)most, (unsigned long long)needed);
    }
}

void setups()
{
    // (the copy of the union box ends the first two)
    setup_launches((int64_t(1) << 26) + 77, 1, 0, 64, ((uint64_t(1) << 26) + 77) * 64);
    setup_launches(INT32_MAX / 2, 1, 0, 64, uint64_t(INT32_MAX / 2) * 64);
    setup_launches(5, 16400, 2, 256, uint64_t(16400) * 16400 * 16);
    setup_launches(5, 3, 2, 256, 9 * 16);
}

// Kernels of one-wave blocks divide their tasks among the XCDs: their grids are
// multiples of eight also on a device whose number of CUs is not.
void grids()
{
    void *p = reinterpret_cast<void *>(uintptr_t(1) << 40);
    const int kinds[][3] = {{3, 3, 6}, {3, 3, 8}, {2, 2, 5}, {3, 2, 7}, {3, 2, 10}, {2, 1, 4}};
    for (int cus : {256, 33, 19, 1})
        for (auto &k : kinds)
            for (int precision : {FPTS_FP64, FPTS_MIXED})
                for (int64_t n : {1, 1000, 3000000}) {
                    // (enough cells that no scan of them takes a block of one wave)
                    fpts_mesh m = shape(k[0], k[1], k[2], 5000, k[0] == 3 ? 18 : 80, 12);
                    m.cus = cus;
                    m.near_npad = (m.NP + 31) / 32 * 32;
                    m.p.max_iter = 50;
                    launches.clear();
                    const int st =
                        fpts_find_eval(&m, n, (double *)p, (int32_t *)p, (int32_t *)p, (double *)p,
                                       (double *)p, precision, 3, k[2], (double *)p, (double *)p, p,
                                       fpts_find_eval_workspace_size(&m, n), nullptr);
                    int waves = 0;
                    for (const Launch &l : launches) {
                        Dl_info info;
                        const bool named = dladdr(l.kernel, &info) && info.dli_sname;
                        // (a block per point, no division)
                        if (named && std::strstr(info.dli_sname, "overflow")) continue;
                        if (l.threads != 64) continue;
                        ++waves;
                        if (l.blocks % 8 == 0) continue;
                        ++failures;
                        std::printf("%d CUs, D %d R %d N %d, %lld points: %llu blocks of %s\n", cus,
                                    k[0], k[1], k[2], (long long)n, (unsigned long long)l.blocks,
                                    named ? info.dli_sname : "?");
                    }
                    if (st != FPTS_OK || waves < 4) {
                        ++failures;
                        std::printf("%d CUs, D %d R %d N %d, %lld points: status %d, %d launches of "
                                    "one-wave blocks\n",
                                    cus, k[0], k[1], k[2], (long long)n, st, waves);
                    }
                }
}

}  // namespace

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "sizes")) sizes();
    else if (!std::strcmp(what, "budgets")) budgets();
    else if (!std::strcmp(what, "setups")) setups();
    else if (!std::strcmp(what, "grids")) grids();
    else return 2;
    std::printf("%s: %d failures\n", what, failures);
    return failures != 0;
}
