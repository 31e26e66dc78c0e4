// Host-only driver for the tile order test: csrc/tile_order.h, the text that the kernels and the host code run, built with the
// host compiler under the sanitizers.  Exit status 0 = every quotient, tile and slice as by plain division.
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "../../paper_2512_19018_amd/csrc/tile_order.h"

using namespace peak;

struct Order {
    int tiles_m, tiles_n, group_m;
    Divisor by_tiles, by_band, by_group, by_last;
};

static int failures = 0;
#define CHECK(c) do { if (!(c)) { if (failures++ < 10) fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); } } while (0)

static uint32_t g_rng = 12345;
static uint32_t next32()
{
    g_rng = g_rng * 1664525u + 1013904223u;
    const uint32_t hi = g_rng >> 16;
    g_rng = g_rng * 1664525u + 1013904223u;
    return hi << 16 | g_rng >> 16;
}

static void check_division(uint32_t n, int d) { CHECK(quotient(n, divisor(d)) == (int)(n / (uint32_t)d)); }

// tile of position L by plain division
static void plain(const Order &o, int64_t L, int &tm, int &tn)
{
    const int64_t band = (int64_t)o.group_m * o.tiles_n, g = L / band, first = g * o.group_m;
    const int64_t rows = o.tiles_m - first < o.group_m ? o.tiles_m - first : o.group_m;
    tm = (int)(first + (L - g * band) % rows);
    tn = (int)((L - g * band) / rows);
}

int main()
{
    const uint32_t top = 0x7FFFFFFF;                        // workgroups of a launch, at most
    std::vector<int> divisors = {1, 2, 3, 4, 7, 8, 255, 256, 65535, 65536, 65537, 1 << 30, 0x7FFFFFFE, 0x7FFFFFFF};
    for (int i = 0; i < 20000; ++i) divisors.push_back(1 + (int)(next32() >> (1 + next32() % 31)) % 0x7FFFFFFF);
    for (int d : divisors) {
        const uint32_t u = (uint32_t)d, whole = top / u * u;
        for (uint32_t n : {0u, 1u, u - 1, u, whole - 1, whole, top - 1, top, next32() >> 1}) if (n <= top) check_division(n, d);
        if (u <= top / 2) { check_division(2 * u - 1, d); check_division(2 * u, d); }
    }

    // small grids: every tile of every slice once, in the order of plain division, on all XCDs' runs together
    for (int tiles_m = 1; tiles_m <= 21; ++tiles_m)
        for (int tiles_n : {1, 2, 3, 5, 8, 13, 16, 17, 31})
            for (int group_m : {1, 4, 8})
                for (int split : {1, 2, 3, 7}) {
                    if (group_m > tiles_m) continue;
                    Order o;
                    set_tile_order(o, tiles_m, tiles_n, group_m);
                    const int tiles = tiles_m * tiles_n;
                    std::vector<int> seen((size_t)tiles * split, 0);
                    for (int block = 0; block < tiles * split; ++block) {
                        const int pos = order_of_block(block, tiles * split);
                        CHECK(pos >= 0 && pos < tiles * split);
                        const int slice = quotient((uint32_t)pos, o.by_tiles);
                        int tm = -1, tn = -1, pm, pn;
                        tile_in_order(o, pos - slice * tiles, tm, tn);
                        plain(o, pos - slice * tiles, pm, pn);
                        CHECK(slice == pos / tiles && tm == pm && tn == pn);
                        if (slice >= 0 && slice < split && tm >= 0 && tm < tiles_m && tn >= 0 && tn < tiles_n) ++seen[((size_t)slice * tiles_m + tm) * tiles_n + tn];
                    }
                    for (int n : seen) CHECK(n == 1);
                }

    // grids up to the limit of a launch: positions at the edges of bands and slices, and anywhere
    const int shapes[][4] = {{1, 0x7FFFFFFF, 1, 1}, {0x7FFFFFFF, 1, 8, 1}, {46340, 46340, 8, 1}, {46341, 46340, 4, 1}, {64, 33554431, 64, 1},
                             {8191, 262143, 8, 1}, {4097, 32768, 4, 15}, {16777216, 2, 8, 63}, {3, 11184810, 3, 64}, {1073741823, 2, 4, 1}};
    for (const int *s : shapes) {
        Order o;
        set_tile_order(o, s[0], s[1], s[2]);
        const int64_t tiles = (int64_t)s[0] * s[1], total = tiles * s[3], band = (int64_t)s[2] * s[1];
        CHECK(total <= (int64_t)top);
        for (int i = 0; i < 4000; ++i) {
            int64_t pos = i % 4 == 0 ? (int64_t)(next32() % (uint32_t)total) : i % 4 == 1 ? next32() % (uint32_t)(tiles / band + 1) * band - i % 3
                        : i % 4 == 2 ? total - 1 - i : (int64_t)(next32() % (uint32_t)s[3]) * tiles - i % 2;
            if (pos < 0 || pos >= total) continue;
            const int slice = quotient((uint32_t)pos, o.by_tiles);
            CHECK(slice == (int)(pos / tiles));
            int tm, tn, pm, pn;
            tile_in_order(o, (int)(pos - (int64_t)slice * tiles), tm, tn);
            plain(o, pos - (int64_t)slice * tiles, pm, pn);
            CHECK(tm == pm && tn == pn);
        }
    }
    if (failures) { fprintf(stderr, "%d checks failed\n", failures); return 1; }
    printf("tile order clean\n");
    return 0;
}
