// Checks the layout of tiled launches (mxr_tiles.h) on the host.  Reads lines
// "first n rows ratio"; prints "ok" or what is wrong, one line each.  Up to 2^22
// rays every tile and lane is walked and every ray counted; beyond that, rays
// from all over the range are looked for in the tile that has to hold them, and
// lanes all over the tiles have to hold rays of the range.
#include <cstdio>
#include <vector>

#include "mxr_tiles.h"

using namespace mxr;

static uint64_t state = 1;
static uint64_t draw(uint64_t below) {
    state += 0x9E3779B97F4A7C15ull;
    uint64_t z = (state ^ (state >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return (z ^ (z >> 31)) % below;
}

static const char *check(uint64_t first, uint64_t n, uint64_t rows, double ratio) {
    const uint32_t rounds = tile_rounds(n), turns = 4u << rounds;
    const TileRange r = tile_range(first, n, rows, ratio, rounds);
    if (row_start(r, 0) != first || row_start(r, (uint32_t)rows) != first + n) return "rows do not cover the range";
    if (r.tiles < n / (256u << rounds)) return "too few tiles";
    uint64_t id;
    if (n <= (1u << 22)) {
        std::vector<unsigned char> seen(n, 0);
        for (uint64_t t = 0; t < r.tiles; ++t) {
            const TileAt at = tile_at(r, rounds, t);
            for (uint32_t turn = 0; turn < turns; ++turn)
                for (uint32_t lane = 0; lane < 64; ++lane)
                    if (tile_ray(r, at, turn, lane, id)) {
                        if (id < first || id - first >= n) return "a ray outside the range";
                        if (seen[id - first]++) return "a ray twice";
                    }
        }
        for (unsigned char s : seen)
            if (!s) return "a ray left out";
        return "ok";
    }
    for (int k = 0; k < 20000; ++k) {
        const uint64_t want = first + (k < 5 ? k : k < 10 ? n - 1 - (k - 5) : draw(n));
        uint64_t row = (uint64_t)((double)(want - first) / (double)n * (double)rows);
        row = row < rows ? row : rows - 1;
        while (row + 1 < rows && row_start(r, (uint32_t)row + 1) <= want) ++row;
        while (row > 0 && row_start(r, (uint32_t)row) > want) --row;
        const uint64_t col = want - row_start(r, (uint32_t)row), per = (256u << rounds) >> r.ht;
        const uint64_t tile = (row >> r.ht) * r.cols + col / per;
        if (tile >= r.tiles) return "a ray left out";
        const TileAt at = tile_at(r, rounds, tile);
        const uint32_t wide = 64u >> r.hw, in_row = (uint32_t)(row - at.row0), in_col = (uint32_t)(col - at.col0);
        const uint32_t turn = (in_row >> r.hw) * (at.per_row / wide) + in_col / wide;
        const uint32_t lane = (in_row & ((1u << r.hw) - 1)) * wide + in_col % wide;
        if (!tile_ray(r, at, turn, lane, id) || id != want) return "a ray not where its tile is";
        const TileAt any = tile_at(r, rounds, draw(r.tiles));
        if (tile_ray(r, any, (uint32_t)draw(turns), (uint32_t)draw(64), id) && (id < first || id - first >= n))
            return "a ray outside the range";
    }
    return "ok";
}

int main() {
    unsigned long long first, n, rows;
    double ratio;
    while (std::scanf("%llu %llu %llu %lf", &first, &n, &rows, &ratio) == 4) std::printf("%s\n", check(first, n, rows, ratio));
    return 0;
}
