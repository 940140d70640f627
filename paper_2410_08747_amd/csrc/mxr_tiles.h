// mxr_tiles.h -- how a tiled launch's rays are laid out: the arithmetic that
// takes a tile and a lane to a ray id, and its host-side plan.  Plain C++, for
// the kernels and for programs that check the layout without a device.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#if defined(__HIPCC__)
#define MXR_HD __host__ __device__ __forceinline__
#else
#define MXR_HD inline
#endif

namespace mxr {

// floor(x / d) from the rounded estimate x * rd (rd = 1/d rounded), for a
// quotient below 2^32 and at most q_max with q_max d < 2^64: the estimate's
// relative error is a few 2^-53, so it lies within 1 of the quotient, and
// one product decides a step down or up.
MXR_HD uint64_t div_est(uint64_t x, uint64_t d, double rd, uint64_t q_max) {
    uint64_t q = (uint64_t)((double)x * rd);
    q = q > q_max ? q_max : q;
    const uint64_t p = q * d;
    if (p > x) q -= 1;
    else if (x - p >= d) q += 1;
    return q;
}

// Rays [first, first + n) of a tiled launch, laid out in `rows` rows of
// consecutive ids: row r begins at first + ceil(r n / rows).  The rows of a
// stratified range are its rows of cells, so the rays at one place of
// neighbouring rows leave in neighbouring directions.  A tile is 2^ht rows of
// (tile rays >> ht) ids each; the tiles run along the rows first, `cols` to a
// block of rows.  A wave takes 2^hw rows of 64 >> hw ids at a time.  A range of
// one row has as many columns as tiles, so they are counted with 64 bits: a run
// may take any number of rays.
struct TileRange {
    uint64_t first, n, q, tiles;  // q = n / rows; tiles of this range
    uint64_t cols;
    uint32_t rows, rem;           // rem = n mod rows
    uint32_t ht, hw;
    double r_rows, r_cols;        // 1 / rows, 1 / cols, rounded
};

// A tile of a range: its first row, its first place in a row and its ids per row.
struct TileAt {
    uint64_t block, col0;
    uint32_t row0, per_row;
};

MXR_HD TileAt tile_at(const TileRange &r, uint32_t rounds, uint64_t tile) {
    TileAt t;
    t.per_row = (256u << rounds) >> r.ht;
    t.block = div_est(tile, r.cols, r.r_cols, r.rows);
    t.col0 = (tile - t.block * r.cols) * t.per_row;
    t.row0 = (uint32_t)(t.block << r.ht);
    return t;
}

// First ray id of a row.
MXR_HD uint64_t row_start(const TileRange &r, uint32_t row) {
    const uint64_t x = (uint64_t)row * r.rem + r.rows - 1;
    return r.first + (uint64_t)row * r.q + div_est(x, r.rows, r.r_rows, r.rows);
}

// The ray of a lane in the turn-th wave's worth of a tile's rays (false: none;
// the lane then holds the range's first id).
MXR_HD bool tile_ray(const TileRange &r, const TileAt &t, uint32_t turn, uint32_t lane, uint64_t &ray_id) {
    const uint32_t wide = 64u >> r.hw;          // ids of a wave's row
    const uint32_t across = t.per_row / wide;   // waves side by side in a tile
    const uint32_t row = t.row0 + ((turn / across) << r.hw) + lane / wide;
    const uint64_t col = t.col0 + (turn % across) * wide + lane % wide;
    const bool in = row < r.rows;
    const uint64_t at = row_start(r, in ? row : 0);
    const uint64_t len = in ? row_start(r, row + 1) - at : 0;
    const bool live = col < len;
    ray_id = live ? at + col : r.first;
    return live;
}

// Rounds of a tile (256 << rounds rays) in a run of n: as many (at most 16
// times 256 rays) as leave 16,384 tiles, some 16 to a work-group's place on the
// chip (of a plain cone's tiles 70 % end at once).
inline uint32_t tile_rounds(uint64_t n) {
    uint32_t rounds = 0;
    while (rounds < 4 && (n >> (8 + 14 + rounds + 1)) > 0) ++rounds;
    return rounds;
}

// Layout of n > 0 rays in rows.  Rows per tile and per wave make both about
// square on the monitor: a cell holds c rays, so a wave covers 64 / c cells,
// `ratio` times as wide as high in a proposal's components.
inline TileRange tile_range(uint64_t first, uint64_t n, uint64_t rows, double ratio, uint32_t rounds) {
    auto log2_of = [](double x, uint32_t most) {
        uint32_t l = 0;
        while (l < most && x > 1.4142 * (double)(1u << l)) ++l;
        return l;
    };
    TileRange r{};
    r.first = first;
    r.n = n;
    r.rows = (uint32_t)rows;
    r.q = n / rows;
    r.rem = (uint32_t)(n % rows);
    r.r_rows = 1.0 / (double)rows;
    const double c = (double)n / ((double)rows * (double)rows);
    uint32_t most = 0;  // at most all rows, and at least 8 ids of a row per wave
    while (most < 3 && (2ull << most) <= rows) ++most;
    r.hw = rows > 1 ? log2_of(std::sqrt(64.0 / c * ratio), most) : 0;
    most = r.hw;
    while (most < r.hw + 2 + rounds && (2ull << most) <= rows) ++most;
    r.ht = rows > 1 ? std::max(r.hw, log2_of(std::sqrt((double)(256u << rounds) / c * ratio), most)) : 0;
    const uint64_t per_row = (256u << rounds) >> r.ht, len = r.q + (r.rem ? 1 : 0);
    r.cols = (len - 1) / per_row + 1;
    r.r_cols = 1.0 / (double)r.cols;
    r.tiles = r.cols * ((rows + (1ull << r.ht) - 1) >> r.ht);
    return r;
}

}  // namespace mxr
