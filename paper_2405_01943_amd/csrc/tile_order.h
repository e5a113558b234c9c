// Which output tile a workgroup of the matrix-core kernels (calib.hip, sparse_down.hip) computes, and how
// large the tiles are.
//
// Consecutive workgroup ids go to different XCDs (8 of them, each with its own L2), and an XCD
// runs about 32 of these workgroups at a time, one per compute unit.  Tiles that share rows of X
// or of W should therefore run on one XCD at one time, and every XCD should get the same number of
// tiles.  Two orders:
//
//   runs (band > 0)   every XCD takes one contiguous run of ceil(N / 8) tiles of a list in which the
//       token tiles are cut into bands of at most 4 (8: max_band) and a band's tiles are listed column of
//       tiles by column of tiles, so 32 neighbours of the list are about a 4 x 8 patch.  The XCDs get equal
//       shares whatever the shape of the grid.
//   patches (band = 0)   the grid is cut into patches of 4 token tiles x 8 column tiles, each taken
//       by one XCD (its L2 serves 13/16 of their reads), and the patches are dealt round-robin from a
//       list whose neighbours share data in the memory-side cache:
//         super_rows = 1: token-major.  The 8 patches in flight lie in one row of patches: X is
//           fetched from HBM by one XCD and found in that cache by the others, and the weights stay
//           cached from one row to the next as long as they fit (+5 % over one band of columns per XCD).
//         super_rows = R > 1, for weights too large to stay cached: R rows of patches at a time, the
//           patch columns outermost.  The patches in flight share a column of the weights, fetched
//           once per super-row, whose X (R x 8 MB at d = 4096) stays cached meanwhile (+7 % at 8192
//           x 28672).  The rows of patches are split evenly over the super-rows: a last super-row of
//           one or two rows left most XCDs without work.
//       A whole patch is a whole round of an XCD, so a grid of few patches leaves XCDs idle.
#pragma once

#include <cstdint>

namespace dass {

struct TileOrder {
    uint32_t tiles_t, tiles_n;   // the grid of tiles
    uint32_t band;               // > 0: runs, bands of this many token tiles; 0: patches
    uint32_t per_xcd;            // runs: tiles of one XCD
    uint32_t super_rows;         // patches: rows of patches taken together
    uint32_t blocks;             // workgroups to launch; 0: more than one launch can hold
};

constexpr uint32_t kPatchT = 4, kPatchN = 8, kXcds = 8, kXcdSlots = kPatchT * kPatchN;

// False: this workgroup has no tile.
__device__ __forceinline__ bool tile_of_block(const TileOrder &o, uint32_t block, uint32_t &tile_t, uint32_t &tile_n)
{
    const uint32_t xcd = block % kXcds, idx = block / kXcds;
    if (o.band > 0) {
        const uint32_t lin = xcd * o.per_xcd + idx;
        if (lin >= o.tiles_t * o.tiles_n)
            return false;
        const uint32_t per_band = o.band * o.tiles_n, b = lin / per_band, rem = lin - b * per_band;
        const uint32_t left = o.tiles_t - b * o.band, rows = left < o.band ? left : o.band;
        tile_n = rem / rows;
        tile_t = b * o.band + (rem - tile_n * rows);
        return true;
    }
    const uint32_t np_t = (o.tiles_t + kPatchT - 1) / kPatchT, np_n = (o.tiles_n + kPatchN - 1) / kPatchN;
    const uint32_t patch = idx / kXcdSlots * kXcds + xcd, within = idx % kXcdSlots;
    const uint32_t per_super = np_n * o.super_rows, sr = patch / per_super, rem = patch - sr * per_super;
    if (sr * o.super_rows >= np_t)
        return false;
    const uint32_t left = np_t - sr * o.super_rows, rows = left < o.super_rows ? left : o.super_rows;
    const uint32_t pcol = rem / rows, prow = sr * o.super_rows + (rem - pcol * rows);
    tile_t = prow * kPatchT + within / kPatchN;
    tile_n = pcol * kPatchN + within % kPatchN;
    return pcol < np_n && tile_t < o.tiles_t && tile_n < o.tiles_n;
}

// Runs up to this many tiles (16 rounds of the chip).  Measured on calib_pipe64_kernel, patches -> runs:
// 6 x 192 tiles 1390 us (super-rows of 8: two of the eight XCDs had work) -> 345, 366 with even
// super-rows; 2 x 86 tiles 87 -> 75 us, 4 x 86 170 -> 157; the plain product with 4 x 16 tiles 251 -> 207 us;
// from about 1000 tiles on either order is within 2.5 % (12 x 86 and 24 x 86 tiles patches 2 % ahead, 12 x 112 and
// 24 x 112 even), with two exceptions: an even number of patch columns of which the last is not whole gives
// the XCDs of one parity all the short patches (12 column tiles, 128 token tiles: 4.6 ms against 3.6), and grids
// narrower than a patch leave most of every patch empty (calib_f32_kernel, 4096 x 1 tiles: 320 us against 127).
constexpr int64_t kRunTiles = 4096;

// weights_cached: the operand that the column tiles read fits the 256 MB memory-side cache.
// max_band: token tiles of a band (runs).  8 for tiles half as high as they are wide, so that 32 neighbours
// stay a square: down projection of 2048 tokens of 4096 x 11008 by 128 x 256 tiles 451 -> 439 us (whole
// dass_mlp_forward), by the sparse kernel 169 -> 162 us with the compression.
// run_tiles: runs up to so many tiles.
inline TileOrder make_tile_order(int64_t tiles_t, int64_t tiles_n, bool weights_cached, int64_t max_band = kPatchT,
                                 int64_t run_tiles = kRunTiles)
{
    TileOrder o = {0, 0, 0, 0, 0, 0};
    const int64_t np_t = (tiles_t + kPatchT - 1) / kPatchT, np_n = (tiles_n + kPatchN - 1) / kPatchN;
    const int64_t n = tiles_t * tiles_n, patches = np_t * np_n;
    const bool short_patches_meet = weights_cached && tiles_n % kPatchN != 0 && np_n % 2 == 0;
    // Whole patches that go round evenly leave no XCD idle, and are then ahead, on weights that stay cached and on
    // others.  Taken in turn, patches against runs: stage 1 with d = 4096, 16 to 32 x 64 tiles 0.7 to 1.4 %, 12 to 20 x
    // 128 0.7 to 1.2 %, 16 x 112 0.6 %; uncached 8 to 20 x 192 (d = 3072) 0.8 to 1.5 %, 8 and 16 x 224 0.5 %, with d =
    // 8192 1.4 and 0.3 %; dass_mlp_forward of 16384 to 32768 tokens of 4096 x 14336 0.2 to 0.8 %, but of 8192 x 8192
    // 2 % behind.
    const bool even_patches = n > 1024 && tiles_t % kPatchT == 0 && tiles_n % kPatchN == 0 && patches % kXcds == 0;
    const bool runs = (n <= run_tiles && !even_patches) || short_patches_meet || tiles_n < kPatchN;
    const int64_t blocks = runs ? (n + kXcds - 1) / kXcds * kXcds : (patches + kXcds - 1) / kXcds * kXcds * kXcdSlots;
    if (blocks > 0x7fffffffLL)
        return o;
    o.tiles_t = (uint32_t)tiles_t;
    o.tiles_n = (uint32_t)tiles_n;
    o.blocks = (uint32_t)blocks;
    if (runs) {
        const int64_t bands = (tiles_t + max_band - 1) / max_band;
        o.band = (uint32_t)((tiles_t + bands - 1) / bands);   // even bands of at most max_band
        o.per_xcd = (uint32_t)((n + kXcds - 1) / kXcds);
    } else {
        const int64_t supers = weights_cached ? np_t : (np_t + 7) / 8;
        o.super_rows = (uint32_t)((np_t + supers - 1) / supers);
    }
    return o;
}

// The tile of a workgroup.  It fills a compute unit, and on grids that do not run for many rounds a slab of
// K takes about as long as its rows take to load, so a shape's time goes as rounds x bytes of a tile's slab.
// Large tiles load least in all and win wherever they fill the chip; small ones win where large ones leave
// compute units idle.
struct TileShape {
    int which;   // 0: the largest, 1: half as many tokens, 2: half of both
    int64_t tiles_t, tiles_n;
};

// tokens, cols: of the three tiles; token_bytes, col_bytes: of a slab, in any unit
inline TileShape cheapest_tile(int64_t T, int64_t n, const int (&tokens)[3], const int (&cols)[3], int token_bytes, int col_bytes)
{
    TileShape best = {0, 0, 0};
    int64_t best_cost = 0;
    for (int k = 0; k < 3; ++k) {
        const TileShape s = {k, (T + tokens[k] - 1) / tokens[k], (n + cols[k] - 1) / cols[k]};
        const int64_t cost = (s.tiles_t * s.tiles_n + 255) / 256 * (tokens[k] * token_bytes + cols[k] * col_bytes);
        if (k == 0 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

// calib_pipe64_kernel for T tokens and n output columns (of each of two matrices for the gated forms, so
// their tiles are half as wide in columns).  256 x 256 against the tile chosen here, whole calls, back to back:
// dass_mlp_forward 128 tokens of 1024 x 4096 98 -> 40 us, 1024 of 4096 x 11008 (64 tiles in the down
// projection) 362 -> 271, 2048 of it (128 tiles) 465 -> 430; dass_calib_norms 300 of 4096 x 1024 73 -> 29, 1024 of 4096 x
// 4096 75 -> 55.  256 x 256 chosen and, in brackets, half as many tokens: 512 of 4096 x 11008 81 (94), 1024 of 4096 x
// 8192 95 (104), 2048 of 4096 x 8192 182 (203); but where its second round is nearly empty the smaller tile is ahead by
// now: 1024 of 4096 x 11008 160 (144), 2048 of 4096 x 5632 159 (143), 3000 of 2048 x 5632 131 (127).
inline TileShape dense_tile_shape(int64_t T, int64_t n, bool gated)
{
    return gated ? cheapest_tile(T, n, {256, 128, 128}, {128, 128, 64}, 1, 2)
                 : cheapest_tile(T, n, {256, 128, 128}, {256, 256, 128}, 1, 1);
}

// down_sparse24_kernel: 64 bytes a feature, 128 a token.  256 x 256 against the tile chosen here, back to back: 2048
// tokens of 4096 x 11008 (128 tiles) 162 -> 107 us, 1024 of it 155 -> 70, 4096 of 2048 x 5632 90 -> 58, 128 of 1024 x
// 4096 58 -> 23.  256 x 256 chosen and, in brackets, half as many tokens: 4096 of 4096 x 11008 (256 tiles) 200 (212), 8192
// of 2048 x 5632 109 (118), 3000 of 4096 x 11008 172 (190); but 6000 of it, whose second round is half empty, 353 (306).
inline TileShape sparse_tile_shape(int64_t T, int64_t d)
{
    return cheapest_tile(T, d, {256, 128, 128}, {256, 256, 128}, 2, 1);
}

}  // namespace dass
