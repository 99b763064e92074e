// Layout of the split coefficient table of the matrix-core forward kernel (kan_matrix.hip), host and device.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace kan {

constexpr int kMxInputs = 4;       // inputs of one step
constexpr int kMxTile = 32;        // outputs of one tile
constexpr int kMxSplits = 3;       // bf16 parts of a float
constexpr int kMxMaxGroups = 12;

// Groups of four positions an input's rows + 1 table rows (the last one w_b) are dealt to; even, so that the groups of a step
// fill whole instructions of eight; at least as many as a window has rows, so that no two rows of a window share a group.
constexpr int mx_groups(int rows, int window)
{
    const int n = (rows + 1 + 7) / 8 * 2, least = (window + 1) / 2 * 2;
    return n < least ? least : n;
}

// Scratch that the kernel can count on where a call brings none of its own: a tile's part of the table has to fit there if the
// folded table does, so that such a call takes the same kernel.
constexpr size_t kMxScratch = 32u << 20;

struct MatrixTable {
    int groups;            // per input; 0: the shape does not qualify
    int n_steps, n_tiles;
    size_t tile_bytes;     // B operands of one tile of outputs, [tile][step][groups / 2][split][half][lane] x 16 bytes
    size_t bytes;          // all tiles, and one word per (tile, step): the part holds values the splits cannot carry
};

inline MatrixTable matrix_table(int n_in, int n_out, int rows, int window)
{
    MatrixTable t = {};
    t.groups = mx_groups(rows, window);
    t.n_steps = (n_in + kMxInputs - 1) / kMxInputs;
    t.n_tiles = (n_out + kMxTile - 1) / kMxTile;
    if (rows < window || n_in < 8 || n_out <= 64 || n_out > 1 << 20 || t.groups > kMxMaxGroups ||
        (int64_t)t.n_steps * t.n_tiles * 32 * t.groups >= 1ll << 31)        // (threads of the launch that splits the table)
        return MatrixTable{};
    t.tile_bytes = (size_t)t.n_steps * (t.groups / 2) * kMxSplits * 2048;
    t.bytes = (t.n_tiles * (t.tile_bytes + (size_t)t.n_steps * 4) + 255) / 256 * 256;
    if (t.tile_bytes + (size_t)t.n_steps * 4 > kMxScratch && (size_t)n_in * (rows + 1) * n_out * 4 <= kMxScratch) return MatrixTable{};
    return t;
}

}  // namespace kan
