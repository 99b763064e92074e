// Which outputs a lane of forward_direct_kernel holds and where their partial sums lie in LDS (plain C++: also
// compiled on the host).
//
// A tile is LPS lanes of T outputs.  Lane l of a tile writes its T sums to its own slots l * T .. l * T + T - 1, so every
// slot has one writer and none lies outside the tile.  What the slots hold: the outputs from direct_first_output on.
// That is the lane's place in the row, l * T after the tile's first output, except in the lane whose T outputs would run
// past the row's end (n_out no multiple of T): it holds n_out - T .. n_out - 1, which may start before the tile.
#pragma once

// first output of the lane whose place in the row is `place` (0: a lane past the row, whose results are dropped)
constexpr int direct_first_output(int place, int T, int n_out)
{
    return place >= n_out ? 0 : (place + T > n_out ? n_out - T : place);
}

// slot of output `out` (out < n_out) of the tile that starts at output `tile0`
constexpr int direct_slot(int out, int tile0, int T, int n_out)
{
    const int lane0 = (out - tile0) / T * T;                             // the slots of the lane that has it
    return lane0 + (out - direct_first_output(tile0 + lane0, T, n_out));
}
