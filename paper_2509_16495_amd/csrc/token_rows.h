// Which token rows the projection kernel's loads fetch for an output tile.  Nothing of HIP in here: the kernel and a host test
// that walks the tiles share the functions.
#pragma once

namespace shiftattn {

// A tile covers token rows m0 and following of a result with rows past the last of the M >= 1 tokens (padding rows, written as
// zeros); a tile may lie wholly among those.  Its loads count from tile_origin(), a row that exists, and row `row` of the tile
// fetches tile_row() rows behind it (never before it: the loads add it as an unsigned offset); rows past the last one fetch
// the last one once more.
constexpr int tile_origin(int m0, int M) { return m0 < M - 1 ? m0 : M - 1; }
constexpr int tile_row(int m0, int row, int M) { return (m0 + row < M - 1 ? m0 + row : M - 1) - tile_origin(m0, M); }

}  // namespace shiftattn
