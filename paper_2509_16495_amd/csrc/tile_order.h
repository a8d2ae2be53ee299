// Which tile, key range and (sequence, head) a workgroup of the prefill kernels takes.  Nothing of HIP in here: the kernels
// and a host test that walks whole grids share the function.
#pragma once

namespace shiftattn {

struct TileItem {
    int rank;   // tile (or pair of tiles) of the sequence
    int split;  // key range
    int sh;     // (sequence, head) index
};

// Workgroup `block` of a grid whose first `decode_wgs` workgroups take decode rows.  The ones behind them are runs of n_sh
// workgroups, one per (sequence, head), a run for every (rank, key range).  range_major: the key ranges outermost (launches
// that carry decode rows: their shorter last ranges start last, on the compute units that the decode rows leave), else the
// ranks.  rotate: rotate_sequences_over_dies() of the batch; the rotation is that of the run, whatever stands in front of it
// in the grid, so a run holds every (sequence, head) once.
// (inlined early and with the divisions in this order: other forms leave the 256-column kernel up to 30 more spilled registers)
[[gnu::always_inline]] constexpr inline TileItem tile_item(int block, int decode_wgs, int n_sh, int ranks, int n_splits,
                                                           bool range_major, bool rotate) {
    const int wg = block - decode_wgs;
    const int per_outer = n_sh * (range_major ? ranks : n_splits), outer = wg / per_outer;
    const int inner = (wg - outer * per_outer) / n_sh;
    int sh = wg - outer * per_outer - inner * n_sh;   // wg - sh: the run times n_sh
    if (rotate) sh = (sh + n_sh - (wg - sh) / (n_sh < 8 ? 8 : n_sh) % n_sh) % n_sh;
    return range_major ? TileItem{inner, outer, sh} : TileItem{outer, inner, sh};
}

}  // namespace shiftattn
