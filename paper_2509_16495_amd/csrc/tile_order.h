// Which tile, key range and (sequence, head) a workgroup of the prefill kernels takes.  Nothing of HIP in here: the kernels
// and a host test that walks whole grids share the function.
#pragma once

namespace shiftattn {

struct TileItem {
    int rank;   // tile (or pair of tiles) of the sequence
    int split;  // key range
    int sh;     // (sequence, head) index
};

// By how much the (sequence, head) index of run `t` of a rotated launch is shifted (runs of n_sh workgroups, for n_sh == 4 pairs of
// them).  The dispatcher hands workgroup i to die i % 8 and there to shader engine (i / 8) % 4, whatever else is free, so what has
// to meet every sequence is each of these 32 engines.  Which members of a run an engine gets repeats after `period` runs; the shift
// grows by `period` + `extra` meanwhile, a number without a common factor with n_sh.  (By `period` alone, which is what one per
// run gives, an engine sees one sequence of n_sh == 4 only and one in four (sequence, head) of n_sh == 8.)  130 random batches of
// two to twelve chunks against one per run: n_sh 4 1.13 times on average, 1.7 at most (4305 + 2070 + 1321 + 5987 tokens, 8 heads
// 240 -> 141 us), 8 1.07, 12 1.03; beyond 16 an engine sees enough of them anyway (2 % slower with it).
[[gnu::always_inline]] constexpr inline int rotation(int t, int n_sh) {
    const int lg = n_sh == 16 ? 1 : n_sh == 12 ? 3 : 2, extra = n_sh > 16 ? 0 : n_sh == 12 ? 3 : 1;
    return t + extra * (t >> lg);
}

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
    if (rotate) sh = (sh + n_sh - rotation((wg - sh) / (n_sh < 8 ? 8 : n_sh), n_sh) % n_sh) % n_sh;
    return range_major ? TileItem{inner, outer, sh} : TileItem{outer, inner, sh};
}

}  // namespace shiftattn
