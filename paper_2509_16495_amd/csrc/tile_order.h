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
// to meet every sequence is each of these 32 engines.  Which members of a run an engine gets repeats after four runs; the shift
// grows by five meanwhile, a number without a common factor with n_sh.  (By four alone, which is what one per run gives, an engine
// sees one sequence of n_sh == 4 only and two of n_sh == 8.)  Random unequal batches against one per run: 60 of n_sh 4 0.94 of the
// time, none slower, 0.62 at best (4305 + 2070 + 1321 + 5987 tokens, 8 heads 240 -> 141 us), 160 of n_sh 8 0.96 (14 more than 3 %
// slower, up to 13).  Beyond 8 an engine sees enough of them by one per run: every engine shown all gave nothing for 12 (160
// batches, 1.00) and 1.3 % more time for 16 (160, up to 1.34 times), 2 % beyond.
[[gnu::always_inline]] constexpr inline int rotation(int t, int n_sh) { return n_sh > 8 ? t : t + (t >> 2); }

// Workgroup `block` of a grid whose first `decode_wgs` workgroups take decode rows.  The ones behind them are runs of n_sh
// workgroups, one per (sequence, head), a run for every (rank, key range).  range_major: the key ranges outermost (launches
// that carry decode rows: their shorter last ranges start last, on the compute units that the decode rows leave), else the
// ranks.  rotate: rotate_sequences_over_dies() of the batch; the rotation is that of the run, whatever stands in front of it
// in the grid, so a run holds every (sequence, head) once.
// (inlined early and with the divisions in this order: other forms cost the kernels at the edge of the register file up to 30 more)
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
