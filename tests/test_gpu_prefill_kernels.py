"""The tuned prefill kernels against the fp64 oracle: tiles of 128 columns in 32-column wavefronts, tiles of 256 in 64-column ones, and
tiles of 128 in two groups of those.  shiftattn_set_option forces the columns of a tile; which of the two 128-column kernels takes a
launch is the planner's choice, so the tests that aim at one choose batches for which it does and ask shiftattn_prefill_plan.

Tolerances as for all bf16 attention: max |err| <= 2e-2 and mean |err| <= 1e-3 against the oracle.
"""
import numpy as np
import pytest

from paper_2509_16495_amd import workloads as W

pytestmark = pytest.mark.gpu

BF16_MAX, BF16_MEAN = 2e-2, 1e-3


@pytest.fixture(scope="module")
def G():
    import gpu_backend
    return gpu_backend


@pytest.fixture
def opts():
    """Sets tuning switches for one test and puts them back to 'decided per call'."""
    from paper_2509_16495_amd import binding as B

    def set_(tile=0, splits=0, pairing=0, scaled_q=0):
        B.set_option(B.OPT_PREFILL_TILE, tile)
        B.set_option(B.OPT_PREFILL_SPLITS, splits)
        B.set_option(B.OPT_PREFILL_PAIRING, pairing)
        B.set_option(B.OPT_PREFILL_SCALED_Q, scaled_q)

    yield set_
    B.set_option(B.OPT_PREFILL_TILE, 0)
    B.set_option(B.OPT_PREFILL_SPLITS, 0)
    B.set_option(B.OPT_PREFILL_PAIRING, 0)
    B.set_option(B.OPT_PREFILL_SCALED_Q, 0)


def _takes(G, case, tile, wave, splits=None, per_wg=None):
    """Asserts which kernel, and how many key ranges and tiles per workgroup, a prefill call on the case takes."""
    p = G.launch_of(case)
    assert (p.tile_columns, p.wave_columns) == (tile, wave)
    assert splits in (None, p.key_ranges) and per_wg in (None, p.tiles_per_wg), (p.key_ranges, p.tiles_per_wg)


# a sequence that makes the two-group form the cheaper 128-column kernel for any batch it joins
LONG = (3, 9000)


def _check(got_bits, want):
    got = W.to_f64(got_bits, "bf16")
    assert got.shape == want.shape
    assert np.all(np.isfinite(got))
    err = np.abs(got - want)
    assert err.max() <= BF16_MAX and err.mean() <= BF16_MEAN, (err.max(), err.mean())


SHAPES = [
    # seqs (q_len, ctx), hq_l, hkv_l
    ([(200, 200), (77, 300), (1, 50), (130, 130)], 8, 1),   # several tiles, ragged tails, chunked, a one-token chunk
    ([(64, 64), (33, 33), (16, 16)], 4, 1),
    ([(150, 150), (5, 260)], 8, 2),                          # two KV heads
    ([(100, 100)], 4, 4),                                    # no GQA sharing: 256 tokens per wide tile
    ([(90, 190)], 6, 2),                                     # three query heads per KV head
    ([(300, 300)], 16, 1),
    ([(0, 10), (40, 40), (0, 0)], 4, 1),                     # empty chunks in the batch
    ([(140, 140), (31, 333)], 5, 1),                         # 40q/8kv model on 8 ranks (Table 4): 51 tokens per wide tile
    ([(129, 200)], 10, 2),
    ([(700, 700)], 8, 1),                                    # 22 wide tiles: pairs, a middle tile on its own
    ([(513, 1100), (31, 31), (257, 257)], 8, 1),             # several sequences of unequal tile counts
    ([(40, 4000)], 7, 1),                                    # 36 tokens per wide tile, long cached context
    # short chunks behind long contexts (longest context >= 16 x longest chunk): the wide kernel takes one tile per
    # workgroup instead of pairs; sequences of 4, 1, 3 and 0 tiles, one of them a prefill from nothing
    ([(100, 2100), (31, 31), (70, 1200), (0, 5)], 8, 1),
    ([(65, 1100), (64, 1040)], 8, 2),
]


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("splits", [0, 3])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", SHAPES)
def test_prefill_kernel_forced(oracle, G, opts, tile, splits, seqs, hq_l, hkv_l):
    from paper_2509_16495_amd import binding as B
    opts(tile=tile, splits=splits)
    assert B.get_option(B.OPT_PREFILL_TILE) == tile and B.get_option(B.OPT_PREFILL_SPLITS) == splits
    case = W.make_attn_case("t", 91, "bf16", seqs, hq_l, hkv_l, 128)
    _takes(G, case, tile, tile // 4, splits or None)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF))   # unwritten slots hold NaN patterns
    _check(got, want)


@pytest.mark.parametrize("pairing", [1, 2])
@pytest.mark.parametrize("splits", [0, 2])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", SHAPES)
def test_wide_prefill_kernel_tiles_in_pairs_and_one_per_workgroup(oracle, G, opts, pairing, splits, seqs, hq_l, hkv_l):
    """The 256-column kernel with its tiles forced two per workgroup (heaviest with lightest) and one per workgroup
    (heaviest first), whatever the planner would choose for the shape."""
    opts(tile=256, splits=splits, pairing=pairing)
    case = W.make_attn_case("t", 93, "bf16", seqs, hq_l, hkv_l, 128)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF))
    _check(got, want)


@pytest.mark.parametrize("splits", [0, 3])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", SHAPES)
def test_wide_prefill_kernel_on_scaled_q(oracle, G, opts, splits, seqs, hq_l, hkv_l):
    """The 256-column kernel with SHIFTATTN_OPT_PREFILL_SCALED_Q (off by default): Q takes the softmax scale when a tile
    fetches it and is rounded to bf16 again, which moves a logit by up to 2^-9 of its value.  An output may then land one
    bf16 step (at most 2^-7 of its magnitude) from the correctly rounded value, so the bound on the largest error is the
    usual one plus that step; the bound on the mean error is the usual one."""
    opts(tile=256, splits=splits, scaled_q=1)
    case = W.make_attn_case("t", 95, "bf16", seqs, hq_l, hkv_l, 128)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = W.to_f64(G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF)), "bf16")
    assert got.shape == want.shape and np.all(np.isfinite(got))
    err = np.abs(got - want)
    assert np.all(err <= BF16_MAX + 2.0 ** -7 * np.abs(want)) and err.mean() <= BF16_MEAN, (err.max(), err.mean())


@pytest.mark.parametrize("tile", [128, 256])
def test_prefill_fused_append_and_fp8_cache_forced(oracle, G, opts, tile):
    from paper_2509_16495_amd import binding as B
    opts(tile=tile)
    case = W.make_attn_case("t", 92, "bf16", [(70, 170), (128, 128), (1, 40), (300, 900)], 8, 1, 128)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    cache = G.cache_for_case(case, only_cached=True)
    _check(G.prefill_case(case, cache, fused_new_kv=True), want)
    assert B.to_host(cache).tobytes() == oracle.cache_for_case(case).tobytes()
    scales = (0.0371, 0.0293)
    ocache = oracle.cache_for_case(case, fp8_scales=scales)
    want = oracle.attention_case(case, ocache, k_scale=scales[0], v_scale=scales[1])
    cache = G.cache_for_case(case, only_cached=True, fp8_scales=scales)
    _check(G.prefill_case(case, cache, fused_new_kv=True, fp8_scales=scales), want)
    assert B.to_host(cache).tobytes() == ocache.tobytes()


def _with_late_outliers(case, rows, key_positions, beta):
    """Copies of the case's K in which, for each listed (query row, key position) pair of sequence 0, the key is beta
    times that row's query vector of head 0: that logit exceeds everything before it by tens of nats."""
    q = W.bf16_bits_to_f32(case.q)
    k = W.bf16_bits_to_f32(case.k_ctx).copy()
    for row, pos in zip(rows, key_positions):
        k[pos, 0] = beta * q[row, 0]
    case.k_ctx = W.f32_to_bf16_bits(k)
    return case


@pytest.mark.parametrize("tile,beta", [(128, 3.0), (256, 3.0), (256, 9.0)])
def test_prefill_reference_maximum_jumps_late(oracle, G, opts, tile, beta):
    """Logits that exceed a column's running maximum by far more than the kernels let their reference lag, long after the
    column has begun to accumulate: the 128-column kernel rescales in place, the 256-column kernel runs the pass again
    from the final reference.  Also a jump inside the very first key tile and one in the last, partial tile.  beta = 3:
    about 50 powers of two above everything before (the 256-column kernel's first attempt, which follows no maximum behind
    the first tile, still holds it); beta = 9: about 150 (its running sums leave the fp32 range it allows itself, the
    pass is run again following the maximum, and once more from the final reference)."""
    opts(tile=tile)
    case = W.make_attn_case("t", 93, "bf16", [(300, 1500)], 8, 1, 128)
    first_new = 1200
    rows = [5, 5, 120, 299, 17]
    keys = [700, 1100, 3, first_new + 299, 40]       # visible to their rows: key <= 1200 + row
    case = _with_late_outliers(case, rows, keys, beta=beta)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = G.prefill_case(case, G.cache_for_case(case))
    _check(got, want)
    # the affected rows are dominated by one key: their result is that key's V row to within the tolerance
    v = W.to_f64(case.v_ctx, "bf16")
    g = W.to_f64(got, "bf16")
    assert np.abs(g[299, 0] - v[first_new + 299, 0]).max() <= BF16_MAX


@pytest.mark.parametrize("tile", [128, 256])
def test_prefill_random_batches(oracle, G, opts, tile):
    """Forty batches of random shape (1-4 sequences, chunks of 1-700 tokens, a third of them behind up to 3000 cached
    tokens, 4 / 5 / 8 / 16 query heads per KV head), N(0,1) data: every output element within the bound.  The first rows of
    a prompt are single V rows of magnitude up to 4, where one bf16 step is 0.031: the bound of 2e-2 holds there only if
    the largest probability of such a row is exact (a softmax without a reference failed two of these forty)."""
    opts(tile=tile)
    rng = np.random.default_rng(123)
    for it in range(40):
        seqs = []
        for _ in range(int(rng.integers(1, 5))):
            q = int(rng.integers(1, 700))
            seqs.append((q, q + int(rng.integers(0, 3) == 0) * int(rng.integers(0, 3000))))
        hq = int(rng.choice([4, 5, 8, 16]))
        case = W.make_attn_case("sweep", 1000 + it, "bf16", seqs, hq, 1, 128)
        want = oracle.attention_case(case, oracle.cache_for_case(case))
        got = G.prefill_case(case, G.cache_for_case(case))
        _check(got, want)


def test_prefill_kernels_agree_on_dispatch(oracle, G, opts):
    """Left to itself the library picks a kernel per launch; whichever it picks, results stay within tolerance of the
    oracle on a shape at the boundary of the choice (enough 256-column tiles to fill the chip, or not)."""
    for n_tok in (1500, 6300):
        case = W.make_attn_case("t", 94, "bf16", [(n_tok, n_tok)], 8, 1, 128)
        rows = np.unique(np.concatenate([np.arange(0, 40), np.arange(n_tok - 40, n_tok),
                                         np.random.default_rng(4).integers(0, n_tok, 24)]))
        want = oracle.attention_case(case, oracle.cache_for_case(case), rows)
        got = G.prefill_case(case, G.cache_for_case(case))
        _check(got[rows], want)


# 32-key tiles a pass walks: every remainder of the loop's four tiles a trip from one tile on, and the ends of the 64 addresses
# that a wavefront holds ready (K runs out after 60 iterations, then after 64 more)
TILE_COUNTS = [1, 2, 3, 4, 5, 6, 7, 8, 59, 60, 61, 62, 63, 64, 65, 66, 123, 124, 125, 129]


@pytest.mark.parametrize("scaled_q", [0, 1])
@pytest.mark.parametrize("tiles", TILE_COUNTS)
def test_wide_prefill_kernel_at_the_ends_of_its_loop(oracle, G, opts, tiles, scaled_q):
    """One workgroup of the 256-column kernel walks exactly `tiles` tiles, the last of them ragged; the scaled-Q bound as above."""
    opts(tile=256, splits=1, pairing=2, scaled_q=scaled_q)
    ctx = 32 * tiles - 5
    case = W.make_attn_case("t", 97 + tiles, "bf16", [(min(20, ctx), ctx)], 8, 1, 128)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = W.to_f64(G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF)), "bf16")
    assert got.shape == want.shape and np.all(np.isfinite(got))
    err = np.abs(got - want)
    assert np.all(err <= BF16_MAX + (2.0 ** -7 * np.abs(want) if scaled_q else 0)) and err.mean() <= BF16_MEAN, (err.max(), err.mean())


@pytest.mark.parametrize("pairing", [1, 2])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("hq_l,hkv_l", [(8, 1), (5, 1), (4, 4), (10, 2)])
def test_two_groups_of_wavefronts_at_the_ends_of_their_loops(oracle, G, opts, pairing, splits, hq_l, hkv_l):
    """Sequences that end after 1, 2, 3, ... tiles of 32 keys, so that one group has a tile more than the other, or none at all, and
    walks past the end of its 64 addresses."""
    opts(tile=128, splits=splits, pairing=pairing)
    seqs = [(1700, 1700), LONG] + [(min(20, 32 * t - 5), 32 * t - 5) for t in (1, 2, 3, 4, 5, 6, 7, 8, 9, 119, 120, 121, 122, 128, 131)]
    case = W.make_attn_case("t", 99, "bf16", seqs, hq_l, hkv_l, 128)
    _takes(G, case, 128, 64, splits, 3 - pairing)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF))
    _check(got, want)


@pytest.mark.parametrize("beta", [3.0, 9.0])
def test_two_groups_of_wavefronts_follow_the_maximum(oracle, G, opts, beta):
    """Logits some 50 and 150 powers of two above everything before them, in tiles of one group or the other: beyond the range of
    the sums both groups run the pass again."""
    opts(tile=128, splits=1)
    case = W.make_attn_case("t", 93, "bf16", [(300, 2500)], 8, 1, 128)
    _takes(G, case, 128, 64, 1)
    first_new = 2200
    case = _with_late_outliers(case, [5, 5, 120, 299, 17], [700, 1124, 3, first_new + 299, 40], beta=beta)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    _check(G.prefill_case(case, G.cache_for_case(case)), want)


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", SHAPES)
def test_two_groups_of_wavefronts_on_all_shapes(oracle, G, opts, splits, seqs, hq_l, hkv_l):
    opts(tile=128, splits=splits, pairing=2)
    case = W.make_attn_case("t", 91, "bf16", seqs + [LONG], hq_l, hkv_l, 128)
    _takes(G, case, 128, 64, splits, 1)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    _check(G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF)), want)


@pytest.mark.parametrize("splits", [1, 2, 3])
def test_two_groups_of_wavefronts_run_a_pass_three_times(oracle, G, opts, splits):
    """Late logits some 150 powers of two above everything before them, in every key range, for a row of each of eight tiles that walk
    101, 103, ... 115 key tiles, all of them full: the attempt that follows the maximum is flagged as well, and the one behind
    it ends with the first group a tile ahead of or behind the second, at every stage of the ring (its count of tiles takes all four
    remainders, with one range and with several)."""
    opts(tile=128, splits=splits, pairing=2)
    case = W.make_attn_case("t", 107, "bf16", [(600, 3800), LONG], 8, 1, 128)
    _takes(G, case, 128, 64, splits, 1)
    rows = [16 * tile + 9 for tile in (0, 4, 8, 12, 16, 20, 24, 28)]
    assert [(3200 + row // 16 * 16 + 15) // 32 + 1 for row in rows] == list(range(101, 117, 2))
    at = (500, 900, 1500, 1900, 2700, 3100)        # two or more in each range, in tiles of either group, behind their first ones
    pairs = [(row, key + 7 * i) for i, row in enumerate(rows) for key in at]
    case = _with_late_outliers(case, [r for r, _ in pairs], [k for _, k in pairs], beta=9.0)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    _check(G.prefill_case(case, G.cache_for_case(case)), want)


@pytest.mark.parametrize("dead", [range(200), list(range(32)) + list(range(64, 96)), list(range(32, 64)) + list(range(96, 128))],
                         ids=["all", "even_tiles", "odd_tiles"])
@pytest.mark.parametrize("tile,wave,splits", [(128, 32, 1), (128, 64, 1), (128, 64, 2), (256, 64, 1), (256, 64, 2)])
def test_keys_whose_logits_overflow_do_not_hide_those_behind_them(oracle, G, opts, tile, wave, splits, dead):
    """K of the lowest bf16 value in one component, where every query is positive: the logits of the first key tiles (of one group of
    wavefronts or of both) are minus infinity, their columns have no reference when the key loop begins, and the keys behind them
    carry the whole result."""
    opts(tile=tile, splits=splits, pairing=2)
    case = W.make_attn_case("t", 101, "bf16", [(40, 400), (33, 333)] + ([LONG] if wave == 64 else []), 8, 1, 128)
    _takes(G, case, tile, wave, splits, 1)
    q, k = W.bf16_bits_to_f32(case.q).copy(), W.bf16_bits_to_f32(case.k_ctx).copy()
    q[:, :, 0] = 4.0
    k[np.array(dead), 0, 0] = -np.float32(2.0 ** 127 * (2 - 2.0 ** -7))       # of the first sequence: k_ctx holds it first
    case.q, case.k_ctx = W.f32_to_bf16_bits(q), W.f32_to_bf16_bits(k)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    _check(G.prefill_case(case, G.cache_for_case(case)), want)


@pytest.mark.parametrize("tile", [128, 256])
def test_wavefronts_without_columns_do_not_hold_up_the_others(G, opts, tile):
    """A tile of three tokens of eight heads fills half a wavefront, the others of its workgroup have no column; it walks the keys of
    a full one.  With selects for masked keys in every iteration of those it took 1.35 times as long as the full tile, without them as
    long (0.99 and 1.00): the bound lies between, a run differs from another by a per cent or two."""
    import torch
    from paper_2509_16495_amd import binding as B
    opts(tile=tile, splits=1, pairing=2)
    calls = []
    for tokens in (3, tile // 8):
        case = W.make_attn_case("t", 109, "bf16", [(tokens, 20000)], 8, 1, 128)
        _takes(G, case, tile, 64, 1, 1)
        cache, q, out = G.cache_for_case(case), G.t(case.q, "bf16"), torch.empty(case.q.shape, dtype=torch.bfloat16, device=G.DEV)
        table, cu, ctx = G.ti(case.block_table, np.int32), G.ti(case.cu_seqlens_q, np.int32), G.ti(case.ctx_lens, np.int32)
        calls.append(lambda c=(q, cache, table, cu, ctx, tokens, 20000, out, case.softmax_scale): B.prefill(*c))
    times = [[], []]
    for _ in range(30):
        for call, us in zip(calls, times):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            call()
            end.record()
            end.synchronize()
            us.append(start.elapsed_time(end) * 1e3)
    few, full = (float(np.median(us[5:])) for us in times)
    print(f"three tokens {few:.1f} us, a full tile {full:.1f} us")
    assert few < 1.15 * full, (few, full)
