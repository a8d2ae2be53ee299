"""Merges of partial attention results at the part counts where they change shape: prefill key ranges around the eight
parts requested at once and the 32 (max, sum) pairs held one per lane, decode parts around the 64 of a wavefront and the
four per group.  max |err| <= 2e-2 and mean |err| <= 1e-3 against the fp64 oracle, as for all bf16 attention."""
import numpy as np
import pytest

from paper_2509_16495_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_backend
    return gpu_backend


def _check(got_bits, want):
    got = W.to_f64(got_bits, "bf16")
    assert np.all(np.isfinite(got))
    err = np.abs(got - want)
    assert err.max() <= 2e-2 and err.mean() <= 1e-3, (err.max(), err.mean())


@pytest.mark.parametrize("splits", [2, 7, 8, 9, 16, 17, 31, 32, 33, 40, 41, 64])
def test_prefill_key_ranges(oracle, G, splits):
    from paper_2509_16495_amd import binding as B
    # 9 x 5 and 13 x 5 rows: neither fills the last workgroup of eight rows; the second chunk has ranges without keys
    case = W.make_attn_case("t", 97, "bf16", [(9, 2500), (13, 200)], 5, 1, 128, pool_factor=1.3)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    cache = G.cache_for_case(case)
    B.set_option(B.OPT_PREFILL_SPLITS, splits)
    try:
        got = G.prefill_case(case, cache)
    finally:
        B.set_option(B.OPT_PREFILL_SPLITS, 0)
    _check(got, want)


@pytest.mark.parametrize("ctx", [
    [64], [65], [64 * 15], [64 * 16 + 1], [64 * 48], [64 * 48 + 1], [64 * 63], [64 * 64], [64 * 64 + 1], [64 * 65 + 40, 3],
    [64 * 63 - 31, 64 * 65, 64 * 130],
    [100] * 127 + [6000],          # 1024 rows: four groups per row, one row with more parts than they request at once
    [70] * 200 + [9000, 31000],  # and one beyond 64 parts
])
def test_decode_parts(oracle, G, ctx):
    case = W.make_attn_case("t", 98, "bf16", [(1, c) for c in ctx], 8, 1, 128, pool_factor=1.1)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = G.decode_case(case, G.cache_for_case(case))
    _check(got, want)
    assert G.decode_case(case, G.cache_for_case(case)).tobytes() == got.tobytes()
