"""The fp32 prefill kernel (head_dim 64 and 128) against the fp64 oracle at the edges of its 16-column tiles, 32-key steps
and eight wavefronts, and against values that are no numbers in tokens a row must not see.  max |err| <= 2e-5: values of
a few units, sums of up to some hundred products in fp32 (2^-24 each), as for the other fp32 attention tests."""
import numpy as np
import pytest

from paper_2509_16495_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_backend
    return gpu_backend


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", [
    ([(1, 1)], 4, 1),
    ([(4, 4), (5, 5), (3, 31), (1, 32), (2, 33), (0, 7)], 4, 1),      # tiles of four tokens; empty chunk
    ([(255, 255), (257, 257), (9, 513)], 4, 1),                       # one, two and three rounds of the wavefronts
    ([(17, 17), (16, 300)], 1, 1),                                    # 16 tokens per tile
    ([(13, 270)], 5, 1),                                              # 15 of 16 columns in use
    ([(7, 40), (20, 20)], 32, 2),                                     # 16 heads per KV head: a token per tile
    ([(n, n + 3) for n in range(1, 71)], 6, 2),                       # more sequences than a wavefront looks at together
])
def test_fp32_prefill(oracle, G, D, seqs, hq_l, hkv_l):
    case = W.make_attn_case("t", 101, "f32", seqs, hq_l, hkv_l, D, pool_factor=1.3)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    got = W.to_f64(G.prefill_case(case, G.cache_for_case(case, fill_byte=0xFF)), "f32")   # (unwritten slots: NaN)
    assert np.all(np.isfinite(got)) and np.abs(got - want).max() <= 2e-5


@pytest.mark.parametrize("D", [64, 128])
def test_rows_in_front_of_a_value_that_is_no_number(oracle, G, D):
    case = W.make_attn_case("t", 102, "f32", [(70, 90)], 4, 1, D, pool_factor=1.3)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    bad = 61   # context position; the first new token sits at 20
    case.v_ctx[bad, 0, 3], case.v_ctx[bad, 0, 5], case.k_ctx[bad + 4, 0, 1] = np.inf, np.nan, np.nan
    got = W.to_f64(G.prefill_case(case, G.cache_for_case(case)), "f32")
    assert np.abs(got[:bad - 20] - want[:bad - 20]).max() <= 2e-5
    assert np.all(np.isnan(got[bad - 20:, :, 5])) and np.all(np.isinf(got[bad - 20:bad + 4 - 20, :, 3]))
    keep = [d for d in range(D) if d not in (3, 5)]
    assert np.abs(got[bad - 20:bad + 4 - 20][:, :, keep] - want[bad - 20:bad + 4 - 20][:, :, keep]).max() <= 2e-5
    assert np.all(np.isnan(got[bad + 4 - 20:]))
