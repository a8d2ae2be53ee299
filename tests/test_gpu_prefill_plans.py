"""Launch plans of the prefill kernels against the fp64 oracle: the 128-column kernel with one tile per workgroup, and
launches whose workspace holds fewer key ranges than the fastest plan takes.  max |err| <= 2e-2 and mean |err| <= 1e-3,
as for all bf16 attention."""
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


@pytest.mark.parametrize("splits", [0, 1, 3, 17])
@pytest.mark.parametrize("seqs,hq_l,hkv_l", [
    ([(1, 1)], 8, 1),
    ([(16, 16), (17, 17), (33, 2050)], 8, 1),            # one tile exactly, one more token, three tiles behind a context
    ([(128, 128), (129, 129), (300, 427)], 5, 1),        # heads not stacked: 128 tokens per tile
    ([(47, 3000), (1, 2900), (0, 0), (90, 95)], 4, 2),   # four (sequence, head) pairs rotated over the dies, empty chunk
    ([(200, 900), (31, 31), (64, 64)], 16, 2),
])
def test_one_tile_per_workgroup(oracle, G, splits, seqs, hq_l, hkv_l):
    from paper_2509_16495_amd import binding as B
    case = W.make_attn_case("t", 99, "bf16", seqs, hq_l, hkv_l, 128, pool_factor=1.3)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    cache = G.cache_for_case(case)
    try:
        B.set_option(B.OPT_PREFILL_TILE, 128)
        B.set_option(B.OPT_PREFILL_PAIRING, 2)
        B.set_option(B.OPT_PREFILL_SPLITS, splits)
        got = G.prefill_case(case, cache)
    finally:
        for opt in (B.OPT_PREFILL_TILE, B.OPT_PREFILL_PAIRING, B.OPT_PREFILL_SPLITS):
            B.set_option(opt, 0)
    _check(got, want)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_workspace_of_any_size_between_the_least_and_the_best(oracle, G, kv):
    """A chunk whose fastest plan takes key ranges and whose plan without a workspace takes none."""
    import torch
    from paper_2509_16495_amd import binding as B
    T, S, hq = 150, 1000, 8
    scales = (0.0371, 0.0293) if kv == "fp8" else None
    case = W.make_attn_case("t", 100, "bf16", [(T, S)], hq, 1, 128, pool_factor=1.1)
    if scales:
        want = oracle.attention_case(case, oracle.cache_for_case(case, fp8_scales=scales), k_scale=scales[0], v_scale=scales[1])
    else:
        want = oracle.attention_case(case, oracle.cache_for_case(case))
    cache = G.cache_for_case(case, fp8_scales=scales)
    ks, vs = scales or (1.0, 1.0)
    q, table, cu, ctx = G.t(case.q, "bf16"), G.ti(case.block_table, np.int32), G.ti(case.cu_seqlens_q, np.int32), G.ti(case.ctx_lens, np.int32)
    out = torch.empty_like(q)
    best = B.prefill_workspace_bytes(1, T, T, S, B.attn_desc(q, cache, table, case.softmax_scale, None, out, ks, vs))
    part, blocks = T * hq * 130 * 4, -(-S // 16)   # one range's partials; blocks widened from FP8, with their table
    fixed = blocks * 2 * 4096 + -(-blocks * 4 // 256) * 256 if scales else 0
    assert (best - fixed) // part >= 2
    for size in (fixed, fixed + 2 * part - 256, fixed + -(-2 * part // 256) * 256, best):
        ws = torch.empty(size + 256, dtype=torch.uint8, device=G.DEV)
        ws[size:].fill_(0x5A)
        out.zero_()
        B.prefill(q, cache, table, cu, ctx, T, S, out, case.softmax_scale, workspace=ws[:size], k_scale=ks, v_scale=vs)
        torch.cuda.synchronize()
        _check(B.to_host(out), want)
        assert torch.all(ws[size:] == 0x5A)


@pytest.mark.parametrize("last,ranges", [(211, 4), (212, 3)])
def test_unequal_chunks_at_the_line_to_whole_rounds(oracle, G, last, ranges):
    """Four chunks of up to 392 tokens: of the 400 workgroups that four key ranges make 217.5 and 217.8 count as busy, and
    the line lies at 217.6."""
    from paper_2509_16495_amd import binding as B
    seqs = [(392, 3000), (70, 2000), (141, 150), (last, 1111)]
    case = W.make_attn_case("t", 101, "bf16", seqs, 8, 1, 128, pool_factor=1.1)
    want = oracle.attention_case(case, oracle.cache_for_case(case))
    cache = G.cache_for_case(case)
    q, table = G.t(case.q, "bf16"), G.ti(case.block_table, np.int32)
    total = sum(n for n, _ in seqs)
    assert B.prefill_workspace_bytes(4, total, 392, 3000, B.attn_desc(q, cache, table, case.softmax_scale, None, q)) == ranges * total * 8 * 130 * 4
    _check(G.prefill_case(case, cache), want)
