"""Host-side checks of the C ABI (no GPU): the library loads, exports every function the header
declares, its index helpers reproduce the paper's worked examples, and every invalid-argument
path returns an error code before anything could be launched."""
import ast
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "shiftattn.h")


@pytest.fixture(scope="module")
def B():
    from paper_2509_16495_amd import binding
    if not binding.is_built():
        from paper_2509_16495_amd import build
        build.build_library()
    binding.lib()
    return binding


def _declared_functions():
    """Every function declared in any header under include/."""
    import glob
    names = set()
    for header in glob.glob(os.path.join(ROOT, "include", "*.h")):
        text = re.sub(r"/\*.*?\*/", "", open(header).read(), flags=re.S)
        names |= set(re.findall(r"\b(shiftattn_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_every_declared_symbol_is_exported(B):
    names = _declared_functions()
    assert {"shiftattn_pack_seq2head", "shiftattn_prefill", "shiftattn_decode", "shiftattn_unpack_head2seq",
            "shiftattn_kv_write", "shiftattn_last_error"} <= set(names)
    for n in names:
        assert hasattr(B.lib(), n), n


def test_options_and_their_bounds(B):
    """The tuning switches: defaults are 0, values are range-checked, unknown options refused."""
    L = B.lib()
    for opt in (B.OPT_PREFILL_TILE, B.OPT_PREFILL_SPLITS, B.OPT_GENERIC_ONLY, B.OPT_PREFILL_PAIRING, B.OPT_PREFILL_SCALED_Q):
        assert B.get_option(opt) == 0
    assert L.shiftattn_set_option(B.OPT_PREFILL_SCALED_Q, 2) == B.EINVAL
    assert L.shiftattn_set_option(B.OPT_PREFILL_PAIRING, 3) == B.EINVAL and L.shiftattn_set_option(B.OPT_PREFILL_PAIRING, -1) == B.EINVAL
    assert L.shiftattn_set_option(B.OPT_PREFILL_TILE, 64) == B.EINVAL
    assert L.shiftattn_set_option(B.OPT_PREFILL_SPLITS, 65) == B.EINVAL and L.shiftattn_set_option(B.OPT_PREFILL_SPLITS, -1) == B.EINVAL
    assert L.shiftattn_set_option(B.OPT_GENERIC_ONLY, 2) == B.EINVAL
    assert L.shiftattn_set_option(17, 0) == B.EINVAL and B.get_option(17) == -1
    a = _attn(B, max_blocks_per_seq=8320)
    auto = B.prefill_workspace_bytes(1, 2048, 2048, 133120, a)
    try:
        B.set_option(B.OPT_PREFILL_SPLITS, 4)
        assert B.get_option(B.OPT_PREFILL_SPLITS) == 4
        assert B.prefill_workspace_bytes(1, 2048, 2048, 133120, a) == 4 * 2048 * 8 * (128 + 2) * 4   # sizes follow the switch
        B.set_option(B.OPT_GENERIC_ONLY, 1)
        assert B.prefill_workspace_bytes(1, 2048, 2048, 133120, a) == 0 and B.decode_workspace_bytes(4, 64, a) == 0
    finally:
        for opt in (B.OPT_PREFILL_TILE, B.OPT_PREFILL_SPLITS, B.OPT_GENERIC_ONLY, B.OPT_PREFILL_PAIRING, B.OPT_PREFILL_SCALED_Q):
            B.set_option(opt, 0)
    assert B.prefill_workspace_bytes(1, 2048, 2048, 133120, a) == auto


def test_launch_plans_follow_the_shape_of_the_batch(B):
    """Host logic behind the workspace queries (no GPU work): how many key ranges a prefill launch takes, seen through
    the size of its partial results, `ranges x rows x heads x (128 + 2) x 4` bytes; and the sizes named for the k ranges of the
    projections.  Shapes: the benchmark's batches (Table 4 head geometries on 8 ranks)."""
    def ranges(num_seqs, total_q, max_q, max_ctx, hq):
        a = _attn(B, num_q_heads=hq, max_blocks_per_seq=(max_ctx + 15) // 16)
        ws = B.prefill_workspace_bytes(num_seqs, total_q, max_q, max_ctx, a)
        assert ws % (total_q * hq * 130 * 4) == 0
        return ws // (total_q * hq * 130 * 4)

    assert ranges(4, 16384, 4096, 4096, 4) == 0         # 256 equal workgroups of 128-column tiles: one round, no split
    assert ranges(1, 16384, 16384, 16384, 8) == 0       # 256 pairs of 256-column tiles
    assert ranges(1, 2048, 2048, 133120, 8) == 4        # 64 tiles, one per workgroup (nothing to level by pairing): four ranges fill the chip
    assert ranges(1, 16384, 16384, 16384, 5) == 2       # 322 tiles, one per workgroup, heaviest first: two ranges bring the heaviest under a compute unit's share
    assert ranges(4, 16384, 4096, 4096, 5) == 0         # short contexts: the merge would cost more than the ragged round
    try:
        B.set_option(B.OPT_PREFILL_TILE, 128)
        assert ranges(1, 2048, 2048, 133120, 8) == 4    # 64 pairs of 128-column tiles
        B.set_option(B.OPT_PREFILL_TILE, 256)
        assert ranges(4, 16384, 4096, 4096, 4) == 2     # 128 pairs of 256-column tiles
        B.set_option(B.OPT_PREFILL_PAIRING, 1)
        assert ranges(1, 2048, 2048, 133120, 8) == 8    # in pairs the chunk is 32 workgroups: eight ranges fill the chip
        assert ranges(1, 16384, 16384, 16384, 5) == 3   # 161 pairs: three ranges make two full rounds
        B.set_option(B.OPT_PREFILL_PAIRING, 2)
        assert ranges(1, 16384, 16384, 16384, 8) == 0   # 512 tiles, heaviest first: the light ones level the chip out
    finally:
        B.set_option(B.OPT_PREFILL_TILE, 0)
        B.set_option(B.OPT_PREFILL_PAIRING, 0)
    # projections: up to 64 rows ranges x rows rounded up to 16, 32 or 64, above them the k ranges of the large-batch kernel while its
    # tiles are few, nothing once they fill the chip
    n, k = 10240, 8192
    assert [B.proj_workspace_bytes(t, n, k) // (n * 4) for t in (1, 16, 17, 32, 33, 64)] == [0, 0, 2 * 32, 2 * 32, 4 * 64, 4 * 64]
    assert B.proj_workspace_bytes(65, n, k) == 6 * 65 * n * 4 and B.proj_workspace_bytes(512, n, k) == 3 * 512 * n * 4
    assert B.proj_workspace_bytes(1024, n, k) == 0 and B.proj_workspace_bytes(16384, n, k) == 0
    # 2048 rows are 320 tiles: six token tiles whole (240 tiles), the last 512 rows in three k ranges (240 work items)
    assert B.proj_workspace_bytes(2048, n, k) == 3 * 512 * n * 4
    assert B.proj_workspace_bytes(8, 6144, 4096) == 0 and B.proj_workspace_bytes(0, n, k) == 0
    # whatever the plan, the workspace is whole fp32 rows of the result: at most 16 ranges of at most all rows, rows of
    # whole leading tiles excluded in steps of 256, and nothing when the tiles are a whole number of rounds of the chip
    for feats, kk in ((10240, 8192), (8192, 8192), (6144, 4096), (2560, 5120), (256, 64)):
        for rows in (65, 100, 255, 256, 257, 511, 777, 1024, 1500, 2048, 2300, 4096, 5000, 8192, 16384, 20000):
            for fp8 in (False, True):
                need = B.proj_workspace_bytes(rows, feats, kk, fp8=fp8)
                assert need % (feats * 4) == 0
                q = need // (feats * 4)   # ranges x rows they cover
                assert q <= 16 * rows
                if q:
                    covered = [r for r in range(rows, 0, -256) if q % r == 0 and 2 <= q // r <= 16]
                    assert covered, (rows, feats, kk, q)
                if (feats // 256) * (-(-rows // 256)) % 256 == 0:
                    assert need == 0, (rows, feats, kk)


@pytest.mark.parametrize("lens,cached,hq,hkv,tile", [
    ([58, 177], 7559, 8, 1, 16), ([222, 85], 8071, 8, 1, 16), ([533, 129], 2897, 4, 1, 32), ([88, 14], 12938, 8, 1, 16),
])
def test_two_unequal_chunks_fit_the_dies_they_run_on(B, lens, cached, hq, hkv, tile):
    """With two (sequence, head) every second die is one sequence's: the long chunk's workgroups are planned for 128 of the
    256 compute units, one round of them."""
    a = _attn(B, num_q_heads=hq, num_kv_heads=hkv, max_blocks_per_seq=(max(lens) + cached + 15) // 16)
    ranges = B.prefill_workspace_bytes(2, sum(lens), max(lens), max(lens) + cached, a) // (sum(lens) * hq * 130 * 4)
    assert 1 < ranges and ranges * ((max(lens) + tile - 1) // tile) <= 128


@pytest.mark.parametrize("lens,cached,hq,hkv", [
    ([9, 33, 51, 36, 20, 48, 37], 3715, 5, 1), ([35, 31, 35, 5, 24, 8], 1112, 10, 2), ([18, 63, 3, 57, 24, 30, 7, 34, 42, 20], 5990, 5, 1),
])
def test_chunks_shorter_than_a_tile_count_as_busy(B, lens, cached, hq, hkv):
    """Every chunk fits one 128-token tile, so every workgroup of every key range has work: one round of 256."""
    a = _attn(B, num_q_heads=hq, num_kv_heads=hkv, max_blocks_per_seq=(max(lens) + cached + 15) // 16)
    ranges = B.prefill_workspace_bytes(len(lens), sum(lens), max(lens), max(lens) + cached, a) // (sum(lens) * hq * 130 * 4)
    assert 1 < ranges and ranges * len(lens) * hq <= 256


def test_struct_layouts_match_header(B):
    assert ctypes.sizeof(B.Xchg) == 20
    assert ctypes.sizeof(B.Attn) == 72 and B.Attn.q_stride.offset == 32 and B.Attn.kv_format.offset == 56


def test_head_block_matches_paper_example(B):
    gold = {}
    for line in open(os.path.join(ROOT, "tests", "golden", "process_groups_sp3_tp2.txt")):
        if line.strip() and not line.startswith("#"):
            k, v = line.split("=", 1)
            gold[k.strip()] = ast.literal_eval(v.strip())
    sp, tp = gold["SP"], gold["TP"]
    blocks = [B.head_block(sp, tp, r) for r in range(sp * tp)]
    for rank, head in gold["HEAD_OF_RANK"].items():
        assert blocks[rank] == head
    assert [blocks.index(b) for b in range(sp * tp)] == gold["SP_TP_GROUP"][0]
    assert B.head_block(3, 2, 6) == -1 and B.head_block(0, 2, 0) == -1 and B.head_block(3, 2, -1) == -1


def test_shift_dispatcher_threshold(B):
    """Algorithm 2: batches larger than the threshold run in the base configuration, the rest in the
    shift configuration."""
    assert B.use_base_config(4097, 4096) == 1 and B.use_base_config(4096, 4096) == 0 and B.use_base_config(0, 0) == 0
    assert B.use_base_config(1, 0) == 1 and B.use_base_config(-1, 5) == -1 and B.use_base_config(5, -1) == -1


def test_replication_and_padding_helpers(B):
    assert [B.kv_head_of_block(p, 8, 4) for p in range(8)] == [0, 0, 1, 1, 2, 2, 3, 3]
    assert [B.kv_head_of_block(p, 4, 8) for p in range(4)] == [0, 2, 4, 6]
    assert B.kv_head_of_block(8, 8, 4) == -1
    assert B.padded_tokens(9, 8) == 16 and B.padded_tokens(16, 8) == 16 and B.padded_tokens(0, 8) == 0
    assert B.padded_tokens(-1, 8) == -1 and B.padded_tokens(5, 0) == -1


def _xchg(B, **kw):
    d = dict(P=2, num_q_heads=8, num_kv_heads=0, head_dim=64, dtype=B.F32)
    d.update(kw)
    return B.Xchg(d["P"], d["num_q_heads"], d["num_kv_heads"], d["head_dim"], d["dtype"])


def _attn(B, **kw):
    d = dict(num_q_heads=8, num_kv_heads=1, head_dim=128, dtype=B.BF16, block_size=16, num_blocks=64,
             max_blocks_per_seq=8, softmax_scale=0.1, q_stride=0, kv_stride=0, out_stride=0, kv_format=0, k_scale=0.0,
             v_scale=0.0, reserved=0)
    d.update(kw)
    return B.Attn(*[d[f[0]] for f in B.Attn._fields_])


FAKE = ctypes.c_void_p(0x1000)  # aligned, never dereferenced: every case below fails validation first


def test_pack_unpack_reject_bad_arguments(B):
    L = B.lib()
    cases = [
        (dict(P=0), 4, 4, B.EINVAL), (dict(P=3), 4, 4, B.EINVAL), (dict(num_kv_heads=3, P=2), 4, 4, B.EINVAL),
        (dict(dtype=7), 4, 4, B.EINVAL), (dict(), 5, 4, B.EINVAL), (dict(), -1, 4, B.EINVAL),
        (dict(head_dim=6), 4, 4, B.EUNSUPPORTED), (dict(head_dim=0), 4, 4, B.EINVAL),
        (dict(num_q_heads=12, num_kv_heads=6, P=4), 4, 4, B.EINVAL),
    ]
    for kw, T, T_pad, code in cases:
        x = _xchg(B, **kw)
        assert L.shiftattn_pack_seq2head(FAKE, FAKE, T, T_pad, ctypes.byref(x), None) == code, kw
        assert B.last_error()
    x = _xchg(B)
    assert L.shiftattn_pack_seq2head(None, FAKE, 4, 4, ctypes.byref(x), None) == B.EINVAL
    assert L.shiftattn_pack_seq2head(FAKE, None, 4, 4, ctypes.byref(x), None) == B.EINVAL
    assert L.shiftattn_pack_seq2head(ctypes.c_void_p(0x1008), FAKE, 4, 4, ctypes.byref(x), None) == B.EINVAL
    assert L.shiftattn_pack_seq2head(FAKE, FAKE, 4, 4, None, None) == B.EINVAL
    assert L.shiftattn_unpack_head2seq(None, FAKE, 4, 4, ctypes.byref(x), None) == B.EINVAL
    assert L.shiftattn_unpack_head2seq(FAKE, FAKE, 4, 3, ctypes.byref(x), None) == B.EINVAL
    # empty problems are valid no-ops and touch nothing
    assert L.shiftattn_pack_seq2head(None, None, 0, 0, ctypes.byref(x), None) == B.OK
    assert L.shiftattn_unpack_head2seq(None, None, 0, 4, ctypes.byref(x), None) == B.OK
    big = _xchg(B, num_q_heads=1 << 20, P=1, head_dim=256)
    assert L.shiftattn_pack_seq2head(FAKE, FAKE, 1 << 20, 1 << 20, ctypes.byref(big), None) == B.EUNSUPPORTED


def test_attention_entry_points_reject_bad_arguments(B):
    L = B.lib()

    def prefill(a, q=FAKE, k=None, v=None, slots=None, cache=FAKE, table=FAKE, cu=FAKE, sl=FAKE, S=1, tq=32, mq=32,
                ms=64, out=FAKE, ws=None, wsb=0):
        return L.shiftattn_prefill(q, k, v, slots, cache, table, cu, sl, S, tq, mq, ms, out, ws, wsb,
                                   None if a is None else ctypes.byref(a), None)

    def decode(a, q=FAKE, k=None, v=None, slots=None, cache=FAKE, table=FAKE, sl=FAKE, S=4, ms=64, out=FAKE, ws=None,
               wsb=0):
        return L.shiftattn_decode(q, k, v, slots, cache, table, sl, S, ms, out, ws, wsb,
                                  None if a is None else ctypes.byref(a), None)

    ok = _attn(B)
    assert prefill(None) == B.EINVAL and decode(None) == B.EINVAL
    for kw, code in [(dict(num_kv_heads=3), B.EINVAL), (dict(num_kv_heads=0), B.EINVAL), (dict(dtype=5), B.EINVAL),
                     (dict(head_dim=100), B.EUNSUPPORTED), (dict(head_dim=512), B.EUNSUPPORTED),
                     (dict(block_size=32), B.EUNSUPPORTED), (dict(softmax_scale=0.0), B.EINVAL),
                     (dict(softmax_scale=-1.0), B.EINVAL), (dict(softmax_scale=float("nan")), B.EINVAL),
                     (dict(q_stride=100), B.EINVAL), (dict(kv_stride=8), B.EINVAL), (dict(out_stride=1028), B.EINVAL),
                     (dict(max_blocks_per_seq=2), B.EINVAL), (dict(kv_format=7), B.EINVAL), (dict(reserved=1), B.EINVAL),
                     (dict(kv_format=B.KV_FP8_E4M3), B.EINVAL),  # scales missing
                     (dict(kv_format=B.KV_FP8_E4M3, k_scale=1.0, v_scale=-1.0), B.EINVAL),
                     (dict(kv_format=B.KV_FP8_E4M3, k_scale=float("inf"), v_scale=1.0), B.EINVAL),
                     (dict(kv_format=B.KV_FP8_E4M3, k_scale=1.0, v_scale=1.0, head_dim=72), B.EUNSUPPORTED)]:
        assert prefill(_attn(B, **kw)) == code, kw
        assert decode(_attn(B, **kw)) == code, kw
    for kw in (dict(q=None), dict(cache=None), dict(table=None), dict(sl=None), dict(out=None)):
        assert prefill(ok, **kw) == B.EINVAL and decode(ok, **kw) == B.EINVAL
    assert prefill(ok, cu=None) == B.EINVAL
    assert prefill(ok, k=FAKE) == B.EINVAL and decode(ok, v=FAKE, slots=FAKE) == B.EINVAL
    assert prefill(ok, q=ctypes.c_void_p(0x1002)) == B.EINVAL
    assert prefill(ok, S=-1) == B.EINVAL and prefill(ok, mq=64, tq=32) == B.EINVAL and prefill(ok, mq=128, tq=128, ms=64) == B.EINVAL
    assert decode(ok, S=-1) == B.EINVAL
    # decode always needs a workspace on the tuned path; a missing or short one is reported, not used
    need = B.decode_workspace_bytes(4, 64, ok)
    assert need > 0
    assert decode(ok) == B.EWORKSPACE and decode(ok, ws=FAKE, wsb=need - 1) == B.EWORKSPACE
    # the variant without a workspace argument: same argument checks; a batch beyond the library's own array is refused
    def decode_static(a, q=FAKE, cache=FAKE, table=FAKE, sl=FAKE, S=4, ms=64, out=FAKE):
        return L.shiftattn_decode_static(q, None, None, None, cache, table, sl, S, ms, out, None if a is None else ctypes.byref(a), None)

    assert decode_static(None) == B.EINVAL and decode_static(_attn(B, head_dim=100)) == B.EUNSUPPORTED
    assert decode_static(ok, S=-1) == B.EINVAL
    assert decode_static(ok, q=None, cache=None, table=None, sl=None, out=None, S=0, ms=0) == B.OK
    wide = _attn(B, num_q_heads=16)
    assert B.decode_workspace_bytes(2048, 64, wide) > B.STATIC_SCRATCH_BYTES
    assert decode_static(wide, S=2048) == B.EWORKSPACE and "scratch" in B.last_error()
    # split prefill (short chunk on a long context) needs one too
    long_ctx = _attn(B, max_blocks_per_seq=8320)
    need = B.prefill_workspace_bytes(1, 2048, 2048, 133120, long_ctx)
    assert need > 0
    assert prefill(long_ctx, tq=2048, mq=2048, ms=133120) == B.EWORKSPACE
    assert B.prefill_workspace_bytes(4, 16384, 4096, 4096, _attn(B, num_q_heads=4, max_blocks_per_seq=256)) == 0
    # empty batches are valid no-ops
    assert prefill(ok, q=None, cache=None, table=None, cu=None, sl=None, out=None, S=0, tq=0, mq=0, ms=0) == B.OK
    assert decode(ok, q=None, cache=None, table=None, sl=None, out=None, S=0, ms=0) == B.OK
    # unified batch: same checks, plus its own
    def mixed(a, q=FAKE, k=None, v=None, slots=None, cache=FAKE, table=FAKE, cu=FAKE, sl=FAKE, Sp=1, tq=32, mq=32, msp=64,
              Sd=4, msd=64, out=FAKE, ws=None, wsb=0):
        return L.shiftattn_mixed(q, k, v, slots, cache, table, cu, sl, Sp, tq, mq, msp, Sd, msd, out, ws, wsb,
                                 None if a is None else ctypes.byref(a), None)

    assert mixed(None) == B.EINVAL and mixed(ok, Sd=-1) == B.EINVAL and mixed(ok, Sp=0, tq=32) == B.EINVAL
    assert mixed(ok, q=None) == B.EINVAL and mixed(ok, cu=None) == B.EINVAL and mixed(ok, k=FAKE) == B.EINVAL
    assert mixed(ok) == B.EWORKSPACE  # the decode part needs one
    assert B.mixed_workspace_bytes(1, 32, 32, 64, 4, 64, ok) == B.decode_workspace_bytes(4, 64, ok)
    assert B.mixed_workspace_bytes(1, 2048, 2048, 133120, 4, 64, long_ctx) == \
        max(B.prefill_workspace_bytes(1, 2048, 2048, 133120, long_ctx), B.decode_workspace_bytes(4, 64, long_ctx))
    assert mixed(ok, q=None, cache=None, table=None, cu=None, sl=None, out=None, Sp=0, tq=0, mq=0, msp=0, Sd=0, msd=0) == B.OK
    # a call that brings new K/V is refused as a whole, before its write is launched, when a part is bad
    need = B.mixed_workspace_bytes(1, 32, 32, 64, 4, 64, ok)
    small = _attn(B, max_blocks_per_seq=2)  # 32 tokens per sequence at most
    for bad in (dict(a=small, msp=32, msd=64), dict(a=small, msp=64, msd=32), dict(a=ok, mq=64), dict(a=ok, out=ctypes.c_void_p(0x1002))):
        a = bad.pop("a")
        assert mixed(a, k=FAKE, v=FAKE, slots=FAKE, ws=FAKE, wsb=need, **bad) == B.EINVAL, bad
    kvw = L.shiftattn_kv_write
    assert kvw(None, FAKE, FAKE, 4, FAKE, ctypes.byref(ok), None) == B.EINVAL
    assert kvw(FAKE, FAKE, FAKE, -1, FAKE, ctypes.byref(ok), None) == B.EINVAL
    assert kvw(None, None, None, 0, None, ctypes.byref(ok), None) == B.OK
    assert B.lib().shiftattn_decode_workspace_bytes(-1, 64, ctypes.byref(ok)) == ctypes.c_size_t(-1).value


def test_projection_entry_points_reject_bad_arguments(B):
    """The fused projections (Algorithm 1, the products next to the two all-to-alls): bf16, head_dim 128 only."""
    L = B.lib()
    ok = dict(P=8, num_q_heads=64, num_kv_heads=8, head_dim=128, dtype=B.BF16)
    x = _xchg(B, **ok)
    q, o = L.shiftattn_qkv_proj_pack, L.shiftattn_unpack_o_proj
    # shapes the GEMM is not built for
    for kw, d_model in [(dict(dtype=B.F32), 8192), (dict(head_dim=64), 8192), (dict(), 8200), (dict(num_q_heads=9, num_kv_heads=1, P=1), 8192)]:
        bad = _xchg(B, **{**ok, **kw})
        assert q(FAKE, FAKE, FAKE, 8, 8, d_model, ctypes.byref(bad), None) == B.EUNSUPPORTED, (kw, d_model)
        assert "projection" in B.last_error()
    for kw, d_model in [(dict(dtype=B.F32), 8192), (dict(head_dim=64), 8192), (dict(), 8192 + 64)]:
        bad = _xchg(B, **{**ok, **kw, "num_kv_heads": 0})
        assert o(FAKE, FAKE, FAKE, 8, 8, d_model, ctypes.byref(bad), None) == B.EUNSUPPORTED, (kw, d_model)
    xo = _xchg(B, **{**ok, "num_kv_heads": 0})
    # invalid arguments: sizes, descriptor, pointers, alignment
    for fn, desc in ((q, x), (o, xo)):
        assert fn(FAKE, FAKE, FAKE, 9, 8, 8192, ctypes.byref(desc), None) == B.EINVAL      # T > T_pad
        assert fn(FAKE, FAKE, FAKE, 8, 8, 0, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, FAKE, FAKE, 8, 8, -64, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, FAKE, FAKE, 8, 8, 8192, None, None) == B.EINVAL
        assert fn(None, FAKE, FAKE, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, None, FAKE, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, FAKE, None, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, ctypes.c_void_p(0x1004), FAKE, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert B.last_error()
    bad_p = _xchg(B, **{**ok, "P": 3})
    assert q(FAKE, FAKE, FAKE, 6, 6, 8192, ctypes.byref(bad_p), None) == B.EINVAL          # heads not divisible by P
    # the forms with a workspace: the same checks, and a workspace must exist and be aligned if a size is given
    qw, ow = L.shiftattn_qkv_proj_pack_ws, L.shiftattn_unpack_o_proj_ws
    for fn, desc in ((qw, x), (ow, xo)):
        assert fn(FAKE, FAKE, FAKE, 9, 8, 8192, ctypes.byref(desc), None, 0, None) == B.EINVAL
        assert fn(None, FAKE, FAKE, 8, 8, 8192, ctypes.byref(desc), None, 0, None) == B.EINVAL
        assert fn(FAKE, FAKE, FAKE, 32, 32, 8192, ctypes.byref(desc), None, 4096, None) == B.EINVAL and "workspace" in B.last_error()
        assert fn(FAKE, FAKE, FAKE, 32, 32, 8192, ctypes.byref(desc), ctypes.c_void_p(0x1004), 4096, None) == B.EINVAL
        assert fn(None, None, None, 0, 0, 8192, ctypes.byref(desc), None, 0, None) == B.OK
    assert L.shiftattn_proj_workspace_bytes(-1, 10240, 8192) == 0 and L.shiftattn_proj_workspace_bytes(8, 0, 8192) == 0
    # empty problems are valid no-ops and touch nothing
    assert q(None, None, None, 0, 0, 8192, ctypes.byref(x), None) == B.OK
    assert o(None, None, None, 0, 8, 8192, ctypes.byref(xo), None) == B.OK


def test_fp8_projection_entry_points_reject_bad_arguments(B):
    """Row quantiser and the projections over FP8 E4M3 codes: every case fails validation before anything is launched."""
    L = B.lib()
    ok = dict(P=8, num_q_heads=64, num_kv_heads=8, head_dim=128, dtype=B.BF16)
    x, xo = _xchg(B, **ok), _xchg(B, **{**ok, "num_kv_heads": 0})
    qr, qv, q8, o8 = L.shiftattn_quantize_rows_fp8, L.shiftattn_quantize_recv_fp8, L.shiftattn_qkv_proj_pack_fp8, L.shiftattn_unpack_o_proj_fp8
    assert qr(FAKE, FAKE, FAKE, -1, 64, None) == B.EINVAL and qr(FAKE, FAKE, FAKE, 4, 0, None) == B.EINVAL
    assert qr(FAKE, FAKE, FAKE, 4, 12, None) == B.EUNSUPPORTED                 # cols no multiple of 8
    assert qr(None, FAKE, FAKE, 4, 64, None) == B.EINVAL and qr(FAKE, None, FAKE, 4, 64, None) == B.EINVAL
    assert qr(FAKE, FAKE, None, 4, 64, None) == B.EINVAL
    assert qr(ctypes.c_void_p(0x1008), FAKE, FAKE, 4, 64, None) == B.EINVAL    # x not 16-byte aligned
    assert qr(FAKE, FAKE, ctypes.c_void_p(0x1002), 4, 64, None) == B.EINVAL    # scales not 4-byte aligned
    assert qr(None, None, None, 0, 64, None) == B.OK
    assert qv(FAKE, FAKE, FAKE, 9, 8, ctypes.byref(xo), None) == B.EINVAL      # T > T_pad
    assert qv(FAKE, FAKE, FAKE, 8, 8, ctypes.byref(_xchg(B, **{**ok, "dtype": B.F32, "num_kv_heads": 0})), None) == B.EUNSUPPORTED
    assert qv(FAKE, FAKE, FAKE, 8, 8, None, None) == B.EINVAL and qv(None, FAKE, FAKE, 8, 8, ctypes.byref(xo), None) == B.EINVAL
    assert qv(None, None, None, 0, 8, ctypes.byref(xo), None) == B.OK
    for kw, d_model in [(dict(dtype=B.F32), 8192), (dict(head_dim=64), 8192), (dict(), 8200), (dict(num_q_heads=9, num_kv_heads=1, P=1), 8192)]:
        bad = _xchg(B, **{**ok, **kw})
        assert q8(FAKE, FAKE, FAKE, FAKE, FAKE, 8, 8, d_model, ctypes.byref(bad), None) == B.EUNSUPPORTED, (kw, d_model)
    assert o8(FAKE, FAKE, FAKE, FAKE, FAKE, 8, 8, 8192 + 64, ctypes.byref(xo), None) == B.EUNSUPPORTED
    for fn, desc in ((q8, x), (o8, xo)):
        assert fn(FAKE, FAKE, FAKE, FAKE, FAKE, 9, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, FAKE, FAKE, FAKE, FAKE, 8, 8, 0, ctypes.byref(desc), None) == B.EINVAL
        assert fn(FAKE, FAKE, FAKE, FAKE, FAKE, 8, 8, 8192, None, None) == B.EINVAL
        for hole in range(5):
            args = [FAKE] * 5
            args[hole] = None
            assert fn(*args, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL, hole
        assert fn(FAKE, ctypes.c_void_p(0x1002), FAKE, FAKE, FAKE, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert fn(ctypes.c_void_p(0x1008), FAKE, FAKE, FAKE, FAKE, 8, 8, 8192, ctypes.byref(desc), None) == B.EINVAL
        assert B.last_error()
    assert q8(None, None, None, None, None, 0, 0, 8192, ctypes.byref(x), None) == B.OK
    assert o8(None, None, None, None, None, 0, 8, 8192, ctypes.byref(xo), None) == B.OK


def test_unified_batches_whose_decode_rows_outweigh_the_chunks_take_two_launches(B):
    """One launch for both kinds of rows holds the partial results of both, two launches share the workspace: where the key
    ranges of the chunks have partial results, the size shows which it is.  With decode rows that outlast the tiles on the
    workgroups that the tiles leave them, one launch took up to 28 % longer than two."""
    def sizes(chunks, num_dec, max_dec, hq, hkv):
        a = _attn(B, num_q_heads=hq, num_kv_heads=hkv, max_blocks_per_seq=(max(max_dec, max(c[1] for c in chunks)) + 15) // 16)
        n, tot, mq, mp = len(chunks), sum(c[0] for c in chunks), max(c[0] for c in chunks), max(c[1] for c in chunks)
        return (B.mixed_workspace_bytes(n, tot, mq, mp, num_dec, max_dec, a),
                max(B.prefill_workspace_bytes(n, tot, mq, mp, a), B.decode_workspace_bytes(num_dec, max_dec, a)))

    for chunks, num_dec, max_dec, hq, hkv in [([(367, 867)] * 4, 115, 12474, 16, 2), ([(968, 968)] * 2, 64, 22991, 16, 2),
                                              ([(263, 2263)] * 6, 105, 19047, 16, 2)]:
        both, larger = sizes(chunks, num_dec, max_dec, hq, hkv)
        assert both == larger, (chunks, num_dec)
    for chunks, num_dec, max_dec, hq, hkv in [([(2048, 133120)], 64, 32768, 8, 1), ([(33, 2000)], 7, 5000, 8, 1)]:
        both, larger = sizes(chunks, num_dec, max_dec, hq, hkv)
        assert both > larger, (chunks, num_dec)


@pytest.mark.parametrize("chunks,num_dec,max_dec,hq", [
    ([(244, 39305)], 19, 2209, 5),     # 55.1 us on the 128-column kernel, 59.9 in two groups of 64-column wavefronts
    ([(1579, 3676)], 31, 5516, 8),     # 53.6 and 58.0
    ([(120, 32556)], 30, 5061, 8),     # 52.9 and 56.2
    ([(545, 8155)], 71, 1094, 8),      # 45.3 and 48.0
    ([(312, 1300)] * 4, 0, 0, 16),     # (alone in ranges of 1400 keys on: 312 tokens on 1799 38.2 and 32.9)
])
def test_short_key_ranges_stay_with_the_128_column_kernel(B, chunks, num_dec, max_dec, hq):
    """What two groups of wavefronts gain in their key loop they lose around it where a range holds few keys: less than 1400, less
    than 2400 beside decode rows."""
    a = _attn(B, num_q_heads=hq, num_kv_heads=2 if hq == 16 else 1, max_blocks_per_seq=(max(max_dec, max(c[1] for c in chunks)) + 15) // 16)
    p = B.prefill_plan(len(chunks), sum(c[0] for c in chunks), max(c[0] for c in chunks), max(c[1] for c in chunks), a, num_dec, max_dec)
    assert (p.tile_columns, p.wave_columns) == (128, 32) and (p.decode_wgs > 0) == (num_dec > 0)


def test_two_unequal_prompts_are_priced_for_the_half_of_the_chip_that_each_sees(B):
    """5068 and 8739 tokens of five heads per KV head: in two groups of wavefronts, heads stacked, the longer prompt runs on every second die
    (176 us); the 128-column kernel takes the heads one by one and meets them all (160)."""
    a = _attn(B, num_q_heads=5, max_blocks_per_seq=547)
    p = B.prefill_plan(2, 5068 + 8739, 8739, 8739, a)
    assert (p.tile_columns, p.wave_columns, p.key_ranges) == (128, 32, 1)


def test_projections_name_a_kernel_that_is_built(B):
    """Every size takes one of the two projection kernels: the weight-streaming one with as many token pieces as cover the rows, in an
    instance that is built (the query fails otherwise), or the tiled one.  40 features a workgroup and more than 96 rows have no
    instance: a ring of one step."""
    for fp8 in (False, True):
        for n in (256, 768, 1280, 2304, 4096, 5120, 6144, 8192, 8448, 10240, 10496, 17408, 20480, 20736):
            for k in (64, 128, 512, 2048, 4096, 5120, 8192, 8256, 16384, 65536):
                for rows in range(1, 131):
                    for ws in (None, 0, 1024):
                        p = B.proj_plan(rows, n, k, fp8, ws)
                        assert p.k_ranges >= 1
                        if p.streams:
                            assert 8 * p.token_pieces >= rows and p.feature_pieces in range(1, 6) and p.token_pieces + p.feature_pieces <= 20
                        else:
                            assert rows > 16 or k % (128 if fp8 else 64), (rows, n, k, fp8, ws)
                            assert p.tile_features in (128, 256) and p.tile_tokens in (128, 256)
    assert [B.proj_plan(r, 10240, 512).streams for r in (96, 97, 128)] == [1, 0, 0]
    assert [B.proj_plan(r, 8192, 512).streams for r in (96, 97, 128, 129)] == [1, 1, 1, 0]
    q = B.lib().shiftattn_proj_plan
    plan = B.ProjPlan()
    assert q(8, 256, 512, 0, 0, None) == B.EINVAL
    assert q(0, 256, 512, 0, 0, ctypes.byref(plan)) == B.EINVAL and q(8, 0, 512, 0, 0, ctypes.byref(plan)) == B.EINVAL
    assert q(8, 128, 512, 0, 0, ctypes.byref(plan)) == B.EUNSUPPORTED and q(8, 256, 96, 0, 0, ctypes.byref(plan)) == B.EUNSUPPORTED
    try:
        B.set_option(B.OPT_GENERIC_ONLY, 1)
        assert B.proj_plan(1, 10240, 8192).streams == 0
    finally:
        B.set_option(B.OPT_GENERIC_ONLY, 0)


def test_few_features_with_long_rows_of_weights_split_k(B):
    """A block's workgroup walks all of k: with few features that is one long chain on part of the chip, so k goes over several
    workgroups where the workspace that the size query names has room for their sums, and never takes more than was given."""
    for fp8 in (False, True):
        e = 1 if fp8 else 2
        for rows in (17, 24, 32, 33, 48, 64):
            for n in (256, 512, 1024, 1536, 2304):
                for k_bytes in (32768, 65536):
                    p = B.proj_plan(rows, n, k_bytes // e, fp8)
                    assert p.k_ranges > 1, (rows, n, k_bytes, fp8)
                    assert not p.streams or p.k_ranges * rows * n * 4 <= B.proj_workspace_bytes(rows, n, k_bytes // e, fp8)
                    room = 2 * rows * n * 4
                    assert B.proj_plan(rows, n, k_bytes // e, fp8, room).k_ranges <= 2
                    assert B.proj_plan(rows, n, k_bytes // e, fp8, room - 1).k_ranges == 1
    assert [B.proj_plan(r, 256, 65536).k_ranges for r in (1, 8, 16)] == [8, 8, 8]
    assert B.proj_plan(48, 3072, 12288).streams == 0   # the tiled kernel is the faster one
    assert B.proj_plan(32, 2304, 16384).streams == 1 and B.proj_plan(64, 1024, 8192).streams == 1
