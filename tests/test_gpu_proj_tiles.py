"""The projections at the edges of the large-batch kernel's tile shapes (256 x 256, 256 x 128 and 128 x 128 features x token
rows, two to four k stages in LDS), and of the streaming kernel for k = 5120, over bf16 and FP8 operands.  The checks
(oracle, tolerances) are those of test_gpu_proj_small.py and test_gpu_proj_fp8.py; the sizes are chosen for what the planner
does with them."""
import pytest
from test_gpu_proj_fp8 import test_o_projection_fp8 as _o_fp8
from test_gpu_proj_fp8 import test_qkv_projection_fp8 as _qkv_fp8
from test_gpu_proj_small import test_small_o_projection as _o_bf16
from test_gpu_proj_small import test_small_qkv_projection as _qkv_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_backend
    return gpu_backend


QKV = [
    # P, h, h_kv, d_model, T, T_pad
    (8, 64, 8, 512, 2100, 2104),   # a round of 256 x 256 tiles, the last token rows in 256 x 128
    (8, 64, 8, 512, 1700, 1700),   # bf16: a round of 256 x 128 tiles, the rest in 256 x 256
    (8, 32, 4, 2048, 900, 904),    # 256 x 128 tiles, the last one 4 rows high; KV replication
    (4, 8, 1, 192, 129, 132),      # 128 x 128: fewer k stages than buffers, half a last stage with FP8, one row in the last tile
    (2, 8, 4, 448, 128, 128),      # half a last stage with FP8: 128 x 128, as many token rows as a tile; bf16: the streaming kernel's 128 rows
    (1, 4, 1, 512, 127, 128),      # streaming kernel: 127 rows and a padding row
    (8, 8, 8, 4096, 260, 264),     # 128 x 128 with k ranges over three token tiles
    (8, 8, 8, 5120, 16, 16),       # streaming kernel: ten (FP8: five) steps of k per wavefront
    (8, 8, 8, 5120, 29, 32),       # four pieces of token rows, padding rows in the last
]
O = [
    # P, hq_l, d_model, T, T_pad
    (2, 4, 768, 385, 390),         # 128 x 128, k through two receive buffers, one row in the last tile
    (4, 10, 2560, 200, 201),       # k = 5120 over four buffers
    (4, 10, 512, 30, 32),
]


@pytest.mark.parametrize("give_workspace", [True, False])
@pytest.mark.parametrize("case", QKV)
def test_qkv(oracle, G, case, give_workspace):
    _qkv_bf16(oracle, G, *case, give_workspace)
    _qkv_fp8(oracle, G, *case, give_workspace)


@pytest.mark.parametrize("give_workspace", [True, False])
@pytest.mark.parametrize("case", O)
def test_o(oracle, G, case, give_workspace):
    _o_bf16(oracle, G, *case, give_workspace)
    _o_fp8(oracle, G, *case, give_workspace)


# One 128 x 128 tile of token rows: full, one row short, and that row as padding.  k is too long for the streaming kernel; 4160 leaves half a last stage with FP8, 4224 does not.
TILE_ROWS = [
    # P, h, h_kv, d_model, T, T_pad
    (2, 8, 4, 4160, 128, 128),
    (1, 4, 1, 4160, 127, 128),
    (1, 4, 1, 4224, 127, 128),
    (2, 8, 4, 4224, 128, 128),
    (4, 8, 8, 4224, 127, 127),
]


@pytest.mark.parametrize("give_workspace", [True, False])
@pytest.mark.parametrize("case", TILE_ROWS)
def test_rows_of_one_tile(oracle, G, case, give_workspace):
    from paper_2509_16495_amd import binding as B
    _, h, h_kv, d_model, _, T_pad = case
    for fp8 in (False, True):
        p = B.proj_plan(T_pad, (h + 2 * h_kv) * 128, d_model, fp8, None if give_workspace else 0)
        assert (p.streams, p.tile_features, p.tile_tokens) == (0, 128, 128)
    _qkv_bf16(oracle, G, *case, give_workspace)
    _qkv_fp8(oracle, G, *case, give_workspace)


# Token tiles that hold padding rows only (of 128 rows, of 256, or both): their loads count from a row that exists, their
# result is zeros.
PADDING = [
    # P, h, h_kv, d_model, T, T_pad
    (8, 64, 8, 512, 128, 129),
    (8, 32, 4, 2048, 384, 385),    # KV replication
    (1, 4, 1, 512, 256, 257),
    (4, 8, 1, 192, 128, 700),      # several tiles behind the last token; half a last stage with FP8
    (2, 8, 4, 448, 1, 300),
    (8, 8, 8, 4096, 130, 520),     # k ranges: the tiles leave no partial results
    (8, 64, 8, 512, 1700, 2300),   # rounds of whole tiles, the rest behind them
]


@pytest.mark.parametrize("give_workspace", [True, False])
@pytest.mark.parametrize("case", PADDING)
def test_tiles_of_padding_rows(oracle, G, case, give_workspace):
    _qkv_bf16(oracle, G, *case, give_workspace)
    _qkv_fp8(oracle, G, *case, give_workspace)
