"""The projections of up to 128 token rows at the edges of the weight-streaming kernel against the CPU float64 oracle: every number
of token pieces (8 rows each) and weight pieces (8 features each) of a workgroup, ragged ones of both, more features than one round of
the chip takes, and k of fewer steps than wavefronts, of a number of steps that eight does not divide, and beyond one pass of the ring; with a
workspace, k in ranges over several workgroups.  The host query names the kernel, so a change of the rule fails here.
Tolerance as for all bf16 projections: one rounding of the result (2^-8 |ref|) and the fp32 sums (1e-3 sqrt(K) covers them for
standard normal operands); FP8 operands are exact products of the codes, so the same holds for them."""
import numpy as np
import pytest

from paper_2509_16495_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    # P, h, h_kv, d_model, T, T_pad
    (1, 2, 1, 256, 1, 1),          # 512 features, 4 per workgroup; 4 (FP8: 2) steps of k for eight wavefronts
    (2, 4, 2, 768, 9, 12),         # 12 (6) steps; two token pieces, the second ragged, padding rows
    (8, 8, 8, 1280, 17, 17),       # three token pieces; 20 (10) steps
    (8, 32, 8, 4096, 24, 25),      # 24 and 16 features per workgroup; padding row opens the fourth token piece
    (8, 40, 8, 5120, 31, 32),      # 28 and 20 features per workgroup: ragged weight pieces
    (8, 64, 8, 1024, 33, 33),      # 40 features per workgroup; five token pieces run as six
    (8, 64, 8, 4096, 49, 56),      # 13 pieces a step: four wavefronts
    (1, 64, 8, 512, 64, 64),       # dense rows, one rank
    (8, 120, 8, 768, 40, 41),      # 17408 features: two rounds of the chip
    (8, 120, 8, 768, 12, 12),      # the same, and 15360 k for the output projection: 240 steps
    (1, 8, 1, 1024, 65, 65),       # twelve token pieces, three of them without a row of their own
    (8, 16, 8, 2048, 96, 96),      # 16 features per workgroup
    (2, 8, 2, 768, 97, 103),       # sixteen token pieces, the padding rows open the thirteenth
    (4, 8, 8, 1024, 128, 128),     # 12 features per workgroup: a ragged weight piece under sixteen token pieces
]


# k in ranges: (projection that has them, k ranges with bf16 and with FP8 operands) beside the sizes
RANGES = [
    # P, h, h_kv, d_model, T, T_pad
    (2, 4, 2, 16384, 9, 12, "qkv", 2, 1),      # padding rows: no partial sums, zeros in the send buffers
    (2, 4, 2, 12288, 64, 64, "qkv", 8, 4),     # 192 (96) steps over 64 (32) wavefronts
    (8, 16, 1, 8192, 45, 48, "qkv", 4, 1),     # KV replication; 36 features per workgroup, sixteen pieces a step
    (8, 64, 8, 512, 32, 33, "o", 2, 1),        # the second range starts in the fifth of eight receive buffers
    (4, 256, 8, 256, 1, 1, "o", 8, 8),         # one row; the blocks of features start further apart than a range is long
    (1, 72, 8, 256, 17, 20, "o", 8, 8),        # 144 (72) steps over 64 wavefronts
]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("P,h,h_kv,d_model,T,T_pad,which,bf16_ranges,fp8_ranges", RANGES)
def test_k_ranges_over_workgroups(oracle, P, h, h_kv, d_model, T, T_pad, which, bf16_ranges, fp8_ranges, fp8):
    from paper_2509_16495_amd import binding as B
    n, k, rows = ((h + 2 * h_kv) * 128, d_model, T_pad) if which == "qkv" else (d_model, h * 128, T)
    plan = B.proj_plan(rows, n, k, fp8)
    assert plan.streams and plan.k_ranges == (fp8_ranges if fp8 else bf16_ranges)
    _both_projections(oracle, P, h, h_kv, d_model, T, T_pad, fp8, workspace=True)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("P,h,h_kv,d_model,T,T_pad", CASES)
def test_stream_kernel_edges(oracle, P, h, h_kv, d_model, T, T_pad, fp8):
    from paper_2509_16495_amd import binding as B
    assert B.proj_plan(T_pad, (h + 2 * h_kv) * 128, d_model, fp8, 0).streams and B.proj_plan(T, d_model, h * 128, fp8, 0).streams
    _both_projections(oracle, P, h, h_kv, d_model, T, T_pad, fp8)


def test_k_ranges_in_a_replayed_graph():
    """Both launches of a call in ranges, captured: replays on other inputs of the same buffers, with eager calls between them, give
    the bits of the eager call."""
    import torch
    import gpu_backend as G
    from paper_2509_16495_amd import binding as B
    T, n, k = 40, 512, 16384
    assert B.proj_plan(T, n, k).streams and B.proj_plan(T, n, k).k_ranges > 1
    g = torch.Generator(device=G.DEV)
    g.manual_seed(9)
    recv = torch.randn((8, T, k // 1024, 128), device=G.DEV, generator=g).to(torch.bfloat16)
    w = torch.randn((n, k), device=G.DEV, generator=g).to(torch.bfloat16)
    ws = torch.empty(B.proj_workspace_bytes(T, n, k), dtype=torch.uint8, device=G.DEV)
    out, eager = (torch.empty((T, n), dtype=torch.bfloat16, device=G.DEV) for _ in range(2))
    B.unpack_o_proj(recv, w, out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.unpack_o_proj(recv, w, out, workspace=ws)
    for _ in range(3):
        recv.copy_(torch.randn(recv.shape, device=G.DEV, generator=g))
        out.view(torch.uint8).fill_(0x55)
        graph.replay()
        torch.cuda.synchronize()
        B.unpack_o_proj(recv, w, eager, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.uint8), eager.view(torch.uint8))


# Every instance of the kernel: pieces of eight token rows x pieces of eight features per workgroup (4, 12, 20, 28 and 36 features on 256
# compute units, so the last piece is half empty).  20 and, with FP8 codes, 10 steps of k: the wavefronts have unequal shares, and the
# rings of two steps of the largest instances turn over.
FEATURES = {1: 1024, 2: 3072, 3: 5120, 4: 7168, 5: 9216}
PIECES = [(x, w) for x in (1, 2, 3, 4, 6, 8, 12, 16) for w in FEATURES if (x, w) != (16, 5)]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("token_pieces,feature_pieces", PIECES)
def test_every_instance(token_pieces, feature_pieces, fp8):
    """Both projections at rows that leave the last token piece ragged, against float64 of the same operands."""
    import torch
    import gpu_backend as G
    from paper_2509_16495_amd import binding as B
    n, k = FEATURES[feature_pieces], 1280
    if token_pieces == 16:   # (up to 2 KiB of weights a row in bf16)
        k = 1024
    T = 8 * token_pieces - 3
    plan = B.proj_plan(T, n, k, fp8, 0)
    assert (plan.streams, plan.k_ranges, plan.token_pieces, plan.feature_pieces) == (1, 1, token_pieces, feature_pieces)
    g = torch.Generator(device=G.DEV)
    g.manual_seed(8)
    a = torch.randn((T, k), device=G.DEV, generator=g).to(torch.bfloat16)
    w = torch.randn((n, k), device=G.DEV, generator=g).to(torch.bfloat16)
    out = torch.empty((T, n), dtype=torch.bfloat16, device=G.DEV)
    send = torch.empty((1, T, n // 128, 128), dtype=torch.bfloat16, device=G.DEV)
    for b in (out, send):
        b.view(torch.uint8).fill_(0x55)
    if fp8:
        ac, asc = torch.empty(a.shape, dtype=torch.uint8, device=G.DEV), torch.empty(T, dtype=torch.float32, device=G.DEV)
        wc, wsc = torch.empty(w.shape, dtype=torch.uint8, device=G.DEV), torch.empty(n, dtype=torch.float32, device=G.DEV)
        B.quantize_rows_fp8(a, ac, asc)
        B.quantize_rows_fp8(w, wc, wsc)
        B.unpack_o_proj_fp8(ac.view(1, T, k // 128, 128), asc, wc, wsc, out)
        B.qkv_proj_pack_fp8(ac, asc, wc, wsc, send, 1, n // 128 - 2, 1)
        value = lambda c, s: c.view(torch.float8_e4m3fn).to(torch.float64) * s.double()[:, None]   # noqa: E731
        want = value(ac, asc) @ value(wc, wsc).T
    else:
        B.unpack_o_proj(a.view(1, T, k // 128, 128), w, out)
        B.qkv_proj_pack(a, w, send, 1, n // 128 - 2, 1)
        want = a.double() @ w.double().T
    torch.cuda.synchronize()
    for got in (out, send.view(T, n)):
        err = (got.double() - want).abs()
        assert bool((err <= 2.0 ** -8 * want.abs() + 1e-3 * k ** 0.5).all()), float(err.max())


def _both_projections(oracle, P, h, h_kv, d_model, T, T_pad, fp8, workspace=False):
    import torch
    import gpu_backend as G
    from paper_2509_16495_amd import binding as B
    rng = np.random.Generator(np.random.PCG64(977))
    D, N, K = 128, (h + 2 * h_kv) * 128, h * 128

    def bf16(shape):
        return W.f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))

    x, w_qkv, recv, w_o = bf16((T, d_model)), bf16((N, d_model)), bf16((P, T_pad, h // P, D)), bf16((d_model, K))
    dev = {n: G.t(a, "bf16") for n, a in (("x", x), ("wq", w_qkv), ("recv", recv), ("wo", w_o))}
    send = torch.empty((P, T_pad, h // P + 2 * B.local_kv_heads(P, h_kv), D), dtype=torch.bfloat16, device=G.DEV)
    out = torch.empty((T, d_model), dtype=torch.bfloat16, device=G.DEV)
    send.view(torch.uint8).fill_(0x55)
    out.view(torch.uint8).fill_(0x55)
    ws_q = ws_o = guard = None
    if workspace:   # as large as the size query says, a guard behind it
        need = max(B.proj_workspace_bytes(T_pad, N, d_model, fp8), B.proj_workspace_bytes(T, d_model, K, fp8))
        guard = torch.full((need + 4096,), 0x77, dtype=torch.uint8, device=G.DEV)
        ws_q, ws_o = guard[:B.proj_workspace_bytes(T_pad, N, d_model, fp8)], guard[:B.proj_workspace_bytes(T, d_model, K, fp8)]
    if fp8:
        def quantised(a):
            codes = torch.empty(a.shape, dtype=torch.uint8, device=G.DEV)
            scales = torch.empty(a.shape[0], dtype=torch.float32, device=G.DEV)
            B.quantize_rows_fp8(a, codes, scales)
            return codes, scales
        (xc, xs), (wqc, wqs), (woc, wos) = quantised(dev["x"]), quantised(dev["wq"]), quantised(dev["wo"])
        rc, rs = torch.zeros(dev["recv"].shape, dtype=torch.uint8, device=G.DEV), torch.empty(T, dtype=torch.float32, device=G.DEV)
        B.quantize_recv_fp8(dev["recv"], rc, rs)
        B.qkv_proj_pack_fp8(xc, xs, wqc, wqs, send, P, h, h_kv, workspace=ws_q)
        B.unpack_o_proj_fp8(rc, rs, woc, wos, out, workspace=ws_o)
        f64 = lambda c: c.view(torch.float8_e4m3fn).to(torch.float64).cpu()   # noqa: E731
        X, WQ, WO = (f64(c) * s.double().cpu()[:, None] for c, s in ((xc, xs), (wqc, wqs), (woc, wos)))
        R = f64(rc)[:, :T].permute(1, 0, 2, 3).reshape(T, K) * rs.double().cpu()[:, None]
        qkv, want_out = (X @ WQ.T).view(T, h + 2 * h_kv, D).numpy(), (R @ WO.T).numpy()
        hl, kl = h // P, B.local_kv_heads(P, h_kv)
        want_send = np.zeros((P, T_pad, hl + 2 * kl, D))
        for p in range(P):
            g = p * h_kv // P
            want_send[p, :T] = np.concatenate([qkv[:, p * hl:(p + 1) * hl], qkv[:, h + g:h + g + kl], qkv[:, h + h_kv + g:h + h_kv + g + kl]], axis=1)
    else:
        B.qkv_proj_pack(dev["x"], dev["wq"], send, P, h, h_kv, workspace=ws_q)
        B.unpack_o_proj(dev["recv"], dev["wo"], out, workspace=ws_o)
        want_send = oracle.qkv_proj_pack(x, w_qkv, P, h, h_kv, D, T_pad, "bf16")
        want_out = oracle.unpack_o_proj(recv, w_o, T, "bf16")
    torch.cuda.synchronize()
    for got, want, k in ((send, want_send, d_model), (out, want_out, K)):
        got = W.to_f64(B.to_host(got), "bf16")
        assert np.all(np.isfinite(got))
        err = np.abs(got - want)
        assert np.all(err <= 2.0 ** -8 * np.abs(want) + 1e-3 * np.sqrt(k)), float(err.max())
    assert not np.any(B.to_host(send)[:, T:])
    assert guard is None or bool((guard[-4096:] == 0x77).all())
