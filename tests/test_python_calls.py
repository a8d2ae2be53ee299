"""What the Python binding's native calls refuse, and with which exception (no GPU work: the checks come before the launch)."""
import contextlib
import ctypes
import os

import numpy as np
import pytest
import torch

BF, F32, U8, I32, I64 = torch.bfloat16, torch.float32, torch.uint8, torch.int32, torch.int64


@pytest.fixture(scope="module")
def B():
    from paper_2509_16495_amd import binding
    if not binding.is_built():
        import __graft_entry__
        __graft_entry__.build()
    binding.lib()
    return binding


def _z(*shape, dtype=BF):
    return torch.zeros(shape, dtype=dtype)


def _attn(**kw):
    a = dict(q=_z(5, 4, 64), cache=_z(3, 1, 2, 16 * 64), table=_z(2, 2, dtype=I32), cu=_z(3, dtype=I32), lens=_z(2, dtype=I32), out=_z(5, 4, 64),
             k=_z(5, 1, 64), v=_z(5, 1, 64), slots=_z(5, dtype=I64), scale=0.1)
    a.update(kw)
    return a


@contextlib.contextmanager
def _no_allocation(B):
    def refused(need, like):
        pytest.fail(f"{need} bytes asked for")
    rebind = lambda f: B._calls.bind(f, *[ctypes.cast(getattr(B.lib(), name), ctypes.c_void_p).value for name in B._calls.names])
    rebind(refused)
    try:
        yield
    finally:
        rebind(B._workspace)


def _prefill(B, ws=_z(64, dtype=U8), **kw):
    a = _attn(**kw)
    B.prefill(a["q"], a["cache"], a["table"], a["cu"], a["lens"], 3, 32, a["out"], a["scale"], a["k"], a["v"], a["slots"], workspace=ws)


def _decode(B, ws=_z(64, dtype=U8), **kw):
    a = _attn(**{"lens": _z(5, dtype=I32), "table": _z(5, 2, dtype=I32), **kw})
    B.decode(a["q"], a["cache"], a["table"], a["lens"], 32, a["out"], a["scale"], a["k"], a["v"], a["slots"], workspace=ws)


def _mixed(B, ws=_z(64, dtype=U8), **kw):
    a = _attn(**{"cu": _z(2, dtype=I32), **kw})
    B.mixed(a["q"], a["cache"], a["table"], a["cu"], a["lens"], kw.get("chunks", 1), 4, 32, 32, a["out"], a["scale"], a["k"], a["v"],
            a["slots"], workspace=ws)


REFUSED = [
    (dict(q=_z(5, 4, 64, dtype=torch.float16), out=_z(5, 4, 64, dtype=torch.float16), cache=_z(3, 1, 2, 1024, dtype=U8)), TypeError),
    (dict(out=_z(5, 4, 64, dtype=F32)), AssertionError),
    (dict(out=_z(5, 5, 64)), AssertionError),
    (dict(q=_z(5, 64), out=_z(5, 64)), ValueError),
    (dict(q=_z(4, 5, 64).transpose(0, 1)), AssertionError),               # heads not dense
    (dict(cache=_z(3, 1, 2, 1000)), AssertionError),
    (dict(cache=_z(3, 1, 2, 1024, dtype=F32)), AssertionError),
    (dict(cache=_z(3, 1, 2, 2048)[..., ::2]), AssertionError),            # not contiguous
    (dict(table=_z(2, 2, dtype=I64)), AssertionError),
    (dict(table=_z(4, dtype=I32)), AssertionError),
    (dict(lens=_z(2, dtype=I64)), AssertionError),
    (dict(scale="x"), TypeError),
    (dict(q=np.zeros((5, 4, 64), np.float32)), TypeError),
]


@pytest.mark.parametrize("call", [_prefill, _decode, _mixed])
@pytest.mark.parametrize("kw,error", REFUSED)
def test_attention_calls_refuse(B, call, kw, error):
    with pytest.raises(error):
        call(B, **kw)


@pytest.mark.parametrize("call", [_prefill, _decode, _mixed])
@pytest.mark.parametrize("kw,error", REFUSED + [(dict(lens=torch.tensor(3, dtype=I32)), IndexError)])
def test_attention_calls_refuse_before_they_ask_for_a_workspace(B, call, kw, error):
    """Without a workspace the refusals are the same, and nothing is allocated before them."""
    with pytest.raises(error):
        call(B, **kw)
    with _no_allocation(B), pytest.raises(error):
        call(B, ws=None, **kw)


def test_batches_whose_counts_do_not_fit_are_refused_before_a_size_is_asked_for(B):
    for kw in (dict(chunks=3), dict(lens=_z(9, dtype=I32), table=_z(9, 2, dtype=I32)), dict(cu=_z(3, dtype=I32)), dict(table=_z(3, 2, dtype=I32))):
        for ws in (_z(64, dtype=U8), None):
            with _no_allocation(B), pytest.raises(AssertionError):
                _mixed(B, ws=ws, **kw)


def _accepted():
    """Any call's arguments are fine but for the place they are in: the last thing asked about."""
    return pytest.raises(RuntimeError, match="a tensor on the GPU is wanted")


@pytest.mark.parametrize("ws", [_z(64, dtype=U8), None])
def test_what_the_refusals_start_from_is_accepted(B, ws):
    for call in (_prefill, _decode, _mixed):
        with _no_allocation(B), _accepted():
            call(B, ws=ws)
        with _no_allocation(B), _accepted():   # more rows than are used, rows of a wider tensor, a single row of whatever stride
            call(B, ws=ws, table=_z(9, 2, dtype=I32) if call is not _mixed else _z(2, 2, dtype=I32), q=_z(5, 6, 64)[:, :4],
                 k=_z(7, 3, 64)[:, :1], v=_z(7, 3, 64)[:, 1:2], slots=_z(8, dtype=I64))


@pytest.mark.parametrize("call", [_prefill, _decode, _mixed])
@pytest.mark.parametrize("kw", [
    dict(table=_z(1, 2, dtype=I32)),                                                           # fewer rows than sequences
    dict(k=_z(4, 1, 64), v=_z(4, 1, 64)), dict(k=_z(5, 2, 64), v=_z(5, 2, 64)),                # fewer new rows than rows, more heads than the cache
    dict(k=_z(5, 1, 64, dtype=F32), v=_z(5, 1, 64, dtype=F32)),
    dict(v=_z(4, 1, 64)), dict(v=_z(5, 2, 64)[:, :1]), dict(v=_z(5, 1, 64, dtype=F32)),          # not as k_new
    dict(slots=_z(5, dtype=I32)), dict(slots=_z(4, dtype=I64)), dict(slots=_z(10, dtype=I64)[::2]),
    dict(q=_z(1, 4, 64).expand(5, 4, 64)), dict(k=_z(1, 1, 64).expand(5, 1, 64), v=_z(1, 1, 64).expand(5, 1, 64)),
    dict(out=_z(1, 4, 64).expand(5, 4, 64)), dict(ws=_z(1, dtype=U8).expand(64)), dict(ws=_z(128, dtype=U8)[::2]),
    dict(lens="every second"), dict(cu="every second"),
])
def test_attention_calls_refuse_what_lies_outside_their_tensors(B, call, kw):
    sizes = {"lens": 5 if call is _decode else 2, "cu": 3 if call is _prefill else 2}
    kw = {k: _z(2 * sizes[k], dtype=I32)[::2] if isinstance(v, str) else v for k, v in kw.items()}
    if call is _decode and "cu" in kw:
        return   # (takes none)
    for ws in (_z(64, dtype=U8), None):
        with _no_allocation(B), pytest.raises(AssertionError):
            call(B, **{"ws": ws, **kw})


def test_layout_calls_refuse_what_lies_outside_their_tensors(B):
    with _accepted():
        B.pack_seq2head(_z(4, 6, 64), _z(2, 4, 4, 64), 2, 4, 1)
    with _accepted():
        B.pack_seq2head(_z(4, 4, 64), _z(2, 4, 2, 64), 2, 4, 0)
    for heads in (1, 3, 5):
        with pytest.raises(AssertionError):
            B.pack_seq2head(_z(4, 6, 64), _z(2, 4, heads, 64), 2, 4, 1)
    k, slots, cache = _z(5, 1, 64), _z(5, dtype=I64), _z(3, 1, 2, 1024)
    for good in (cache, _z(3, 1, 2, 1024, dtype=U8)):
        with _accepted():
            B.kv_write(k, k, slots, good)
    for args in ((_z(5, 1, 64, dtype=F32), _z(5, 1, 64, dtype=F32), slots, cache), (k, _z(5, 1, 64, dtype=F32), slots, cache),
                 (k, k, _z(10, dtype=I64)[::2], cache), (_z(1, 1, 64).expand(5, 1, 64), _z(1, 1, 64).expand(5, 1, 64), slots, cache)):
        with pytest.raises(AssertionError):
            B.kv_write(*args)
    for ws, error in ((None, _accepted()), (_z(64, dtype=U8), _accepted()), (_z(128, dtype=U8)[::2], pytest.raises(AssertionError))):
        with error:
            B.qkv_proj_pack(_z(4, 256), _z(768, 256), _z(1, 4, 6, 128), 1, 4, 1, ws)
        with error:
            B.unpack_o_proj(_z(1, 4, 2, 128), _z(256, 256), _z(4, 256), ws)


def test_other_calls_refuse(B):
    with pytest.raises(AssertionError):
        _prefill(B, cu=_z(2, dtype=I32))
    with pytest.raises(AssertionError):
        _prefill(B, k=_z(1, 5, 64).transpose(0, 1).expand(5, 2, 64))
    with pytest.raises(AssertionError):
        _mixed(B, chunks=3)
    for args in ((_z(4, 6, 64), _z(2, 4, 3, 64), 2, 4, 2), (_z(4, 6, 64), _z(2, 4, 4, 64, dtype=F32), 2, 4, 1), (_z(4, 6, 64), _z(3, 4, 4, 64), 2, 4, 1),
                 (_z(6, 4, 64).transpose(0, 1), _z(2, 4, 4, 64), 2, 4, 1)):
        with pytest.raises(AssertionError):
            B.pack_seq2head(*args)
    with pytest.raises(TypeError):
        B.pack_seq2head(_z(4, 6, 64), _z(2, 4, 4, 64), 2.0, 4, 1)
    for args in ((_z(2, 4, 2, 64), _z(4, 5, 64)), (_z(2, 4, 2, 64), _z(4, 4, 64, dtype=F32)), (_z(2, 4, 2, 64), _z(4, 4, 32))):
        with pytest.raises(AssertionError):
            B.unpack_head2seq(*args)
    with pytest.raises(AssertionError):
        B.kv_write(_z(5, 1, 64), _z(5, 1, 64), _z(5, dtype=I32), _z(3, 1, 2, 1024))
    with pytest.raises(AssertionError):
        B.qkv_proj_pack(_z(4, 256), _z(768, 128), _z(1, 4, 6, 128), 1, 4, 1)
    with pytest.raises(AssertionError):
        B.unpack_o_proj(_z(1, 4, 2, 128), _z(256, 128), _z(4, 256))
    with pytest.raises(AssertionError):
        B.quantize_rows_fp8(_z(4, 64), _z(4, 64, dtype=U8), _z(5, dtype=F32))
    with pytest.raises(AssertionError):
        B.quantize_recv_fp8(_z(1, 4, 2, 128), _z(1, 4, 2, 64, dtype=U8), _z(4, dtype=F32))
    with pytest.raises(AssertionError):
        B.qkv_proj_pack_fp8(_z(4, 256, dtype=U8), _z(3, dtype=F32), _z(768, 256, dtype=U8), _z(768, dtype=F32), _z(1, 4, 6, 128), 1, 4, 1)
    with pytest.raises(AssertionError):
        B.unpack_o_proj_fp8(_z(1, 4, 2, 128, dtype=U8), _z(3, dtype=F32), _z(256, 256, dtype=U8), _z(256, dtype=F32), _z(4, 256))


def test_functions_are_matched_by_name(B):
    """The native calls name the functions they want, in their own order; each is one that the header declares."""
    import re
    from paper_2509_16495_amd import _calls
    header = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "shiftattn.h")).read()
    assert len(set(_calls.names)) == len(_calls.names) >= 15
    assert all(re.search(rf"\b{name}\s*\(", header) and hasattr(B.lib(), name) for name in _calls.names)


@pytest.mark.parametrize("missing", ["libshiftattn.so", "_calls.so"])
def test_a_missing_file_is_named_with_the_way_to_build_it(B, tmp_path, missing):
    """A package with one of its two built files only (such files stay behind when the sources move on)."""
    import subprocess
    import sys
    pkg = tmp_path / "paper_2509_16495_amd"
    pkg.mkdir()
    here = os.path.dirname(os.path.abspath(B.__file__))
    for name in {"__init__.py", "binding.py", "libshiftattn.so", "_calls.so"} - {missing}:
        os.symlink(os.path.join(here, name), pkg / name)
    src = "from paper_2509_16495_amd import binding\ntry: binding.lib()\nexcept RuntimeError as e: print('RuntimeError', e)"
    env = {k: v for k, v in os.environ.items() if k != "SHIFTATTN_LIB"}
    out = subprocess.run([sys.executable, "-c", src], cwd=tmp_path, env={**env, "PYTHONPATH": str(tmp_path)}, capture_output=True, text=True)
    assert out.stdout.startswith("RuntimeError") and missing in out.stdout and "paper_2509_16495_amd.build" in out.stdout, out.stdout + out.stderr


@pytest.mark.gpu
def test_a_size_that_the_library_does_not_have_is_left_to_its_own_refusal(B):
    """No workspace given and none computed (head_dim 4): the library says what it refuses."""
    t = lambda *shape, dtype=BF: torch.zeros(shape, dtype=dtype, device="cuda:0")
    q, cache, table, lens, out = t(5, 4, 4), t(3, 1, 2, 64), t(5, 2, dtype=I32), t(5, dtype=I32), t(5, 4, 4)
    with pytest.raises(B.ShiftAttnError, match="head_dim"):
        B.prefill(q, cache, table, t(6, dtype=I32), lens, 3, 32, out, 0.1)
    with pytest.raises(B.ShiftAttnError, match="head_dim"):
        B.decode(q, cache, table, lens, 32, out, 0.1)
    with pytest.raises(B.ShiftAttnError, match="head_dim"):
        B.mixed(q, cache, table, t(2, dtype=I32), lens, 1, 1, 32, 32, out, 0.1)


@pytest.mark.gpu
def test_host_memory_is_refused_unless_the_gpu_can_reach_it(B):
    x = torch.arange(4 * 6 * 64, dtype=torch.int32).remainder(251).to(BF).view(4, 6, 64)
    want, send = torch.zeros((2, 4, 4, 64), dtype=BF, device="cuda:0"), torch.zeros((2, 4, 4, 64), dtype=BF, device="cuda:0")
    B.pack_seq2head(x.to("cuda:0"), want, 2, 4, 1)
    with _accepted():
        B.pack_seq2head(x, send, 2, 4, 1)
    pinned = torch.empty(x.shape, dtype=BF, pin_memory=True)
    pinned.copy_(x)
    B.pack_seq2head(pinned, send, 2, 4, 1)
    assert torch.equal(send, want) and bool(want.any())
