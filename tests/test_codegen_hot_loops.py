"""Host-side check of the generated code (no GPU): the steady-state loops of the two MFMA-bound kernels that run one
wavefront per SIMD hold no register spills.

Both kernels sit at the edge of the register file, and a spill that lands inside the loop costs far more than its
instruction: a scratch load shares the vector-memory counter with the direct-to-LDS loads.  A wait for all of them then
waits for it too (a one-line change of a loop bound that moved one scratch load into the 256-column prefill kernel's loop
made every launch 4-5 % slower, with every test green), and a wait that counts the newest loads, as the 64-column
wavefronts' does, would let the tile it needs be one load short.  The check compiles the source to assembly with the
build's own flags and looks at the basic blocks that carry the loops' MFMAs.
"""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2509_16495_amd import build as BLD

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc to compile to assembly")


@functools.lru_cache(maxsize=None)
def _assembly(source):
    """Lines of the source's gfx950 assembly, compiled once with the build's own flags."""
    flags = [f for f in BLD.FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, source + ".s")
        subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", os.path.join(BLD.CSRC, source), "-o", out],
                              cwd=BLD.CSRC, stderr=subprocess.DEVNULL)
        return tuple(open(out))


def _kernel_lines(source, kernel_substr):
    """Those of the kernel whose mangled name contains `kernel_substr`."""
    lines, inside = [], False
    for line in _assembly(source):
        if re.match(r"^[A-Za-z_$][\w.$]*:", line):
            inside = kernel_substr in line
        elif line.startswith(".Lfunc_end"):
            inside = False
        elif inside:
            lines.append(line)
    return lines


def _blocks_of(source, kernel_substr, tmp_path):
    """Basic blocks of the kernel whose mangled name contains `kernel_substr`: [label, mfmas, spill ops, instructions]."""
    out = os.path.join(str(tmp_path), source + ".s")
    flags = [f for f in BLD.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", os.path.join(BLD.CSRC, source), "-o", out],
                          cwd=BLD.CSRC, stderr=subprocess.DEVNULL)
    blocks, cur, inside = [], None, False
    for line in open(out):
        s = line.strip()
        m = re.match(r"^([A-Za-z_.$][\w.$]*):", line)
        if m and not m.group(1).startswith(".L"):      # a function label
            inside = kernel_substr in m.group(1)
            cur = None
            continue
        if not inside:
            continue
        if m:
            cur = [m.group(1), 0, 0, 0]
            blocks.append(cur)
        elif cur is not None and s and not s.startswith((";", ".")):
            cur[3] += 1
            cur[1] += "v_mfma" in s
            cur[2] += ("scratch_" in s) or ("v_readlane" in s) or ("v_writelane" in s)
    return blocks


# template arguments <decode role, scaled Q, groups> of the instances of the 64-column wavefronts' kernel
PREFILL64 = [(d, q, 1) for q in (0, 1) for d in (0, 1, 2)] + [(d, 0, 2) for d in (0, 1, 2)]


@pytest.mark.parametrize("decode,scaled_q,groups", PREFILL64)
def test_prefill64_steady_state_loops_have_no_spills(decode, scaled_q, groups):
    """Every instance holds fourteen bodies of an iteration, 32 MFMAs each in two blocks (the second with the direct-to-LDS loads of a tile,
    twice as many with two groups): four of the steady loop and three behind it, whose MFMAs carry wait states, for the first attempt at a
    pass and as many, with a maximum per two logits, for those that follow the maximum."""
    blocks = []
    for line in _kernel_lines("prefill_mfma64.hip", f"prefill64_kernelILi{decode}ELb{scaled_q}ELi{groups}E"):
        text = line.split(";")[0].strip()
        if re.match(r"^\.LBB", line):
            blocks.append([])
        elif blocks and text and not text.startswith("."):
            blocks[-1].append(text.split()[0])
    assert not [op for b in blocks for op in b if op.startswith("scratch_")]

    def count(ops, *names):
        return sum(op.startswith(names) for op in ops)

    kinds = {}
    for front, body in zip(blocks, blocks[1:]):
        if count(body, "global_load_lds_dwordx4") != 4 * groups or count(body, "v_mfma") < 20:
            continue
        both = front + body
        assert count(both, "v_mfma") == 32 and count(front, "s_barrier") == 1
        waits = sum(a == "s_nop" and b.startswith("v_mfma") for a, b in zip(both, both[1:]))
        follows = count(both, "v_max3_f32")
        assert waits in (0, 32) and follows in (0, 16)
        kinds[waits > 0, follows > 0] = kinds.get((waits > 0, follows > 0), 0) + 1
        # (the rare attempts of two groups want one scalar register too many: it comes back from a vector lane once a trip)
        allowed = 0 if follows == 0 or groups == 1 else 1 if waits == 0 else 2
        assert count(both, "v_readlane", "v_writelane") <= allowed
    assert kinds == {(False, False): 4, (True, False): 3, (False, True): 4, (True, True): 3}


def test_proj_gemm_main_loop_has_no_spills(tmp_path):
    for kernel in ("proj_gemm_kernelILb0ELb0", "proj_gemm_kernelILb1ELb0"):   # bf16 and FP8, not split over k
        blocks = _blocks_of("proj_gemm.hip", kernel, tmp_path)
        loops = [b for b in blocks if b[1] >= 64]                # a stage pair of the main loop: 128 (bf16) or 64 (FP8) MFMAs
        assert loops, (kernel, [tuple(b) for b in blocks if b[1]])
        for b in loops:
            assert b[2] == 0, ("spill traffic in the main loop", kernel, tuple(b))


@pytest.mark.parametrize("fp8", [0, 1])
def test_kv_append_streams_the_rows_of_runs(tmp_path, fp8):
    """Rows of new tokens are read once: the 16-byte loads of the three places that write a run carry the streaming hint, which
    they lose where the compiler merges them with another source (rows written by the kernel in front, 600000 tokens: 123 -> 147 us).
    The two loads of the token-by-token path (windows of many short runs) do without it."""
    out = os.path.join(str(tmp_path), "layout.s")
    flags = [f for f in BLD.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", os.path.join(BLD.CSRC, "layout_kernels.hip"), "-o", out],
                          cwd=BLD.CSRC, stderr=subprocess.DEVNULL)
    loads, inside = [], False
    for line in open(out):
        if re.match(r"^[A-Za-z_$]", line):
            inside = f"kv_write_block_kernelILb{fp8}E" in line.split(":")[0]
        elif inside and "global_load_dwordx4" in line:
            loads.append(line.split("//")[0].rstrip().endswith(" nt"))
    assert loads.count(True) >= 4 and loads.count(False) <= 2, loads


def test_prefill_key_loop_forms_its_addresses_in_scalar_registers(tmp_path):
    """128-column kernel, the steady-state loop of two tiles a trip: block ids are uniform, so their addresses cost the vector unit
    nothing; an id that the compiler takes for different per lane moves three multiplications and the loads' bases there."""
    out = os.path.join(str(tmp_path), "prefill.s")
    flags = [f for f in BLD.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", os.path.join(BLD.CSRC, "prefill_mfma.hip"), "-o", out],
                          cwd=BLD.CSRC, stderr=subprocess.DEVNULL)
    blocks, kernel = [], ""
    for line in open(out):
        m = re.match(r"^([A-Za-z_.$][\w.$]*):", line)
        if m and not m.group(1).startswith(".L"):
            kernel = m.group(1)
        elif m:
            blocks.append((kernel, []))
        elif blocks and line.startswith("\t") and line[1:2].isalpha():
            blocks[-1][1].append(line.split()[0])
    loops = [i for i, (k, b) in enumerate(blocks) if "prefill_kernelILi" in k and sum("mfma" in x for x in b) >= 16 and b.count("global_load_lds_dwordx4") == 8]
    assert len(loops) == 3, [(k, len(b)) for k, b in (blocks[i] for i in loops)]   # one of each instance
    for i in loops:
        for k, b in blocks[i:i + 2]:
            assert sum("mfma" in x for x in b) >= 15
            assert not [x for x in b if x.startswith(("v_readfirstlane", "v_readlane", "v_mul_lo_u32", "v_mad_u64_u32"))], k


def _unsynchronised_parks(lines):
    """Of one kernel's assembly: (parks seen, those of them that an MFMA reaches without an s_barrier in between).  A park is a run of
    sixteen 16-byte LDS stores 1 KiB apart: what a lane leaves for the other group."""
    blocks, labels = [[]], {}
    for line in lines:
        s = line.split(";")[0].strip()
        m = re.match(r"^(\.LBB[\w.$]*):", line)
        if m:
            blocks.append([])
            labels[m.group(1)] = len(blocks) - 1
        elif s and not s.startswith(".") and not s.endswith(":"):
            blocks[-1].append(s.split())
            if s.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                blocks.append([])

    def walk(i, dirty):
        """Through block i, entered with an MFMA behind the last barrier or not: (the same at its end, parks, those that are dirty)."""
        run = parks = bad = 0
        for op in blocks[i]:
            if op[0].startswith("v_mfma"):
                dirty = True
            elif op[0] == "s_barrier":
                dirty, run = False, 0
            elif op[0] == "ds_write_b128":
                offset = next((int(x[7:]) for x in op if x.startswith("offset:")), 0)
                run = run + 1 if offset == 1024 * run else int(offset == 0)
                parks += run == 16
                bad += run == 16 and dirty
        return dirty, parks, bad

    def successors(i):
        last = blocks[i][-1] if blocks[i] else [""]
        if last[0].startswith(("s_cbranch", "s_branch")):
            yield labels[last[1]]
        if not last[0].startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            yield i + 1

    entered, work = [False] * len(blocks), list(range(len(blocks)))
    while work:
        i = work.pop()
        if walk(i, entered[i])[0]:
            for n in successors(i):
                if not entered[n]:
                    entered[n] = True
                    work.append(n)
    found = [walk(i, entered[i]) for i in range(len(blocks))]
    return sum(f[1] for f in found), sum(f[2] for f in found)


@pytest.mark.parametrize("decode", [0, 1, 2])
def test_two_groups_exchange_their_sums_behind_a_barrier(decode):
    """The two-group form of the 64-column wavefronts parks accumulators in the bytes of its key rings.  Whichever attempt a pass ends
    with, a barrier lies between the last product of every wavefront and the first parked accumulator: one group may be a whole tile
    ahead of the other, whose operands it would overwrite."""
    parks, bad = _unsynchronised_parks(_kernel_lines("prefill_mfma64.hip", f"prefill64_kernelILi{decode}ELb0ELi2E"))
    assert parks >= 1 and bad == 0, (parks, bad)
