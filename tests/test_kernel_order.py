"""What the compiler cannot see, in the assembly of the kernels as built (no GPU): products written as asm, whose results it takes to be
there at once, have every other instruction that touches such a result far enough behind them; barriers written by hand, which it
does not wait in front of, have no LDS read of a buffer they free behind them; requests written as asm, which it does not count, are
waited for by no wait of its own inside a loop."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_13333_amd import build as B

PRODUCT = 8   # wait states of a 32x32x16 product (8 passes)
NEEDED = 24   # three products; the hardware asks for 11 wait states


def _regs(op):
    m = re.match(r"v\[(\d+):(\d+)\]$", op)
    if m:
        return range(int(m[1]), int(m[2]) + 1)
    m = re.match(r"v(\d+)$", op)
    return [int(m[1])] if m else []


def _blocks(lines):
    """Basic blocks of a kernel: lists of (mnemonic, operands, written as asm), and the successors of each."""
    blocks, names, asm = [[]], {}, False
    for line in lines:
        asm = (asm or "ASMSTART" in line) and "ASMEND" not in line
        t = line.split(";")[0].strip()
        if re.match(r"\.?L?\w*:$", t) and t.startswith(".L"):
            blocks.append([])
            names[t[:-1]] = len(blocks) - 1
        elif t and not t.startswith(".") and not t.endswith(":"):
            p = t.replace(",", " ").split()
            blocks[-1].append((p[0], p[1:], asm))
            if p[0].startswith(("s_branch", "s_cbranch", "s_endpgm")):
                blocks.append([])
    succ = []
    for i, b in enumerate(blocks):
        last = b[-1] if b else ("", [], False)
        s = [names[last[1][-1]]] if last[0].startswith(("s_branch", "s_cbranch")) else []
        if not last[0].startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            s.append(i + 1)
        succ.append(s)
    return blocks, succ


def shortest_distances(lines):
    """Per kernel: the smallest number of wait states, over all paths, between an asm product into VGPRs and the first
    instruction that is no product and reads or writes them; only products and s_nop are counted."""
    blocks, succ = _blocks(lines)
    entry = [None] * len(blocks)
    entry[0] = {}
    work, least, seen = [0], 10 ** 6, 0
    while work:
        i = work.pop()
        state = dict(entry[i])
        for op, args, asm in blocks[i]:
            if op.startswith("v_mfma"):
                state = {r: d + PRODUCT for r, d in state.items() if d + PRODUCT < 8 * NEEDED}
                if asm and args[0].startswith("v"):
                    seen += 1
                    state.update((r, 0) for r in _regs(args[0]))
            elif op == "s_nop":
                state = {r: d + int(args[0]) + 1 for r, d in state.items()}
            elif op.startswith(("v_", "ds_", "buffer_", "global_")):
                for r in {r for a in args for r in _regs(a)}:
                    least = min(least, state.pop(r, 10 ** 6))
        for j in succ[i]:
            if entry[j] is None:
                entry[j] = state
                work.append(j)
            else:
                merged = {r: min(entry[j].get(r, 10 ** 6), state.get(r, 10 ** 6)) for r in {*entry[j], *state}}
                if merged != entry[j]:
                    entry[j] = merged
                    work.append(j)
    return least, seen


def _assembly(tmp_path_factory, source):
    if not shutil.which("hipcc"):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("asm") / "kernels.s"
    subprocess.run(["hipcc", *B.FLAGS, "-w", "--offload-device-only", "-S", os.path.join(B.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    return out.read_text()


def test_fp32_attention_up_to_heads_of_96_uses_no_scratch_memory(tmp_path_factory):
    """(Above that the dK / dV part spills.)"""
    text = _assembly(tmp_path_factory, "attention_f32.hip")
    scratch = {m[1]: int(m[2]) for m in re.finditer(r"\.name:\s+(\S*attn_\w+)\n\s+\.private_segment_fixed_size:\s+(\d+)", text)}
    assert len(scratch) == 16
    assert all(n == 0 for k, n in scratch.items() if "kernelILi4E" not in k), scratch


@pytest.fixture(scope="module")
def attention_asm(tmp_path_factory):
    kernels, cur = {}, None
    for line in _assembly(tmp_path_factory, "attention_bf16.hip").splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = kernels.setdefault(m[1], [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            cur.append(line)
    return kernels


@pytest.mark.parametrize("form", ["ILi64ELi1E", "ILi128ELi1E", "ILi128ELi2E"])
def test_first_reader_of_an_asm_product(attention_asm, form):
    (lines,) = [v for k, v in attention_asm.items() if "attn_dkv_kernel" + form in k]
    least, seen = shortest_distances(lines)
    assert seen >= 8  # the kernel has such products
    assert NEEDED <= least < 10 ** 6, least


def test_first_reader_of_an_asm_product_where_ds_is_stored(attention_asm):
    (lines,) = [v for k, v in attention_asm.items() if "attn_dkv_ds_kernel" in k]
    least, seen = shortest_distances(lines)
    assert seen >= 8
    assert NEEDED <= least < 10 ** 6, least


@pytest.mark.parametrize("form", ["ILi64E", "ILi128E"])
def test_first_reader_of_an_asm_product_in_the_shared_launch(attention_asm, form):
    (lines,) = [v for k, v in attention_asm.items() if "attn_bwd_kernel" + form in k]
    least, seen = shortest_distances(lines)
    assert seen >= 8
    assert NEEDED <= least < 10 ** 6, least


def test_only_the_kernel_of_few_workgroups_stores_ds(attention_asm):
    """Two stores through a buffer descriptor per step and key tile there; the other forms of the kernel hold none of it."""
    stores = {k: sum("buffer_store" in line for line in v) for k, v in attention_asm.items() if "attn_dkv" in k}
    assert len(stores) == 4
    for k, n in stores.items():
        assert n == (2 if "attn_dkv_ds_kernel" in k else 0), k


def reads_at_barriers(lines):
    """For every barrier of a kernel the largest number of LDS reads, over all paths, that may not have returned there."""
    blocks, succ = _blocks(lines)
    entry, work, at = {0: 0}, [0], {}
    while work:
        i = work.pop()
        n = entry[i]
        for j, (op, args, _) in enumerate(blocks[i]):
            if op.startswith("ds_read"):
                n = min(n + 1, 64)
            elif op == "s_waitcnt":
                n = min([n] + [int(m[1]) for m in (re.match(r"lgkmcnt\((\d+)\)", a) for a in args) if m])
            elif op == "s_barrier":
                at[i, j] = max(at.get((i, j), 0), n)
        for k in succ[i]:
            if k not in entry or entry[k] < n:
                entry[k] = n
                work.append(k)
    return list(at.values())


@pytest.mark.parametrize("kernel", ["attn_fwd_pair_kernelILi64E", "attn_fwd_pair_kernelILi128E", "attn_fwd_kernelILi64E", "attn_fwd_kernelILi128E",
                                    "attn_dq_kernelILi64E", "attn_dq_kernelILi128E", "attn_dq_ds_kernelILi128E"])
def test_no_lds_read_is_under_way_at_a_barrier_that_frees_its_buffer(attention_asm, kernel):
    """Behind the barrier any wavefront may have the buffer filled again."""
    (lines,) = [v for k, v in attention_asm.items() if kernel in k]
    at = reads_at_barriers(lines)
    assert at and max(at) == 0, at


def compiler_waits_in_loops(lines):
    """The waits for memory requests inside a kernel's loops that are not written as asm."""
    blocks, succ = _blocks(lines)

    def in_loop(i):
        seen, work = set(), list(succ[i])
        while work:
            k = work.pop()
            if k not in seen:
                seen.add(k)
                work += succ[k]
        return i in seen
    return [a for i, b in enumerate(blocks) if in_loop(i) for op, args, asm in b if op == "s_waitcnt" and not asm for a in args if a.startswith("vmcnt")]


@pytest.mark.parametrize("kernel", ["attn_fwd_pair_kernelILi64E", "attn_fwd_pair_kernelILi128E", "attn_fwd_kernelILi64E", "attn_fwd_kernelILi128E",
                                    "attn_bwd_kernelILi64E", "attn_bwd_kernelILi128E", "attn_dq_kernelILi64E", "attn_dq_kernelILi128E",
                                    "attn_dkv_kernelILi64ELi1E", "attn_dkv_kernelILi128ELi1E", "attn_dkv_kernelILi128ELi2E", "attn_dkv_ds_kernelILi128ELi1E"])
def test_the_compiler_waits_for_no_request_of_the_loop(attention_asm, kernel):
    """Its wait for what it loaded before the loop (rows of Q or dO, row statistics) would be one for the next block's requests too."""
    (lines,) = [v for k, v in attention_asm.items() if kernel in k]
    assert compiler_waits_in_loops(lines) == []
