"""Registers of the kernels, as the compiler reports them for gfx950 (no GPU needed)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2601_07353_amd import build as B


SOURCES = ("attention.hip", "ahead.hip", "expand.hip", "literal.hip", "select.hip", "accept.hip")


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """{source: (what the compiler says about its kernels, its assembly)}"""
    folder = tmp_path_factory.mktemp("s")

    def one(source):
        path = str(folder / (source + ".s"))
        said = subprocess.run([B._hipcc(), *B.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-S",
                               os.path.join(B.CSRC, source), "-o", path], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True)
        return said.stdout, open(path).read().splitlines()
    with ThreadPoolExecutor(max_workers=6) as ex:
        return dict(zip(SOURCES, ex.map(one, SOURCES)))


@pytest.fixture(scope="module")
def attention_kernels(compiled):
    """{(Dh, wavefronts, balanced): {resource: number}} of tree_attention_kernel."""
    kernels, at = {}, None
    for line in compiled["attention.hip"][0].splitlines():
        name = re.search(r"Function Name: (\S+)", line)
        if name:
            m = re.search(r"tree_attention_kernelILi(\d+)ELi(\d+)ELb([01])E", name.group(1))
            at = kernels.setdefault((int(m.group(1)), int(m.group(2)), m.group(3) == "1"), {}) if m else None
            continue
        value = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if value and at is not None:
            at[value.group(1)] = int(value.group(2))
    return kernels


def test_attention_kernels_do_not_spill(attention_kernels):
    """All eight: 256 vector registers (two wavefronts per SIMD) and no scratch memory.  The unbalanced ones,
    which equal-length batches and single sequences run, keep their scalars in scalar registers too:
    spilling ten of them into vector lanes cost 1 % of a call."""
    assert len(attention_kernels) == 8
    for key, r in attention_kernels.items():
        assert r["VGPRs"] <= 256 and r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (key, r)
        if not key[2]:
            assert r["SGPRs Spill"] == 0, (key, r)


@pytest.mark.parametrize("source,kernels", [("expand.hip", 6), ("ahead.hip", 2), ("accept.hip", 3)])
def test_scans_do_not_spill(source, kernels, compiled):
    """The kernels that stream rows for capped trees, and the target argmax: no scratch memory."""
    found = re.findall(r"Function Name: (\S*(?:expand_(?:tree_)?kernel|build_ahead_kernel|argmax_\w+_kernel)\S*).*?ScratchSize \[bytes/lane\]: (\d+)",
                       compiled[source][0], re.S)
    assert len(found) == kernels and all(size == "0" for _, size in found), found


def barriers_of_parts(lines):
    """Barriers that every path reaches with lanes of the wavefront taken out: (line number, text).  Follows each kernel's
    branches.  The depth of a point is how many of the instructions that take lanes out are open there; where paths meet, the
    smallest counts, and an instruction that brings lanes back closes one, whichever it was, so nothing is reported wrongly."""
    found, at, functions = [], 0, []
    for n, line in enumerate(lines):                       # functions: [first line, end)
        if re.match(r"_Z\w+:", line):
            at = n
        elif re.match(r"\s*\.size\s+_Z", line):
            functions.append((at, n))
    for first, end in functions:
        blocks, label_of, current = [[]], {}, 0            # straight pieces of code and the labels in front of them
        for n in range(first, end):
            text = lines[n].split(";")[0].strip()
            if re.match(r"\.LBB\w+:", text):
                blocks.append([])
                label_of[text[:-1]] = len(blocks) - 1
            elif text and not text.startswith(".") and not text.endswith(":"):
                blocks[-1].append((n, text.split()))
                if text.startswith(("s_branch", "s_cbranch", "s_endpgm", "s_setpc")):
                    blocks.append([])
        depth_in = [None] * len(blocks)
        depth_in[0], work = 0, [0]
        while work:
            current = work.pop()
            depth, out = depth_in[current], [current + 1]
            for _, op in blocks[current]:
                depth = max(0, depth + change(op))
            if blocks[current]:
                op = blocks[current][-1][1]
                if op[0] in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    out = []
                if op[0].startswith(("s_branch", "s_cbranch")) and op[-1] in label_of:
                    out.append(label_of[op[-1]])
            for b in out:
                if b < len(blocks) and (depth_in[b] is None or depth < depth_in[b]):
                    depth_in[b] = depth
                    work.append(b)
        for block, depth in zip(blocks, depth_in):
            for n, op in block if depth is not None else ():
                if op[0] == "s_barrier" and depth > 0:
                    found.append((n + 1, lines[n]))
                depth = max(0, depth + change(op))
    return found


def change(op):
    """What an instruction does to the number of open ones that take lanes out."""
    writes_exec = len(op) > 1 and op[1].startswith("exec")
    if op[0].startswith("s_and_saveexec") or op[0].startswith("s_and_b64") and writes_exec or op[0].startswith("s_xor_b64") and writes_exec:
        return 1
    if op[0].startswith("s_or_saveexec") or op[0] in ("s_or_b64", "s_mov_b64") and writes_exec:
        return -1
    return 0       # (s_andn2_saveexec: the other side of a branch; s_andn2_b64 exec: lanes that leave a loop, until it ends)


@pytest.mark.parametrize("source", SOURCES)
def test_no_barrier_runs_for_a_part_of_a_wavefront(source, compiled):
    """A loop that starts with `if (threadIdx.x == 0)` right behind another such condition got two entries from
    the compiler, and its barriers ran once for thread 0 and once for the others."""
    assert barriers_of_parts(compiled[source][1]) == []


def test_the_barrier_check_follows_branches():
    text = """
_Zk:
  s_and_saveexec_b64 s[2:3], vcc
  s_cbranch_execz .LBB0_2
.LBB0_1:
  v_mov_b32 v0, v1
  s_barrier
  s_andn2_b64 exec, exec, s[4:5]
  s_cbranch_execnz .LBB0_1
.LBB0_2:
  s_or_b64 exec, exec, s[2:3]
  s_barrier
  s_endpgm
  .size _Zk, 1
"""
    assert [line.split()[0] for _, line in barriers_of_parts(text.split("\n"))] == ["s_barrier"]
    assert barriers_of_parts(text.replace("s_and_saveexec_b64 s[2:3], vcc", "s_nop 0").split("\n")) == []
