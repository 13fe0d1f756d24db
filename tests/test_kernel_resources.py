"""Registers of the kernels, as the compiler reports them for gfx950 (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2601_07353_amd import build as B


@pytest.fixture(scope="module")
def attention_kernels(tmp_path_factory):
    """{(Dh, wavefronts, balanced): {resource: number}} of tree_attention_kernel."""
    out = subprocess.run([B._hipcc(), *B.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(B.CSRC, "attention.hip"), "-o", str(tmp_path_factory.mktemp("o") / "attention.o")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout
    kernels, at = {}, None
    for line in out.splitlines():
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
def test_scans_do_not_spill(source, kernels, tmp_path_factory):
    """The kernels that stream rows for capped trees, and the target argmax: no scratch memory."""
    out = subprocess.run([B._hipcc(), *B.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(B.CSRC, source), "-o", str(tmp_path_factory.mktemp("o") / "out.o")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True).stdout
    found = re.findall(r"Function Name: (\S*(?:expand_(?:tree_)?kernel|build_ahead_kernel|argmax_\w+_kernel)\S*).*?ScratchSize \[bytes/lane\]: (\d+)",
                       out, re.S)
    assert len(found) == kernels and all(size == "0" for _, size in found), found


def _assembly(source, tmp_path_factory):
    path = str(tmp_path_factory.mktemp("s") / "out.s")
    subprocess.run([B._hipcc(), *B.FLAGS, "--cuda-device-only", "-S", os.path.join(B.CSRC, source), "-o", path],
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT, check=True)
    return open(path).read().splitlines()


@pytest.mark.parametrize("source", ["ahead.hip"])
def test_no_barrier_runs_for_a_part_of_a_wavefront(source, tmp_path_factory):
    """A loop that starts with `if (threadIdx.x == 0)` right behind another such condition got two entries from
    the compiler, and its barriers ran once for thread 0 and once for the others: a barrier right behind the
    instruction that takes lanes out."""
    narrowed = False
    for line in _assembly(source, tmp_path_factory):
        op = line.split(";")[0].split()
        if not op or op[0].startswith("."):
            continue
        if op[0].endswith(":") or op[0] in ("s_branch", "s_endpgm"):
            narrowed = False
        elif "saveexec" in op[0]:
            narrowed = True
        elif len(op) > 1 and op[1].startswith("exec") and op[0] in ("s_or_b64", "s_mov_b64"):
            narrowed = False
        assert not (narrowed and op[0] == "s_barrier"), line
