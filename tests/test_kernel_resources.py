"""Registers of the attention kernels, as the compiler reports them for gfx950 (no GPU needed)."""
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
