"""Registers and scratch of the kernels whose launch counts on several workgroups per compute unit, as the compiler
states them (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2605_30010_amd.build import CSRC, FLAGS, HIPCC


@pytest.fixture(scope="module")
def dense(tmp_path_factory):
    """(vector registers, scratch bytes per lane) by kernel of dense_kernels.hip."""
    obj = str(tmp_path_factory.mktemp("resources") / "dense.o")
    run = subprocess.run([HIPCC] + FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                                            os.path.join(CSRC, "dense_kernels.hip"), "-o", obj], check=True, capture_output=True, text=True)
    out, name, vgprs = {}, None, 0
    for line in run.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r" VGPRs: (\d+)", line)
        if m:
            vgprs = int(m.group(1))
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m:
            out[name] = (vgprs, int(m.group(1)))
    return out


@pytest.mark.parametrize("head_dim,workgroups", [(16, 3), (32, 3), (64, 3), (72, 3), (80, 3), (96, 2), (128, 1)])
def test_attention_workgroups_per_compute_unit(dense, head_dim, workgroups):
    """A SIMD has 512 registers per lane, given out in eights: 168 for each of three wavefronts, 256 for each of two."""
    kernels = {k: v for k, v in dense.items() if "attention_dma_kernelILi%dE" % head_dim in k}
    assert kernels
    assert all(scratch == 0 for _, scratch in kernels.values()), kernels
    assert min(vgprs for vgprs, _ in kernels.values()) <= {1: 512, 2: 256, 3: 168}[workgroups], kernels
