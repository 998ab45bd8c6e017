"""Registers and scratch of kernels, as the compiler reports them for the
library's own flags: no GPU is needed."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2609_18077_amd import build

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _scratch(source):
    """Kernel name -> bytes of scratch a lane."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not available")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, *build.SOURCE_FLAGS.get(source, []), "--offload-device-only",
                          "-Rpass-analysis=kernel-resource-usage", "-I", os.path.join(build.ROOT, "include"), "-c",
                          os.path.join(build.HERE, "csrc", source), "-o", os.devnull],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    names = re.findall(r"Function Name: (\S+)", res.stderr)
    sizes = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", res.stderr)]
    assert names and len(names) == len(sizes)
    return dict(zip(names, sizes))


@pytest.mark.parametrize("source,kernels", [("attn_fwd_split.hip", 4), ("rope3d.hip", 2), ("qknorm.hip", 3)])
def test_latency_bound_kernels_use_no_scratch(source, kernels):
    """A short launch of these is one workgroup's chain of memory latencies, to
    which every spilled register (or array held in memory) adds."""
    got = _scratch(source)
    assert len(got) == kernels
    assert all(x == 0 for x in got.values()), got


def _ir(source):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc is not available")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run([HIPCC, *flags, *build.SOURCE_FLAGS.get(source, []), "--offload-device-only", "-S", "-emit-llvm",
                          "-I", os.path.join(build.ROOT, "include"), os.path.join(build.HERE, "csrc", source), "-o", "-"],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    return {m.group(1): m.group(2) for m in re.finditer(r"^define [^\n]*@(\w+)\([^\n]*\{\n(.*?)^\}", res.stdout, re.S | re.M)}


@pytest.mark.parametrize("source,kernel,least", [
    ("rope3d.hip", "rope3d_kernelILb1E", 2),
    ("qknorm.hip", "qk_norm_kernelILb1ELb1E", 2),
    ("attn_bwd.hip", "bwd_dkdv_kernel", 2),
    ("attn_bwd.hip", "bwd_dq4_kernel", 1),
    ("attn_fwd_split.hip", "attn_fwd_split_kernelILb1ELb0ELb1E", 3),
])
def test_lanes_hand_over_through_lds_with_a_fence(source, kernel, least):
    """Where the lanes of a wave write LDS that its other lanes read (no barrier:
    one wave's accesses are in order), the order is stated to the compiler: a
    wavefront fence and a wave barrier."""
    bodies = [b for n, b in _ir(source).items() if kernel in n]
    assert len(bodies) == 1, kernel
    assert bodies[0].count('fence syncscope("wavefront") acq_rel') >= least
    assert len(re.findall(r"call void @llvm.amdgcn.wave.barrier", bodies[0])) >= least
