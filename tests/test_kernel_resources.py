"""Registers and LDS of the built kernels that the launch rules count on."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_14107_amd import dejavu as dj

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled name -> metadata of every kernel in the library."""
    dj.load()
    d = tmp_path_factory.mktemp("lib")
    so = shutil.copy(dj.LIB_PATH, d)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", so], check=True,
                   capture_output=True, cwd=d)
    out = {}
    for obj in glob.glob(os.path.join(str(d), "*gfx950")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], check=True,
                               capture_output=True, text=True).stdout
        for k in re.split(r"\n  - (?=\.agpr)", notes)[1:]:
            name = re.search(r"\n    \.name: +(\S+)", k).group(1)
            out[name] = {f: int(re.search(rf"\.{f}: +(\d+)", k).group(1)) for f in
                         ("group_segment_fixed_size", "vgpr_count", "agpr_count")}
    return out


def of(kernels, fragment):
    found = [v for k, v in kernels.items() if fragment in k]
    assert found, fragment
    return found


def test_layernorm_rows_take_no_lds(kernels):
    """LN2's blocks fit beside another handle's GEMM block, which holds all LDS of its compute unit; only
    a launch that touches weights asks for some."""
    assert all(v["group_segment_fixed_size"] == 0 for v in of(kernels, "ln_rows_k"))


def test_per_frame_attention_blocks_per_compute_unit(kernels):
    """Blocks of eight wavefronts, 512 registers per SIMD lane: two blocks (four wavefronts a SIMD) at head
    dim 64, one (two a SIMD) at 128, and no such kernel at the other head dims."""
    assert sum("attn_mfma_k" in k for k in kernels) == 2
    assert of(kernels, "attn_mfma_kILi64E")[0]["vgpr_count"] <= 128
    assert 128 < of(kernels, "attn_mfma_kILi128E")[0]["vgpr_count"] <= 256
    assert all(v["group_segment_fixed_size"] == 0 for v in of(kernels, "attn_mfma_k"))
