"""The rules that choose tiles, kernels and grids, run on the host for the shapes they decide on."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2506_14107_amd", "csrc")
CUS = 256


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("plans") / "plans.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-shared", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", CSRC,
                    os.path.join(HERE, "plans.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("Nout,esz", [(9728, 2), (9984, 2), (16128, 2), (4864, 4)])
def test_tail_rows_are_stored_nowhere(lib, Nout, esz):
    """Packed outputs (QKV, out-projection, MLP hidden rows) of batches whose rows, padded to 256, stay
    below 2^32 bytes as handles require: a tile's rows past the live ones keep off the live ones on any
    number of compute units.  192-row tiles reach up to 128 rows past the padding, where 32-bit products
    wrap to the first rows (on 228 units: 9728 outputs, 220672 rows)."""
    lib.t_stray_rows.restype = ctypes.c_longlong
    last = ((1 << 32) - 1) // (Nout * esz) // 256 * 256
    for cus in (CUS, 304, 255, 240, 228, 192, 128):
        for M in range(last - 255, last + 1):
            assert lib.t_stray_rows(M, Nout, esz, cus) == 0, (M, cus)
