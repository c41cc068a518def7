"""The rules that choose tiles, kernels and grids, run on the host for the shapes they decide on."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from . import test_gpu_tiles as tiles

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


def gemm(lib, M, Nout):
    head = ctypes.c_int()
    return lib.t_gemm_plan(M, Nout, CUS, ctypes.byref(head)), head.value


def test_batches_of_the_tile_test_reach_every_tail(lib):
    """What test_tile_plan_bitwise compares: every tail shape of the 256-wide plan with rows in large
    tiles and without, and every one of the 128-wide plan's."""
    wide, narrow = set(), set()
    for m in (tiles.WIDE, tiles.NARROW, tiles.ODD_K):
        for k in tiles.TILE_BATCHES:
            for Nout in (3 * m.width, m.width, m.mlp):
                tail, head = gemm(lib, k * m.n_tokens, Nout)
                if Nout % 256 == 0:
                    wide.add((tail, head > 0))
                else:
                    narrow.add(tail)
    assert {t for t, h in wide if h} == set(range(6)), wide
    assert {t for t, h in wide if not h} == {1, 2, 3, 4, 5}, wide
    assert narrow >= {0, 3, 4, 5}, narrow


def test_odd_slice_test_walks_several_rounds(lib):
    m = tiles.ODD_K_ROUNDS
    assert (3 * m.patch ** 2 + 63) // 64 % 2 == 1 and m.width % 256 == 0
    assert gemm(lib, 700 * m.n_patches, m.width)[1] // 256 * (m.width // 256) >= 2 * CUS
    assert gemm(lib, 100 * m.n_patches, m.width)[1] == 0


STREAM, FRAME, UNIT = range(3)


def attn(lib, dh, F, N, H, G=0, star=True):
    out = (ctypes.c_longlong * 3)()
    route = lib.t_attn_plan(dh, F, N, H, G, int(star), CUS, out)
    return route, out[0], out[1], out[2]


def test_attention_plan_is_of_the_launch_alone(lib):
    """The per-frame grid follows from the launch's own sizes: two blocks per compute unit at head dim
    64 and one at 128, also after a model of 577 tokens whose keys fill the LDS of a unit."""
    want = attn(lib, 64, 128, 257, 16)
    assert want[:2] == (FRAME, 2 * CUS) and 2 * want[2] <= 160 << 10
    assert attn(lib, 64, 128, 577, 16)[0] == STREAM
    assert attn(lib, 64, 64, 197, 12, G=4)[:2] == (FRAME, 2 * CUS)
    assert attn(lib, 64, 128, 257, 16) == want
    assert attn(lib, 128, 64, 257, 8, G=8)[:2] == (FRAME, CUS)


def test_attention_routes(lib):
    """Each route of the rule, at the sizes around its lines."""
    assert attn(lib, 64, 256, 257, 16, G=8)[0] == UNIT          # 512 units: two whole rounds
    assert attn(lib, 64, 192, 257, 16, G=8)[0] == STREAM        # 384: a round and a half
    assert attn(lib, 64, 256, 257, 16, G=8, star=False)[0] == STREAM
    assert attn(lib, 64, 16, 257, 16, G=8)[0] == STREAM
    assert attn(lib, 64, 32, 257, 16)[0] == STREAM              # no more items than resident blocks
    assert attn(lib, 64, 33, 257, 16)[0] == FRAME
    assert attn(lib, 64, 64, 320, 16)[0] == FRAME               # two blocks' keys: 160 KB
    assert attn(lib, 64, 64, 321, 16)[0] == STREAM
    assert attn(lib, 64, 64, 257, 16, G=4, star=False)[0] == STREAM
    assert attn(lib, 128, 32, 257, 8, G=8)[0] == STREAM
    assert attn(lib, 128, 33, 257, 8, G=8)[0] == FRAME
    for dh in (80, 96):
        assert attn(lib, dh, 256, 257, 16)[0] == STREAM
    for dh, F, N, H, G in [(64, 256, 257, 16, 8), (64, 512, 289, 16, 8), (64, 512, 17, 2, 4)]:
        route, grid, lds, pcap = attn(lib, dh, F, N, H, G)
        assert route == UNIT and pcap >= N and lds <= 160 << 10 and grid <= CUS


@pytest.mark.parametrize("N", [17, 257, 577])
@pytest.mark.parametrize("H", [1, 3, 12, 16, 18])
def test_streamed_blocks(lib, N, H):
    """Every query tile has one block, at most twice as many blocks are dealt as have work (a few per
    XCD more where units are few), and a group's blocks of one head share an XCD where groups are
    kept: whole batches, the first call of a stream, calls that continue one."""
    lib.t_stream_grid.restype = ctypes.c_longlong
    q = ((N + 31) // 32 + 3) // 4
    for G in (0, 1, 4, 8, 12, 64, 256):
        for F, skip in [(1, 0), (4, 0), (5, 0), (8, 0), (13, 0), (20, 0), (131, 0), (256, 0), (5, 4),
                        (8, 4), (12, 7), (67, 63), (252, 248), (259, 255), (260, 250)]:
            if skip and skip >= max(G, 1):
                continue
            together = ctypes.c_longlong()
            grid = lib.t_stream_grid(F, skip, N, H, G, ctypes.byref(together))
            busy = (F - skip) * H * q
            assert busy <= grid <= 2 * busy + 8 * q, (F, skip, G)
            if H >= 8 and F % max(G, 1) == 0 and skip == 0:
                assert together.value == busy, (F, skip, G)


def test_streamed_blocks_at_scratch_limits(lib):
    """Two-token frames, as many as 32-bit offsets allow, in one group: the launch stays in range."""
    lib.t_stream_grid.restype = ctypes.c_longlong
    together = ctypes.c_longlong()
    for H, F in [(1, 5592000), (10, 559000)]:
        for G, skip in [(F, 0), (F - 1, 0), (F, F - 1), (1, 0)]:
            grid = lib.t_stream_grid(F, skip, 2, H, G, ctypes.byref(together))
            assert 0 < grid * 256 < 1 << 32, (H, F, G, skip)


@pytest.mark.parametrize("name", tiles.ATTENTION)
def test_routes_of_the_attention_test(lib, name):
    S, p, D, H, G, n = tiles.ATTENTION[name]
    N = (S // p) ** 2 + 1
    assert attn(lib, D // H, n, N, H, G)[0] == {"stream": STREAM, "frame": FRAME, "unit": UNIT}[
        name.split("-")[2]]
    assert attn(lib, D // H, 2 * G, N, H, G)[0] == STREAM
    assert attn(lib, D // H, 5 + G, N, H, G, star=False)[0] == STREAM


def test_launchers_keep_no_unsynchronised_state():
    """Local statics of the host code are constants (initialised once, whatever threads come first):
    handles of several threads launch at the same time."""
    mutable = re.compile(r"^[ \t]+static (?!const |constexpr |inline )\w+[ \w:*]* \w+ *(?:=|;)", re.M)
    for name in sorted(os.listdir(CSRC)):
        assert not mutable.findall(open(os.path.join(CSRC, name)).read()), name
