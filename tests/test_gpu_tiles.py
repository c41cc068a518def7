"""The bf16 GEMM's tile plan: every tile shape gives the same bits, at the edges of each shape."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from synth.configs import ModelConfig

from .gpu_util import check_close, dev, encoder, host, require_gpu

pytestmark = pytest.mark.gpu

# outputs 768 / 256 / 1024 (256-wide large tiles) and 1152 / 384 / 1536 (128-wide for the first
# two); 50 tokens.  Patch 8 gives the patch GEMM three k-slices (odd), patch 16 twelve.
WIDE = ModelConfig(112, 16, 1, 256, 4, 1024, "bf16")
NARROW = ModelConfig(112, 16, 1, 384, 6, 1536, "bf16")
ODD_K = ModelConfig(56, 8, 1, 256, 4, 512, "bf16")
TILE_BATCHES = (2, 7, 21, 61, 122, 190, 328, 350, 415, 700)   # frames; test_plans.py checks that they reach
                                                         # every tail shape
# three k-slices and four tile columns: 700 frames are two whole rounds of large tiles, whose blocks go
# from one tile to the next with no slice copied ahead
ODD_K_ROUNDS = ModelConfig(56, 8, 1, 1024, 16, 1024, "bf16")


@pytest.mark.parametrize("m", [WIDE, NARROW, ODD_K], ids=["wide", "narrow", "odd-k"])
def test_tile_plan_bitwise(m):
    """One frame at a time (50 rows, the smallest tiles) against batches whose row counts take
    every tile shape, whole rounds of large tiles with and without a remainder among them."""
    torch = require_gpu()
    n = 700
    blob = synth.make_blob(m, 51)
    base = np.random.default_rng(52).standard_normal((8, 3, m.image_size, m.image_size))
    gain = np.linspace(0.5, 1.5, n).reshape(n, 1, 1, 1)
    fr = (base[np.arange(n) % 8] * gain).astype(np.float32)
    off = float("-inf")
    big = encoder(m, blob, n)
    one = encoder(m, blob, 1)
    want = one.encode(dev(fr), 1, off, want_masks=False, want_tokens=True)
    torch.cuda.synchronize()
    for k in TILE_BATCHES:
        got = big.encode(dev(fr[:k]), 1, off, want_masks=False, want_tokens=True)
        torch.cuda.synchronize()
        for x, y in ((got[0], want[0]), (got[2], want[2])):
            assert np.array_equal(host(x), host(y)[:k]), f"{k} frames"
    ref = oracle.dense_vit(fr[-2:], blob, m.as_dict(), return_tokens=True)
    check_close(host(got[0])[-2:], ref[0], "bf16", "embeddings")
    check_close(host(got[2])[-2:], ref[1], "bf16", "tokens")


def test_odd_slices_over_several_rounds_bitwise():
    """The patch GEMM of 700 frames against batches of 100, which stay below one round."""
    torch = require_gpu()
    m, n = ODD_K_ROUNDS, 700
    blob = synth.make_blob(m, 63)
    fr = np.random.default_rng(64).standard_normal((n, 3, 56, 56)).astype(np.float32)
    off = float("-inf")
    got = encoder(m, blob, n).encode(dev(fr), 1, off, want_masks=False, want_tokens=True)
    few = encoder(m, blob, 100).encode(dev(fr), 1, off, want_masks=False, want_tokens=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(got[0]), host(few[0]))
    assert np.array_equal(host(got[2]), host(few[2]))
    for k in (0, 349, 698):
        ref = oracle.dense_vit(fr[k:k + 2], blob, m.as_dict(), return_tokens=True)
        check_close(host(got[2])[k:k + 2], ref[1], "bf16", "tokens")


# fp32: head dims 16 to 128 (one attention variant each), token counts around its 64-key steps and
# 16-query tiles, widths that are odd multiples of 64; 700 frames take the 64 x 64 GEMM tiles
@pytest.mark.parametrize("S,p,D,H,n", [
    (112, 16, 192, 3, 700), (64, 8, 192, 12, 9), (224, 14, 192, 6, 5), (64, 16, 384, 8, 30),
    (128, 16, 320, 4, 11), (112, 16, 192, 2, 7), (112, 16, 448, 4, 7), (112, 16, 256, 2, 7)])
def test_fp32_tiles_bitwise(S, p, D, H, n):
    """One frame at a time (32 x 32 tiles) against the batch bit for bit, and the oracle."""
    torch = require_gpu()
    m = ModelConfig(S, p, 1, D, H, 4 * D, "f32")
    blob = synth.make_blob(m, 53)
    base = np.random.default_rng(54).standard_normal((8, 3, S, S))
    gain = np.linspace(0.5, 1.5, n).reshape(n, 1, 1, 1)
    fr = (base[np.arange(n) % 8] * gain).astype(np.float32)
    off = float("-inf")
    got = encoder(m, blob, n).encode(dev(fr), 1, off, want_masks=False, want_tokens=True)
    one = encoder(m, blob, 1).encode(dev(fr), 1, off, want_masks=False, want_tokens=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(got[0]), host(one[0]))
    assert np.array_equal(host(got[2]), host(one[2]))
    ref = oracle.dense_vit(fr[-2:], blob, m.as_dict(), return_tokens=True)
    check_close(host(got[0])[-2:], ref[0], "f32", "embeddings")
    check_close(host(got[2])[-2:], ref[1], "f32", "tokens")


@pytest.mark.parametrize("G,n", [(8, 480), (4, 240), (4, 264)],
                         ids=["unit-G8", "unit-G4", "frame-G4"])
def test_attention_routes_bitwise(G, n):
    """Per-unit blocks (240 pairs of a group and a head), per-frame blocks (264 pairs, two rounds of
    units mostly empty) and streamed blocks (internal batches of two groups; streamed calls of five
    frames): the same bits."""
    torch = require_gpu()
    m = ModelConfig(112, 16, 2, 256, 4, 512, "bf16")
    blob = synth.make_blob(m, 55)
    rng = np.random.default_rng(56)
    fr = rng.standard_normal((n, 3, 112, 112)).astype(np.float32)
    for f in range(n):   # patches of each group's first frame, a third of them with noise
        keep = rng.random((1, 7, 1, 7, 1)) < 0.66
        own, ref = (fr[k].reshape(3, 7, 16, 7, 16) for k in (f, f // G * G))
        fr[f] = np.where(keep, ref + 0.05 * own, own).reshape(3, 112, 112)
    fr = dev(fr)
    big = encoder(m, blob, n)
    want = big.encode(fr, G, 0.9, want_tokens=True)
    few = encoder(m, blob, 2 * G).encode(fr, G, 0.9, want_tokens=True)
    parts = [big.stream_encode(fr[f:f + 5], G, 0.9, want_tokens=True) for f in range(0, n, 5)]
    torch.cuda.synchronize()
    reuse = host(want[1]).mean()
    assert 0.2 < reuse < 0.8, reuse
    for k in range(3):
        assert np.array_equal(host(want[k]), host(few[k])), k
        assert np.array_equal(host(want[k]), np.concatenate([host(p[k]) for p in parts])), k


# image, patch, width, heads, group, frames: one to five steps of 64 keys with a ragged last one, every
# head dim, batches on both sides of the rule's lines (test_plans.py checks the routes)
ATTENTION = {
    "dh64-50-unit": (112, 16, 256, 4, 8, 480), "dh64-145-unit": (192, 16, 256, 4, 8, 480),
    "dh64-257-unit": (224, 14, 256, 4, 8, 480), "dh64-145-frame": (192, 16, 256, 4, 4, 264),
    "dh64-257-frame": (224, 14, 256, 4, 4, 264), "dh64-577-stream": (336, 14, 256, 4, 4, 24),
    "dh80-50-stream": (112, 16, 640, 8, 4, 24), "dh80-257-stream": (224, 14, 640, 8, 4, 24),
    "dh96-50-stream": (112, 16, 384, 4, 4, 24), "dh96-257-stream": (224, 14, 384, 4, 8, 32),
    "dh128-50-frame": (112, 16, 256, 2, 4, 140), "dh128-145-frame": (192, 16, 256, 2, 8, 136),
    "dh128-257-frame": (224, 14, 256, 2, 8, 136), "dh128-257-stream": (224, 14, 256, 2, 8, 120)}


@pytest.mark.parametrize("name", ATTENTION)
def test_attention_steps_bitwise(name):
    """Batches on the named route against streamed blocks (internal batches of two groups; stream calls
    of five frames): the same bits, and the last group against the oracle on the same maps."""
    torch = require_gpu()
    S, p, D, H, G, n = ATTENTION[name]
    m = ModelConfig(S, p, 2, D, H, 2 * D, "bf16")
    blob = synth.make_blob(m, 65)
    rng = np.random.default_rng(66)
    fr = rng.standard_normal((n, 3, S, S)).astype(np.float32)
    g = S // p
    for f in range(n):   # patches of each group's first frame, a third of them with noise
        keep = rng.random((1, g, 1, g, 1)) < 0.66
        own, ref = (fr[k].reshape(3, g, p, g, p) for k in (f, f // G * G))
        fr[f] = np.where(keep, ref + 0.05 * own, own).reshape(3, S, S)
    x = dev(fr)
    big = encoder(m, blob, n)
    want = big.encode(x, G, 0.9, want_tokens=True)
    few = encoder(m, blob, 2 * G).encode(x, G, 0.9, want_tokens=True)
    parts = [big.stream_encode(x[f:f + 5], G, 0.9, want_tokens=True) for f in range(0, n, 5)]
    torch.cuda.synchronize()
    masks = host(want[1])
    assert 0.2 < masks.mean() < 0.8, masks.mean()
    for k in range(3):
        assert np.array_equal(host(want[k]), host(few[k])), k
        assert np.array_equal(host(want[k]), np.concatenate([host(q[k]) for q in parts])), k
    ref = oracle.encode(fr[-G:], blob, m.as_dict(), G, masks=masks[-G:])
    check_close(host(want[0])[-G:], ref["emb"], "bf16", "embeddings")
    check_close(host(want[2])[-G:], ref["tokens"], "bf16", "tokens")


@pytest.mark.parametrize("S,p,n,shift", [(224, 14, 40, 0), (112, 16, 80, 0), (112, 16, 80, 1),
                                         (60, 12, 110, 0), (70, 14, 110, 0), (63, 7, 70, 0)])
def test_patch_gather_routes_bitwise(S, p, n, shift):
    """Whole batches (strips through LDS where size, parity and alignment allow; shift: frames that
    start 4 bytes off 16) against one frame at a time (the plain gather): the same bits."""
    torch = require_gpu()
    m = ModelConfig(S, p, 1, 128, 2, 128, "bf16")
    blob = synth.make_blob(m, 57)
    rng = np.random.default_rng(58)
    flat = dev(rng.standard_normal(n * 3 * S * S + 4).astype(np.float32))
    fr = flat[shift:shift + n * 3 * S * S].view(n, 3, S, S)
    off = float("-inf")
    got = encoder(m, blob, n).encode(fr, 1, off, want_masks=False, want_tokens=True)
    one = encoder(m, blob, 1).encode(fr, 1, off, want_masks=False, want_tokens=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(got[0]), host(one[0]))
    assert np.array_equal(host(got[2]), host(one[2]))
    ref = oracle.dense_vit(host(fr)[-1:], blob, m.as_dict(), return_tokens=True)
    check_close(host(got[2])[-1:], ref[1], "bf16", "tokens")


@pytest.mark.parametrize("reuse", [False, True])
def test_weights_touched_ahead_bitwise(reuse):
    """277 MB of weights: batches of up to 8192 tokens touch them ahead of the GEMMs (one frame: more
    wavefronts without a row than with one; 28 frames), 8500 tokens do not.  The same bits."""
    torch = require_gpu()
    m = ModelConfig(64, 16, 11, 1024, 16, 4096, "bf16")
    blob = synth.make_blob(m, 59)
    n = 500
    rng = np.random.default_rng(60)
    base = rng.standard_normal((n // 4, 3, 64, 64))
    fr = dev((np.repeat(base, 4, 0) + 0.3 * rng.standard_normal((n, 3, 64, 64))).astype(np.float32))
    tau = 0.9 if reuse else float("-inf")
    want = encoder(m, blob, n).encode(fr, 4, tau, want_tokens=True)
    few = encoder(m, blob, 28).encode(fr[:196], 4, tau, want_tokens=True)
    one = encoder(m, blob, 4).encode(fr[:8], 4, tau, want_tokens=True)
    torch.cuda.synchronize()
    for k in range(3):
        assert np.array_equal(host(want[k])[:196], host(few[k])), k
        assert np.array_equal(host(want[k])[:8], host(one[k])), k


@pytest.mark.parametrize("dtype,mlp", [("f32", (1 << 19) + 128), ("bf16", (1 << 20) + 128)])
def test_weight_matrices_past_4_gib(dtype, mlp):
    """W_1 [mlp, 2048] and W_2 [2048, mlp] of 2^32 + 2^20 bytes, zero but for the first and the last
    64 hidden units (on both sides of the 4 GiB line of W_1): the bits of the model that has these
    128 units alone, since the others add exact zeros and leave every sum's order as it is."""
    torch = require_gpu()
    small = ModelConfig(32, 16, 1, 2048, 16, 128, dtype)
    w = synth.weights.make_weights(small, 61, perturb_ln=True)
    large = dataclasses.replace(small, mlp=mlp)
    blob = np.zeros(synth.weights.blob_floats(large), np.float32)   # pages never written stay unmapped
    off = 0
    for name, shape in synth.weights.weight_layout(large):
        v = blob[off:off + int(np.prod(shape))].reshape(shape)
        off += v.size
        s = w[name]
        if name in ("l0.W_1", "l0.b_1"):
            v[:64], v[-64:] = s[:64], s[64:]
        elif name == "l0.W_2":
            v[:, :64], v[:, -64:] = s[:, :64], s[:, 64:]
        else:
            v[...] = s
    fr = np.random.default_rng(62).standard_normal((3, 3, 32, 32)).astype(np.float32)
    out = []
    for m, b in ((small, synth.weights.pack_weights(w, small)), (large, blob)):
        enc = encoder(m, b, 3)
        out.append(enc.encode(dev(fr), 1, float("-inf"), want_masks=False, want_tokens=True))
        torch.cuda.synchronize()
        enc.close()
    assert np.array_equal(host(out[0][0]), host(out[1][0]))
    assert np.array_equal(host(out[0][2]), host(out[1][2]))
    ref = oracle.dense_vit(fr, synth.weights.pack_weights(w, small), small.as_dict(), return_tokens=True)
    check_close(host(out[0][2]), ref[1], dtype, "tokens")
