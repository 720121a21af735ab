"""The fixed-order product on the matrix cores (patch embedding) equals the
oracle's scalar fma chain bit for bit: every tile per wave (1 x 1, 1 x 2,
2 x 4 by the number of output tiles), rows that are not a multiple of 16 bytes
(odd P), a K tail inside and before a 16-deep half chunk, K shorter than a
chunk, ragged token counts, both weight types, and one non-finite token."""
import numpy as np
import pytest
import torch

from oracle import pinned
from paper_2607_12287_amd import incvit, synth
from tests.gpu_util import say, workspace_arrays

pytestmark = pytest.mark.gpu

CASES = {
    # name: (channels, patch, grid_h, grid_w, dim, streams): P, tiles
    "p3_1x1": (3, 1, 5, 5, 32, 1),            # P = 3: one step of a chunk
    "p75_1x1": (3, 5, 7, 9, 96, 2),           # P = 75: odd rows, tail in the first half chunk
    "p49_1x1": (1, 7, 4, 5, 64, 3),           # P = 49: one value past the first half of the tail chunk
    "p588_1x2": (3, 14, 17, 19, 1152, 2),     # 21 token tiles per stream, 3024 tiles; D not a multiple of 128
    "p108_1x2_d96": (3, 6, 33, 31, 672, 1),   # 64 x 42 = 2688 tiles; D % 64 != 0
    "p48_2x4": (3, 4, 33, 31, 1024, 4),       # 64 x 64 x 4 = 16384 tiles, N = 1023
    "p192_2x4": (3, 8, 32, 33, 512, 8),       # 66 x 32 x 8 = 16896 tiles, whole chunks only
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_embedding_bit_exact(name, dtype):
    ch, patch, gh, gw, dim, B = CASES[name]
    m = synth.ModelShape(gh * patch, gw * patch, ch, patch, dim, 1, dim // 32, 32, dtype)
    w = synth.make_weights(m, 77 + dim)
    rng = np.random.default_rng(dim + patch)
    patches = rng.standard_normal((B, m.n_tokens, m.patch_dim)).astype(np.float32)
    patches[0, m.n_tokens // 2, -1] = np.inf  # its own row only
    say(f"[fixed product {name} {dtype}] N={m.n_tokens} P={m.patch_dim} D={dim} B={B}")
    enc = incvit.Encoder(m, synth.flatten_weights(m, w), max_streams=B)
    buf, caches = enc.new_caches(B)
    enc.full_encode(torch.from_numpy(patches).cuda(), caches)
    t0 = workspace_arrays(enc, B)["t0"]
    for v in sorted({0, B - 1}):
        ref = pinned.embed_f32(patches[v], w["w_pe"], w["b_pe"], w["pos"])
        assert np.array_equal(t0[v], ref, equal_nan=True), (name, v)
        assert np.isfinite(ref).sum() >= ref.size - dim
