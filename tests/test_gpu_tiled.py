"""The large-row GEMM (bf16 calls with hundreds of rows known on the host:
full encodes, pure top-k steps) against the oracle, with ragged row tiles
(rows not a multiple of 64 or 128), a ragged column tile (the MLP width padded
to 544 = 4 x 128 + 32 columns), both tile heights (64 and 128 rows), and the
same calls on the weight-streaming GEMM (tuning tiled = 1) for comparison."""
import numpy as np
import pytest

from paper_2607_12287_amd import incvit, synth
from tests.gpu_util import Pair, say

pytestmark = pytest.mark.gpu

CASES = {
    # name: (dim, depth, heads, mlp, img, patch, B, top-k caps of the two steps)
    "rows600_cols544": (256, 2, 4, 520, 40, 4, 6, ([100, 100, 60, 100, 100, 100], [100, 37, 100, 100, 100, 100])),
    "rows2048_tile128": (768, 1, 12, 1024, 128, 4, 2, ([300, 200], [1024, 1])),
}


@pytest.mark.parametrize("tiled,fc2_mode", [(0, 0), (0, 2), (1, 0)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_large_row_gemm(name, tiled, fc2_mode):
    """fc2_mode 0: the down projection split over K (its tiles are fewer than
    the CUs here); 2: unsplit, the residual and the cache write in its
    epilogue."""
    dim, depth, heads, mlp, img, patch, B, caps = CASES[name]
    m = synth.small_model(dim=dim, depth=depth, heads=heads, mlp=mlp, img=img, patch=patch, dtype="bf16")
    w = synth.make_weights(m, 2500 + dim)
    say(f"[large-row GEMM {name} tiled={tiled} fc2_mode={fc2_mode}] N={m.n_tokens} B={B} rows={B * m.n_tokens} "
        f"D={dim} F={mlp}")
    its = [synth.RefillRectStream(m, 2510 + v, v, 3 * patch + 1, 5 * patch).frames(3) for v in range(B)]
    frames = [np.stack([synth.patchify(next(it), patch) for it in its]) for _ in range(3)]
    p = Pair(m, w, B)
    incvit._check(incvit.incvit_set_tuning(p.enc.h, tiled=tiled, fc2_mode=fc2_mode), p.enc.h)
    p.full_encode(frames[0])
    tf = p.check_layers(None, "full")
    fr = p.check_caches("full")
    say(f"  full encode: per-layer worst {tf:.2e}, free-running worst {fr:.2e}")
    for t in (1, 2):
        idx, count, refreshed, res = p.step(frames[t], np.inf, caps[t - 1])
        p.check_step(idx, count, refreshed, res, f"step {t}")
        tf = p.check_layers(lambda v: idx[v, :count[v]], f"step {t}")
        fr = p.check_caches(f"step {t}")
        say(f"  step {t}: rows {int(count.sum())} per-layer worst {tf:.2e}, free-running worst {fr:.2e}")



# one case per tile of the launch rule, at its edges: one row short of and one
# past a row tile, a ragged last column tile, one and several tiles to a
# workgroup, an odd number of 32-deep chunks (dim 224: 7, fewer than the ring's
# slots) and an even one
TILES = {
    # name: (dim, heads, mlp, rows): the tile that the MLP up projection takes
    "64x128": (224, 7, 2912, 513),             # 9 x 23 = 207 (64 x 64: 414)
    "64x64": (128, 2, 1056, 641),              # 11 x 17 = 187
    "128x128": (224, 7, 2912, 1023),           # 64 x 128: 16 x 23 = 368; 256 x 128: 92
    "256x128": (128, 2, 4096, 1025),           # 5 x 32 = 160
    "256x256": (128, 2, 8192, 1985),           # 8 x 32 = 256
    # as many chunks as the staging runs ahead of the products (3 and 5): tiles
    # beyond the chip's places need a workgroup of their own
    "128x128_short_k": (96, 3, 2688, 4096),    # 32 x 21 = 672 (256 x 128: 336, a last round of a third)
    "256x128_short_k": (160, 5, 3584, 4096),   # 16 x 28 = 448
}


@pytest.mark.parametrize("name", sorted(TILES))
def test_tiles_against_the_weight_streaming_gemm(name):
    """Full encodes on the large-row GEMM against the same encodes on the
    weight-streaming one (tuning tiled = 1), one layer: both round every
    operation once, so they differ by the fp32 order of a product's sum, which
    moves a bf16 result by at most one step (2^-8 relative) at a tie; the
    residual sum, the MLP and the final LayerNorm pass such steps on, hence four
    of them on the largest value (the bar of the per-layer oracle checks)."""
    import torch

    dim, heads, mlp, rows = TILES[name]
    m = synth.ModelShape(4, 4 * rows, 3, 4, dim, 1, heads, mlp, "bf16")
    gen = torch.Generator(device="cuda").manual_seed(4200 + rows)
    w = torch.empty(synth.canonical_weight_count(m), device="cuda").normal_(0.0, 0.02, generator=gen)
    o = 0
    for pname, shape in synth.param_shapes(m):
        n = int(np.prod(shape))
        if pname.endswith("_g"):
            w[o:o + n] += 1.0
        o += n
    patches = torch.rand((1, rows, 48), device="cuda", generator=gen)
    got = []
    for tiled in (0, 1):
        enc = incvit.Encoder(m, w, max_streams=1)
        incvit._check(incvit.incvit_set_tuning(enc.h, tiled=tiled), enc.h)
        buf, caches = enc.new_caches(1)
        y = torch.zeros((1, rows, dim), dtype=torch.bfloat16, device="cuda")
        idx = torch.zeros((1, rows), dtype=torch.int32, device="cuda")
        count = torch.zeros((1,), dtype=torch.int32, device="cuda")
        enc.encode_frame(patches, caches, 0, 1, 0.98, [rows], out=(idx, count, y))
        torch.cuda.synchronize()
        got.append((y.float(), enc.export_raw(caches[0])))
    del buf
    a, b = got[0][0], got[1][0]
    err = float((a - b).abs().max() / b.abs().max())
    say(f"[tile {name}] rows={rows} D={dim} F={mlp}: largest difference {err:.2e} of the largest value")
    assert int(count[0]) == rows and torch.isfinite(a).all()
    assert err <= 4 * 2.0 ** -8
    # keys, values and layer inputs (after the fp32 references)
    sa, sb = (s[rows * dim * 4:].view(torch.bfloat16).float() for _, s in got)
    assert float((sa - sb).abs().max() / sb.abs().max()) <= 4 * 2.0 ** -8
