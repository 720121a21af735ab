"""The large-row GEMM (bf16 calls with hundreds of rows known on the host:
full encodes, pure top-k steps) against the oracle, with ragged row tiles
(rows not a multiple of 64 or 128) and a ragged column tile (the MLP width
padded to 544 = 4 x 128 + 32 columns), and the same calls on the
weight-streaming GEMM (tuning tiled = 1) for comparison; then every tile of the
launch rule, with one and with several tiles to a workgroup, against the
weight-streaming GEMM."""
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


@pytest.mark.parametrize("tiled,fc2_mode", [(0, 0), (0, 1), (0, 2), (1, 0)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_large_row_gemm(name, tiled, fc2_mode):
    """fc2_mode 1: the down projection split over K; 2: unsplit, the residual
    and the cache write in its epilogue; 0: by its number of 64 x 128 tiles,
    split for the 600 rows (20 tiles), unsplit for the 2048 (192)."""
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



# One case per tile of the launch rule, at its edges: one row short of and one
# past a row tile, a ragged last column tile, one and several tiles to a
# workgroup, an odd number of 32-deep chunks (dim 224: 7, fewer than the ring's
# slots) and an even one.  A workgroup takes several tiles when they outnumber
# the places on the chip (256; 512 for 128 x 128) and each has more slots than
# the staging runs ahead.
TILES = {
    # name: (dim, heads, mlp, rows of a stream, streams, MLP reading)
    # the tile that the MLP up projection takes:
    "64x128": (224, 7, 2912, 513, 1, "reuse"),             # 9 x 23 = 207 (64 x 64: 414)
    "64x64": (128, 2, 1056, 641, 1, "reuse"),              # 11 x 17 = 187
    "128x128": (224, 7, 2912, 1023, 1, "reuse"),           # 64 x 128: 16 x 23 = 368; 256 x 128: 92
    "256x128": (128, 2, 4096, 1025, 1, "reuse"),           # 5 x 32 = 160
    "256x256": (128, 2, 8192, 1985, 1, "reuse"),           # 8 x 32 = 256
    # as many chunks as the staging runs ahead of the products (3 and 5): tiles
    # beyond the chip's places need a workgroup of their own
    "128x128_short_k": (96, 3, 2688, 4096, 1, "reuse"),    # 32 x 21 = 672 (256 x 128: 336, a last round of a third)
    "256x128_short_k": (160, 5, 3584, 4096, 1, "reuse"),   # 16 x 28 = 448
    # several tiles to a workgroup
    "256x256_several": (128, 2, 8192, 4096, 1, "reuse"),   # 16 x 32 = 512, 4 slots (2 ahead)
    "256x128_several": (224, 7, 3584, 4095, 1, "reuse"),   # 16 x 28 = 448, 7 slots (5 ahead)
    "128x128_several": (160, 5, 2688, 4095, 1, "reuse"),   # 32 x 21 = 672, 5 slots (3 ahead)
    # the other products on several tiles to a workgroup: QKV on 256 x 256 (512
    # tiles), and on 256 x 128 (896 and 1344) with the output and down projections
    # on 128 x 128 (224 x 3 = 672) and 256 x 128 (112 x 4 = 448), their residual
    # in the epilogue, as partial sums (the last layer) and, with every row in the
    # MLP, as the attention branch
    "qkv_256x256": (128, 2, 512, 4096, 16, "reuse"),
    "down_128x128": (320, 5, 640, 4095, 7, "reuse"),
    "down_256x128": (512, 8, 512, 4095, 7, "reuse"),
    "branch_128x128": (320, 5, 640, 4095, 7, "all"),
    "branch_256x128": (512, 8, 512, 4095, 7, "all"),
}


def _random_encoder(m, streams, mlp, seed):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.empty(synth.canonical_weight_count(m), device="cuda").normal_(0.0, 0.02, generator=gen)
    o = 0
    for pname, shape in synth.param_shapes(m):
        n = int(np.prod(shape))
        if pname.endswith("_g"):
            w[o:o + n] += 1.0
        o += n
    patches = torch.rand((streams, m.n_tokens, m.patch_dim), device="cuda", generator=gen)
    return (lambda: incvit.Encoder(m, w, max_streams=streams, mlp=mlp)), patches


def _worst(a, b):
    """Largest difference over the largest value, stream by stream of bf16 states."""
    return max(float((x.float() - y.float()).abs().max() / y.float().abs().max()) for x, y in zip(a, b))


@pytest.mark.parametrize("name", sorted(TILES))
def test_tiles_against_the_weight_streaming_gemm(name):
    """Full encodes on the large-row GEMM against the same encodes on the
    weight-streaming one (tuning tiled = 1): both round every operation once, so
    they differ by the fp32 order of a product's sum, which moves a bf16 result
    by at most one step (2^-8 relative) at a tie; the residual sum, the MLP and
    the final LayerNorm pass such steps on, hence four of them on the largest
    value per layer (the bar of the per-layer oracle checks).  One layer, two
    where a product's epilogue differs in the last one."""
    import torch

    dim, heads, mlp, rows, streams, reading = TILES[name]
    depth = 1 if streams == 1 else 2
    m = synth.ModelShape(4, 4 * rows, 3, 4, dim, depth, heads, mlp, "bf16")
    say(f"[tile {name}] rows={rows} x {streams} D={dim} F={mlp} depth={depth}")
    make, patches = _random_encoder(m, streams, reading, 4200 + rows)
    ys, states = [], []
    for tiled in (0, 1):
        enc = make()
        incvit._check(incvit.incvit_set_tuning(enc.h, tiled=tiled), enc.h)
        buf, caches = enc.new_caches(streams)
        y = torch.zeros((streams, rows, dim), dtype=torch.bfloat16, device="cuda")
        idx = torch.zeros((streams, rows), dtype=torch.int32, device="cuda")
        count = torch.zeros((streams,), dtype=torch.int32, device="cuda")
        enc.encode_frame(patches, caches, 0, 1, 0.98, [rows] * streams, out=(idx, count, y))
        torch.cuda.synchronize()
        assert count.tolist() == [rows] * streams and torch.isfinite(y).all()
        ys.append(y)
        # keys, values and layer inputs (after the fp32 references)
        states.append([enc.export_raw(c)[rows * dim * 4:].view(torch.bfloat16) for c in caches])
        torch.cuda.synchronize()
        enc.close()
    del buf
    err, err_state = _worst(*ys), _worst(*states)
    say(f"  largest difference {err:.2e} of the largest value (state {err_state:.2e})")
    assert err <= depth * 4 * 2.0 ** -8
    assert err_state <= depth * 4 * 2.0 ** -8


@pytest.mark.parametrize("row_groups", [3, 8])
def test_rows_beyond_the_expected(row_groups):
    """A threshold step whose caller expects 96 or 256 rows (the MLP up
    projection then takes 64 x 64 or 64 x 128 tiles: 136 of them, of eight slots,
    two or four more than the staging runs ahead) gets none, a few, as many and
    all 1024: the launch covers every row, and 1088 and 544 tiles over 256
    workgroups give each several.  Against the weight-streaming GEMM, one layer,
    bar as above."""
    import torch

    m = synth.ModelShape(4 * 32, 4 * 32, 3, 4, 512, 1, 8, 4304, "bf16")
    N = m.n_tokens
    make, first = _random_encoder(m, 1, "reuse", 4300 + row_groups)
    got = []
    for tiled in (0, 1):
        enc = make()
        incvit._check(incvit.incvit_set_tuning(enc.h, row_groups=row_groups, tiled=tiled), enc.h)
        buf, caches = enc.new_caches(1)
        frame = first.clone()
        enc.full_encode(frame, caches)
        out = []
        for rows in (0, 5, 32 * row_groups, N, 1):
            frame = frame.clone()
            frame[:, :rows] = -frame[:, :rows]  # far from its reference
            y = torch.zeros((1, N, m.dim), dtype=torch.bfloat16, device="cuda")
            idx = torch.zeros((1, N), dtype=torch.int32, device="cuda")
            count = torch.zeros((1,), dtype=torch.int32, device="cuda")
            enc.step(frame, caches, 0.5, [N], out=(idx, count, y))
            torch.cuda.synchronize()
            say(f"[rows beyond the expected, row_groups={row_groups} tiled={tiled}] {int(count[0])} of {rows}")
            assert int(count[0]) == rows
            out.append(y[:, :rows].clone())
            out.append(enc.export_raw(caches[0])[N * m.dim * 4:].view(torch.bfloat16).clone())
        got.append([x for x in out if x.numel()])
        torch.cuda.synchronize()
        enc.close()
    del buf
    err = _worst(*got)
    say(f"  largest difference {err:.2e} of the largest value")
    assert err <= 4 * 2.0 ** -8
