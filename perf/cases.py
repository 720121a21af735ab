"""The work a program gives this library, as cases that can be timed and compared.

A program that watches cameras makes an `Encoder` from its model's weights, encodes the first frame of every stream in
full and then calls a step per frame (eagerly, or as a captured graph into whose fixed input it copies the frame).
Every case here is one such call on one model, with synthetic frames of the kind the repository's own workloads use:
smooth noise, a textured square that moves four pixels a frame, fresh sensor noise.  A state holds a ring of frames, so
that one pass follows another as frames follow each other, on a cache that the pass before it left behind: what a pass
leaves there (keys, values and references) is what the next pass's outputs are made from, and the resumed stream returns
all of it.

`depth` is the number of encoder layers.  Two bf16 cases run a whole 27-layer stack; the others run fewer layers of the
same width, whose roundings travel less far, so that their tolerance says something about each layer.
"""
import math

import torch

from paper_2607_12287_amd import incvit, synth

RING = 4        # frames of a state's stream after its first one
SPEED = 4       # pixels that the square moves per frame
TAU = 0.98      # similarity below which a token is refreshed

# The shapes that this repository names (224x224 frames unless said otherwise).
TINY = dict(img_h=224, img_w=224, patch=16, dim=192, heads=3, mlp=768, dtype="f32")
SO400M = dict(img_h=224, img_w=224, patch=14, dim=1152, heads=16, mlp=4304, dtype="bf16")
SO400M_448 = dict(SO400M, img_h=448, img_w=448)
VIT_L = dict(img_h=224, img_w=224, patch=14, dim=1024, heads=16, mlp=4096, dtype="bf16")


def _case(name, model, depth, streams, call, *, graph=False, cap=0, side=0, row_groups=0, score="embed", mlp_rows="reuse"):
    c = dict(model, depth=depth, streams=streams, call=call, graph=graph, cap=cap, side=side, row_groups=row_groups, score=score,
             mlp_rows=mlp_rows)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a small fp32 model on one camera, a captured step of a dozen rows; launches set its time
        _case("tiny_step", TINY, 12, 1, "step", graph=True, side=48),
        # the benchmark's headline: one camera, about a tenth of the tokens move, whole stack, captured step
        _case("so400m_step", SO400M, 27, 1, "step", graph=True, side=56),
        # a robot with three cameras, eager calls, rows not known on the host
        _case("so400m_x3_step", SO400M, 9, 3, "step", side=77, row_groups=4),
        # a server of eight cameras, captured step
        _case("vitl_x8_step", VIT_L, 12, 8, "step", graph=True, side=49, row_groups=6),
        # a large frame with a fixed share of rows: a tenth (captured) and a half (eager)
        _case("448_top_k_10", SO400M_448, 9, 1, "top_k", graph=True, cap=102),
        _case("448_top_k_50", SO400M_448, 9, 1, "top_k", cap=512),
        # full frames: what every stream starts with and what the refresh schedule repeats; one camera, a large frame,
        # and many cameras at once (the largest call)
        _case("so400m_encode", SO400M, 27, 1, "encode"),
        _case("448_encode", SO400M_448, 9, 1, "encode"),
        _case("vitl_x32_encode", VIT_L, 6, 32, "encode"),
        # the key score (the paper's eq. 3 as printed) on odd frames: 13 x 21 tokens, two cameras
        _case("key_step_odd", dict(img_h=182, img_w=294, patch=14, dim=768, heads=12, mlp=3072, dtype="bf16"), 8, 2, "step",
              side=63, score="key"),
        # the reading in which every token goes through the MLP, two cameras
        _case("mlp_all_step", SO400M, 6, 2, "step", graph=True, side=56, mlp_rows="all"),
        # a stream that moves between processes: its saved state is loaded, one frame is encoded, the state is saved (fp32)
        _case("resume_step_f32", dict(img_h=224, img_w=224, patch=16, dim=384, heads=6, mlp=1536, dtype="f32"), 8, 1, "resume",
              side=48),
    ]


def draw(rng):
    """A case of the same ranges: calls, types, widths, frame sizes and stream counts, odd ones among them."""
    most = _cost(listed()[8])

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        patch = rng.choice([14, 16])
        head = rng.choice([32, 64, 64, 72, 80, 96])
        heads = rng.choice([3, 4, 6, 8, 12, 16])
        dim = head * heads
        if dim % 32 or not 192 <= dim <= 1280:
            continue
        model = dict(img_h=patch * spread(9, 33), img_w=patch * spread(9, 33), patch=patch, dim=dim, heads=heads,
                     mlp=int(dim * rng.uniform(2.5, 4.5)), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
        n = (model["img_h"] // patch) * (model["img_w"] // patch)
        streams = spread(1, 24)
        call = rng.choice(["step", "step", "top_k", "encode", "encode", "resume"])
        score = "key" if call == "step" and rng.random() < 0.25 else "embed"
        mlp_rows = "all" if call == "step" and score == "embed" and rng.random() < 0.2 else "reuse"
        small = min(model["img_h"], model["img_w"])
        case = _case("", model, spread(2, 12), 1 if call == "resume" else streams, call,
                     graph=call in ("step", "top_k") and rng.random() < 0.5,
                     cap=max(1, int(n * rng.uniform(0.03, 0.7))) if call == "top_k" else 0,
                     side=0 if call in ("top_k", "encode") else max(patch, int(small * rng.uniform(0.15, 0.45))),
                     score=score, mlp_rows=mlp_rows)
        if _cost(case) <= most:
            return case


# ---------------------------------------------------------------- inputs --


def _model(case):
    return synth.ModelShape(case["img_h"], case["img_w"], 3, case["patch"], case["dim"], case["depth"], case["heads"],
                            case["mlp"], case["dtype"])


def _seed(seed, what):
    return (int(seed) * 1000003 + what * 7919 + 17) % (1 << 62)


def _weights(m, seed):
    """Canonical fp32 vector on the GPU: 0.02 N(0, 1), LayerNorm gains around one (synth.make_weights' distributions)."""
    gen = torch.Generator(device="cuda").manual_seed(_seed(seed, 1))
    w = torch.empty(synth.canonical_weight_count(m), device="cuda").normal_(0.0, 0.02, generator=gen)
    o = 0
    for name, shape in synth.param_shapes(m):
        n = math.prod(shape)
        if name.endswith("_g"):
            w[o:o + n] += 1.0
        o += n
    return w


def _smooth(gen, b, h, w, cell):
    """[b][3][h][w] of bilinear noise: a U[0,1) lattice value every `cell` pixels."""
    gh, gw = -(-h // cell) + 1, -(-w // cell) + 1
    lat = torch.rand((b, 3, gh, gw), device="cuda", generator=gen)
    full = torch.nn.functional.interpolate(lat, size=((gh - 1) * cell + 1, (gw - 1) * cell + 1), mode="bilinear", align_corners=True)
    return full[:, :, :h, :w]


def _side(case, v):
    """Side of the moving square of stream v in pixels."""
    m = min(case["img_h"], case["img_w"])
    if case["call"] == "top_k":  # a quarter more tokens change than are refreshed
        return min(m, case["patch"] * math.ceil(math.sqrt(1.25 * case["cap"])))
    if case["call"] == "encode":
        return max(1, m // 4)
    return max(1, min(m, case["side"] * (2 + v % 3) // 3) if case["streams"] > 1 else min(m, case["side"]))


def _frames(case, seed):
    """[RING + 1][B][N][P]: the first frame and the ring; a square moves to and fro over a still background, with fresh
    sensor noise in every frame (top-k calls: with a fresh texture in every frame)."""
    gen = torch.Generator(device="cuda").manual_seed(_seed(seed, 2))
    host = torch.Generator().manual_seed(_seed(seed, 3))
    B, h, w, p = case["streams"], case["img_h"], case["img_w"], case["patch"]
    clean = _smooth(gen, B, h, w, 8)
    out = []
    side = [_side(case, v) for v in range(B)]
    reach = SPEED * (RING // 2)
    at = [(int(torch.randint(0, h - s + 1, (1,), generator=host)), int(torch.randint(0, max(1, w - s - reach + 1), (1,), generator=host)))
          for s in side]
    big = max(side)
    tex = _smooth(gen, B, big, big, 4)
    for t in range(RING + 1):
        f = clean.clone()
        if case["call"] == "top_k" and t:
            tex = _smooth(gen, B, big, big, 4)
        dx = SPEED * (t if t <= RING // 2 else RING - t)
        for v, (y, x) in enumerate(at):
            s = side[v]
            x1 = min(x + dx, w - s)
            f[v, :, y:y + s, x1:x1 + s] = tex[v, :, :s, :s]
        f = (f + 0.005 * torch.randn(f.shape, device="cuda", generator=gen)).clamp_(0.0, 1.0)
        out.append(f.reshape(B, 3, h // p, p, w // p, p).permute(0, 2, 4, 1, 3, 5).reshape(B, (h // p) * (w // p), 3 * p * p))
    return torch.stack(out).contiguous()


def _selection(case, n):
    return (math.inf, [case["cap"]] * case["streams"]) if case["call"] == "top_k" else (TAU, [n] * case["streams"])


class State:
    """An encoder with its caches, its frames and its output buffers, as a program keeps them."""

    graph = None

    def __del__(self):
        if self.graph is not None:
            incvit.Encoder.drop_graph(self.graph)


def prepare(case, seed):
    m = _model(case)
    s = State()
    s.case, s.t = case, 0
    B = case["streams"]
    s.enc = incvit.Encoder(m, _weights(m, seed), max_streams=B, score=case["score"], mlp=case["mlp_rows"])
    if case["row_groups"]:  # what a caller that expects about 32 * row_groups rows sets
        incvit._check(incvit.incvit_set_tuning(s.enc.h, row_groups=case["row_groups"]), s.enc.h)
    frames = _frames(case, seed)
    s.first, s.ring = frames[0].contiguous(), [f.contiguous() for f in frames[1:]]
    s.buf, s.caches = s.enc.new_caches(B)
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    s.out = (torch.zeros((B, m.n_tokens), dtype=torch.int32, device="cuda"), torch.zeros((B,), dtype=torch.int32, device="cuda"),
             torch.zeros((B, m.n_tokens, m.dim), dtype=dt, device="cuda"))
    s.tau, s.caps = _selection(case, m.n_tokens)
    if case["call"] != "encode":
        s.enc.full_encode(s.first, s.caches)
    if case["call"] == "resume":
        s.saved = s.enc.export_raw(s.caches[0])
        s.nd = m.n_tokens * m.dim
    if case["graph"]:
        s.input = s.first.clone()
        s.graph = s.enc.step_graph(s.input, s.caches, s.tau, s.caps, s.out)
    return s


def run(s):
    frame = s.ring[s.t % RING]
    s.t += 1
    call = s.case["call"]
    if call == "encode":
        out = s.enc.encode_frame(frame, s.caches, 0, 1, s.tau, s.caps, out=s.out)
        return {"idx": out[0], "count": out[1], "refreshed": out[2]}
    if s.graph is not None:
        s.input.copy_(frame)
        s.enc.launch(s.graph)
        return {"idx": s.out[0], "count": s.out[1], "refreshed": s.out[2]}
    if call == "resume":
        s.enc.import_raw(s.saved, s.caches[0])
        out = s.enc.step(frame, s.caches, s.tau, s.caps, out=s.out)
        s.saved = s.enc.export_raw(s.caches[0])
        ref = s.saved[: s.nd * 4].view(torch.float32)
        return {"idx": out[0], "count": out[1], "refreshed": out[2], "ref": ref, "state": s.saved[s.nd * 4:].view(out[2].dtype)}
    out = s.enc.step(frame, s.caches, s.tau, s.caps, out=s.out)
    return {"idx": out[0], "count": out[1], "refreshed": out[2]}


# ------------------------------------------------------------------ work --


def _rows(case):
    """(tokens per stream, refreshed rows of the call)."""
    p = case["patch"]
    n = (case["img_h"] // p) * (case["img_w"] // p)
    if case["call"] == "encode":
        return n, n * case["streams"]
    if case["call"] == "top_k":
        return n, min(case["cap"], n) * case["streams"]
    rows = 0
    for v in range(case["streams"]):  # the tokens that a square at a random place and its former place touch
        s = _side(case, v)
        rows += min(n, round((s / p + 1) * ((s + SPEED) / p + 1)))
    return n, rows


def work(case):
    n, rows = _rows(case)
    B, D, F, L, P = case["streams"], case["dim"], case["mlp"], case["depth"], 3 * case["patch"] ** 2
    e = 2 if case["dtype"] == "bf16" else 4
    every = case["mlp_rows"] == "all"
    mlp = B * n if every else rows
    read = (P * D + L * (4 * D * D + 2 * D * F)) * e + n * D * 4 + B * n * P * 4
    flops = 2.0 * B * n * P * D + L * (2.0 * rows * 4 * D * D + 4.0 * mlp * D * F + 4.0 * rows * n * D)
    write = rows * D * (4 + e) + L * 2 * rows * D * e + (L + 1) * mlp * D * e + mlp * D * e  # ref, refreshed; K, V; X; Y
    if case["call"] != "encode":
        read += B * n * D * 4 + L * 2 * (B * n - rows) * D * e  # references; keys and values of the kept rows
    if every:
        read += L * (B * n - rows) * D * e
        write += L * rows * D * e
    if case["score"] == "key":
        flops += 2.0 * B * n * D * D
    if case["call"] == "resume":  # the saved state in and out
        state = n * D * 4 + (3 * L + 2) * n * D * e
        read += state
        write += state
    return {"bytes": float(read + write), "flops": float(flops)}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / (6e14 if case["dtype"] == "bf16" else 4e13)) + 2e-5 * case["depth"]


def tolerance(case):
    # Measured with the sums in another order (other K splits, columns per workgroup and attention waves through the tuning
    # call), and against 64 bits: fp32 stacks differ by 3e-7 (largest value 6e-6) and are 5e-7 from 64 bits.  bf16 storage
    # rounds every operation's result, and one rounding that falls the other way travels through the residual stream: two
    # orders differ by 7.3e-3 (6 layers) to 1.35e-2 (27 layers), the largest value by 0.05 to 0.2, and
    # each is as far from 64 bits.  About four times that.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 3e-5}
    return {"rel": 0.03, "max": 0.6}


# ----------------------------------------------------------------- exact --


def _exact_params(m, seed):
    w = _weights(m, seed)
    if m.dtype == "bf16":
        w = w.to(torch.bfloat16)
    par, o = {}, 0
    for name, shape in synth.param_shapes(m):
        n = math.prod(shape)
        par[name] = w[o:o + n].double().reshape(shape)
        o += n
    return par


def _norm(x, g, b, eps):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), g, b, eps)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


class _Plain:
    """The method in plain torch and 64 bits, one stream: state = reference, layer inputs, keys, values, branches, output."""

    def __init__(self, m, par, case):
        self.m, self.par, self.case = m, par, case

    def tokens(self, patches):
        return patches.double() @ self.par["w_pe"] + self.par["b_pe"] + self.par["pos"]

    def score(self, t0):
        if self.case["score"] == "embed":
            return t0
        D = self.m.dim
        x = t0.to(torch.bfloat16).double() if self.m.dtype == "bf16" else t0
        x = _norm(x, self.par["l0.ln1_g"], self.par["l0.ln1_b"], self.m.ln_eps)
        return x @ self.par["l0.w_qkv"][:, D:2 * D] + self.par["l0.b_qkv"][D:2 * D]

    def layers(self, st, rows, x_all):
        """Rows `rows` through every layer (x_all: their, or with every row in the MLP all rows', layer-0 inputs)."""
        m, par, every = self.m, self.par, self.case["mlp_rows"] == "all"
        H, dh, N = m.heads, m.head_dim, m.n_tokens
        x = x_all
        for l in range(m.depth):
            p = {k: par["l%d.%s" % (l, k)] for k in synth.LAYER_PARAMS}
            if every:
                st["X"][l][:] = x
            else:
                st["X"][l][rows] = x
            u = x[rows] if every else x
            if len(rows):
                q, k, v = (_norm(u, p["ln1_g"], p["ln1_b"], m.ln_eps) @ p["w_qkv"] + p["b_qkv"]).chunk(3, dim=-1)
                st["K"][l][rows], st["V"][l][rows] = k, v
                qh = q.reshape(-1, H, dh).transpose(0, 1).contiguous()
                kh = st["K"][l].reshape(N, H, dh).permute(1, 2, 0).contiguous()
                vh = st["V"][l].reshape(N, H, dh).transpose(0, 1).contiguous()
                o = torch.softmax((qh @ kh) / math.sqrt(dh), dim=-1) @ vh
                a = o.transpose(0, 1).reshape(-1, m.dim) @ p["w_o"] + p["b_o"]
                if every:
                    st["A"][l][rows] = a
            if every:
                a = st["A"][l]
            h = x + a
            x = h + _gelu(_norm(h, p["ln2_g"], p["ln2_b"], m.ln_eps) @ p["w_1"] + p["b_1"]) @ p["w_2"] + p["b_2"]
        y = _norm(x, par["lnf_g"], par["lnf_b"], m.ln_eps)
        if every:
            st["X"][m.depth][:], st["Y"][:] = x, y
            return y[rows]
        st["X"][m.depth][rows], st["Y"][rows] = x, y
        return y

    def encode(self, patches):
        m = self.m
        z = lambda n: torch.zeros((n, m.n_tokens, m.dim), dtype=torch.float64, device="cuda")  # noqa: E731
        t0 = self.tokens(patches)
        st = {"ref": self.score(t0), "X": z(m.depth + 1), "K": z(m.depth), "V": z(m.depth), "A": z(m.depth), "Y": z(1)[0]}
        self.layers(st, torch.arange(m.n_tokens, device="cuda"), t0)
        return st

    def step(self, st, patches, tau, cap):
        t0 = self.tokens(patches)
        sc = self.score(t0)
        sim = (sc * st["ref"]).sum(-1) / (sc.norm(dim=-1) * st["ref"].norm(dim=-1)).clamp_min(1e-8)
        rows = torch.nonzero(sim < tau).flatten()
        if len(rows) > cap:
            rows = rows[torch.argsort(sim[rows], stable=True)[:cap]].sort().values
        st["ref"][rows] = sc[rows]
        return rows, self.layers(st, rows, t0 if self.case["mlp_rows"] == "all" else t0[rows])


def exact(case, seed):
    m = _model(case)
    B, N = case["streams"], m.n_tokens
    plain = _Plain(m, _exact_params(m, seed), case)
    frames = _frames(case, seed)
    tau, caps = _selection(case, N)
    idx = torch.zeros((B, N), dtype=torch.int32, device="cuda")
    count = torch.zeros((B,), dtype=torch.int32, device="cuda")
    out = torch.zeros((B, N, m.dim), dtype=torch.float64, device="cuda")
    for v in range(B):
        if case["call"] == "encode":
            st = plain.encode(frames[1, v])
            rows, y = torch.arange(N, device="cuda"), st["Y"]
        else:
            st = plain.encode(frames[0, v])
            rows, y = plain.step(st, frames[1, v], tau, caps[v])
        idx[v, :len(rows)], count[v], out[v, :len(rows)] = rows.int(), len(rows), y
    got = {"idx": idx, "count": count, "refreshed": out}
    if case["call"] == "resume":
        got["ref"] = st["ref"].flatten()
        got["state"] = torch.cat([st[k].flatten() for k in ("X", "K", "V", "Y")])
    return got
