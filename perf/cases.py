"""Timed cases of the decode, training and export paths, through the public Python entry points.

Each case is a dict of plain values; `prepare` makes what a program holds before the call (model
buffers, queries or requests, a context with its reservation and launch shape, a trainer), `run`
is one pass, `work` the bytes and operations that the pass cannot do without and `exact` the same
outputs in 64-bit torch arithmetic, written from the storage formats and the method alone.

Kinds:
  query         Context.decode: random access to a BC4 + grid model
  pages         Context.decode_pages: virtual-texturing pages of one or several maps
  hybrid_query  Context.hybrid_decode: random access to a model in the paper's hybrid layout
  hybrid_pages  Context.hybrid_decode_pages: per-tile models, one page each, with a border
  train         Trainer.step, or forward and backward through autograd, under BC simulation
  hybrid_train  HybridTrainer.step of several per-tile models
  encode        HybridTrainer.encode: export of trained tile models as BC7 or BC4 blocks
"""
import math

import numpy as np
import torch

from paper_2604_12625_amd import inputs as I
from paper_2604_12625_amd import ndgi as N
from paper_2604_12625_amd import train as TR

DEV = "cuda"
PREC = {"f16": N.PREC_F16, "f32": N.PREC_F32}
TORCH = {"f16": torch.float16, "f32": torch.float32}
BYTES = {"f16": 2, "f32": 4}
GAMMA = 2.2
MLP_FLOP = 2 * (16 * 32 + 32 * 32 + 32 * 3)


def listed():
    return [
        # the tiny parity map, one sweep's worth of queries: latency of the smallest call
        dict(name="query_small_f32", kind="query", W=64, H=64, Gw=16, Gh=16, T=8, store="f32", prec="f32", n=4096,
             reserve=False),
        # shading points scattered over a large map, too few a tile to be worth binning
        dict(name="query_sparse_f16", kind="query", W=2048, H=2048, Gw=512, Gh=512, T=24, store="f16", prec="f16",
             n=200003, reserve=False),
        # a batch on a 48-key model in full precision (baking checks), binned, an odd count
        dict(name="query_48keys_f32", kind="query", W=1024, H=1024, Gw=256, Gh=256, T=48, store="f16", prec="f32",
             n=1000003, reserve=True),
        # the benchmark's random leg: 16,000,000 queries of the 4096^2 x 24 model
        dict(name="query_16m_f16", kind="query", W=4096, H=4096, Gw=1024, Gh=1024, T=24, store="f16", prec="f16",
             n=16000000, reserve=True),
        # the benchmark's frame: every 128^2 page of the 4096^2 map at one time
        dict(name="frame_4096_f16", kind="pages", maps=1, W=4096, H=4096, ratio=4, T=24, store="f16", prec="f16",
             page=128, requests=0, tile_w=2, tile_h=16, graph=False),
        # one virtual-texturing frame: 2000 requests over 32 maps of 256 .. 4096 texels a side
        dict(name="vt_frame_f16", kind="pages", maps=32, W=0, H=0, ratio=4, T=24, store="f16", prec="f16", page=128,
             requests=2000, tile_w=2, tile_h=16, graph=True),
        # a whole map in full precision, its grid at no simple ratio of the texels
        dict(name="pages_ragged_f32", kind="pages", maps=1, W=1600, H=1152, ratio=0, T=16, store="f32", prec="f32",
             page=64, requests=0, tile_w=1, tile_h=4, graph=False),
        # the paper's storage: a 1024^2 lightmap as 64 tile models with 4-texel mirrored borders
        dict(name="hybrid_tiles_m_f16", kind="hybrid_pages", profile="M", codec=1, modes="6", prec="f16", models=64,
             page=128, border=4),
        # random access to the widest decoder's layout
        dict(name="hybrid_query_m64_f16", kind="hybrid_query", profile="M.64", codec=0, modes="", prec="f16", W=128,
             H=128, n=300007),
        # one optimisation step of a 1024^2 x 24 model, 2^18 samples
        dict(name="train_1024", kind="train", W=1024, H=1024, Gw=256, Gh=256, T=24, n=262144, mode="step"),
        # one optimisation step of 64 tile models, the paper's batch of 4096 samples each
        dict(name="hybrid_train_m", kind="hybrid_train", profile="M", codec=1, models=64, per_model=4096, noise=True),
        # the paper's export of eight trained tile models
        dict(name="encode_bc7_m", kind="encode", profile="M", state=1, codec=1, models=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    return max(lo, min(hi, 4 * int(round(_log(rng, lo, hi) / 4))))


def draw(rng):
    kind = rng.choice(["query", "query", "pages", "pages", "hybrid_query", "hybrid_pages", "train", "hybrid_train",
                       "encode"])
    if kind == "query":
        W, H = _side(rng, 64, 4096), _side(rng, 64, 4096)
        four = rng.random() < 0.7
        Gw, Gh = (W // 4, H // 4) if four else (_log(rng, 8, W // 3), _log(rng, 8, H // 3))
        T = rng.randint(2, 48)
        return dict(kind=kind, W=W, H=H, Gw=Gw, Gh=Gh, T=T, store=rng.choice(["f16", "f16", "f32"]),
                    prec=rng.choice(["f16", "f16", "f32"]), n=_log(rng, 1000, 8000000), reserve=rng.random() < 0.6)
    if kind == "pages":
        page = rng.choice([64, 128, 128, 256])
        prec = rng.choice(["f16", "f16", "f32"])
        if rng.random() < 0.5:
            return dict(kind=kind, maps=rng.randint(2, 32), W=0, H=0, ratio=4, T=rng.randint(2, 24), store="f16",
                        prec=prec, page=128, requests=_log(rng, 5, 1500), tile_w=rng.choice([1, 2]),
                        tile_h=rng.choice([4, 16]), graph=rng.random() < 0.5)
        four = rng.random() < 0.6
        return dict(kind=kind, maps=1, W=page * rng.randint(1, 3072 // page), H=page * rng.randint(1, 3072 // page),
                    ratio=4 if four else 0, T=rng.randint(2, 24), store=rng.choice(["f16", "f16", "f32"]), prec=prec,
                    page=page, requests=0, tile_w=rng.choice([1, 2]), tile_h=rng.choice([4, 16]), graph=False)
    profile = rng.choice(["L", "M", "H", "M.64"])
    codec = rng.choice([1, 1, 0])
    modes = rng.choice(["6", "456"]) if codec else ""
    if kind == "hybrid_query":
        return dict(kind=kind, profile=profile, codec=codec, modes=modes, prec=rng.choice(["f16", "f32"]),
                    W=4 * rng.randint(16, 128), H=4 * rng.randint(16, 128), n=_log(rng, 1000, 2000000))
    if kind == "hybrid_pages":
        return dict(kind=kind, profile=profile, codec=codec, modes=modes, prec=rng.choice(["f16", "f16", "f32"]),
                    models=_log(rng, 1, 128), page=128, border=rng.choice([0, 4, 4, 7]))
    if kind == "train":
        W, H = _side(rng, 64, 1024), _side(rng, 64, 1024)
        four = rng.random() < 0.7
        return dict(kind=kind, W=W, H=H, Gw=W // 4 if four else _log(rng, 8, W // 3),
                    Gh=H // 4 if four else _log(rng, 8, H // 3), T=rng.randint(2, 24), n=_log(rng, 1000, 262144),
                    mode=rng.choice(["step", "step", "autograd"]))
    if kind == "hybrid_train":
        models = _log(rng, 1, 64)
        return dict(kind=kind, profile=profile, codec=codec, models=models, per_model=64 * _log(rng, 8, 64),
                    noise=rng.random() < 0.8)
    return dict(kind="encode", profile=rng.choice(["L", "M", "H"]), state=rng.choice([1, 0]), codec=codec,
                models=rng.randint(1, 3 if codec else 1))


# ------------------------------------------------------------------------------- inputs

def _scene_frames(side_w, side_h, times, seed, purpose):
    """Frames [k][H][W][3] FP16 of a synthetic temporal lightmap of side_w x side_h texels."""
    scene = I.light_scene(max(side_w, side_h), max(side_w, side_h), I.rng(purpose, I.P_TARGET, seed))
    scene = dict(scene, W=side_w, H=side_h)
    return torch.stack([I.scene_frame_torch(scene, float(t), device=DEV).to(torch.float16) for t in times])


def _grid_dims(c):
    return (c["W"] // 4, c["H"] // 4) if c["ratio"] == 4 else (c["W"] // 8, c["H"] // 8)


def _page_inputs(c, seed):
    """(model tensors, request columns, dst texels, pitch) of a pages case."""
    page = c["page"]
    if c["maps"] == 1:
        sides = [(c["W"], c["H"]) + _grid_dims(c)]
    else:
        s = [int(x) for x in I.vt_map_sides(c["maps"], I.rng(3, I.P_MODEL, c["maps"]))]
        sides = [(x, x, x // 4, x // 4) for x in s]
    models = [I.random_model_torch(w, h, gw, gh, c["T"], seed=1000 * (seed % 100003) + i, device=DEV,
                                   grid_dtype="float16" if c["store"] == "f16" else "float32",
                                   mlp_dtype="float16" if c["store"] == "f16" else "float32")
              for i, (w, h, gw, gh) in enumerate(sides)]
    if c["maps"] == 1:
        py, px = np.meshgrid(np.arange(c["H"] // page), np.arange(c["W"] // page), indexing="ij")
        px, py = px.ravel(), py.ravel()
        mi = np.zeros(px.size, np.int32)
        t = np.full(px.size, np.float32(I.rng(3, I.P_REQ, seed).random()), np.float32)
        off, pitch, texels = (py * page * c["W"] + px * page).astype(np.int64), c["W"], c["W"] * c["H"]
    else:
        mi, px, py, t = I.vt_requests([s[0] for s in sides], c["requests"], I.rng(3, I.P_REQ, seed), page=page)
        k, row = np.arange(c["requests"]), 50
        pitch = row * page
        off = ((k // row) * page * pitch + (k % row) * page).astype(np.int64)
        texels = -(-c["requests"] // row) * page * pitch
    return models, (mi, px, py, t, off), texels, pitch


def _hybrid_numpy(c, seed, i, W=128, H=128):
    modes = tuple(int(x) for x in c["modes"]) or (6,)
    return I.random_hybrid_model(W=W, H=H, profile=c["profile"], config=6 + 16 * (seed % 100003), index=i,
                                 codec=c["codec"], bc7_modes=modes)


def _hybrid_requests(c, seed):
    n, R = c["models"], c["page"] + 2 * c["border"]
    per_row = min(8, n)
    k = np.arange(n)
    pitch = per_row * R
    off = ((k // per_row) * R * pitch + (k % per_row) * R).astype(np.int64)
    t = np.float32(I.rng(6, I.P_REQ, seed).random())
    return t, off, pitch, -(-n // per_row) * R * pitch


def _train_inputs(c, seed):
    """(initial state, target [T][H][W][3] FP16, packed samples, Adam moments) of a train case: a
    state some steps into a run, its moments of the size of the gradients."""
    W, H, T, n = c["W"], c["H"], c["T"], c["n"]
    tgt = _scene_frames(W, H, [k / T for k in range(T)], seed, 4)
    mean = tgt.float().mean(dim=(0, 1, 2)).cpu().numpy()
    init = I.train_init_torch(W, H, c["Gw"], c["Gh"], T, mean, seed=seed, device=DEV)
    smp = I.train_samples_torch(n, W, H, T, seed=seed + 1, device=DEV)
    return init, tgt, smp, _moments(init["flat"].numel(), N.MLP_SIZE, 0.3 / n, seed)


def _moments(count, n_mlp, size, seed):
    """Adam moments (m, v): sqrt(v) of `size` for features and of 0.05 for the last n_mlp."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 2)
    s = torch.full((count,), size, dtype=torch.float32, device=DEV)
    s[count - n_mlp:] = 0.05
    v = (s * (0.5 + torch.rand(count, generator=gen, device=DEV))) ** 2
    m = 0.1 * s * torch.randn(count, generator=gen, device=DEV)
    return m, v


def _htrain_init(c, seed, i, keys, codec):
    return I.hybrid_train_init(128, 128, c["profile"], len(keys), keys, I.rng(7, I.P_INIT, 4096 * (seed % 100003) + i),
                               codec=codec)


def _htrain_inputs(c, seed):
    """(initial states, key times, normalised float target [M][frames][128][128][3], samples, moments)."""
    keys = I.lightmap_key_times(I.rng(6, I.P_MODEL, 1))
    M, B = c["models"], c["per_model"]
    inits = [_htrain_init(c, seed, i, keys, c["codec"]) for i in range(M)]
    cols = min(8, M)
    rows = -(-M // cols)
    full = _scene_frames(128 * cols, 128 * rows, keys, seed, 7)
    tiles = full.view(len(keys), rows, 128, cols, 128, 3).permute(1, 3, 0, 2, 4, 5)
    tiles = tiles.reshape(rows * cols, len(keys), 128, 128, 3)[:M]
    y = tiles.float() ** (1.0 / GAMMA)
    tgt = (y / y.double().mean(dim=(2, 3), keepdim=True).float()).contiguous()
    smp = I.train_samples_torch(M * B, 128, 128, len(keys), seed=seed + 1, device=DEV, border=4)
    hid = I.HYBRID_PROFILES[c["profile"]][1]
    n_par = sum(np.asarray(inits[0][k]).size for k in TR.HYB_KEYS) * M
    return inits, keys, tgt, smp, _moments(n_par, M * I.hybrid_mlp_size(hid), 1.0 / B, seed)


# ------------------------------------------------------------------------- prepare, run

def prepare(case, seed):
    c = case
    s = dict(case=c, ctx=N.Context(0))
    if c["kind"] == "query":
        dt = "float16" if c["store"] == "f16" else "float32"
        m = I.random_model_torch(c["W"], c["H"], c["Gw"], c["Gh"], c["T"], seed=seed, device=DEV, grid_dtype=dt,
                                 mlp_dtype=dt)
        s["model"] = N.DeviceModel(c["W"], c["H"], c["Gw"], c["Gh"], c["T"], m["bc4"], m["grid"], m["mlp"])
        s["q"] = I.uniform_queries_torch(c["n"], seed=seed + 1, device=DEV)
        s["out"] = torch.zeros((c["n"], 3), dtype=TORCH[c["prec"]], device=DEV)
        if c["reserve"]:
            s["ctx"].reserve_decode(s["model"], c["n"])
    elif c["kind"] == "pages":
        models, (mi, px, py, t, off), texels, pitch = _page_inputs(c, seed)
        s["models"] = [N.DeviceModel(m["W"], m["H"], m["Gw"], m["Gh"], m["T"], m["bc4"], m["grid"], m["mlp"])
                       for m in models]
        s["marr"] = N.models_array(s["models"])
        s["rq"] = N.page_requests(mi, px, py, t, off)
        s["n"], s["pitch"] = len(mi), pitch
        s["nreq"] = torch.tensor([len(mi)], dtype=torch.int32, device=DEV)
        s["out"] = torch.zeros((texels, 3), dtype=TORCH[c["prec"]], device=DEV)
        s["ctx"].set_launch(c["tile_w"], c["tile_h"], 32)
    elif c["kind"] == "hybrid_query":
        s["model"] = N.HybridModel.from_numpy(_hybrid_numpy(c, seed, 0, c["W"], c["H"]))
        s["q"] = I.uniform_queries_torch(c["n"], seed=seed + 1, device=DEV)
        s["out"] = torch.zeros((c["n"], 3), dtype=TORCH[c["prec"]], device=DEV)
    elif c["kind"] == "hybrid_pages":
        t, off, pitch, texels = _hybrid_requests(c, seed)
        n = c["models"]
        s["models"] = [N.HybridModel.from_numpy(_hybrid_numpy(c, seed, i)) for i in range(n)]
        s["marr"] = N.models_array(s["models"])
        zero = np.zeros(n, np.int32)
        s["rq"] = N.page_requests(np.arange(n, dtype=np.int32), zero, zero, np.full(n, t, np.float32), off)
        s["nreq"] = torch.tensor([n], dtype=torch.int32, device=DEV)
        s["pitch"], s["widths"] = pitch, 2 if I.HYBRID_PROFILES[c["profile"]][1] == 64 else 1
        s["out"] = torch.zeros((texels, 3), dtype=TORCH[c["prec"]], device=DEV)
    elif c["kind"] == "train":
        init, tgt, s["smp"], (m, v) = _train_inputs(c, seed)
        s["tr"] = TR.Trainer(s["ctx"], init, lr_feat=1e-2, lr_mlp=1e-3)
        s["tr"].m.copy_(m)
        s["tr"].v.copy_(v)
        s["tr"].state.step = 1000
        s["tgt"] = tgt.view(torch.int16)
        s["tr"].params.requires_grad_(c["mode"] == "autograd")
        if c["mode"] == "autograd":
            gen = torch.Generator(device=DEV)
            gen.manual_seed(seed + 3)
            s["gp"] = torch.randn((c["n"], 3), generator=gen, device=DEV) / c["n"]
    elif c["kind"] == "hybrid_train":
        inits, _, s["tgt"], s["smp"], (m, v) = _htrain_inputs(c, seed)
        s["tr"] = TR.HybridTrainer(s["ctx"], inits, lr_feat=1e-3, lr_mlp=1e-3, seed=1, per_model=c["per_model"])
        s["tr"].m.copy_(m)
        s["tr"].v.copy_(v)
        s["tr"].state.step = 1000
    else:
        keys = I.lightmap_key_times(I.rng(6, I.P_MODEL, 1))
        inits = [_htrain_init(c, seed, i, keys, c["state"]) for i in range(c["models"])]
        s["tr"] = TR.HybridTrainer(s["ctx"], inits, lr_feat=1e-3, lr_mlp=1e-3, seed=1, per_model=4096)
    return s


def run(state):
    s, c = state, state["case"]
    ctx = s["ctx"]
    if c["kind"] == "query":
        return ctx.decode(s["model"], s["q"], PREC[c["prec"]], out=s["out"])
    if c["kind"] == "pages":
        return ctx.decode_pages(s["marr"], len(s["models"]), s["rq"], s["nreq"], s["n"], c["page"], s["out"],
                                s["pitch"], PREC[c["prec"]], graph=c["graph"])
    if c["kind"] == "hybrid_query":
        return ctx.hybrid_decode(s["model"], s["q"], PREC[c["prec"]], out=s["out"])
    if c["kind"] == "hybrid_pages":
        return ctx.hybrid_decode_pages(s["marr"], c["models"], s["rq"], s["nreq"], c["models"], c["page"], s["out"],
                                       s["pitch"], PREC[c["prec"]], widths=s["widths"], border=c["border"])
    if c["kind"] == "train":
        if c["mode"] == "step":
            return [s["tr"].step(s["smp"], s["tgt"]), s["tr"].params]
        p = s["tr"].params
        p.grad = None
        pred = TR.ndgi_apply(s["tr"], s["smp"])
        pred.backward(s["gp"])
        return [pred, p.grad]
    if c["kind"] == "hybrid_train":
        return [s["tr"].step(s["smp"], s["tgt"], N.HTRAIN_NOISE if c["noise"] else 0), s["tr"].params]
    out = []
    for m in range(c["models"]):
        e = s["tr"].encode(0, c["codec"], N.DTYPE_F16, model=m).arrays
        out.append([e[0], e[1], e[2], e[3], e[5]])
    return out


# -------------------------------------------------------------------------------- work

def work(case):
    c = case
    if c["kind"] == "query":
        node = 8 * BYTES[c["store"]]
        # a map that the queries cover is read once; a sparse batch reads a footprint and eight nodes a query
        maps = min(c["W"] * c["H"] * 4, 64 * c["n"]) + min(c["T"] * c["Gw"] * c["Gh"] * node, 8 * node * c["n"])
        return dict(bytes=maps + c["n"] * (12 + 3 * BYTES[c["prec"]]), flops=MLP_FLOP * c["n"])
    if c["kind"] == "pages":
        if c["maps"] == 1:
            texels = c["W"] * c["H"]
            gw, gh = _grid_dims(c)
            maps = texels * 4 + 2 * gw * gh * 8 * BYTES[c["store"]]
        else:
            texels = c["requests"] * c["page"] ** 2
            maps = texels * (4 + 2)   # at most: a page asked for twice is read once
        return dict(bytes=maps + texels * 3 * BYTES[c["prec"]], flops=MLP_FLOP * texels)
    if c["kind"] in ("hybrid_query", "hybrid_pages"):
        side, hid = I.HYBRID_PROFILES[c["profile"]]
        bpt = 1 if c["codec"] else 2
        if c["kind"] == "hybrid_query":
            n, slices, M, W, H = c["n"], 12, 1, c["W"], c["H"]
            extra = 12 * n + 2 * 64 * 24 * 2
        else:
            n, slices, M, W, H = c["models"] * (c["page"] + 2 * c["border"]) ** 2, 2, c["models"], 128, 128
            extra = 2 * 2 * 128
        per = (W * H + slices * side * side) * bpt + 2 * I.hybrid_mlp_size(hid)
        return dict(bytes=M * per + extra + n * 3 * BYTES[c["prec"]], flops=n * 2 * (16 * hid + hid * hid + 3 * hid))
    if c["kind"] == "train":
        n_par = c["W"] * c["H"] * 9 + c["T"] * c["Gw"] * c["Gh"] * 8 + N.MLP_SIZE
        b = c["n"] * (4 + 6) + n_par * 24 if c["mode"] == "step" else c["n"] * (4 + 24) + n_par * 8
        return dict(bytes=b, flops=3 * MLP_FLOP * c["n"])
    side, hid = I.HYBRID_PROFILES[c["profile"]]
    cw = 1 if c["codec" if c["kind"] == "hybrid_train" else "state"] else 4
    texels = 128 * 128 + 12 * side * side
    n_par = c["models"] * (texels // 2 + texels * cw + 2 * 64 * 24 * 2 + I.hybrid_mlp_size(hid))
    if c["kind"] == "hybrid_train":
        n = c["models"] * c["per_model"]
        return dict(bytes=n * (4 + 12) + n_par * 24, flops=3 * n * 2 * (16 * hid + hid * hid + 3 * hid))
    return dict(bytes=4 * n_par + c["models"] * texels * (1 if c["codec"] else 2), flops=0)


# ------------------------------------------------------------- the same in 64-bit torch

def _axis(c, size):
    """Texel-centre bilinear neighbours of normalised coordinate c (float64): i0, i1, w1."""
    q = c * size - 0.5
    f = torch.floor(q)
    w = q - f
    inside = (q >= -1.0) & (q <= size)
    i = f.clamp(-2, size + 1).long()
    return i.clamp(0, size - 1), (i + 1).clamp(0, size - 1), torch.where(inside, w, torch.zeros_like(w))


def _bc4_texels(blocks, C):
    """[H/4][W/4][C][8] BC4 blocks to texels [H][W][C] (uint8)."""
    hb, wb = blocks.shape[:2]
    out = torch.empty((hb, 4, wb, 4, C), dtype=torch.uint8, device=blocks.device)
    for y0 in range(0, hb, 64):
        b = blocks[y0:y0 + 64].to(torch.int32)
        e0, e1 = b[..., 0], b[..., 1]
        sel = sum(b[..., 2 + k].long() << (8 * k) for k in range(6))
        eight = e0 > e1
        for s in range(16):
            k = ((sel >> (3 * s)) & 7).to(torch.int32)
            j8 = torch.where(k == 0, 0, torch.where(k == 1, 7, k - 1))
            j6 = torch.where(k == 0, 0, torch.where(k == 1, 5, k - 1)).clamp(max=5)
            v8 = ((7 - j8) * e0 + j8 * e1 + 3) // 7
            v6 = ((5 - j6) * e0 + j6 * e1 + 2) // 5
            v6 = torch.where(k == 6, 0, torch.where(k == 7, 255, v6))
            out[y0:y0 + 64, s >> 2, :, s & 3] = torch.where(eight, v8, v6).to(torch.uint8)
    return out.reshape(4 * hb, 4 * wb, C)


def _bc7_texels(blocks):
    """[H/4][W/4][16] BC7 blocks of modes 4, 5 and 6 to texels [H][W][4] (int64)."""
    hb, wb = blocks.shape[:2]
    bit = (blocks.long()[..., None] >> torch.arange(8, device=blocks.device)) & 1
    bit = bit.reshape(hb, wb, 128)

    def bits(pos, n):
        return sum(bit[..., pos + k] << k for k in range(n))

    def index(pos, b, s):
        return bits(pos, b - 1) if s == 0 else bits(pos + b - 1 + b * (s - 1), b)

    def expand(v, n):
        return (v << (8 - n)) | (v >> (2 * n - 8)) if n < 8 else v

    def weight(j, b):
        return (64 * j + ((1 << b) - 1) // 2) // ((1 << b) - 1)

    def lerp(w, a, b):
        return ((64 - w) * a + w * b + 32) >> 6

    def rotate(t, rot):
        t = list(t)
        a = t[3]
        new = [torch.where(rot == c + 1, a, t[c]) for c in range(3)]
        alpha = torch.where(rot == 1, t[0], torch.where(rot == 2, t[1], torch.where(rot == 3, t[2], a)))
        return torch.stack(new + [alpha], -1)

    low = blocks[..., 0].long()
    m6, m5, m4 = (low & 0x7f) == 0x40, (low & 0x3f) == 0x20, (low & 0x1f) == 0x10
    out = torch.zeros((hb, 4, wb, 4, 4), dtype=torch.int64, device=blocks.device)
    for s in range(16):
        w = weight(index(65, 4, s), 4)
        t6 = torch.stack([lerp(w, (bits(7 + 14 * c, 7) << 1) | bits(63, 1), (bits(14 + 14 * c, 7) << 1) | bits(64, 1))
                          for c in range(4)], -1)
        wc, wa = weight(index(66, 2, s), 2), weight(index(97, 2, s), 2)
        t5 = rotate([lerp(wc, expand(bits(8 + 14 * c, 7), 7), expand(bits(15 + 14 * c, 7), 7)) for c in range(3)]
                    + [lerp(wa, bits(50, 8), bits(58, 8))], bits(6, 2))
        w2, w3, sel = weight(index(50, 2, s), 2), weight(index(81, 3, s), 3), bits(7, 1) == 1
        wc, wa = torch.where(sel, w3, w2), torch.where(sel, w2, w3)
        t4 = rotate([lerp(wc, expand(bits(8 + 10 * c, 5), 5), expand(bits(13 + 10 * c, 5), 5)) for c in range(3)]
                    + [lerp(wa, expand(bits(38, 6), 6), expand(bits(44, 6), 6))], bits(5, 2))
        t = torch.where(m6[..., None], t6, torch.where(m5[..., None], t5, torch.where(m4[..., None], t4, 0)))
        out[:, s >> 2, :, s & 3] = t
    return out.reshape(4 * hb, 4 * wb, 4)


def _bilinear(tex, u, v):
    """tex [H][W][C] sampled at (u, v), in float64."""
    x0, x1, wx = _axis(u, tex.shape[1])
    y0, y1, wy = _axis(v, tex.shape[0])
    f = lambda y, x: tex[y, x].double()  # noqa: E731
    wx, wy = wx[:, None], wy[:, None]
    return (1 - wy) * ((1 - wx) * f(y0, x0) + wx * f(y0, x1)) + wy * ((1 - wx) * f(y1, x0) + wx * f(y1, x1))


def _mlp(p, x, hid, act, last):
    p = p.double()
    o1 = hid * 16
    o2 = o1 + hid
    o3 = o2 + hid * hid
    o4 = o3 + hid
    o5 = o4 + 3 * hid
    h = act(x @ p[:o1].view(hid, 16).T + p[o1:o2])
    h = act(h @ p[o2:o3].view(hid, hid).T + p[o3:o4])
    return last(h @ p[o4:o5].view(3, hid).T + p[o5:])


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _same(x):
    return x


def _decode64(m, tex, u, v, t):
    """A BC4 + grid model (texels decoded) at float64 (u, v, t): RGB."""
    T, Gh, Gw = m["grid"].shape[:3]
    tw = t - torch.floor(t)
    k = torch.floor(tw * T).long().clamp(max=T - 1)
    w = (tw * T - k)[:, None]
    flat = m["grid"].reshape(T * Gh, Gw, 8)
    x0, x1, wx = _axis(u, Gw)
    y0, y1, wy = _axis(v, Gh)
    wx, wy = wx[:, None], wy[:, None]
    g = 0.0
    for key, wk in ((k, 1 - w), ((k + 1) % T, w)):
        f = lambda y, x: flat[key * Gh + y, x].double()  # noqa: E731
        g = g + wk * ((1 - wy) * ((1 - wx) * f(y0, x0) + wx * f(y0, x1)) + wy * ((1 - wx) * f(y1, x0) + wx * f(y1, x1)))
    return _mlp(m["mlp"], torch.cat([_bilinear(tex, u, v) / 255.0, g], 1), 32, torch.relu, torch.exp)


def _nodes(tau, n):
    p = tau * (n - 1)
    i = torch.floor(p).long().clamp(0, max(n - 2, 0))
    return i, (i + 1).clamp(max=n - 1), p - i


def _tau(t, keys):
    n = keys.numel()
    if n == 0:
        return t
    k = keys.double()
    i = (torch.searchsorted(k, t.contiguous(), right=True) - 1).clamp(0, n - 2)
    return ((i + (t - k[i]) / (k[i + 1] - k[i])) / (n - 1)).clamp(0, 1)


def _gamma(t):
    return torch.stack([torch.sin(math.pi * t), torch.cos(math.pi * t), torch.sin(2 * math.pi * t),
                        torch.cos(2 * math.pi * t)], 1)


def _hybrid_maps(m, codec):
    """Decoded maps of a numpy hybrid model on the device."""
    d = {k: torch.from_numpy(m[k]).to(DEV) for k in ("fuv", "fuvt", "fut", "fvt", "keys", "mlp")}
    dec = _bc7_texels if codec else (lambda b: _bc4_texels(b, 4))
    s = d["fuvt"].shape[0]
    d["uvt"] = torch.cat([dec(d["fuvt"][k]) for k in range(s)], 0)     # [S Gv][Gu][4]
    d["uv"] = dec(d["fuv"])
    return d


def _hybrid64(d, m, u, v, t):
    t = t.clamp(0, 1)
    tau = _tau(t, d["keys"])
    s0, s1, ws = _nodes(tau, m["S"])
    x0, x1, wx = _axis(u, m["Gu"])
    y0, y1, wy = _axis(v, m["Gv"])
    wx, wy = wx[:, None], wy[:, None]
    V = 0.0
    for s, w in ((s0, 1 - ws), (s1, ws)):
        f = lambda y, x: d["uvt"][s * m["Gv"] + y, x].double()  # noqa: E731
        V = V + w[:, None] * ((1 - wy) * ((1 - wx) * f(y0, x0) + wx * f(y0, x1))
                              + wy * ((1 - wx) * f(y1, x0) + wx * f(y1, x1)))
    k0, k1, wk = _nodes(tau, m["Tt"])
    planes = []
    for c, size, p in ((u, m["U"], d["fut"]), (v, m["V"], d["fvt"])):
        a0, a1, wa = _axis(c, size)
        wa, w = wa[:, None], wk[:, None]
        planes.append((1 - w) * ((1 - wa) * p[k0, a0].double() + wa * p[k0, a1].double())
                      + w * ((1 - wa) * p[k1, a0].double() + wa * p[k1, a1].double()))
    x = torch.cat([V / 255.0, _bilinear(d["uv"], u, v) / 255.0, planes[0] / 255.0, planes[1] / 255.0, _gamma(t)], 1)
    return _mlp(d["mlp"], x, m["hidden"], _gelu, _same)


def _adam64(p, g, m, v, lr, step=1001, b1=0.9, b2=0.999, eps=1e-8):
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    return p - lr * (m / (1 - b1 ** step)) / (torch.sqrt(v / (1 - b2 ** step)) + eps)


def _samples(smp):
    s = smp.long() & 0xffffffff
    return s & 0xfff, (s >> 12) & 0xfff, s >> 24


def _train64(c, seed):
    """Outputs of a train case: loss and stepped parameters, or prediction and gradient."""
    init, tgt, smp, (m, v) = _train_inputs(c, seed)
    W, H, Gw, Gh, T = c["W"], c["H"], c["Gw"], c["Gh"], c["T"]
    p = init["flat"].double().requires_grad_(True)
    n_e, n_w = W * H, W * H * 8
    n_f = n_e + n_w + T * Gh * Gw * 8
    x, y, k = _samples(smp)
    ep = p[:n_e].view(H // 4, W // 4, 8, 2)[y >> 2, x >> 2]
    w = p[n_e:n_e + n_w].view(H, W, 8)[y, x]
    E = torch.round(255.0 * ep.detach().float()).double()      # the simulation rounds single-precision products
    J = torch.round(7.0 * w.detach().float()).double()
    val = torch.floor(((7 - J) * E[..., 0] + J * E[..., 1] + 3) / 7) / 255.0
    lin = ep[..., 0] * (1 - J / 7) + ep[..., 1] * (J / 7) + w * (E[..., 1] - E[..., 0]) / 255.0
    grid = p[n_e + n_w:n_f].view(T * Gh, Gw, 8)
    u64, v64 = (x.double() + 0.5) / W, (y.double() + 0.5) / H
    x0, x1, wx = _axis(u64, Gw)
    y0, y1, wy = _axis(v64, Gh)
    wx, wy = wx[:, None], wy[:, None]
    f = lambda yy, xx: grid[k * Gh + yy, xx]  # noqa: E731
    g = (1 - wy) * ((1 - wx) * f(y0, x0) + wx * f(y0, x1)) + wy * ((1 - wx) * f(y1, x0) + wx * f(y1, x1))
    pred = _mlp(p[n_f:], torch.cat([val + (lin - lin.detach()), g], 1), 32, torch.relu, torch.exp)
    if c["mode"] == "autograd":
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed + 3)
        gp = torch.randn((c["n"], 3), generator=gen, device=DEV) / c["n"]
        pred.backward(gp.double())
        return [pred.detach(), p.grad]
    loss = ((pred - tgt[k, y, x].double()) ** 2).mean()
    loss.backward()
    with torch.no_grad():
        m, v, q = m.double(), v.double(), p.detach()
        feat = _adam64(q[:n_f], p.grad[:n_f], m[:n_f], v[:n_f], 1e-2)
        feat[:n_e + n_w].clamp_(0, 1)
        mlp = _adam64(q[n_f:], p.grad[n_f:], m[n_f:], v[n_f:], 1e-3)
        return [loss.detach().reshape(1), torch.cat([feat, mlp])]


def _noise64(seed, step, n):
    """U(-1/2, 1/2) of samples 0 .. n-1, channels 0 .. 11: SplitMix64 of a counter, top 24 bits."""
    wrap = lambda a: (a + (1 << 63)) % (1 << 64) - (1 << 63)  # noqa: E731
    shr = lambda a, k: (a >> k) & ((1 << (64 - k)) - 1)  # noqa: E731
    base = wrap(seed * 0x9E3779B97F4A7C15 + (step << 32) + 0x9E3779B97F4A7C15)
    z = torch.arange(n, device=DEV)[:, None] * 16 + torch.arange(12, device=DEV)[None] + base
    z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    return shr(z, 40).double() / (1 << 24) - 0.5


def _htrain64(c, seed):
    inits, keys, tgt, smp, (m, v) = _htrain_inputs(c, seed)
    M, B, d = c["models"], c["per_model"], inits[0]["dims"]
    side, hid = d["Gu"], d["hidden"]
    sizes = [np.asarray(inits[0][k]).size for k in TR.HYB_KEYS]
    n_feat, n_mlp = sum(sizes[:-1]), sizes[-1]
    flat = np.concatenate([np.concatenate([np.asarray(i[k], np.float32).ravel() for k in TR.HYB_KEYS[:-1]]) for i in inits]
                          + [np.asarray(i["mlp"], np.float32).ravel() for i in inits])
    p = torch.from_numpy(flat).to(DEV).double().requires_grad_(True)
    feats = p[:M * n_feat].view(M, n_feat)
    seg = dict(zip(TR.HYB_KEYS, torch.split(feats, sizes[:-1], dim=1)))
    x, y, f = _samples(smp)
    mi = torch.arange(M, device=DEV).repeat_interleave(B)
    cw = 1 if c["codec"] else 4
    fuv_ep, fuv_w = seg["fuv_ep"].reshape(M, 32, 32, 4, 2), seg["fuv_w"].reshape(M, 128, 128, cw)
    uvt_ep = seg["fuvt_ep"].reshape(M, 12, side // 4, side // 4, 4, 2)
    uvt_w = seg["fuvt_w"].reshape(M, 12, side, side, cw)
    fut, fvt = seg["fut"].reshape(M, 24, 64, 2), seg["fvt"].reshape(M, 24, 64, 2)

    def lerp(ep, w):
        return (1 - w) * ep[..., 0] + w * ep[..., 1]

    tau = f.double() / (d["frames"] - 1)
    t = torch.from_numpy(np.asarray(keys, np.float32)).to(DEV).double()[f]
    u64, v64 = (x.double() + 0.5) / 128, (y.double() + 0.5) / 128
    V = 0.0
    x0, x1, wx = _axis(u64, side)
    y0, y1, wy = _axis(v64, side)
    s0, s1, ws = _nodes(tau, 12)
    for ss, wgt in ((s0, 1 - ws), (s1, ws)):
        for yy, wyy in ((y0, 1 - wy), (y1, wy)):
            for xx, wxx in ((x0, 1 - wx), (x1, wx)):
                V = V + (wgt * wyy * wxx)[:, None] * lerp(uvt_ep[mi, ss, yy >> 2, xx >> 2], uvt_w[mi, ss, yy, xx])
    uv = lerp(fuv_ep[mi, y >> 2, x >> 2], fuv_w[mi, y, x])
    k0, k1, wk = _nodes(tau, 24)
    planes = []
    for coord, arr in ((u64, fut), (v64, fvt)):
        a0, a1, wa = _axis(coord, 64)
        planes.append(sum((wt * wp)[:, None] * arr[mi, kk, aa] for kk, wt in ((k0, 1 - wk), (k1, wk))
                          for aa, wp in ((a0, 1 - wa), (a1, wa))))
    z = torch.cat([V, uv, planes[0], planes[1]], 1)
    if c["noise"]:
        z = z + _noise64(1, 1000, M * B) / 256.0
    z = torch.cat([z, _gamma(t)], 1)
    pred = torch.cat([_mlp(p[M * n_feat + i * n_mlp:M * n_feat + (i + 1) * n_mlp], z[i * B:(i + 1) * B], hid, _gelu, _same)
                      for i in range(M)])
    loss = ((pred - tgt[mi, f, y, x].double()) ** 2).mean()      # models of equal batches
    (M * loss).backward()
    with torch.no_grad():
        q = _adam64(p.detach(), p.grad, m.double(), v.double(), 1e-3)
        q[:M * n_feat].clamp_(0, 1)
        return [loss.detach().reshape(1), q]


def exact(case, seed):
    c = case
    if c["kind"] == "query":
        dt = "float16" if c["store"] == "f16" else "float32"
        m = I.random_model_torch(c["W"], c["H"], c["Gw"], c["Gh"], c["T"], seed=seed, device=DEV, grid_dtype=dt,
                                 mlp_dtype=dt)
        tex = _bc4_texels(m["bc4"], 8)
        q = I.uniform_queries_torch(c["n"], seed=seed + 1, device=DEV).double()
        return torch.cat([_decode64(m, tex, b[:, 0], b[:, 1], b[:, 2]) for b in torch.split(q, 1 << 20)])
    if c["kind"] == "pages":
        models, (mi, px, py, t, off), texels, pitch = _page_inputs(c, seed)
        out = torch.zeros((texels, 3), dtype=torch.float64, device=DEV)
        i = torch.arange(c["page"], device=DEV)
        for k, m in enumerate(models):
            mine = np.nonzero(np.asarray(mi) == k)[0]
            if not mine.size:
                continue
            tex = _bc4_texels(m["bc4"], 8)
            for b in np.array_split(mine, -(-mine.size * c["page"] ** 2 // (1 << 20))):
                col = lambda a: torch.from_numpy(np.asarray(a)[b]).to(DEV)[:, None, None]  # noqa: E731
                x, y = (col(px) * c["page"] + i[None, None, :]), (col(py) * c["page"] + i[None, :, None])
                x, y, tt = torch.broadcast_tensors((x.double() + 0.5) / m["W"], (y.double() + 0.5) / m["H"], col(t).double())
                at = (col(off) + i[None, :, None] * pitch + i[None, None, :]).reshape(-1)
                out[at] = _decode64(m, tex, x.reshape(-1), y.reshape(-1), tt.reshape(-1))
        return out
    if c["kind"] == "hybrid_query":
        m = _hybrid_numpy(c, seed, 0, c["W"], c["H"])
        d = _hybrid_maps(m, c["codec"])
        q = I.uniform_queries_torch(c["n"], seed=seed + 1, device=DEV).double()
        return torch.cat([_hybrid64(d, m, b[:, 0], b[:, 1], b[:, 2]) for b in torch.split(q, 1 << 18)])
    if c["kind"] == "hybrid_pages":
        t, off, pitch, texels = _hybrid_requests(c, seed)
        out = torch.zeros((texels, 3), dtype=torch.float64, device=DEV)
        R = c["page"] + 2 * c["border"]
        i = torch.arange(R, device=DEV)
        x = i - c["border"]
        x = torch.where(x < 0, -1 - x, torch.where(x >= 128, 255 - x, x))
        u = (x.double() + 0.5) / 128
        for k in range(c["models"]):
            m = _hybrid_numpy(c, seed, k)
            at = (int(off[k]) + i[:, None] * pitch + i[None, :]).reshape(-1)
            uu, vv = u[None, :].expand(R, R).reshape(-1), u[:, None].expand(R, R).reshape(-1)
            out[at] = _hybrid64(_hybrid_maps(m, c["codec"]), m, uu, vv, torch.full_like(uu, float(t)))
        return out
    if c["kind"] == "train":
        return _train64(c, seed)
    if c["kind"] == "hybrid_train":
        return _htrain64(c, seed)
    keys = I.lightmap_key_times(I.rng(6, I.P_MODEL, 1))
    return [[None, None, None, None, torch.from_numpy(np.asarray(_htrain_init(c, seed, i, keys, c["state"])["mlp"])).double()]
            for i in range(c["models"])]
