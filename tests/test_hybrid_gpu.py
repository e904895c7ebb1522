"""GPU parity of the hybrid-layout decode (Sec. 3.3, Eq. 4: F_uvt, F_uv, F_ut, F_vt,
gamma(t) into the GELU decoder) against the CPU oracle, through the C ABI.

The decoder output is linear, so a plain relative error is undefined where the output
crosses zero.  The statistic is |gpu - oracle| / max(|oracle|, rms), with rms the root mean
square of the oracle's outputs over the compared set: a relative error for outputs of
typical size and an error relative to the output scale near zero.  Bounds: 2e-3 on the
FP16 path, 1e-5 on the FP32 path (max over the compared set)."""
import numpy as np
import pytest

from oracle import ndgi_oracle as O
from paper_2604_12625_amd import inputs as I
from tests.gpu_util import torch_cuda

pytestmark = pytest.mark.gpu

TOL = {1: 2e-3, 0: 1e-5}


def scaled_err(gpu, ref):
    gpu = np.asarray(gpu, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    rms = np.sqrt(np.mean(ref[np.isfinite(ref)] ** 2))
    return np.abs(gpu - ref) / np.maximum(np.abs(ref), rms)


def assert_close(gpu, ref, tol, what=""):
    e = scaled_err(gpu, ref)
    worst = float(np.max(e)) if e.size else 0.0
    assert worst <= tol, f"{what}: max scaled err {worst:.3e} > {tol:.1e} (p99.9 {np.quantile(e, 0.999):.3e})"
    return worst


@pytest.fixture(scope="module")
def N():
    torch_cuda()
    from paper_2604_12625_amd import ndgi
    return ndgi


@pytest.fixture(scope="module")
def ctx(N):
    c = N.Context(0)
    yield c
    c.close()


def _dec(N, ctx, m, q, prec):
    import torch
    hm = N.HybridModel.from_numpy(m)
    out = ctx.hybrid_decode(hm, torch.from_numpy(q).cuda(), prec)
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


@pytest.mark.parametrize("profile", ["L", "M", "H", "M.64"])
@pytest.mark.parametrize("prec", [1, 0])
def test_hybrid_queries_match_oracle(N, ctx, profile, prec):
    m = I.random_hybrid_model(profile=profile, config=40)
    q = I.uniform_queries(4096 + 37, I.rng(40, I.P_QUERY))
    assert_close(_dec(N, ctx, m, q, prec), O.hybrid_decode(m, q), TOL[prec], f"{profile} prec {prec}")


@pytest.mark.parametrize("prec", [1, 0])
def test_hybrid_fp32_weights_no_keys_single_slice(N, ctx, prec):
    m = I.random_hybrid_model(192, 96, profile="M", slices=1, plane=(48, 96, 1), mlp_dtype=np.float32,
                              keys=False, config=41, uvt_side=(24, 16))
    q = I.uniform_queries(3000, I.rng(41, I.P_QUERY))
    assert_close(_dec(N, ctx, m, q, prec), O.hybrid_decode(m, q), TOL[prec], "S = 1, Tt = 1")
    m = I.random_hybrid_model(256, 128, profile="M.64", slices=5, plane=(256, 3, 7), mlp_dtype=np.float32,
                              keys=False, config=42, uvt_side=(256, 128))
    q = I.uniform_queries(3000, I.rng(42, I.P_QUERY))
    assert_close(_dec(N, ctx, m, q, prec), O.hybrid_decode(m, q), TOL[prec], "full-res F_uvt")


def test_hybrid_edges_clamp_time_and_nan(N, ctx):
    m = I.random_hybrid_model(profile="M", config=43)
    q = np.array([[-0.5, 0.5, 0.2], [1.7, 0.5, 0.2], [0.5, -3.0, 0.2], [0.5, 9.0, 0.2],
                  [0.3, 0.6, -0.5], [0.3, 0.6, 1.5], [0.3, 0.6, 0.0], [0.3, 0.6, 1.0],
                  [0.3, 0.6, float(m["keys"][3])], [0.3, 0.6, float(m["keys"][-1])],
                  [np.nan, 0.5, 0.5], [0.5, np.inf, 0.5], [0.5, 0.5, -np.inf]], dtype=np.float32)
    for prec in (1, 0):
        got = _dec(N, ctx, m, q, prec)
        ref = O.hybrid_decode(m, q)
        assert np.isnan(got[-3:]).all()
        assert_close(got[:-3], ref[:-3], TOL[prec], f"edges prec {prec}")


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 100_003])
def test_hybrid_ragged_counts(N, ctx, n):
    import torch
    m = I.random_hybrid_model(profile="M.64", config=44)
    q = I.uniform_queries(max(n, 1), I.rng(44, I.P_QUERY, n))[:n]
    hm = N.HybridModel.from_numpy(m)
    out = torch.full((n + 5, 3), -7.0, dtype=torch.float16, device="cuda")
    ctx.hybrid_decode(hm, torch.from_numpy(q).cuda(), 1, out=out[:n] if n else out[:0])
    torch.cuda.synchronize()
    o = out.float().cpu().numpy()
    np.testing.assert_array_equal(o[n:], -7.0)
    if n:
        sel = np.arange(n) if n < 5000 else np.random.default_rng(n).integers(0, n, 5000)
        assert_close(o[sel], O.hybrid_decode(m, q[sel]), TOL[1], f"n={n}")


def test_hybrid_argument_errors(N, ctx):
    import torch
    m = I.random_hybrid_model(profile="M", config=45)
    hm = N.HybridModel.from_numpy(m)
    q = torch.zeros((4, 3), dtype=torch.float32, device="cuda")
    for field, val in (("hidden", 32), ("Gu", 256), ("U", 0), ("S", 0), ("n_keys", 1), ("n_keys", 300),
                       ("W", 130), ("codec", 2), ("codec", -1), ("mlp_dtype", 7)):
        bad = N.HybridModel.from_numpy(m)
        setattr(bad.desc, field, val)
        with pytest.raises(N.NdgiError):
            ctx.hybrid_decode(bad, q, 1)
    with pytest.raises(N.NdgiError):
        ctx.hybrid_decode(hm, q, 5)
    assert ctx.hybrid_decode(hm, q[:0], 1).shape == (0, 3)


# ------------------------------------------------------------------------------ pages
def _hyb_vt(seed):
    """Eight per-tile models (all four profiles, mixed widths) plus two 256^2 maps; page
    requests over them, some invalid (model index or page out of range)."""
    models = [I.random_hybrid_model(profile=p, config=50 + seed, index=i, keys=(i % 3 != 0))
              for i, p in enumerate(["L", "M", "H", "M.64", "M", "L", "M.64", "H"])]
    models.append(I.random_hybrid_model(256, 256, profile="M", plane=(128, 128, 24), config=50 + seed, index=8,
                                        uvt_side=(64, 64)))
    models.append(I.random_hybrid_model(256, 256, profile="M.64", plane=(128, 128, 24), config=50 + seed,
                                        index=9, uvt_side=(64, 64)))
    g = np.random.default_rng(seed)
    reqs = []
    for r in range(40):
        mi = int(g.integers(0, len(models)))
        n = models[mi]["W"] // 128
        px, py = int(g.integers(0, n)), int(g.integers(0, n))
        reqs.append((mi, px, py, float(np.float32(g.random() * 1.2 - 0.1)), (r // 8) * 128 * 1024 + (r % 8) * 128))
    reqs[5] = (len(models) + 3, 0, 0, 0.5, reqs[5][4])       # model out of range
    reqs[11] = (1, 1, 0, 0.5, reqs[11][4])                   # page outside a 128^2 map
    reqs[17] = (8, 0, 2, 0.5, reqs[17][4])                   # page outside a 256^2 map
    return models, reqs


def _run_hpages(N, ctx, models, reqs, prec, graph=False, widths=0, border=0, rows=None):
    import torch
    hms = [N.HybridModel.from_numpy(m) for m in models]
    marr = N.models_array(hms)
    r = np.array(reqs, dtype=object)
    rq = N.page_requests(r[:, 0].astype(np.int32), r[:, 1].astype(np.int32), r[:, 2].astype(np.int32),
                         r[:, 3].astype(np.float32), r[:, 4].astype(np.int64))
    nreq = torch.tensor([len(reqs)], dtype=torch.int32, device="cuda")
    rows = rows or (len(reqs) + 7) // 8 * 128
    dt = torch.float16 if prec else torch.float32
    dst = torch.full((rows * 1024, 3), -7.0, dtype=dt, device="cuda")
    ctx.hybrid_decode_pages(marr, len(models), rq, nreq, len(reqs), 128, dst, 1024, prec, widths=widths,
                            border=border, graph=graph)
    torch.cuda.synchronize()
    return dst.float().cpu().numpy(), (hms, marr, rq, nreq, dst)


@pytest.mark.parametrize("prec", [1, 0])
def test_hybrid_pages_many_models_and_bad_requests(N, ctx, prec):
    models, reqs = _hyb_vt(3)
    out, _ = _run_hpages(N, ctx, models, reqs, prec)
    assert ctx.error_flags() & N.FLAG_BAD_PAGE_REQUEST
    ref = np.full(out.shape, -7.0)
    assert O.hybrid_decode_pages(models, reqs, 128, ref, 1024) == 3
    valid = ref[:, 0] != -7.0
    assert_close(out[valid], ref[valid], TOL[prec], "hybrid pages")
    np.testing.assert_array_equal(out[~valid], -7.0)


def test_hybrid_pages_width_mask(N, ctx):
    """Naming only width 16 skips and flags the requests of width-64 models; the rest
    decode as with both widths."""
    models, reqs = _hyb_vt(6)
    out, _ = _run_hpages(N, ctx, models, reqs, 1, widths=1)
    assert ctx.error_flags() & N.FLAG_BAD_PAGE_REQUEST
    narrow = [r if (0 <= r[0] < len(models) and models[r[0]]["hidden"] == 16) else (len(models), 0, 0, 0.0, r[4])
              for r in reqs]
    ref = np.full(out.shape, -7.0)
    O.hybrid_decode_pages(models, narrow, 128, ref, 1024)
    valid = ref[:, 0] != -7.0
    assert valid.any() and not valid.all()
    assert_close(out[valid], ref[valid], TOL[1], "width 16 only")
    np.testing.assert_array_equal(out[~valid], -7.0)
    with pytest.raises(N.NdgiError):
        _run_hpages(N, ctx, models, reqs, 1, widths=4)


def test_hybrid_pages_graph_replay_with_new_requests(N, ctx):
    models, reqs = _hyb_vt(4)
    reqs = [r for i, r in enumerate(reqs) if i not in (5, 11, 17)][:24]
    reqs = [(m, px, py, t, (r // 8) * 128 * 1024 + (r % 8) * 128) for r, (m, px, py, t, _) in enumerate(reqs)]
    out1, keep = _run_hpages(N, ctx, models, reqs, 1, graph=True)
    hms, marr, rq, nreq, dst = keep
    ref = np.full(out1.shape, -7.0)
    O.hybrid_decode_pages(models, reqs, 128, ref, 1024)
    v = ref[:, 0] != -7.0
    assert_close(out1[v], ref[v], TOL[1], "graph #1")
    reqs2 = [(m, px, py, float(np.float32((t + 0.37) % 1.0)), off) for (m, px, py, t, off) in reqs]
    r = np.array(reqs2, dtype=object)
    rq.copy_(N.page_requests(r[:, 0].astype(np.int32), r[:, 1].astype(np.int32), r[:, 2].astype(np.int32),
                             r[:, 3].astype(np.float32), r[:, 4].astype(np.int64)))
    nreq.fill_(16)
    import torch
    for _ in range(3):
        dst.fill_(-7.0)
        ctx.hybrid_decode_pages(marr, len(models), rq, nreq, len(reqs), 128, dst, 1024, 1, graph=True)
        torch.cuda.synchronize()
        out2 = dst.float().cpu().numpy()
        ref2 = np.full(out1.shape, -7.0)
        O.hybrid_decode_pages(models, reqs2[:16], 128, ref2, 1024)
        v = ref2[:, 0] != -7.0
        assert_close(out2[v], ref2[v], TOL[1], "graph replay")
        np.testing.assert_array_equal(out2[~v], -7.0)


def test_hybrid_pages_nan_time_and_page_size(N, ctx):
    import torch
    models, reqs = _hyb_vt(5)
    reqs = [(1, 0, 0, float("nan"), 0), (2, 0, 0, 0.25, 128)]
    out, _ = _run_hpages(N, ctx, models, reqs, 1)
    assert np.isnan(out.reshape(128, 1024, 3)[:, :128]).all()
    ref = np.full(out.shape, -7.0)
    O.hybrid_decode_pages(models, reqs[1:], 128, ref, 1024)
    v = ref[:, 0] != -7.0
    assert_close(out[v], ref[v], TOL[1], "page next to a NaN page")
    hm = N.HybridModel.from_numpy(models[0])
    marr = N.models_array([hm])
    rq = N.page_requests([0], [0], [0], [0.5], [0])
    nreq = torch.tensor([1], dtype=torch.int32, device="cuda")
    dst = torch.empty((128 * 128, 3), dtype=torch.float16, device="cuda")
    for page in (0, -32, 8192):
        with pytest.raises(N.NdgiError):
            ctx.hybrid_decode_pages(marr, 1, rq, nreq, 1, page, dst, 128, 1)
    with pytest.raises(N.NdgiError):     # border wider than the page
        ctx.hybrid_decode_pages(marr, 1, rq, nreq, 1, 8, dst, 128, 1, border=9)


def _bordered(reqs, border):
    """Requests re-addressed to non-overlapping (128 + 2 border)^2 regions in a 1024-wide
    destination; returns (requests, destination rows)."""
    R = 128 + 2 * border
    per = 1024 // R
    out = [(m, px, py, t, (r // per) * R * 1024 + (r % per) * R) for r, (m, px, py, t, _) in enumerate(reqs)]
    return out, (len(reqs) + per - 1) // per * R


@pytest.mark.parametrize("border", [4, 1, 32])
@pytest.mark.parametrize("prec", [1, 0])
def test_hybrid_pages_with_mirrored_border(N, ctx, border, prec):
    """Bordered regions (ragged sub-tiles, mirror addressing at map edges, neighbours inside
    the map) over per-tile models of both codecs and widths and two 256^2 maps."""
    models, reqs = _hyb_vt(6)
    models[2] = I.random_hybrid_model(profile="H", config=83, index=2, codec=1)
    models[3] = I.random_hybrid_model(profile="M.64", config=83, index=3, codec=1)
    reqs, rows = _bordered(reqs, border)
    out, _ = _run_hpages(N, ctx, models, reqs, prec, border=border, rows=rows)
    ref = np.full(out.shape, -7.0)
    assert O.hybrid_decode_pages(models, reqs, 128, ref, 1024, border=border) == 3
    assert ctx.error_flags() & N.FLAG_BAD_PAGE_REQUEST
    valid = ref[:, 0] != -7.0
    assert_close(out[valid], ref[valid], TOL[prec], f"border {border}")
    np.testing.assert_array_equal(out[~valid], -7.0)


def test_hybrid_pages_border_graph_and_errors(N, ctx):
    import torch
    ctx.error_flags()
    models, reqs = _hyb_vt(7)
    reqs = [r for i, r in enumerate(reqs) if i not in (5, 11, 17)][:20]
    reqs, rows = _bordered(reqs, 4)
    out, keep = _run_hpages(N, ctx, models, reqs, 1, graph=True, border=4, rows=rows)    # capture
    hms, marr, rq, nreq, dst = keep
    ref = np.full(out.shape, -7.0)
    O.hybrid_decode_pages(models, reqs, 128, ref, 1024, border=4)
    v = ref[:, 0] != -7.0
    for rep in range(3):
        if rep:              # replays into a cleared destination
            dst.fill_(-7.0)
            ctx.hybrid_decode_pages(marr, len(models), rq, nreq, len(reqs), 128, dst, 1024, 1, border=4, graph=True)
            torch.cuda.synchronize()
            out = dst.float().cpu().numpy()
        assert_close(out[v], ref[v], TOL[1], f"bordered graph, run {rep}")
        np.testing.assert_array_equal(out[~v], -7.0)
    for border, pitch in ((-1, 1024), (33, 1024), (4, 135), (32, 191)):
        with pytest.raises(N.NdgiError):
            ctx.hybrid_decode_pages(marr, len(models), rq, nreq, len(reqs), 128, dst, pitch, 1, border=border)
    ctx.hybrid_decode_pages(marr, len(models), rq, nreq, len(reqs), 128, dst, 136, 1, border=4)
    torch.cuda.synchronize()
    assert ctx.error_flags() == 0


@pytest.mark.parametrize("profile", ["M", "M.64"])
def test_hybrid_1024_map_of_tile_models_sampled(N, ctx, profile):
    """A 1024 x 1024 lightmap as 64 per-tile models of 128 x 128 texels (the paper's
    production setting), decoded at one t through the page decoder at its real size and
    checked on sampled texels."""
    import torch
    models = [I.random_hybrid_model(profile=profile, config=46, index=i) for i in range(64)]
    hms = [N.HybridModel.from_numpy(m) for m in models]
    marr = N.models_array(hms)
    t = 0.6180339
    idx = np.arange(64)
    rq = N.page_requests(idx.astype(np.int32), np.zeros(64, np.int32), np.zeros(64, np.int32),
                         np.full(64, t, np.float32), ((idx // 8) * 128 * 1024 + (idx % 8) * 128).astype(np.int64))
    nreq = torch.tensor([64], dtype=torch.int32, device="cuda")
    g = np.random.default_rng(47)
    sel = g.integers(0, 1024 * 1024, 4096)
    xs, ys = sel % 1024, sel // 1024
    tile = (ys // 128) * 8 + xs // 128
    ref = np.zeros((sel.size, 3))
    for k in np.unique(tile):
        s = tile == k
        ref[s] = O.hybrid_decode_f64(models[k], (xs[s] % 128 + 0.5) / 128, (ys[s] % 128 + 0.5) / 128,
                                     np.full(s.sum(), np.float64(np.float32(t))))
    for prec in (1, 0):
        dst = torch.empty((1024 * 1024, 3), dtype=torch.float16 if prec else torch.float32, device="cuda")
        ctx.hybrid_decode_pages(marr, 64, rq, nreq, 64, 128, dst, 1024, prec, widths=1 if profile == "M" else 2)
        got = dst[torch.from_numpy(sel).cuda()].float().cpu().numpy()
        assert_close(got, ref, TOL[prec], f"{profile} 1024^2 prec {prec}")
    assert ctx.error_flags() == 0


# ------------------------------------------------------------------------- BC7 modes 4-6
@pytest.mark.parametrize("profile", ["L", "M.64"])
@pytest.mark.parametrize("prec", [1, 0])
def test_bc7_queries_match_oracle(N, ctx, profile, prec):
    """F_uv and F_uvt as BC7 blocks (codec 1): random blocks of modes 4, 5 and 6 mixed, every
    index pattern, rotation, index selection and p-bit, decoded at random points."""
    m = I.random_hybrid_model(profile=profile, config=80, codec=1)
    assert m["fuv"].shape[-1] == 16
    q = I.uniform_queries(4096 + 91, I.rng(80, I.P_QUERY))
    assert_close(_dec(N, ctx, m, q, prec), O.hybrid_decode(m, q), TOL[prec], f"bc7 {profile} prec {prec}")


def test_bc7_full_resolution_uvt_and_edges(N, ctx):
    m = I.random_hybrid_model(256, 128, profile="M", slices=4, plane=(64, 32, 5), mlp_dtype=np.float32,
                              keys=False, config=81, uvt_side=(256, 128), codec=1)
    q = np.concatenate([I.uniform_queries(3000, I.rng(81, I.P_QUERY)),
                        np.array([[-0.5, 0.5, 0.2], [1.7, 1.5, 1.2], [0.0, 0.0, 0.0], [1.0, 1.0, 1.0]],
                                 dtype=np.float32)])
    for prec in (1, 0):
        assert_close(_dec(N, ctx, m, q, prec), O.hybrid_decode(m, q), TOL[prec], f"bc7 full-res prec {prec}")


@pytest.mark.parametrize("prec", [1, 0])
def test_bc7_pages_with_mixed_codecs(N, ctx, prec):
    """One page launch over BC4 and BC7 tile models: each request decodes with its model's
    block format."""
    models, reqs = _hyb_vt(5)
    rebuilt = []
    for i, m in enumerate(models):
        if i % 2:
            m = I.random_hybrid_model(m["W"], m["H"], profile=["L", "M", "H", "M.64", "M", "L", "M.64", "H", "M",
                                                               "M.64"][i], plane=(m["U"], m["V"], m["Tt"]),
                                      config=82, index=i, uvt_side=(m["Gu"], m["Gv"]), codec=1)
        rebuilt.append(m)
    out, _ = _run_hpages(N, ctx, rebuilt, reqs, prec)
    ref = np.full(out.shape, -7.0)
    assert O.hybrid_decode_pages(rebuilt, reqs, 128, ref, 1024) == 3
    valid = ref[:, 0] != -7.0
    assert_close(out[valid], ref[valid], TOL[prec], "bc7 pages")
    np.testing.assert_array_equal(out[~valid], -7.0)


def _bc7_all_texels(blocks):
    """Oracle decode of every texel of [n][16] BC7 blocks -> [n][16][4]."""
    n = blocks.shape[0]
    ys, xs = np.meshgrid(np.arange(4), np.arange(4), indexing="ij")
    b = np.repeat(blocks[:, None, :], 16, axis=1)
    return O.bc7_texels(b, np.broadcast_to(xs.ravel(), (n, 16)), np.broadcast_to(ys.ravel(), (n, 16)))


def test_bc7_block_decode_is_bit_exact(N):
    """The device BC7 texel decode, byte for byte: the hand-built golden blocks, 200,003
    random mode-6 blocks (every index pattern and p-bit) and 200,003 random blocks of modes
    4, 5 and 6 mixed (every rotation and index selection), against the oracle; a block of
    another mode decodes to 0."""
    import torch
    from tests.test_oracle_hybrid import _golden_bc7
    rows = _golden_bc7()
    gold = np.stack([b for b, _ in rows])
    got = N.bc7_decode_blocks(torch.from_numpy(gold).cuda()).cpu().numpy()
    for i, (_, want) in enumerate(rows):
        np.testing.assert_array_equal(got[i], want)
    blocks = I.random_bc7m6((200_003,), np.random.default_rng(84))
    got = N.bc7_decode_blocks(torch.from_numpy(blocks).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, _bc7_all_texels(blocks))
    mixed = I.random_bc7((200_003,), np.random.default_rng(85))
    mixed[:7, 0] = [0x00, 0x01, 0x02, 0x04, 0x08, 0x80, 0x00]     # modes 0-3 and 7, no mode
    got = N.bc7_decode_blocks(torch.from_numpy(mixed).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, _bc7_all_texels(mixed))
    np.testing.assert_array_equal(got[:7], 0)
    assert N.bc7_decode_blocks(torch.from_numpy(blocks[:0]).cuda()).shape == (0, 16, 4)
    with pytest.raises(N.NdgiError):   # misaligned source
        raw = torch.from_numpy(blocks[:5]).cuda().view(-1)
        N.bc7_decode_blocks(raw[8:8 + 64].view(4, 16))


@pytest.mark.parametrize("page,border", [(100, 0), (100, 7), (40, 32), (5, 5)])
def test_hybrid_pages_of_any_size(N, ctx, page, border):
    """Pages need not be multiples of 32: 100-texel pages of 200 x 300 maps (ragged
    sub-tiles), 40-texel pages with a 32-texel border, 5-texel pages."""
    import torch
    ctx.error_flags()   # clear what earlier tests left
    models = [I.random_hybrid_model(200, 300, profile=p, plane=(100, 150, 24), config=85, index=i,
                                    uvt_side=(48, 64), codec=i % 2) for i, p in enumerate(["M", "M.64", "L", "H"])]
    R = page + 2 * border
    g = np.random.default_rng(page + border)
    reqs = []
    for r in range(12):
        mi = int(g.integers(0, 4))
        px, py = int(g.integers(0, 200 // page)), int(g.integers(0, 300 // page))
        reqs.append((mi, px, py, float(np.float32(g.random())), (r // 4) * R * 1024 + (r % 4) * R))
    rows = 3 * R
    hms = [N.HybridModel.from_numpy(m) for m in models]
    marr = N.models_array(hms)
    r = np.array(reqs, dtype=object)
    rq = N.page_requests(r[:, 0].astype(np.int32), r[:, 1].astype(np.int32), r[:, 2].astype(np.int32),
                         r[:, 3].astype(np.float32), r[:, 4].astype(np.int64))
    nreq = torch.tensor([len(reqs)], dtype=torch.int32, device="cuda")
    dst = torch.full((rows * 1024, 3), -7.0, dtype=torch.float16, device="cuda")
    ctx.hybrid_decode_pages(marr, 4, rq, nreq, len(reqs), page, dst, 1024, 1, border=border)
    torch.cuda.synchronize()
    out = dst.float().cpu().numpy()
    assert ctx.error_flags() == 0
    ref = np.full(out.shape, -7.0)
    assert O.hybrid_decode_pages(models, reqs, page, ref, 1024, border=border) == 0
    valid = ref[:, 0] != -7.0
    assert valid.sum() == len(reqs) * R * R
    assert_close(out[valid], ref[valid], TOL[1], f"page {page} border {border}")
    np.testing.assert_array_equal(out[~valid], -7.0)


@pytest.mark.parametrize("profile", ["M", "M.64"])
@pytest.mark.parametrize("dtype", ["float16", "float32"])
def test_decoder_weights_at_any_alignment(N, ctx, profile, dtype):
    """Decoder vectors that start one element past an aligned address (quads of weights then
    load one by one) give the bits of the aligned ones, for queries and pages."""
    import torch
    m = I.random_hybrid_model(64, 64, profile=profile, plane=(32, 32, 8), config=91, uvt_side=(16, 16))
    hm = N.HybridModel.from_numpy(m)
    w = torch.from_numpy(m["mlp"]).to("cuda", getattr(torch, dtype))
    room = torch.zeros(w.numel() + 1, dtype=w.dtype, device="cuda")
    room[1:] = w
    d = hm.desc
    models = [N.HybridModel(d.W, d.H, d.Gu, d.Gv, d.S, d.U, d.V, d.Tt, d.hidden, *hm.arrays[:5], v)
              for v in (w, room[1:])]
    assert models[1].desc.mlp % (4 * w.element_size())
    q = torch.from_numpy(np.random.default_rng(92).random((300, 3)).astype(np.float32)).cuda()
    rq = N.page_requests(np.zeros(1, np.int32), np.zeros(1, np.int32), np.zeros(1, np.int32),
                         np.full(1, 0.3, np.float32), np.zeros(1, np.int64))
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    for prec in (1, 0):
        got = []
        for hm in models:
            dst = torch.zeros((64 * 64, 3), dtype=(torch.float16 if prec else torch.float32), device="cuda")
            ctx.hybrid_decode_pages(N.models_array([hm]), 1, rq, one, 1, 64, dst, 64, prec)
            got.append((ctx.hybrid_decode(hm, q, prec).cpu().numpy(), dst.cpu().numpy()))
        for a, b in zip(*got):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("page,border", [(64, 4), (34, 0), (35, 1)])
def test_pages_of_every_block_mode(N, ctx, page, border):
    """Random BC7 blocks of modes 4, 5 and 6 (every rotation and index selection) and of modes
    that decode to 0, in the sub-tiles' staged texels and in F_uvt: pages against the oracle."""
    import torch
    g = np.random.default_rng(93)
    m = I.random_hybrid_model(72, 140, profile="M", plane=(36, 70, 6), config=94, uvt_side=(72, 140), codec=1)
    for k in ("fuv", "fuvt"):
        b = g.integers(0, 256, m[k].shape, dtype=np.uint8)
        mode = g.integers(0, 8, b.shape[:-1])
        first = b[..., 0]
        for i, (keep, bit) in enumerate([(0xE0, 0x10), (0xC0, 0x20), (0x80, 0x40)]):
            sel = (mode < 7) & (mode % 3 == i)
            first[sel] = (first[sel] & keep) | bit
        m[k] = b
    R = page + 2 * border
    reqs = [(0, px, py, float(np.float32(g.random())), (py * 8 + px) * R) for px in range(72 // page) for py in range(140 // page)]
    r = np.array(reqs, dtype=object)
    rq = N.page_requests(r[:, 0].astype(np.int32), r[:, 1].astype(np.int32), r[:, 2].astype(np.int32),
                         r[:, 3].astype(np.float32), r[:, 4].astype(np.int64))
    nreq = torch.tensor([len(reqs)], dtype=torch.int32, device="cuda")
    pitch = 64 * R
    dst = torch.full((R * pitch, 3), -7.0, dtype=torch.float32, device="cuda")
    ctx.hybrid_decode_pages(N.models_array([N.HybridModel.from_numpy(m)]), 1, rq, nreq, len(reqs), page, dst, pitch, 0,
                            border=border)
    out = dst.cpu().numpy()
    ref = np.full(out.shape, -7.0)
    assert O.hybrid_decode_pages([m], reqs, page, ref, pitch, border=border) == 0
    valid = ref[:, 0] != -7.0
    assert valid.sum() == len(reqs) * R * R
    assert_close(out[valid], ref[valid], TOL[0], f"page {page} border {border}")
    np.testing.assert_array_equal(out[~valid], -7.0)
