"""GPU parity of the hybrid-layout training path (ndgi_hybrid_train_step, ndgi_hybrid_export,
the target preprocessing) against the CPU oracle, through the C ABI.

Bounds: forward outputs and the loss within 1e-5 relative (FP32 on the GPU against FP64);
gradients within 1e-4 relative plus 1e-6 of the array's largest entry (FP32 atomics and
wave reductions reorder the sums); export bytes bit-exact."""
import numpy as np
import pytest

from oracle import ndgi_oracle as O
from paper_2604_12625_amd import inputs as I
from tests.gpu_util import torch_cuda
from tests.test_oracle_hybrid import tiny_hybrid_state

pytestmark = pytest.mark.gpu


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


def _state(hidden, seed, frames=3, keys=True, on_grid=False, bigger=False, codec=0):
    st = tiny_hybrid_state(hidden, seed=seed, frames=frames, keys=keys, on_grid=on_grid)
    if bigger:   # a 64 x 48 map, F_uvt 16 x 12 x 5, planes 32 x 4 and 48 x 4
        g = np.random.default_rng(seed + 100)
        d = dict(st["dims"], W=64, H=48, Gu=16, Gv=12, S=5, U=32, V=48, Tt=4)
        st = dict(dims=d)
        st["fuv_ep"] = g.uniform(0, 1, (12, 16, 4, 2))
        st["fuv_w"] = g.uniform(0, 1, (48, 64, 4))
        st["fuvt_ep"] = g.uniform(0, 1, (5, 3, 4, 4, 2))
        st["fuvt_w"] = g.uniform(0, 1, (5, 12, 16, 4))
        st["fut"] = g.uniform(0, 1, (4, 32, 2))
        st["fvt"] = g.uniform(0, 1, (4, 48, 2))
        st["mlp"] = I.hybrid_mlp(hidden, np.float64, g)
    if codec == 1:   # BC7: one weight per texel
        g = np.random.default_rng(seed + 200)
        st["dims"] = dict(st["dims"], codec=1)
        st["fuv_w"] = g.uniform(0, 1, st["fuv_w"].shape[:-1])
        st["fuvt_w"] = g.uniform(0, 1, st["fuvt_w"].shape[:-1])
    # the GPU holds float32 masters: the oracle reads the same values
    for k in O.HYB_KEYS:
        st[k] = np.asarray(st[k], dtype=np.float32).astype(np.float64)
    return st


def _samples(st, n, seed):
    g = np.random.default_rng(seed)
    d = st["dims"]
    x, y, f = g.integers(0, d["W"], n), g.integers(0, d["H"], n), g.integers(0, d["frames"], n)
    tgt = g.normal(0.5, 0.5, (d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    return x, y, f, tgt


def _dev(N, x, y, f, tgt):
    import torch
    smp = torch.from_numpy(I.pack_samples(x, y, f).view(np.int32)).cuda()
    return smp, torch.from_numpy(tgt).cuda()


def _close(got, ref, rel, what, floor=1e-6):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    tol = rel * np.abs(ref) + floor * max(float(np.max(np.abs(ref))), 1e-30)
    bad = np.abs(got - ref) > tol
    assert not bad.any(), f"{what}: {int(bad.sum())} of {bad.size} off, worst {np.max(np.abs(got - ref) - tol):.3e}"


@pytest.mark.parametrize("hidden", [16, 64])
@pytest.mark.parametrize("flags", [0, 2, 1 | 2, 1 | 4, 8 | 2, 8 | 4])
@pytest.mark.parametrize("bigger", [False, True])
def test_hybrid_loss_grad_and_forward_match_oracle(N, ctx, hidden, flags, bigger):
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(hidden, seed=hidden + flags, bigger=bigger)
    x, y, f, tgt = _samples(st, 700, seed=7 + flags)
    smp, tg = _dev(N, x, y, f, tgt)
    tr = HybridTrainer(ctx, st, seed=11)
    pred = tr.forward(smp, flags).cpu().numpy()
    ref_pred = O.hybrid_train_forward(st, x, y, f, flags, seed=11, step=0)
    _close(pred, ref_pred, 1e-5, "forward", floor=1e-6)
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, flags).item())
    ref_loss, ref_g = O.hybrid_train_grads(st, x, y, f, tgt[f, y, x], flags, seed=11, step=0)
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    got = tr.split(tr.grads)
    for k in O.HYB_KEYS:
        _close(got[k].cpu().numpy(), ref_g[k], 1e-4, k)


def test_hybrid_adam_steps_match_oracle(N, ctx):
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(16, seed=3)
    ref = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in st.items()}
    opt = dict(step=0, lr_feat=1e-2, lr_mlp=1e-3, m={k: 0.0 for k in O.HYB_KEYS}, v={k: 0.0 for k in O.HYB_KEYS})
    tr = HybridTrainer(ctx, st, lr_feat=1e-2, lr_mlp=1e-3, seed=5)
    flags = O.HT_NOISE            # the paper's phase 1: continuous endpoints and weights, noise
    for it in range(3):
        x, y, f, tgt = _samples(st, 500, seed=20 + it)
        smp, tg = _dev(N, x, y, f, tgt)
        loss = float(tr.step(smp, tg, flags).item())
        ref_loss = O.hybrid_train_step(ref, opt, x, y, f, tgt[f, y, x], flags, seed=5)
        assert abs(loss - ref_loss) <= 1e-4 * abs(ref_loss), (it, loss, ref_loss)
    assert tr.state.step == 3
    got = tr.split(tr.params)
    for k in O.HYB_KEYS:
        g = got[k].cpu().numpy().astype(np.float64)
        # no quantisation in these steps; Adam turns FP32 noise on a cancelling gradient sum
        # into a fraction of lr, hence the lr-scaled absolute floor (as for the other layout)
        diff = np.abs(g - ref[k])
        tol = 1e-4 * np.abs(ref[k]) + 3e-3 * (1e-2 if k != "mlp" else 1e-3)
        assert not (diff > tol).any(), (k, int((diff > tol).sum()), float(diff.max()))


def test_hybrid_export_is_exact_and_decodes_to_the_simulated_forward(N, ctx):
    import torch
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(64, seed=8, bigger=True)
    tr = HybridTrainer(ctx, st)
    hm = tr.export(N.DTYPE_F32)
    ref = O.hybrid_export(st)
    for k in ("fuv", "fuvt", "fut", "fvt"):
        np.testing.assert_array_equal(getattr(hm, "arrays")[("fuv", "fuvt", "fut", "fvt").index(k)].cpu().numpy(),
                                      ref[k], err_msg=k)
    d = st["dims"]
    g = np.random.default_rng(9)
    n = 3000
    x, y, f = g.integers(0, d["W"], n), g.integers(0, d["H"], n), g.integers(0, d["frames"], n)
    fwd = O.hybrid_train_forward(st, x, y, f, 1 | 4)
    t = np.asarray(d["keys"], dtype=np.float32)[f]
    q = np.stack([(x + 0.5) / d["W"], (y + 0.5) / d["H"], t], 1).astype(np.float32)
    out = ctx.hybrid_decode(hm, torch.from_numpy(q).cuda(), N.PREC_F32).cpu().numpy()
    rms = np.sqrt(np.mean(fwd ** 2))
    assert np.max(np.abs(out - fwd) / np.maximum(np.abs(fwd), rms)) <= 1e-5


def test_target_normalisation_and_restore(N, ctx):
    import torch
    from paper_2604_12625_amd.train import hybrid_normalize_target, hybrid_restore
    g = np.random.default_rng(12)
    tgt = g.uniform(0.01, 5.0, (4, 40, 24, 3)).astype(np.float16)
    out, means = hybrid_normalize_target(ctx, torch.from_numpy(tgt.view(np.int16)).cuda(), 2.2)
    ref, ref_means = O.hybrid_normalise_target(tgt.astype(np.float64), 2.2)
    _close(out.cpu().numpy(), ref, 1e-5, "normalised target")
    _close(means.cpu().numpy(), ref_means, 1e-6, "means")
    back = hybrid_restore(ctx, out[2].reshape(-1, 3), means[2], 2.2).cpu().numpy()
    _close(back, O.hybrid_restore(ref[2].reshape(-1, 3), ref_means[2], 2.2), 1e-5, "restore")
    _close(back, tgt[2].reshape(-1, 3).astype(np.float64), 1e-5, "round trip")


@pytest.mark.parametrize("hidden", [16, 64])
def test_many_models_in_one_launch(N, ctx, hidden):
    """Three models trained together: each model's gradients are those of its own loss (the
    mean over its own samples), and the launch reports the mean of the models' losses."""
    from paper_2604_12625_amd.train import HybridTrainer
    M, Bm = 3, 128
    sts = [_state(hidden, seed=40 + i) for i in range(M)]
    for st in sts[1:]:
        st["dims"] = sts[0]["dims"]          # models trained together share sizes and key times
    g = np.random.default_rng(41)
    d = sts[0]["dims"]
    xs, ys, fs = (g.integers(0, d["W"], M * Bm), g.integers(0, d["H"], M * Bm), g.integers(0, d["frames"], M * Bm))
    tgt = g.normal(0.5, 0.5, (M, d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    smp, tg = _dev(N, xs, ys, fs, tgt)
    flags = 1 | 2
    tr = HybridTrainer(ctx, sts, seed=13, per_model=Bm)
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, flags).item())
    ref_loss = 0.0
    for m in range(M):
        sl = slice(m * Bm, (m + 1) * Bm)
        lm, gm = O.hybrid_train_grads(sts[m], xs[sl], ys[sl], fs[sl], tgt[m][fs[sl], ys[sl], xs[sl]], flags, seed=13,
                                      step=0, s_offset=m * Bm)
        ref_loss += lm / M
        got = tr.split(tr.grads, m)
        for k in O.HYB_KEYS:
            _close(got[k].cpu().numpy(), gm[k], 1e-4, f"model {m} {k}")
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    # a bad per-model count is rejected
    tr2 = HybridTrainer(ctx, sts, seed=13, per_model=100)
    with pytest.raises(N.NdgiError):
        tr2.loss_grad(smp, tg, flags)


# ------------------------------------------------------------------------- BC7 mode 6
@pytest.mark.parametrize("hidden", [16, 64])
@pytest.mark.parametrize("flags", [0, 2, 1 | 2, 1 | 4])
def test_bc7_loss_grad_and_forward_match_oracle(N, ctx, hidden, flags):
    """The BC7 simulation (one weight per texel shared by the 4 channels, Eq. 6): forward,
    loss and every gradient, including the shared weights' channel sums."""
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(hidden, seed=60 + hidden + flags, bigger=True, codec=1)
    x, y, f, tgt = _samples(st, 900, seed=61 + flags)
    smp, tg = _dev(N, x, y, f, tgt)
    tr = HybridTrainer(ctx, st, seed=17)
    assert tr.split(tr.params)["fuv_w"].shape == (48, 64)
    pred = tr.forward(smp, flags).cpu().numpy()
    _close(pred, O.hybrid_train_forward(st, x, y, f, flags, seed=17, step=0), 1e-5, "forward")
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, flags).item())
    ref_loss, ref_g = O.hybrid_train_grads(st, x, y, f, tgt[f, y, x], flags, seed=17, step=0)
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    got = tr.split(tr.grads)
    for k in O.HYB_KEYS:
        _close(got[k].cpu().numpy(), ref_g[k], 1e-4, k)


def test_bc7_adam_steps_match_oracle(N, ctx):
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(16, seed=63, codec=1)
    ref = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in st.items()}
    opt = dict(step=0, lr_feat=1e-2, lr_mlp=1e-3, m={k: 0.0 for k in O.HYB_KEYS}, v={k: 0.0 for k in O.HYB_KEYS})
    tr = HybridTrainer(ctx, st, lr_feat=1e-2, lr_mlp=1e-3, seed=6)
    for it in range(3):
        x, y, f, tgt = _samples(st, 500, seed=64 + it)
        smp, tg = _dev(N, x, y, f, tgt)
        loss = float(tr.step(smp, tg, O.HT_NOISE).item())
        ref_loss = O.hybrid_train_step(ref, opt, x, y, f, tgt[f, y, x], O.HT_NOISE, seed=6)
        assert abs(loss - ref_loss) <= 1e-4 * abs(ref_loss), (it, loss, ref_loss)
    got = tr.split(tr.params)
    for k in O.HYB_KEYS:
        diff = np.abs(got[k].cpu().numpy().astype(np.float64) - ref[k])
        tol = 1e-4 * np.abs(ref[k]) + 3e-3 * (1e-2 if k != "mlp" else 1e-3)
        assert not (diff > tol).any(), (k, int((diff > tol).sum()), float(diff.max()))


@pytest.mark.parametrize("on_grid", [False, True])
def test_bc7_export_is_exact_and_decodes_to_the_simulated_forward(N, ctx, on_grid):
    """Mode-6 blocks bit-identical to the oracle's encoder (p-bits, anchor swaps) and their
    decode at the training samples equal to the simulated forward."""
    import torch
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(64, seed=65, bigger=True, codec=1)
    if on_grid:   # weights at index boundaries 1/30 + J/15 and endpoints on the 8-bit grid
        g = np.random.default_rng(66)
        for k in ("fuv_w", "fuvt_w"):
            st[k] = np.clip(g.integers(0, 16, st[k].shape) / 15.0 + g.choice([-1, 0, 1], st[k].shape) / 30.0, 0, 1)
            st[k] = st[k].astype(np.float32).astype(np.float64)
        for k in ("fuv_ep", "fuvt_ep"):
            st[k] = (g.integers(0, 256, st[k].shape) / 255.0).astype(np.float32).astype(np.float64)
    tr = HybridTrainer(ctx, st)
    hm = tr.export(N.DTYPE_F32)
    ref = O.hybrid_export(st)
    for i, k in enumerate(("fuv", "fuvt", "fut", "fvt")):
        np.testing.assert_array_equal(hm.arrays[i].cpu().numpy(), ref[k], err_msg=k)
    assert hm.desc.codec == 1
    d = st["dims"]
    g = np.random.default_rng(67)
    n = 3000
    x, y, f = g.integers(0, d["W"], n), g.integers(0, d["H"], n), g.integers(0, d["frames"], n)
    fwd = O.hybrid_train_forward(st, x, y, f, 1 | 4)
    t = np.asarray(d["keys"], dtype=np.float32)[f]
    q = np.stack([(x + 0.5) / d["W"], (y + 0.5) / d["H"], t], 1).astype(np.float32)
    out = ctx.hybrid_decode(hm, torch.from_numpy(q).cuda(), N.PREC_F32).cpu().numpy()
    rms = np.sqrt(np.mean(fwd ** 2))
    assert np.max(np.abs(out - fwd) / np.maximum(np.abs(fwd), rms)) <= 1e-5


def test_bc7_many_models_in_one_launch(N, ctx):
    from paper_2604_12625_amd.train import HybridTrainer
    M, Bm = 2, 192
    sts = [_state(16, seed=70 + i, codec=1) for i in range(M)]
    for st in sts[1:]:
        st["dims"] = sts[0]["dims"]
    g = np.random.default_rng(71)
    d = sts[0]["dims"]
    xs, ys, fs = (g.integers(0, d["W"], M * Bm), g.integers(0, d["H"], M * Bm), g.integers(0, d["frames"], M * Bm))
    tgt = g.normal(0.5, 0.5, (M, d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    smp, tg = _dev(N, xs, ys, fs, tgt)
    tr = HybridTrainer(ctx, sts, seed=19, per_model=Bm)
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, 1 | 2).item())
    ref_loss = 0.0
    for m in range(M):
        sl = slice(m * Bm, (m + 1) * Bm)
        lm, gm = O.hybrid_train_grads(sts[m], xs[sl], ys[sl], fs[sl], tgt[m][fs[sl], ys[sl], xs[sl]], 1 | 2, seed=19,
                                      step=0, s_offset=m * Bm)
        ref_loss += lm / M
        got = tr.split(tr.grads, m)
        for k in O.HYB_KEYS:
            _close(got[k].cpu().numpy(), gm[k], 1e-4, f"model {m} {k}")
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    hm = tr.export(N.DTYPE_F16, model=1)
    np.testing.assert_array_equal(hm.arrays[0].cpu().numpy(), O.hybrid_export(sts[1])["fuv"])


@pytest.mark.parametrize("codec", [0, 1])
def test_large_single_model_batch_matches_oracle(N, ctx, codec):
    """A batch large enough for four-wave workgroups whose F_uvt endpoint and plane
    gradients are summed in LDS per chunk (20000 samples: a partial last chunk)."""
    from paper_2604_12625_amd.train import HybridTrainer
    st = _state(16, seed=90 + codec, codec=codec)
    x, y, f, tgt = _samples(st, 20000, seed=91)
    smp, tg = _dev(N, x, y, f, tgt)
    tr = HybridTrainer(ctx, st, seed=23)
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, 1 | 2).item())
    ref_loss, ref_g = O.hybrid_train_grads(st, x, y, f, tgt[f, y, x], 1 | 2, seed=23, step=0)
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    got = tr.split(tr.grads)
    for k in O.HYB_KEYS:
        _close(got[k].cpu().numpy(), ref_g[k], 1e-4, k)


@pytest.mark.parametrize("codec", [0, 1])
def test_production_size_multi_model_batch_matches_oracle(N, ctx, codec):
    """Four tile models x 4096 samples (the map workload's per-model batch): four-wave
    workgroups over chunks of one model's samples with the F_uvt endpoint and plane
    gradients summed in LDS, several chunks per model; the paper's phase-1 flags (noise on the
    continuous endpoint / weight maps)."""
    from paper_2604_12625_amd.train import HybridTrainer
    M, Bm = 4, 4096
    sts = [_state(16, seed=120 + i, bigger=True, codec=codec) for i in range(M)]
    for st in sts[1:]:
        st["dims"] = sts[0]["dims"]
    g = np.random.default_rng(121)
    d = sts[0]["dims"]
    xs, ys, fs = (g.integers(0, d["W"], M * Bm), g.integers(0, d["H"], M * Bm), g.integers(0, d["frames"], M * Bm))
    tgt = g.normal(0.5, 0.5, (M, d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    smp, tg = _dev(N, xs, ys, fs, tgt)
    tr = HybridTrainer(ctx, sts, seed=29, per_model=Bm)
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, N.HTRAIN_NOISE).item())
    ref_loss = 0.0
    for m in range(M):
        sl = slice(m * Bm, (m + 1) * Bm)
        lm, gm = O.hybrid_train_grads(sts[m], xs[sl], ys[sl], fs[sl], tgt[m][fs[sl], ys[sl], xs[sl]], O.HT_NOISE,
                                      seed=29, step=0, s_offset=m * Bm)
        ref_loss += lm / M
        got = tr.split(tr.grads, m)
        for k in O.HYB_KEYS:
            _close(got[k].cpu().numpy(), gm[k], 1e-4, f"model {m} {k}")
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)


@pytest.mark.parametrize("codec,sizes", [
    (1, (100, 60, 36, 20, 5, 37, 53, 7)),    # F_uvt's endpoints, weights and the planes summed in LDS
    (0, (100, 60, 36, 20, 5, 37, 53, 7)),    # four weights a texel: endpoints and planes only
    (1, (92, 68, 64, 64, 5, 31, 5, 2)),      # one weight a texel, which no longer fit
    (1, (92, 68, 64, 64, 9, 92, 68, 3)),     # the endpoints no longer fit either
])
def test_every_gradient_sum_at_ragged_sizes_matches_oracle(N, ctx, codec, sizes):
    """Grids, planes and maps whose sizes do not divide each other (every interpolation weight
    a different one), at both sides of the sizes up to which gradients are summed in LDS; a
    partial last chunk.  Tolerances as for the other batches of this size."""
    from paper_2604_12625_amd.train import HybridTrainer
    W, H, Gu, Gv, S, U, V, Tt = sizes
    st = _state(16, seed=170 + codec, frames=6, codec=codec)
    g = np.random.default_rng(171)
    f32 = lambda *shape: g.uniform(0, 1, shape).astype(np.float32).astype(np.float64)
    st["dims"] = dict(st["dims"], W=W, H=H, Gu=Gu, Gv=Gv, S=S, U=U, V=V, Tt=Tt)
    cw = () if codec else (4,)
    st.update(fuv_ep=f32(H // 4, W // 4, 4, 2), fuv_w=f32(H, W, *cw), fuvt_ep=f32(S, Gv // 4, Gu // 4, 4, 2),
              fuvt_w=f32(S, Gv, Gu, *cw), fut=f32(Tt, U, 2), fvt=f32(Tt, V, 2))
    x, y, f, tgt = _samples(st, 16700, seed=172)
    smp, tg = _dev(N, x, y, f, tgt)
    tr = HybridTrainer(ctx, st, seed=31)
    pred = tr.forward(smp, 0).cpu().numpy()
    _close(pred, O.hybrid_train_forward(st, x, y, f, 0, seed=31, step=0), 1e-5, "forward")
    tr.zero_grad()
    loss = float(tr.loss_grad(smp, tg, 0).item())
    ref_loss, ref_g = O.hybrid_train_grads(st, x, y, f, tgt[f, y, x], 0, seed=31, step=0)
    assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss), (loss, ref_loss)
    got = tr.split(tr.grads)
    for k in O.HYB_KEYS:
        _close(got[k].cpu().numpy(), ref_g[k], 1e-4, k)


def test_short_chunks_keep_their_speed(N, ctx):
    """100 BC7 M-profile models x 1920 samples (chunks of 640) take little longer than 64 x 4096 (chunks of
    1024): 1.2 times, and 1.7 where the short chunks also summed F_uvt's weights in LDS."""
    import torch
    from paper_2604_12625_amd.train import HybridTrainer
    keys = I.lightmap_key_times(I.rng(6, I.P_MODEL, 1))
    st = I.hybrid_train_init(128, 128, "M", len(keys), keys, I.rng(7, I.P_INIT, 1), codec=1)
    best = {}
    for models, per in ((100, 1920), (64, 4096)):
        tr = HybridTrainer(ctx, [st] * models, seed=1, per_model=per)
        smp = I.train_samples_torch(models * per, 128, 128, len(keys), seed=2, device="cuda")
        tgt = torch.ones((models, len(keys), 128, 128, 3), device="cuda")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                tr.step(smp, tgt, N.HTRAIN_NOISE)
            b.record()
            b.synchronize()
            best[per] = min(best.get(per, 1e9), a.elapsed_time(b))
    assert best[1920] <= 1.4 * best[4096], best


@pytest.mark.parametrize("hidden", [16, 64])
def test_rounds_of_a_chunk_equal_separate_calls(N, ctx, hidden):
    """Eight models x 32768 samples run several 256-sample rounds per chunk (four on a
    256-CU GPU), where h = 16 carries the decoder's weight-gradient sums across the rounds
    in its MFMA chains; the same samples as four calls of each model's quarters (one round
    per chunk) must give four times the gradients and the loss (each call normalises by its
    own per-model count).  No noise, so that the draws do not depend on a sample's index."""
    from paper_2604_12625_amd.train import HybridTrainer
    M, Bm = 8, 32768
    sts = [_state(hidden, seed=140 + i, bigger=True, codec=1) for i in range(M)]
    for st in sts[1:]:
        st["dims"] = sts[0]["dims"]
    g = np.random.default_rng(141)
    d = sts[0]["dims"]
    xs, ys, fs = (g.integers(0, d["W"], M * Bm), g.integers(0, d["H"], M * Bm), g.integers(0, d["frames"], M * Bm))
    tgt = g.normal(0.5, 0.5, (M, d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    smp, tg = _dev(N, xs, ys, fs, tgt)
    one = HybridTrainer(ctx, sts, seed=3, per_model=Bm)
    one.zero_grad()
    loss_one = float(one.loss_grad(smp, tg, 0).item())
    q = Bm // 4
    four = HybridTrainer(ctx, sts, seed=3, per_model=q)
    four.zero_grad()
    loss_four = 0.0
    for k in range(4):
        idx = np.concatenate([np.arange(m * Bm + k * q, m * Bm + (k + 1) * q) for m in range(M)])
        sk, _ = _dev(N, xs[idx], ys[idx], fs[idx], tgt)
        loss_four += float(four.loss_grad(sk, tg, 0).item())
    assert abs(loss_four - 4 * loss_one) <= 1e-5 * abs(loss_four), (loss_four, loss_one)
    _close(four.grads.cpu().numpy(), 4.0 * one.grads.cpu().numpy(), 1e-4, "gradients")


def test_identical_models_trained_together_equal_one_trained_alone(N, ctx):
    """Per-model normalisation: M copies of a model with the same samples, trained together,
    stay equal step for step to the model trained alone (Adam is not invariant to a common
    gradient scale, so a batch-wide mean would drift)."""
    from paper_2604_12625_amd.train import HybridTrainer
    M, Bm = 4, 1024
    st = _state(16, seed=130, bigger=True)
    d = st["dims"]
    alone = HybridTrainer(ctx, st, lr_feat=1e-2, lr_mlp=1e-3, seed=31)
    many = HybridTrainer(ctx, [st] * M, lr_feat=1e-2, lr_mlp=1e-3, seed=31, per_model=Bm)
    g = np.random.default_rng(131)
    tgt = g.normal(0.5, 0.5, (d["frames"], d["H"], d["W"], 3)).astype(np.float32)
    for it in range(3):
        x, y, f = g.integers(0, d["W"], Bm), g.integers(0, d["H"], Bm), g.integers(0, d["frames"], Bm)
        smp, tg = _dev(N, x, y, f, tgt)
        smp_m, tg_m = _dev(N, np.tile(x, M), np.tile(y, M), np.tile(f, M), np.stack([tgt] * M))
        la = float(alone.step(smp, tg, 0).item())
        lm = float(many.step(smp_m, tg_m, 0).item())
        assert abs(la - lm) <= 1e-6 * abs(la), (it, la, lm)
    pa = alone.split(alone.params)
    for m in range(M):
        pm = many.split(many.params, m)
        for k in O.HYB_KEYS:
            a, b = pa[k].cpu().numpy(), pm[k].cpu().numpy()
            # same samples, same arithmetic; only the order of float atomics differs
            assert np.max(np.abs(a - b)) <= 1e-5 * max(float(np.max(np.abs(a))), 1e-30) + 1e-7, (m, k)


# ------------------------------------------------------------ export path and the ablation arm
def _blocks_bc4(seed):
    g = np.random.default_rng(seed)
    dec = g.integers(0, 256, (64, 8)).astype(np.uint8)
    dec[:32, 0] = np.maximum(dec[:32, 0], dec[:32, 1] + 1)
    dec[32:, 0] = np.minimum(dec[32:, 0], dec[32:, 1])
    smooth = np.clip(np.round(np.linspace(g.uniform(0, 120, (48, 1)), g.uniform(130, 255, (48, 1)), 16, axis=1)[..., 0]
                              + g.normal(0, 4, (48, 16))), 0, 255)
    return np.concatenate([g.integers(0, 256, (48, 16)), g.integers(100, 108, (16, 16)),
                           O.bc4_decode_blocks(dec).astype(np.int64), smooth.astype(np.int64),
                           np.full((2, 16), 100), np.full((2, 16), 255), np.zeros((2, 16), np.int64)]).astype(np.uint8)


@pytest.mark.parametrize("codec", [0, 1])
def test_checkpoint_resumes_the_run(N, ctx, tmp_path, codec):
    """HybridTrainer.save / load of a two-model state with key times: the state comes back
    exactly, and the resumed trainer's next noisy steps see the uninterrupted one's losses
    (the noise is a function of seed and step)."""
    import torch
    from paper_2604_12625_amd.train import HybridTrainer
    sts = [_state(16, seed=170 + i, codec=codec) for i in range(2)]
    a = HybridTrainer(ctx, sts, lr_feat=1e-2, lr_mlp=1e-3, seed=9, per_model=256)
    x, y, f, tgt = _samples(sts[0], 512, seed=171)
    smp, tg = _dev(N, x, y, f, np.concatenate([tgt, tgt]))
    for _ in range(3):
        a.step(smp, tg, N.HTRAIN_NOISE)
    p = tmp_path / "hyb.npz"
    a.save(p)
    b = HybridTrainer.load(ctx, p)
    assert b.state.step == a.state.step == 3 and b.M == 2 and b.codec == codec
    for name in ("params", "m", "v"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert torch.equal(a.keys, b.keys)
    # the first step reads identical parameters (its FP64 loss sums differ in order only);
    # the second follows updates whose FP32 gradient sums were added in another order
    for rel in (1e-12, 1e-6):
        la = float(a.step(smp, tg, N.HTRAIN_NOISE).item())
        lb = float(b.step(smp, tg, N.HTRAIN_NOISE).item())
        assert abs(la - lb) <= rel * abs(la), (la, lb, rel)
    m = b.export(N.DTYPE_F16, model=1)
    m.save(tmp_path / "m.npz")
    m2 = N.HybridModel.load(tmp_path / "m.npz")
    for u, v in zip(m.arrays, m2.arrays):
        assert torch.equal(u, v)


def test_bc4_encoder_matches_oracle_bit_for_bit(N, ctx):
    import torch
    tex = _blocks_bc4(140)
    got = N.bc4_encode_blocks(torch.from_numpy(tex).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, O.encode_bc4(tex))


def _blocks_bc7(seed):
    """Encoder inputs [n][16][4]: random, smooth and grey texels (_test_blocks), decodes of
    random mode-6 blocks and of random mode-4 and mode-5 blocks, constant blocks."""
    from tests.test_oracle_encode import _test_blocks
    g = np.random.default_rng(seed)
    dec6 = np.stack([O.bc7_decode_block(b) for b in I.random_bc7m6((40,), g)])
    dec45 = np.stack([O.bc7_decode_block(b) for b in I.random_bc7((60,), g, modes=(4, 5))])
    const = np.repeat(g.integers(0, 256, (8, 1, 4)), 16, axis=1)
    return np.concatenate([_test_blocks(seed + 1), dec6, dec45, const,
                           np.zeros((1, 16, 4)), np.full((1, 16, 4), 255)]).astype(np.uint8)


def test_bc7_encoder_matches_oracle_bit_for_bit(N, ctx):
    """The multi-mode encoder (modes 6, 5 and 4, each block its least-error candidate) writes
    the oracle's blocks, byte for byte; and the decode of what it wrote is the oracle's decode
    of it (both decoders pinned)."""
    import torch
    tex = _blocks_bc7(141)
    got = N.bc7_encode_blocks(torch.from_numpy(tex).cuda()).cpu().numpy()
    want = O.encode_bc7(tex)
    np.testing.assert_array_equal(got, want)
    modes = [O.bc7_mode(b) for b in want]
    assert {4, 5, 6} <= set(modes)                  # every mode occurs among the winners
    np.testing.assert_array_equal(N.bc7_decode_blocks(torch.from_numpy(got).cuda()).cpu().numpy(),
                                  np.stack([O.bc7_decode_block(b) for b in got]))


@pytest.mark.parametrize("n", [1, 3, 5, 24])
def test_block_encoders_at_extremes_match_oracle(N, ctx, n):
    """Blocks at the ends of the searches' ranges (values 0 and 255, one texel apart from the
    rest, two values, steps of one), in counts around the four BC4 blocks of a workgroup: byte
    for byte the oracle's."""
    import torch
    g = np.random.default_rng(147 + n)
    one = np.full((n, 16, 4), 255)
    one[np.arange(n), g.integers(0, 16, n)] = g.integers(0, 256, (n, 4))
    kinds = [g.choice([0, 255], (n, 16, 4)), one, 255 - one,
             np.where(g.random((n, 16, 1)) < 0.5, g.integers(0, 256, (n, 1, 4)), g.integers(0, 256, (n, 1, 4))),
             np.clip(g.choice([0, 254], (n, 1, 1)) + g.integers(0, 2, (n, 16, 4)), 0, 255)]
    tex = np.stack([kinds[i % len(kinds)][i] for i in range(n)]).astype(np.uint8)
    got = N.bc7_encode_blocks(torch.from_numpy(tex).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, O.encode_bc7(tex))
    tex4 = np.ascontiguousarray(tex[..., 0])
    got = N.bc4_encode_blocks(torch.from_numpy(tex4).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, O.encode_bc4(tex4))


def test_bc4_encoder_of_few_blocks(N, ctx):
    """Up to eight blocks a CU go one to a workgroup: the bytes of the kernel for more, and a small call
    in less than half the time of the largest such one (0.13 of it; 0.83 where a wave took each block)."""
    import torch
    few = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    g = np.random.default_rng(11)
    x = np.clip(g.integers(0, 256, (few + 1, 1)) + g.normal(0, 1, (few + 1, 16)) * np.exp(g.uniform(0, 5, (few + 1, 1))), 0, 255)
    x[:256] = np.arange(256)[:, None]
    t = torch.from_numpy(x.astype(np.uint8)).cuda()
    more = N.bc4_encode_blocks(t)
    assert torch.equal(N.bc4_encode_blocks(t[:few]), more[:few])
    assert torch.equal(torch.cat([N.bc4_encode_blocks(t[i:i + 1]) for i in range(0, few, 64)]), more[:few:64])
    best = {}
    for _ in range(8):
        for n in (64, few):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                N.bc4_encode_blocks(t[:n], out=more[:n])
            b.record()
            b.synchronize()
            best[n] = min(best.get(n, 1e9), a.elapsed_time(b))
    assert best[64] <= 0.5 * best[few], best


def test_block_encoders_at_scale_match_oracle_on_a_sample(N, ctx):
    """65,536 blocks per encoder in one launch each (the grid-stride loops run many blocks
    per wave): a sample of them against the oracle, byte for byte, and every block decodes."""
    import torch
    g = np.random.default_rng(145)
    n = 65536
    base = g.integers(0, 256, (n, 1, 4))
    tex7 = np.clip(base + g.normal(0, 10, (n, 16, 4)), 0, 255).astype(np.uint8)
    got7 = N.bc7_encode_blocks(torch.from_numpy(tex7).cuda()).cpu().numpy()
    sel = g.choice(n, 96, replace=False)
    np.testing.assert_array_equal(got7[sel], O.encode_bc7(tex7[sel]))
    modes = np.array([O.bc7_mode(b) for b in got7[:4096]])
    assert set(modes.tolist()) <= {4, 5, 6}
    tex4 = np.clip(g.integers(0, 256, (n, 1)) + g.normal(0, 12, (n, 16)), 0, 255).astype(np.uint8)
    got4 = N.bc4_encode_blocks(torch.from_numpy(tex4).cuda()).cpu().numpy()
    sel = g.choice(n, 24, replace=False)
    np.testing.assert_array_equal(got4[sel], O.encode_bc4(tex4[sel]))


@pytest.mark.parametrize("state_codec,flags,codec", [(0, 0, 0), (0, 0, 1), (1, 0, 1), (1, 0, 0), (0, 8, 0), (0, 8, 1),
                                                     (0, 1, 0), (1, 1, 1)])
def test_hybrid_encode_matches_oracle(N, ctx, state_codec, flags, codec):
    """The paper's export: reconstruct (lerp, direct or rounded), quantise, encode; every
    output bit for bit."""
    from paper_2604_12625_amd.train import HybridTrainer
    # BC4 output: the oracle's exhaustive encoder takes tens of ms per block, so the 8 x 8 map
    st = _state(16, seed=150 + 3 * state_codec + flags, bigger=codec == 1, codec=state_codec)
    tr = HybridTrainer(ctx, st)
    hm = tr.encode(flags, codec, N.DTYPE_F32)
    ref = O.hybrid_encode(st, flags, codec)
    for i, k in enumerate(("fuv", "fuvt", "fut", "fvt")):
        np.testing.assert_array_equal(hm.arrays[i].cpu().numpy(), ref[k], err_msg=k)
    np.testing.assert_array_equal(hm.arrays[5].cpu().numpy(), ref["mlp"])
    assert hm.desc.codec == codec


def test_hybrid_encode_rejects_bad_flags(N, ctx):
    from paper_2604_12625_amd.train import HybridTrainer
    tr = HybridTrainer(ctx, _state(16, seed=160, codec=1))
    with pytest.raises(N.NdgiError):
        tr.encode(N.HTRAIN_DIRECT, 1)          # a directly optimised map has the BC4 layout
    tr0 = HybridTrainer(ctx, _state(16, seed=161))
    with pytest.raises(N.NdgiError):
        tr0.encode(N.HTRAIN_DIRECT | N.HTRAIN_BCSIM, 1)
    with pytest.raises(N.NdgiError):
        tr0.encode(0, 7)
    with pytest.raises(N.NdgiError):          # DIRECT training on a BC7-layout state
        import torch
        tr.loss_grad(torch.zeros(64, dtype=torch.int32, device="cuda"),
                     torch.zeros((3, 8, 8, 3), dtype=torch.float32, device="cuda"), N.HTRAIN_DIRECT)


@pytest.mark.parametrize("codec", [0, 1])
def test_import_equals_oracle_and_fine_tune_reads_the_decode(N, ctx, codec):
    """ndgi_hybrid_import writes the oracle's imported state bit for bit; a DIRECT | QPLANES
    forward on it equals the FP32 decode of the model (the final stage trains on what a decode
    reads)."""
    import torch
    from paper_2604_12625_amd.train import hybrid_import_models
    m = I.random_hybrid_model(W=64, H=48, profile="L", slices=5, plane=(32, 48, 4), keys=True, config=170 + codec,
                              codec=codec, uvt_side=(16, 12), mlp_dtype=np.float16)
    hm = N.HybridModel.from_numpy(m)
    frames = len(m["keys"])
    tr = hybrid_import_models(ctx, [hm], frames, keys=m["keys"])
    ref = O.hybrid_import(m, frames)
    got = tr.split(tr.params)
    for k in O.HYB_KEYS:
        np.testing.assert_array_equal(got[k].cpu().numpy(), ref[k].astype(np.float32), err_msg=k)
    g = np.random.default_rng(171)
    n = 5000
    x, y, f = g.integers(0, m["W"], n), g.integers(0, m["H"], n), g.integers(0, frames, n)
    smp, _ = _dev(N, x, y, f, np.zeros((frames, m["H"], m["W"], 3), np.float32))
    fwd = tr.forward(smp, N.HTRAIN_DIRECT | N.HTRAIN_QPLANES).cpu().numpy()
    q = np.stack([(x + 0.5) / m["W"], (y + 0.5) / m["H"], np.asarray(m["keys"], np.float32)[f]], 1).astype(np.float32)
    dec = ctx.hybrid_decode(hm, torch.from_numpy(q).cuda(), N.PREC_F32).cpu().numpy()
    rms = np.sqrt(np.mean(dec.astype(np.float64) ** 2))
    assert np.max(np.abs(fwd - dec) / np.maximum(np.abs(dec), rms)) <= 1e-5
