"""The guide network on the matrix cores against the oracle: forward
outputs, loss, gradient, and a training run that fits a known direction
field."""
import math

import numpy as np
import pytest
import torch

from gpu_common import ctx
from oracle import guide as G
from paper_1902_01137_amd import api

pytestmark = pytest.mark.gpu


def _records(n, seed):
    rng = np.random.default_rng(seed)
    rec = np.zeros((n, 12), np.float32)
    rec[:, 0:3] = rng.uniform(-1, 1, (n, 3))
    d = rng.standard_normal((n, 3))
    rec[:, 3:6] = d / np.linalg.norm(d, axis=1, keepdims=True)
    rec[:, 6] = np.log1p(rng.exponential(20.0, n))
    o = rng.standard_normal((n, 3))
    rec[:, 7:10] = o / np.linalg.norm(o, axis=1, keepdims=True)
    rec[:, 10] = rng.exponential(1.0, n)
    return rec


def test_forward_matches_oracle():
    c = ctx()
    gd = api.Guide(c, seed=3)
    p = G.init_params(11)
    gd.set_params(torch.from_numpy(p))
    rec = _records(1003, 1)          # ragged: not a multiple of the 16-row tile
    out = gd.forward(torch.from_numpy(rec).cuda()).cpu().numpy().astype(np.float64)
    ref, _ = G.forward(p, rec[:, :7].astype(np.float64))
    err = np.linalg.norm(out - ref) / np.linalg.norm(ref)
    assert err < 1e-2, err
    assert np.max(np.abs(out - ref)) < 0.05 * (np.max(np.abs(ref)) + 1.0)
    assert np.allclose(gd.get_params().cpu().numpy(), p)


def test_loss_and_gradient_match_oracle():
    c = ctx()
    gd = api.Guide(c, seed=4)
    p = G.init_params(12) * 0.5
    gd.set_params(torch.from_numpy(p))
    rec = _records(4099, 2)
    g, loss = gd.gradient(torch.from_numpy(rec).cuda())
    torch.cuda.synchronize()
    g = g.cpu().numpy().astype(np.float64)
    lv = loss.cpu().numpy()
    X, wo, w = rec[:, :7].astype(np.float64), rec[:, 7:10].astype(np.float64), rec[:, 10].astype(np.float64)
    L_ref, g_ref = G.loss_grad(p, X, wo, w)
    assert lv[1] == pytest.approx(w.sum(), rel=1e-6)
    assert lv[0] / lv[1] == pytest.approx(L_ref, rel=2e-3)
    cos = g @ g_ref / (np.linalg.norm(g) * np.linalg.norm(g_ref))
    rel = np.linalg.norm(g - g_ref) / np.linalg.norm(g_ref)
    assert cos > 0.999 and rel < 1e-2, (cos, rel)


@pytest.mark.parametrize("n", [1, 17, 300, 70001])
def test_gradient_per_layer_matches_oracle(n):
    """Every layer's weight and bias gradient on its own against the
    oracle's (a mistake confined to one block, such as a bias or the input
    layer, must not hide in the norm of the whole vector); record counts from
    a single record through ragged tiles to several hundred workgroups.
    Bound: bf16 operands in the backward products (the oracle keeps the
    output gradient in float64) cost at most 0.4 % per block in a float64
    emulation of the rounding at these sizes; 2 % leaves room for the float32
    loss terms."""
    c = ctx()
    gd = api.Guide(c, seed=5)
    p = G.init_params(13) * 0.5
    gd.set_params(torch.from_numpy(p))
    rec = _records(n, 3 + n)
    g, _ = gd.gradient(torch.from_numpy(rec).cuda())
    torch.cuda.synchronize()
    g = g.cpu().numpy().astype(np.float64)
    X, wo, w = rec[:, :7].astype(np.float64), rec[:, 7:10].astype(np.float64), rec[:, 10].astype(np.float64)
    _, g_ref = G.loss_grad(p, X, wo, w)
    for layer, ((gW, gb), (rW, rb)) in enumerate(zip(G.unpack(g), G.unpack(g_ref))):
        for name, a, b in (("W", gW, rW), ("b", gb, rb)):
            rel = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
            assert rel < 2e-2, (n, layer, name, rel)


def test_gradient_is_repeatable():
    """The partial gradients are written, not accumulated: two calls on the
    same records give the same gradient, and a call on fewer records after a
    larger one is not polluted by the earlier call's rows."""
    c = ctx()
    gd = api.Guide(c, seed=6)
    gd.set_params(torch.from_numpy(G.init_params(14) * 0.5))
    big = torch.from_numpy(_records(20000, 7)).cuda()
    small = torch.from_numpy(_records(1000, 8)).cuda()
    g_small, _ = gd.gradient(small)
    g_small = g_small.clone()
    gd.gradient(big)
    g_again, _ = gd.gradient(small)
    torch.cuda.synchronize()
    assert torch.equal(g_small, g_again)


def test_adam_steps_and_repacked_weights_match_oracle():
    """Two Adam steps (bias corrections at t = 1 and 2) on the library's own
    gradient against the oracle's update of the float32 master weights; then
    a forward pass with the updated network, whose bf16 copies the same
    kernel rewrote, against the oracle's forward."""
    c = ctx()
    gd = api.Guide(c, seed=7)
    p = (G.init_params(15) * 0.5).astype(np.float32)
    gd.set_params(torch.from_numpy(p))
    rec_np = _records(2000, 9)
    rec = torch.from_numpy(rec_np).cuda()
    m = np.zeros(p.shape)
    v = np.zeros(p.shape)
    lr = 1e-3
    for t in (1, 2):
        g, _ = gd.gradient(rec)
        g = g.cpu().numpy().astype(np.float64)
        gd.train_step(rec, lr)
        p, m, v = G.adam_step(p, m, v, g, t, lr)
        got = gd.get_params().cpu().numpy()
        np.testing.assert_allclose(got, p, rtol=1e-5, atol=1e-8)
    out = gd.forward(rec).cpu().numpy().astype(np.float64)
    ref, _ = G.forward(got.astype(np.float64), rec_np[:, :7].astype(np.float64))
    err = np.linalg.norm(out[:, :40] - ref) / np.linalg.norm(ref)
    assert err < 1e-2, err


def test_training_fits_a_direction_field():
    """Outgoing directions drawn from a vMF whose mean depends on the
    position: the trained mixture must put much more density on them."""
    c = ctx()
    gd = api.Guide(c, seed=5)
    rng = np.random.default_rng(6)
    n = 1 << 15
    rec = _records(n, 7)
    x = rec[:, 0:3].astype(np.float64)
    mu = np.stack([np.sin(2 * x[:, 0]), np.cos(2 * x[:, 0]), 0.5 * x[:, 1]], axis=1)
    mu /= np.linalg.norm(mu, axis=1, keepdims=True)
    rec[:, 7:10] = G.vmf_sample(mu, np.full(n, 30.0), rng.random(n), rng.random(n))
    rec[:, 10] = 1.0
    t = torch.from_numpy(rec).cuda()
    p0 = gd.get_params().cpu().numpy()
    L0 = G.loss_grad(p0, rec[:, :7].astype(np.float64), rec[:, 7:10].astype(np.float64), np.ones(n))[0]
    for it in range(400):
        idx = torch.randint(0, n, (4096,), device="cuda")
        loss = gd.train_step(t[idx], 3e-3)
    torch.cuda.synchronize()
    p1 = gd.get_params().cpu().numpy()
    L1 = G.loss_grad(p1, rec[:, :7].astype(np.float64), rec[:, 7:10].astype(np.float64), np.ones(n))[0]
    # the density of a kappa = 30 lobe at its mean is ~4.8/sr; uniform is 1/(4 pi)
    assert L1 < L0 - 2.0, (L0, L1)


def _hg(g, mu):
    return (1 - g * g) / (4 * math.pi * (1 + g * g - 2 * g * mu) ** 1.5)


def test_guided_sampling_step_against_oracle():
    """The renderer's guided step on given vertices: the mixture density it
    reports at the drawn direction matches the oracle's network and mixture,
    p is HG at that direction, and the weight factor is p / (c q + (1-c) p)."""
    c = ctx()
    gd = api.Guide(c, seed=17)
    prm = gd.get_params().cpu().numpy()
    n = 20011
    rec = _records(n, 3)
    X = np.zeros((n, 8), np.float32)
    X[:, :7] = rec[:, :7]
    U = np.random.default_rng(4).random((n, 4)).astype(np.float32)
    gf, g = 0.5, 0.85
    out = gd.sample(torch.from_numpy(X).cuda(), torch.from_numpy(U).cuda(), gf, g).cpu().numpy().astype(np.float64)
    d = out[:, :3]
    assert np.allclose(np.linalg.norm(d, axis=1), 1.0, atol=1e-5)
    z, _ = G.forward(prm, X[:, :7].astype(np.float64))
    # the tracer keeps the network outputs in bf16 (sampling and density use the same rounded values)
    q_ref = G.mixture_pdf(G.bf16_round(z), d)
    rel = np.abs(out[:, 4] - q_ref) / q_ref
    assert np.median(rel) < 0.01 and np.quantile(rel, 0.99) < 0.1, (np.median(rel), np.quantile(rel, 0.99))
    p_ref = _hg(g, np.sum(d * X[:, 3:6], axis=1))
    assert np.allclose(out[:, 5], p_ref, rtol=1e-4)
    w_ref = out[:, 5] / (gf * out[:, 4] + (1 - gf) * out[:, 5])
    assert np.allclose(out[:, 3], w_ref, rtol=1e-5)


@pytest.mark.parametrize("gf", [0.5, 0.9])
def test_guided_sampling_step_is_unbiased(gf):
    """Over the mixture proposal, E[w] = 1 and E[w omega] = g omega_in (the
    HG mean cosine) exactly, for any network."""
    c = ctx()
    gd = api.Guide(c, seed=17)
    g = 0.85
    rec = _records(4, 5)
    m = 1 << 18
    X = np.zeros((4 * m, 8), np.float32)
    X[:, :7] = np.repeat(rec[:, :7], m, axis=0)
    U = np.random.default_rng(6).random((4 * m, 4)).astype(np.float32)
    out = gd.sample(torch.from_numpy(X).cuda(), torch.from_numpy(U).cuda(), gf, g).cpu().numpy().astype(np.float64)
    for v in range(4):
        o = out[v * m:(v + 1) * m]
        w = o[:, 3]
        wd = w[:, None] * o[:, :3]
        se_w = w.std() / math.sqrt(m)
        assert abs(w.mean() - 1.0) < 5 * se_w + 1e-6, (v, w.mean(), se_w)
        exp = g * rec[v, 3:6].astype(np.float64)
        se = wd.std(axis=0) / math.sqrt(m)
        assert np.all(np.abs(wd.mean(axis=0) - exp) < 5 * se + 1e-6), (v, wd.mean(axis=0), exp, se)


@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 4099, 150_001])
def test_forward_of_any_tile_position(n):
    """The last tile in part, fewer records than one workgroup takes and more
    than all resident ones take at once: a record's outputs depend on no other record."""
    gd = api.Guide(ctx(), seed=3)
    gd.set_params(torch.from_numpy(G.init_params(11)))
    base = _records(61, 5)          # (prime: every record meets every place in a tile)
    one = gd.forward(torch.from_numpy(base).cuda())
    out = gd.forward(torch.from_numpy(np.resize(base, (n, 12))).cuda())
    assert torch.equal(out, one.repeat(n // 61 + 1, 1)[:n])


@pytest.mark.parametrize("n", [15, 63, 64, 65, 129, 2049])
def test_gradient_at_the_edges_of_a_chunk(n):
    """Parts of the 64 records a workgroup takes at a time and of its chunk (bounds as for the whole gradient above)."""
    gd = api.Guide(ctx(), seed=4)
    p = G.init_params(12) * 0.5
    gd.set_params(torch.from_numpy(p))
    rec = _records(n, 6)
    g, loss = gd.gradient(torch.from_numpy(rec).cuda())
    g = g.cpu().numpy().astype(np.float64)
    w = rec[:, 10].astype(np.float64)
    L_ref, g_ref = G.loss_grad(p, rec[:, :7].astype(np.float64), rec[:, 7:10].astype(np.float64), w)
    lv = loss.cpu().numpy()
    assert lv[1] == pytest.approx(w.sum(), rel=1e-6)
    assert lv[0] / lv[1] == pytest.approx(L_ref, rel=2e-3)
    cos = g @ g_ref / (np.linalg.norm(g) * np.linalg.norm(g_ref))
    assert cos > 0.999 and np.linalg.norm(g - g_ref) < 1e-2 * np.linalg.norm(g_ref), cos
